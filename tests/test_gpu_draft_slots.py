"""The draft step's slots: one chunk up to 256 chunks a row (1,024 bf16 or 512 fp32 elements),
runs of chunks beyond.  Rows at both sides of the line, against the oracle's draws."""
import pytest
import torch

from paper_2608_24411_amd import synth
from test_gpu_draft import check_draws, compare_draft, gpu_draft, oracle_draft

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("V,dtype", [(131072, "f32"), (131076, "f32"), (262144, "bf16"), (262152, "bf16"),
                                     (262145, "bf16"), (524296, "bf16")])
@pytest.mark.parametrize("worep", [False, True])
def test_draft_slots(gpu_lib, V, dtype, worep):
    print("draft slots", V, dtype, worep, flush=True)
    w = synth.make_workload(4, device="cuda", B=1, V=V, dtype=dtype)
    # mass at the row's end, in its last slot
    w["draft"][0, 1, -3:] = 4.0
    g = gpu_draft(gpu_lib, w, 9, 2, worep)
    compare_draft(g, oracle_draft(w, 9, 2, worep))
    check_draws(g, w, 9, 2, worep)
    assert (g["status"] == 0).all()
