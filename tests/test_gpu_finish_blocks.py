"""The second launch of the deferred schedule takes 768 threads a sequence up to one sequence
per CU and 512 beyond.  Walks that end at a leaf, at a rejected single candidate and at a row
of several candidates give the same bits with either, and those of the schedule in which
every row draws."""
import pytest
import torch

from paper_2608_24411_amd import synth
from parity_util import gpu_tree
from test_gpu_path import same

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("V,dtype", [(2048, "f32"), (2051, "f32"), (3072, "bf16"), (3075, "bf16")])
@pytest.mark.parametrize("mode", ("resispec", "specinfer"))
def test_finish_blocks_agree(gpu_lib, V, dtype, mode):
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    print("finish blocks", V, dtype, mode, cus, flush=True)
    w = synth.make_workload(2, device="cuda", B=cus + 1, V=V, dtype=dtype)
    keys = ("target", "draft", "node_token", "parent", "u_accept", "u_resample")
    ref = gpu_tree(gpu_lib, w, mode)
    ends = set()
    for B in (cus + 1, cus):
        ws = torch.empty(gpu_lib.resispec_deferred_workspace_bytes(B, w["N"]), dtype=torch.uint8, device="cuda")
        t, l, s = gpu_lib.resispec_verify_tree_deferred(*[w[k][:B] for k in keys], temperature=w["temperature"],
                                                        max_depth=w["max_depth"], mode=mode, workspace=ws)
        torch.cuda.synchronize()
        same(dict(tokens=t, accepted_len=l, status=s), {k: ref[k][:B] for k in ("tokens", "accepted_len", "status")})
        ends |= set(l.tolist())
    assert {0, 1, 4} <= ends     # ended at a root, at a rejected chain candidate, at a leaf
