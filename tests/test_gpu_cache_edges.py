"""The path schedule's residual cache where the last slot of a row is partial: its chunks past
the row belong neither to the sequence's share of the workspace nor, for the last sequence, to
the workspace.  Roots that reject at least three candidates in a row, with much of the mass on
the row's first tokens (where a neighbour's surplus chunk would land), give the bits of the
path without a workspace, and the bytes behind the workspace stay as they were."""
import pytest
import torch

from parity_util import gpu_tree
from test_gpu_path import _chain_workload, group_tree, path_tree, same

pytestmark = pytest.mark.gpu

GUARD = 1 << 16


@pytest.mark.parametrize("V,dtype", [(132000, "bf16"), (151669, "bf16"), (151936, "bf16"), (131073, "bf16"),
                                     (140001, "f32"), (201088, "f32")])
def test_partial_last_slot(gpu_lib, V, dtype):
    w, kids_of = _chain_workload(V, dtype, False, V)
    B = w["parent"].shape[0]
    kids = torch.zeros((B, w["parent"].shape[1], V), dtype=torch.bool)
    for n, ks in kids_of.items():
        if ks:
            kids[:, n].scatter_(1, w["node_token"][:, torch.as_tensor(ks)].cpu().long(), True)
    # (the candidates keep their logits, so they are rejected as before)
    first = torch.arange(V) < 1024
    w["target"] += 4.0 * (first & ~kids).cuda()
    w["draft"] += 4.0 * (first & ~kids).cuda()
    need = gpu_lib.resispec_path_workspace_bytes(B, V)
    for mode in ("resispec", "specinfer"):
        print("partial last slot", V, dtype, mode, flush=True)
        ref = path_tree(gpu_lib, w, mode)
        same(ref, gpu_tree(gpu_lib, w, mode))
        buf = torch.full((need + GUARD,), 0xA5, dtype=torch.uint8, device="cuda")
        for g in (1, 2, 3, 0):
            same(group_tree(gpu_lib, w, mode, g, workspace=buf[:need]), ref)
        assert bool((buf[need:] == 0xA5).all())
