"""Rows that are no multiple of 16 bytes, and tensors that start off a 16-byte boundary: the
vector that crosses a row's end, at the edges of vectors, chunks (1,024 bf16 or 512 fp32
elements) and slots, in every schedule, against the oracle.  The schedules agree bit for bit;
the oracle's bar is that of the other parity tests (flag window 1e-6)."""
import pytest
import torch

from paper_2608_24411_amd import synth
from parity_util import compare_walk, gpu_tree, host_tree, oracle_walk
from test_gpu_draft import check_draws, compare_draft, gpu_draft, oracle_draft
from test_gpu_path import path_tree, same

pytestmark = pytest.mark.gpu

SIZES = {"bf16": (8, 9, 15, 1023, 1025, 1031, 8193, 32001, 131073),
         "f32": (4, 5, 7, 511, 513, 515, 4097, 32001, 65537)}
CASES = [(d, V, 0) for d in SIZES for V in SIZES[d]] + [
    # whole vectors in a tensor that starts one element late, and three late
    ("bf16", 32000, 1), ("f32", 32000, 1), ("bf16", 1027, 3), ("f32", 513, 3)]


def late(x, n):
    """The same tensor, n elements after a 16-byte boundary."""
    return torch.empty(x.numel() + n, dtype=x.dtype, device=x.device)[n:].view(x.shape).copy_(x)


@pytest.mark.parametrize("dtype,V,shift", CASES)
@pytest.mark.parametrize("mode", ("resispec", "specinfer"))
def test_odd_rows(gpu_lib, dtype, V, shift, mode):
    print("odd rows", dtype, V, shift, mode, flush=True)
    w = synth.make_workload(1, device="cuda", B=3, V=V, dtype=dtype)
    # the last elements of some rows carry most of the mass: draws and tests reach them
    w["target"][1, :, -1] = 9.0
    w["draft"][2, :, -1] = 9.0
    w["node_token"][2, 1:4] = V - 1
    if shift:
        w["target"], w["draft"] = late(w["target"], shift), late(w["draft"], shift)
    ref = gpu_tree(gpu_lib, w, mode)
    same(path_tree(gpu_lib, w, mode), ref)
    args = [w[k] for k in ("target", "draft", "node_token", "parent", "u_accept", "u_resample")]
    kw = dict(temperature=w["temperature"], max_depth=w["max_depth"], mode=mode)
    for entry, more in ((gpu_lib.resispec_verify_tree_deferred, {}),
                        (gpu_lib.resispec_verify_tree_path_group, dict(group_size=0)),
                        (gpu_lib.resispec_verify_tree_group, dict(group_size=0))):
        t, l, s = entry(*args, **kw, **more)
        torch.cuda.synchronize()
        same(dict(tokens=t, accepted_len=l, status=s), ref)
    # a group may have as many members as a row has runs of 256 elements, at most 16
    if V > 256:
        S = min(16, (V + 255) // 256)
        ws = torch.empty(gpu_lib.resispec_path_workspace_bytes(3, V), dtype=torch.uint8, device="cuda")
        t, l, s = gpu_lib.resispec_verify_tree_path_group(*args, **kw, group_size=S, workspace=ws) \
            if (V * w["target"].element_size()) % 16 or shift else (ref["tokens"], ref["accepted_len"], ref["status"])
        torch.cuda.synchronize()
        same(dict(tokens=t, accepted_len=l, status=s), ref)
        if S * 63 <= 512 and ((V * w["target"].element_size()) % 16 or shift):
            t, l, s = gpu_lib.resispec_verify_tree_group(*args, **kw, group_size=S)
            torch.cuda.synchronize()
            same(dict(tokens=t, accepted_len=l, status=s), ref)
    h = host_tree(w)
    compare_walk(ref, oracle_walk(h, w, mode), h, w, mode)


@pytest.mark.parametrize("dtype,V,shift", CASES)
def test_odd_rows_draft(gpu_lib, dtype, V, shift):
    print("odd rows, draft step", dtype, V, shift, flush=True)
    w = synth.make_workload(1, device="cuda", B=2, V=V, dtype=dtype)
    w["draft"][1, :, -1] = 9.0
    if shift:
        w["draft"] = late(w["draft"], shift)
    for worep in (False, True) if V > 64 else (False,):
        g = gpu_draft(gpu_lib, w, 3, 1, worep)
        compare_draft(g, oracle_draft(w, 3, 1, worep))
        check_draws(g, w, 3, 1, worep)
