"""Few long rows in the pool's row groups where rows differ from the usual: no candidates, faults
of every kind, rows that take the exact-maximum pass (the members' maxima are exchanged), and
trees whose candidates were drawn without replacement.  Every row gives the bits of the same
row in a batch too large for groups, and no state stays behind."""
import numpy as np
import pytest
import torch

from paper_2608_24411_amd import synth
from test_gpu_pool import equal, flat

pytestmark = pytest.mark.gpu
MODES = ("resispec", "specinfer")
SHAPES = [(41472, "f32"), (82001, "bf16")]     # whole and odd vectors, at least 160 KiB a row


def rows_both_ways(gpu_lib, w, mode, sizes=(1, 29, 64, 100)):
    """The outcomes of w's 160 rows as one batch (no groups), and as batches that take groups."""
    ref = flat(gpu_lib, w, mode=mode)
    for B in sizes:
        for lo in (0, 60):
            equal(flat(gpu_lib, w, B, lo, mode=mode), [x[lo:lo + B] for x in ref])
    assert gpu_lib.resispec_debug_pool_held() == 0
    return ref


@pytest.mark.parametrize("V,dtype", SHAPES)
@pytest.mark.parametrize("mode", MODES)
def test_no_candidates(gpu_lib, V, dtype, mode):
    print("pool, no candidates", V, dtype, mode, flush=True)
    w = synth.make_workload(0, device="cuda", B=160, V=V, dtype=dtype)
    w["cand_ids"] = w["cand_ids"][:, :0].contiguous()
    w["u_accept"] = w["u_accept"][:, :0].contiguous()
    ref = rows_both_ways(gpu_lib, w, mode)
    assert (ref[2] == 0).all() and (ref[1] == 0).all()


@pytest.mark.parametrize("V,dtype", SHAPES)
@pytest.mark.parametrize("mode", MODES)
def test_faults(gpu_lib, V, dtype, mode):
    """Bad tokens, uniforms out of range at a test and at the draw, candidates without draft
    mass, and rows without any: each status, beside rows that have none."""
    print("pool, faults", V, dtype, mode, flush=True)
    w = synth.make_workload(0, device="cuda", B=160, V=V, dtype=dtype)
    b = torch.arange(160, device="cuda")
    w["cand_ids"][b % 8 == 1, 0] = V
    w["cand_ids"][b % 8 == 2, 0] = -3
    w["u_accept"][b % 8 == 3, 0] = 1.0
    late = torch.nonzero(b % 8 == 4).flatten()     # no target mass at any candidate: all rejected
    w["target"][late[:, None], w["cand_ids"][late].long()] = float("-inf")
    w["u_resample"][late] = -0.5
    zero = torch.nonzero(b % 8 == 5).flatten()
    w["draft"][zero, w["cand_ids"][zero, 0].long()] = float("-inf")
    w["target"][b % 8 == 6] = float("-inf")
    ref = rows_both_ways(gpu_lib, w, mode)
    st = ref[2].cpu().numpy()
    for k, want in ((0, 0), (1, 1), (2, 1), (3, 5), (4, 5), (5, 2), (6, 3), (7, 0)):
        assert (st[np.arange(160) % 8 == k] == want).all(), k


@pytest.mark.parametrize("V,dtype", SHAPES)
@pytest.mark.parametrize("mode", MODES)
def test_exact_maximum_pass(gpu_lib, V, dtype, mode):
    """A logit far above those that set the exponent reference, in the last member's share, in
    another's, or in the draft alone."""
    print("pool, exact maximum", V, dtype, mode, flush=True)
    w = synth.make_workload(0, device="cuda", B=160, V=V, dtype=dtype)
    b = torch.arange(160, device="cuda")
    w["target"][b % 4 == 1, V - 2] = 300.0
    w["target"][b % 4 == 2, V // 2] = 250.0
    w["draft"][b % 4 == 3, V - 7] = 300.0
    ref = rows_both_ways(gpu_lib, w, mode)
    assert (ref[0][(b % 4 == 1) & (ref[1] == 0)] == V - 2).all()


@pytest.mark.parametrize("mode", MODES)
@pytest.mark.parametrize("cfg,V", [(4, 82944), (3, 82001)])
def test_without_replacement(gpu_lib, mode, cfg, V):
    """Trees with and without replacement: verify_tree and verify_nodes take groups; the group
    entry with one member does not."""
    w = synth.make_workload(cfg, device="cuda", B=2, V=V, dtype="bf16")
    args = [w[k] for k in ("target", "draft", "node_token", "parent", "u_accept", "u_resample")]
    for worep in (True, False):
        print("pool, trees", cfg, V, mode, worep, flush=True)
        kw = dict(temperature=w["temperature"], mode=mode, without_replacement=worep)
        a = gpu_lib.resispec_verify_tree(*args, **kw, max_depth=w["max_depth"])
        b = gpu_lib.resispec_verify_tree_group(*args, **kw, max_depth=w["max_depth"], group_size=1)
        ws = torch.empty(gpu_lib.resispec_workspace_bytes(2, w["N"]), dtype=torch.uint8, device="cuda")
        gpu_lib.resispec_verify_nodes(*args, **kw, workspace=ws)
        nodes = gpu_lib.resispec_node_outcomes(ws, 2, w["N"])
        # every node again in batches of 2 * 6 trees, more rows than take groups
        many = [torch.cat([x] * 6) for x in args]
        wsm = torch.empty(gpu_lib.resispec_workspace_bytes(12, w["N"]), dtype=torch.uint8, device="cuda")
        gpu_lib.resispec_verify_nodes(*many, **kw, workspace=wsm)
        ref = gpu_lib.resispec_node_outcomes(wsm, 12, w["N"])
        torch.cuda.synchronize()
        assert 2 * w["N"] <= 128 < 12 * w["N"]
        equal(a, b)
        for x, y in zip(nodes, ref):
            assert torch.equal(x, y[:2]) and torch.equal(x, y[10:])
        assert gpu_lib.resispec_debug_pool_held() == 0
