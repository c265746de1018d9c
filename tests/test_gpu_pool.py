"""Row groups whose states come from the library's pool (few long rows, no group workspace):
the flat entry and the all-nodes schedule.  Every size of the range gives the bits of the
ordinary kernel (the same rows in a batch too large for groups), also when groups do not
form, when their exchanges time out, when launches on several streams hold states at once,
and on every replay of a graph."""
import threading

import pytest
import torch

from paper_2608_24411_amd import synth
from test_gpu_parity import _flat_check

pytestmark = pytest.mark.gpu

KEYS = ("target", "draft", "cand_ids", "u_accept", "u_resample")
# rows of at least 160 KiB; odd and whole vectors
SHAPES = [(41472, "f32"), (41001, "f32"), (82944, "bf16"), (82001, "bf16")]


def flat(native, w, B=None, lo=0, **kw):
    part = [w[k][lo:(w["B"] if B is None else lo + B)] for k in KEYS]
    return native.resispec_verify(*part, temperature=w["temperature"], **kw)


def rows(out, lo, B):
    return [x[lo:lo + B] for x in out]


def equal(a, b):
    assert all(torch.equal(x, y) for x, y in zip(a, b))


@pytest.fixture(scope="module", params=SHAPES, ids=lambda s: "%d-%s" % s)
def many(request, gpu_lib):
    V, dtype = request.param
    w = synth.make_workload(0, device="cuda", B=300, V=V, dtype=dtype)
    ref = {m: flat(gpu_lib, w, mode=m) for m in ("resispec", "specinfer")}   # 300 rows: no groups
    torch.cuda.synchronize()
    return w, ref


@pytest.mark.parametrize("mode", ("resispec", "specinfer"))
def test_sizes(gpu_lib, many, mode):
    w, ref = many
    # 8 members down to 2, one more row than groups take
    for B in (1, 3, 31, 32, 33, 64, 85, 128, 129):
        print("pool", w["V"], mode, B, flush=True)
        out = flat(gpu_lib, w, B, 7, mode=mode)
        torch.cuda.synchronize()
        equal(out, rows(ref[mode], 7, B))
    part = dict(w, B=40, **{k: w[k][:40] for k in KEYS})
    _flat_check(part, *rows(ref[mode], 0, 40), mode)


def test_groups_that_fail(gpu_lib, many):
    """No formation, and exchanges that time out: the row is done by one workgroup."""
    w, ref = many
    for waits in (dict(formation=0), dict(barrier=0), dict(barrier=0, formation=0)):
        print("pool, waits", w["V"], waits, flush=True)
        gpu_lib.resispec_debug_set_group_waits(**waits)
        try:
            for _ in range(3):
                out = flat(gpu_lib, w, 60, 5)
                torch.cuda.synchronize()
                equal(out, rows(ref["resispec"], 5, 60))
        finally:
            gpu_lib.resispec_debug_set_group_waits()


def test_streams_and_threads(gpu_lib, many):
    """Four threads with a stream each, 85 rows a launch: more groups than the pool holds."""
    w, ref = many
    got = {}
    torch.cuda.synchronize()

    def work(t):
        s = torch.cuda.Stream()
        with torch.cuda.stream(s):
            got[t] = [(40 * t + i, flat(gpu_lib, w, 85, 40 * t + i)) for i in range(12)]
        s.synchronize()

    threads = [threading.Thread(target=work, args=(t,)) for t in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert len(got) == 4
    for outs in got.values():
        for lo, out in outs:
            equal(out, rows(ref["resispec"], lo, 85))


def test_graph_replays(gpu_lib, many):
    w, ref = many
    args = [w[k][:50].clone() for k in KEYS]
    out = [torch.empty(50, dtype=torch.int32, device="cuda") for _ in range(3)]
    kw = dict(temperature=w["temperature"], out_token=out[0], out_accepted_len=out[1], out_status=out[2])
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(s):
        gpu_lib.resispec_verify(*args, **kw)
    torch.cuda.current_stream().wait_stream(s)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        gpu_lib.resispec_verify(*args, **kw)
    for lo in (0, 100, 33, 250):
        print("pool, graph", w["V"], lo, flush=True)
        for a, k in zip(args, KEYS):
            a.copy_(w[k][lo:lo + 50])
        other = flat(gpu_lib, w, 20, lo)         # eager work between replays
        g.replay()
        torch.cuda.synchronize()
        equal(out, rows(ref["resispec"], lo, 50))
        equal(other, rows(ref["resispec"], lo, 20))


def test_tree_rows(gpu_lib):
    """One and two trees: verify_tree and verify_nodes take groups, the group entry with one
    member does not."""
    w = synth.make_workload(2, device="cuda", B=2, V=82001)
    for B in (1, 2):
        args = [w[k][:B] for k in ("target", "draft", "node_token", "parent", "u_accept", "u_resample")]
        kw = dict(temperature=w["temperature"], max_depth=w["max_depth"])
        a = gpu_lib.resispec_verify_tree(*args, **kw)
        b = gpu_lib.resispec_verify_tree_group(*args, **kw, group_size=1)
        torch.cuda.synchronize()
        equal(a, b)
