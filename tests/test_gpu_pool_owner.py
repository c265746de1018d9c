"""Whose group states are whose, in batches of few long rows: ownership goes by the launch and
needs no memory of the caller's, so outputs may lie where inputs do or be shared by calls that
ignore them, calls without a workspace that overlap leave the states of others alone, and every
state comes back."""
import threading

import pytest
import torch

from paper_2608_24411_amd import synth
from parity_util import gpu_tree
from test_gpu_pool import KEYS, equal, flat

pytestmark = pytest.mark.gpu
V = 82944   # bf16: 162 KiB a row


def workload(k, B):
    cfg = dict(synth.CONFIGS[0], B=B, V=V, dtype="bf16", k=k)
    return synth.make_workload(cfg, device="cuda")


@pytest.fixture(scope="module")
def one(gpu_lib):
    """140 rows of one candidate: more than take groups, so the reference has none."""
    w = workload(1, 140)
    return w, flat(gpu_lib, w)


@pytest.mark.parametrize("where", ["cand_ids", "u_accept", "u_resample"])
def test_lengths_in_place_of_inputs(gpu_lib, one, where):
    w, ref = one
    for B in (1, 33, 64, 128):
        print("pool, lengths over", where, B, flush=True)
        args = {k: w[k][5:5 + B].clone() for k in KEYS}
        room = args[where].view(torch.int32).view(B)
        out = gpu_lib.resispec_verify(*args.values(), temperature=w["temperature"], out_accepted_len=room)
        torch.cuda.synchronize()
        equal(out, [x[5:5 + B] for x in ref])
        assert gpu_lib.resispec_debug_pool_held() == 0


def test_lengths_shared_by_threads(gpu_lib, one):
    """Four threads with a stream each; one array takes everyone's lengths and statuses."""
    w, ref = one
    print("pool, shared lengths", flush=True)
    junk = torch.empty(32, dtype=torch.int32, device="cuda")
    got = {}
    torch.cuda.synchronize()

    def work(t):
        s = torch.cuda.Stream()
        with torch.cuda.stream(s):
            got[t] = [(20 * t + i, flat(gpu_lib, w, 32, 20 * t + i, out_accepted_len=junk, out_status=junk)[0])
                      for i in range(20)]
        s.synchronize()

    threads = [threading.Thread(target=work, args=(t,)) for t in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert len(got) == 4
    for outs in got.values():
        for lo, token in outs:
            assert torch.equal(token, ref[0][lo:lo + 32])
    assert gpu_lib.resispec_debug_pool_held() == 0


def test_calls_without_a_workspace(gpu_lib, one):
    """resispec_verify_tree_noalloc on three streams at once (their outcomes race, and are not
    looked at) beside flat calls on a fourth, which are right; then alone, where it is too."""
    w, ref = one
    t = synth.make_workload(2, device="cuda", B=2, V=V)
    args = [t[k] for k in ("target", "draft", "node_token", "parent", "u_accept", "u_resample")]
    kw = dict(temperature=t["temperature"], max_depth=t["max_depth"])

    def noalloc():
        out = [torch.empty(s, dtype=torch.int32, device="cuda") for s in ((2, t["max_depth"] + 1), (2,), (2,))]
        return gpu_lib.resispec_verify_tree_noalloc(*args, **kw, out_tokens=out[0], out_accepted_len=out[1],
                                                    out_status=out[2])

    print("pool, no workspace", flush=True)
    streams = [torch.cuda.Stream() for _ in range(4)]
    torch.cuda.synchronize()
    outs = []
    for i in range(12):
        for s in streams[:3]:
            with torch.cuda.stream(s):
                noalloc()
        with torch.cuda.stream(streams[3]):
            outs.append(flat(gpu_lib, w, 24, i))
    torch.cuda.synchronize()
    for i, out in enumerate(outs):
        equal(out, [x[i:i + 24] for x in ref])
    assert gpu_lib.resispec_debug_pool_held() == 0
    a = noalloc()
    b = gpu_lib.resispec_verify_tree_group(*args, **kw, group_size=1)
    torch.cuda.synchronize()
    equal(a, b)


def test_many_launches(gpu_lib, one):
    """One state after another: row counts that do not divide the pool, far more launches than
    it has states, and a graph whose replays meet eager launches on another stream."""
    w, ref = one
    side = torch.cuda.Stream()
    out = [torch.empty(30, dtype=torch.int32, device="cuda") for _ in range(3)]
    call = dict(out_token=out[0], out_accepted_len=out[1], out_status=out[2])
    with torch.cuda.stream(side):
        flat(gpu_lib, w, 30, 50, **call)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=side):
        flat(gpu_lib, w, 30, 50, **call)
    print("pool, many launches", flush=True)
    for i in range(400):
        B = 1 + (i * 7) % 37
        if i % 5 == 0:
            for x in out:
                x.fill_(-7)
            side.wait_stream(torch.cuda.current_stream())
            with torch.cuda.stream(side):
                g.replay()
        got = flat(gpu_lib, w, B, i % 100)
        if i % 5 == 0:
            torch.cuda.synchronize()
            equal(out, [x[50:80] for x in ref])
        equal(got, [x[i % 100:i % 100 + B] for x in ref])
    assert gpu_lib.resispec_debug_pool_held() == 0


def test_launches_that_meet(gpu_lib, one):
    """Launches of 64 and 128 rows on two and four streams: some take groups and some do not,
    every row is right, and the count of workgroups under way ends at 0."""
    w, ref = one
    for B, ns in ((64, 2), (128, 2), (128, 4), (20, 4)):
        print("pool, launches that meet", B, ns, flush=True)
        streams = [torch.cuda.Stream() for _ in range(ns)]
        torch.cuda.synchronize()
        outs = []
        for i in range(12):
            for s in streams:
                with torch.cuda.stream(s):
                    outs.append((i, flat(gpu_lib, w, B, i)))
        torch.cuda.synchronize()
        for i, out in outs:
            equal(out, [x[i:i + B] for x in ref])
        assert gpu_lib.resispec_debug_pool_held() == 0


def test_a_launch_that_fails_keeps_no_state(gpu_lib, one):
    w, ref = one
    print("pool, failed launches", flush=True)
    gpu_lib.resispec_debug_fail_pool_launches(3)
    try:
        for B in (128, 1, 60):
            with pytest.raises(RuntimeError):
                flat(gpu_lib, w, B)
        assert gpu_lib.resispec_debug_pool_held() == 0
        equal(flat(gpu_lib, w, 64, 9), [x[9:73] for x in ref])     # the fourth does not fail
    finally:
        gpu_lib.resispec_debug_fail_pool_launches(0)
    assert gpu_lib.resispec_debug_pool_held() == 0
