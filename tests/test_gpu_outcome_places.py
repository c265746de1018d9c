"""Node outcomes go wherever a copy of the runtime goes: arrays on the device
(one kernel), pinned and pageable host memory and addresses off a word (copies), alone or
mixed, eagerly and from a graph."""
import ctypes

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

B, N = 5, 51
ROWS = B * N


@pytest.fixture(scope="module")
def outcomes(gpu_lib):
    ws = torch.randint(0, 255, (gpu_lib.resispec_workspace_bytes(B, N),), dtype=torch.uint8, device="cuda")
    stride = ws.numel() // 12
    words = ws.view(torch.int32).cpu().numpy()
    return ws, [words[k * stride:k * stride + ROWS].copy() for k in range(3)]


def copy_out(gpu_lib, ws, addresses):
    st = gpu_lib.lib.resispec_node_outcomes(
        ctypes.c_void_p(ws.data_ptr()), ctypes.c_size_t(ws.numel()), B, N, *[ctypes.c_void_p(a) for a in addresses],
        ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
    torch.cuda.synchronize()
    return st


def place(kind):
    """An array of the kind, its address, and its words on the host."""
    if kind == "pageable":
        x = np.full(ROWS, -9, dtype=np.int32)
        return x, x.ctypes.data, lambda: x
    if kind == "pinned":
        x = torch.full((ROWS,), -9, dtype=torch.int32).pin_memory()
        return x, x.data_ptr(), lambda: x.numpy()
    room = torch.zeros(4 * ROWS + 8, dtype=torch.uint8, device="cuda")
    off = 1 if kind == "off a word" else 0
    return room, room.data_ptr() + off, lambda: np.frombuffer(room.cpu().numpy().tobytes()[off:off + 4 * ROWS],
                                                              dtype=np.int32)


@pytest.mark.parametrize("kinds", [("device",) * 3, ("pinned",) * 3, ("pageable",) * 3, ("off a word",) * 3,
                                   ("device", "pageable", "pinned"), ("pinned", "device", "device"),
                                   ("device", "device", "pageable")], ids=lambda k: "-".join(k).replace(" ", "_"))
def test_destinations(gpu_lib, outcomes, kinds):
    print("outcome places", kinds, flush=True)
    ws, want = outcomes
    places = [place(k) for k in kinds]
    assert copy_out(gpu_lib, ws, [p[1] for p in places]) == 0
    for p, w in zip(places, want):
        assert np.array_equal(p[2](), w)


def test_graph(gpu_lib, outcomes):
    print("outcome places, graph", flush=True)
    ws, want = outcomes
    src = ws.clone()
    side = torch.cuda.Stream()
    out = [torch.empty((B, N), dtype=torch.int32, device="cuda") for _ in range(3)]
    addresses = [ctypes.c_void_p(x.data_ptr()) for x in out]
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=side):
        assert gpu_lib.lib.resispec_node_outcomes(ctypes.c_void_p(src.data_ptr()), ctypes.c_size_t(src.numel()), B, N,
                                                  *addresses, ctypes.c_void_p(side.cuda_stream)) == 0
    for i in range(3):
        src.copy_(ws if i != 1 else torch.zeros_like(ws))
        g.replay()
        torch.cuda.synchronize()
        for x, w in zip(out, want):
            assert np.array_equal(x.cpu().numpy().ravel(), w if i != 1 else 0 * w)
