"""The path schedule keeps one tree node per thread up to 512 nodes and reads the tree at
every row beyond: trees of 511, 512 and 513 nodes, walked as the all-nodes schedule does."""
import numpy as np
import pytest
import torch

from paper_2608_24411_amd import synth
from parity_util import gpu_tree
from test_gpu_path import path_tree, same

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N", [511, 512, 513])
@pytest.mark.parametrize("mode", ("resispec", "specinfer"))
def test_tree_sizes(gpu_lib, N, mode):
    print("held tree", N, mode, flush=True)
    cfg = dict(synth.CONFIGS[3], B=4, V=2048, tree=("random_bfs", N, 12, (0.4, 0.3, 0.2, 0.1)))
    w = synth.make_workload(cfg, device="cuda")
    # accepted chains down to the last nodes: the deepest path of each tree takes any draw
    par = synth.to_host(w["parent"])
    for b in range(4):
        n = N - 1
        while n > 0:
            w["u_accept"][b, n] = 0.0
            n = int(par[b, n])
    ref = gpu_tree(gpu_lib, w, mode)
    same(path_tree(gpu_lib, w, mode), ref)
    ws = torch.empty(gpu_lib.resispec_path_workspace_bytes(4, 2048), dtype=torch.uint8, device="cuda")
    t, l, s = gpu_lib.resispec_verify_tree_path_group(
        *[w[k] for k in ("target", "draft", "node_token", "parent", "u_accept", "u_resample")],
        temperature=w["temperature"], max_depth=w["max_depth"], mode=mode, workspace=ws)
    torch.cuda.synchronize()
    same(dict(tokens=t, accepted_len=l, status=s), ref)
    assert int(l.max()) >= 2
