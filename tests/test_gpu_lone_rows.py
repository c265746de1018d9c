"""The row kernel's two block sizes: batches of no more rows than the device has CUs take
768 threads a row, larger ones 512.  The results do not depend on it: rows of the largest
batch of the first kind equal the same rows in a batch with one row more, bit for bit, and
the oracle's outcomes."""
import pytest
import torch

from paper_2608_24411_amd import synth
from test_gpu_parity import _flat_check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("V,dtype", [(3000, "f32"), (3001, "f32"), (12288, "bf16"), (12291, "bf16")])
@pytest.mark.parametrize("mode", ("resispec", "specinfer"))
def test_block_sizes_agree(gpu_lib, V, dtype, mode):
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    print("block sizes", V, dtype, mode, cus, flush=True)
    w = synth.make_workload(0, device="cuda", B=cus + 1, V=V, dtype=dtype)
    got = []
    for B in (cus + 1, cus):
        part = dict(w, **{k: w[k][:B].contiguous() for k in ("target", "draft", "cand_ids", "u_accept", "u_resample")})
        out = gpu_lib.resispec_verify(part["target"], part["draft"], part["cand_ids"], part["u_accept"],
                                      part["u_resample"], temperature=w["temperature"], mode=mode)
        torch.cuda.synchronize()
        got.append(out)
        _flat_check(dict(part, B=B), *out, mode)
    for a, b in zip(*got):
        assert torch.equal(a[:cus], b)


@pytest.mark.parametrize("B,N", [(1, 1), (5, 51), (1, 256), (257, 1)])
def test_node_outcomes_copies_every_row(gpu_lib, B, N):
    """255, 256 and 257 rows around a block of the copy, and a single one."""
    ws = torch.randint(0, 255, (gpu_lib.resispec_workspace_bytes(B, N),), dtype=torch.uint8, device="cuda")
    stride = ws.numel() // 12
    want = ws.view(torch.int32)
    for k, x in enumerate(gpu_lib.resispec_node_outcomes(ws, B, N)):
        assert torch.equal(x.flatten(), want[k * stride:k * stride + B * N])
