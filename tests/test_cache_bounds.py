"""The path schedule's residual cache against the row layouts, on the host: whatever V, a pass
touches only the elements that the caller's workspace holds (cache_bounds.cpp, compiled with
the kernels' own layout and bounds)."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    from paper_2608_24411_amd import build
    env = {k: v for k, v in os.environ.items() if k != "LD_PRELOAD"}     # (a sanitizer's runtime)
    exe = str(tmp_path_factory.mktemp("cache") / "bounds")
    subprocess.run([build.HIPCC, "--offload-host-only", "-x", "hip", "-std=c++17", "-O1", "-w", "-I",
                    os.path.join(build.HERE, "csrc"), "-I", os.path.join(build.ROOT, "include"),
                    os.path.join(HERE, "cache_bounds.cpp"), "-o", exe], check=True, env=env)
    return exe


def test_cache_bounds(program):
    """Every size up to 1,200, then sizes spread to the largest, the ends of chunks and the
    sizes whose last slot is partial among them."""
    # (not at import: the library would come before torch, and with it another HIP runtime)
    from paper_2608_24411_amd import native
    edges = [k * 1024 + d for k in (128, 129, 130, 148, 149, 191, 257, 385, 1000, 4095) for d in (-1, 0, 1, 512, 513)]
    sizes = sorted(set(range(1, 1200)) | set(range(1201, 1 << 22, 4973)) | set(edges) |
                   {128256, 131073, 132000, 140000, 140001, 151643, 151669, 151936, 152064, 201088, 1 << 22})
    r = subprocess.run([program] + [str(v) for v in sizes], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout[-200:]
    surplus = dict(tuple(map(int, line.split())) for line in r.stdout.split("\n") if line)
    assert set(surplus) == set(sizes)
    # without the bound these would be touched past the sequence's share
    assert surplus[151936] == 1024 and surplus[132000] > 0 and surplus[128256] == 0
    # a sequence's share of the workspace: R and Q
    for v in (1, 1024, 132000, 151936):
        half = (v + 1023) // 1024 * 1024
        state = native.resispec_path_workspace_bytes(1, v) - 8 * half
        assert native.resispec_path_workspace_bytes(16, v) == 16 * (state + 8 * half)
