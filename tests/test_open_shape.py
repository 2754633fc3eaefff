"""Host-side check (no GPU): a batched launch opens the next step of every chain
exactly once, whatever the height of the cluster tiles, whose workgroups have
16 threads per row."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)


@pytest.mark.parametrize("tile_h", [16, 32, 64])
def test_every_chain_opened_once(tmp_path, tile_h):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not available")
    exe = str(tmp_path / "open_shape")
    subprocess.run([hipcc, "-O1", "-std=c++17", f"-DCVF_SW_TILE_H={tile_h}", "-I", os.path.join(ROOT, "include"),
                    "-I", os.path.join(ROOT, "paper_2505_05919_amd", "csrc"),
                    os.path.join(HERE, "helpers", "open_shape.cpp"), "-o", exe], check=True)
    counts = list(range(1, 20)) + [63, 64, 65, 300]
    out = subprocess.run([exe], input="\n".join(map(str, counts)), capture_output=True, text=True, check=True).stdout
    lines = [list(map(int, line.split())) for line in out.splitlines()]
    assert [r[0] for r in lines] == counts
    for count, waves, *opened in lines:
        assert waves == tile_h // 4
        assert opened == [1] * (2 * count)
