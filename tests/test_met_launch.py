"""Host-side check (no GPU) of the Metropolis launch as a chain takes it: quads
for every even L, one row per wavefront up to L = 2046 and blocks of whole row
pairs beyond, every row covered once, no lane with more cells than its packed
counters hold."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)


@pytest.fixture(scope="module")
def launches(tmp_path_factory):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not available")
    exe = str(tmp_path_factory.mktemp("met") / "met_launch_shapes")
    subprocess.run([hipcc, "-O1", "-std=c++17", "-I", os.path.join(ROOT, "paper_2505_05919_amd", "csrc"),
                    os.path.join(HERE, "helpers", "met_launch_shapes.cpp"), "-o", exe], check=True)
    Ls = range(2, 32768, 2)
    out = subprocess.run([exe], input="\n".join(map(str, Ls)), capture_output=True, text=True, check=True).stdout
    rows = [tuple(map(int, line.split())) for line in out.splitlines()]
    assert [r[0] for r in rows] == list(Ls)
    return rows


def test_launches_cover_the_lattice(launches):
    for L, quad, rows, row_blocks, _ in launches:
        assert quad == (1 if L % 4 == 0 else 2), L
        if L <= 2046:
            assert rows == 1, L
        else:
            assert rows % 2 == 0 and 2 <= rows <= 32, L    # whole row pairs
        assert 4 * rows * row_blocks >= L > 4 * rows * (row_blocks - 1), L
        assert 2 * rows <= 64, L                           # two cells of a quad per row and colour
        assert row_blocks + 1 <= 65535, L                  # grid.y, with the row that opens the next step


def test_launch_of_the_benchmark_lattice(launches):
    (shape,) = [r[1:4] for r in launches if r[0] == 4096]
    assert shape == (1, 16, 64)                            # 1024 workgroups of four wavefronts


def test_unaligned_rows_stay_in_cache_on_large_lattices(launches):
    for L, quad, _, _, through in launches:
        assert through == (quad == 1 or L <= 3740), L
