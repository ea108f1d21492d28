"""Row chunks of the Gram products (host code, no GPU).

The FP32 products of the mixed-precision split Rayleigh-Ritz sum a chunk's rows
in FP32 and the chunks in FP64, so a chunk may not hold more rows than the
chunk count it stands for gives it: M / (4096 / blocks), and no more than by
128 x 128 tiles in 1024 workgroups.  Limits: at least 256 rows per chunk, and
less than 2 GB of the widest operand."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
DRIVER = os.path.join(ROOT, "tests", "native", "gram_chunks.cpp")

WIDTHS = [1, 16, 64, 65, 128, 129, 160, 256, 257, 512, 1024, 1408, 1473, 1536, 2048, 2304, 3300, 3328, 4096, 5760,
          5824, 8192]
ROWS = [27, 256, 257, 5000, 216000, 373248, 2985984]


@pytest.fixture(scope="module")
def chunks(tmp_path_factory):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ not available")
    exe = str(tmp_path_factory.mktemp("gram") / "gram_chunks")
    r = subprocess.run([gxx, "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", DRIVER, "-o", exe],
                       capture_output=True, text=True)
    if r.returncode != 0 and "hip_runtime" in r.stderr:
        pytest.skip("HIP headers not available for a host build")
    assert r.returncode == 0, r.stderr

    def run(cases):
        text = "".join("%d %d %d %d\n" % c for c in cases)
        out = subprocess.run([exe], input=text, capture_output=True, text=True, check=True).stdout
        return [tuple(int(v) for v in line.split()) for line in out.splitlines()]
    return run


@pytest.mark.parametrize("single", [0, 1])
def test_chunk_rows(chunks, single):
    cases = [(M, n, n, single) for M in ROWS for n in WIDTHS]
    for (M, n, ld, _), (ch, blocks) in zip(cases, chunks(cases)):
        nb = -(-n // 64)
        assert blocks == nb * (nb + 1) // 2
        rows = -(-M // ch)
        assert ch >= 1 and rows * ld * 8 < 2 ** 31
        if not single:
            continue
        tiles = -(-n // 128)
        tiles = tiles * (tiles + 1) // 2
        longest = max(min(M * blocks / 4096, M / -(-1024 // tiles)), M / -(-M // 256))
        assert M / ch <= longest, (M, n, ch)
