"""The packed layouts of the fp32 path, on the host: the pack kernel's piece
order (row_piece) against the positions at which the gate and head kernels
read a value, written out here, and the split activations' offsets
(split_offset) as a bijection onto part 0 of each packed tile. Whole and
ragged last row blocks, one row, one k tile. Compiled for the host only."""
import os
import shutil
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SRC = r'''
#include <cstdio>
#include <cstdlib>
#include "zo_pack.hpp"
int main(int, char** argv) {
  const int64_t n = atoll(argv[1]), K = atoll(argv[2]);
  for (int64_t u = 0; u < n * K / 4; ++u) {
    const zo::RowPiece p = zo::row_piece((uint64_t)u, n, K);
    std::printf("%lld %d\n", (long long)p.row, p.k);
  }
  for (int64_t r = 0; r < n; ++r)
    for (int k = 0; k < K; ++k) std::printf("%zu 0\n", zo::split_offset(r >> 4, (int)(r & 15), k, (int)K));
  return 0;
}
'''


@pytest.fixture(scope="module")
def exe(tmp_path_factory):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not available")
    d = tmp_path_factory.mktemp("pack")
    (d / "pack.cpp").write_text(SRC)
    subprocess.run([hipcc, "-std=c++17", "-O1", "-x", "hip", "--offload-arch=gfx950", "-I",
                    os.path.join(ROOT, "paper_2505_17852_amd", "csrc"), str(d / "pack.cpp"), "-o", str(d / "pack")],
                   check=True, capture_output=True)
    return str(d / "pack")


@pytest.mark.parametrize("n,K", [(1, 32), (15, 64), (16, 32), (17, 96), (128, 32), (300, 64), (1027, 256)])
def test_f32_packed_layouts(exe, n, K):
    out = subprocess.run([exe, str(n), str(K)], check=True, capture_output=True, text=True).stdout
    a = np.array(out.split(), np.int64).reshape(-1, 2)
    pieces, split = a[: n * K // 4], a[n * K // 4:, 0]

    # the packed matrix by the pack kernel's order: value (row, k) holds row K + k
    packed = (pieces[:, :1] * K + pieces[:, 1:] + np.arange(4)).reshape(-1)
    # and as the kernels read it: block b of R rows at 16 b K values, its k tile kt
    # 32 R values further each, the halves 16 R apart, lane (row, kg) at (kg R + row) 4
    row, k = (x.reshape(-1) for x in np.meshgrid(np.arange(n), np.arange(K), indexing="ij"))
    b = row // 16
    R = np.minimum(16, n - 16 * b)
    kt, kg, half = k // 32, k % 32 // 8, k % 8 // 4
    at = 16 * b * K + kt * 32 * R + half * 16 * R + (kg * R + row % 16) * 4 + k % 4
    assert np.array_equal(np.sort(at), np.arange(n * K))
    assert np.array_equal(packed[at], row * K + k)

    # part 0 of tile (rt, kt): 1 KB at 3 KB steps, every 2-byte value once
    tile = (row // 16) * (K // 32) + kt
    assert np.array_equal(split // 3072, tile)
    assert np.all(split % 3072 < 1024) and np.all(split % 2 == 0)
    assert np.unique(split).size == n * K
    assert np.array_equal(split % 1024, (row % 16 + 16 * kg) * 16 + 2 * (k % 8))
