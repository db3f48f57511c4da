"""The few-row GEMM kernel (K taken whole by each workgroup) and its dispatch
against the oracle, bit for bit: x small multiples of 1/4 and scales powers of
two, so that every partial sum is exact in binary32 in any order.

Row counts at the edges of 16-, 32- and 64-row groups and over one; weight rows
that do not fill a workgroup of 16, 32, 48 or 64; K of fewer steps than waves,
an odd number of them, and of several rounds; x small enough to be staged whole
and not; every block size, with as many scales as can be staged and more (the
split kernels take those); K >= 4 N, where K is split over the grid (the
weight-streaming kernel, the few-row kernel with K in ranges, and for (40, 96,
9600) 128 x 256 tiles).
"""
import numpy as np
import pytest
import torch

import oracle
import paper_2501_04266_amd as zq
from paper_2501_04266_amd import workloads as wl
from tests.gpu_util import from_dev, poisoned, to_dev

pytestmark = pytest.mark.gpu

# (M, N, K, B)
CASES = [(1, 1, 64, 32), (1, 2049, 2048, 256), (2, 6143, 1088, 64), (4, 16385, 192, 128), (3, 100, 320, 1024),
         (5, 2050, 5120, 256), (16, 6145, 2048, 32), (16, 1023, 1600, 128), (9, 16400, 2880, 256),
         (17, 2047, 2048, 256), (24, 16433, 640, 128), (32, 1500, 1984, 512), (31, 16384, 128, 32),
         (33, 2048, 2048, 128), (64, 2049, 1024, 256), (48, 12320, 448, 64), (63, 16390, 1024, 256),
         (65, 1000, 1088, 256), (130, 2065, 960, 128), (256, 2048, 2048, 256), (200, 333, 704, 1024),
         (16, 64, 4160, 256), (20, 130, 24640, 32), (40, 96, 9600, 32), (1, 300, 24576, 32),
         # K in a few ranges: whole, ragged and odd ones, blocks that straddle rows and ranges
         (16, 6144, 24576, 256), (9, 6100, 24640, 512), (32, 6144, 24576, 1024), (24, 4111, 16448, 256),
         (17, 3000, 12352, 512), (30, 2000, 8256, 1024)]


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("M,N,K,B", CASES)
def test_few_rows_exact(M, N, K, B, dtype):
    rng = np.random.default_rng(M * 13 + N + K)
    x = wl.to_storage((rng.integers(-8, 9, M * K) / 4.0).astype(np.float32), dtype).reshape(M, K)
    codes = rng.integers(-127, 128, N * K).astype(np.int8)
    # powers of two that differ from block to block: a wrong scale shows
    scales = (2.0 ** -rng.integers(6, 9, -(-(N * K) // B))).astype(np.float32)
    want = oracle.qwz_dequant_gemm(x, codes, scales, N, B, dtype)
    buf = poisoned(M * N + 2, torch.float32)
    guard = buf.clone()
    y = buf[1:1 + M * N].view(M, N)  # 4 bytes past a 16-byte boundary
    zq.qwz_dequant_gemm(to_dev(x, dtype).reshape(M, K), to_dev(codes), to_dev(scales), N, B, y=y)
    torch.cuda.synchronize()
    got = from_dev(y).astype(np.float64)
    bad = np.flatnonzero(got != want)
    assert bad.size == 0, f"{bad.size} of {got.size} differ; first at {np.unravel_index(bad[0], got.shape)}"
    assert torch.equal(buf[[0, -1]].view(torch.int32), guard[[0, -1]].view(torch.int32))


# the tiled kernel's shapes: 256 x 192 (first two), 256 x 128 (next two), with K
# split in two (fifth) and (900, 4000, 2048); ragged rows and columns, blocks whose
# scales start inside a tile's first row group.  The other three run the few-row
# kernel's wide variants.  (Every shape, whole and split: test_gpu_gemm_routes.py.)
TILES = [(300, 18431, 640, 256), (257, 18432, 320, 1024), (500, 12280, 640, 128), (511, 12289, 192, 32),
         (400, 6100, 3072, 256), (520, 2050, 4096, 512), (300, 2000, 6144, 64), (900, 4000, 2048, 256),
         (1030, 2049, 1088, 1024)]


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("M,N,K,B", TILES)
def test_tile_shapes_exact(M, N, K, B, dtype):
    test_few_rows_exact(M, N, K, B, dtype)


def test_few_rows_same_bits_twice():
    """Without a split over the grid the sums run in one fixed order."""
    rng = np.random.default_rng(3)
    M, N, K, B = 16, 6144, 2048, 256
    x = to_dev(wl.to_storage(rng.standard_normal(M * K).astype(np.float32), "bf16"), "bf16").reshape(M, K)
    codes, scales = oracle.qwz_quantize((rng.standard_normal(N * K) * 0.02).astype(np.float32), B, "f32")
    args = (x, to_dev(codes), to_dev(scales), N, B)
    a, b = zq.qwz_dequant_gemm(*args), zq.qwz_dequant_gemm(*args)
    torch.cuda.synchronize()
    assert torch.equal(a, b)
