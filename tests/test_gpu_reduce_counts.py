"""Reduce levels of every slice count at which a kernel's structure changes,
against the oracle, bit for bit: the counts fixed at compile time (1 to 8 on
large levels; 2, 4 and 8 on small ones), and by batches (of 6 on small levels,
of 4 and 3 on large ones) every size of the first batch with none, one, two and
three whole batches after it.  Whole and ragged lengths, plain, fused and
gathered, and one block whose 16 s overflows.

Blocks of 1024 take the large level's kernels at every length, so most counts
run there on short levels; one long level for each other block size.
"""
import numpy as np
import pytest
import torch

import oracle
import paper_2501_04266_amd as zq
from tests.gpu_util import assert_bits_equal, from_dev, to_dev

pytestmark = pytest.mark.gpu

LARGE = 4096 * 2048  # elements from which blocks of up to 512 take the large level's kernels
COUNTS = list(range(1, 19)) + [24, 25, 64]
CASES = ([(P, 8192 * 2 + 1024 * (P % 3), 1024) for P in COUNTS] + [(P, 8192 + 7, 1024) for P in (1, 5, 11, 15)] +
         [(P, 2048 * 3 + B * (P % 2), B) for P in COUNTS for B in (32, 256, 512)] +
         [(P, 4096 + 33, 512) for P in (1, 6, 9, 14)] +
         [(1, LARGE + 32 * 70, 32), (2, LARGE + 512 * 3, 512), (3, LARGE + 64, 64), (5, LARGE + 17, 128),
          (6, LARGE + 256 * 9, 256), (7, LARGE + 512, 512), (8, LARGE + 32 * 33, 32), (9, LARGE + 128 * 11, 128),
          (11, LARGE + 64 * 5, 64), (13, LARGE + 512 * 7 + 5, 512), (14, LARGE + 256, 256)])


@pytest.mark.parametrize("P,m,B", CASES)
def test_reduce_counts(P, m, B):
    rng = np.random.default_rng(1000 * P + m % 997 + B)
    nb, ns = (m + 1) // 2, -(-m // B)
    packed = rng.integers(0, 256, (P, nb), dtype=np.uint8)
    if m % 2:
        packed[:, -1] &= 0x0F
    scales = rng.uniform(2e-4, 1e-3, (P, ns)).astype(np.float32)
    scales[P - 1, ns // 2] = 1.5 * 2.0 ** 124
    op, os_ = oracle.qgz_reduce_level(packed.reshape(-1), scales.reshape(-1), P, m, B)
    what = f"P={P} m={m} B={B}"
    dp, ds = to_dev(packed.reshape(-1)), to_dev(scales.reshape(-1))
    bufs, sbufs = [to_dev(p) for p in packed], [to_dev(s) for s in scales]
    noalloc = (torch.full((nb,), 0xA5, dtype=torch.uint8, device="cuda"),
               torch.full((ns,), -1.0, dtype=torch.float32, device="cuda"))
    results = [("plain", zq.qgz_reduce_level(dp, ds, P, m, B)),
               ("tables", zq.qgz_reduce_level_gather(bufs, sbufs, m, B)),
               ("arguments", zq.qgz_reduce_level_gather_noalloc(bufs, sbufs, m, B, *noalloc))]
    y = zq.qgz_reduce_dequantize(dp, ds, P, m, B, out_dtype=torch.bfloat16)
    torch.cuda.synchronize()
    for form, (gp, gs) in results:
        assert_bits_equal(from_dev(gp), op, f"{what} {form} codes", B // 2)
        assert_bits_equal(from_dev(gs), os_, f"{what} {form} scales")
    assert_bits_equal(from_dev(y), oracle.qgz_dequantize(op, os_, m, B, "bf16"), what + " fused", B)
