"""Reduce levels of any length against the oracle: slices that start at odd
byte addresses (m % 32 != 0), a last group that does not divide the full
blocks, a short last block in the same launch, levels smaller than one group,
and slice counts that fill whole, partial and single batches.

A group is 2048 elements on small levels (8 per lane) and 8192 on large ones
(32 per lane, from 4096 such waves: m of about 8.4 million; every m at
B = 1024).  Everything is bit-exact.
"""
import numpy as np
import pytest
import torch

import oracle
import paper_2501_04266_amd as zq
from tests.gpu_util import assert_bits_equal, from_dev, to_dev

pytestmark = pytest.mark.gpu

LARGE = 4096 * 2048
CASES = [(1, 2047, 32), (1, 2048, 32), (3, 2049, 64), (7, 2048 + 97, 128), (8, 4095, 256), (9, 6143, 512),
         (17, 2048 * 3 + 512 + 1, 512), (4, 10239, 64), (5, 31, 32), (8, 8191, 1024), (12, 8192, 1024),
         (3, 8192 + 1024 + 7, 1024), (2, LARGE + 8193, 128), (4, LARGE + 333, 256), (8, LARGE + 64 * 129, 64),
         (3, LARGE + 1, 64), (5, LARGE + 12345, 512), (6, LARGE + 32 * 300 + 16, 32)]


def _slices(P, m, B, seed):
    rng = np.random.default_rng(seed)
    nb, ns = (m + 1) // 2, -(-m // B)
    packed = rng.integers(0, 256, (P, nb), dtype=np.uint8)
    if m % 2:
        packed[:, -1] &= 0x0F
    scales = rng.uniform(2e-4, 1e-3, (P, ns)).astype(np.float32)
    scales[:, -1] *= 3  # the last block's scale is its own
    scales[0, ns // 2] = 1.5 * 2.0 ** 124  # one block whose 16 s overflows
    return packed, scales


@pytest.mark.parametrize("P,m,B", CASES)
def test_reduce_ragged(P, m, B):
    packed, scales = _slices(P, m, B, 100 * P + m % 1000 + B)
    op, os_ = oracle.qgz_reduce_level(packed.reshape(-1), scales.reshape(-1), P, m, B)
    dp, ds = to_dev(packed.reshape(-1)), to_dev(scales.reshape(-1))
    what = f"P={P} m={m} B={B}"
    gp, gs = zq.qgz_reduce_level(dp, ds, P, m, B)
    torch.cuda.synchronize()
    assert_bits_equal(from_dev(gp), op, what + " codes", B // 2)
    assert_bits_equal(from_dev(gs), os_, what + " scales")
    for out, dt in (("f32", torch.float32), ("bf16", torch.bfloat16)):
        y = zq.qgz_reduce_dequantize(dp, ds, P, m, B, out_dtype=dt)
        torch.cuda.synchronize()
        assert_bits_equal(from_dev(y), oracle.qgz_dequantize(op, os_, m, B, out), what + " fused " + out, B)
    bufs, sbufs = [to_dev(p) for p in packed], [to_dev(s) for s in scales]
    if m % 32:  # slices of any alignment are accepted: every other one starts 1 byte in
        bufs = [torch.cat([b[:1], b])[1:] if p % 2 else b for p, b in enumerate(bufs)]
    gp, gs = zq.qgz_reduce_level_gather(bufs, sbufs, m, B)
    torch.cuda.synchronize()
    assert_bits_equal(from_dev(gp), op, what + " gathered codes", B // 2)
    assert_bits_equal(from_dev(gs), os_, what + " gathered scales")


# up to 64 slices their addresses are kernel arguments, beyond that a device
# table; small and large levels, levels of one group and less
@pytest.mark.parametrize("P,m,B", [(1, 4096, 128), (2, LARGE + 33, 64), (6, 2049, 128), (8, 6000, 256), (3, 1000, 1024),
                                   (63, 2048 + 17, 32), (64, 8192, 1024), (64, 4096 + 5, 64), (65, 4096 + 5, 64)])
def test_gather_noalloc_slice_counts(P, m, B):
    packed, scales = _slices(P, m, B, 7 * P + m % 1000)
    op, os_ = oracle.qgz_reduce_level(packed.reshape(-1), scales.reshape(-1), P, m, B)
    bufs, sbufs = [to_dev(p) for p in packed], [to_dev(s) for s in scales]
    out = (torch.full((op.size,), 0xA5, dtype=torch.uint8, device="cuda"),
           torch.full((os_.size,), -1.0, dtype=torch.float32, device="cuda"))
    zq.qgz_reduce_level_gather_noalloc(bufs, sbufs, m, B, *out)
    torch.cuda.synchronize()
    assert_bits_equal(from_dev(out[0]), op, f"P={P} m={m} B={B} codes", B // 2)
    assert_bits_equal(from_dev(out[1]), os_, f"P={P} m={m} B={B} scales")


def test_gather_noalloc_two_streams():
    """Calls on different streams do not share their addresses (up to 64 slices)."""
    P, m, B = 8, 1 << 20, 128
    work = []
    for k in range(2):
        packed, scales = _slices(P, m, B, 40 + k)
        want = oracle.qgz_reduce_level(packed.reshape(-1), scales.reshape(-1), P, m, B)
        out = (torch.empty(m // 2, dtype=torch.uint8, device="cuda"),
               torch.empty(m // B, dtype=torch.float32, device="cuda"))
        work.append(([to_dev(p) for p in packed], [to_dev(s) for s in scales], out, want, torch.cuda.Stream()))
    torch.cuda.synchronize()
    for _ in range(20):
        for bufs, sbufs, out, _w, st in work:
            zq.qgz_reduce_level_gather_noalloc(bufs, sbufs, m, B, *out, stream=st)
    torch.cuda.synchronize()
    for k, (_b, _s, out, want, _st) in enumerate(work):
        assert_bits_equal(from_dev(out[0]), want[0], f"stream {k} codes", B // 2)
        assert_bits_equal(from_dev(out[1]), want[1], f"stream {k} scales")
