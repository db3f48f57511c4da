"""Every kernel of the dequantise-on-load GEMM, in every variant that its plan
chooses, against the oracle bit for bit, with ragged rows and columns; and the
paths that split K (a zero fill, then additions into y) captured in a graph.
The shapes and the kernels they run are in tests/gemm_routes.py, which a CPU test
holds against the plan.

Exact: x small multiples of 1/4 and scales powers of two, so that every partial
sum is a multiple of 2^-11 and, at these lengths, far below 2^13.
"""
import numpy as np
import pytest
import torch

import oracle
import paper_2501_04266_amd as zq
from paper_2501_04266_amd import workloads as wl
from tests.gemm_routes import ROUTES
from tests.gpu_util import from_dev, poisoned, to_dev

pytestmark = pytest.mark.gpu

SHAPES = [r for r in ROUTES if r[0] != "plain"]  # (test_dequant_gemm_long_k runs that one)


def _inputs(M, N, K, B, dtype):
    rng = np.random.default_rng(M * 17 + N + K)
    x = wl.to_storage((rng.integers(-4, 5, M * K) / 4.0).astype(np.float32), dtype).reshape(M, K)
    codes = rng.integers(-127, 128, N * K).astype(np.int8)
    # powers of two that differ from block to block: a wrong scale shows
    scales = (2.0 ** -rng.integers(7, 10, -(-(N * K) // B))).astype(np.float32)
    return x, codes, scales


def _assert_equal(y, want, what):
    got = from_dev(y).astype(np.float64)
    bad = np.flatnonzero(got != want)
    assert bad.size == 0, f"{what}: {bad.size} of {got.size} differ; first at {np.unravel_index(bad[0], got.shape)}"


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("route,M,N,K,B", SHAPES)
def test_route_exact(route, M, N, K, B, dtype):
    x, codes, scales = _inputs(M, N, K, B, dtype)
    want = oracle.qwz_dequant_gemm(x, codes, scales, N, B, dtype)
    buf = poisoned(M * N + 2, torch.float32)
    guard = buf.clone()
    y = buf[1:1 + M * N].view(M, N)
    zq.qwz_dequant_gemm(to_dev(x, dtype).reshape(M, K), to_dev(codes), to_dev(scales), N, B, y=y)
    torch.cuda.synchronize()
    _assert_equal(y, want, route)
    assert torch.equal(buf[[0, -1]].view(torch.int32), guard[[0, -1]].view(torch.int32))


SPLIT = [r for r in SHAPES if r[0].startswith("ranges") or r[0].endswith("split")]
SPLIT = [r for r in SPLIT if r[1] * r[2] * r[3] < 2e9] + [r for r in SHAPES if r[0] == "tiles:256x128"]


@pytest.mark.parametrize("route,M,N,K,B", SPLIT)
def test_route_graph_capture(route, M, N, K, B):
    """The zero fill and the kernel that adds into y replay from a graph, as the
    one launch of whole tiles does; y is overwritten eagerly between replays."""
    x, codes, scales = _inputs(M, N, K, B, "bf16")
    want = oracle.qwz_dequant_gemm(x, codes, scales, N, B, "bf16")
    xd, cd, sd = to_dev(x, "bf16").reshape(M, K), to_dev(codes), to_dev(scales)
    y = poisoned(M * N, torch.float32).reshape(M, N)
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.stream(s):
        with torch.cuda.graph(graph, stream=s):
            zq.qwz_dequant_gemm(xd, cd, sd, N, B, y=y)
    torch.cuda.synchronize()
    for rep in range(3):
        y.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        _assert_equal(y, want, f"{route} replay {rep}")
