"""The dequantise-on-load GEMM's plan (csrc/zq_gemm_plan.h, host arithmetic),
compiled with the host compiler and asked without a GPU: which kernel runs the
shapes of the GPU tests, that no plan exceeds what its kernels can hold or sums
longer chains than the plans it is compared with, and the edges of its rules."""
import os
import random
import subprocess

import pytest

from tests.gemm_routes import ROUTES

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2501_04266_amd", "csrc")


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("plan") / "gemm_plan")
    subprocess.run(["g++", "-std=c++17", "-O2", "-Wall", "-Wextra", "-Werror", "-I", CSRC,
                    os.path.join(HERE, "c", "gemm_plan.cpp"), "-o", exe], check=True)

    def ask(shapes, cus=256):
        text = "".join(f"{M} {N} {K} {B} {cus}\n" for M, N, K, B in shapes)
        out = subprocess.run([exe], input=text, capture_output=True, text=True, check=True).stdout.splitlines()
        rows = []
        for line in out:
            name, mt, nt, splits, grid, us, drift, limit = line.split()
            rows.append((name, int(mt), int(nt), int(splits), int(grid), float(us), float(drift), float(limit)))
        assert len(rows) == len(shapes)
        return rows
    return ask


def test_gpu_shapes_run_the_kernels_they_name(plan):
    got = plan([r[1:] for r in ROUTES])
    wrong = [(want, g[0], s) for (want, *s), g in zip(ROUTES, got) if want != g[0]]
    assert not wrong, wrong


def _shapes(count, seed):
    rng = random.Random(seed)
    out = []
    for _ in range(count):
        M = int(2 ** rng.uniform(0, 13.3))
        N = int(2 ** rng.uniform(0, 17))
        K = 64 * int(2 ** rng.uniform(0, 11))
        out.append((M, N, K, rng.choice([32, 64, 128, 256, 512, 1024])))
    return out


@pytest.mark.parametrize("cus", [256, 64, 32])
def test_plans_fit_their_kernels(plan, cus):
    shapes = _shapes(20000, 5) + [(M, N, 64 * k, 1024) for M in (1, 16, 32) for N in (1, 64, 90, 96)
                                  for k in (1 << 14, 40000, 174762, 174763, 1 << 18)]
    for (M, N, K, B), (name, mt, nt, splits, grid, us, drift, limit) in zip(shapes, plan(shapes, cus)):
        what = (M, N, K, B, name, splits)
        kind, _, rest = name.partition(":")
        assert 0 < grid < 2 ** 31, what
        if kind in ("rows", "ranges"):
            m16, n16 = (int(v) for v in rest.split(",")[0].split("x"))
            assert nt * 16 * n16 >= N > (nt - 1) * 16 * n16 and mt * 16 * m16 >= M, what
            # byte offsets of weight rows and of x stay below the mark of a dead load
            assert 16 * n16 * K < 2 ** 30 and 2 * 16 * m16 * K < 2 ** 30, what
            if kind == "rows":
                assert 16 * n16 * K // B + 1 <= 8192, what  # scales in LDS
                assert grid >= nt * mt and splits == 1, what
                if "staged" in rest:
                    assert 2 * M * K <= 49152, what
            else:
                assert mt == 1 and 2 <= splits <= K // 1024, what
                assert -(-nt // 8) * splits <= cus // 8, what  # one round on the XCD that has the most
                pairs = K // 128
                for s in range(splits):  # a row's scales of one range fit its 64 places, wherever it starts
                    lo, hi = s * pairs // splits * 128, (s + 1) * pairs // splits * 128
                    hi = K if s == splits - 1 else hi
                    for r in (0, 1, 95):
                        assert (r * K + hi - 1) // B - (r * K + lo) // B + 1 <= 64, what
        elif kind == "stream":
            assert M <= 16 and nt == -(-N // 64) and splits == (-(-K // int(rest.split(",")[0])) or 1), what
        elif kind == "tiles":
            bm, bn = (int(v) for v in rest.split(",")[0].split("x"))
            assert nt == -(-N // bn) and mt == -(-M // bm) and 1 <= splits <= max(1, min(16, K // 64)), what
            assert K <= 2 ** 21 and grid == mt * nt * splits, what


@pytest.mark.parametrize("cus", [256, 64])
def test_no_plan_sums_longer_chains(plan, cus):
    shapes = _shapes(20000, 11)
    for s, (name, *_, drift, limit) in zip(shapes, plan(shapes, cus)):
        assert name == "plain" or drift <= limit + 0.051, (s, name, drift, limit)
    # 256 x 192 tiles of whole K, one set of accumulators, where tiles of 256 columns
    # would be split: longer chains, not taken
    (name, _, _, splits, *_), = plan([(260, 18432, 6144, 256)], cus=256)
    assert name == "tiles:256x256,split" and splits == 3


def test_edges(plan):
    # more ranges of K than 1024 allows: as many as it does, not none
    (name, _, _, splits, *_), = plan([(32, 2048, 8192, 256)])
    assert (name, splits) == ("ranges:2x6,waves8,sets2", 8)
    # no plan that takes K whole (its scales do not fit LDS): the ranges are still compared
    (name, *_), = plan([(32, 2048, 16384, 64)])
    assert name == "ranges:2x6,waves8,sets2"
    # K a little below 4 N: the streaming kernel where splitting K over the grid is faster
    (name, *_), = plan([(16, 2048, 4096, 256)])
    assert name.startswith("stream:")
    # the number of compute units reaches both models: as many weight rows a workgroup
    # as leave one workgroup for each
    (few, *_), (many, *_) = plan([(16, 6144, 2048, 256)], cus=64) + plan([(16, 6144, 2048, 256)], cus=256)
    assert few == "rows:1x6,waves8" and many == "rows:1x2,waves16,sets2"
    # no columns of K at all
    assert [r[0] for r in plan([(1, 64, 0, 256), (17, 64, 0, 256)])] == ["stream:256", "tiles:128x256"]
