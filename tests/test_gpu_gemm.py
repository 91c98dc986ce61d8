"""GPU parity of the matrix-core GEMM's block shapes (wq_gemm.hip): every
compiled shape (forced with WQ_GEMM_CONFIG, in single, planned and listed
launches) at sizes that leave remainders in M, N and K, with scales on both
sides of the short dequantization's limit and scale arrays that start in the
middle of a dword.

Inputs are integer-exact: x in {-4..4} and scales 2^e, e in [-10, -2], so every
product is a multiple of 2^-10 and every sum of K = 1056 of them at most
4 * 8 * 2^-2 * 1056 < 2^14; all partial sums are exact in fp32 and the result
is unique up to its one fp16 rounding, so the comparison is bit for bit.
"""

from __future__ import annotations

import os
import re

import numpy as np
import pytest

import oracle
from gpu_util import announce, gpu_gemv, to_dev, to_host
from paper_2412_15803_amd import workloads as wl
from paper_2412_15803_amd import wq

pytestmark = pytest.mark.gpu



def _block_shapes():
    """The rows of the source's WQ_GEMM_CONFIGS: what index WQ_GEMM_CONFIG
    names.  The library forces a shape on M > 64 if TM >= 2 and R = 16, on
    2 <= M <= 64 if TM <= 4, and picks its own where it cannot."""
    names = ("tm", "tn", "nw", "kw", "xk", "ck", "w", "r", "occ")
    table = open(os.path.join(os.path.dirname(wq.__file__), "csrc", "wq_gemm.hip")).read()
    table = table[table.index("#define WQ_GEMM_CONFIGS(X)"):table.index("struct Config {")]
    return [dict(zip(names, map(int, row.split(",")))) for row in re.findall(r"X\(([\d, ]+)\)", table)]


SHAPES = _block_shapes()
TALL = [i for i, c in enumerate(SHAPES) if c["r"] == 16]  # 16 rows of x per tile, or each of 4 in four places
SMALL_BATCH = [i for i, c in enumerate(SHAPES) if c["tm"] <= 4]
PROMPT = [i for i in TALL if SHAPES[i]["tm"] >= 2]
LINES = [i for i, c in enumerate(SHAPES) if c["ck"] == 256]
assert len(SHAPES) >= 24 and len(LINES) >= 16 and all(SHAPES[i]["tm"] <= 4 for i in LINES)


def _case(m, n, k, seed, shift=0, lo=-10, hi=-2):
    import torch

    packed = wl.random_words_host(seed, n, k)
    scales = wl.pow2_scales_host(seed + 1, n, k, lo, hi)
    x = wl.small_int_x_host(seed + 2, m, k)
    ng = k // 32
    buf = torch.zeros(n * ng + shift, dtype=torch.int16, device="cuda:0")
    buf[shift:] = to_dev(scales).reshape(-1)
    return packed, scales, x, buf[shift:].view(n, ng)


def _check(m, n, k, seed, shift=0):
    packed, scales, x, sd = _case(m, n, k, seed, shift)
    y = to_host(gpu_gemv(to_dev(packed), sd, to_dev(x)), np.uint16)
    ref = oracle.gemv(packed, scales, x, n, k).view(np.uint16)
    bad = np.argwhere(y != ref)
    assert bad.size == 0, f"{len(bad)} mismatches, first {bad[:5].tolist()}"


@pytest.mark.parametrize("shift", [0, 1])
@pytest.mark.parametrize("config", TALL)
def test_block_shape_exact(config, shift, monkeypatch):
    """One block past a whole number of them in N, a ragged M over two or
    more blocks of rows, and K = 4 whole stages and one group."""
    monkeypatch.setenv("WQ_GEMM_CONFIG", str(config))
    m = 131 if config in PROMPT else 19
    announce(f"gemm config {config} M={m} N=530 K=1056 scale shift {shift}")
    _check(m, 530, 1056, 100 * config + shift, shift)


def _check_list(m, shapes, seed, lo=-10, hi=-2):
    """Independent linears through wq_decode_linears, every second one with
    scales that start in the middle of a dword."""
    import torch

    cases = [_case(m, n, k, seed + 10 * i, i % 2, lo, hi) for i, (n, k) in enumerate(shapes)]
    lins = [(to_dev(p), sd, to_dev(x), torch.full((m, p.shape[0]), float("nan"), dtype=torch.float16, device="cuda:0"))
            for p, _, x, sd in cases]
    wq.wq_decode_linears(lins, m=m)
    torch.cuda.synchronize()
    for (p, s, x, _), (*_, y), (n, k) in zip(cases, lins, shapes):
        bad = np.argwhere(to_host(y, np.uint16) != oracle.gemv(p, s, x, n, k).view(np.uint16))
        assert bad.size == 0, f"{n} x {k}: {len(bad)} mismatches, first {bad[:5].tolist()}"


@pytest.mark.parametrize("config", SMALL_BATCH)
def test_block_shape_planned_exact(config, monkeypatch):
    """Several linears in one planned launch, a block of rows of x and part of
    a second one where 64 rows allow it."""
    monkeypatch.setenv("WQ_GEMM_CONFIG", str(config))
    m = min(SHAPES[config]["r"] * SHAPES[config]["tm"] + 3, 61)
    announce(f"gemm config {config} planned M={m}")
    _check_list(m, [(275, 352), (530, 1056), (17, 96), (1, 32)], 300 * config)


@pytest.mark.parametrize("config", PROMPT)
def test_block_shape_listed_exact(config, monkeypatch):
    monkeypatch.setenv("WQ_GEMM_CONFIG", str(config))
    announce(f"gemm config {config} listed M=131")
    _check_list(131, [(275, 352), (530, 1056), (17, 96), (1, 32)], 400 * config)


@pytest.mark.parametrize("config", LINES)
def test_block_shape_turned_exact(config, monkeypatch):
    """K = 8192 and one block of rows of x: the blocks of a linear start their
    walk along K at different windows, in single and in planned launches.
    Sums below 4 * 8 * 2^-4 * 8192 = 2^14."""
    monkeypatch.setenv("WQ_GEMM_CONFIG", str(config))
    c = SHAPES[config]
    m, rows = c["r"] * c["tm"] - 1, 16 * c["tn"] * c["nw"]
    n = 3 * rows + 5
    announce(f"gemm config {config} turned M={m} N={n}")
    packed, scales, x, sd = _case(m, n, 8192, 500 * config, 0, -10, -4)
    y = to_host(gpu_gemv(to_dev(packed), sd, to_dev(x)), np.uint16)
    assert np.array_equal(y, oracle.gemv(packed, scales, x, n, 8192).view(np.uint16))
    _check_list(m, [(rows + 5, 8192), (40, 64)], 600 * config, lo=-10, hi=-4)


@pytest.mark.parametrize("m,n,k", [(3, 1, 32), (3, 17, 64), (16, 33, 2080), (17, 257, 96), (48, 65, 8224), (49, 31, 224),
                                   (64, 300, 288), (65, 1, 32), (97, 700, 352), (129, 129, 608)])
def test_picked_shape_exact(m, n, k):
    """The shape that the size rule picks, at the smallest sizes and at
    remainders of the tiles and stages."""
    announce(f"gemm M={m} N={n} K={k}")
    _check(m, n, k, m + n + k, shift=n % 2)


@pytest.mark.parametrize("m", [5, 40, 100])
def test_rows_and_columns_stay_apart(m):
    """A NaN row of x reaches only its own outputs and a NaN scale only its
    own column, also where K ends inside a stage."""
    n, k = 70, 352
    packed, scales, x, _ = _case(m, n, k, 7 * m)
    ref = oracle.gemv(packed, scales, x, n, k).view(np.uint16)
    xb, sb = x.copy(), scales.copy()
    xb[1] = np.nan
    sb[33, 0] = 0x7E00
    announce(f"gemm NaN row and column M={m}")
    y = to_host(gpu_gemv(to_dev(packed), to_dev(sb), to_dev(xb)), np.uint16)
    keep_r, keep_c = np.arange(m) != 1, np.arange(n) != 33
    assert np.array_equal(y[np.ix_(keep_r, keep_c)], ref[np.ix_(keep_r, keep_c)])
    assert np.isnan(y[1].view(np.float16)).all() and np.isnan(y[:, 33].view(np.float16)).all()


def test_prompt_list_of_many_linears_exact():
    """70 independent linears and a dependent one at M = 66: more than one
    launch's worth of descriptors, in one call, bit for bit."""
    import torch

    m, lins, refs = 66, [], []
    announce("gemm list of 71 linears at M=66")
    for i in range(70):
        n, k = (64 if i == 8 else 1 + 37 * (i % 9)), 32 * (1 + i % 5)
        packed, scales, x, sd = _case(m, n, k, 1000 + i, lo=-7, hi=-6)
        lins.append((to_dev(packed), sd, to_dev(x), torch.empty((m, n), dtype=torch.float16, device="cuda:0")))
        refs.append(oracle.gemv(packed, scales, x, n, k))
    # Outputs are multiples of 2^-7 below 2^7, so this sum of 64 is exact too.
    packed, scales, _, sd = _case(m, 40, 64, 2000, lo=-5, hi=-5)
    lins.append((to_dev(packed), sd, lins[8][3], torch.empty((m, 40), dtype=torch.float16, device="cuda:0")))
    refs.append(oracle.gemv(packed, scales, refs[8], 40, 64))
    wq.wq_decode_linears(lins, m=m)
    torch.cuda.synchronize()
    for (_, _, _, y), ref in zip(lins, refs):
        assert np.array_equal(to_host(y, np.uint16), ref.view(np.uint16))


# Blocks that hold four rows of x per tile, each in the places of four lane
# groups, so that a tile's sums are those of single groups.
GROUP_CONFIGS = [i for i, c in enumerate(SHAPES) if c["r"] == 4 or (c["tn"], c["kw"]) == (1, 8)]


@pytest.mark.parametrize("m", [2, 3, 4, 5, 8, 19])
@pytest.mark.parametrize("config", GROUP_CONFIGS)
def test_group_sum_shape_exact(config, m, monkeypatch):
    """Ragged rows in one block, or several blocks of rows; K of four whole
    stages and one group."""
    monkeypatch.setenv("WQ_GEMM_CONFIG", str(config))
    announce(f"gemm config {config} M={m} N=275 K=1056")
    _check(m, 275, 1056, 100 * config + m, shift=m % 2)


@pytest.mark.parametrize("m,n,k", [(2, 1, 32), (2, 17, 64), (4, 33, 2080), (5, 257, 96), (8, 65, 8224), (7, 31, 224),
                                   (2, 300, 16384), (8, 1000, 8192)])
def test_group_sum_picked_exact(m, n, k):
    announce(f"gemm M={m} N={n} K={k}")
    if k > 8224:  # keep every sum exact: at most 4 * 8 * 2^-4 * 16384 = 2^15
        # In a list: alone, two rows of so deep a K take the vector kernel.
        _check_list(m, [(n, k), (n, k)], m + n, lo=-10, hi=-4)
    else:
        _check(m, n, k, m + n + k, shift=n % 2)


@pytest.mark.parametrize("n,k", [(1, 3584), (17, 3552), (2048, 3584), (2049, 3584), (2049, 8192), (300, 16384), (2050, 13824),
                                 (8193, 4096), (10241, 4096), (17, 3072), (17, 3104), (3072, 6176), (3073, 8192),
                                 (10240, 4096), (5120, 14336)])
def test_two_rows_on_either_kernel_exact(n, k):
    """Both sides of the line between the vector kernel and the GEMM at
    M = 2, through wq_gemv and as the second of two dependent linears."""
    import torch

    announce(f"two rows N={n} K={k}")
    packed, scales, x, sd = _case(2, n, k, n + k, n % 2, -10, -7)  # sums below 4 * 8 * 2^-7 * 16384 = 2^12
    ref = oracle.gemv(packed, scales, x, n, k).view(np.uint16)
    pd = to_dev(packed)
    assert np.array_equal(to_host(gpu_gemv(pd, sd, to_dev(x)), np.uint16), ref)
    # x of the second linear is the first one's y: one nonzero weight per row, code 9 at a scale of 1.
    ident = np.full((k, 4), 0x88888888, dtype=np.uint32)
    r = np.arange(k)
    ident[r, r % 32 // 8] += np.uint32(1) << (4 * (r % 8)).astype(np.uint32)
    first_x = np.zeros((2, 32), dtype=np.float16)
    first_x[:, :8] = wl.small_int_x_host(n, 2, 8)
    x2 = first_x[:, np.arange(k) % 32]
    ref2 = oracle.gemv(packed, scales, x2, n, k).view(np.uint16)
    ones = torch.ones((k, 1), dtype=torch.float16, device="cuda:0")
    mid = torch.full((2, k), float("nan"), dtype=torch.float16, device="cuda:0")
    y = torch.full((2, n), float("nan"), dtype=torch.float16, device="cuda:0")
    wq.wq_decode_linears([(to_dev(ident), ones, to_dev(first_x), mid), (pd, sd, mid, y)], m=2)
    torch.cuda.synchronize()
    assert np.array_equal(to_host(y, np.uint16), ref2)


@pytest.mark.parametrize("m", [2, 4, 7])
def test_group_sum_special_values(m):
    """An infinity in x gives what the sum of its products gives (infinite,
    or no number at a weight of zero), the largest x stays finite, and other
    rows keep their bits."""
    n, k = 70, 352
    packed, scales, x, _ = _case(m, n, k, 9 * m)
    ref = oracle.gemv(packed, scales, x, n, k).view(np.uint16)
    w = oracle.dequant(packed, scales, n, k)
    xb = x.copy()
    xb[1, 300] = np.inf
    announce(f"gemm infinity M={m}")
    y = to_host(gpu_gemv(to_dev(packed), to_dev(scales), to_dev(xb)), np.uint16)
    keep = np.arange(m) != 1
    assert np.array_equal(y[keep], ref[keep])
    with np.errstate(invalid="ignore"):
        want = np.inf * w[:, 300]
    assert np.array_equal(y[1].view(np.float16).astype(np.float64), want, equal_nan=True)
    xb = np.zeros_like(x)
    xb[1, ::32] = 65504.0
    s = np.full_like(scales, 0x0001)  # 2^-24
    y = to_host(gpu_gemv(to_dev(packed), to_dev(s), to_dev(xb)), np.uint16)
    assert np.array_equal(y, oracle.gemv(packed, s, xb, n, k).view(np.uint16))


@pytest.mark.parametrize("big", [1000.0, 10000.0, 60000.0])
@pytest.mark.parametrize("scale", [0.02, 0.2, 1.0])
@pytest.mark.parametrize("m", [2, 3, 4])
def test_outliers_at_zero_weights(m, scale, big):
    """Activations of up to 6e4 in every group, where the code is 8 (weight
    zero), among small ones: their products are exactly zero, so they add
    nothing to the documented bound and must add nothing to the error."""
    import torch

    n, k = 70, 352
    packed = wl.random_words_host(31 * m, n, k)
    col = np.arange(5, k, 32)  # element 5 of its word
    packed[:, col // 8] = (packed[:, col // 8] & ~np.uint32(0xF << 20)) | np.uint32(8 << 20)
    scales = np.full((n, k // 32), scale, dtype=np.float16).view(np.uint16)
    rng = np.random.default_rng(int(big) + m)
    x = (0.01 * rng.standard_normal((m, k))).astype(np.float16)
    x[:, col] = np.where(rng.random((m, col.size)) < 0.5, big, -big)
    ref, bound = oracle.gemv(packed, scales, x, n, k), oracle.tol_bound(packed, scales, x, n, k)
    announce(f"gemm outliers M={m} scale {scale} x {big}")
    pd, sd, xd = to_dev(packed), to_dev(scales), to_dev(x)
    y = to_host(gpu_gemv(pd, sd, xd), np.float16)
    assert np.all(oracle.within_tolerance(y, ref, bound))
    yd = torch.full((m, n), float("nan"), dtype=torch.float16, device="cuda:0")
    wq.wq_decode_linears([(pd, sd, xd, yd)], m=m)
    torch.cuda.synchronize()
    assert np.all(oracle.within_tolerance(to_host(yd, np.float16), ref, bound))
