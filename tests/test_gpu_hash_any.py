"""The any-shape matrix-core hashing kernel (DESSERT_HASH_AUTO where no fixed-shape kernel exists) against the CPU oracle and
against the plain kernel (DESSERT_HASH_SCALAR)."""
import numpy as np
import pytest
import torch

import paper_2210_15748_amd as dz
from oracle import oracle as orc

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def both(xt, pk, X, R, L, Cb):
    ix = dz.create(X.shape[1], L, Cb, dtype=dz.I8 if xt == "i8" else dz.F16,
                   proj_kind=dz.PROJ_RADEMACHER_I8 if pk == "pm1" else dz.PROJ_GAUSSIAN_F32, proj=torch.from_numpy(R).to(DEV))
    Xd = torch.from_numpy(X).to(DEV)
    auto = dz.hash(ix, Xd).cpu().numpy()
    dz.set_algo(ix, dz.HASH_SCALAR)
    return auto, dz.hash(ix, Xd).cpu().numpy()


def i8_inputs(rng, n, d, P):
    X = rng.integers(-127, 128, (n, d)).astype(np.int8)
    X[0] = 0
    return X, (rng.integers(0, 2, (P, d)) * 2 - 1).astype(np.int8)


# d: one k-step of 32, either side of whole k-steps, the largest.  L, C: tables that divide unevenly over the two lane halves
# (12, 20, 28), several segments of 16 tables a half (36, 96, 100), code bits that straddle M-tiles, one-byte and 16-bit codes.
# n: a lone vector, either side of a wave's 32 and of a workgroup's 128 vectors (one n-tile per wave, up to 65 536 vectors by segments); the
# next test has the two-tile forms
@pytest.mark.parametrize("d,L,Cb,n", [(32, 20, 5, 1), (33, 4, 1, 63), (47, 12, 7, 65), (63, 28, 8, 255), (96, 24, 6, 257), (100, 96, 3, 300),
                                      (127, 100, 4, 333), (200, 8, 11, 1000), (255, 36, 9, 129), (300, 48, 16, 70), (383, 24, 13, 31),
                                      (384, 128, 8, 140), (200, 16, 5, 140_003)])
def test_i8_any_shape_bit_exact(d, L, Cb, n):
    print("[case]", d, L, Cb, n, flush=True)
    rng = np.random.default_rng(d * 7 + L)
    X, R = i8_inputs(rng, n, d, L * Cb)
    auto, scalar = both("i8", "pm1", X, R, L, Cb)
    assert np.array_equal(auto, scalar)
    if n <= 1000:
        want = orc.hash_i8(X, R, L, Cb)
        assert np.array_equal(auto, want)


# Two n-tiles per wave, from 65 537 vectors (times segments) on: either side of that line, ragged ends of a wave's 64 and a workgroup's 256
# vectors, every step of KS; beyond 131 072 vectors all of R in LDS where it fits 80 KB, a tile at a time where it does not.  All rows
# against the plain kernel, the first and the last workgroups' against the oracle
@pytest.mark.parametrize("d,L,Cb,n", [(64, 12, 7, 65_536), (64, 12, 7, 65_537), (128, 24, 6, 65_600), (200, 20, 5, 65_793), (384, 16, 3, 65_599),
                                      (96, 40, 8, 32_769), (100, 36, 9, 40_003), (47, 12, 7, 140_003), (255, 100, 4, 131_137), (300, 96, 7, 140_001)])
def test_i8_two_tiles_per_wave(d, L, Cb, n):
    print("[case]", d, L, Cb, n, flush=True)
    rng = np.random.default_rng(d + n)
    X, R = i8_inputs(rng, n, d, L * Cb)
    auto, scalar = both("i8", "pm1", X, R, L, Cb)
    assert np.array_equal(auto, scalar)
    for part in (slice(0, 300), slice(n - 300, n)):
        assert np.array_equal(auto[part], orc.hash_i8(X[part], R, L, Cb))


# fp32 sums of exact products: a sign may differ from the 64-bit one only where the projection is within the rounding of the
# sum, at most (d + 2^3) * 2^-24 * sum |r_i x_i| with any order of adding, plus 2^-23 of every |r_i x_i| for the two-part matrix
@pytest.mark.parametrize("xt,pk", [("f16", "gauss"), ("f16", "pm1"), ("i8", "gauss")])
@pytest.mark.parametrize("d,L,Cb,n", [(16, 8, 8, 33), (17, 12, 3, 500), (50, 24, 11, 300), (200, 8, 11, 70_001), (200, 96, 5, 257), (255, 20, 7, 100),
                                      (300, 24, 12, 1000), (384, 4, 16, 65),
                                      # two n-tiles per wave at every step of KS, with ragged ends
                                      (50, 24, 11, 65_537), (100, 8, 7, 65_793), (200, 12, 3, 65_599), (250, 8, 5, 65_600), (384, 4, 6, 65_601),
                                      # beyond 131 072 vectors: all of R in LDS where it fits, a tile at a time where it does not
                                      (200, 8, 11, 140_003), (50, 12, 4, 131_073), (250, 24, 6, 131_137)])
def test_fp_any_shape_signs_within_rounding(xt, pk, d, L, Cb, n):
    print("[case]", xt, pk, d, L, Cb, n, flush=True)
    rng = np.random.default_rng(d + L * Cb)
    if xt == "i8":
        X = rng.integers(-127, 128, (n, d)).astype(np.int8)
    else:
        X = (rng.standard_normal((n, d)) / np.sqrt(d)).astype(np.float16)
    X[0] = 0
    R = (rng.integers(0, 2, (L * Cb, d)) * 2 - 1).astype(np.int8) if pk == "pm1" else rng.standard_normal((L * Cb, d)).astype(np.float32)
    if pk == "gauss":
        R[1] *= 1e-12          # rows far from unit scale, and an all-zero one: the sign does not depend on a row's scale
        R[2] *= 1e12
        R[3] = 0
    auto, _ = both(xt, pk, X, R, L, Cb)
    X64, R64 = X.astype(np.float64), R.astype(np.float64)
    p = X64 @ R64.T
    bound = ((d + 8) * 2.0 ** -24 + 2.0 ** -23) * (np.abs(X64) @ np.abs(R64).T)
    bits = ((auto.astype(np.int64)[:, :, None] >> np.arange(Cb)) & 1).reshape(n, L * Cb)
    diff = bits != (p >= 0)
    assert auto.astype(np.int64).max() < (1 << Cb)
    assert np.all(np.abs(p)[diff] <= bound[diff])
    assert diff.mean() <= 1e-4


def test_fp_any_shape_infinite_and_nan_elements_as_the_plain_kernel():
    """Rows with infinities (their sign decides), opposed infinities and NaN (not >= 0: bit 0), and neighbours that must
    not see them, at a dimension whose last k-step overlaps the one before."""
    rng = np.random.default_rng(5)
    for d in (50, 200):
        X = (rng.standard_normal((300, d)) / np.sqrt(d)).astype(np.float16)
        X[3, 5], X[4, d - 1], X[5, 0] = np.inf, -np.inf, np.nan
        X[8, 1], X[8, d - 2] = np.inf, np.inf
        R = rng.standard_normal((24 * 7, d)).astype(np.float32)
        auto, scalar = both("f16", "gauss", X, R, 24, 7)
        special = [3, 4, 5, 8]
        assert np.array_equal(auto[special], scalar[special])
        assert (auto != scalar).mean() <= 1e-4


def test_any_shape_at_unaligned_vector_addresses():
    """Vectors that start at an odd element: the kernel's loads take any element's address."""
    rng = np.random.default_rng(6)
    d, L, Cb, n = 100, 24, 6, 300
    X, R = i8_inputs(rng, n, d, L * Cb)
    ix = dz.create(d, L, Cb, proj=torch.from_numpy(R).to(DEV))
    room = torch.zeros(n * d + 16, dtype=torch.int8, device=DEV)
    for shift in (1, 2, 7):
        v = room[shift:shift + n * d].view(n, d)
        v.copy_(torch.from_numpy(X).to(DEV))
        assert np.array_equal(dz.hash(ix, v).cpu().numpy(), orc.hash_i8(X, R, L, Cb))


# Rows of which half the entries lie `span` below the largest, and vectors that are zero where a row is large: the sums of the small
# entries alone.  Down to 2^-28 the two parts hold an entry to 2^-23 of itself; matrices that span more are for the plain kernel
@pytest.mark.parametrize("xt", ["f16", "i8"])
@pytest.mark.parametrize("span", [1e-3, 1e-6, 2.0 ** -27, 1e-10, 1e-12, 1e-30])
def test_rows_of_wide_range_keep_their_small_entries(xt, span):
    print("[case]", xt, span, flush=True)
    rng = np.random.default_rng(11)
    d, L, Cb, n = 100, 24, 7, 2000
    X = np.zeros((n, d), np.int8 if xt == "i8" else np.float16)
    X[:, d // 2:] = rng.integers(-127, 128, (n, d - d // 2)) if xt == "i8" else rng.standard_normal((n, d - d // 2))
    R = rng.uniform(1, 2, (L * Cb, d)).astype(np.float32) * rng.choice([-1, 1], (L * Cb, d))
    R[:, d // 2:] *= span
    R = R.astype(np.float32)
    auto, _ = both(xt, "gauss", X, R, L, Cb)
    X64, R64 = X.astype(np.float64), R.astype(np.float64)
    p = X64 @ R64.T
    bound = ((d + 8) * 2.0 ** -24 + 2.0 ** -22) * (np.abs(X64) @ np.abs(R64).T)
    bits = ((auto.astype(np.int64)[:, :, None] >> np.arange(Cb)) & 1).reshape(n, L * Cb)
    diff = bits != (p >= 0)
    assert np.all(np.abs(p)[diff] <= bound[diff])
    assert diff.mean() <= 1e-4


def test_infinite_elements_against_entries_far_below_the_largest():
    """A lone infinite element decides the sign of every bit whose entry is not zero, however small beside its row: powers of
    two, which the two parts hold exactly."""
    rng = np.random.default_rng(12)
    d, L, Cb = 50, 24, 7
    R = (2.0 ** rng.integers(-40, 1, (L * Cb, d)) * rng.choice([-1, 1], (L * Cb, d))).astype(np.float32)
    X = rng.standard_normal((2 * d, d)).astype(np.float16)
    X[np.arange(d), np.arange(d)] = np.inf
    X[d + np.arange(d), np.arange(d)] = -np.inf
    auto, scalar = both("f16", "gauss", X, R, L, Cb)
    want = (np.concatenate([R.T, -R.T]) > 0).astype(np.int64)       # [2 d][L C]
    bits = ((auto.astype(np.int64)[:, :, None] >> np.arange(Cb)) & 1).reshape(2 * d, L * Cb)
    assert np.array_equal(bits, want)
    assert np.array_equal(auto, scalar)
