"""The binary16 split of the matrix-core distances (Eq4/Eq10).

The kernels compute S = |X|^2 + |P|^2 - 2 X.P as kBase A + R with the palette
split -2P = kBase hi + lo, in binary32 matrix products that are exact as long
as every partial sum stays below 2^24.  The CPU test bounds those sums for the
base that the sources use; the GPU test drives them: every harmonic count
with its own operand layout, both dtypes, channels at the clamp bounds, far
beyond them, on rounding ties of the 1/4096 grid, subnormal, infinite and NaN,
bit-exact against the oracle.
"""
import math
import os
import re

import numpy as np
import pytest

import oracle

_CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2609_16874_amd", "csrc")
X_MAX, P_MAX, CHANNELS = 6144, 4096, 32      # |X|, |P| per channel, channels per axis at 16 harmonics


def _base():
    with open(os.path.join(_CSRC, "cpe_common.hpp")) as fh:
        m = re.search(r"constexpr int kDistBase = (\d+);", fh.read())
    assert m, "kDistBase not found in cpe_common.hpp"
    return int(m.group(1))


def test_every_partial_sum_is_exact():
    base = _base()
    f1, f2 = divmod(2 ** 10, base), divmod(2 ** 20, base)
    for v in (*f1, *f2, 1024 + 1023, 576):
        assert float(np.float16(v)) == v              # coefficients and fields are binary16 numbers
    n_half = CHANNELS // 2 * X_MAX ** 2               # one lane half's part of |X|^2
    assert n_half >> 20 <= 576
    fields = (2047, 2047, n_half >> 20)               # offset 1024 included in the low two
    offset = 2 * 1024
    lo = base // 2
    # R: the lo products term by term, then the norms of both halves and the constant
    r = CHANNELS * X_MAX * lo + 2 * (fields[0] + fields[1] * f1[1] + fields[2] * f2[1]) + base + offset * (1 + f1[1])
    # A: the hi products by Cauchy-Schwarz (|hi| <= (|2P| + |lo|) / base), the norms
    x = math.sqrt(CHANNELS) * X_MAX
    p = P_MAX * math.sqrt(CHANNELS / 2) + 0.5 * math.sqrt(CHANNELS)
    a = x * (2 * p + lo * math.sqrt(CHANNELS)) / base + 2 * (fields[1] * f1[0] + fields[2] * f2[0])
    a += p * p / base + offset * f1[0]
    assert r < 2 ** 24 and a < 2 ** 24, (r, a)


def test_search_keys_keep_the_fast_gap():
    """The assignment search compares sums whose low kStepBits are replaced
    by a step number: a pixel that its test decides has batch sums at least
    kFastGap binary32 steps apart, and the winner's key is the smaller sum."""
    with open(os.path.join(_CSRC, "k_mfma.hpp")) as fh:
        src = fh.read()
    gap, bits = (int(re.search(rf"constexpr int {n} = (\d+);", src).group(1)) for n in ("kFastGap", "kStepBits"))
    need = (gap + 2 * ((1 << bits) - 1)) >> bits
    rng = np.random.default_rng(5)
    s = rng.integers(0x3c000000, 0x44000000, 400000)
    t = s + rng.integers(-64, 65, s.size)
    key = lambda v: (v >> bits << bits) | rng.integers(0, 1 << bits, v.size)
    ks, kt = key(s), key(t)
    lo, hi = np.minimum(ks, kt), np.maximum(ks, kt)
    decided = (hi >> bits) - (lo >> bits) >= need
    assert 0.2 < decided.mean() < 0.9
    assert ((t - s)[decided & (ks < kt)] >= gap).all()
    assert ((s - t)[decided & (kt < ks)] >= gap).all()


def _values(rng, dtype, shape):
    """Channels that reach every branch of the input conversion."""
    n = int(np.prod(shape))
    ties = (rng.integers(-6200, 6201, n) + 0.5) / 4096.0
    unit = rng.uniform(-1.0, 1.0, n)
    edge = rng.choice([1.5, -1.5, 1.4998, -1.4998, 1.5007, 0.25, -0.25, 0.12497, 40.0, -60000.0], n)
    odd = rng.choice([np.inf, -np.inf, np.nan, 0.0, -0.0, 6e-8, -3e-5, 1.3e-4], n)
    v = np.where(rng.random(n) < 0.4, ties, unit)
    v = np.where(rng.random(n) < 0.2, edge, v)
    v = np.where(rng.random(n) < 0.02, odd, v)
    return v.astype(dtype).reshape(shape)


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [np.float16, np.float32])
@pytest.mark.parametrize("n_freq", [1, 3, 4, 6, 8, 9, 12, 15, 16])
def test_distances_of_extreme_inputs(n_freq, dtype):
    torch = pytest.importorskip("torch")
    from paper_2609_16874_amd import native
    H, W, bw, bh = 45, 53, 32, 27
    rng = np.random.default_rng(100 * n_freq + np.dtype(dtype).itemsize)
    fx, fy = (2.0 * math.pi * 2.0 ** np.arange(n_freq) / e for e in (W, H))
    emb = _values(rng, dtype, (H, W, 4 * n_freq))
    # a row of pixels on the palette itself (S near 0), one at the clamp
    # bounds against it (the largest S) and one along it
    ref = oracle.decode(emb[:1, :1].copy(), None, fx, fy, bw, bh)
    pal = np.concatenate([ref["pal_x"][rng.integers(0, bw, W)], ref["pal_y"][rng.integers(0, bh, W)]], axis=1)
    emb[0] = (pal / 4096.0).astype(dtype)
    emb[1] = np.where(pal < 0, 1.5, -1.5).astype(dtype)
    emb[2] = np.where(pal < 0, -1.5, 1.5).astype(dtype)
    fg = rng.uniform(0.0, 1.0, (H, W)).astype(dtype)
    fg[:3] = 1.0
    cap = ((bw + 1) // 2) * ((bh + 1) // 2)
    name = "f16" if dtype == np.float16 else "f32"
    e, g = torch.from_numpy(emb).cuda(), torch.from_numpy(fg).cuda()
    for plane, thr in ((g, 0.5), (None, 0.0)):
        ref = oracle.decode(emb, fg if plane is not None else None, fx, fy, bw, bh, cap, thr, 0.0)
        dec = native.Decoder(H, W, n_freq, name, fx, fy, bw, bh, cap)
        hist = torch.empty((bh, bw), dtype=torch.int64, device="cuda")
        for mode, score in ((0, True), (0, False), (2, False)):     # exact search, default, fast search
            assert dec.test_search_mode(mode) == 0
            got = dec.run(e, plane, thr, 0.0, score=score, tau=math.inf)
            assert dec.histogram(hist) == 0
            torch.cuda.synchronize()
            assert np.array_equal(hist.cpu().numpy().view(np.uint64), ref["hist"])
            assert got["K"] == ref["K"]
            assert np.array_equal(got["labels"], ref["labels"])
            assert np.array_equal(got["centroids"], ref["centroids"])
            if score:
                np.testing.assert_allclose(got["score_map"], ref["score_map"], rtol=1e-5, atol=0)
        dec.close()
