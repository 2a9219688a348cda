"""The launches of frames above 2^21 pixels, at sizes that the oracle decodes
quickly (a test hook takes them there): the pixels listed by a launch of their
own (aligned and misaligned foreground planes, both dtypes) or not at all
(no foreground channel), the vote and the assignment on that list, for one
block of 32 x 32 bins and for two x blocks per pass, in both searches, with
score map and mask threshold.  Bit-exact against the oracle (Eq5-Eq8)."""
import math

import numpy as np
import pytest

import oracle

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# H, W, bins_w, bins_h, harmonics, dtype, share of the largest vote mass
CASES = [(133, 127, 32, 32, 8, np.float32, 0.0), (133, 127, 23, 9, 16, np.float16, 0.1),
         (133, 127, 33, 31, 4, np.float32, 0.1), (64, 128, 64, 64, 16, np.float16, 0.1),
         (131, 63, 65, 33, 9, np.float32, 0.1), (133, 127, 65, 97, 3, np.float16, 0.0),
         (97, 85, 128, 128, 16, np.float32, 0.1), (1, 1, 40, 33, 5, np.float16, 0.0),
         (279, 271, 40, 72, 6, np.float16, 0.1), (279, 271, 72, 40, 4, np.float32, 0.1)]


@pytest.mark.parametrize("case", CASES, ids=["%dx%d_b%dx%d_F%d_%s" % (*c[:5], np.dtype(c[5]).name) for c in CASES])
def test_separately_listed_pixels(case):
    from paper_2609_16874_amd import native
    H, W, bw, bh, F, dtype, share = case
    rng = np.random.default_rng(H * 131 + bw)
    fx, fy = (2.0 * math.pi * 2.0 ** np.arange(F) / e for e in (W, H))
    cx, cy = rng.uniform(0, W, 12), rng.uniform(0, H, 12)
    inst = rng.integers(0, 12, (H, W))
    px, py = cx[inst][..., None] * fx, cy[inst][..., None] * fy
    emb = np.stack([np.sin(px), np.cos(px), np.sin(py), np.cos(py)], -1)            # [H][W][F][4]
    emb = np.concatenate([emb[..., :2].reshape(H, W, -1), emb[..., 2:].reshape(H, W, -1)], -1)
    emb = (emb + rng.normal(0.0, 0.15, emb.shape)).astype(dtype)
    fg = rng.uniform(0.0, 1.0, (H, W)).astype(dtype)
    fg.reshape(-1)[8192:16384] = 0.0                                                # a slice without a pixel
    fg[0, 0] = 1.0
    cap = ((bw + 1) // 2) * ((bh + 1) // 2)
    e = torch.from_numpy(emb).cuda()
    shifted = torch.empty(H * W + 1, dtype=e.dtype, device="cuda")[1:].view(H, W)   # aligned to its element only
    shifted.copy_(torch.from_numpy(fg))
    dec = native.Decoder(H, W, F, "f16" if dtype == np.float16 else "f32", fx, fy, bw, bh, cap)
    assert dec.test_separate_list(2) == native.CPE_ERR_INVALID_ARG
    assert dec.test_separate_list(True) == 0 and dec.launch_count() == 3
    hist = torch.empty((bh, bw), dtype=torch.int64, device="cuda")
    for plane, planes in ((fg, (torch.from_numpy(fg).cuda(), shifted)), (None, (None,))):
        theta = share * oracle.decode(emb, plane, fx, fy, bw, bh, cap, 0.4, 0.0)["hist"].max() * 2.0 ** -30
        base = oracle.decode(emb, plane, fx, fy, bw, bh, cap, 0.4, theta)
        for t in (math.inf, -math.log(np.median(base["score_map"][base["labels"] > 0]))):
            ref = oracle.decode(emb, plane, fx, fy, bw, bh, cap, 0.4, theta, tau=t)
            for g in planes:
                for mode, score in ((0, True), (0, False), (2, False), (1, False)):
                    print(case, "no plane" if g is None else "plane", t, mode, score, flush=True)
                    assert dec.test_search_mode(mode) == 0
                    got = dec.run(e, g, 0.4, theta, score=score, tau=t)
                    assert dec.histogram(hist) == 0
                    torch.cuda.synchronize()
                    assert np.array_equal(hist.cpu().numpy().view(np.uint64), ref["hist"])
                    assert got["K"] == ref["K"] > 0
                    assert np.array_equal(got["labels"], ref["labels"])
                    assert np.array_equal(got["centroids"], ref["centroids"])
                    if score:
                        np.testing.assert_allclose(got["score_map"], ref["score_map"], rtol=1e-5, atol=0)
    assert dec.test_separate_list(False) == 0
    assert dec.launch_count() == (2 if max(bw, bh) <= 32 else 3)
    dec.close()
