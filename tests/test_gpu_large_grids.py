"""The assignment of bin grids above 32 x 32 and its plan (Eq5-Eq8, Section
3.2), bit-exact against the oracle at the edges of the plan: one more bin than
a block of 32 or a mask word of 64, single rows and columns, the largest grid,
noise frames whose thousands of candidates leave the LDS one or two waves and
count past the privatised ones, capacities that cut a row's candidates, no
candidate, with and without foreground, score map and mask threshold, in both
searches."""
import math

import numpy as np
import pytest

import oracle

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# bins_w, bins_h, harmonics, dtype, theta, capacity (None: every candidate)
CASES = [(33, 1, 4, np.float32, 0.0, None), (1, 40, 3, np.float16, 0.0, None), (33, 33, 8, np.float16, 0.0, 37),
         (64, 48, 16, np.float16, 0.0, None), (65, 34, 6, np.float32, 0.0, None), (128, 128, 8, np.float16, 0.0, None),
         (128, 128, 16, np.float32, 0.0, 1500), (97, 128, 9, np.float16, 0.0, 1), (40, 40, 4, np.float32, 1e9, None)]


@pytest.mark.parametrize("case", CASES, ids=["%dx%d_F%d_%s_t%g_cap%s" % (c[0], c[1], c[2], np.dtype(c[3]).name, c[4], c[5])
                                             for c in CASES])
def test_large_grid_assignment(case):
    from paper_2609_16874_amd import native
    bw, bh, F, dtype, theta, cap = case
    H, W = 47, 61
    rng = np.random.default_rng(bw * 131 + bh)
    fx, fy = (2.0 * math.pi * 2.0 ** np.arange(F) / e for e in (W, H))
    emb = rng.normal(0.0, 0.7, (H, W, 4 * F)).astype(dtype)
    fg = rng.uniform(0.0, 1.0, (H, W)).astype(dtype)
    cap = cap or ((bw + 1) // 2) * ((bh + 1) // 2)
    name = "f16" if dtype == np.float16 else "f32"
    e, g = torch.from_numpy(emb).cuda(), torch.from_numpy(fg).cuda()
    dec = native.Decoder(H, W, F, name, fx, fy, bw, bh, cap)
    hist = torch.empty((bh, bw), dtype=torch.int64, device="cuda")
    for plane, thr, tau in ((g, 0.4, math.inf), (None, 0.0, math.inf), (g, 0.4, 1.9 * math.sqrt(F))):
        ref = oracle.decode(emb, fg if plane is not None else None, fx, fy, bw, bh, cap, thr, theta, tau=tau)
        for mode, score in ((0, True), (0, False), (2, False), (1, False)):
            assert dec.test_search_mode(mode) == 0
            got = dec.run(e, plane, thr, theta, score=score, tau=tau)
            assert dec.histogram(hist) == 0
            torch.cuda.synchronize()
            assert np.array_equal(hist.cpu().numpy().view(np.uint64), ref["hist"])
            assert got["K"] == ref["K"]
            assert np.array_equal(got["labels"], ref["labels"]), (mode, score)
            assert np.array_equal(got["centroids"], ref["centroids"]), (mode, score)
            if score:
                np.testing.assert_allclose(got["score_map"], ref["score_map"], rtol=1e-5, atol=0)
    dec.close()
