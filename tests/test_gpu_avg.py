"""GPU check of the coefficient average and reconstruction (flr_apply with
averaging) against a 64-bit evaluation of its definition: odd widths (lanes of
four columns cut by the image's right end, images narrower than four columns),
strips of one column more or less than a whole one, single rows, every radius
form (r < 8, r = 8, 8 < r <= 32) and every tile height.

Tolerance: window sums, products and the mean are 64-bit on FP32 inputs, so
an output differs from the exact one by its rounding to FP32 (2^-24 relative)
and by 64-bit rounding of the summed magnitudes (below 1e-12 of their sum).
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import paper_2410_11625_amd as flr  # noqa: E402

pytestmark = pytest.mark.gpu


def _box(x, r):
    """Clipped window sums of the last two axes."""
    for ax in (-2, -1):
        n = x.shape[ax]
        c = np.concatenate([np.zeros_like(x.take([0], ax)), np.cumsum(x, ax)], ax)
        i = np.arange(n)
        x = c.take(np.minimum(i + r, n - 1) + 1, ax) - c.take(np.maximum(i - r, 0), ax)
    return x


@pytest.mark.parametrize("H,W,Q,C,r", [
    (1, 1, 1, 1, 8), (3, 3, 2, 3, 8), (5, 2, 1, 2, 3), (2, 5, 3, 1, 1), (7, 239, 2, 3, 8),
    (9, 240, 2, 1, 8), (18, 241, 3, 2, 8), (33, 257, 1, 3, 8), (35, 515, 2, 3, 8),
    (6, 245, 2, 3, 5), (37, 506, 2, 1, 3), (21, 300, 1, 1, 0), (5, 233, 2, 2, 9),
    (70, 461, 1, 3, 16), (66, 390, 2, 1, 32), (40, 1030, 4, 4, 8),
])
@pytest.mark.parametrize("rows", [0, 1, 3, 8])
@pytest.mark.parametrize("pair", [False, True])
def test_apply_average(H, W, Q, C, r, rows, pair):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    rng = np.random.default_rng(H * 1000 + W + Q + C + r)
    F = Q + 2 if pair else Q + 1
    co = rng.standard_normal((F, C, H, W)).astype(np.float32)
    co[:, :, rng.integers(0, H), rng.integers(0, W)] *= 1e3
    g = rng.standard_normal((Q, H, W)).astype(np.float32)
    dev = torch.device("cuda:0")
    out = flr.apply(torch.from_numpy(g).to(dev), torch.from_numpy(co.reshape(F * C, H, W)).to(dev),
                    r, tile_rows=rows, intercept_pair=pair).cpu().numpy()
    n = _box(np.ones((H, W)), r)
    w = np.concatenate([np.ones((1, H, W)), g.astype(np.float64)] +
                       ([np.ones((1, H, W))] if pair else []))
    want = (w[:, None] * _box(co.astype(np.float64), r)).sum(0) / n
    mag = (np.abs(w)[:, None] * _box(np.abs(co).astype(np.float64), r)).sum(0) / n
    # cumulative sums of the whole row here: their rounding is bounded by the
    # whole frame's magnitude
    tol = 2.0 ** -24 * np.abs(want) + 1e-12 * (mag + np.abs(co).sum() * np.abs(w).max() / n)
    bad = np.abs(out - want) > tol
    assert not bad.any(), (np.argwhere(bad)[:4], np.abs(out - want).max())
