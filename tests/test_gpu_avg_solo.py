"""GPU check of the averaging with one tile per wavefront (many tiles of few
planes): flr_apply against a 64-bit evaluation in each radius form, with and
without tiles inside the image, last workgroups filled in part, images narrower
than four columns; and batches against flr_denoise, bit for bit.

Tolerance: window sums, products and the mean are 64-bit on FP32 inputs, so
an output differs from the exact one by its rounding to FP32 and by 64-bit
rounding of the summed magnitudes.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import paper_2410_11625_amd as flr  # noqa: E402
from synth import make_config  # noqa: E402
from tests.test_gpu_avg import _box  # noqa: E402

pytestmark = pytest.mark.gpu


# tiles of four rows x strips x channels: at or past the line, 2 to 6 planes
@pytest.mark.parametrize("H,W,Q,C,r,pair", [
    (2731, 37, 1, 3, 8, False), (2731, 37, 1, 3, 8, True), (1399, 600, 1, 2, 8, False),
    (2733, 241, 2, 2, 8, False), (6150, 20, 4, 4, 8, False), (6150, 9, 4, 4, 8, True),
    (4109, 3, 2, 2, 8, False), (3075, 10, 1, 4, 3, False), (4101, 260, 1, 3, 20, False),
    (6201, 2, 1, 2, 12, False)])
def test_tile_per_wavefront(H, W, Q, C, r, pair):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    dev = torch.device("cuda:0")
    rng = np.random.default_rng(H + W + Q + C + r)
    F = Q + 2 if pair else Q + 1
    co = rng.standard_normal((F, C, H, W)).astype(np.float32)
    g = rng.standard_normal((Q, H, W)).astype(np.float32)
    out = flr.apply(torch.from_numpy(g).to(dev), torch.from_numpy(co.reshape(F * C, H, W)).to(dev),
                    r, intercept_pair=pair).cpu().numpy()
    n = _box(np.ones((H, W)), r)
    w = np.concatenate([np.ones((1, H, W)), g.astype(np.float64)] +
                       ([np.ones((1, H, W))] if pair else []))
    want = (w[:, None] * _box(co.astype(np.float64), r)).sum(0) / n
    # the reference's cumulative sums round with the whole frame's magnitude
    tol = 2.0 ** -24 * np.abs(want) + 1e-12 * np.abs(co).sum() * np.abs(w).max() / n
    bad = np.abs(out - want) > tol
    assert not bad.any(), (np.argwhere(bad)[:4], np.abs(out - want).max())


@pytest.mark.parametrize("Q,sizes", [(1, [(2731, 50), (70, 80)]), (4, [(8197, 12), (64, 300)])])
@pytest.mark.parametrize("blocks", [0, None])
def test_batch_equals_denoise(Q, sizes, blocks):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    dev = torch.device("cuda:0")
    frames = []
    for k, (h, w) in enumerate(sizes):
        fr = make_config(1, seed=30 + k, h=h, w=w)
        frames.append(dict(guides=torch.from_numpy(fr["guides"][:Q].astype(np.float32)).to(dev),
                           noisy=torch.from_numpy(fr["noisy"].astype(np.float32)).to(dev)))
    b = flr.Batch(frames, radius=8, persistent_blocks=blocks)
    for _ in range(2):
        outs = [o.clone() for o in b.run()]
    assert not b.failed()
    for f, o in zip(frames, outs):
        assert torch.equal(o, flr.denoise(f["noisy"], f["guides"], radius=8, fused="two_pass"))
