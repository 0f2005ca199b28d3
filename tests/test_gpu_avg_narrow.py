"""GPU check of the averaging of images narrower than four columns, at the
tile heights that tall ones take: flr_apply against a 64-bit evaluation, and
batches that mix them with wide frames against flr_denoise, bit for bit.

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


@pytest.mark.parametrize("W", [1, 2, 3, 4])
@pytest.mark.parametrize("H,C,r", [(2407, 1, 8), (803, 3, 3), (1203, 2, 20)])
@pytest.mark.parametrize("pair", [False, True])
def test_tall_narrow(H, W, C, r, pair):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    dev = torch.device("cuda:0")
    rng = np.random.default_rng(H + W + r)
    Q, F = 2, 4 if pair else 3
    co = rng.standard_normal((F, C, H, W)).astype(np.float32)
    g = rng.standard_normal((Q, H, W)).astype(np.float32)
    gt, ct = torch.from_numpy(g).to(dev), torch.from_numpy(co.reshape(F * C, H, W)).to(dev)
    n = _box(np.ones((H, W)), r)
    w = np.concatenate([np.ones((1, H, W)), g.astype(np.float64)] +
                       ([np.ones((1, H, W))] if pair else []))
    want = (w[:, None] * _box(co.astype(np.float64), r)).sum(0) / n
    mag = np.abs(co).sum() * np.abs(w).max() / n
    for rows in (0, 2, 4):
        out = flr.apply(gt, ct, r, tile_rows=rows, intercept_pair=pair).cpu().numpy()
        bad = np.abs(out - want) > 2.0 ** -24 * np.abs(want) + 1e-12 * mag
        assert not bad.any(), (rows, np.argwhere(bad)[:4], np.abs(out - want).max())


@pytest.mark.parametrize("sizes", [[(2500, 3)], [(2500, 3), (300, 700), (11, 2)],
                                   [(40, 50), (2500, 1)]])
@pytest.mark.parametrize("blocks", [0, None])
def test_batches_with_narrow_frames(sizes, blocks):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    dev = torch.device("cuda:0")
    frames = []
    for k, (h, w) in enumerate(sizes):
        fr = make_config(1, seed=20 + k, h=h, w=w)
        frames.append(dict(guides=torch.from_numpy(fr["guides"][:3].astype(np.float32)).to(dev),
                           noisy=torch.from_numpy(fr["noisy"].astype(np.float32)).to(dev)))
    b = flr.Batch(frames, radius=8, persistent_blocks=blocks)
    for _ in range(2):
        outs = [o.clone() for o in b.run()]
    assert not b.failed()
    for f, o in zip(frames, outs):
        assert torch.equal(o, flr.denoise(f["noisy"], f["guides"], radius=8, fused="two_pass"))
