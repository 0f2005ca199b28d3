"""GPU checks at the edges of the launch rules that choose a kernel form.

* Moment and coefficient walks: up to 39 moment channels (one LDS group,
  several workgroups per CU), 40 to 78 (two groups walked by a producer and a
  consumer half), above 78 (split), with narrow and wide prefix segments, on
  strips of 256 columns plus or minus one and frames shorter than a window.
  Tolerance 1e-4 against the oracle, on guides whose windows are well
  conditioned (at most about 20 with eps 0.1): relative to the output (the
  FP32 path's own measure) for the two-pass path; relative to the output or
  its rms for the stages, whose FP32 moment planes (2^-24) enter amplified by
  the condition and by the sum over at most 11 guides of magnitude 3 (4e-5).
* Batched averaging with frames of two- and of four-row tiles in one launch:
  bit for bit the single frames, by both schedules.
* Model interpolation staged in 8, 4, 2, 1 or no rows, and upsampling tiles:
  FP64 up to the output, so 1e-6 (see the bilinear
  models' own tests).
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import paper_2410_11625_amd as flr  # noqa: E402
from oracle import flr_lowres, flr_ref  # noqa: E402
from synth import make_config, random_frame  # noqa: E402

pytestmark = pytest.mark.gpu


def _t(a):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).to("cuda:0")


def _rel(got, want, floor=1e-3):
    rms = max(float(np.sqrt(np.mean(want ** 2))), 1e-30)
    return float(np.max(np.abs(got - want) / np.maximum(np.abs(want), floor * rms)))


def _f32(x):
    return float(np.float32(x))


# (Q, C): 5, 34, 38 | 41, 44, 67, 71, 76 | 80, 89 moment channels
@pytest.mark.parametrize("Q,C", [(1, 1), (4, 4), (5, 3), (6, 2), (5, 4), (7, 4), (8, 3), (10, 1),
                                 (8, 4), (11, 1)])
@pytest.mark.parametrize("H,W,r", [(3, 17, 8), (41, 255, 8), (70, 257, 4), (29, 300, 11)])
def test_walk_forms(Q, C, H, W, r):
    fr = random_frame(H, W, Q, C, seed=Q * 100 + C, offset=1.0)
    y, g = fr["noisy"], fr["guides"]
    want = flr_ref.flr_reference(y, g, r, _f32(1e-1))
    for path, floor in (("two_pass", 1e-3), ("stages", 1.0)):
        got = flr.denoise(_t(y), _t(g), r, eps=1e-1, fused=path).cpu().numpy()
        assert _rel(got, want, floor) <= 1e-4, path


@pytest.mark.parametrize("blocks", [0, 5])
def test_batch_mixed_averaging_tiles(blocks):
    frames = []
    for k, (h, w) in enumerate([(33, 256), (820, 230), (1, 241), (64, 90)]):
        fr = make_config(1, seed=30 + k, h=h, w=w)
        frames.append(dict(guides=_t(fr["guides"]), noisy=_t(fr["noisy"])))
    b = flr.Batch(frames, persistent_blocks=blocks)
    outs = b.run()
    torch.cuda.synchronize()
    for f, out in zip(frames, outs):
        assert torch.equal(out, flr.denoise(f["noisy"], f["guides"], fused="two_pass"))


@pytest.mark.parametrize("Q,C,block", [(1, 1, 16), (6, 2, 4), (8, 3, 4), (4, 2, 1), (12, 2, 2),
                                       (12, 4, 1)])
def test_interpolation_rows(Q, C, block):
    fr = random_frame(53, 259, Q, C, seed=Q + C, smooth=1.5, offset=1.0)
    y, g = fr["noisy"], fr["guides"]
    got = flr.denoise_lowres(_t(y), _t(g), block=block).cpu().numpy()
    want = flr_lowres.lowres_reference(y, g, block, _f32(1.25), 4, _f32(1e-3))
    assert _rel(got, want) <= 1e-6


@pytest.mark.parametrize("Q,C", [(8, 3), (7, 4)])
@pytest.mark.parametrize("up,H,W", [(2, 62, 258), (4, 44, 516), (8, 24, 264)])
def test_upsampling_rows(Q, C, up, H, W):
    hi = random_frame(H, W, Q, C, seed=7, smooth=6.0, offset=1.0)["guides"]
    lo = random_frame(H // up, W // up, Q, C, seed=8, offset=1.0)
    b = flr.Batch([dict(guides=_t(hi), guides_low=_t(lo["guides"]), noisy=_t(lo["noisy"]))],
                  eps=1e-1)
    out = b.run()[0].cpu().numpy()
    _, A = flr_ref.flr_reference(lo["noisy"], lo["guides"], 8, _f32(1e-1), return_coeffs=True)
    A = flr_lowres.bilinear_upsample(flr_ref.average_coefficients(A, 8), H, W, up)
    assert _rel(out, flr_ref.apply_model(A, hi)) <= 1e-6
