"""GPU check of flr_denoise's fused path in both forms: two kernels where the
workspace holds the coefficient image (what flr_denoise_workspace_bytes asks
for), one kernel with its ring where it holds only that.

With the image the outputs are the two-pass path's bit for bit; the one-kernel
form computes the same in 64 bits from coefficients stored relative to a
workgroup's anchor, so both lie within the FP32 path's 1e-4 of each other.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import paper_2410_11625_amd as flr  # noqa: E402
from paper_2410_11625_amd.api import make_params, workspace_bytes  # noqa: E402
from synth import make_config  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,W,Q,C,r,mode", [(5, 7, 2, 1, 2, "ridge"), (40, 70, 4, 1, 8, "paper"),
                                            (61, 259, 5, 3, 3, "ridge"),
                                            (33, 90, 12, 3, 8, "ridge"),
                                            (700, 900, 3, 1, 3, "ridge")])
def test_fused_forms(H, W, Q, C, r, mode):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    dev = torch.device("cuda:0")
    fr = make_config(1, h=H, w=W)
    g8 = fr["guides"][:min(Q, 8)]
    guides = np.concatenate([g8, 0.5 * g8[:Q - len(g8)] ** 2]).astype(np.float32)
    g = torch.from_numpy(np.ascontiguousarray(guides)).to(dev)
    y = torch.from_numpy(np.ascontiguousarray(fr["noisy"][:C], dtype=np.float32)).to(dev)
    kw = dict(radius=r, eps=1e-2, mode=mode, eps_mul=0.05 if mode == "paper" else 0.0)
    two = flr.denoise(y, g, fused="two_pass", **kw)
    assert torch.equal(flr.denoise(y, g, fused="fused", **kw), two)
    need = workspace_bytes(make_params(H, W, Q, C, r, fused="fused"))
    small = torch.empty(need - 1, dtype=torch.uint8, device=dev)
    if (H, W) == (700, 900):  # the ring is smaller than the image here
        one = flr.denoise(y, g, fused="fused", workspace=small, **kw)
        rms = two.square().mean().sqrt()
        rel = ((one - two).abs() / torch.maximum(two.abs(), 1e-3 * rms)).max()
        assert rel <= 2e-4, float(rel)
    else:
        with pytest.raises(flr.FLRError):
            flr.denoise(y, g, fused="fused", workspace=small, **kw)
