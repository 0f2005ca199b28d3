"""GPU check of flr_net_backward's wide data-gradient tiles (64 pixels, at
stride 2 32) at their edges: FLR_DGRAD_WIDE_PX=0 gives them to every grid. Against
the oracle's backward on the device's own activations, and bit for bit against
the narrow tiles; frames that reach them by themselves, too.

Tolerance as for the narrow tiles: FP32 sums over a frame, 1e-4 of a layer's
largest gradient.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import paper_2410_11625_amd as flr  # noqa: E402
from oracle import net_adjoint  # noqa: E402
from paper_2410_11625_amd.api import net_forward_trace  # noqa: E402
from synth import make_config  # noqa: E402
from synth.net_weights import LAYERS, flatten_net_weights, make_net_weights  # noqa: E402
from tests.test_gpu_net_backward_tiles import TOL, _device_cache  # noqa: E402

pytestmark = pytest.mark.gpu


def _frame(H, W):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    dev = torch.device("cuda:0")
    weights = make_net_weights(2)
    p = torch.from_numpy(flatten_net_weights(weights).astype(np.float32)).to(dev)
    fr = make_config(1, seed=8, h=H, w=W)
    g = torch.from_numpy(fr["guides"].astype(np.float32)).to(dev)
    y = torch.from_numpy(fr["noisy"].astype(np.float32)).to(dev)
    G = np.random.default_rng(H * W + 1).standard_normal((4, H, W)).astype(np.float32)
    return weights, p, flr.net_pack(p), g, y, G


@pytest.mark.parametrize("H,W", [(2, 1), (4, 64), (5, 65), (9, 129), (66, 127), (130, 66)])
def test_wide_tiles_match_oracle_and_narrow(H, W, monkeypatch):
    weights, p, packed, g, y, G = _frame(H, W)
    Gd = torch.from_numpy(G).to(g.device)
    monkeypatch.setenv("FLR_DGRAD_WIDE_PX", "0")
    got = flr.net_backward(g, y, p, packed, Gd)
    monkeypatch.setenv("FLR_DGRAD_WIDE_PX", str(1 << 40))
    assert torch.equal(got, flr.net_backward(g, y, p, packed, Gd))
    got = got.cpu().numpy()
    out, acts = net_forward_trace(g, y, packed)
    want = net_adjoint.net_backward(_device_cache(acts, out, weights), G.astype(np.float64))
    o = 0
    for name, _, _, _ in LAYERS:
        for ref in want[name]:
            n = ref.size
            e = np.abs(got[o:o + n].astype(np.float64).reshape(ref.shape) - ref).max()
            assert e <= TOL * max(np.abs(ref).max(), 1e-30), (name, e, np.abs(ref).max())
            o += n
    assert o == got.size


# 257 x 321: wide at stride 1; 413 x 523: every layer but the coarsest
@pytest.mark.parametrize("H,W", [(257, 321), (413, 523)])
def test_widths_by_grid_equal_narrow(H, W, monkeypatch):
    weights, p, packed, g, y, G = _frame(H, W)
    Gd = torch.from_numpy(G).to(g.device)
    monkeypatch.delenv("FLR_DGRAD_WIDE_PX", raising=False)
    got = flr.net_backward(g, y, p, packed, Gd)
    monkeypatch.setenv("FLR_DGRAD_WIDE_PX", str(1 << 40))
    narrow = flr.net_backward(g, y, p, packed, Gd)
    assert torch.isfinite(got).all() and torch.equal(got, narrow)
