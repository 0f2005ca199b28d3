"""GPU check of flr_net_backward's rounding error against 64 bits, under loss
gradients of random signs: a frame's gradients cancel, so an error that leans
one way shows, as does one that grows with the length of a chain of sums.

The reference differentiates the network at the activations that the device
stored (flr_net_forward_trace), in torch float64 on the device, as sums over
taps of plain matrix products. Errors are root mean squares over a layer's
weights (or biases), relative to that of the layer's gradient, in units of
2^-24 (half a unit in the last place of an FP32 number just below two).

A sum of K products of random signs rounds K times at the size it has grown
to: sqrt(K / 2) / sqrt(3) units. The ten data gradients' K add up to about
2700 (21 units), a weight gradient's chain of 128 products and its later
levels to about 6; twice their sum bounds what uncorrelated rounding gives.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import paper_2410_11625_amd as flr  # noqa: E402
from paper_2410_11625_amd.api import net_forward_trace  # noqa: E402
from synth import make_config  # noqa: E402
from synth.net_weights import LAYERS, flatten_net_weights, make_net_weights  # noqa: E402

pytestmark = pytest.mark.gpu

UNIT = 2.0 ** -24
TOL = 2 * (21 + 6)
D = torch.float64


def _grads(x, w, dz, s, need_dx=True):
    """Gradients of a layer's weights, biases and input."""
    k = w.shape[2]
    c, H, W = x.shape
    o, Ho, Wo = dz.shape
    p = k // 2
    xp = torch.zeros((c, H + 2 * p + s, W + 2 * p + s), dtype=D, device=x.device)
    xp[:, p:p + H, p:p + W] = x
    dxp = torch.zeros_like(xp) if need_dx else None
    z = dz.reshape(o, -1).contiguous()
    dW = torch.empty((o, c, k, k), dtype=D, device=x.device)
    for u in range(k):
        for v in range(k):
            xs = xp[:, u:u + s * Ho:s, v:v + s * Wo:s].reshape(c, -1)
            dW[:, :, u, v] = torch.mm(z, xs.t().contiguous())
            if need_dx:
                dxp[:, u:u + s * Ho:s, v:v + s * Wo:s] += \
                    torch.mm(w[:, :, u, v].t().contiguous(), z).reshape(c, Ho, Wo)
    return dW, dz.sum((1, 2)), dxp[:, p:p + H, p:p + W] if need_dx else None


def _up(x, like):
    return x.repeat_interleave(2, 1).repeat_interleave(2, 2)[:, :like.shape[1], :like.shape[2]]


def _down(g):
    c, H, W = g.shape
    q = torch.zeros((c, (H + 1) // 2 * 2, (W + 1) // 2 * 2), dtype=D, device=g.device)
    q[:, :H, :W] = g
    return q.reshape(c, q.shape[1] // 2, 2, q.shape[2] // 2, 2).sum((2, 4))


def _reference(acts, out, weights, G, layers=12):
    """{layer: (dW, db)} of the last `layers` layers (2: the head and out3)."""
    dev = G.device
    a = {k: (t.to(torch.int32) << 16).view(torch.float32).to(D).permute(2, 0, 1).contiguous()
         for k, t in acts.items()}
    w = {n: torch.from_numpy(v[0].astype(np.float32)).to(dev).bfloat16().to(D)
         for n, v in weights.items()}
    s = out.to(D)
    r = {}

    def layer(name, x, g, stride=1, need_dx=True):
        r[name] = _grads(x, w[name], g, stride, need_dx)
        return r[name][2]

    def relu(g, act):
        return torch.where(a[act] > 0, g, torch.zeros_like(g))
    g = relu(layer("out1", a["out3"], G.to(D) * s * (1 - s)), "out3")
    g = layer("out3", a["d0b"], g)
    if layers > 2:
        e0, e1, e2, d1 = a["in1"], a["e1b"], a["e2b"], a["d1b"]
        g = relu(layer("d0b", a["d0a"], relu(g, "d0b")), "d0a")
        g = layer("d0a", torch.cat([_up(d1, e0), e0]), g)
        ge0 = g[32:]
        g = relu(layer("d1b", a["d1a"], relu(_down(g[:32]), "d1b")), "d1a")
        g = layer("d1a", torch.cat([_up(e2, e1), e1]), g)
        ge1 = g[64:]
        g = relu(layer("e2b", a["e2a"], relu(_down(g[:64]), "e2b"), 2), "e2a")
        g = relu(layer("e2a", e1, g) + ge1, "e1b")
        g = relu(layer("e1b", a["e1a"], g, 2), "e1a")
        g = relu(layer("e1a", e0, g) + ge0, "in1")
        g = relu(layer("in1", a["in3"], g), "in3")
        layer("in3", a["x0"][:11], g, 1, False)
    return r


def _errors(H, W, layers):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    dev = torch.device("cuda:0")
    weights = make_net_weights(2)
    p = torch.from_numpy(flatten_net_weights(weights).astype(np.float32)).to(dev)
    packed = flr.net_pack(p)
    fr = make_config(1, seed=6, h=H, w=W)
    g = torch.from_numpy(fr["guides"].astype(np.float32)).to(dev)
    y = torch.from_numpy(fr["noisy"].astype(np.float32)).to(dev)
    G = np.random.default_rng(H + W).standard_normal((4, H, W)).astype(np.float32) / (H * W)
    G = torch.from_numpy(G).to(dev)
    got = flr.net_backward(g, y, p, packed, G).to(D)
    out, acts = net_forward_trace(g, y, packed)
    want = _reference(acts, out, weights, G, layers)
    errs, o = {}, 0
    for name, _, _, _ in LAYERS:
        for tag, v in zip("wb", weights[name]):
            n = v.size
            if name in want:
                ref = want[name]["wb".index(tag)].reshape(-1)
                e = got[o:o + n] - ref
                errs[name + "." + tag] = float(e.square().mean().sqrt() /
                                               ref.square().mean().sqrt()) / UNIT
            o += n
    assert o == got.numel()
    return errs


@pytest.mark.parametrize("H,W", [(256, 256), (257, 321)])
def test_net_backward_rounding_does_not_lean(H, W):
    errs = _errors(H, W, 12)
    assert len(errs) == 24 and max(errs.values()) <= TOL, errs


def test_weight_gradient_chains_stay_short():
    """Sums over a large frame: the last two layers, whose dz carries next to
    no error of its own. One chain of a chunk's 3264 products would give 23
    units, chains of 128 give 5 and their second level of 26 sums 2; twice
    that."""
    errs = _errors(1080, 1920, 2)
    assert len(errs) == 4 and max(errs.values()) <= 14, errs
