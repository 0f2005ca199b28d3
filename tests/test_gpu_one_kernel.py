"""GPU check of the fused path's one-kernel form, run by a workspace of
min_workspace_bytes: against the oracle, and at full size against the two-pass
path (both within the FP32 path's 1e-4 of the exact output)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import paper_2410_11625_amd as flr  # noqa: E402
from oracle import flr_ref  # noqa: E402
from paper_2410_11625_amd import api  # noqa: E402
from synth import make_config  # noqa: E402

pytestmark = pytest.mark.gpu


def _frame(H, W, Q, C):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    fr = make_config(1, h=H, w=W)
    g8 = fr["guides"][:min(Q, 8)]
    guides = np.concatenate([g8, 0.5 * g8[:Q - len(g8)] ** 2]).astype(np.float32)
    noisy = fr["noisy"][:C].astype(np.float32)
    dev = torch.device("cuda:0")
    return guides, noisy, torch.from_numpy(np.ascontiguousarray(guides)).to(dev), \
        torch.from_numpy(np.ascontiguousarray(noisy)).to(dev)


def _one_kernel(y, g, r, rows=0, **kw):
    Q, H, W = g.shape
    p = flr.make_params(H, W, Q, y.shape[0], r, tile_rows=rows, fused="fused", **kw)
    least = flr.min_workspace_bytes(p)
    image = flr.workspace_bytes(flr.make_params(H, W, Q, y.shape[0], r, fused="two_pass"))
    assert least < image  # the one kernel runs
    ws = torch.empty(least, dtype=torch.uint8, device=g.device)
    return flr.denoise(y, g, r, fused="fused", workspace=ws, tile_rows=rows, **kw)


def _rel(got, want):
    rms = max(np.sqrt(np.mean(np.square(want, dtype=np.float64))), 1e-30)  # an all-zero frame
    return float((np.abs(got - want) / np.maximum(np.abs(want), 1e-3 * rms)).max())


@pytest.mark.parametrize("H,W,Q,C,r,rows,mode", [
    (61, 300, 8, 3, 8, 31, "ridge"), (70, 227, 8, 3, 8, 70, "paper"),
    (113, 250, 4, 1, 16, 113, "paper"), (97, 200, 8, 3, 12, 97, "ridge"),
    (140, 120, 2, 1, 32, 140, "ridge"), (33, 90, 3, 2, 0, 11, "ridge"),
    (50, 500, 12, 3, 2, 25, "paper")])          # vertical sums outside LDS
def test_one_kernel_matches_oracle(H, W, Q, C, r, rows, mode):
    guides, noisy, g, y = _frame(H, W, Q, C)
    em = 0.05 if mode == "paper" else 0.0
    got = _one_kernel(y, g, r, rows, eps=1e-3, mode=mode, eps_mul=em).cpu().numpy()
    want = flr_ref.flr_reference(noisy, guides, r, float(np.float32(1e-3)), mode,
                                 eps_mul=float(np.float32(em)))
    assert _rel(got, want) <= 1e-4


@pytest.mark.parametrize("H,W,Q,C,r", [(1080, 1920, 8, 3, 8), (717, 1283, 6, 3, 5),
                                       (1080, 1920, 12, 3, 8), (1440, 2560, 3, 1, 16)])
def test_one_kernel_full_frames(H, W, Q, C, r):
    _, _, g, y = _frame(H, W, Q, C)
    one = _one_kernel(y, g, r).cpu().numpy()
    two = flr.denoise(y, g, r, fused="two_pass").cpu().numpy()
    assert np.isfinite(one).all() and _rel(one, two) <= 2e-4


def test_smaller_workspace_where_memory_is_short(monkeypatch):
    """denoise and flnr_denoise fall back on the smaller workspace."""
    _, _, g, y = _frame(600, 900, 12, 3)
    p = flr.make_params(600, 900, 12, 3, 8, fused="fused")
    packed = flr.net_pack(0.05 * torch.randn(flr.net_num_params(), device=g.device))
    full = {flr.workspace_bytes(p), flr.flnr_workspace_bytes(p)}
    assert flr.min_workspace_bytes(p) < min(full)
    two = flr.denoise(y, g, 8, fused="fused")
    g12 = g.clone()
    flnr = flr.flnr_denoise(y, g12, packed, fused="fused")
    empty, refused = torch.empty, []

    def short(size, *a, **kw):
        if size in full:
            refused.append(size)
            raise torch.OutOfMemoryError("short")
        return empty(size, *a, **kw)
    monkeypatch.setattr(api.torch, "empty", short)
    one = flr.denoise(y, g, 8, fused="fused")
    small = flr.flnr_denoise(y, g12, packed, fused="fused")
    with pytest.raises(torch.OutOfMemoryError):
        flr.denoise(y, g, 8, fused="two_pass")
    monkeypatch.undo()
    assert len(refused) == 3
    assert _rel(one.cpu().numpy(), two.cpu().numpy()) <= 2e-4
    assert _rel(small.cpu().numpy(), flnr.cpu().numpy()) <= 2e-4


@pytest.mark.parametrize("H,W,Q,C,r", [(1, 1, 1, 1, 0), (7, 9, 2, 1, 1), (64, 96, 3, 1, 1),
                                       (200, 160, 1, 3, 1), (90, 300, 6, 3, 0)])
def test_small_windows_in_either_form(H, W, Q, C, r):
    """Small windows on small frames run as one kernel in the workspace that
    they ask for, and as the two-pass path in one that only holds its image."""
    guides, noisy, g, y = _frame(H, W, Q, C)
    p = flr.make_params(H, W, Q, C, r, fused="fused")
    image = flr.workspace_bytes(flr.make_params(H, W, Q, C, r, fused="two_pass"))
    need = flr.workspace_bytes(p)
    assert need > image
    one = flr.denoise(y, g, r, fused="fused")
    ws = torch.empty(need, dtype=torch.uint8, device=g.device)
    assert torch.equal(one, flr.denoise(y, g, r, fused="fused", workspace=ws))
    two = flr.denoise(y, g, r, fused="fused", workspace=ws[:image])
    assert torch.equal(two, flr.denoise(y, g, r, fused="two_pass"))
    want = flr_ref.flr_reference(noisy, guides, r, float(np.float32(1e-3)), "ridge")
    assert _rel(one.cpu().numpy(), want) <= 1e-4 and _rel(two.cpu().numpy(), want) <= 1e-4
