"""GPU check of the memory that FLNRTrainer keeps for crops side by side: it
stays within SIDE_BYTES over batches of ever new sizes, smaller bounds take
fewer streams down to one, the step is the same bit for bit, and a captured
step keeps its buffers."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import paper_2410_11625_amd as flr  # noqa: E402
from synth import make_training_batch  # noqa: E402
from synth.net_weights import flatten_net_weights, make_net_weights  # noqa: E402

pytestmark = pytest.mark.gpu


def _dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch.device("cuda:0")


def _crops(dev, n, count):
    c = make_training_batch(n=1, crop=n, frame_h=96, frame_w=128)[0]
    return [{k: torch.from_numpy(np.ascontiguousarray(v * (1.0 + 0.1 * i), dtype=np.float32))
             .to(dev) for k, v in c.items()} for i in range(count)]


def _trainer(dev, side_bytes):
    p = torch.from_numpy(flatten_net_weights(make_net_weights(2)).astype(np.float32)).to(dev)
    tr = flr.FLNRTrainer(p, lr=1e-3)
    tr.SIDE_BYTES = side_bytes
    return tr


def _set_bytes(n):
    tr = _trainer(_dev(), 0)
    tr.step(_crops(_dev(), n, 1))
    return sum(t.numel() * t.element_size() for b in tr._bufs.values() for t in b.values())


def test_side_buffers_stay_within_their_bound():
    dev = _dev()
    sizes = [64, 40, 56, 44, 60, 48, 52, 64]
    batches = [_crops(dev, n, 4) for n in sizes]
    one = {n: _set_bytes(n) for n in sizes}
    bound = 4 * max(one.values())
    want = _trainer(dev, 0)
    want_losses = [want.step(b).clone() for b in batches]
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    before = torch.cuda.memory_allocated()
    tr = _trainer(dev, bound)
    losses = [tr.step(b).clone() for b in batches]
    torch.cuda.synchronize()
    kept = torch.cuda.memory_allocated() - before
    # one set per size, the bound, and the trainer's own vectors
    assert kept <= sum(one[n] for n in set(sizes)) + bound + (8 << 20), kept
    assert kept > sum(one[n] for n in set(sizes))  # crops did run side by side
    assert all(torch.equal(a, b) for a, b in zip(losses, want_losses))
    assert torch.equal(tr.params, want.params)


@pytest.mark.parametrize("sets,streams", [(0, 1), (1, 2), (2, 3), (3, 4)])
def test_bound_sets_the_streams(sets, streams):
    dev = _dev()
    crops = _crops(dev, 48, 5)
    tr = _trainer(dev, sets * _set_bytes(48))
    tr.step(crops)
    torch.cuda.synchronize()
    assert len({k[2] for k in tr._side}) == streams - 1


def test_captured_step_keeps_its_buffers():
    dev = _dev()
    crops = _crops(dev, 48, 3)
    ref, tr = _trainer(dev, 0), _trainer(dev, 2 * _set_bytes(48))
    for t in (ref, tr):
        t.step(crops)
    state = tr.params.clone(), tr.m.clone(), tr.v.clone()
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=s):
        losses = tr.step(crops)
    want = ref.step(crops)
    held = dict(tr._side)
    for n in (40, 56, 64):  # other sizes do not take the captured step's sets
        tr.step(_crops(dev, n, 6))
    assert all(tr._side.get(k) is b for k, b in held.items())
    for _ in range(3):
        for t, v in zip((tr.params, tr.m, tr.v), state):
            t.copy_(v)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(losses, want) and torch.equal(tr.params, ref.params)
        tr.step(_crops(dev, 40, 2))
