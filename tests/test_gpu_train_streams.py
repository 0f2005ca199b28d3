"""GPU check of FLNRTrainer.step's side-by-side crops: the same step, bit for
bit, as the crops one after the other, over several steps, for uneven crop
sizes, for more crops than streams, on a caller's own stream, and where a
buffer shared between crops makes the trainer run them in turn."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import paper_2410_11625_amd as flr  # noqa: E402
from synth import make_training_batch  # noqa: E402
from synth.net_weights import flatten_net_weights, make_net_weights  # noqa: E402

pytestmark = pytest.mark.gpu


def _crops(dev, sizes):
    out = []
    for i, n in enumerate(sizes):
        c = make_training_batch(n=1, crop=n, frame_h=96, frame_w=128)[0]
        out.append({k: torch.from_numpy(np.ascontiguousarray(v * (1.0 + 0.1 * i),
                                                             dtype=np.float32)).to(dev)
                    for k, v in c.items()})
    return out


def _run(crops, side, dev, steps=2):
    p = torch.from_numpy(flatten_net_weights(make_net_weights(2)).astype(np.float32)).to(dev)
    tr = flr.FLNRTrainer(p, lr=1e-3, learn_eps=True)
    tr.SIDE_STREAMS = side
    losses = [tr.step(crops).clone() for _ in range(steps)]
    return torch.stack(losses), tr.grad.clone(), tr.params.clone(), tr.reg.clone()


@pytest.mark.parametrize("sizes", [(48, 48), (48, 32, 64, 48, 40, 48, 56), (64, 64, 64, 64, 64)])
@pytest.mark.parametrize("own_stream", [False, True])
def test_side_by_side_equals_in_turn(sizes, own_stream):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    dev = torch.device("cuda:0")
    crops = _crops(dev, sizes)
    want = _run(crops, 1, dev)
    s = torch.cuda.Stream() if own_stream else torch.cuda.current_stream()
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(s):
        got = _run(crops, 4, dev)
    torch.cuda.synchronize()
    for a, b in zip(got, want):
        assert torch.equal(a, b)


def test_shared_guide_buffer_runs_in_turn():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    dev = torch.device("cuda:0")
    a, b = _crops(dev, (48, 48))
    g12 = torch.zeros((12, 48, 48), device=dev)
    g12[:8] = a["guides"]
    shared = [dict(guides12=g12, noisy=c["noisy"], target=c["target"]) for c in (a, b)]
    plain = [dict(guides=a["guides"], noisy=c["noisy"], target=c["target"]) for c in (a, b)]
    tr = flr.FLNRTrainer(torch.from_numpy(
        flatten_net_weights(make_net_weights(2)).astype(np.float32)).to(dev))
    assert tr._side_streams(shared) == 1 and tr._side_streams(plain) == 2
    for x, y in zip(_run(shared, 4, dev), _run(plain, 4, dev)):
        assert torch.equal(x, y)
