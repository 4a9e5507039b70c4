"""A network on a stream that is not torch's current one: what its calls return
belongs to the work they queued there."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("given", [True, False], ids=["stream given", "built under the stream"])
def test_training_loss_of_its_own_step(given):
    import torch

    from paper_2607_06794_amd import surrogate as SU

    side = torch.cuda.Stream()
    if given:
        net = SU.UNet(8, 8, 16, ch=(8, 16, 24, 40), stream=side)
    else:
        with torch.cuda.stream(side):
            net = SU.UNet(8, 8, 16, ch=(8, 16, 24, 40))
    torch.cuda.synchronize()
    net.init(3)
    gen = torch.Generator().manual_seed(5)
    x, tgt, far = (torch.rand(net.P[0], 8, generator=gen) for _ in range(3))
    x[:, 6] = 1.0
    x, tgt, far = (t.reshape(-1).to("cuda:0") for t in (x, tgt, 3.0 * far))
    torch.cuda.synchronize()
    net.forward(net.prepare(x))
    want = net.loss(x, tgt, 1.0)
    other = net.loss(x, far, 1.0)  # what an early read would find
    assert other[0] != want[0] and np.isfinite(want).all()
    assert torch.cuda.current_stream() != side
    print(f"[gpu] train step behind a busy stream, given={given}", flush=True)
    with torch.cuda.stream(side):
        torch.cuda._sleep(100_000_000)  # the step's kernels wait behind this, about 50 ms
    got = net.train_step(None, x, tgt, lam=1.0)
    assert got == want
