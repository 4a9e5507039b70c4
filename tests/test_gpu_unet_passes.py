"""The elementwise passes of the U-Net in both widths (eight channels per thread,
one where the channel count or a pointer's alignment asks for it), the weight
packing at the edges of its tiles, and a network's gradients where each layer's
input gradient goes out as the next one's pre-activation gradient.

Sums of eight FP32 values against the same sums in torch's order of magnitude:
2e-7 of the largest (eight roundings of 6e-8, partly cancelling); values that
are only copied, halved or rounded once to BF16 must be equal."""
import ctypes as ct

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def dev(n, dtype, off=0):
    import torch

    return torch.zeros(n + off, dtype=dtype, device="cuda:0")[off:]


@pytest.mark.parametrize("D,H,W,C", [(2, 2, 2, 8), (4, 6, 10, 24), (2, 4, 6, 5), (8, 16, 32, 128)])
@pytest.mark.parametrize("off", [0, 1])
def test_pooling_both_ways(D, H, W, C, off):
    import torch

    from paper_2607_06794_amd import _lib as L

    lib, s = L.load(), ct.c_void_p(torch.cuda.current_stream().cuda_stream)
    p = lambda t: ct.c_void_p(t.data_ptr())
    gen = torch.Generator().manual_seed(C + off)
    rnd = lambda *sh: torch.randn(sh, generator=gen)
    P, Pc = D * H * W, D * H * W // 8
    held = []  # inputs stay alive until the end

    def put(t):
        held.append(dev(t.numel(), t.dtype, off).copy_(t.reshape(-1)))
        return held[-1]

    kids = lambda t: t.reshape(D // 2, 2, H // 2, 2, W // 2, 2, -1).permute(0, 2, 4, 1, 3, 5, 6).reshape(Pc, 8, -1)
    print(f"[gpu] pooling {D} x {H} x {W} x {C}, offset {off}", flush=True)
    x = rnd(P, C).bfloat16()
    y = dev(Pc * C, torch.bfloat16, off)
    L.check(lib.lb_pool2(p(put(x)), D, H, W, C, p(y), s))
    want = kids(x.float()).sum(1) * 0.125
    assert (y.cpu().float() - want.reshape(-1)).abs().max() <= 2.0 ** -8 * want.abs().max()
    st, so = C + 8, 4
    gc, skip = rnd(Pc, C), rnd(P, st)
    g = dev(P * C, torch.float32, off)
    L.check(lib.lb_pool2_backward(p(put(gc)), p(put(skip)), st, so, D, H, W, C, p(g), s))
    up = gc.reshape(D // 2, 1, H // 2, 1, W // 2, 1, C).expand(D // 2, 2, H // 2, 2, W // 2, 2, C).reshape(P, C)
    assert torch.equal(g.cpu().reshape(P, C), up * 0.125 + skip[:, so:so + C])
    gf, gq = rnd(P, st), dev(Pc * C, torch.float32, off)
    L.check(lib.lb_up2_backward(p(put(gf)), st, C, D, H, W, p(gq), s))
    want = kids(gf[:, :C].double()).sum(1)
    assert (gq.cpu().double() - want.reshape(-1)).abs().max() <= 2e-7 * 8 * gf.abs().max()
    dy, yy, gb = rnd(P * C), rnd(P * C).bfloat16(), dev(P * C, torch.bfloat16, off)
    for relu in (0, 1):
        L.check(lib.lb_relu_grad(p(put(dy)), p(put(yy)), P * C, relu, p(gb), s))
        want = torch.where(yy.float() > 0, dy, torch.zeros(())) if relu else dy
        assert torch.equal(gb.cpu(), want.bfloat16())


@pytest.mark.parametrize("cin,cout", [(8, 8), (40, 72), (64, 64), (24, 136)])
def test_packing(cin, cout):
    import torch

    from paper_2607_06794_amd import _lib as L

    lib, s = L.load(), ct.c_void_p(torch.cuda.current_stream().cuda_stream)
    w = torch.arange(27 * cin * cout, dtype=torch.int32).to(torch.int16).reshape(27 * cin, cout)
    a, b = w.to("cuda:0"), torch.zeros(27 * cin * cout, dtype=torch.int16, device="cuda:0")
    L.check(lib.lb_conv_pack_weights(ct.c_void_p(a.data_ptr()), cin, cout, ct.c_void_p(b.data_ptr()), s))
    assert torch.equal(b.cpu().reshape(cout, 27 * cin), w.T.contiguous())


def test_network_packing_is_layer_packing():
    import torch

    from paper_2607_06794_amd import _lib as L
    from paper_2607_06794_amd import surrogate as SU

    net = SU.UNet(8, 8, 16, ch=(8, 16, 24, 40)).init(3)
    want = net.pt.clone()
    net.pt.zero_()
    for name, c1, c2, co, _, _ in net.layers:
        o = net.off[name][0]
        L.check(net.lib.lb_conv_pack_weights(ct.c_void_p(net.pb.data_ptr() + 2 * o), c1 + c2, co,
                                             ct.c_void_p(net.pt.data_ptr() + 2 * o), net._s()))
    assert torch.equal(net.pt, want) and np.isfinite(net.p.cpu().numpy()).all()
