"""Convolutions with K cut inside a work-group: tiles of 64 and of 128 with rows and
columns past the volume and the channels, two inputs whose border lies between
operands, an upsampled input, and a network whose levels take two, three and four
parts.

Layers against PyTorch FP64 on the CPU: BF16 operands and FP32 sums, an element of
K terms off by about sqrt(K) 2^-24 of its magnitude, so 2e-5 of the largest result.
A network adds its parts in one order whichever kernel sums them: the digests are
those of a build in which conv_small took every such layer.  Its inputs and weights
are binary fractions made from integers, exact on every machine."""
import ctypes as ct
import hashlib

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

CASES = [  # D, H, W, c1, c2, cout, up1
    (12, 20, 52, 64, 32, 64, 0),  # tiles of 64, three parts; the gradient too
    (12, 20, 52, 32, 0, 104, 0),  # columns past a tile
    (12, 28, 60, 64, 32, 40, 1),  # upsampled, two inputs
    (12, 28, 60, 32, 32, 48, 0),
    (12, 30, 46, 72, 0, 64, 0),  # the gradient: tiles of 128, two parts, columns past it
    (12, 30, 46, 64, 0, 104, 0),  # the forward
    (15, 31, 63, 104, 0, 32, 0),  # the gradient: rows past a tile
    (15, 31, 63, 32, 0, 104, 0),  # the forward
]
NETWORKS = {  # canvas: digest of the output, of the input gradients at the decoder
    (32, 56, 128): ("e83c8b3e22386000bcf3a1aa105b5c6d", "4d0639e5c5420c8a7e48a172627dff57"),  # level 1: two parts
    (24, 56, 120): ("d134869c6e9641fd8352d750ae58b097", "d8235619d3b9ac41f0ebbd14826bd759"),  # three
    (32, 40, 96): ("6307d9a1a12af9656311b216a28cf355", "ee905c5517f6b8c1a506b8869d79c7c5"),  # four
}


@pytest.mark.parametrize("case", CASES)
def test_layer_both_ways(case):
    import torch

    from paper_2607_06794_amd import _lib as L

    D, H, W, c1, c2, co, up = case
    cin, P = c1 + c2, D * H * W
    gen = torch.Generator().manual_seed(P + cin)
    rnd = lambda *s: torch.randn(s, generator=gen).bfloat16()
    x1, x2 = rnd(D >> up, H >> up, W >> up, c1), rnd(D, H, W, c2) if c2 else None
    w, b, g = rnd(27, cin, co), torch.randn(co, generator=gen), rnd(D, H, W, co)
    x = x1.double()
    if up:
        for d in range(3):
            x = x.repeat_interleave(2, dim=d)
    if c2:
        x = torch.cat([x, x2.double()], dim=-1)
    pad = lambda t: torch.nn.functional.pad(t, (0, 0, 1, 1, 1, 1, 1, 1))
    xp, gp, wd = pad(x), pad(g.double()), w.double()
    cut = lambda t, z, y, q: t[z:z + D, y:y + H, q:q + W].reshape(P, -1)
    taps = [(t // 9, t // 3 % 3, t % 3) for t in range(27)]
    ref = {"y": sum(cut(xp, *o) @ wd[t] for t, o in enumerate(taps)) + b.double(),
           "dx": sum(cut(gp, 2 - o[0], 2 - o[1], 2 - o[2]) @ wd[t].T for t, o in enumerate(taps))}
    dev = lambda t: t.to("cuda:0").contiguous()
    lib, s = L.load(), ct.c_void_p(torch.cuda.current_stream().cuda_stream)
    p = lambda t: ct.c_void_p(t.data_ptr())
    tx1, tx2, tw, tb, tg = dev(x1), dev(x2) if c2 else None, dev(w), dev(b), dev(g)
    f32 = lambda *sh: torch.zeros(sh, dtype=torch.float32, device="cuda:0")
    acc, wt = f32(P, co), torch.zeros(27 * cin * co, dtype=torch.bfloat16, device="cuda:0")
    print(f"[gpu] convolution {case}", flush=True)
    L.check(lib.lb_conv_pack_weights(p(tw), cin, co, p(wt), s))
    runs = []
    for _ in range(2):
        out = {"y": f32(P, co), "dx": f32(P, cin)}
        cv = L.LbConv()
        cv.x1, cv.c1, cv.up1, cv.x2, cv.c2 = tx1.data_ptr(), c1, up, tx2.data_ptr() if c2 else None, c2
        cv.w, cv.wt, cv.b = tw.data_ptr(), wt.data_ptr(), tb.data_ptr()
        cv.y, cv.yf, cv.acc = None, out["y"].data_ptr(), acc.data_ptr()
        cv.D, cv.H, cv.W, cv.cout, cv.relu = D, H, W, co, 0
        L.check(lib.lb_conv3d_forward(ct.byref(cv), s))
        L.check(lib.lb_conv3d_backward_data(ct.byref(cv), p(tg), p(out["dx"]), s))
        torch.cuda.synchronize()
        runs.append(out)
    for k, v in runs[0].items():
        err = float((v.cpu().double() - ref[k]).abs().max() / ref[k].abs().max())
        assert np.isfinite(err) and err <= 2e-5, (k, err)
        assert torch.equal(v, runs[1][k])


def fractions(n, seed, scale):
    """n values in (-scale, scale), multiples of scale / 1024 (scale a power of two)."""
    i = np.arange(n, dtype=np.uint64) * np.uint64(0x9E3779B97F4A7C15) + np.uint64(seed)
    i = (i ^ (i >> np.uint64(29))) * np.uint64(0xBF58476D1CE4E5B9)
    return ((i >> np.uint64(40)) % np.uint64(2047)).astype(np.float32) / 1024 * scale - (1023 / 1024) * scale


@pytest.mark.parametrize("canvas", sorted(NETWORKS), ids=lambda c: "x".join(map(str, c)))
def test_network_sums_in_one_order(canvas):
    import torch

    from paper_2607_06794_amd import surrogate as SU

    net = SU.UNet(*canvas)
    flat = np.zeros(net.nparam, np.float32)
    for k, (name, c1, c2, co, _, _) in enumerate(net.layers):
        o, nw, ob, _ = net.off[name]
        flat[o:o + nw] = fractions(nw, k, 2.0 ** -round(np.log2(27 * (c1 + c2)) / 2 - 1))
        flat[ob:ob + co] = fractions(co, 100 + k, 2.0 ** -5)
    net.set_flat(flat)
    dev = lambda a: torch.from_numpy(a).to("cuda:0")
    x, gout = dev(fractions(net.P[0] * 8, 7, 1.0)), dev(fractions(net.P[0] * 8, 8, 1.0))
    print(f"[gpu] network {canvas}", flush=True)
    net.zero_grad()
    net.forward(dev(x.cpu().bfloat16().view(torch.int16).numpy()))
    net.backward(gout)
    torch.cuda.synchronize()
    digest = lambda *ts: hashlib.sha256(b"".join((t.cpu().numpy() + 0.0).tobytes() for t in ts)).hexdigest()[:32]
    assert net.out.abs().max() > 0.01 and all(g.abs().max() > 0 for g in net.gcat)
    got = digest(net.out), digest(*net.gcat)
    print(canvas, got, flush=True)
    assert got == NETWORKS[canvas]
