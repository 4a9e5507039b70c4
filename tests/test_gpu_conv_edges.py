"""Convolutions at the edges of their tiles: volumes of one cell and of odd
extents, one more and one less than a brick, channel counts below, at and above
the 32-channel operand and the 128-channel stage, a concatenation whose border
lies inside an operand, upsampled inputs, and volumes on both sides of the
borders between the kernels.  Forward, input gradient, weight and bias
gradients against PyTorch FP64 on the CPU.

The operands are BF16 and the sums FP32: an element of K terms is off by about
sqrt(K) 2^-24 of its magnitude, at most 1e-5 of the largest result for the
K <= 27 x 264 and the positions <= 20 000 here, so 2e-5 as in the layer tests."""
import ctypes as ct

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

CASES = [  # D, H, W, c1, c2, cout, up1
    (1, 1, 1, 8, 0, 8, 0),
    (1, 2, 3, 24, 0, 40, 0),
    (3, 5, 7, 8, 8, 16, 0),
    (2, 4, 4, 32, 0, 64, 0),
    (3, 5, 5, 128, 0, 72, 0),
    (4, 6, 10, 136, 0, 24, 0),
    (4, 8, 8, 256, 8, 32, 1),
    (4, 4, 6, 16, 24, 104, 1),
    (5, 9, 9, 40, 40, 33 * 8, 0),
    (2, 6, 6, 160, 96, 256, 0),  # K in 27 parts, four rounds of eight wavefronts
    (3, 18, 20, 96, 64, 160, 0),  # 16 parts, two column tiles per work-group
    (8, 16, 64, 8, 0, 32, 0),  # 8 192 positions
    (9, 16, 64, 32, 0, 64, 0),  # more, whole bricks in y and x only
    (4, 40, 56, 32, 16, 32, 0),  # whole bricks
    (10, 30, 31, 16, 0, 8, 0),  # no whole bricks, few tiles
    (2, 72, 136, 8, 8, 160, 1),  # whole bricks, wide: the GEMM
]


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
    ref = {
        "y": sum(cut(xp, *o) @ wd[t] for t, o in enumerate(taps)) + b.double(),
        "dx": sum(cut(gp, 2 - o[0], 2 - o[1], 2 - o[2]) @ wd[t].T for t, o in enumerate(taps)),
        "dw": torch.stack([cut(xp, *o).T @ g.double().reshape(P, -1) for o in taps]),
        "db": g.double().reshape(P, -1).sum(0),
    }
    dev = lambda t: t.to("cuda:0").contiguous()
    lib, s = L.load(), ct.c_void_p(torch.cuda.current_stream().cuda_stream)
    p = lambda t: ct.c_void_p(t.data_ptr())
    tx1, tx2, tw, tb, tg = dev(x1), dev(x2) if c2 else None, dev(w), dev(b), dev(g)
    f32 = lambda *sh: torch.zeros(sh, dtype=torch.float32, device="cuda:0")
    out = {"y": f32(P, co), "dx": f32(P, cin), "dw": f32(27, cin, co), "db": f32(co)}
    wt = torch.zeros(27 * cin * co, dtype=torch.bfloat16, device="cuda:0")
    print(f"[gpu] convolution {case}", flush=True)
    L.check(lib.lb_conv_pack_weights(p(tw), cin, co, p(wt), s))
    cv = L.LbConv()
    cv.x1, cv.c1, cv.up1, cv.x2, cv.c2 = tx1.data_ptr(), c1, up, tx2.data_ptr() if c2 else None, c2
    cv.w, cv.wt, cv.b = tw.data_ptr(), wt.data_ptr(), tb.data_ptr()
    cv.y, cv.yf, cv.acc = None, out["y"].data_ptr(), None
    cv.D, cv.H, cv.W, cv.cout, cv.relu = D, H, W, co, 0
    L.check(lib.lb_conv3d_forward(ct.byref(cv), s))
    L.check(lib.lb_conv3d_backward_data(ct.byref(cv), p(tg), p(out["dx"]), s))
    L.check(lib.lb_conv3d_backward_weights(ct.byref(cv), p(tg), p(out["dw"]), p(out["db"]), s))
    torch.cuda.synchronize()
    for k, v in out.items():
        r = ref[k].reshape(v.shape)
        err = float((v.cpu().double() - r).abs().max() / r.abs().max())
        assert np.isfinite(err) and err <= 2e-5, (k, err)
