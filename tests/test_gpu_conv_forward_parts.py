"""Forward convolutions whose sum over K may go in parts (a layer given its
scratch acc): volumes of one cell and of odd extents, channel counts inside a
32-channel operand, at and beyond a stage of 128 or 256 channels, a concatenation
whose border lies inside an operand, an upsampled input, one and two column
tiles per work-group.  Against PyTorch FP64 on the CPU, with and without acc;
two runs with acc are the same bits, and the BF16 output is the FP32 one rounded.

BF16 operands, FP32 sums: an element of K terms is off by about sqrt(K) 2^-24
of its magnitude, 7e-6 for K = 27 x 520, so 2e-5 of the largest result."""
import ctypes as ct

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

CASES = [  # D, H, W, c1, c2, cout, up1
    (1, 1, 1, 64, 0, 8, 0),  # parts, one cell
    (1, 2, 3, 24, 0, 40, 0),  # one stage, the operand's last eight channels missing
    (3, 5, 7, 40, 40, 72, 0),  # the concatenation's border inside an operand
    (3, 18, 20, 64, 0, 160, 0),  # parts of at most 128 channels, two column tiles
    (2, 6, 6, 160, 96, 256, 0),  # parts of 256 channels
    (3, 18, 20, 96, 64, 160, 0),  # the same, two column tiles
    (4, 6, 10, 136, 0, 24, 0),  # two stages, the second of eight channels
    (3, 18, 20, 128, 8, 160, 0),  # the same, two column tiles
    (4, 4, 6, 256, 8, 104, 1),  # three stages, upsampled
    (2, 3, 5, 512, 8, 16, 0),  # five stages
    (5, 9, 9, 40, 40, 264, 0),
]


@pytest.mark.parametrize("case", CASES)
def test_forward_in_parts(case):
    import torch

    from paper_2607_06794_amd import _lib as L

    D, H, W, c1, c2, co, up = case
    cin, P = c1 + c2, D * H * W
    gen = torch.Generator().manual_seed(P + cin)
    rnd = lambda *s: torch.randn(s, generator=gen).bfloat16()
    x1, x2 = rnd(D >> up, H >> up, W >> up, c1), rnd(D, H, W, c2) if c2 else None
    w, b = rnd(27, cin, co), torch.randn(co, generator=gen)
    x = x1.double()
    if up:
        for d in range(3):
            x = x.repeat_interleave(2, dim=d)
    if c2:
        x = torch.cat([x, x2.double()], dim=-1)
    xp = torch.nn.functional.pad(x, (0, 0, 1, 1, 1, 1, 1, 1))
    ref = b.double() + sum(xp[t // 9:t // 9 + D, t // 3 % 3:t // 3 % 3 + H, t % 3:t % 3 + W].reshape(P, -1) @ w[t].double()
                           for t in range(27))
    dev = lambda t: t.to("cuda:0").contiguous()
    lib, s = L.load(), ct.c_void_p(torch.cuda.current_stream().cuda_stream)
    tx1, tx2, tw, tb = dev(x1), dev(x2) if c2 else None, dev(w), dev(b)
    wt = torch.zeros(27 * cin * co, dtype=torch.bfloat16, device="cuda:0")
    acc = torch.zeros(P * co, dtype=torch.float32, device="cuda:0")
    print(f"[gpu] forward {case}", flush=True)
    L.check(lib.lb_conv_pack_weights(ct.c_void_p(tw.data_ptr()), cin, co, ct.c_void_p(wt.data_ptr()), s))

    def run(scratch, relu):
        yf, y = (torch.zeros((P, co), dtype=t, device="cuda:0") for t in (torch.float32, torch.bfloat16))
        cv = L.LbConv()
        cv.x1, cv.c1, cv.up1, cv.x2, cv.c2 = tx1.data_ptr(), c1, up, tx2.data_ptr() if c2 else None, c2
        cv.w, cv.wt, cv.b = tw.data_ptr(), wt.data_ptr(), tb.data_ptr()
        cv.y, cv.yf, cv.acc = y.data_ptr(), yf.data_ptr(), scratch
        cv.D, cv.H, cv.W, cv.cout, cv.relu = D, H, W, co, relu
        L.check(lib.lb_conv3d_forward(ct.byref(cv), s))
        torch.cuda.synchronize()
        return yf.cpu(), y.cpu()

    whole, parts, again, relu = run(None, 0), run(acc.data_ptr(), 0), run(acc.data_ptr(), 0), run(acc.data_ptr(), 1)
    for yf, y in (whole, parts):
        err = float((yf.double() - ref).abs().max() / ref.abs().max())
        assert np.isfinite(err) and err <= 2e-5, err
        assert torch.equal(y, yf.bfloat16())
    assert torch.equal(again[0], parts[0])
    assert torch.equal(relu[0], parts[0].clamp(min=0.0)) and torch.equal(relu[1], relu[0].bfloat16())
