"""Convs whose channel counts are multiples of 16 but not of the tiles, and any
number of output channels (the flat direct-to-LDS kernel and the split weight
gradient): steps that straddle taps, several taps per step, ragged reductions,
rows and columns, strides and dilations, every tile size, all three directions
and output modes against exact library sums."""
import numpy as np
import pytest

from paper_2011_14504_amd import synth

pytestmark = pytest.mark.gpu

# (N, H, W, C, K, R, stride, padding, dilation)
CASES = [
    (1, 1, 1, 16, 16, 1, 1, 0, 1), (1, 5, 7, 16, 16, 3, 1, 1, 1), (2, 9, 11, 48, 32, 3, 2, 1, 1),
    (1, 17, 13, 80, 48, 5, 1, 2, 1), (3, 13, 9, 96, 160, 3, 2, 1, 1), (1, 20, 21, 144, 64, 3, 1, 4, 4),
    (1, 15, 15, 208, 16, 1, 3, 0, 1), (2, 8, 8, 64, 19, 1, 1, 0, 1), (2, 9, 9, 128, 150, 3, 1, 1, 1),
    (1, 65, 63, 32, 48, 3, 1, 1, 1), (1, 7, 7, 256, 21, 1, 1, 0, 1), (1, 11, 6, 336, 80, 2, 1, 0, 2),
    # input channels padded to 16
    (2, 9, 11, 20, 32, 3, 2, 1, 1), (1, 10, 12, 36, 48, 3, 1, 1, 1),
    # enough tiles for the large ones, ragged both ways
    (9, 65, 63, 80, 144, 3, 1, 1, 1), (17, 45, 45, 16, 272, 1, 1, 0, 1), (33, 33, 33, 112, 96, 3, 2, 1, 1),
]


def _taps(H, W, R, st, pad, dil):
    P, Q = (H + 2 * pad - dil * (R - 1) - 1) // st + 1, (W + 2 * pad - dil * (R - 1) - 1) // st + 1
    for r in range(R):
        for s in range(R):
            yield r, s, slice(r * dil, r * dil + st * (P - 1) + 1, st), slice(s * dil, s * dil + st * (Q - 1) + 1, st), P, Q


@pytest.mark.parametrize("case", CASES, ids=str)
def test_conv_flat(orc, case):
    import torch
    from paper_2011_14504_amd import iseg
    N, H, W, C, K, R, st, pad, dil = case
    print(f"[conv flat] {case}", flush=True)
    dev = "cuda:0"
    e = [torch.tensor([v], dtype=torch.int32, device=dev) for v in (-7, -9)]
    x = torch.from_numpy(synth.int_codes(60, (N, H, W, C), -128, 127)).to(dev)
    w = torch.from_numpy(synth.int_codes(61, (K, R, R, C), -128, 127)).to(dev)
    xp = torch.zeros((N, H + 2 * pad, W + 2 * pad, C), dtype=torch.float64, device=dev)
    xp[:, pad:pad + H, pad:pad + W] = x
    ref = 0
    for r, s, hs, ws, P, Q in _taps(H, W, R, st, pad, dil):
        ref = ref + xp[:, hs, ws].reshape(-1, C) @ w[:, r, s].double().t().contiguous()
    ref = ref.cpu().numpy().astype(np.int64).reshape(N, P, Q, K)
    dy = torch.from_numpy(synth.int_codes(62, ref.shape, -128, 127)).to(dev)
    dxp = torch.zeros_like(xp)
    gref = torch.zeros((K, R, R, C), dtype=torch.float64, device=dev)
    for r, s, hs, ws, P, Q in _taps(H, W, R, st, pad, dil):
        gref[:, r, s] = dy.double().reshape(-1, K).t().contiguous() @ xp[:, hs, ws].reshape(-1, C)
        dxp[:, hs, ws] += (dy.double().reshape(-1, K) @ w[:, r, s].double()).view(N, P, Q, C)
    dref = dxp[:, pad:pad + H, pad:pad + W].cpu().numpy().astype(np.int64)
    for mode in (iseg.ISEG_OUT_RAW, iseg.ISEG_OUT_Q8):
        fwd = iseg.conv_fwd(x, e[0], w, e[1], st, pad, dil, mode)
        plans = [iseg.iseg_conv_last_plan()]
        bwd = iseg.conv_bwd_data(dy, e[0], w, e[1], x.shape, st, pad, dil, mode)
        plans.append(iseg.iseg_conv_last_plan())
        # backward-data: strided convs from few channels and strided 1x1 have paths of their own, and
        # dy of other channel counts takes the generic or (padded) the direct-to-LDS kernel
        assert plans[0] == "flat" and (plans[1] == "flat") == (K % 16 == 0 and not (st > 1 and (R == 1 or K <= 32)))
        for out, oe, want in ((*fwd, ref), (*bwd, dref)):
            r, re = (want, -16) if mode == iseg.ISEG_OUT_RAW else orc.requant(want, -16, 8)
            assert np.array_equal(out.cpu().numpy().astype(np.int64), r) and int(oe.item()) == re
    g, ge = iseg.conv_bwd_weight(dy, e[0], x, e[1], w.shape, st, pad, dil, iseg.ISEG_G_RAW)
    gref = gref.cpu().numpy().astype(np.int64)
    assert K % 16 or C % 16 or iseg.iseg_conv_last_plan() in ("wgrad_tr", "wgrad_rows")
    assert np.array_equal(g.cpu().numpy(), gref) and int(ge.item()) == -16
    g, ge = iseg.conv_bwd_weight(dy, e[0], x, e[1], w.shape, st, pad, dil, seed=5, tensor_id=16, step=2)
    r, re = orc.requant(gref, -16, 8, stochastic=True, keep_scale=True, seed=5, tensor_id=16, step=2)
    assert np.array_equal(g.cpu().numpy().astype(np.int64), r) and int(ge.item()) == re
