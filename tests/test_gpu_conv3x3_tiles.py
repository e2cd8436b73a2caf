"""3x3 stride-1 convs and their backward-data at the edges of the 32-wide tiles:
images smaller than a tile and ragged ones, both tile heights, one and several
64-channel chunks, both dilations in either axis and every output mode (raw sums, recomputed codes, staged sums) against exact
library sums."""
import numpy as np
import pytest

from paper_2011_14504_amd import synth

pytestmark = pytest.mark.gpu

# (N, H, W, C, K, padding (h, w), dilation (h, w))
CASES = [
    (1, 1, 1, 64, 64, (1, 1), (1, 1)), (2, 7, 31, 128, 64, (1, 1), (1, 1)), (1, 9, 33, 64, 192, (1, 1), (1, 1)),
    (2, 8, 32, 192, 128, (2, 2), (2, 2)), (1, 17, 65, 256, 64, (1, 2), (1, 2)), (3, 16, 30, 128, 256, (2, 1), (2, 1)),
    (1, 12, 40, 320, 64, (0, 0), (1, 1)), (2, 11, 20, 64, 64, (3, 0), (2, 2)), (1, 33, 32, 512, 128, (2, 2), (2, 2)),
    # enough tiles for the tall ones (but where both dilations are 2)
    (17, 65, 97, 64, 128, (1, 1), (1, 1)), (16, 17, 33, 192, 512, (1, 1), (1, 1)), (33, 16, 64, 128, 512, (1, 2), (1, 2)),
    (25, 30, 33, 64, 256, (1, 1), (1, 1)), (33, 30, 32, 192, 512, (2, 1), (2, 1)), (33, 16, 32, 192, 1024, (2, 2), (2, 2)),
]


def _sums(x, w, pad, dil):
    """exact conv sums, x [N][H][W][C], w [K][3][3][C], in float64 on the GPU"""
    import torch
    N, H, W, C = x.shape
    xp = torch.zeros((N, H + 2 * pad[0], W + 2 * pad[1], C), dtype=torch.float64, device="cuda:0")
    xp[:, pad[0]:pad[0] + H, pad[1]:pad[1] + W] = torch.from_numpy(x).to("cuda:0")
    P, Q = H + 2 * pad[0] - 2 * dil[0], W + 2 * pad[1] - 2 * dil[1]
    wd = torch.from_numpy(w).to("cuda:0").double()
    out = torch.zeros((N * P * Q, w.shape[0]), dtype=torch.float64, device="cuda:0")
    for r in range(3):
        for s in range(3):
            t = xp[:, r * dil[0]:r * dil[0] + P, s * dil[1]:s * dil[1] + Q].reshape(-1, C)
            out += t @ wd[:, r, s].t().contiguous()
    return out.view(N, P, Q, -1).cpu().numpy().astype(np.int64)


@pytest.mark.parametrize("case", CASES, ids=str)
def test_conv3x3_tiles(orc, case):
    import torch
    from paper_2011_14504_amd import iseg
    N, H, W, C, K, pad, dil = case
    print(f"[conv3x3 tiles] {case}", flush=True)
    dev = "cuda:0"
    e = [torch.tensor([v], dtype=torch.int32, device=dev) for v in (-7, -9)]
    x = synth.int_codes(50, (N, H, W, C), -128, 127)
    w = synth.int_codes(51, (K, 3, 3, C), -128, 127)
    ref = _sums(x, w, pad, dil)
    xd, wd = torch.from_numpy(x).to(dev), torch.from_numpy(w).to(dev)
    for mode in (iseg.ISEG_OUT_RAW, iseg.ISEG_OUT_Q8):
        y, ye = iseg.conv_fwd(xd, e[0], wd, e[1], 1, pad, dil, mode)
        assert iseg.iseg_conv_last_plan() == "m32"
        r, re = (ref, -16) if mode == iseg.ISEG_OUT_RAW else orc.requant(ref, -16, 8)
        assert np.array_equal(y.cpu().numpy().astype(np.int64), r) and int(ye.item()) == re
    # backward-data: the adjoint is the conv of dy with the flipped, transposed filter
    dy = synth.int_codes(52, ref.shape, -128, 127)
    wt = np.ascontiguousarray(w[:, ::-1, ::-1].transpose(3, 1, 2, 0))
    ref = _sums(dy, wt, (2 * dil[0] - pad[0], 2 * dil[1] - pad[1]), dil)
    dyd = torch.from_numpy(dy).to(dev)
    for mode in (iseg.ISEG_OUT_RAW, iseg.ISEG_OUT_Q8):
        dx, dxe = iseg.conv_bwd_data(dyd, e[0], wd, e[1], x.shape, 1, pad, dil, mode)
        assert iseg.iseg_conv_last_plan() == "m32"
        r, re = (ref, -16) if mode == iseg.ISEG_OUT_RAW else orc.requant(ref, -16, 8)
        assert np.array_equal(dx.cpu().numpy().astype(np.int64), r) and int(dxe.item()) == re
