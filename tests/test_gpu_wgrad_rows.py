"""Weight gradients of 3x3 stride-1 convs with padding = dilation (the row
kernel: x rows shared by the taps over rows extended by the dilation) against
exact library sums: both tile widths, rows narrower and wider than a step,
images smaller than a chunk, dilations up to the limit and past it, one and many
splits, and every reduction of the splits."""
import numpy as np
import pytest

from paper_2011_14504_amd import synth

pytestmark = pytest.mark.gpu

# (N, H, W, C, K, dilation, kernel): "taps" where the row kernel's extended rows
# and 128-pixel blocks cost more than its shared loads save
CASES = [
    (1, 1, 1, 64, 64, 1, "taps"), (1, 2, 3, 64, 128, 1, "taps"), (3, 7, 5, 64, 64, 2, "taps"),
    (2, 9, 70, 64, 128, 1, "rows"), (1, 40, 129, 64, 64, 1, "rows"), (1, 13, 40, 128, 192, 6, "rows"),
    (2, 16, 16, 64, 256, 18, "taps"), (1, 70, 66, 64, 64, 63, "rows"), (1, 70, 66, 64, 64, 64, "rows"),
    (1, 70, 70, 64, 64, 65, "taps"), (1, 3, 200, 192, 128, 3, "rows"), (5, 33, 31, 128, 128, 1, "rows"),
    (2, 64, 64, 64, 64, 1, "rows"), (16, 56, 56, 64, 64, 1, "rows"), (1, 65, 63, 512, 384, 2, "rows"),
    # the row kernel on images smaller than a chunk, and with rows no longer than the dilation
    (300, 2, 3, 320, 192, 1, "rows"), (60, 7, 5, 64, 64, 2, "rows"), (200, 7, 5, 64, 64, 2, "rows"),
    (2, 16, 16, 64, 64, 18, "rows"), (1, 64, 64, 64, 64, 63, "rows"),
    # narrow maps under strong dilation, and little work
    (8, 8, 8, 512, 256, 18, "taps"), (8, 8, 8, 512, 256, 1, "taps"), (4, 16, 16, 512, 128, 36, "taps"),
    (3, 13, 7, 128, 64, 64, "taps"),
]


@pytest.mark.parametrize("case", CASES, ids=str)
def test_wgrad_rows(orc, case):
    import torch
    from paper_2011_14504_amd import iseg
    N, H, W, C, K, d, kernel = case
    print(f"[wgrad rows] {case}", flush=True)
    x = synth.int_codes(40, (N, H, W, C), -128, 127)
    dy = synth.int_codes(41, (N, H, W, K), -128, 127)
    dev = "cuda:0"
    e = [torch.tensor([v], dtype=torch.int32, device=dev) for v in (-20, -7)]
    args = (torch.from_numpy(dy).to(dev), e[0], torch.from_numpy(x).to(dev), e[1], (K, 3, 3, C), 1, d, d)
    raw, re = iseg.conv_bwd_weight(*args, g_mode=iseg.ISEG_G_RAW)
    assert iseg.iseg_conv_last_plan() == "wgrad_" + kernel
    # per tap: dy^T x over the shifted pixels, exact in float64
    xp = np.zeros((N, H + 2 * d, W + 2 * d, C), np.float64)
    xp[:, d:d + H, d:d + W] = x
    dyf = torch.from_numpy(dy.reshape(-1, K).astype(np.float64)).to(dev)
    ref = np.zeros((K, 3, 3, C), np.int64)
    for r in range(3):
        for s in range(3):
            t = torch.from_numpy(np.ascontiguousarray(xp[:, r * d:r * d + H, s * d:s * d + W]).reshape(-1, C)).to(dev)
            ref[:, r, s] = (dyf.t().contiguous() @ t).cpu().numpy().astype(np.int64)
    assert np.array_equal(raw.cpu().numpy(), ref) and int(re.item()) == -27
    g, ge = iseg.conv_bwd_weight(*args, seed=5, tensor_id=16, step=2)
    rc, rce = orc.requant(ref, -27, 8, stochastic=True, keep_scale=True, seed=5, tensor_id=16, step=2)
    assert np.array_equal(g.cpu().numpy().astype(np.int64), rc) and int(ge.item()) == rce
