"""The softmax cross-entropy's kernel variants against the oracle: class counts
on both sides of every register width, runs longer than one pass of rows, odd
ratios, one-pixel and single-row maps."""
import numpy as np
import pytest

from paper_2011_14504_amd import synth

pytestmark = pytest.mark.gpu

# (N, h, w, K, H, W, logit exponent)
CASES = [(1, 2, 3, k, 29, 47, -4) for k in (1, 24, 25, 48, 64, 65, 96, 97, 128, 129, 152, 153, 176, 177, 192, 193)]
CASES += [
    (2, 3, 2, 21, 3 * 40, 2 * 24, -3),     # 40 rows per cell: three passes, the last half empty
    (1, 1, 1, 19, 17, 33, -5),             # one low-res element: every run is clamped
    (1, 2, 2, 150, 35, 200, -5),           # runs of 17 or 18 rows and 100 columns
    (1, 4, 6, 59, 4, 6, -2),               # no upsampling: one pixel per cell
    (1, 5, 4, 150, 5 * 16 - 3, 4 * 16 - 5, -5),
]


@pytest.mark.parametrize("case", CASES, ids=str)
def test_softmax_ce_paths(orc, case):
    import torch
    from paper_2011_14504_amd import iseg
    N, h, w, K, H, W, le = case
    print(f"[loss paths] {case}", flush=True)
    logits = synth.int_codes(90 + K, (N, h, w, K))
    labels = synth.labels(91, (N, H, W), K)
    labels[:, : H // 2] = labels[:, :1, :1]          # a region of one class
    dev = "cuda:0"
    e = torch.tensor([le], dtype=torch.int32, device=dev)
    args = (torch.from_numpy(logits).to(dev), e, torch.from_numpy(labels).to(dev))
    loss, grad, err, ee = iseg.softmax_ce(*args, want_grad=True)
    rl, rg = orc.softmax_ce(logits, le, labels)
    g = grad.cpu().numpy()
    # one class: the loss is zero up to the sums' rounding of terms of size |logit|
    assert abs(float(loss.item()) - rl) <= 1e-12 * max(abs(rl), 128 * 2.0 ** le)
    assert np.max(np.abs(g - rg)) <= 1e-12 * max(np.max(np.abs(rg)), 1.0 / (N * h * w) if K == 1 else 0.0)
    if K > 1:
        rc, re = orc.quantize_f64(rg, 8)
        assert int(ee.item()) == re
        assert np.array_equal(err.cpu().numpy().astype(np.int64).ravel(), rc.ravel())
    # the same bits again: every sum has one order
    loss2, grad2, err2, _ = iseg.softmax_ce(*args, want_grad=True)
    assert torch.equal(loss, loss2) and torch.equal(grad, grad2) and torch.equal(err, err2)


@pytest.mark.parametrize("case", [(1, 2, 2, 5, 1200, 400, -1), (1, 3, 3, 150, 900, 120, -2)], ids=str)
def test_softmax_ce_long_runs(orc, case):
    """Cells of hundreds of rows and columns: the error of the exps grows with
    rows times columns, 2.5e-16 each (an exp's and a rounding's error per step)."""
    import torch
    from paper_2011_14504_amd import iseg
    N, h, w, K, H, W, le = case
    print(f"[loss long runs] {case}", flush=True)
    logits = synth.int_codes(90 + K, (N, h, w, K))
    labels = synth.labels(91, (N, H, W), K)
    dev = "cuda:0"
    e = torch.tensor([le], dtype=torch.int32, device=dev)
    loss, grad, err, ee = iseg.softmax_ce(torch.from_numpy(logits).to(dev), e, torch.from_numpy(labels).to(dev),
                                          want_grad=True)
    rl, rg = orc.softmax_ce(logits, le, labels)
    tol = 2.5e-16 * (H / h + 1) * (W / w + 1)
    assert abs(float(loss.item()) - rl) <= tol * abs(rl)
    assert np.max(np.abs(grad.cpu().numpy() - rg)) <= tol * np.max(np.abs(rg))
    rc, re = orc.quantize_f64(rg, 8)
    assert int(ee.item()) == re and np.array_equal(err.cpu().numpy().astype(np.int64).ravel(), rc.ravel())
