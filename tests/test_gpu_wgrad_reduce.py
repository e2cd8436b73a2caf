"""The sums over a weight gradient's splits against exact library sums: split
counts on both sides of every choice of waves per block, the last steps of four
and eight splits full and ragged, few and many blocks."""
import numpy as np
import pytest

from paper_2011_14504_amd import synth

pytestmark = pytest.mark.gpu

# (splits, C, K): 1x1 convs of 256 pixels per split
CASES = [(s, 64, 64) for s in (9, 15, 16, 17, 24, 25, 33, 64, 65, 80, 81, 128, 129, 200)]
CASES += [(9, 16, 16), (27, 48, 16), (100, 16, 80), (9, 512, 512), (12, 512, 512), (40, 192, 128)]


@pytest.mark.parametrize("case", CASES, ids=str)
def test_wgrad_split_sums(orc, case):
    import torch
    from paper_2011_14504_amd import iseg
    splits, C, K = case
    print(f"[wgrad reduce] {case}", flush=True)
    x = synth.int_codes(50, (1, splits, 256, C), -128, 127)
    dy = synth.int_codes(51, (1, splits, 256, K), -128, 127)
    dev = "cuda:0"
    e = [torch.tensor([v], dtype=torch.int32, device=dev) for v in (-20, -7)]
    xd, dyd = torch.from_numpy(x).to(dev), torch.from_numpy(dy).to(dev)
    args = (dyd, e[0], xd, e[1], (K, 1, 1, C))
    raw, re = iseg.conv_bwd_weight(*args, g_mode=iseg.ISEG_G_RAW)
    assert iseg.iseg_conv_last_plan() == "wgrad_tr"
    ref = (dyd.reshape(-1, K).double().t().contiguous() @ xd.reshape(-1, C).double()).cpu().numpy().astype(np.int64)
    ref = ref.reshape(K, 1, 1, C)
    assert np.array_equal(raw.cpu().numpy(), ref) and int(re.item()) == -27
    g, ge = iseg.conv_bwd_weight(*args, seed=5, tensor_id=16, step=2)
    rc, rce = orc.requant(ref, -27, 8, stochastic=True, keep_scale=True, seed=5, tensor_id=16, step=2)
    assert np.array_equal(g.cpu().numpy().astype(np.int64), rc) and int(ge.item()) == rce
