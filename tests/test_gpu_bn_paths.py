"""L1BN forward and backward against the oracle where the kernels' slices, row
tiles and load widths change: channel counts that leave a slice partly empty,
row counts around the tiles' edges, rows that only allow 4-byte loads, codes on
the edge of the range and channels whose mean is a code (sgn 0)."""
import numpy as np
import pytest

from paper_2011_14504_amd import synth

pytestmark = pytest.mark.gpu


def _dev(a, off=0):
    """a on the GPU, its first byte `off` bytes past an aligned address."""
    import torch
    b = torch.empty(a.size + 64, dtype=torch.int8, device="cuda:0")[off:off + a.size].view(a.shape)
    b.copy_(torch.from_numpy(np.ascontiguousarray(a)))
    return b


# (M, C, byte offset of the tensors, input exponent, configuration, codes)
CASES = [
    (1, 16, 0, -9, {}, "u"), (4095, 16, 0, -9, {}, "u"), (4097, 16, 0, -6, {}, "u"),
    (2047, 32, 0, -8, {}, "u"), (2049, 32, 0, -8, dict(relu=0), "u"),
    (1023, 48, 0, -7, {}, "u"), (1025, 80, 0, -7, dict(k_E2=8), "u"), (1024, 144, 0, -5, {}, "n"),
    (3, 208, 0, -6, {}, "u"), (257, 20, 0, -7, {}, "u"), (255, 268, 4, -8, {}, "n"),
    (1025, 64, 4, -7, {}, "n"), (1025, 64, 8, -7, dict(k_E2=8), "n"), (4096 * 3 + 5, 16, 0, -4, {}, "n"),
    # more row tiles than blocks
    (1024 * 70 + 3, 256, 0, -6, {}, "n"),
    # several slices, the last of 16 to 48 channels, with as many tiles as blocks and
    # one more, and where their blocks are cut to a multiple of eight
    (256 * 120 + 1, 80, 0, -6, {}, "n"), (1024 * 41, 272, 0, -6, {}, "n"), (1024 * 37 + 700, 160, 0, -6, dict(k_E2=8), "n"),
    (64 * 1500 + 63, 144, 0, -5, {}, "n"), (512 * 150 + 511, 48, 0, -7, {}, "u"), (40000, 176, 0, -6, dict(k_E2=8), "u"),
    (64 * 2100 + 1, 100, 0, -6, {}, "n"), (70001, 36, 0, -6, dict(k_E2=8), "n"), (70000, 12, 4, -6, {}, "n"),
    (50003, 80, 4, -6, {}, "n"), (4 * 64 * 51 * 5 + 64, 336, 8, -6, {}, "n"),
    # more slices than XCDs have blocks for: paired slices, an odd number of them
    (3100, 2112, 0, -6, {}, "n"), (1500, 2084, 0, -6, dict(k_E2=8), "u"),
    # constant channels, the extremes of the code range, coarse and fine grids
    (700, 64, 0, -20, {}, "edge"), (700, 64, 0, -14, {}, "edge"), (700, 64, 0, 16, {}, "edge"),
    (700, 64, 0, -40, {}, "edge"), (1500, 48, 0, -4, dict(k_mu=2, k_sigma=2), "edge"),
    (1500, 48, 0, -40, dict(k_mu=2, k_sigma=3), "edge"), (1100, 64, 0, -9, dict(k_mu=8, k_xhat=8, eps_code=32768), "n"),
    # small even codes around zero: many channels whose mean is exactly a code
    (2048, 128, 0, -6, {}, "sym"), (2048, 128, 0, -6, dict(relu=0), "sym"),
    # several channel groups per finalize block, the last one partly empty
    # (and, past 512 channels, the backward's per-channel kernel with all classes in one thread)
    (70, 512, 0, -6, dict(k_E2=8), "n"), (70, 516, 0, -6, {}, "n"), (70, 516, 0, -6, dict(k_E2=8), "n"),
    (65, 1040, 0, -6, {}, "n"), (33, 2320, 0, -7, dict(k_E2=8), "u"), (9, 6148, 0, -7, {}, "n"),
    # denominators in a kernel of their own
    (5, 2048, 0, -7, {}, "n"), (5, 2052, 0, -7, {}, "n"), (3, 65536, 0, -6, {}, "u"),
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: f"{c[0]}x{c[1]}+{c[2]}e{c[3]}{c[5]}{len(c[4])}")
def test_bn_paths(orc, case):
    import torch
    from paper_2011_14504_amd import iseg
    M, C, off, xe, kw, codes = case
    print(f"[bn paths] {case}", flush=True)
    if codes == "n":
        x = synth.gaussian_codes(71, (M, C), 30) // 2 + (np.arange(C) % 61 - 30).astype(np.int8)[None, :]
    elif codes == "sym":
        h = synth.int_codes(72, (M // 2, C), -3, 3)
        x = np.concatenate([h, -h])
        x[:, ::3] += 2
    else:
        x = synth.int_codes(73, (M, C))
    x = np.ascontiguousarray(x.astype(np.int8))
    if codes == "edge":
        for k, v in enumerate((127, -127, -128, 126, 0, 1)):
            x[:, k] = v
        x[:, 6] = np.where(np.arange(M) % 2, 127, -128)
        x[0, 7:9] = (127, -128)
    gq, bq = synth.int_codes(74, (C,)), synth.int_codes(75, (C,))
    dy = synth.int_codes(76, (M, C))
    cfg = dict(orc.BN_DEFAULT, **kw)
    c = iseg.bn_cfg(**cfg)

    def E(v):
        return torch.tensor([v], dtype=torch.int32, device="cuda:0")
    xd, dyd, g = _dev(x, off), _dev(dy, off), _dev(gq)
    status = torch.zeros(1, dtype=torch.int32, device="cuda:0")
    y, ye, saved = iseg.bn_fwd(xd, E(xe), g, _dev(bq), c, status=status)
    r = orc.bn_fwd(x, xe, gq, bq, cfg)
    sv = {k: v.cpu().numpy() for k, v in iseg.bn_saved_view(saved, C).items()}
    assert int(status.item()) == 0
    assert np.array_equal(sv["n_mu"], r["n_mu"]) and np.array_equal(sv["n_sigma"], r["n_sigma"])
    assert int(sv["hdr"][0]) == r["b"]
    assert np.array_equal(sv["xcode"][np.arange(C)[None, :], x.astype(np.int64) + 128], r["xhat"])
    assert np.array_equal(sv["qmin"], x.min(0)) and np.array_equal(sv["qmax"], x.max(0))
    assert np.array_equal(y.cpu().numpy(), r["y"]) and int(ye.item()) == r["y_exp"]
    # the saved A table holds the same codes
    assert np.array_equal(sv["acode"][np.arange(C)[None, :], x.astype(np.int64) + 128], r["y"])
    dx, dxe, dg, db, dge, dbe = iseg.bn_bwd(dyd, E(-20), xd, g, saved, c, status=status)
    rb = orc.bn_bwd(dy, -20, x, xe, gq, bq, cfg)
    assert np.array_equal(dg.cpu().numpy(), rb["dgamma"]) and int(dge.item()) == rb["dgamma_exp"]
    assert np.array_equal(db.cpu().numpy(), rb["dbeta"]) and int(dbe.item()) == rb["dbeta_exp"]
    assert np.array_equal(dx.cpu().numpy(), rb["dx"]) and int(dxe.item()) == rb["dx_exp"]


@pytest.mark.parametrize("shape", [(700, 80, 16), (700, 80, 8), (65, 2320, 16), (65, 2320, 8), (5000, 12, 8)], ids=str)
def test_bn_dirty_buffers(orc, shape):
    """Workspaces and the saved state full of ones before the calls."""
    import torch
    from paper_2011_14504_amd import iseg
    M, C, k_E2 = shape
    print(f"[bn dirty] {shape}", flush=True)
    x, dy = synth.int_codes(81, (M, C)), synth.int_codes(82, (M, C))
    gq, bq = synth.int_codes(83, (C,)), synth.int_codes(84, (C,))
    cfg = dict(orc.BN_DEFAULT, k_E2=k_E2)
    c = iseg.bn_cfg(**cfg)
    dev = "cuda:0"

    def ones(n, dt=torch.uint8):
        return torch.full((int(n),), 255 if dt == torch.uint8 else -1, dtype=dt, device=dev)
    xd, dyd, g, b = _dev(x), _dev(dy), _dev(gq), _dev(bq)
    xe, dye = (torch.tensor([v], dtype=torch.int32, device=dev) for v in (-7, -20))
    L = iseg.lib()
    y, dx = (ones(M * C, torch.int8).view(M, C) for _ in range(2))
    e = [ones(1, torch.int32) for _ in range(4)]
    dg, db = ones(C, torch.int64), ones(C, torch.int64)
    saved = ones(L.iseg_bn_saved_bytes(C))
    iseg.iseg_bn_fwd(xd, xe, M, C, g, b, c, y, e[0], saved, ones(L.iseg_bn_fwd_ws(M, C)))
    iseg.iseg_bn_bwd(dyd, dye, xd, M, C, g, c, saved, dx, e[1], dg, db, e[2], e[3], ones(L.iseg_bn_bwd_ws(M, C)))
    r = orc.bn_fwd(x, -7, gq, bq, cfg)
    assert np.array_equal(y.cpu().numpy(), r["y"]) and int(e[0].item()) == r["y_exp"]
    rb = orc.bn_bwd(dy, -20, x, -7, gq, bq, cfg)
    assert np.array_equal(dx.cpu().numpy(), rb["dx"]) and int(e[1].item()) == rb["dx_exp"]
    assert np.array_equal(dg.cpu().numpy(), rb["dgamma"]) and np.array_equal(db.cpu().numpy(), rb["dbeta"])
    assert [int(v.item()) for v in e[2:]] == [rb["dgamma_exp"], rb["dbeta_exp"]]
