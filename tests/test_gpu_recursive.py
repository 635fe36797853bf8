"""Maps for large widths by recursive filtering: the HIP path against the
oracle's Young-van Vliet maps (FP64 recursions on both sides, FP32 maps), and
the fit on those maps against the oracle's lattice fit on the same maps."""
import math

import numpy as np
import pytest
import torch

import oracle as O
from paper_1310_7114_amd import synth as S

pytestmark = pytest.mark.gpu


def normwise(a, b):
    return float(np.linalg.norm(a - b) / max(np.linalg.norm(b), 1e-300))


def gpu_rec(itc, img, sigma, scale=1.0, pitch=None):
    H, W = img.shape
    if pitch is None:
        x = torch.from_numpy(img).cuda()
    else:
        buf = torch.zeros((H, pitch), dtype=torch.from_numpy(img).dtype, device="cuda")
        buf[:, :W] = torch.from_numpy(img).cuda()
        x = buf[:, :W]
    m = itc.precompute_recursive(x, sigma, scale=scale)
    torch.cuda.synchronize()
    return m, [p.cpu().double().numpy() for p in m.planes()], float(m.s_x.cpu()[0])


CASES = [
    ("ellipses64_s2", lambda: S.config1_case(1).img, 2.0, 1.0),
    ("ellipses64_s6", lambda: S.config1_case(2).img, 6.0, 1.0),
    ("ragged70x133_s4", lambda: (np.random.default_rng(1).uniform(size=(70, 133)) < 0.3).astype(np.uint8), 4.0, 1.0),
    ("gray100x77_s12", lambda: S.gray_gaussians((7, 0), H=100, W=77, n=8, major=(5, 30)), 12.0, 1 / 255),
    ("f32_90x200_s25", lambda: np.random.default_rng(2).uniform(size=(90, 200)).astype(np.float32), 25.0, 1.0),
    ("tiny1x1_s1", lambda: np.ones((1, 1), np.uint8), 1.0, 1.0),
    ("small3x5_s0.5", lambda: np.array([[0, 1, 1, 0, 1], [1, 1, 0, 0, 1], [0, 0, 1, 1, 1]], np.uint8), 0.5, 1.0),
    ("shapes512_s40", lambda: S.config2_case(0).img, 40.0, 1.0),
]


@pytest.mark.parametrize("name,build,sigma,scale", CASES, ids=[c[0] for c in CASES])
def test_recursive_maps(gpu_lib, name, build, sigma, scale):
    img = build()
    m, got, sx = gpu_rec(gpu_lib, img, sigma, scale)
    A, Mu, Mv, sx_ref = O.recursive_maps(img.astype(np.float64) * scale, sigma)
    for g, r in zip(got, (A, Mu, Mv)):
        assert normwise(g, r) <= 1e-6
    assert sx == pytest.approx(sx_ref, rel=1e-6)
    # columns past the width inside the last map panel are written as zero
    H, W = img.shape
    full = (W + 15) // 16 * 16
    if full > W:
        n = gpu_lib.plane_elems(m.desc)
        flat = m.buf[: 3 * n * 4].view(torch.float32)
        for i in range(3):
            assert torch.all(gpu_lib.panel_view(flat[i * n:(i + 1) * n], H, full)[:, W:] == 0)


# sigma = 4: lines of W + 26 and H + 26 entries around the compiled segment lengths (64 segments of 7, 13, 19, 25,
# 35 and 39 entries along rows, 48 of 8, 16, 25, 34, 45 and 52 along columns) and past the longest of each; one and
# two S_X row groups; widths around the 8-column runs of the column pass
@pytest.mark.parametrize("H,W,dt", [(358, 422, np.uint8), (359, 423, np.float32), (742, 806, np.uint8), (743, 807, np.uint8),
                                    (17, 1190, np.uint8), (66, 1191, np.uint8), (1174, 15, np.float64), (1175, 18, np.uint8),
                                    (33, 2214, np.uint8), (1606, 9, np.uint8), (1607, 8, np.uint8), (2134, 31, np.uint8),
                                    (2135, 16, np.uint8), (2470, 33, np.uint8), (2471, 33, np.uint8), (34, 2470, np.uint8),
                                    (35, 2471, np.uint8), (64, 64, np.float64), (65, 63, np.float64), (129, 1, np.uint8)])
def test_recursive_line_lengths(gpu_lib, H, W, dt):
    img = (np.random.default_rng(H * 4096 + W).uniform(size=(H, W)) * (255 if dt == np.uint8 else 1)).astype(dt)
    _, got, sx = gpu_rec(gpu_lib, img, 4.0, 0.5)
    A, Mu, Mv, sx_ref = O.recursive_maps(img.astype(np.float64) * 0.5, 4.0)
    for g, r in zip(got, (A, Mu, Mv)):
        assert normwise(g, r) <= 1e-6
    assert sx == pytest.approx(sx_ref, rel=1e-6)


def test_recursive_pitch(gpu_lib):
    img = (np.random.default_rng(3).uniform(size=(45, 70)) < 0.4).astype(np.uint8)
    _, got, _ = gpu_rec(gpu_lib, img, 5.0, pitch=128)
    A, Mu, Mv, _ = O.recursive_maps(img.astype(np.float64), 5.0)
    for g, r in zip(got, (A, Mu, Mv)):
        assert normwise(g, r) <= 1e-6


@pytest.mark.parametrize("H,pitch,dt", [(60, 35_000_000, torch.uint8), (100, 5_000_000, torch.float32)])
def test_recursive_wide_pitch(gpu_lib, H, pitch, dt):
    """A cross-section of a large buffer: H + ceil(6 sigma) rows of the pitch pass 4 GiB, so a 32-bit row offset
    past the image would come back inside the buffer, whose other columns are not zero."""
    W, sigma = 70, 40.0
    img = np.random.default_rng(H).uniform(size=(H, W)) * 255
    img = img.astype(np.uint8) if dt == torch.uint8 else img.astype(np.float32)
    buf = torch.full((H, pitch), 255, dtype=dt, device="cuda")
    buf[:, :W] = torch.from_numpy(img).cuda()
    m = gpu_lib.precompute_recursive(buf[:, :W], sigma, scale=0.5)
    torch.cuda.synchronize()
    A, Mu, Mv, sx_ref = O.recursive_maps(img.astype(np.float64) * 0.5, sigma)
    for g, r in zip(m.planes(), (A, Mu, Mv)):
        assert normwise(g.cpu().double().numpy(), r) <= 1e-6
    assert float(m.s_x.cpu()[0]) == pytest.approx(sx_ref, rel=1e-6)


def test_fit_on_recursive_maps(gpu_lib):
    """512 x 512 shapes, M = 100, sigma = 16 (beyond the masks' radius limit).

    At this width the sweeps amplify any perturbation by about 1.15 per sweep
    (the oracle's own codebook moves by 2e-6 px after 10 sweeps and 2e-4 px
    after 40 when only its maps are rounded to FP32), so the codebook is
    compared after one sweep and after 10, with the bars of the mask path;
    D is compared over 40 sweeps."""
    case = S.config2_case(0)
    sigma = 16.0
    m, _, _ = gpu_rec(gpu_lib, case.img, sigma)
    A, Mu, Mv, _ = O.recursive_maps(case.weights, sigma)
    U, V = np.meshgrid(np.arange(512.0), np.arange(512.0), indexing="ij")
    maps = (A, U * A - Mu, V * A - Mv)  # the oracle reads B = x A - M
    for sweeps, bar in ((1, 1e-4), (10, 1e-3)):
        w, _, _ = gpu_lib.fit(m, torch.from_numpy(case.w0).cuda(), sweeps)
        torch.cuda.synchronize()
        W_ref, _, _, _ = O.fit_lattice(case.weights, case.w0, sigma, 0, sweeps, maps=maps)
        assert float(np.linalg.norm(w.cpu().double().numpy() - W_ref, axis=1).max()) <= bar
    _, tr, _ = gpu_lib.fit(m, torch.from_numpy(case.w0).cuda(), 40)
    _, tr_ref, _, _ = O.fit_lattice(case.weights, case.w0, sigma, 0, 40, maps=maps)
    assert np.abs(tr.cpu().numpy() - tr_ref).max() <= 1e-5 * max(1.0, abs(tr_ref).max())


def test_recursive_rejects(gpu_lib):
    x = torch.ones((8, 8), dtype=torch.uint8, device="cuda")
    with pytest.raises(gpu_lib.ItcError):
        gpu_lib.precompute_recursive(x, 0.3)
