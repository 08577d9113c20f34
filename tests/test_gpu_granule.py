"""The granule scan (the automatic schedule's forward and adjoint) against the float64 oracle at the
sizes where it can go wrong: rows around a granule (256 positions) and a run (16), pieces that start
inside and past the first window, outputs that start off a 128-byte line, every slot count of the
states, windows longer than the row, and non-finite inputs."""
import sys

import numpy as np
import pytest
import torch

from oracle import morlet_oracle as O

pytestmark = pytest.mark.gpu
# float32 outputs from float64 states: the K-term products round at 2^-24 of the terms, which exceed
# the result by less than 30 in these configurations
TOL = 2e-6


@pytest.fixture(scope="module", autouse=True)
def _device():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2110_11866_amd  # noqa: F401
    yield


def _rel(a, b):
    return float(np.linalg.norm(a - b) / max(np.linalg.norm(b), 1e-300))


def _say(*a):
    print("[case]", *a, flush=True)
    sys.stdout.flush()


@pytest.mark.parametrize("K", [1, 4, 5, 8, 9, 12])
@pytest.mark.parametrize("N", [1, 15, 16, 17, 255, 256, 257, 4095, 5003])
def test_slots_and_lengths(N, K):
    import paper_2110_11866_amd as M
    sigma, L = 11.0, 40
    x = np.random.default_rng(N + K).standard_normal(N).astype(np.float32)
    xt = torch.from_numpy(x).cuda()
    for mode in ("sft", "asft"):
        _say("slots", N, K, mode)
        plan = M.MorletPlan(N, sigma, 6 / sigma, K, L, mode=mode)
        info = plan.info()
        p = O.plan_morlet(sigma, 6 / sigma, K, L, mode=mode, n0=info["n0"] if mode == "asft" else None, P_S=info["P_S"])
        assert _rel(plan.forward(xt).cpu().numpy(), O.forward(x.astype(np.float64), p)) <= TOL
        g = np.random.default_rng(N).standard_normal((N, 2)).astype(np.float32).view(np.complex64)[:, 0]
        gx, _ = plan.backward(None, torch.from_numpy(g).cuda(), want_params=False)
        assert _rel(gx.cpu().numpy(), O.adjoint(g.astype(np.complex128), p)) <= TOL


@pytest.mark.parametrize("off", [0, 1, 3, 15, 16, 31])
@pytest.mark.parametrize("dtype", [torch.float32, torch.float16, torch.bfloat16])
def test_unaligned_views(off, dtype):
    # inputs and outputs that are views: any sample alignment, any output line offset
    import paper_2110_11866_amd as M
    N, sigma, K, L = 3001, 37.0, 5, 97
    buf = torch.from_numpy(np.random.default_rng(off).standard_normal(N + 64).astype(np.float32)).cuda().to(dtype)
    x = buf[off:off + N]
    xd = x.double().cpu().numpy()
    for kind in ("morlet", "gauss"):
        _say("views", off, dtype, kind)
        if kind == "morlet":
            plan = M.MorletPlan(N, sigma, 6 / sigma, K, L, mode="asft")
            p = O.plan_morlet(sigma, 6 / sigma, K, L, mode="asft", n0=plan.info()["n0"], P_S=plan.info()["P_S"])
        else:
            plan = M.GaussPlan(N, sigma, K, L, mode="asft")
            p = O.plan_gauss(sigma, K, L, mode="asft", n0=plan.info()["n0"])
        full = torch.full((N + 64,), 7.0, dtype=torch.complex64 if kind == "morlet" else torch.float32, device="cuda")
        plan.forward(x, out=full[off:off + N])
        torch.cuda.synchronize()
        got = full.cpu().numpy()
        assert _rel(got[off:off + N], O.forward(xd, p)) <= TOL
        assert (got[:off] == 7).all() and (got[off + N:] == 7).all()


@pytest.mark.parametrize("mode", ["sft", "asft"])
def test_pieces_and_windows(mode):
    # 70 001 samples in several pieces: windows shorter than a piece, of several pieces, and longer
    # than the row
    import paper_2110_11866_amd as M
    N = 70001
    x = np.random.default_rng(3).standard_normal(N).astype(np.float32)
    xt = torch.from_numpy(x).cuda()
    for sigma, L in [(5.0, 13), (300.0, 901), (3000.0, 9001), (30000.0, 90001)]:
        _say("pieces", mode, sigma, L)
        plan = M.MorletPlan(N, sigma, 6 / sigma, 6, L, mode=mode)
        info = plan.info()
        p = O.plan_morlet(sigma, 6 / sigma, 6, L, mode=mode, n0=info["n0"] if mode == "asft" else None, P_S=info["P_S"])
        assert _rel(plan.forward(xt).cpu().numpy(), O.forward(x.astype(np.float64), p)) <= 1e-5


@pytest.mark.parametrize("bad", [float("inf"), float("-inf"), float("nan")])
def test_non_finite_input_reaches_no_earlier_output(bad):
    # output n reads inputs up to n - n0 + L: everything before stays what it is without the bad one
    import paper_2110_11866_amd as M
    N, sigma, K, L = 4096, 20.0, 5, 64
    x = np.random.default_rng(8).standard_normal(N).astype(np.float32)
    for at in (900, 1007, 1008, 2500):
        for plan in (M.MorletPlan(N, sigma, 6 / sigma, K, L, mode="asft"), M.GaussPlan(N, sigma, K, L)):
            _say("non-finite", bad, at, plan.kind)
            clean = plan.forward(torch.from_numpy(x).cuda()).cpu().numpy()
            y = x.copy()
            y[at] = bad
            got = plan.forward(torch.from_numpy(y).cuda()).cpu().numpy()
            first = at + plan.info()["n0"] - L
            assert np.isfinite(got[:first]).all()
            assert _rel(got[:first], clean[:first]) <= TOL
            assert not np.isfinite(got[first:first + 2 * L + 1]).any()


@pytest.mark.parametrize("H,W", [(1, 1), (15, 63), (16, 64), (17, 65), (33, 130), (200, 31), (5, 300)])
@pytest.mark.parametrize("K", [4, 6, 12])
def test_columns(H, W, K):
    # the image filters' second axis: rows around a run, columns around a wave's 64, both directions
    import paper_2110_11866_amd as M
    img = np.random.default_rng(H * W + K).standard_normal((H, W)).astype(np.float32)
    xt = torch.from_numpy(img).cuda()
    for mode in ("sft", "asft"):
        _say("columns", H, W, K, mode)
        plan = M.Gauss2DPlan(H, W, 5.0, 4.0, K, 19, 15, mode=mode)
        px, py = (O.plan_gauss(s, K, L, mode=mode, n0=plan.axis_info(a)["n0"] if mode == "asft" else None)
                  for a, s, L in ((0, 4.0, 15), (1, 5.0, 19)))
        assert _rel(plan.forward(xt).cpu().numpy(), O.gauss_smooth_2d(img, px, py)) <= TOL
        want = np.stack([O.adjoint(img[:, c].astype(np.complex128), py) for c in range(W)], axis=1)
        want = np.stack([O.adjoint(r.astype(np.complex128), px) for r in want])
        assert _rel(plan.backward(xt).cpu().numpy(), want) <= TOL
        gab = M.Gabor2DPlan(H, W, 4.0, 1.2, K, 5.0, 4, 15, 19, mode=mode)
        gx, gy = gab.axis_info(0), gab.axis_info(1)
        px = O.plan_morlet(4.0, 1.2, K, 15, mode=mode, n0=gx["n0"] if mode == "asft" else None)
        py = O.plan_gauss(5.0, 4, 19, mode=mode, n0=gy["n0"] if mode == "asft" else None)
        assert _rel(gab.forward(xt).cpu().numpy(), O.gabor_2d(img, px, py)) <= TOL
        g = np.random.default_rng(K).standard_normal((H, W, 2)).astype(np.float32).view(np.complex64)[..., 0]
        assert _rel(gab.backward(torch.from_numpy(g).cuda()).cpu().numpy(), O.gabor_2d_adjoint(g, px, py)) <= TOL


def test_columns_in_pieces_and_non_finite():
    # 900 rows in several pieces; an infinite pixel reaches no row before its window
    import paper_2110_11866_amd as M
    H, W, L = 900, 70, 54
    img = np.random.default_rng(4).standard_normal((H, W)).astype(np.float32)
    plan = M.Gauss2DPlan(H, W, 16.0, 2.0, 4, L, 7, mode="sft")
    px, py = O.plan_gauss(2.0, 4, 7), O.plan_gauss(16.0, 4, L)
    clean = plan.forward(torch.from_numpy(img).cuda()).cpu().numpy()
    assert _rel(clean, O.gauss_smooth_2d(img, px, py)) <= TOL
    for at in (400, 415, 416):
        bad = img.copy()
        bad[at, 33] = np.inf
        got = plan.forward(torch.from_numpy(bad).cuda()).cpu().numpy()
        assert np.array_equal(got[:at - L, :], clean[:at - L, :]) or _rel(got[:at - L], clean[:at - L]) <= TOL
        assert not np.isfinite(got[at - L:at + L + 1, 33]).any()


@pytest.mark.parametrize("W", [31, 32, 33, 97])
@pytest.mark.parametrize("K", [4, 9])
def test_columns_around_a_waves_width(W, K):
    # a wave of the column scan takes 32 columns, two a lane
    test_columns(40, W, K)
