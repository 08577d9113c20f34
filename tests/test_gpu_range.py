"""Inputs at the ends of float32's range through the granule and the carried scan, whose float32 products run
on bfloat16 thirds: a third that rounds past the range or vanishes below it must not show in the outputs."""
import sys

import numpy as np
import pytest
import torch

from oracle import morlet_oracle as O

pytestmark = pytest.mark.gpu
TOP = float(np.finfo(np.float32).max)
# (N, sigma, L): granule scan, carried scan
SIZES = [(4096, 20.0, 64), (60000, 6000.0, 20000)]
# as for the granule scan (2e-6) and, over long windows, the carried scan (1e-5)
TOL = {4096: 2e-6, 60000: 1e-5}


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


def _plans(kind, N, sigma, L, mode):
    import paper_2110_11866_amd as M
    if kind == "morlet":
        plan = M.MorletPlan(N, sigma, 6 / sigma, 5, L, mode=mode)
        i = plan.info()
        return plan, O.plan_morlet(sigma, 6 / sigma, 5, L, mode=mode, n0=i["n0"] if mode == "asft" else None, P_S=i["P_S"])
    plan = M.GaussPlan(N, sigma, 5, L, mode=mode)
    return plan, O.plan_gauss(sigma, 5, L, mode=mode, n0=plan.info()["n0"] if mode == "asft" else None)


@pytest.mark.parametrize("bad", [TOP, -TOP, 3.397e38])
@pytest.mark.parametrize("mode", ["sft", "asft"])
@pytest.mark.parametrize("N,sigma,L", SIZES)
def test_largest_values(N, sigma, L, mode, bad):
    # one value at the top of the range (a mask's): the outputs before its reach are what they are without
    # it, those of its window follow the oracle, in both directions and at several places of a run
    for kind in ("morlet", "gauss"):
        plan, p = _plans(kind, N, sigma, L, mode)
        n0 = plan.info()["n0"]
        x = np.random.default_rng(8).standard_normal(N).astype(np.float32)
        g = np.random.default_rng(9).standard_normal((N, 2)).astype(np.float32).view(np.complex64)[:, 0]
        g = g if kind == "morlet" else g.real.copy()
        clean = plan.forward(torch.from_numpy(x).cuda()).cpu().numpy()
        clean_g = plan.backward(None, torch.from_numpy(g).cuda(), want_params=False)[0].cpu().numpy()
        for at in (N // 2 + 7, N // 2 + 8):
            _say("largest", kind, N, mode, bad, at)
            y, h = x.copy(), g.copy()
            y[at] = bad
            h[at] = bad
            got = plan.forward(torch.from_numpy(y).cuda()).cpu().numpy()
            gx = plan.backward(None, torch.from_numpy(h).cuda(), want_params=False)[0].cpu().numpy()
            first, last = max(at + n0 - L, 0), min(at + n0 + L + 1, N)
            assert np.isfinite(got).all()
            assert _rel(got[:first], clean[:first]) <= TOL[N]
            assert _rel(got[first:last], O.forward(y.astype(np.float64), p)[first:last]) <= TOL[N]
            # the adjoint runs from the row's end: what lies past the value's reach comes first
            first, last = max(at - n0 - L, 0), min(at - n0 + L + 1, N)
            assert np.isfinite(gx).all()
            assert _rel(gx[last:], clean_g[last:]) <= TOL[N]
            assert _rel(gx[first:last], O.adjoint(h.astype(np.complex128), p)[first:last]) <= TOL[N]


@pytest.mark.parametrize("N,sigma,L", SIZES)
def test_largest_states(N, sigma, L):
    # inputs inside the range whose running sum (the constant term's state) ends within a bfloat16
    # rounding of the range's end
    plan, p = _plans("gauss", N, sigma, L, "sft")
    for at in (N // 2, N // 2 + 5):
        _say("states", N, at)
        y = np.zeros(N, np.float32)
        y[at:at + 2] = 1.6995e38
        got = plan.forward(torch.from_numpy(y).cuda()).cpu().numpy()
        assert _rel(got, O.forward(y.astype(np.float64), p)) <= TOL[N]


@pytest.mark.parametrize("scale", [1e-30, 1e-33, 1e-35, 1e-36])
@pytest.mark.parametrize("mode", ["sft", "asft"])
@pytest.mark.parametrize("N,sigma,L", SIZES)
def test_smallest_values(N, sigma, L, mode, scale):
    # a whole signal (its first part zero) near the lower end: as accurate as at any other size
    for kind in ("morlet", "gauss"):
        _say("smallest", kind, N, mode, scale)
        plan, p = _plans(kind, N, sigma, L, mode)
        x = (np.random.default_rng(8).standard_normal(N) * scale).astype(np.float32)
        x[:N // 3] = 0
        got = plan.forward(torch.from_numpy(x).cuda()).cpu().numpy()
        assert _rel(got / scale, O.forward(x.astype(np.float64), p) / scale) <= TOL[N]
        gx = plan.backward(None, torch.from_numpy(x.astype(got.dtype)).cuda(), want_params=False)[0].cpu().numpy()
        assert _rel(gx / scale, O.adjoint(x.astype(np.complex128), p) / scale) <= TOL[N]


@pytest.mark.parametrize("scale", [1e-33, 1e-35, 1e-36])
@pytest.mark.parametrize("mode", ["sft", "asft"])
@pytest.mark.parametrize("N,sigma,L", [(8192, 200.0, 600), (60000, 6000.0, 20000)])
def test_smallest_states(N, sigma, L, mode, scale):
    # a short signal near the lower end, then zeros over more than a granule: those outputs come from the state alone
    for kind in ("morlet", "gauss"):
        _say("smallest states", kind, N, mode, scale)
        plan, p = _plans(kind, N, sigma, L, mode)
        n0 = plan.info()["n0"]
        at = N // 2
        x = np.zeros(N, np.float32)
        x[at:at + 40] = np.random.default_rng(8).standard_normal(40) * scale
        got = plan.forward(torch.from_numpy(x).cuda()).cpu().numpy()
        ref = O.forward(x.astype(np.float64), p)
        seen = slice(at + n0 - L // 2, at + n0 + L // 2)
        assert _rel(got[seen] / scale, ref[seen] / scale) <= 1e-5
        gx = plan.backward(None, torch.from_numpy(x.astype(got.dtype)).cuda(), want_params=False)[0].cpu().numpy()
        ref = O.adjoint(x.astype(np.complex128), p)
        seen = slice(at - n0 - L // 2, at - n0 + L // 2)
        assert _rel(gx[seen] / scale, ref[seen] / scale) <= 1e-5
