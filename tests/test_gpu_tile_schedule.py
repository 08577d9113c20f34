"""The tile scan, which the automatic schedule leaves for the granule and carried scans in most calls, asked for by
name: every term count in both directions, a row of look-backs over many tiles, and the no-allocation forward's
fixed array used by launches of every kind in turn."""
import sys

import numpy as np
import pytest
import torch

from oracle import morlet_oracle as O

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _device():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2110_11866_amd  # noqa: F401
    yield


def _rel(a, b):
    return float(np.linalg.norm(np.asarray(a) - np.asarray(b)) / max(np.linalg.norm(np.asarray(b)), 1e-300))


def _say(*a):
    print("[case]", *a, flush=True)
    sys.stdout.flush()


def _noalloc(plan, x, W):
    from paper_2110_11866_amd import _abi
    _abi.morlet_forward_noalloc(plan.handle, x.data_ptr(), _abi.MORLET_F32, W.data_ptr(), torch.cuda.current_stream().cuda_stream)


@pytest.mark.parametrize("K", list(range(1, 13)))
def test_every_term_count(K):
    # as test_gpu_all_terms.py, whose calls run the granule scan
    import paper_2110_11866_amd as M
    N, sigma = 20011, 12.0
    L = max(48, K + 1)
    rng = np.random.default_rng(100 + K)
    x = rng.standard_normal(N).astype(np.float32)
    g = (rng.standard_normal(N) + 1j * rng.standard_normal(N)).astype(np.complex64)
    xt, gt = torch.from_numpy(x).cuda(), torch.from_numpy(g).cuda()
    for mode in ("sft", "asft"):
        _say("terms", K, mode)
        plan = M.MorletPlan(N, sigma, 6.0 / sigma, K, L, mode=mode).set_schedule("tiles")
        i = plan.info()
        p = O.plan_morlet(sigma, 6.0 / sigma, K, L, mode=mode, n0=i["n0"] if mode == "asft" else None, P_S=i["P_S"])
        assert _rel(plan.forward(xt).cpu().numpy(), O.forward(x.astype(np.float64), p)) <= 1e-5
        assert _rel(plan.backward(None, gt, want_params=False)[0].cpu().numpy(), O.adjoint(g.astype(np.complex128), p)) <= 1e-5
        plan = M.GaussPlan(N, sigma, K, L, mode=mode).set_schedule("tiles")
        p = O.plan_gauss(sigma, K, L, mode=mode, n0=plan.info()["n0"] if mode == "asft" else None)
        assert _rel(plan.forward(xt).cpu().numpy(), O.forward(x.astype(np.float64), p)) <= 1e-5
        gr = np.ascontiguousarray(g.real)
        assert _rel(plan.backward(None, torch.from_numpy(gr).cuda(), want_params=False)[0].cpu().numpy(), O.adjoint(gr.astype(np.complex128), p)) <= 1e-5


def test_long_row_lookback_and_repeats():
    # 257 tiles in one row; the workspace, re-armed by the kernel, gives the same bits again
    import paper_2110_11866_amd as M
    _say("long row")
    N, sigma, K, L = 1 << 20, 512.0, 5, 2048
    x = np.random.default_rng(21).standard_normal(N).astype(np.float32)
    xt = torch.from_numpy(x).cuda()
    plan = M.MorletPlan(N, sigma, 6.0 / sigma, K, L).set_schedule("tiles")
    outs = [plan.forward(xt).clone() for _ in range(3)]
    assert _rel(outs[0].cpu().numpy(), O.forward(x.astype(np.float64), O.plan_morlet(sigma, 6.0 / sigma, K, L))) <= 1e-5
    assert torch.equal(outs[0], outs[1]) and torch.equal(outs[0], outs[2])


def test_noalloc_array_in_turn():
    # tile states of a large launch, a smaller launch of other shape over them, the carried scan's sums, tiles again
    import paper_2110_11866_amd as M
    rng = np.random.default_rng(71)
    for N, sigma, K, L, mode, schedule in [(1 << 20, 64.0, 5, 160, "asft", "tiles"), (5000, 16.0, 4, 64, "sft", "tiles"),
                                           (102400, 8192.0, 6, 32768, "asft", "auto"), (70000, 30.0, 7, 90, "sft", "tiles"),
                                           (102400, 8192.0, 6, 32768, "sft", "auto"), (5000, 16.0, 4, 64, "sft", "segments")]:
        _say("noalloc", N, K, mode, schedule)
        x = torch.from_numpy(rng.standard_normal(N).astype(np.float32)).cuda()
        plan = M.MorletPlan(N, sigma, 6.0 / sigma, K, L, mode=mode).set_schedule(schedule)
        want = plan.forward(x)
        got = torch.full_like(want, float("nan"))
        _noalloc(plan, x, got)
        torch.cuda.synchronize()
        assert torch.equal(got, want)


def test_noalloc_takes_the_scan_that_fits():
    # 36 000 tiles, whose states do not fit the array; windows so long that the tile scan is the faster one
    import paper_2110_11866_amd as M
    _say("noalloc large")
    B, N, sigmas = 64, 1 << 20, [16384.0, 65536.0]
    plan = M.ScalogramPlan([N] * B, sigmas, [6.0 / s for s in sigmas], 5, 2.6, mode="asft")
    x = torch.randn(B * N, generator=torch.Generator(device="cuda").manual_seed(2), device="cuda")
    want = plan.forward(x)
    got = torch.full_like(want, float("nan"))
    _noalloc(plan, x, got)
    torch.cuda.synchronize()
    assert float((got - want).norm() / want.norm()) <= 2e-5
