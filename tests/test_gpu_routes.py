"""The automatic schedule where windows are long against the pieces of the rows: it takes the scan whose estimated
time is least, so a call never takes a multiple of the tiles schedule's time, and both agree."""
import sys

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu
# both sides within 1e-5 of the oracle over such windows (test_gpu_carry.py)
TOL = 2e-5
# by the wrong scan these calls took 4 to 40 times the tiles schedule's time; the estimates are good to about
# 1.2, and timing to a few percent
FACTOR = 1.5


@pytest.fixture(scope="module", autouse=True)
def _device():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2110_11866_amd  # noqa: F401
    yield


def _rel(a, b):
    return float((a - b).norm() / b.norm())


def _us(call):
    for _ in range(3):
        call()
    best = float("inf")
    for _ in range(5):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        for _ in range(10):
            call()
        b.record()
        torch.cuda.synchronize()
        best = min(best, a.elapsed_time(b) * 100)
    return best


def _compare(name, plan, calls):
    auto = [(c().clone(), _us(c)) for c in calls]
    plan.set_schedule("tiles")
    for (out, us), c in zip(auto, calls):
        want, tiles = c(), _us(c)
        print("[case]", name, "auto %.1f us, tiles %.1f us" % (us, tiles), flush=True)
        sys.stdout.flush()
        assert _rel(out, want) <= TOL
        assert us <= FACTOR * tiles


@pytest.mark.parametrize("mode", ["sft", "asft"])
@pytest.mark.parametrize("lengths,widest,S,K", [([1 << 20], 131072.0, 2, 5), ([262144] * 2, 32768.0, 8, 5),
                                                ([100003, 70001, 99], 12000.0, 3, 9), ([50000] * 60, 6000.0, 1, 9)])
def test_scalograms_with_wide_windows(lengths, widest, S, K, mode):
    import paper_2110_11866_amd as M
    sig = [widest / 8 * 8 ** (i / max(S - 1, 1)) for i in range(S)][-S:] if S > 1 else [widest]
    plan = M.ScalogramPlan(lengths, sig, [6 / s for s in sig], K, 2.6 if K < 9 else 4.0, mode=mode)
    n = sum(lengths)
    x = torch.from_numpy(np.random.default_rng(1).standard_normal(n).astype(np.float32)).cuda()
    g = torch.view_as_complex(torch.from_numpy(np.random.default_rng(2).standard_normal((n * S, 2)).astype(np.float32)).cuda())
    out = torch.empty(n * S, dtype=torch.complex64, device="cuda")
    ws = plan.workspace(x.device, backward=True)
    _compare((lengths[0], S, K, mode), plan,
             [lambda: plan.forward(x, out=out, ws=ws), lambda: plan.backward(None, g, want_params=False)[0]])


@pytest.mark.parametrize("H,W,L,K", [(4000, 500, 2000, 8), (2000, 40, 1000, 12), (20000, 16, 1250, 4), (1080, 1920, 30, 4)])
def test_images_with_wide_windows(H, W, L, K):
    # down the columns every piece sums its window; between transposes the lines take the cheapest scan
    import paper_2110_11866_amd as M
    img = torch.from_numpy(np.random.default_rng(3).standard_normal((H, W)).astype(np.float32)).cuda()
    for mode in ("sft", "asft"):
        plan = M.Gauss2DPlan(H, W, L / 3.3, 2.0, K, L, max(K, 7), mode=mode)
        _compare(("image", H, W, L, K, mode), plan, [lambda: plan.forward(img), lambda: plan.backward(img)])
        gab = M.Gabor2DPlan(H, W, 3.0, 2.0, 5, L / 3.3, K, 9, L, mode=mode)
        cot = torch.view_as_complex(torch.stack([img, img.flip(0)], dim=-1).contiguous())
        _compare(("gabor", H, W, L, K, mode), gab, [lambda: gab.forward(img), lambda: gab.backward(cot)])
