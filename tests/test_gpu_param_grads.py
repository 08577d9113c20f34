"""The parameter-gradient pass against the float64 oracle: every tile shape (the moments' sums run from each
chunk's start), one and many terms, windows that put x[j - 2L] and the cotangent off 16 bytes, inputs
that are views, rows that end inside a chunk. The pass is float64 throughout, so its error is that of sums of
10^4 terms that cancel by up to 10^5."""
import sys

import numpy as np
import pytest
import torch

from oracle import morlet_oracle as O

pytestmark = pytest.mark.gpu
TOL = 1e-8


@pytest.mark.parametrize("tile", [4, 8, 16, 32])
@pytest.mark.parametrize("K", [1, 5, 6, 12])
@pytest.mark.parametrize("L", [40, 41, 63])
def test_tiles_terms_and_alignments(tile, K, L):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2110_11866_amd as M
    sigma = 17.0
    for N in (9001, 37):
        rng = np.random.default_rng(N + K + L)
        x = torch.from_numpy(rng.standard_normal(N + 1).astype(np.float32)).cuda()[1:]
        xd = x.double().cpu().numpy()
        for kind in ("morlet", "gauss"):
            for mode in ("sft", "asft"):
                print("[case]", tile, K, L, N, kind, mode, flush=True)
                sys.stdout.flush()
                if kind == "morlet":
                    plan = M.MorletPlan(N, sigma, 6 / sigma, K, L, mode=mode)
                    i = plan.info()
                    p = O.plan_morlet(sigma, 6 / sigma, K, L, mode=mode, n0=i["n0"] if mode == "asft" else None, P_S=i["P_S"])
                    # the cotangent of sum w |W|^2: one that the gradient does not average out of
                    g = (2 * rng.uniform(size=N) * O.forward(xd, p)).astype(np.complex64)
                    gt = torch.from_numpy(np.concatenate([g[:1], g])).cuda()[1:]
                else:
                    plan = M.GaussPlan(N, sigma, K, L, mode=mode)
                    p = O.plan_gauss(sigma, K, L, mode=mode, n0=plan.info()["n0"] if mode == "asft" else None)
                    g = (2 * rng.uniform(size=N) * O.forward(xd, p).real).astype(np.float32)
                    gt = torch.from_numpy(np.concatenate([g[:1], g])).cuda()[1:]
                plan.set_tile(tile)
                got = plan.backward(x, gt)[1].cpu().numpy()
                want = O.param_grads(xd, g.astype(np.complex128), p)
                size = np.abs(want).max() + 1e-30
                assert np.abs(got - want).max() <= TOL * size, (got, want)


@pytest.mark.parametrize("tile", [4, 8, 32])
@pytest.mark.parametrize("K", [2, 3, 4, 7, 8, 9, 10, 11])
def test_terms_between_at_every_tile(tile, K):
    # the other term counts, each its own kernels, with float32 and (at tile 32, where the inputs are loaded
    # again) 16-bit inputs
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    test_tiles_terms_and_alignments(tile, K, 41)
    import paper_2110_11866_amd as M
    N, sigma, L = 9001, 17.0, 41
    rng = np.random.default_rng(K)
    for dtype in (torch.float16, torch.bfloat16) if tile == 32 else ():
        x = torch.from_numpy(rng.standard_normal(N + 1).astype(np.float32)).cuda().to(dtype)[1:]
        xd = x.double().cpu().numpy()
        for mode in ("sft", "asft"):
            print("[case]", tile, K, dtype, mode, flush=True)
            sys.stdout.flush()
            plan = M.MorletPlan(N, sigma, 6 / sigma, K, L, mode=mode).set_tile(tile)
            i = plan.info()
            p = O.plan_morlet(sigma, 6 / sigma, K, L, mode=mode, n0=i["n0"] if mode == "asft" else None, P_S=i["P_S"])
            g = (2 * rng.uniform(size=N) * O.forward(xd, p)).astype(np.complex64)
            got = plan.backward(x, torch.from_numpy(g).cuda())[1].cpu().numpy()
            want = O.param_grads(xd, g.astype(np.complex128), p)
            assert np.abs(got - want).max() <= TOL * (np.abs(want).max() + 1e-30), (got, want)
