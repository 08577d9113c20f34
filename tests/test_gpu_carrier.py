"""The multiplication method's carrier kernels (four samples a thread) against the float64 oracle, forward and
backward: lengths around the four samples and a block's 1024, odd lengths (rows off 16 bytes), each input
type, views at any alignment."""
import sys

import numpy as np
import pytest
import torch

from oracle import morlet_oracle as O

pytestmark = pytest.mark.gpu
TOL = 1e-5   # as for the multiplication method at any length


@pytest.mark.parametrize("dtype", [torch.float32, torch.float16, torch.bfloat16])
@pytest.mark.parametrize("N", [1, 2, 3, 4, 5, 1023, 1025, 4099])
def test_lengths_types_and_views(N, dtype):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2110_11866_amd as M
    sigma, PM = 8.0, 2
    rng = np.random.default_rng(N)
    buf = torch.from_numpy(rng.standard_normal(N + 3).astype(np.float32)).cuda().to(dtype)
    gb = torch.from_numpy(rng.standard_normal((N + 1, 2)).astype(np.float32)).cuda().view(torch.complex64)[:, 0]
    for mode in ("sft", "asft"):
        plan = M.MultiplyPlan(N, sigma, 0.75, PM, mode=mode)
        i = plan.info()
        p = O.plan_multiply(sigma, 0.75, PM, i["L"], mode=mode, n0=i["n0"] if mode == "asft" else None)
        for off in (0, 3):
            print("[case]", N, dtype, mode, off, flush=True)
            sys.stdout.flush()
            x = buf[off:off + N]
            want = O.forward(x.double().cpu().numpy(), p)
            full = torch.full((N + 2,), 7.0, dtype=torch.complex64, device="cuda")
            plan.forward(x, out=full[1:N + 1])
            assert np.linalg.norm(full[1:N + 1].cpu().numpy() - want) <= TOL * np.linalg.norm(want)
            assert complex(full[0]) == 7 and complex(full[N + 1]) == 7
            g = gb[off // 3:off // 3 + N].contiguous()
            want = O.adjoint(g.cpu().numpy().astype(np.complex128), p)
            gx = plan.backward(None, g)[0].cpu().numpy()
            assert np.linalg.norm(gx - want) <= TOL * np.linalg.norm(want)
