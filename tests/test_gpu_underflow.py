"""Solves that run on after their residual has left the normal range.

rtol = 0 with a large iteration limit asks for exactly that: ||r||^2 loses about 20
decimal digits per hundred iterations here and reaches 1e-308 after 700 to 1700.
The iterate found by then has to stay: the call ends at the limit (or with an exactly
zero residual) and p is the solution.  One shape for each form of the FP64 loop."""

import numpy as np
import pytest

import oracle as O

pytestmark = [pytest.mark.gpu, pytest.mark.filterwarnings("ignore::RuntimeWarning")]


@pytest.mark.parametrize("n", [(64, 64), (512, 256), (1024, 1024), (256, 2048), (32, 16, 32)])
def test_residual_below_the_normal_range(n):
    import torch

    from paper_2606_06720_amd import nf as NF

    T = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")
    rng = np.random.default_rng(3)
    shape = n[::-1]
    m = T(rng.uniform(-1.0, 1.0, (len(n),) + shape))
    r = T(rng.uniform(0.05, 0.15, shape))
    S = rng.standard_normal(shape)
    S = T(S - S.mean())
    L = tuple(v / min(n) for v in n)
    with NF.Grid(n, L) as g:
        ref, p = torch.zeros_like(r), torch.zeros_like(r)
        g.pressure_solve(m, r, S, ref, rtol=1e-13)
        rc, info = g.pressure_solve(m, r, S, p, rtol=0.0, max_iter=4000, allow_notconv=True)
        assert info.iters <= 4000 and info.true_rel_res <= 1e-11
        assert float((p - ref).norm()) <= 1e-10 * float(ref.norm())
        # a source whose squares are not representable: no iteration can be taken
        rc, info = g.pressure_solve(m, r, S * 1e-162, torch.zeros_like(r), rtol=1e-10, max_iter=50, allow_notconv=True)
        assert info.iters <= 50


@pytest.mark.parametrize("n", [(64, 64), (512, 256), (1024, 1024), (256, 2048), (32, 16, 32)])
def test_refined_solve_whose_scalars_start_below_the_normal_range(n):
    # ||r||^2 of the first residual is a subnormal number, <r, M^-1 r> 0 by rounding; the
    # scaled FP32 residual is of order 1, so the corrections can still be computed
    import torch

    from paper_2606_06720_amd import nf as NF

    rng = np.random.default_rng(1)
    shape = n[::-1]
    L = tuple(v / min(n) for v in n)
    m = torch.from_numpy(rng.uniform(-1.0, 1.0, (len(n),) + shape)).to("cuda:0")
    r = torch.from_numpy(rng.uniform(0.05, 0.15, shape)).to("cuda:0")
    S = rng.standard_normal(shape)
    S = torch.from_numpy(S - S.mean()).to("cuda:0") * 1e-160
    with NF.Grid(n, L, dtype=NF.NF_F32_REFINED) as g:
        p = torch.zeros_like(r)
        rc, info = g.pressure_solve(m, r, S, p, rtol=1e-10, max_iter=500, allow_notconv=True)
        assert info.iters <= 500 and bool(torch.isfinite(p).all())
