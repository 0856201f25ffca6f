"""The two-pass PCG loop against the oracle's textbook PCG, iterate by iterate.

The loop takes its step lengths from the single-reduction recurrences, so the
first iterations (which start the recurrences) and the last ones (far below the
tolerances in use, where rounding decides) are the places where it could leave
the textbook iterates.  Iterates after one to four iterations are compared at
1e-10 relative L2 (the FP64 bound of the pressure), on grids whose row and column
tiles have remainders, a single line, or several small lines."""

import numpy as np
import pytest

import oracle as O

pytestmark = [pytest.mark.gpu, pytest.mark.filterwarnings("ignore::RuntimeWarning")]

TOL = 1e-10

SHAPES = [((8, 8), (1.0, 1.0)), ((50, 16), (1.0, 0.5)), ((64, 64), (1.0, 1.0)), ((200, 128), (1.0, 1.0)),
          ((256, 512), (1.0, 2.0)), ((800, 32), (1.0, 0.04)), ((16, 2048), (1.0 / 128, 1.0)),
          # 3D: the smallest tiles, z tiles of one and of several lines, a long row
          ((8, 8, 8), (1.0, 1.0, 1.0)), ((16, 8, 512), (1.0, 0.5, 32.0)), ((64, 32, 16), (1.0, 0.5, 0.25)),
          ((512, 8, 16), (32.0, 0.5, 1.0))]


def rel(a, b):
    return float(np.linalg.norm(np.ravel(a - b)) / np.linalg.norm(np.ravel(b)))


@pytest.mark.parametrize("n,L", SHAPES)
def test_first_iterates_and_attainable_accuracy(n, L):
    import torch

    from paper_2606_06720_amd import nf as NF

    T = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")
    rng = np.random.default_rng(41)
    shape = n[::-1]
    m = rng.uniform(-1.0, 1.0, (len(n),) + shape)
    r = rng.uniform(0.05, 0.15, shape)
    S = rng.standard_normal(shape)
    S -= S.mean()
    p0 = rng.standard_normal(shape)
    with NF.Grid(n, L) as g:
        for k in (1, 2, 3, 4):
            want, io = O.pressure_pcg(m, r, S, p0, 1e-13, k, L)
            p = T(p0)
            rc, info = g.pressure_solve(T(m), T(r), T(S), p, rtol=1e-13, max_iter=k, allow_notconv=True)
            assert info.iters == io.iters
            assert rel(p.cpu().numpy(), want) <= TOL, k
            assert abs(info.rel_res - io.rel_res) <= 1e-9 * io.rel_res
        # a tolerance below the attainable accuracy: the recurrence residual still reaches it
        want, _ = O.pressure_pcg(m, r, S, None, 1e-13, 4000, L)
        p = T(np.zeros(shape))
        rc, info = g.pressure_solve(T(m), T(r), T(S), p, rtol=1e-15, max_iter=4000)
        assert info.converged and info.true_rel_res <= 1e-11
        assert rel(p.cpu().numpy(), want) <= TOL


@pytest.mark.parametrize("n,L", [((2048, 8), (1.0, 1.0 / 256)), ((4096, 50), (1.0, 1.0 / 80)),
                                 ((16, 4096), (1.0 / 256, 1.0))])
def test_sequential_field_tiles_match_oracle(n, L):
    """Rows of 2048 and more (and FP32 columns of 4096) with one field at a time in
    LDS: the tiles a handle takes when the tuner is off."""
    import torch

    from paper_2606_06720_amd import nf as NF

    T = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")
    rng = np.random.default_rng(43)
    shape = n[::-1]
    m = rng.uniform(-1.0, 1.0, (2,) + shape)
    r = rng.uniform(0.05, 0.15, shape)
    S = rng.standard_normal(shape)
    S -= S.mean()
    want, io = O.pressure_pcg(m, r, S, None, 1e-12, 4000, L)
    NF.nf_set_autotune(0)
    try:
        for dtype in (NF.NF_F64, NF.NF_F32_REFINED):
            with NF.Grid(n, L, dtype=dtype) as g:
                p = T(np.zeros(shape))
                rc, info = g.pressure_solve(T(m), T(r), T(S), p, rtol=1e-12, max_iter=4000)
                assert info.converged
                if dtype == NF.NF_F64:
                    assert abs(info.iters - io.iters) <= 1
                assert rel(p.cpu().numpy(), want) <= TOL
    finally:
        NF.nf_set_autotune(2)
