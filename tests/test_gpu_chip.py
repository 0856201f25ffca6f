"""The team over the chip (the whole PCG loop of a mid-size 2D grid in one launch)
against the oracle and against the same passes as launches.

Shapes: the smallest grids with such a team, one to sixteen rows or columns per
tile, tiles that do not fill their threads, one and two launched tiles per member, more
row than column tiles and the reverse, and shapes just outside its limits.  A handle
that times a kernel runs the passes as launches, so the two can be compared on
one handle: the tiles' work and the order of every sum are the same, so the
results agree bit for bit.  Against the oracle: 1e-10 relative L2, the FP64 bound
of the pressure; the larger grids check the residual the solve reports (computed
from b - A x at the end) instead."""

import threading

import numpy as np
import pytest

import oracle as O

pytestmark = [pytest.mark.gpu, pytest.mark.filterwarnings("ignore::RuntimeWarning")]

TOL = 1e-10


def rel(a, b):
    return float(np.linalg.norm(np.ravel(a - b)) / np.linalg.norm(np.ravel(b)))


def fields(n, seed, a=1.0, r0=0.1):
    rng = np.random.default_rng(seed)
    shape = n[::-1]
    m = rng.uniform(-a, a, (2,) + shape)
    r = r0 * rng.uniform(0.5, 1.5, shape)
    S = rng.standard_normal(shape)
    S -= S.mean()
    return m, r, S


@pytest.fixture(scope="module")
def env():
    import torch

    from paper_2606_06720_amd import nf as NF

    T = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")
    return NF, T, torch


SHAPES = [(512, 256), (256, 512), (200, 400), (1024, 128), (128, 1024), (2048, 64), (1600, 100), (400, 256), (400, 400),
          (512, 512), (400, 1024), (512, 800), (512, 1024), (1024, 512), (800, 800), (1600, 400), (2048, 512),
          (1024, 1024), (2048, 1024)]


@pytest.mark.parametrize("n", SHAPES)
def test_chip_team_matches_oracle_and_its_passes_as_launches(env, n):
    NF, T, torch = env
    L = tuple(v / min(n) for v in n)
    m, r, S = fields(n, 53)
    small = n[0] * n[1] <= 131072
    if small:
        want, io = O.pressure_pcg(m, r, S, None, 1e-11, 4000, L)
    for dtype in (NF.NF_F64, NF.NF_F32_REFINED):
        with NF.Grid(n, L, dtype=dtype) as g:
            got = []
            for timed in (-1, 0):  # -1: the team where the grid has one; 0: passes as launches
                g.time_kernel(timed)
                print("solve", n, dtype, timed, flush=True)
                p = T(np.zeros(n[::-1]))
                rc, info = g.pressure_solve(T(m), T(r), T(S), p, rtol=1e-11, max_iter=4000)
                assert info.converged and info.true_rel_res <= 2e-11
                if small:
                    if dtype == NF.NF_F64:
                        assert abs(info.iters - io.iters) <= 1
                    assert rel(p.cpu().numpy(), want) <= TOL
                got.append((info.iters, p.cpu().numpy()))
            assert got[0][0] == got[1][0] and np.array_equal(got[0][1], got[1][1])
            g.time_kernel(-1)
            for k in (1, 2):
                p = T(np.zeros(n[::-1]))
                rc, info = g.pressure_solve(T(m), T(r), T(S), p, rtol=1e-11, max_iter=k, allow_notconv=True)
                assert rc == NF.NF_ENOTCONV and info.iters == k and not info.converged


def test_more_iterations_than_one_launch(env):
    # an ill-conditioned tensor and a tolerance that is not reached: the solve
    # goes on from one team launch to the next and stops at the cap
    NF, T, torch = env
    n = (512, 256)
    m, r, S = fields(n, 41, a=100.0, r0=1e-7)
    with NF.Grid(n, (2.0, 1.0)) as g:
        got = []
        for timed in (-1, 0):
            g.time_kernel(timed)
            p = T(np.zeros(n[::-1]))
            rc, info = g.pressure_solve(T(m), T(r), T(S), p, rtol=1e-14, max_iter=8300, allow_notconv=True)
            got.append((info.iters, p.cpu().numpy()))
        assert got[0][0] > 8192
        assert got[0][0] == got[1][0] and np.array_equal(got[0][1], got[1][1])


def test_concurrent_chip_teams_are_bitwise_sequential_runs(env):
    # four handles on four streams and threads, whose teams need the same compute units
    NF, T, torch = env
    shapes = [(512, 512), (1024, 512), (256, 256), (512, 256)]
    prm = (25.0, 1e-3, 0.75, 1e-3)
    data = [tuple(T(v) for v in fields(n, 60 + i)) for i, n in enumerate(shapes)]
    grids = [NF.Grid(n) for n in shapes]

    def go(i, out):
        m, r, S = data[i]
        mm, p = m.abs().clone(), torch.zeros_like(r)
        for _ in range(3):
            grids[i].step(*prm, mm, p, r, S, rtol=1e-10)
        out[i] = (mm, p)

    seq, par = {}, {}
    for i in range(len(shapes)):
        go(i, seq)
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream() for _ in shapes]

    def run(i):
        with torch.cuda.stream(streams[i]):
            go(i, par)

    th = [threading.Thread(target=run, args=(i,)) for i in range(len(shapes))]
    for t in th:
        t.start()
    for t in th:
        t.join()
    torch.cuda.synchronize()
    for i in range(len(shapes)):
        assert torch.equal(seq[i][0], par[i][0]) and torch.equal(seq[i][1], par[i][1])
    for g in grids:
        g.close()
