"""The small-grid team (the whole PCG loop of a grid of up to 65536 points in one
launch) against the oracle and against the same passes as launches.

Shapes: the smallest grids, one column or one row per member, odd half lengths,
radix-5 lengths, partly filled teams, the largest tiles, and shapes just outside
the team's limits.  A handle that times a kernel runs the passes as launches of
their own, so the two can be compared on one handle: the members' work and the
order of every sum are the same, so the results agree bit for bit.  Against the
oracle: 1e-10 relative L2, the FP64 bound of the pressure."""

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


SHAPES = [(8, 8), (16, 8), (8, 1024), (50, 50), (50, 64), (64, 50), (100, 32), (128, 256), (200, 200), (256, 256),
          (400, 128), (512, 64), (64, 512), (800, 64), (1024, 64), (64, 1024), (1600, 32), (2048, 32), (32, 2048),
          (4096, 16), (256, 400)]


@pytest.mark.parametrize("n", SHAPES)
def test_team_matches_oracle_and_its_passes_as_launches(env, n):
    NF, T, torch = env
    L = tuple(v / min(n) for v in n)
    m, r, S = fields(n, 47)
    want, io = O.pressure_pcg(m, r, S, None, 1e-11, 4000, L)
    for dtype in (NF.NF_F64, NF.NF_F32_REFINED):
        with NF.Grid(n, L, dtype=dtype) as g:
            got = []
            for timed in (-1, 0):  # -1: the team where the grid has one; 0: passes as launches
                g.time_kernel(timed)
                p = T(np.zeros(n[::-1]))
                rc, info = g.pressure_solve(T(m), T(r), T(S), p, rtol=1e-11, max_iter=4000)
                assert info.converged and info.true_rel_res <= 2e-11
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
    # an ill-conditioned tensor: about 9600 iterations, more than two team launches
    NF, T, torch = env
    n = (64, 64)
    m, r, S = fields(n, 41, a=100.0, r0=1e-6)
    with NF.Grid(n) as g:
        its = []
        for timed in (-1, 0):
            g.time_kernel(timed)
            p = T(np.zeros(n[::-1]))
            rc, info = g.pressure_solve(T(m), T(r), T(S), p, rtol=1e-10, max_iter=40000)
            assert info.converged and info.true_rel_res <= 1e-8
            its.append(info.iters)
        assert min(its) > 8192
        assert its[0] == its[1]


def test_concurrent_teams_are_bitwise_sequential_runs(env):
    # ten handles (more than there are XCDs) on ten streams and threads
    NF, T, torch = env
    shapes = [(64, 64), (128, 128), (256, 256), (200, 100), (64, 32), (256, 128), (128, 64), (100, 100), (512, 64),
              (256, 256)]
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
        # also where a team could not form in time and left its solve to launches
        assert torch.equal(seq[i][0], par[i][0]) and torch.equal(seq[i][1], par[i][1])
    for g in grids:
        g.close()
