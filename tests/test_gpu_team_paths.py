"""Which form of the PCG loop runs, and the ways between the forms.

The tests of the one-launch loops compare them bitwise with the same passes as launches;
here it is the handle's own record that says that a team formed for the shapes that
have one (and that none is tried for shapes outside the limits).  Formation that gives
up is forced from the host by a launch with too few workgroups, at the start of a
loop and where a loop of more than 4096 iterations goes on from one team launch to the
next.  A handle that times a kernel runs launches only and gives the expected bits."""

import threading
import time

import numpy as np
import pytest

pytestmark = [pytest.mark.gpu, pytest.mark.filterwarnings("ignore::RuntimeWarning")]

CHUNK = 4096  # iterations per team launch


def fields(n, seed, a=1.0, r0=0.1):
    import torch

    rng = np.random.default_rng(seed)
    shape = n[::-1]
    m = rng.uniform(-a, a, (2,) + shape)
    r = r0 * rng.uniform(0.5, 1.5, shape)
    S = rng.standard_normal(shape)
    S -= S.mean()
    return tuple(torch.from_numpy(v).to("cuda:0") for v in (m, r, S))


def box(n):
    return tuple(v / min(n) for v in n)


def solve(g, m, r, S, **kw):
    import torch

    p = torch.zeros_like(r)
    rc, info = g.pressure_solve(m, r, S, p, allow_notconv=True, **kw)
    return info, p


XCD = [(8, 8), (50, 50), (64, 32), (200, 200), (256, 256), (2048, 32), (64, 1024)]
CHIP = [(512, 256), (200, 400), (2048, 64), (128, 1024), (512, 512), (1600, 400), (800, 800), (1024, 1024),
        (256, 400)]
NONE = [(4096, 16), (32, 2048), (2048, 1024), (100, 800)]


@pytest.mark.parametrize("n", XCD + CHIP + NONE)
def test_form_of_the_loop(n):
    from paper_2606_06720_amd import nf as NF

    kind = 1 if n in XCD else (2 if n in CHIP else 0)
    m, r, S = fields(n, 5)
    for dtype in (NF.NF_F64, NF.NF_F32_REFINED):
        with NF.Grid(n, box(n), dtype=dtype) as g:
            assert g.team()["kind"] == kind and (g.team()["members"] > 0) == (kind > 0)
            info, p = solve(g, m, r, S, rtol=1e-10)
            assert info.converged
            t = g.team()
            assert t["missed"] == 0
            if kind:
                assert t["formed"] >= 1
            else:
                assert t["formed"] == 0 and t["as_launches"] >= 1
            g.time_kernel(0)
            solve(g, m, r, S, rtol=1e-10)
            assert g.team()["formed"] == t["formed"]  # timed handles run launches


# row pass (rows, threads) and column pass (columns, threads) as launches, FP64
TILES = [((64, 64), (2, 64, 1, 64)), ((256, 256), (8, 512, 4, 512)), ((512, 512), (2, 256, 1, 256)),
         ((256, 512), (4, 256, 1, 256)), ((1024, 1024), (4, 512, 1, 256))]


@pytest.mark.parametrize("n,want", TILES)
def test_tiles_in_use(n, want):
    from paper_2606_06720_amd import nf as NF

    with NF.Grid(n) as g:
        t = g.team()
        assert tuple(t[k] for k in ("row_rows", "row_threads", "col_cols", "col_threads")) == want
        g.set_tiles(1, 1, 1)  # the untuned passes from here on
        t, tun = g.team(), g.tuning()
        assert t["kind"] == 0
        assert t["row_rows"] == tun["flux_rows"] and t["col_cols"] == tun["update_cols"]
        assert t["row_threads"] == tun["flux_threads"] and t["col_threads"] == tun["update_threads"]


@pytest.mark.parametrize("n", [(64, 64), (512, 256), (1024, 1024)])
def test_formation_that_gives_up(n):
    import torch

    from paper_2606_06720_amd import nf as NF

    m, r, S = fields(n, 6)
    for dtype in (NF.NF_F64, NF.NF_F32_REFINED):
        with NF.Grid(n, box(n), dtype=dtype) as g:
            _, want = solve(g, m, r, S, rtol=1e-10)
            formed = g.team()["formed"]
            g.team_force(NF.NF_FORCE_MISS, 0)
            _, p = solve(g, m, r, S, rtol=1e-10)
            assert g.team()["missed"] == 1
            assert torch.equal(p, want)
            _, p = solve(g, m, r, S, rtol=1e-10)
            assert g.team()["missed"] == 1 and g.team()["formed"] > formed
            assert torch.equal(p, want)
            with pytest.raises(NF.NfError):
                g.team_force(9, 0)


@pytest.mark.parametrize("n", [(64, 64), (512, 256), (1024, 1024)])
def test_loops_of_more_than_one_launch(n):
    import torch

    from paper_2606_06720_amd import nf as NF

    # ill-conditioned, so that the loop reaches its limit; in FP32 the first correction
    # does if it is asked for a reduction that it cannot have by then
    m, r, S = fields(n, 41, a=100.0, r0=1e-7)
    kw = dict(rtol=1e-14, max_iter=CHUNK + 200)
    for dtype in (NF.NF_F64, NF.NF_F32_REFINED):
        with NF.Grid(n, box(n), dtype=dtype) as g:
            if dtype == NF.NF_F32_REFINED:
                g.set_inner_tolerance(1e-30)
            g.time_kernel(0)
            info, want = solve(g, m, r, S, **kw)
            assert info.iters == kw["max_iter"] and g.team()["formed"] == 0
            g.time_kernel(-1)
            info, p = solve(g, m, r, S, **kw)
            assert info.iters == kw["max_iter"] and g.team()["formed"] == 2
            assert torch.equal(p, want)
            # the second launch of the loop gives up: launches go on from its state
            g.team_force(NF.NF_FORCE_MISS, 1)
            info, p = solve(g, m, r, S, **kw)
            assert info.iters == kw["max_iter"] and g.team()["formed"] == 3 and g.team()["missed"] == 1
            assert torch.equal(p, want)


@pytest.mark.parametrize("n", [(64, 64), (512, 256)])
def test_misses_do_not_end_the_use_of_teams(n):
    import torch

    from paper_2606_06720_amd import nf as NF

    m, r, S = fields(n, 8)
    with NF.Grid(n, box(n)) as g:

        def go(miss=False):
            if miss:
                g.team_force(NF.NF_FORCE_MISS, 0)
            before = g.team()
            _, p = solve(g, m, r, S, rtol=1e-10)
            return {k: v - before[k] for k, v in g.team().items()}, p

        did, want = go()
        assert did["formed"] == 1
        # misses with a formed team between them: the next loop is tried again
        for _ in range(3):
            did, p = go(miss=True)
            assert did["missed"] == 1 and torch.equal(p, want)
            did, p = go()
            assert did["formed"] == 1 and torch.equal(p, want)
        # two in a row: 64 loops as launches, then teams again
        go(miss=True)
        go(miss=True)
        assert g.team()["pause"] == 64
        for _ in range(64):
            did, p = go()
            assert did["as_launches"] == 1 and did["formed"] == 0
        assert torch.equal(p, want)
        did, p = go()
        assert did["formed"] == 1 and torch.equal(p, want)


@pytest.mark.parametrize("n", [(8, 8), (64, 64), (256, 256), (512, 256), (1024, 1024)])
def test_member_that_stops_waiting_at_the_last_barrier(n):
    # the first member passes that barrier and finds the solve stopped; the others have
    # left without their part of the solution
    import torch

    from paper_2606_06720_amd import nf as NF

    m, r, S = fields(n, 10)
    for dtype in (NF.NF_F64, NF.NF_F32_REFINED):
        with NF.Grid(n, box(n), dtype=dtype) as g:
            info, want = solve(g, m, r, S, rtol=1e-10, max_iter=5)
            assert info.iters == 5
            g.team_force(NF.NF_FORCE_LOSE, 4)
            with pytest.raises(NF.NfError) as e:
                solve(g, m, r, S, rtol=1e-10, max_iter=5)
            assert e.value.code == NF.NF_EDEVICE
            info, p = solve(g, m, r, S, rtol=1e-10, max_iter=5)
            assert info.iters == 5 and torch.equal(p, want)


def test_no_team_over_the_chip_beside_an_ensemble():
    import torch

    from paper_2606_06720_amd import nf as NF

    m, r, S = fields((512, 256), 9)
    shapes = [(64, 64), (128, 64)]
    data = [fields(n, 20 + i) for i, n in enumerate(shapes)]
    with NF.Grid((512, 256), (2.0, 1.0)) as g, NF.Batch(shapes) as b:
        b.set_partitions(1)
        _, want = solve(g, m, r, S, rtol=1e-10)
        assert g.team()["formed"] == 1

        def ensemble():
            with torch.cuda.stream(torch.cuda.Stream()):
                b.run([(25.0, 1e-3, 0.75)] * 2, 1e-3, 1500, [d[0].abs() for d in data],
                      [torch.zeros_like(d[1]) for d in data], [d[1] for d in data], [d[2] for d in data])

        torch.cuda.synchronize()
        th = threading.Thread(target=ensemble)
        th.start()
        t0 = time.time()
        while g.team()["as_launches"] == 0 and time.time() - t0 < 1.0:
            _, p = solve(g, m, r, S, rtol=1e-10)
        before = g.team()
        for _ in range(10):
            _, p = solve(g, m, r, S, rtol=1e-10)
            assert torch.equal(p, want)
        after, alive = g.team(), th.is_alive()
        th.join()
        assert alive, "the ensemble ended before the solves"
        assert after["as_launches"] == before["as_launches"] + 10 and after["formed"] == before["formed"]
        _, p = solve(g, m, r, S, rtol=1e-10)
        assert torch.equal(p, want) and g.team()["formed"] == after["formed"] + 1
