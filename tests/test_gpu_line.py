"""Lines of cells in registers (chunks of 56 cells per wavefront): the batched
tubes, split over teams of workgroups or not, at the edges of chunks and
slices, against the FP64 oracle and against each other."""
import numpy as np
import pytest

import oracle
from paper_1207_3392_amd import workloads as wl

pytestmark = pytest.mark.gpu
hydro = pytest.importorskip("paper_1207_3392_amd.hydro")


def _gpu():
    try:
        import torch
        return torch.cuda.is_available()
    except Exception:
        return False


if not _gpu():
    pytest.skip("no GPU", allow_module_level=True)

KINDS = (wl.BC_OUTFLOW, wl.BC_REFLECT, wl.BC_PERIODIC)


def tube(n, bc, seed, theta=1.4):
    pr = wl.random_smooth_patch(1, (n,), seed=seed, bc=bc, theta=theta)
    pr.bc = ((bc, bc), (0, 0), (0, 0)) if not isinstance(bc, tuple) else (bc, (0, 0), (0, 0))
    return pr


@pytest.mark.parametrize("solver", [hydro.HLL, hydro.HLLC])
def test_tubes_at_chunk_edges(solver):
    """One and two chunks, the last one of 1 .. 4 cells (copies of the far
    end, wall ghosts and wraps then reach into the chunk before it)."""
    sizes = (4, 7, 55, 56, 57, 58, 59, 60, 61, 111, 112, 113, 114, 115, 116, 120)
    probs = [tube(n, b, 10 * n + k) for n in sizes for k, b in enumerate(KINDS + ((1, 2), (2, 1)))]
    t_end = 4.0 / max(sizes) / 2.0
    B = hydro.Batch(probs)
    B.run_to(t_end, 0.4, solver)
    for i, pr in enumerate(probs):
        d = oracle.Desc.from_problem(pr, solver=solver)
        U, steps = oracle.run(d, oracle.prim_to_cons(d, pr.flat()), t_end, 0.4)
        ref = oracle.cons_to_prim(d, U)
        got = B.get_state(i, hydro.PRIMITIVE)
        assert abs(B.status(i)[0] - steps) <= 1
        assert np.max(np.abs(got - ref)) < 2e-5 * np.max(np.abs(ref)), (pr.n[0], pr.bc, np.abs(got - ref).max())
    B.close()


@pytest.mark.parametrize("bc", KINDS + ((1, 2),))
def test_shared_tubes_equal_unshared(bc):
    """A tube alone, which a team of workgroups shares from some 830 cells on,
    equals, bit for bit, the same tube among so many that none is shared, and
    (up to 1023 cells) the oracle."""
    for n in (256, 257, 370, 459, 1023, 1795, 6144):
        pr = tube(n, bc, n)
        t_end = 12.0 / n / 3.0
        one = hydro.Batch([pr])
        one.run_to(t_end, 0.4, hydro.HLLC)
        a, sa = one.get_state(0, hydro.CONSERVED), one.status(0)
        many = hydro.Batch([pr] * 700)
        many.run_to(t_end, 0.4, hydro.HLLC)
        for i in (0, 350, 699):
            assert many.status(i) == sa
            assert np.array_equal(many.get_state(i, hydro.CONSERVED), a), (n, bc, i)
        one.run_to(t_end, 0.4, hydro.HLLC)  # a replay from the new state shares again
        many.run_to(t_end, 0.4, hydro.HLLC)
        assert np.array_equal(many.get_state(5, hydro.CONSERVED), one.get_state(0, hydro.CONSERVED))
        if n <= 1023:
            d = oracle.Desc.from_problem(pr, solver=oracle.HLLC)
            U, steps = oracle.run(d, oracle.prim_to_cons(d, pr.flat()), t_end, 0.4)
            assert np.max(np.abs(a - U)) < 2e-5 * np.max(np.abs(U))
        one.close()
        many.close()


def patch_case(n, bc, solver, prec, steps, accel=0.0, check=True):
    pr = tube(n, bc, 3 * n + prec)
    pr.accel = (accel, 0.0, 0.0)
    d = oracle.Desc.from_problem(pr, solver=solver)
    p = hydro.Patch(pr, precision=prec)
    U = p.get_state(hydro.CONSERVED)
    dts = []
    for _ in range(steps):
        dts.append(oracle.cfl_dt(d, U, 0.4))
        U = oracle.step(d, U, dts[-1])
    s = np.max(np.abs(U), axis=1, keepdims=True)
    s[1] = max(s[1, 0], np.sqrt(2 * s[0, 0] * s[2, 0]))
    tol = 1e-12 if prec == 64 else 2e-5
    p.advance(steps, 0.4, solver=solver)  # dt from the device
    assert np.max(np.abs(p.get_state(hydro.CONSERVED) - U) / s) < tol, (n, bc, solver)
    assert abs(p.time() - sum(dts)) <= (1e-13 if prec == 64 else 2e-6) * sum(dts)
    nxt = oracle.cfl_dt(d, U, 0.4)
    assert abs(p.cfl_dt(0.4) - nxt) <= (1e-12 if prec == 64 else 2e-6) * nxt
    p.step(nxt, solver)  # dt from the host
    assert np.max(np.abs(p.get_state(hydro.CONSERVED) - oracle.step(d, U, nxt)) / s) < tol, (n, bc, solver)
    p.close()


@pytest.mark.parametrize("prec", [32, 64])
@pytest.mark.parametrize("solver", [hydro.HLL, hydro.HLLC])
def test_patches_at_chunk_edges(prec, solver):
    for n in (2, 3, 55, 56, 57, 60, 113, 897):
        for k, bc in enumerate(KINDS + ((1, 2),)):
            patch_case(n, bc, solver, prec, 3, accel=0.1 * k)


@pytest.mark.parametrize("prec", [32, 64])
def test_patches_around_the_longest_line(prec):
    """Patches past the longest run of steps in one launch, where the stage
    kernels take over (the two routes are compared bit for bit below)."""
    n = 5376 if prec == 32 else 3584
    for k in (0, 1):
        patch_case(n + k, wl.BC_REFLECT, hydro.HLLC, prec, 2)


def test_runs_longer_than_a_launch():
    """5001 steps in one call (more than one launch, an odd count) equal the
    same steps in several calls and as a graph; t_end stops the clock."""
    pr = tube(40, wl.BC_PERIODIC, 5)
    a, b, c = hydro.Patch(pr), hydro.Patch(pr), hydro.Patch(pr)
    a.advance(5001, 0.4)
    for k in (1, 2000, 2999, 1):
        b.advance(k, 0.4)
    c.advance_graph(5001, 0.4)
    assert np.array_equal(a.get_state(), b.get_state()) and a.time() == b.time()
    assert np.array_equal(a.get_state(), c.get_state()) and a.time() == c.time()
    assert a.cfl_dt(0.4) == b.cfl_dt(0.4) == c.cfl_dt(0.4)
    end = a.time() + 2.5 * a.cfl_dt(0.4)
    a.advance(7, 0.4, end)
    assert a.time() == pytest.approx(end, rel=1e-14)
    u = a.get_state()
    a.advance(3, 0.4, end)
    assert np.array_equal(u, a.get_state()) and a.time() == pytest.approx(end, rel=1e-14)
    for p in (a, b, c):
        p.close()


@pytest.mark.parametrize("prec", [32, 64])
@pytest.mark.parametrize("solver", [hydro.HLL, hydro.HLLC])
def test_timed_and_replayed_runs_equal_the_others(prec, solver):
    """Per-kernel timing launches the stages one by one, a graph or a plain
    call may take whole runs of steps in one launch: the same state, time and
    next CFL step, bit for bit, of every patch."""
    for n in (2, 57, 600, 2500):
        for k, bc in enumerate(KINDS + ((1, 2),)):
            pr = tube(n, bc, n + k)
            pr.accel = (0.3 * (k % 2), 0.0, 0.0)
            got = []
            for how in ("plain", "timed", "graph", "one by one"):
                p = hydro.Patch(pr, precision=prec)
                p.set_timing(how == "timed")
                if how == "graph":
                    p.advance_graph(7, 0.4, solver=solver)
                elif how == "one by one":
                    for _ in range(7):
                        p.advance(1, 0.4, solver=solver)
                else:
                    p.advance(7, 0.4, solver=solver)
                p.step(0.5 * p.cfl_dt(0.4), solver)
                got.append((p.get_state(hydro.CONSERVED), p.time(), p.cfl_dt(0.4)))
                p.close()
            for g in got[1:]:
                assert np.array_equal(g[0], got[0][0]) and g[1:] == got[0][1:], (n, bc)


def test_kernel_config_names_the_kernel_that_runs():
    def name(ndim, n, prec=32, timing=False):
        p = hydro.Patch(wl.random_smooth_patch(ndim, n, seed=1), precision=prec)
        p.set_timing(timing)
        s = p.kernel_config()
        p.close()
        return s

    for prec, t in ((32, "f32"), (64, "f64")):
        assert name(1, (600,), prec) == f"k_line<nd=1,{t}> threads=1024"
        assert name(1, (600,), prec, True) == f"k_stage<nd=1,{t},tile=64x1> zchunk=1"
        assert name(1, (9000,), prec) == f"k_stage<nd=1,{t},tile=64x1> zchunk=1"
        assert name(2, (70, 40), prec) == f"k_strip<nd=2,{t}> threads=256 rows=1"
        assert name(3, (20, 12, 9), prec).startswith(f"k_stage<nd=3,{t},tile=")


@pytest.mark.parametrize("prec", [32, 64])
def test_route_of_a_run_changes_nothing(prec):
    """Either side of the sizes and run lengths where a run of steps goes
    from one launch to the stage kernels, against the timed run (which takes
    the stage kernels): the same bits; and which of the two a size takes."""
    t = f"f{prec}"
    line, stage = f"k_line<nd=1,{t}> threads=1024", f"k_stage<nd=1,{t},tile=64x1> zchunk=1"
    names = {32: {1792: line, 2500: line, 3584: line, 3585: stage, 5376: stage},
             64: {896: line, 1792: line, 2300: stage, 3584: stage}}[prec]
    for n in (896, 897, 1406, 1408, 1792, 1793, 1960, 2070, 2200, 2252, 2254, 2300, 2500, 3583, 3584, 3585, 5376):
        pr = tube(n, wl.BC_REFLECT, n)
        a, b = hydro.Patch(pr, precision=prec), hydro.Patch(pr, precision=prec)
        b.set_timing(True)
        if n in names:
            assert a.kernel_config().startswith(names[n]), (n, a.kernel_config())
        for m in (1, 2, 3, 5, 14, 40):
            for p in (a, b):
                p.advance(m, 0.4)
        assert np.array_equal(a.get_state(), b.get_state()) and a.time() == b.time(), n
        assert a.cfl_dt(0.4) == b.cfl_dt(0.4)
        a.close()
        b.close()


def test_autotune_times_each_size_as_it_would_run():
    """Each workgroup size is tried with the split of its own number of
    workgroups: the size that autotune keeps runs within 20 % of the fastest,
    whichever size it started from (with the starting size's split for all, it
    kept 256 threads here, 1.45 times slower)."""
    a, b = tube(1700, wl.BC_OUTFLOW, 1), tube(100, wl.BC_OUTFLOW, 2)
    B = hydro.Batch([a] * 200 + [b] * 500)

    def ms(threads):
        B.set_block(threads)
        out = []
        for _ in range(3):
            for i, pr in enumerate(B.problems):
                B.set_state(i, pr.W)
            B.run_to(0.05, 0.4)
            out.append(B.last_ms())
        return min(out)

    own = {t: ms(t) for t in (256, 512, 1024)}
    for start in (256, 1024):
        B.set_block(start)
        for i, pr in enumerate(B.problems):
            B.set_state(i, pr.W)
        kept, t = B.autotune(0.05, 0.4)
        assert B.block() == kept
        assert own[kept] <= 1.2 * min(own.values()) and t <= 1.2 * min(own.values()), (start, kept, t, own)
    B.close()


def test_a_run_after_a_change_costs_little_more():
    """Setting one of many short tubes anew makes the next run order its
    queue again, on the host: a small part of the run, not several times it."""
    import time

    import torch

    pr = tube(64, wl.BC_OUTFLOW, 3)
    B = hydro.Batch([pr] * 2000)

    def best(fn):
        out = []
        for _ in range(12):
            torch.cuda.synchronize()
            t = time.perf_counter()
            fn()
            torch.cuda.synchronize()
            out.append(time.perf_counter() - t)
        return min(out)

    def again():
        B.set_state(0, pr.W)
        B.run_to(0.02, 0.4)

    plain, changed = best(lambda: B.run_to(0.02, 0.4)), best(again)
    assert changed < 3.0 * plain, (plain, changed)
    B.close()


def test_setting_a_tube_is_refused_under_capture():
    import torch

    pr = tube(100, wl.BC_OUTFLOW, 4)
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        B = hydro.Batch([pr, pr])
        before = B.get_state(0)
        x = torch.zeros(4, device="cuda")
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=s):
            x += 1.0
            with pytest.raises(hydro.HydroError):
                B.set_state(0, 2.0 * pr.W)
        g.replay()
        assert np.array_equal(B.get_state(0), before) and x.sum().item() == 4.0
        B.close()


@pytest.mark.parametrize("threads", [256, 512, 1024])
def test_teams_at_slice_edges(threads):
    """A tube that a team shares (the members that ran are asked for) equals
    the same tube on one workgroup, bit for bit, where the members' slices end
    in a chunk of 1, 2, 3 or 4 cells (copies then reach past the chunk before),
    of other counts and of all 56, for every kind of end and workgroup size."""
    ends = set()
    for k, n in enumerate((897, 898, 900, 903, 904, 1351, 1353, 5555, 5566, 5577, 5588, 5590, 6144)):
        bc = (KINDS + ((1, 2),))[k % 4]
        t_end = 12.0 / n / 3.0
        for b in (bc, wl.BC_PERIODIC):
            pr = tube(n, b, n)
            one, many = hydro.Batch([pr]), hydro.Batch([pr] * 600)
            for B in (one, many):
                B.set_block(threads)
                B.run_to(t_end, 0.4, hydro.HLLC)
            M = one.members(0)
            assert M > 1 and all(many.members(i) == 1 for i in (0, 300, 599)), (n, M)
            ends |= {(n // M + (r < n % M)) % 56 for r in range(M)}
            for i in (0, 599):
                assert many.status(i) == one.status(0)
                assert np.array_equal(many.get_state(i, hydro.CONSERVED), one.get_state(0, hydro.CONSERVED)), (n, b, M)
            one.close()
            many.close()
    assert {0, 1, 2, 3, 4} <= ends and len(ends) > 6, ends


def test_a_bad_state_in_one_share_of_a_team():
    """A negative pressure in a cell of one member's share: that tube reports
    it, the others are as in a batch without it."""
    good, bad = tube(1795, wl.BC_OUTFLOW, 5), tube(5555, wl.BC_OUTFLOW, 6)
    bad.W = np.array(bad.W, copy=True)
    bad.W[2].ravel()[3000] = -0.5
    t_end = 12.0 / 5555 / 3.0
    A, B = hydro.Batch([good, good]), hydro.Batch([good, bad, good])
    for x in (A, B):
        x.run_to(t_end, 0.4)
    assert B.members(1) > 1
    for call in (lambda: B.get_state(1), lambda: B.status(1)):
        with pytest.raises(hydro.HydroError) as err:
            call()
        assert err.value.status == hydro.HY_ESTATE
    for i, j in ((0, 0), (1, 2)):
        assert np.array_equal(A.get_state(i, hydro.CONSERVED), B.get_state(j, hydro.CONSERVED))
        assert A.status(i) == B.status(j)
    B.set_state(1, tube(5555, wl.BC_OUTFLOW, 6).W)
    B.run_to(t_end, 0.4)  # the latch is the run's
    assert B.status(1)[1] == pytest.approx(t_end, rel=1e-12)
    A.close()
    B.close()


@pytest.mark.parametrize("prec", [32, 64])
def test_a_bad_state_in_a_run_of_steps(prec):
    """A state that turns bad between the first and the last step of one
    launch is reported, by a run of steps as by the stage kernels."""
    for timing in (False, True):
        p = hydro.Patch(tube(300, wl.BC_PERIODIC, 7), precision=prec)
        p.set_timing(timing)
        p.advance(3, 0.4)
        p.get_state()
        p.step(40.0 * p.cfl_dt(0.4))
        p.advance(5, 0.4)
        for call in (p.get_state, p.time, lambda: p.cfl_dt(0.4)):
            with pytest.raises(hydro.HydroError) as err:
                call()
            assert err.value.status == hydro.HY_ESTATE
        p.set_state(p.problem.W)
        p.advance(5, 0.4)
        assert np.all(np.isfinite(p.get_state()))
        p.close()
