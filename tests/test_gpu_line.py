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
    """A tube that a team of workgroups shares equals, bit for bit, the same
    tube among so many that none is shared, at slices whose last chunk has 1
    to 4 cells and others."""
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

