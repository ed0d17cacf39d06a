"""The planes per workgroup that a 3D patch takes by itself: within the patch
at sizes with one chunk, several and a short last one, and the results those of
one chunk, bit for bit."""
import numpy as np
import pytest

from paper_1207_3392_amd import workloads as wl

pytestmark = pytest.mark.gpu
hydro = pytest.importorskip("paper_1207_3392_amd.hydro")


@pytest.mark.parametrize("precision", [32, 64])
@pytest.mark.parametrize("n", [(5, 6, 7), (65, 9, 17), (60, 70, 67), (130, 24, 45)])
@pytest.mark.parametrize("solver", [hydro.HLL, hydro.HLLC, hydro.HLLC_SWITCH])
def test_default_chunks(n, solver, precision):
    prob = wl.random_smooth_patch(3, n, seed=sum(n), bc=wl.BC_OUTFLOW)
    out = []
    for zchunk in (None, n[2]):
        p = hydro.Patch(prob, precision=precision)
        if zchunk:
            p.set_launch_cfg(64, 8, zchunk)
        else:
            assert 1 <= p.launch_cfg()[2] <= n[2]
        p.advance(3, 0.3, solver=solver)
        out.append(p.get_state(hydro.CONSERVED))
        p.close()
    assert np.array_equal(out[0], out[1])
