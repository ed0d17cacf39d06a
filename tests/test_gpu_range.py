"""FP64 states far from 1.  Multiplying density and pressure by lam and
velocities by mu (pressure by lam mu^2) multiplies every term of the method by
a power of lam and mu, so a step of the scaled state is the scaled step.
Tolerance: a step's roundings, each 2^-53 of a variable's scale, 1e-13 with
room (the parity tests hold the unscaled step to the oracle)."""
import numpy as np
import pytest

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

# (lam, mu, the unscaled state's velocities times): the product of density and
# pressure leaves the range of FP64 in all but the last.  (Momenta whose square
# overflows are refused by set_state, hence the slow flow at large densities.)
SCALES = ((1e-200, 1.0, 1.0), (2.0 ** -900, 1.0, 1.0), (1e-160, 1e-40, 1.0), (1e-250, 1e30, 1.0),
          (1e157, 1.0, 1e-6), (1e-24, 1e5, 1.0))


def stepped(prob, lam, mu, slow, solver, dt, steps):
    """Two steps of dt / mu (dt > 0), or an advance of so many steps, of the
    scaled state: the conserved state scaled back, and the next CFL step."""
    W = np.array(prob.W, dtype=np.float64, copy=True)
    W[0] *= lam
    W[1:-1] *= mu * slow
    W[-1] *= lam * mu * mu
    p = hydro.Patch(prob, precision=64, set_initial=False)
    p.set_state(W)
    if dt:
        for _ in range(2):
            p.step(dt / mu, solver)
    if steps:
        p.advance(steps, 0.4, solver=solver)
    U, nxt = p.get_state(hydro.CONSERVED) / lam, p.cfl_dt(0.4) * mu
    U[1:-1] /= mu
    U[-1] /= mu * mu
    p.close()
    return U, nxt


@pytest.mark.parametrize("n", [(90,), (6000,), (70, 9), (40, 10, 9)])
@pytest.mark.parametrize("solver", [hydro.HLL, hydro.HLLC, hydro.HLLC_SWITCH])
def test_scaled_state_steps_alike(n, solver):
    for bc in (wl.BC_PERIODIC, wl.BC_REFLECT):
        prob = wl.random_smooth_patch(len(n), n, seed=len(n), bc=bc)
        for steps in (0, 3):
            base = {}
            for lam, mu, slow in SCALES:
                if slow not in base:
                    base[slow] = stepped(prob, 1.0, 1.0, slow, solver, 0.1 / max(n), steps)
                U1, dt1 = base[slow]
                s = np.max(np.abs(U1), axis=1, keepdims=True)
                s[1:-1] = np.maximum(s[1:-1], np.sqrt(2 * s[0] * s[-1]))
                U, dt = stepped(prob, lam, mu, slow, solver, 0.1 / max(n), steps)
                assert abs(dt - dt1) <= 1e-13 * dt1, (lam, mu, dt, dt1)
                assert np.all(np.abs(U - U1) <= 1e-13 * s), (lam, mu, np.abs(U - U1).max())
