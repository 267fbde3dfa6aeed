"""The reverse of the gas faces, short form and general form, through one recorded step: the
dot product <lam, dE> of the oracle's forward-mode derivative against <dJ/dE0, v> of the GPU
adjoint, with perturbations on both sides of the short form's bounds (relative pressure jumps
of 1/512 and 1/16) on a grid that fills no tile evenly.  Tolerance as the dot-product tests
of the whole adjoint: ten times the change of the oracle's own product when its base state
moves by 1e-14 relative, and at least 1e-10."""
import numpy as np
import pytest

import oracle
from paper_2207_04252_amd import synth
from tests.parity import sound_speed
from tests.test_gpu_adjoint import local_scale

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def rb():
    import torch
    assert torch.cuda.is_available(), "GPU test on a machine without a GPU"
    from paper_2207_04252_amd import rossbi
    rossbi.load()
    return rossbi


@pytest.mark.parametrize("nr,nth,nz", [(20, 72, 8), (9, 130, 5), (20, 72, 1)])
@pytest.mark.parametrize("amp", [1e-4, 2e-3, 0.03, 0.15])
def test_adjoint_face_ranges(rb, amp, nr, nth, nz):
    cfg = synth.C2_DISC.scaled(nr, nth, nz).with_(vortex_amp=0.0, noise_amp=0.0)
    print(f"[adjoint faces] amplitude {amp} grid {nr}x{nth}x{nz}", flush=True)
    E = oracle.Oracle(cfg).state()
    cs, p = sound_speed(E, cfg.gamma)
    rng = np.random.default_rng(11)
    d = rng.uniform(-amp, amp, (5, *E.shape[1:]))
    rho = E[4] * (1.0 + d[4])
    v = [E[f] / E[4] + d[f] * cs for f in range(3)]
    p = p * (1.0 + d[3])
    x0 = np.stack([rho * v[0], rho * v[1], rho * v[2],
                   p / (cfg.gamma - 1.0) + 0.5 * rho * (v[0] ** 2 + v[1] ** 2 + v[2] ** 2), rho])
    # (a short step: at the full one the strongest perturbations empty the thin top cells)
    o = oracle.Oracle(cfg)
    o.set_state(x0)
    dts = np.array([0.02 * o.cfl_dt()])
    sim = rb.Sim(cfg)
    sim.set_fields(x0)
    assert np.array_equal(sim.record(1, 1, dt_list=dts), dts)
    sc = local_scale(cfg, x0)
    live = np.broadcast_to(x0[4] >= 1e-2 * x0[4].max(axis=0, keepdims=True), x0.shape)
    lam = rng.uniform(-1, 1, size=x0.shape) / sc * live
    g0 = sim.adjoint(lam)[0].cpu().numpy()
    sim.close()
    w = rng.uniform(-1, 1, size=x0.shape) * sc * live
    x1 = x0 * (1 + 1e-14 * np.random.default_rng(5).uniform(-1, 1, size=x0.shape))
    st, _, dx = oracle.tangent_state(cfg, x0, w, None, dts)
    st1, _, dx1 = oracle.tangent_state(cfg, x1, w, None, dts)
    assert st == 0 and st1 == 0
    lhs, mag = float(np.sum(lam * dx)), float(np.sum(np.abs(lam * dx)))
    err = abs(lhs - float(np.sum(g0 * w))) / mag
    tol = max(1e-10, 10.0 * abs(float(np.sum(lam * dx1)) - lhs) / mag)
    print(f"[adjoint faces] rel {err:.2e} (tol {tol:.1e})", flush=True)
    assert err <= tol
