"""The FP32-perturbation gas faces' short form and the general form behind it, through the
spatial operator against the FP64 oracle: perturbations from far below to above the short
form's bounds (a tenth of the background, a star pressure a quarter off), on a grid that fills
no tile evenly.  Bound: each face flux carries some fifty FP32 roundings of the perturbation
flux, at most its amplitude times the face term |E| A (|v| + c): 50 x 2^-24 = 3e-6, taken as
1e-5 of the amplitude times the largest face term."""
import numpy as np
import pytest

import oracle
from paper_2207_04252_amd import synth
from tests.parity import sound_speed

pytestmark = pytest.mark.gpu

CFG = synth.C2_DISC.scaled(20, 72, 8).with_(vortex_amp=0.0, noise_amp=0.0)


@pytest.fixture(scope="module")
def rb():
    import torch
    assert torch.cuda.is_available(), "GPU test on a machine without a GPU"
    from paper_2207_04252_amd import rossbi
    rossbi.load()
    return rossbi


@pytest.mark.parametrize("nz", [8, 1])
@pytest.mark.parametrize("amp", [1e-6, 1e-3, 0.03, 0.09, 0.11, 0.2])
def test_pert_face_amplitudes(rb, amp, nz):
    cfg = CFG.scaled(20, 72, nz)
    print(f"[pert faces] amplitude {amp} nz {nz}", flush=True)
    o = oracle.Oracle(cfg)
    E = o.state()
    cs, p = sound_speed(E, cfg.gamma)
    rng = np.random.default_rng(3)
    d = rng.uniform(-amp, amp, (5, *E.shape[1:]))
    rho = E[4] * (1.0 + d[4])
    v = [E[f] / E[4] + d[f] * cs for f in range(3)]
    p = p * (1.0 + d[3])
    E = np.stack([rho * v[0], rho * v[1], rho * v[2],
                  p / (cfg.gamma - 1.0) + 0.5 * rho * (v[0] ** 2 + v[1] ** 2 + v[2] ** 2), rho])
    o.set_state(E)
    sim = rb.Sim(cfg, precision=rb.RB_FP32_PERT)
    sim.set_fields(E)
    G, Go = sim.operator(), o.eval_G()
    resolved = sim.diagnostics().fp64_resolves
    sim.close()
    # (on so coarse a grid the thin top layers' faces see strong perturbations early)
    assert resolved == 0 if amp <= 1e-6 else resolved > 0 or amp < 0.11, resolved
    g = o.geometry()
    amax = max(g["Ar"].max(), g["Ath"].max(), g["Az"].max() if nz > 1 else 0.0)
    speed = (np.sqrt(v[0] ** 2 + v[1] ** 2 + v[2] ** 2) + cs).max()
    for f in range(5):
        mag = (rho * np.maximum(np.abs(v[f]), cs)).max() if f < 3 else np.abs(E[f]).max()
        err = np.max(np.abs(G[f] - Go[f])) / (mag * amax * speed)
        print(f"[pert faces] field {f}: err/scale {err:.2e}", flush=True)
        assert err <= 1e-5 * amp, (f, err)
