"""The FP64 gas faces' short form and the general form behind it, through the spatial operator
against the FP64 oracle, on a grid that fills no tile evenly: perturbations on both sides of
the short form's bounds (relative pressure jumps of 1/512 and 1/16), radial flows on both
sides of 0.9 sound speeds and supersonic both ways, and a gamma without a short form.  Bound:
both solvers stop at a relative change of the star pressure of 1e-12; six faces of a cell make
6e-12 of the largest face term |E| A (|v| + c), taken as 1e-11."""
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


@pytest.mark.parametrize("gamma", [1.4, 5.0 / 3.0])
@pytest.mark.parametrize("nz", [8, 1])
@pytest.mark.parametrize("amp,mach", [(1e-4, 0.0), (2e-3, 0.0), (0.05, 0.0), (0.2, 0.0),
                                      (1e-3, 0.9), (0.02, -0.9), (0.02, 1.3), (0.02, -1.3)])
def test_gas_face_ranges(rb, amp, mach, nz, gamma):
    cfg = CFG.scaled(20, 72, nz).with_(gamma=gamma)
    print(f"[gas faces] amplitude {amp} mach {mach} nz {nz} gamma {gamma:.3f}", flush=True)
    o = oracle.Oracle(cfg)
    E = o.state()
    cs, p = sound_speed(E, cfg.gamma)
    rng = np.random.default_rng(3)
    d = rng.uniform(-amp, amp, (5, *E.shape[1:]))
    rho = E[4] * (1.0 + d[4])
    v = [E[f] / E[4] + d[f] * cs for f in range(3)]
    v[0] = v[0] + mach * cs
    p = p * (1.0 + d[3])
    E = np.stack([rho * v[0], rho * v[1], rho * v[2],
                  p / (cfg.gamma - 1.0) + 0.5 * rho * (v[0] ** 2 + v[1] ** 2 + v[2] ** 2), rho])
    o.set_state(E)
    sim = rb.Sim(cfg)
    sim.set_fields(E)
    G, Go = sim.operator(), o.eval_G()
    sim.close()
    g = o.geometry()
    amax = max(g["Ar"].max(), g["Ath"].max(), g["Az"].max() if nz > 1 else 0.0)
    speed = (np.sqrt(v[0] ** 2 + v[1] ** 2 + v[2] ** 2) + cs).max()
    for f in range(5):
        mag = (rho * np.maximum(np.abs(v[f]), cs)).max() if f < 3 else np.abs(E[f]).max()
        err = np.max(np.abs(G[f] - Go[f])) / (mag * amax * speed)
        print(f"[gas faces] field {f}: err/scale {err:.2e}", flush=True)
        assert err <= 1e-11, (f, err)
