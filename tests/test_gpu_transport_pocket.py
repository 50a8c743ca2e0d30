"""Mixture-averaged transport in a single fluid cell closed in by solids and filled with one pure
species.  No face of it carries a flux, so its undefined diffusion coefficient (0/0 for a pure
species) must not enter: composition and temperature stay, the step stays finite, and every
other cell is the oracle's."""
import numpy as np
import pytest
import torch

import lbm_inputs as L
from gpu_helpers import fetch, gpu_state, make_solver, oracle_ghat, oracle_state, random_state
from oracle import step as OS

pytestmark = pytest.mark.gpu
BOUND = {"fp64": (1e-12, 1e-12), "fp32": (2e-7, 2e-6)}      # one step, as in the parity tests


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("lattice,shape", [("D2Q9", (1, 13, 70)), ("D3Q27", (7, 8, 64))])
def test_pocket_of_a_pure_species(lattice, shape, precision):
    nz, ny, nx = shape
    p = L.base_params(lattice, nx, ny, nz, physics="two_step", visc_law="const_mu", nu_ref=0.01, cs_smag=0.17,
                      thickening=2.0, chem=L.two_step_chem(B1=50.0, B2=5.0), T_ref=320.0, precision=precision,
                      weno_scale=[1630.0, 0.05, 0.22, 0.05, 0.13, 0.11], transport_model="mixture",
                      transport=L.mixture_transport(0.01),
                      face_bc=["periodic", "periodic", "wall", "wall", "periodic", "periodic"])
    ghat, scal = random_state(p, 47)
    z, y, x = nz // 2, ny // 2, 20
    solid = np.zeros(shape, bool)
    solid[max(z - 1, 0):z + 2, y - 1:y + 2, x - 1:x + 2] = True
    solid[z, y, x] = False
    scal[1:, z, y, x] = 0.0                                  # nitrogen alone
    s = make_solver(p)
    s.set_geometry(torch.from_numpy(solid.astype(np.uint8)))
    gpu_state(s, ghat, scal)
    s.step(1)
    pops, sc, _ = fetch(s)                                   # raises if the step went non-finite
    s.close()
    assert np.isfinite(pops).all() and np.array_equal(sc[1:, z, y, x], np.zeros(5))
    tg, ts = BOUND[precision]
    assert abs(sc[0, z, y, x] - scal[0, z, y, x]) <= ts * 1630.0
    # the oracle with another mixture in the pocket, which nothing outside it sees
    scal[1:, z, y, x] = scal[1:, 0, 0, 0]
    st, _ = OS.step(p, oracle_state(p, ghat, scal, solid))
    live = ~solid
    live[z, y, x] = False
    want = oracle_ghat(p, st)
    assert (np.abs(pops - want) <= tg)[:, live].all()
    ref = st["scal"].numpy()
    scale = np.maximum(np.array(p["weno_scale"][:6]).reshape(-1, 1, 1, 1), np.abs(ref))
    assert (np.abs(sc - ref) <= ts * scale)[:, live].all()
