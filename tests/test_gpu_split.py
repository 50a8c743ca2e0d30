"""GPU tests of the step's cell kinds: the one-launch split of D2Q9 (listed boundary cells and
interior tiles), used where the tiles exceed one pass over the chip, against the one-instance
step of a small box, and the instances for domains without boundaries against the oracle.

The channel has walls in y, solid blocks, one-step chemistry, and is periodic in x: n copies
of a box side by side evolve as the box.  The box runs as one instance, the copies split.
Instances round differently: per step each is within the one-step bounds against the oracle
(FP64 1e-12, FP32 2e-7 in ghat; 1e-12, 2e-6 of each scalar's range), so after 3 steps the two
differ by at most 6 of those."""
import numpy as np
import pytest
import torch

import lbm_inputs as L
from gpu_helpers import fetch, gpu_state, make_solver, oracle_ghat, oracle_state, random_state
from oracle import step as OS

pytestmark = pytest.mark.gpu
ONE_STEP = {"fp64": (1e-12, 1e-12), "fp32": (2e-7, 2e-6)}


def _channel(nx, ny, precision):
    return L.base_params("D2Q9", nx, ny, 1, physics="one_step", visc_law="const_mu", nu_ref=0.005, prandtl=0.7,
                         thickening=2.0, cs_smag=0.17, precision=precision,
                         face_bc=["periodic", "periodic", "wall", "wall", "periodic", "periodic"],
                         weno_scale=[1700.0, 1.0], chem=[4.0, 15000.0, 300.0, 2000.0, 1.0])


@pytest.mark.parametrize("observed", [False, True])
@pytest.mark.parametrize("nx,ny,copies,precision", [
    (64, 40, 103, "fp64"),      # 64x4 tiles, 1030 of them (one pass: 1024)
    (50, 37, 143, "fp64"),      # linear tiles, the last one partly filled
    (64, 40, 206, "fp32"),      # 2060 tiles (one pass: 2048)
    (45, 33, 355, "fp32"),
])
def test_split_channel_matches_small_box(nx, ny, copies, precision, observed):
    p = _channel(nx, ny, precision)
    ghat, scal = random_state(p, seed=3, amp=0.002)
    solid = np.zeros((1, ny, nx), dtype=np.uint8)
    solid[0, ny // 3:ny // 3 + 3, 5:9] = 1
    solid[0, ny - 4:, nx - 1] = 1               # touches the wall and the periodic seam
    out = []
    for n in (1, copies):
        q = dict(p, nx=n * nx)
        s = make_solver(q)
        s.set_geometry(torch.from_numpy(np.tile(solid, (1, 1, n))))
        gpu_state(s, np.tile(ghat, (1, 1, 1, n)), np.tile(scal, (1, 1, 1, n)))
        if observed:
            s.set_statistics(1)
            s.set_probes([nx * 2 * n + 3, nx * n - 1], capacity=3)
        s.step(3)
        sums = np.array(s.step_sums())
        extra = [t.cpu().numpy() for t in s.statistics()[:2]] + [s.probes().cpu().numpy()] if observed else []
        out.append(fetch(s)[:2] + (sums / n, extra))
        s.close()
    (g0, s0, sums0, x0), (g1, s1, sums1, x1) = out
    tg, ts = ONE_STEP[precision]
    assert np.abs(g1 - np.tile(g0, (1, 1, 1, copies))).max() <= 6 * tg
    for k, span in enumerate((1700.0, 1.0)):
        assert np.abs(s1[k] - np.tile(s0[k], (1, 1, copies))).max() <= 6 * ts * span
    # the sums are FP64 sums of per-cell values that differ by the same bounds
    assert np.abs(sums1 - sums0).max() <= 6 * 6 * ts * np.abs(sums0).max()
    if observed:
        for a, b in zip(x0[:2], x1[:2]):
            assert np.abs(b - np.tile(a, (1, 1, 1, copies))).max() <= 6 * 9 * tg + 6 * ts
        assert np.abs(x0[2][:, :, 2] - x1[2][:, :, 2]).max() <= 6 * 9 * tg + 6 * ts


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("lattice,nx,ny,nz,physics", [
    ("D2Q9", 64, 4, 1, "isothermal"), ("D2Q9", 65, 5, 1, "passive"), ("D2Q9", 2, 1, 1, "isothermal"),
    ("D3Q27", 64, 4, 3, "isothermal"), ("D3Q27", 64, 8, 5, "passive"), ("D3Q27", 7, 5, 3, "passive"),
    ("D3Q27", 64, 4, 5, "two_step"), ("D3Q27", 9, 6, 5, "two_step"),
])
def test_without_boundaries_matches_oracle(lattice, nx, ny, nz, physics, precision):
    kw = {}
    if physics == "two_step":
        kw = dict(chem=L.two_step_chem(), T_ref=320.0, visc_law="const_mu",
                  weno_scale=[1630.0, 0.05, 0.22, 0.05, 0.13, 0.1])
    p = L.base_params(lattice, nx, ny, nz, physics=physics, nu_ref=0.01, cs_smag=0.17, precision=precision, **kw)
    ghat, scal = random_state(p, seed=11)
    s = make_solver(p)
    gpu_state(s, ghat, scal)
    s.step(1)
    g, sc, _ = fetch(s)
    s.close()
    st, _ = OS.run(p, oracle_state(p, ghat, scal), 1)
    tg, ts = ONE_STEP[precision]
    assert np.abs(g - oracle_ghat(p, st)).max() <= tg
    ref = st["scal"].numpy()
    for k in range(ref.shape[0]):
        assert np.abs(sc[k] - ref[k]).max() <= ts * max(np.ptp(ref[k]), np.abs(ref[k]).max())
