"""GPU tests of the initial state's storage rounding, the reduction of the block records at
its launch boundaries (one launch up to 4096 records of 256 cells) and the state copies."""
import numpy as np
import pytest
import torch

import lbm_inputs as L
from gpu_helpers import make_solver
from oracle import step as OS
from paper_2207_11567_amd import Solver

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lattice,nx,ny,nz", [("D2Q9", 33, 7, 1), ("D3Q27", 16, 9, 5)])
def test_fp16_initial_state_is_the_nearest_half(lattice, nx, ny, nz):
    p = L.base_params(lattice, nx, ny, nz, precision="fp16s")
    rng = np.random.default_rng(4)
    D = 2 if lattice == "D2Q9" else 3
    P = (1 + 10.0 ** rng.uniform(-9, 0, (nz, ny, nx)) * rng.choice([-1, 1], (nz, ny, nx))) / 3
    u = 10.0 ** rng.uniform(-9, -1, (D, nz, ny, nx)) * rng.choice([-1, 1], (D, nz, ny, nx))
    s = make_solver(p)
    s.init_fields(torch.from_numpy(P), torch.from_numpy(u))
    got = s.get_state()[0].cpu().numpy()
    s.close()
    ref = OS.to_storage(p, OS.init_state(p, torch.from_numpy(P), torch.from_numpy(u), None)["pops"]).numpy()
    # the FP64 values of the two sides differ by a few 1e-17: away from a tie the halves are equal
    near = ref.astype(np.float16)
    gap = np.abs(np.spacing(near).astype(np.float64))
    tie = np.abs(np.abs(ref - near.astype(np.float64)) - 0.5 * gap) < 1e-15
    assert (got == near)[~tie].all() and tie.mean() < 1e-3


@pytest.mark.parametrize("nx,ny", [(33, 7), (1024, 1024), (1025, 1024), (2048, 1100)])
def test_sums_match_the_fields(nx, ny):
    p = L.base_params("D2Q9", nx, ny, 1, physics="one_step", weno_scale=[1700.0, 1.0],
                      chem=[4.0, 15000.0, 300.0, 2000.0, 1.0])
    rng = np.random.default_rng(nx)
    P = (1 + 0.01 * rng.standard_normal((1, ny, nx))) / 3
    u = 0.05 * rng.standard_normal((2, 1, ny, nx))
    scal = np.stack([300 + 1700 * rng.random((1, ny, nx)), rng.random((1, ny, nx))])
    s = Solver(p, device="cuda:0")
    s.init_fields(torch.from_numpy(P), torch.from_numpy(u), torch.from_numpy(scal))
    f = s.fields()
    sums = np.array(f["sums"])
    dev = torch.empty(1, dtype=torch.float64, device=s.device)
    surface = s.flame_surface(300.0, 2000.0)
    assert s.flame_surface_noalloc(300.0, 2000.0, dev).item() == surface
    again = np.array(s.fields()["sums"])
    pops, sc, _ = s.get_state()
    s.close()
    rho, Ph, uu = f["rho"], f["P_h"], f["u"]
    want = [rho.sum(), Ph.sum(), (rho * uu[0]).sum(), (rho * uu[1]).sum(), torch.zeros(()),
            (0.5 * rho * (uu ** 2).sum(0)).sum(), (1 / f["scal"][0]).sum(), (rho * f["scal"][1]).sum()]
    want = np.array([float(w) for w in want])
    # FP64 sums of N terms in two orders: N eps of the sum of magnitudes at most
    scale = np.array([float(rho.sum()), float(Ph.sum())] + [float((rho * uu.abs().amax()).sum())] * 3 + list(want[5:]))
    assert (np.abs(sums - want) <= nx * ny * 2.3e-16 * np.abs(scale) + 1e-300).all()
    assert np.array_equal(sums, again)
    T = f["scal"][0]
    assert torch.equal(sc[0], T) and pops.shape == (9, 1, ny, nx)


@pytest.mark.parametrize("precision", ["fp64", "fp32", "fp16s"])
@pytest.mark.parametrize("nx,ny,nz", [(7, 5, 3), (16, 4, 4), (64, 8, 9)])
def test_state_round_trip(nx, ny, nz, precision):
    # byte counts that are and are not multiples of the copy's 16-byte words
    p = L.base_params("D3Q27", nx, ny, nz, physics="passive", precision=precision)
    s = make_solver(p)
    g = torch.Generator(device="cuda").manual_seed(1)
    pops = (0.01 * torch.randn((27, nz, ny, nx), generator=g, device="cuda")).to(s.pop_dtype)
    scal = torch.rand((1, nz, ny, nx), generator=g, device="cuda").to(s.scal_dtype)
    s.set_state(pops, scal, 5)
    a, b, step = s.get_state()
    s.close()
    assert torch.equal(a, pops) and torch.equal(b, scal) and step == 5
