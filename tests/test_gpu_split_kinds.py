"""GPU tests of the one-launch split of D2Q9 (listed boundary cells beside interior tiles)
against the oracle, one step from a random state, for every kind of instance it selects: walls,
inlet and outlet, solids, one- and two-step chemistry, mixture transport, BGK, the three
storage precisions, observables, cached pulls (population copies over 256 MB).

A channel periodic in x made of n copies of a box evolves as the box does, so the oracle
steps the box.  Bounds per step as in the one-step parity tests: ghat 1e-12 (FP64), 2e-7
(FP32), plus half an FP16 ulp where that is the storage; scalars 1e-12 and 2e-6 of the larger of
range and value.  A sum over the cells is bounded by its own terms: each term passes through
fewer than 64 roundings of the compute precision's epsilon, at the magnitude below, and P_h
carries the temperature's bound through Lambda."""
import ctypes

import numpy as np
import pytest
import torch

import lbm_inputs as L
from gpu_helpers import make_solver, oracle_ghat, oracle_state, random_state
from oracle import step as OS
from paper_2207_11567_amd import _capi as C

pytestmark = pytest.mark.gpu
BOUND = {"fp64": (1e-12, 1e-12, 2.3e-16), "fp32": (2e-7, 2e-6, 6e-8), "fp16s": (2e-7, 2e-6, 6e-8)}
WALLS = ["periodic", "periodic", "wall", "wall", "periodic", "periodic"]
OPEN = ["periodic", "periodic", "inlet", "outlet", "periodic", "periodic"]


def _params(nx, ny, physics, precision, faces, **kw):
    yf, yo, _ = L.fresh_ch4_air(0.83)
    two = physics in ("two_step", "mixture")
    p = L.base_params("D2Q9", nx, ny, 1, physics="two_step" if two else "one_step", precision=precision, nu_ref=0.01,
                      visc_law="const_mu", prandtl=0.7, thickening=2.0, cs_smag=0.17, face_bc=faces, omega_bulk=1.2,
                      T_ref=320.0 if two else 300.0, inlet_T=320.0 if two else 300.0, inlet_u=[0.02, 0.03, 0.0],
                      inlet_Y=[yf, yo] + [0.0] * 6 if two else [1.0] + [0.0] * 7, outlet_P=1.001 / 3.0,
                      weno_scale=[1630.0, 0.05, 0.22, 0.05, 0.13, 0.11, 1.0, 1.0] if two else [1700.0] + [1.0] * 7,
                      chem=L.two_step_chem(B1=50.0, B2=5.0) if two else [4.0, 15000.0, 300.0, 2000.0, 1.0])
    if physics == "mixture":
        p.update(transport_model="mixture", transport=L.mixture_transport(0.01))
    p.update(kw)
    return p


def _solids(nx, ny):
    solid = np.zeros((1, ny, nx), dtype=np.uint8)
    solid[0, ny // 3:ny // 3 + 3, 5:9] = 1
    solid[0, ny // 2:ny // 2 + 4, nx - 1] = 1       # touches the seam between two copies
    return solid


def _check(p, ghat, scal, solid, copies, observed):
    """One step of `copies` copies of the box against the oracle's box."""
    nx, ny, N = p["nx"], p["ny"], p["nx"] * p["ny"]
    prec = p["precision"]
    tg, ts, eps = BOUND[prec]
    s = make_solver(dict(p, nx=copies * nx))
    assert s.N // 256 > (1024 if prec == "fp64" else 2048)        # more than one pass over the chip
    s.set_geometry(torch.from_numpy(solid).cuda().tile((1, 1, copies)))
    s.set_state(torch.from_numpy(ghat).to("cuda", s.pop_dtype).tile((1, 1, 1, copies)),
                torch.from_numpy(scal).to("cuda", s.scal_dtype).tile((1, 1, 1, copies)), 0)
    cells = [3 + copies * nx * 2, nx * (copies // 2) - 2 + copies * nx * (ny // 2), copies * nx * (ny - 1)]
    if observed:
        s.set_statistics(1)
        s.set_probes(cells, capacity=1)
    s.step(1)
    pops, sc, _ = s.get_state()
    sums = np.array(s.step_sums()) / copies

    state = oracle_state(p, ghat, scal, solid)
    P_o, rho_o, u_o, _, sums_o = OS.fields(p, state)
    st, _ = OS.step(p, state)
    fluid = torch.from_numpy(solid == 0)[0].cuda()[:, None, :]    # [ny, 1, nx]

    def off(got, want, bound):
        """Largest |got - want| / bound over the copies' fluid cells; want, bound [ny, nx]."""
        worst = 0.0
        for g, w, b in zip(got, want, bound):
            d = (g.reshape(ny, copies, nx).double() - w.cuda()[:, None, :]).abs() / b.cuda()[:, None, :]
            worst = max(worst, torch.where(fluid, d, 0.0).max().item())
        return worst

    want = torch.from_numpy(oracle_ghat(p, st))[:, 0]
    half = 2.0 ** -11 if prec == "fp16s" else 0.0
    assert off(pops[:, 0], want, tg + half * want.abs()) <= 1
    want = st["scal"][:, 0]
    scale = torch.tensor(p["weno_scale"][:len(want)], dtype=torch.float64)[:, None, None].expand_as(want)
    assert off(sc[:, 0], want, ts * torch.maximum(scale, want.abs())) <= 1

    # per cell: |u| <= 3 P0 / rho sum |ghat|, and Lambda carries the scalars' bounds
    rho, T = rho_o.max().item(), scal[0].min()
    ua, du = u_o.abs().max().item(), 64 * eps * 9 * np.abs(ghat).max() / rho_o.min().item()
    two = len(scal) == 6
    dLam = ts * (scal[0].max() / T + (1.75 * sum(p["weno_scale"][1:6]) if two else 0.0))
    dP = 64 * eps + rho / 6 * dLam
    per_cell = np.array([64 * eps * rho, dP, rho * du, rho * du, 0.0, 2 * rho * ua * du,
                         64 * eps * (0.0444 if two else 1.0) / T, 64 * eps * rho * np.abs(scal[1]).max()])
    assert (np.abs(sums - sums_o.numpy()) <= N * per_cell).all(), (sums, sums_o, N * per_cell)
    if observed:
        mean, rms, k = s.statistics()
        val = torch.cat([u_o[:, 0], P_o])
        bound = torch.tensor([du, du, dP], dtype=torch.float64)[:, None, None].expand_as(val)
        assert k == 1 and off(mean[:, 0], val, bound) <= 1 and off(rms[:, 0], 0 * val, bound) <= 1
        rows = s.probes().cpu()
        for j, n in enumerate(cells):
            y, x = divmod(n, copies * nx)
            d = (rows[0, j] - val[:, y, x % nx]).abs()
            assert (d <= bound[:, 0, 0]).all(), (n, rows[0, j], val[:, y, x % nx])
    s.close()


# copies: just over one pass (1024 tiles FP64, 2048 otherwise), and for FP32 with two scalars also
# just over the lines it splits from (4096 64x4 tiles, 2600 linear ones); 64 x 40 on 64x4 tiles, the
# others on linear tiles, the last one partly filled
@pytest.mark.parametrize("observed", [False, True])
@pytest.mark.parametrize("nx,ny,copies,precision", [
    (64, 40, 103, "fp64"), (50, 37, 143, "fp64"), (64, 40, 206, "fp32"), (45, 33, 355, "fp32"), (64, 40, 206, "fp16s"),
    (45, 33, 355, "fp16s"), (64, 40, 411, "fp32"), (45, 33, 450, "fp32"),
])
@pytest.mark.parametrize("physics,faces", [
    ("one_step", WALLS), ("one_step", OPEN), ("two_step", OPEN), ("mixture", OPEN),
])
def test_split_channel_matches_oracle(physics, faces, nx, ny, copies, precision, observed):
    p = _params(nx, ny, physics, precision, faces)
    ghat, scal = random_state(p, seed=31)
    _check(p, ghat, scal, _solids(nx, ny), copies, observed)


@pytest.mark.parametrize("nx,ny,copies,precision", [(64, 40, 103, "fp64"), (45, 33, 355, "fp32"), (45, 33, 450, "fp32")])
def test_split_bgk_channel_matches_oracle(nx, ny, copies, precision):
    p = _params(nx, ny, "one_step", precision, OPEN, collision="bgk")
    ghat, scal = random_state(p, seed=33)
    _check(p, ghat, scal, _solids(nx, ny), copies, False)


@pytest.mark.parametrize("nx,ny,copies,precision", [
    (64, 40, 1460, "fp64"), (50, 37, 2020, "fp64"), (64, 40, 2920, "fp32"), (64, 40, 5850, "fp16s"),
])
def test_split_channel_with_cached_pulls_matches_oracle(nx, ny, copies, precision):
    p = _params(nx, ny, "one_step", precision, OPEN)
    ghat, scal = random_state(p, seed=35)
    size = {"fp64": 8, "fp32": 4, "fp16s": 2}[precision]
    assert 9 * nx * ny * copies * size > 256 << 20
    _check(p, ghat, scal, _solids(nx, ny), copies, False)


def test_split_corners_with_inlet_noise_match_oracle():
    # inlet and outlet in x between walls: the links of a corner pass through two faces; 1075 tiles
    p = _params(1100, 250, "one_step", "fp64", ["inlet", "outlet", "wall", "wall", "periodic", "periodic"],
                inlet_noise=0.05)
    ghat, scal = random_state(p, seed=37)
    _check(p, ghat, scal, _solids(1100, 250), 1, True)


@pytest.mark.parametrize("precision", ["fp64", "fp32", "fp16s"])
@pytest.mark.parametrize("lattice,nx,ny,nz,physics", [
    ("D2Q9", 64, 8, 1, "passive"), ("D2Q9", 65, 5, 1, "isothermal"), ("D3Q27", 64, 4, 3, "isothermal"),
    ("D3Q27", 7, 5, 3, "passive"), ("D3Q27", 64, 4, 5, "two_step"), ("D3Q27", 9, 6, 5, "two_step"),
])
def test_periodic_box_matches_oracle(lattice, nx, ny, nz, physics, precision):
    kw = {}
    if physics == "two_step":
        kw = dict(chem=L.two_step_chem(), T_ref=320.0, visc_law="const_mu",
                  weno_scale=[1630.0, 0.05, 0.22, 0.05, 0.13, 0.1, 1.0, 1.0])
    p = L.base_params(lattice, nx, ny, nz, physics=physics, nu_ref=0.01, cs_smag=0.17, precision=precision, **kw)
    ghat, scal = random_state(p, seed=39)
    s = make_solver(p)
    s.set_state(torch.from_numpy(ghat), torch.from_numpy(scal) if len(scal) else None, 0)
    s.step(1)
    pops, sc, _ = (t.double().cpu().numpy() if torch.is_tensor(t) else t for t in s.get_state())
    s.close()
    st, _ = OS.step(p, oracle_state(p, ghat, scal))
    want, (tg, ts, _) = oracle_ghat(p, st), BOUND[precision]
    half = 2.0 ** -11 if precision == "fp16s" else 0.0
    assert (np.abs(pops - want) <= tg + half * np.abs(want)).all()
    ref = st["scal"].numpy()
    scale = np.maximum(np.array(p["weno_scale"][:len(ref)]).reshape(-1, 1, 1, 1), np.abs(ref))
    assert (np.abs(sc - ref) <= ts * scale).all()


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("shift", [(0, 8), (8, 0), (8, 8)])
def test_state_copy_to_any_element_alignment(precision, shift):
    # byte counts are multiples of 16, the destinations' addresses (populations, scalars) are not
    p = L.base_params("D3Q27", 16, 4, 4, physics="passive", precision=precision)
    s = make_solver(p)
    g = torch.Generator(device="cuda").manual_seed(2)
    pops = (0.01 * torch.randn((27, 4, 4, 16), generator=g, device="cuda")).to(s.pop_dtype)
    scal = torch.rand((1, 4, 4, 16), generator=g, device="cuda").to(s.scal_dtype)
    s.set_state(pops, scal, 7)
    out = []
    for t, k in zip((pops, scal), shift):
        room = torch.zeros(t.numel() * t.element_size() + 16, dtype=torch.uint8, device="cuda")
        out.append(room[k:k + room.numel() - 16])
    n = ctypes.c_int64()
    C.check(C.lib().lbm_get_state(s._h, ctypes.c_void_p(out[0].data_ptr()), ctypes.c_void_p(out[1].data_ptr()),
                                  ctypes.byref(n)), s._h)
    s.close()
    assert n.value == 7
    assert torch.equal(out[0], pops.view(torch.uint8).flatten()) and torch.equal(out[1], scal.view(torch.uint8).flatten())
