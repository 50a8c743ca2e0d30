"""The FP32 one-launch split of D2Q9 is as accurate as the one-instance step: a cold vortex flow
between walls, 24 steps, once as a box periodic in x (one instance) and once as copies of it
(split), both against the FP64 solver's box, whose own error is 1e-13.  The two differ at most by the
order in which products are contracted, so their errors may differ by a few per cent."""
import numpy as np
import pytest
import torch

import lbm_inputs as L
from gpu_helpers import make_solver

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny,copies", [(256, 320, 14), (250, 330, 14)])     # 64x4 tiles, linear tiles
@pytest.mark.parametrize("kind", ["one_step", "two_step", "two_step observed", "mixture"])
def test_split_is_as_accurate_as_one_instance(nx, ny, copies, kind):
    x, y = np.arange(nx)[None, None, :] + 0.5, np.arange(ny)[None, :, None] + 0.5
    kx, ky = 8 * np.pi / nx, 8 * np.pi / ny
    u = 0.005 * np.stack([np.sin(kx * x) * np.cos(ky * y), -kx / ky * np.cos(kx * x) * np.sin(ky * y)])
    full = np.ones((1, ny, nx))
    yf, yo, _ = L.fresh_ch4_air(0.83)
    two = kind != "one_step"
    scal = np.stack([320 * full, yf * full, yo * full] + [0 * full] * 3) if two else np.stack([300 * full, full])
    kw = dict(physics="one_step", weno_scale=[1700.0] + [1.0] * 7, chem=[4.0, 15000.0, 300.0, 2000.0, 1.0])
    if two:
        kw = dict(physics="two_step", T_ref=320.0, chem=L.two_step_chem(B1=50.0, B2=5.0),
                  weno_scale=[1630.0, 0.05, 0.22, 0.05, 0.13, 0.11, 1.0, 1.0])
    if kind == "mixture":
        kw.update(transport_model="mixture", transport=L.mixture_transport(0.7 * 0.03 / 4))

    def run(precision, n):
        s = make_solver(L.base_params("D2Q9", n * nx, ny, 1, precision=precision, visc_law="const_mu",
                                      nu_ref=0.7 * 0.03 / 4, thickening=4.0, cs_smag=0.17,
                                      face_bc=["periodic", "periodic", "wall", "wall", "periodic", "periodic"], **kw))
        s.init_fields(torch.full((1, ny, n * nx), 1 / 3, dtype=torch.float64), torch.from_numpy(np.tile(u, (1, 1, 1, n))),
                      torch.from_numpy(np.tile(scal, (1, 1, 1, n))))
        if kind.endswith("observed"):
            s.set_statistics(1)
        s.step(24)
        pops = s.get_state()[0].double()
        s.close()
        return pops

    assert nx * ny <= 1024 * 256 and 4096 * 256 < copies * nx * ny
    ref = run("fp64", 1)
    one, many = run("fp32", 1) - ref, run("fp32", copies) - ref.tile((1, 1, 1, copies))
    e1, en = one.norm().item(), many.norm().item() / copies ** 0.5
    m1, mn = one.mean().abs().item(), many.mean().abs().item()
    print(f"error norm {e1:.3e}, split {en:.3e}; mean {m1:.3e}, split {mn:.3e}", flush=True)
    assert en <= 1.05 * e1 and mn <= 1.2 * m1
