"""One reverse step on a small box and on copies of it side by side.  The box (54 blocks) takes
blocks in linear order and ordinary loads, the copies XCD order and, in FP32, streaming loads of the
incoming adjoint (arrays beyond 256 MB); the adjoint of the tiled state under the tiled
incoming adjoint is the tiled adjoint.  Both instances use the same formulas, so values
differ by at most their rounding: fewer than 64 roundings at the array's largest magnitude."""
import pytest
import torch

import lbm_inputs as L
from gpu_helpers import make_solver

pytestmark = pytest.mark.gpu
EPS = {"fp64": 2.3e-16, "fp32": 6e-8}


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("physics", ["isothermal", "passive"])
@pytest.mark.parametrize("n,reps", [((24, 24, 24), (4, 4, 4)), ((25, 23, 22), (4, 4, 4)), ((5, 3, 2), (4, 8, 16))])
def test_reverse_step_of_a_tiled_box(n, reps, physics, precision):
    g = torch.Generator(device="cuda").manual_seed(5)
    real = torch.float64 if precision == "fp64" else torch.float32
    nx, ny, nz = n

    def field(k, amp):
        return (amp * torch.randn((k, nz, ny, nx), generator=g, device="cuda", dtype=torch.float64)).to(real)
    k = 1 if physics == "passive" else 0
    ghat, T, lp, ls = field(27, 0.01), field(k, 1.0), field(27, 1.0), field(k, 1.0)
    out = []
    for r in ((1, 1, 1), reps):
        p = L.base_params("D3Q27", r[0] * nx, r[1] * ny, r[2] * nz, physics=physics, nu_ref=0.01, cs_smag=0.17,
                          precision=precision, prandtl=0.7, weno_scale=[1.0] * 8)
        s = make_solver(p)
        tile = (1, r[2], r[1], r[0])
        a = [v.tile(tile) if v.shape[0] else v.new_empty((0,) + s.shape) for v in (ghat, T, lp, ls)]
        _, _, work = s.adjoint_buffers()
        got = s.adjoint_step((a[0], a[1]), a[2], a[3], work)
        out.append([v.clone() for v in got])
        torch.cuda.synchronize()
        s.close()
    for a, b in zip(*out):
        if a.shape[0]:
            assert torch.isfinite(b).all()
            want = a.tile((1, reps[2], reps[1], reps[0]))
            assert (b - want).abs().max().item() <= 64 * EPS[precision] * want.abs().max().item()
