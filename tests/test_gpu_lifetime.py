"""GPU tests of a solver's lifetime: destroying one waits for no work but its own, and the
synchronising calls read the same results from a pooled pinned block and, with more solvers
alive than the pool has blocks (64), by a copy."""
import pytest
import torch

import lbm_inputs as L
from paper_2207_11567_amd import Solver

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lattice,nx,ny,nz", [("D2Q9", 32, 16, 1), ("D3Q27", 16, 8, 4)])
def test_destroy_leaves_other_streams_running(lattice, nx, ny, nz):
    s = Solver(L.base_params(lattice, nx, ny, nz))
    s.init_fields(torch.full((nz, ny, nx), 1 / 3), torch.zeros((s.D, nz, ny, nx)))
    s.step(2)
    s.step_sums()
    a = torch.rand((8192, 8192), device="cuda")
    out = torch.empty_like(a)
    other, done = torch.cuda.Stream(), torch.cuda.Event()
    other.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(other):
        torch.mm(a, a, out=out)                 # the library's set-up for the stream
        other.synchronize()
        for _ in range(40):                     # 1.1e12 operations each: a few ms
            torch.mm(a, a, out=out)
        done.record()
    before = done.query()
    s.close()
    after = done.query()
    other.synchronize()
    assert not before and not after


def test_more_solvers_than_pinned_blocks():
    def sums(k, s):
        p = 1 / 3 + 1e-3 * k
        s.init_fields(torch.full((1, 3, 5), p, dtype=torch.float64), torch.zeros((2, 1, 3, 5)))
        f = s.fields()["sums"]
        # FP64 sums of 15 values each
        assert abs(f[1] - 15 * p) <= 15 * 2.3e-16 * 15 and abs(f[0] - 15) <= 15 * 2.3e-16 * 15
        s.step(1)
        assert abs(s.step_sums()[0] - 15) <= 15 * 2.3e-16 * 15
        assert s.thermo_pressure() == (1.0, 0.0, 0.0)
        _, _, n = s.get_state()
        assert n == 1

    made = [Solver(L.base_params("D2Q9", 5, 3, 1)) for _ in range(150)]
    for k, s in enumerate(made):
        sums(k, s)
    for s in made[::2]:
        s.close()
    made = made[1::2] + [Solver(L.base_params("D2Q9", 5, 3, 1)) for _ in range(75)]
    for k, s in enumerate(made):
        sums(150 + k, s)
    # blocks of two solvers in turn
    a, b = made[0], made[-1]
    for k in range(3):
        sums(300 + k, a)
        sums(400 + k, b)
    for s in made:
        s.close()
