"""GPU: several plain steps per launch on tiles, the default of lattices that
do not run two per launch in the row walk.

Every site goes through the arithmetic of the one-step kernel, so the fields
must be bit-identical to one step per launch: for lattices whose tiles wrap
around, ragged last tiles, every number of steps and threads that the tile
rule chooses, runs that leave a shorter launch, and half storage's stochastic
rounding.
"""
import numpy as np
import pytest

from paper_1008_2865_amd import inputs

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no HIP device", allow_module_level=True)

from paper_1008_2865_amd.sim import LBSim  # noqa: E402

G1, G2 = inputs.couplings(0.1)


def run(rho, storage, chunks, spl, **kw):
    sim = LBSim(rho, G1=G1, G2=G2, storage=storage, steps_per_launch=spl, **kw)
    for n in chunks:
        sim.step(n)
    out = sim.get_state().view(np.uint8), sim.trace() if kw.get("log_every") else None, sim.t
    sim.close()
    return out


@pytest.mark.parametrize("nx,ny", [
    (5, 5), (6, 9), (8, 8),       # one or two steps: the region wraps the lattice
    (33, 20), (64, 64),           # 4 x 4 tiles, five steps
    (100, 70), (257, 131),        # four and three steps, ragged
    (400, 389), (449, 447),       # one tile per CU, three steps
    (512, 509),                   # 32 x 32, two steps
    (601, 640), (997, 701),       # 512 threads, three steps
    (1030, 1021),                 # 512 threads, two steps; 256 in double precision
    (24, 1100),                   # narrow
])
@pytest.mark.parametrize("storage", ["f64", "f32", "f16dev"])
def test_fields_are_those_of_one_step_per_launch(nx, ny, storage):
    print(f"tile {storage} {nx}x{ny}", flush=True)
    rho = inputs.rho_noise(nx, ny, nx + ny)
    a, _, ta = run(rho, storage, [23], 1)
    b, _, tb = run(rho, storage, [1, 2, 3, 17], 0)
    assert ta == tb == 23 and np.array_equal(a, b)


@pytest.mark.parametrize("storage", ["f64", "f32", "f16dev"])
@pytest.mark.parametrize("nx,ny,tau", [(48, 60, 0.8), (260, 200, 1.3), (620, 600, 0.8)])
def test_other_tau_and_logging(nx, ny, tau, storage):
    print(f"tile {storage} {nx}x{ny} tau {tau}", flush=True)
    rho = inputs.rho_noise(nx, ny, 3)
    a, tra, _ = run(rho, storage, [40], 1, tau=tau, log_every=9, max_steps=40)
    b, trb, _ = run(rho, storage, [4, 30, 6], 0, tau=tau, log_every=9, max_steps=40)
    assert np.array_equal(a, b)
    assert tra.shape == trb.shape
    np.testing.assert_allclose(trb, tra, rtol=1e-13, atol=0)
