"""GPU: the adjoint's tiles against the oracle, and against themselves.

Lattices that the tile rule splits in one, two and three steps per launch,
with ragged and wrapping tiles; and every split of a run into launches must
give the same bits, since a tile's own sites and the same sites in a
neighbour's halo go through one arithmetic.
"""
import numpy as np
import pytest

from oracle import adjoint as OA
from paper_1008_2865_amd import inputs

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no HIP device", allow_module_level=True)

from paper_1008_2865_amd.adjoint import DropletLoss  # noqa: E402

G1, G2 = inputs.couplings(0.1)


@pytest.mark.parametrize("nx,ny,tau,steps", [
    (5, 5, 1.0, 7),      # 2 x 2 tiles, one step: the region wraps the lattice
    (8, 13, 0.8, 8),
    (37, 90, 1.0, 11),   # three steps, ragged
    (261, 199, 1.0, 7),  # 16 x 16 and beyond
    (523, 301, 0.8, 5),  # two steps
])
def test_gradients_match_oracle(nx, ny, tau, steps):
    print(f"adjoint tile f64 {nx}x{ny} tau={tau} T={steps}", flush=True)
    rho = inputs.rho_noise(nx, ny, 9)
    target, beta, eps = -0.6 * nx * ny, 0.2, 1e-6
    L, dG1, dG2, drho, _, _ = OA.loss_and_grads(rho, G1, G2, steps, tau, target, beta, eps)
    dl = DropletLoss(nx, ny, steps, E_target=target, beta=beta, eps=eps, tau=tau, storage="f64",
                     checkpoint_every=4)
    got = dl.forward(rho, G1, G2)[0]
    g1, g2, gr = dl.backward()
    dl.close()
    # The tolerances of the adjoint's other oracle test.
    assert abs(got - L) <= 1e-10 * abs(L)
    assert abs(g1 - dG1) <= 1e-9 * abs(dG1) and abs(g2 - dG2) <= 1e-9 * abs(dG2)
    assert float(np.max(np.abs(gr.cpu().numpy() - drho))) <= 1e-9 * float(np.max(np.abs(drho)))


@pytest.mark.parametrize("storage", ["f32", "f64"])
@pytest.mark.parametrize("nx,ny", [(24, 31), (150, 97), (400, 260), (700, 650)])
def test_launch_splits_give_the_same_bits(nx, ny, storage):
    print(f"adjoint tile {storage} {nx}x{ny}", flush=True)
    rho = torch.tensor(inputs.rho_noise(nx, ny, 4), device="cuda")
    ref = None
    for every in (13, 1, 2, 5):
        dl = DropletLoss(nx, ny, 13, E_target=-0.5 * nx * ny, beta=0.1, storage=storage, checkpoint_every=every)
        out = dl.forward(rho, G1, G2) + dl.backward()
        dl.close()
        if ref is None:
            ref = out
        assert out[:6] == ref[:6] and torch.equal(out[6], ref[6]), every
