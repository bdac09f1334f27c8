"""GPU: a batch of many small lattices runs on tiles, in the two-step walk once a
height is set, and on tiles again, with the same bits."""
import numpy as np
import pytest

from paper_1008_2865_amd import inputs

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no HIP device", allow_module_level=True)

from paper_1008_2865_amd.sim import LBBatch  # noqa: E402


@pytest.mark.parametrize("storage", ["f32", "f16dev"])
def test_height_set_and_taken_back(storage):
    G1, G2 = inputs.couplings(0.1)
    lats = [dict(rho_init=inputs.rho_noise(40, 48, i), G1=G1, G2=G2) for i in range(467)]
    with torch.cuda.stream(torch.cuda.Stream()):
        walk = LBBatch(lats, storage=storage, steps_per_launch=1)
        batch = LBBatch(lats, storage=storage)
        for ty in (None, 16, 64, 0):
            if ty is not None:
                batch.set_two_step_tile(ty)
                assert batch.two_step_shape()[:2] == ((128, ty) if ty else (0, 0))
            print(f"{storage} height {ty}", flush=True)
            for n in (5, 2):
                walk.step(n)
                batch.step(n)
            for i in (0, 200, 466):
                assert np.array_equal(walk[i].get_state().view(np.uint8), batch[i].get_state().view(np.uint8)), (ty, i)
        walk.close()
        batch.close()
