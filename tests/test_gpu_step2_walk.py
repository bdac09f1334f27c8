"""GPU: the two-step row walk against one step per launch.

The walk is unrolled by the length of its LDS rings (8), alternates its
direction from launch to launch and has a kernel of its own for tau = 1, so
the shapes here end a walk at every position of the unrolled loop, start runs
at odd and even time levels and hold tau at 1 and beside it.  Every kernel
rounds a site's update identically, so the populations are bit-identical.
"""
import numpy as np
import pytest

from paper_1008_2865_amd import inputs

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no HIP device", allow_module_level=True)

from paper_1008_2865_amd.sim import LBBatch, LBSim  # noqa: E402

WORD = {"f32": np.uint32, "f16dev": np.uint16}


@pytest.mark.parametrize("storage", ["f32", "f16dev"])
@pytest.mark.parametrize("tau", [1.0, 0.8])
@pytest.mark.parametrize("nx,ny,tile_x,tile_y", [
    (5, 9, 64, 8), (58, 17, 64, 8), (59, 35, 64, 9), (123, 41, 128, 10), (130, 47, 128, 11), (244, 50, 128, 12),
    (251, 53, 256, 13), (300, 59, 256, 14), (257, 64, 128, 15)])
def test_walk_matches_one_step_per_launch(storage, tau, nx, ny, tile_x, tile_y):
    print(f"{storage} tau {tau} {nx}x{ny} tile {tile_x}x{tile_y}", flush=True)
    G1, G2 = inputs.couplings(0.07)
    out = []
    for spl in (1, 2):
        sim = LBSim(inputs.rho_noise(nx, ny, 5), G1=G1, G2=G2, tau=tau, storage=storage, tile_x=tile_x,
                    tile_y=tile_y, steps_per_launch=spl)
        for n in (2, 1, 6, 3, 8):  # both directions from odd and even levels
            sim.step(n)
        out.append(sim.get_state().view(WORD[storage]))
        sim.close()
    assert np.array_equal(out[0], out[1])


@pytest.mark.parametrize("storage", ["f32", "f16dev"])
@pytest.mark.parametrize("taus", [(1.0, 1.0, 1.0), (0.8, 0.8, 0.8), (1.0, 0.9, 1.0)])
def test_batch_walk_matches_single_lattices(storage, taus):
    lats = []
    for k, (tau, (nx, ny)) in enumerate(zip(taus, [(130, 47), (70, 33), (256, 29)])):
        G1, G2 = inputs.couplings(0.02 * k)
        lats.append(dict(rho_init=inputs.rho_noise(nx, ny, 40 + k), G1=G1, G2=G2, tau=tau))
    print(f"{storage} taus {taus}", flush=True)
    with torch.cuda.stream(torch.cuda.Stream()):
        batch = LBBatch(lats, storage=storage, tile_x=64, steps_per_launch=2)
        for n in (3, 6):
            batch.step(n)
        for k, L in enumerate(lats):
            one = LBSim(L["rho_init"], G1=L["G1"], G2=L["G2"], tau=L["tau"], storage=storage, tile_x=64,
                        steps_per_launch=1)
            one.step(9)
            assert np.array_equal(batch[k].get_state().view(WORD[storage]), one.get_state().view(WORD[storage])), k
            one.close()
        batch.close()
