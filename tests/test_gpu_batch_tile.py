"""GPU: a batch whose plain steps run several per launch on tiles.

Every lattice of the batch must hold the bits of a run of its own at one step
per launch: lattices of very different sizes (those that wrap in one tile
among them), logged and unlogged, replayed from graphs and launched, chunked
so that launches of every length occur, in every storage.
"""
import numpy as np
import pytest

from paper_1008_2865_amd import inputs

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no HIP device", allow_module_level=True)

from paper_1008_2865_amd.sim import LBBatch, LBSim  # noqa: E402

SIZES = {
    "tiny": [(5, 7), (24, 9)],                          # one step per launch
    "small": [(64, 64), (33, 90), (130, 20)],           # four and five
    "middle": [(300, 257), (96, 128), (512, 500)],      # three and two
    "large": [(700, 900), (1024, 130), (256, 256)],     # 512 threads
}


@pytest.mark.parametrize("storage", ["f64", "f32", "f16dev"])
@pytest.mark.parametrize("group", list(SIZES))
@pytest.mark.parametrize("use_graphs", [True, False])
def test_lattices_hold_the_bits_of_their_own_runs(group, storage, use_graphs):
    print(f"batch tile {storage} {group} graphs {use_graphs}", flush=True)
    lats = []
    for k, (nx, ny) in enumerate(SIZES[group]):
        G1, G2 = inputs.couplings(0.04 * k)
        lats.append(dict(rho_init=inputs.rho_noise(nx, ny, 60 + k), G1=G1, G2=G2, tau=(1.0, 0.8)[k % 2]))
    chunks = [1, 7, 13, 13, 4]
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        batch = LBBatch(lats, storage=storage, tile_x=64, log_every=10, max_steps=sum(chunks),
                        use_graphs=use_graphs)
        assert batch.two_step_shape() == (0, 0, 0)
        for n in chunks:
            batch.step(n)
            torch.cuda.synchronize()
            _ = batch[0].pseudo_energy()  # eager work between graph replays
        for k, L in enumerate(lats):
            single = LBSim(L["rho_init"], G1=L["G1"], G2=L["G2"], tau=L["tau"], storage=storage, tile_x=64,
                           log_every=10, max_steps=sum(chunks), steps_per_launch=1)
            single.step(sum(chunks))
            assert batch[k].t == sum(chunks)
            assert np.array_equal(batch[k].get_state().view(np.uint8), single.get_state().view(np.uint8)), k
            # The batch records the state it stops in, if due; a single run
            # records it on the way out.
            ta, tb = batch[k].trace(), single.trace()
            assert ta.shape == tb.shape and np.array_equal(ta, tb), k
            single.close()
        batch.close()


@pytest.mark.parametrize("storage", ["f64", "f32", "f16dev"])
@pytest.mark.parametrize("tau", [1.0, 1.3])
@pytest.mark.parametrize("group", ["small", "large"])
def test_one_tau_for_every_lattice(group, tau, storage):
    # A batch whose lattices all have tau = 1 runs a kernel of its own.
    print(f"batch tile {storage} {group} tau {tau}", flush=True)
    lats = []
    for k, (nx, ny) in enumerate(SIZES[group]):
        G1, G2 = inputs.couplings(0.03 * k)
        lats.append(dict(rho_init=inputs.rho_noise(nx, ny, 80 + k), G1=G1, G2=G2, tau=tau))
    with torch.cuda.stream(torch.cuda.Stream()):
        batch = LBBatch(lats, storage=storage, tile_x=64)
        batch.step(9)
        for k, L in enumerate(lats):
            single = LBSim(L["rho_init"], G1=L["G1"], G2=L["G2"], tau=tau, storage=storage, tile_x=64,
                           steps_per_launch=1)
            single.step(9)
            assert np.array_equal(batch[k].get_state().view(np.uint8), single.get_state().view(np.uint8)), k
            single.close()
        batch.close()
