"""GPU: kernel variants and input paths that the tests by size do not reach.

The double-precision tiles of 256 threads with tau other than 1 and in a batch,
the adjoint's tiles of 512 threads in single precision, energies into pageable
memory, and device fields that are refused.
"""
import numpy as np
import pytest

from paper_1008_2865_amd import inputs

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no HIP device", allow_module_level=True)

from paper_1008_2865_amd import binding as B  # noqa: E402
from paper_1008_2865_amd.adjoint import DropletLoss  # noqa: E402
from paper_1008_2865_amd.sim import LBBatch, LBSim  # noqa: E402

G1, G2 = inputs.couplings(0.1)


def bits(a):
    return a.view(np.uint8)


@pytest.mark.parametrize("tau", [1.0, 0.8])
def test_double_precision_tiles_of_256_threads(tau):
    rho = inputs.rho_noise(1030, 1027, 5)  # above 1 050 000 sites
    states = []
    for spl in (1, 0):
        print(f"f64 1030x1027 tau {tau} steps_per_launch {spl}", flush=True)
        sim = LBSim(rho, G1=G1, G2=G2, tau=tau, storage="f64", steps_per_launch=spl)
        sim.step(5)
        states.append(sim.get_state())
        sim.close()
    assert np.array_equal(bits(states[0]), bits(states[1]))


@pytest.mark.parametrize("taus", [(1.0,), (0.8, 1.0)])
def test_double_precision_batch_tiles_of_256_threads(taus):
    shapes = [(470 + 3 * i, 465 - 7 * i) for i in range(5)]  # 1 080 000 sites
    lats = [dict(rho_init=inputs.rho_noise(nx, ny, i), G1=G1, G2=G2, tau=taus[i % len(taus)])
            for i, (nx, ny) in enumerate(shapes)]
    states = []
    for spl in (1, 0):
        print(f"f64 batch tau {taus} steps_per_launch {spl}", flush=True)
        batch = LBBatch(lats, storage="f64", steps_per_launch=spl)
        batch.step(5)
        batch.step(1)
        states.append([m.get_state() for m in batch.members])
        batch.close()
    assert all(np.array_equal(bits(a), bits(b)) for a, b in zip(*states))


def test_f32_adjoint_tiles_of_512_threads_against_f64():
    # Tolerances of the 512^2 test at its short horizon.
    nx, ny, steps = 600, 560, 40  # above 262 144 sites
    rho = inputs.rho_noise(nx, ny, 1)
    probe = LBSim(rho, G1=G1, G2=G2, storage="f64")
    probe.step(steps)
    row = probe.pseudo_energy()
    probe.close()
    out = {}
    for storage in ("f64", "f32"):
        print(f"adjoint {storage} {nx}x{ny}", flush=True)
        loss = DropletLoss(nx, ny, steps, E_target=1.01 * (row[2] + row[3]), beta=1.0 / (nx * ny), storage=storage,
                           checkpoint_every=15)
        out[storage] = loss.forward(rho, G1, G2) + loss.backward()
        loss.close()
    a, b = out["f64"], out["f32"]
    assert abs(b[1] - a[1]) <= 1e-5 * abs(a[1])
    assert all(abs(b[i] - a[i]) <= 1e-4 * abs(a[i]) for i in (4, 5))
    assert float(torch.linalg.norm(b[6] - a[6])) <= 1e-4 * float(torch.linalg.norm(a[6]))


@pytest.mark.parametrize("storage", ["f64", "f32", "f16dev"])
def test_energies_into_pageable_memory(storage):
    sim = LBSim(inputs.rho_noise(96, 80, 2), G1=G1, G2=G2, storage=storage)
    sim.step(7)
    pinned = sim.pseudo_energy()
    pageable = np.full(6, -1.0)
    B.lb_pseudo_energy(sim.ctx, pageable)
    part = torch.full((16,), -1.0, dtype=torch.float64, pin_memory=True)
    B.lb_pseudo_energy(sim.ctx, part[5:11])
    sim.close()
    assert np.array_equal(pinned, pageable) and np.array_equal(pinned, part[5:11].numpy())
    assert part[:5].tolist() == [-1.0] * 5 and part[11:].tolist() == [-1.0] * 5


def fields(nx, ny):
    return torch.full((ny, nx), 0.7, dtype=torch.float64, device="cuda")


# Checked through a copy, by the kernel, and by its second turn (above 524 288 sites).
@pytest.mark.parametrize("nx, ny", [(16, 16), (300, 200), (1030, 600)])
def test_device_fields_are_refused(nx, ny):
    rho, u, v = fields(nx, ny), torch.zeros((ny, nx), dtype=torch.float64, device="cuda"), fields(nx, ny)
    v[:] = 0.0
    loss = DropletLoss(nx, ny, 2, E_target=-1.0, beta=0.1, storage="f32")
    for at in (0, nx * ny // 2, nx * ny - 1):
        for value in (float("nan"), float("inf"), -float("inf"), 0.0, -0.5):
            rho.view(-1)[at] = value
            with pytest.raises(B.LBError) as err:
                LBSim(rho, G1=G1, G2=G2, storage="f32")
            assert err.value.code == B.LB_ERR_INVALID and f"rho_init[{at}]" in str(err.value)
            with pytest.raises(B.LBError) as err:
                loss.forward(rho, G1, G2)
            assert err.value.code == B.LB_ERR_INVALID and f"rho_init[{at}]" in str(err.value)
            rho.view(-1)[at] = 0.7
        for name, w in (("ux_init", u), ("uy_init", v)):
            w.view(-1)[at] = float("nan")
            with pytest.raises(B.LBError) as err:
                LBSim(rho, ux_init=u, uy_init=v, G1=G1, G2=G2, storage="f32")
            assert err.value.code == B.LB_ERR_INVALID and f"{name}[{at}]" in str(err.value)
            w.view(-1)[at] = -0.01  # negative velocities are fine
    sim = LBSim(rho, ux_init=u, uy_init=v, G1=G1, G2=G2, storage="f32")
    sim.step(1)
    sim.close()
    loss.forward(rho, G1, G2)
    loss.close()


def test_a_refused_density_leaves_the_last_run():
    nx, ny = 160, 150  # by the kernel's check
    rho = torch.tensor(inputs.rho_noise(nx, ny, 3), device="cuda")
    loss = DropletLoss(nx, ny, 9, E_target=-0.5 * nx * ny, beta=0.1, storage="f64", checkpoint_every=4)
    loss.forward(rho, G1, G2)
    want = loss.backward()
    loss.forward(rho, G1, G2)
    bad = rho.clone()
    bad[3, 4] = -1.0
    for field in (bad, bad.cpu().numpy()):
        with pytest.raises(B.LBError):
            loss.forward(field, 2 * G1, G2)
    got = loss.backward()
    loss.close()
    assert got[:2] == want[:2] and torch.equal(got[2], want[2])
