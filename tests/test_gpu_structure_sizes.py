"""GPU: the structure factor over the factorisations its transform meets.

Sides with every radix of the mixed-radix passes (8, 4, 2, 5, 3, 7), sides by
convolution (a prime factor above 7), odd sides (no l = L/2 column), sides whose
columns run one, two and four to a workgroup, and the smallest and largest of
the range, against the oracle.  Tolerances are those of the random-field test:
the transforms' rounding is a few ulp per pass, far below.
"""
import numpy as np
import pytest

from oracle import structure as OS
from paper_1008_2865_amd import inputs

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no HIP device", allow_module_level=True)

from paper_1008_2865_amd.structure import StructureFactor  # noqa: E402


@pytest.mark.parametrize("L", [5, 6, 7, 9, 11, 16, 33, 49, 128, 250, 331, 540, 662, 700, 1000, 1021, 1025, 1372, 1536, 2002, 2045,
                               2046, 2047])
def test_sides_match_oracle(L):
    print(f"structure factor L={L}", flush=True)
    rho = inputs.rho_noise(L, L, L, amp=0.2)
    tol = 1e-12 if L <= 512 else 1e-11
    sk = StructureFactor(L)
    Sn, counts, kbar, _, spec = sk(torch.tensor(rho, device="cuda"), spectrum=True)
    plain = sk(rho)
    sk.close()
    want, want_counts = OS.shells(rho)
    full = OS.spectrum(rho)
    assert np.array_equal(counts, want_counts)
    assert float(np.max(np.abs(spec.cpu().numpy() - full))) <= tol * float(full.max())
    assert float(np.max(np.abs(Sn - want))) <= tol * float(full.max())
    assert abs(kbar - OS.kbar(want)) <= tol * kbar
    # Without the spectrum and from host memory: the same bits.
    assert np.array_equal(plain[0], Sn) and plain[2] == kbar
