"""GPU: the structure factor of small fluctuations on a large mean.

Along both axes, S(0, m) and S(m, 0) are as accurate as the fluctuation's own
transform: the rounding of the mean enters neither.  Tolerance: a transform of
2^p points carries an error of order p ulp of its norm (by convolution three
times that), squared here, so about 100 ulp = 2e-14 of the axis' largest value
at the sizes below; 1e-12 leaves room for the oracle's own.  A uniform field has
no fluctuation at all and is refused at every size.
"""
import numpy as np
import pytest

from oracle import structure as OS

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no HIP device", allow_module_level=True)

from paper_1008_2865_amd import binding as B  # noqa: E402
from paper_1008_2865_amd.structure import StructureFactor  # noqa: E402

# A row or a column of one, two and four columns per workgroup, even, odd, and by convolution.
SIDES = [5, 13, 64, 100, 331, 512, 1000, 1021, 2048]


@pytest.mark.parametrize("L", SIDES)
def test_axes_of_small_fluctuations(L):
    print(f"structure factor of small fluctuations L={L}", flush=True)
    noise = np.random.default_rng(L).random((L, L)) - 0.5
    fields = {"noise 0.01": 0.7 + 0.01 * noise, "noise 1e-6": 0.7 + 1e-6 * noise,
              "rows": 0.7 + 1e-6 * noise[:, :1] * np.ones((1, L)),
              "columns": 0.7 + 1e-6 * noise[:1] * np.ones((L, 1)), "large mean": 1e6 + noise}
    fields["one site apart"] = fields["noise 1e-6"].copy()
    fields["one site apart"][0, 0] = 1.2
    sk = StructureFactor(L)
    got = {name: sk(torch.tensor(f, device="cuda"), spectrum=True) for name, f in fields.items()}
    sk.close()
    for name, f in fields.items():
        spec, want = got[name][4].cpu().numpy(), OS.spectrum(f)
        scale = float(want.max())
        for axis, a, b in (("S(0, m)", spec[1:, 0], want[1:, 0]), ("S(m, 0)", spec[0, 1:], want[0, 1:])):
            # An axis without power of its own (rows, columns) has only the rounding of the other.
            top = float(b.max())
            if top < 1e-10 * scale:
                top = scale
            assert float(np.max(np.abs(a - b))) <= 1e-12 * top, (name, axis)
        # The mean itself is subtracted to a few ulp.
        assert abs(spec[0, 0]) <= 1e-12 * scale + L * L * (4 * np.spacing(np.mean(f))) ** 2, name


@pytest.mark.parametrize("L", SIDES)
@pytest.mark.parametrize("value", [0.3, 0.7, 1.0])
def test_uniform_field_is_refused(L, value):
    sk = StructureFactor(L)
    with pytest.raises(B.LBError) as err:
        sk(torch.full((L, L), value, dtype=torch.float64, device="cuda"))
    sk.close()
    assert err.value.code == B.LB_ERR_NONFINITE
