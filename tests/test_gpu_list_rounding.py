"""GPU checks of what rounding leaves of the list path's results where terms cancel: the gradient of the scale with a bias many times
the scores."""
import numpy as np
import pytest

from paper_2506_16640_amd import synth
from tests.parity_util import gpu_run, oracle_run, rel_err

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("use_saved", [False, True])
@pytest.mark.parametrize("d,dtype", [(64, "bf16"), (128, "bf16"), (64, "fp32")])
def test_scale_gradient_beside_a_large_bias(d, dtype, use_saved):
    """Scale 1e-4 with the bias outside it: in units of the scores the bias term is some 1e4 to 1e5, and dP has a common part of some
    hundred that mu takes off again.  The kernels' scores carry the bias in fp32, so that a score is good to 2^-24 1e5 = 6e-3 of
    a spread of sqrt(d) >= 8, 1e-3 at the worst row, less in the sums over rows; an error of rounding of the common part
    times the bias, 400 * 2^-24 * 1e5 = 2 a row, is far beyond the bar."""
    data = synth.make_inputs(B=1, H=2, n=600, nk=600, d=d, dtype=dtype, scale="head", seed=5)
    data["beta"][:], data["gamma"][:], data["delta"] = 1e-4, 0.0, 0.0
    data["V"][:] = synth.bf16_round(data["V"] + 8.0)
    data["dO"][:] = np.abs(data["dO"])
    kw = dict(slopes=np.array([0.25, 0.5], dtype=np.float32), bias_mode=1)
    g = gpu_run(data, 1.5, dtype, use_saved=use_saved, **kw)
    r = oracle_run(data, 1.5, **kw)
    errs = {n: rel_err(g[n], r[n]) for n in ("dbeta", "dQ", "dV")}
    print(d, dtype, errs, g["dbeta"], r["dbeta"])
    assert errs["dbeta"] <= 2e-3, errs
