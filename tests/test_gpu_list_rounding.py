"""GPU checks of what rounding leaves of the list path's results: the gradient of the scale with a bias many times the scores, rows of one
key, and rows whose scores' rounding is as wide as the threshold's bracket."""
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


@pytest.mark.parametrize("alpha", [1.5, 2.0, 1.25, 1.7])
@pytest.mark.parametrize("d", [64, 128])
def test_rows_of_one_key(d, alpha):
    """A row of one key has p = 1 whatever order its score was summed in: y = a d and tau = y - 1 are rounded to fp32, half a unit in the last
    place of y each, and p = (a d - tau)^r is off by r times that (and a few roundings of values near 1)."""
    n, r = 400, 1.0 / (alpha - 1.0)
    data = synth.make_inputs(B=2, H=2, n=n, nk=n, d=d, dtype="fp32", scale="head", seed=9)
    data["beta"][:], data["gamma"][:], data["delta"] = 1.0, 0.0, 11.0  # scale 12
    g = gpu_run(data, alpha, "fp32", bwd=False)
    y = 12.0 * (alpha - 1.0) / np.sqrt(d) * np.matmul(data["Q"].astype(np.float64), data["K"].transpose(0, 1, 3, 2).astype(np.float64))
    y = np.where(np.tril(np.ones((n, n), dtype=bool)), y, -np.inf)
    two = np.sort(y, axis=-1)[..., -2:]
    one = two[..., 1] - two[..., 0] > 1.01
    value = np.take_along_axis(data["V"], y.argmax(-1)[..., None], axis=2).astype(np.float64)
    p = (g["O"] * value).sum(-1) / (value * value).sum(-1)
    bar = r * np.spacing(np.abs(two[..., 1]).astype(np.float32)) + 4 * 2.0 ** -24
    print(d, alpha, "rows", int(one.sum()), "p off by", np.abs(p - 1.0)[one].max(), "of the bar", (np.abs(p - 1.0) / bar)[one].max())
    assert one.sum() > 500 and (np.abs(p - 1.0) <= bar)[one].all()


@pytest.mark.parametrize("size", [1024.0, 2048.0, 4096.0, 8192.0])
@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("d,dtype", [(64, "bf16"), (128, "bf16"), (64, "fp32")])
def test_scores_that_round_by_the_width_of_the_bracket(d, dtype, causal, size):
    """Half of the products are +- size^2 and cancel: the sums round by a hundredth of the bracket's width to several times it, another way in
    every order of summation.  Which keys a row has is then a matter of rounding, but its probabilities add up to one."""
    data = synth.make_inputs(B=2, H=3, n=500, nk=500, d=d, dtype=dtype, scale="none", seed=4)
    sign = np.where(np.arange(d // 2) % 2 == 0, 1.0, -1.0)
    data["Q"][..., : d // 2] = size * np.random.default_rng(8).permuted(np.broadcast_to(sign, data["Q"].shape[:3] + (d // 2,)), axis=-1)
    data["K"][..., : d // 2] = size
    data["Q"][..., d // 2:] *= 16.0
    data["V"][:] = 1.0
    g = gpu_run(data, 1.5, dtype, causal=causal, bwd=False, stats=True)
    off = np.abs(g["O"] - 1.0).max(-1)
    print(d, dtype, causal, size, "largest deviation", off.max(), {k: v for k, v in g["stats"].items() if v and k.startswith("fwd")})
    assert off.max() <= 1e-2  # (O is rounded to bf16: 4e-3)
