"""GPU parity of the list kernel's memory of large scores at its edges: rows whose large scores lie in fewer, as many and more
32-key blocks than a lane has places, all-equal rows, and sequences whose group numbers take many bits of the remembered
scores.  The bars are the parity tests' (2e-2 on O, 1e-3 on tau: bf16 inputs, sums in fp32)."""
import numpy as np
import pytest

from paper_2506_16640_amd import synth
from tests.parity_util import compare, gpu_run, oracle_run

pytestmark = pytest.mark.gpu


def _data(nq, nk, d, dtype="bf16", seed=0):
    return synth.make_inputs(B=1, H=2, n=nq, nk=nk, d=d, dtype=dtype, scale="head", seed=seed)


@pytest.mark.parametrize("d,dtype", [(64, "bf16"), (128, "bf16"), (64, "fp32"), (128, "fp32")])
@pytest.mark.parametrize("blocks", [1, 5, 6, 7, 12, 20])
def test_large_scores_in_so_many_blocks(blocks, d, dtype):
    """One key in each of `blocks` 32-key blocks, all in the same lane half, points along a common direction that every
    query carries: their scores lie close together, well above the others."""
    data = _data(768, 768, d, dtype, seed=blocks)
    rng = np.random.default_rng(blocks)
    u = np.ones(d, dtype=np.float32)  # (exact in bf16, as are its products below)
    data["Q"][:] = data["Q"] * 0.125 + 0.25 * u
    at = 32 * np.arange(blocks) + 8 * rng.integers(0, 4, size=blocks) + rng.integers(0, 4, size=blocks)
    data["K"][:, :, at] = (2.0 + 0.0625 * rng.integers(0, 3, size=blocks)).astype(np.float32)[:, None] * u
    if dtype == "bf16":  # both sides see the same bf16 values
        import torch
        data["Q"][:] = torch.from_numpy(np.ascontiguousarray(data["Q"])).bfloat16().float().numpy()
    for alpha in (1.5, 2.0, 1.25, 1.7):
        g = gpu_run(data, alpha, dtype, bwd=False)
        compare(g, oracle_run(data, alpha, bwd=False), bwd=False, label="blocks %d alpha %g" % (blocks, alpha))


@pytest.mark.parametrize("n", [31, 170, 200, 1000])
def test_rows_of_equal_scores(n):
    """Zero queries: every score is exactly zero, and its bits next to a group's number are a denormal."""
    data = _data(n, n, 64, seed=3)
    data["Q"][:, :, ::3] = 0.0
    for alpha in (1.5, 2.0):
        compare(gpu_run(data, alpha, "bf16", bwd=False), oracle_run(data, alpha, bwd=False), bwd=False, label="zero rows %d" % n)


@pytest.mark.parametrize("nk,d", [(28 * 1024, 64), (28 * 1024 + 709, 64), (128 * 1024 + 165, 128)])
def test_sequences_longer_than_the_marks(nk, d):
    data = _data(129, nk, d, seed=5)
    compare(gpu_run(data, 1.5, "bf16", bwd=False), oracle_run(data, 1.5, bwd=False), bwd=False, label="nk %d" % nk)
