"""How much of the scores the forward's list kernel computes (its counters), where a rule decides between ways to the same result: dense rows
that leave it on the first tile, rows of weak scales that are swept a second time.  Results against the oracle as in the parity tests."""
import numpy as np
import pytest

from paper_2506_16640_amd import synth
from tests.parity_util import compare, gpu_run, oracle_run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["bf16", "fp32"])
@pytest.mark.parametrize("n", [257, 300, 352, 500, 640])
def test_dense_ragged_blocks_leave_on_their_first_tile(n, dtype):
    """A head's last block with 1, 44, 96, 116 and 128 rows: waves without rows have no say.  Only the first block, which no key tile is whole
    for, may be swept (10 tiles of 32 x 32, at most twice); the others compute at most two tiles a wave."""
    data = synth.make_inputs(B=1, H=2, n=n, nk=n, d=64, dtype=dtype, scale="dense", seed=4)
    g = gpu_run(data, 1.5, dtype, stats=True, path=0)
    st = {k: v for k, v in g["stats"].items() if v}
    print(n, dtype, compare(g, oracle_run(data, 1.5), label="ragged dense %d %s" % (n, dtype)), st)
    assert st["fwd_list_qk"] <= 2 * (2 * 10 + 8 * ((n + 127) // 128 - 1)), st


@pytest.mark.parametrize("d,dtype", [(64, "bf16"), (128, "bf16"), (64, "fp32")])
@pytest.mark.parametrize("causal,bias", [(True, False), (True, True), (False, False), (False, True)])
def test_second_sweep_of_few_and_many_tiles(causal, bias, d, dtype):
    """Rows without a scale keep tens of their keys.  One, two and three 128-key tiles, whole and ragged: a thread's first cells wait in LDS where
    the second sweep has at most two tiles.  With bias: windows that start behind the first tile."""
    for n in (60, 97, 128, 129, 200, 256, 257, 384, 400):
        data = synth.make_inputs(B=1, H=2, n=n, nk=n, d=d, dtype=dtype, scale="none", seed=n)
        kw = dict(causal=causal, slopes=np.array([0.0, 0.05], dtype=np.float32)) if bias else dict(causal=causal)
        for alpha in (1.5, 1.7):
            g = gpu_run(data, alpha, dtype, stats=True, path=0, use_saved=True, **kw)
            st = {k: v for k, v in g["stats"].items() if v}
            label = "second sweep n%d a%g c%d b%d d%d %s" % (n, alpha, causal, bias, d, dtype)
            print(label, compare(g, oracle_run(data, alpha, **kw), label=label), st)
            if not bias and st.get("fwd_blocks", 0) == 0:
                assert st["fwd_list_qk"] > st["fwd_tiles_visible"] or n == 60, st
