"""How much of the scores the forward's list kernel computes (its counters), where a rule decides between ways to the same result: dense rows
that leave it on the first tile.  Results against the oracle as in the parity tests."""
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
