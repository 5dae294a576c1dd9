"""Heads whose query blocks are split between the backward's list kernels and its tiled kernels: dK and dV are the sum of
both shares and are rounded to the output type once."""
import numpy as np
import pytest

from tests.parity_util import gpu_run

pytestmark = pytest.mark.gpu


def _shares(list_blocks, d):
    """Inputs (sparsemax, 64 keys, not causal) in which both shares and their sum are exact.  Rows of the first
    `list_blocks` blocks see two equal keys far above the others (p = 1/2); the last block's scores are all zero
    (p = 1/64, 32 keys of each half row: too many for the backward's lists).  The tiled share of every element is
    +-257, nine bits and more than a 16-bit float holds, the lists' share is -+1."""
    nk, nl = 64, 128 * list_blocks
    pair, j = np.arange(nl) % 32, np.arange(nk)
    sign = np.where(j % 8 < 4, 1.0, -1.0).astype(np.float32)  # a pair: key j and key j + 4, in different half rows
    Q = np.zeros((1, 1, nl + 128, d), np.float32)
    K, V, dO = np.zeros((1, 1, nk, d), np.float32), np.zeros((1, 1, nk, d), np.float32), np.zeros_like(Q)
    K[0, 0, j, j // 8 * 4 + j % 4] = 8.0
    V[0, 0, :, 0] = sign  # dP_ij = +-dO_i[0]: mu = 0 exactly
    # rows on the lists: q[pair] = 16 (score 16 for the pair's keys), q[32:64] for their share of dK
    per_pair = nl // 32  # rows that name a key
    Q[0, 0, np.arange(nl), pair] = 16.0
    Q[0, 0, :nl, 32:64] = 4.0
    dO[0, 0, :nl] = -2.0 / per_pair  # sum of p dO: -1; sum of c dS q: (1/8) per_pair (-2/per_pair) 4 = -1
    # the tiled block: c dS = dO / 8 per row; 127 rows of 128 and one of 192: sum of dO / 64 = 257 = sum of dO / 8 q, q = 1/8
    Q[0, 0, nl:, 32:64] = 0.125
    dO[0, 0, nl:] = 128.0
    dO[0, 0, nl] = 192.0
    return dict(Q=Q, K=K, V=V, dO=dO, beta=None, gamma=None, delta=1.0), sign


@pytest.mark.parametrize("dtype", ["bf16", "fp32"])
@pytest.mark.parametrize("use_saved", [False, True])
@pytest.mark.parametrize("list_blocks", [1, 4])  # keys of 4 and of 16 list entries (a lane group, a wave)
@pytest.mark.parametrize("d", [64, 128])
def test_shares_are_added_before_rounding(list_blocks, use_saved, dtype, d):
    data, sign = _shares(list_blocks, d)
    g = gpu_run(data, 2.0, dtype, causal=False, stats=True, use_saved=use_saved, saved_factor=4)
    st = g["stats"]
    print(list_blocks, use_saved, dtype, d, {k: v for k, v in st.items() if v})
    assert st["bwd_support"] == 2 * 128 * list_blocks and st["bwd_dkv_tiles"] > 0  # both paths at work
    tol = 0.0 if dtype == "bf16" else 2e-3  # bf16: 256 +- 1e-3 is 256; fp32: 1e-6 of 257
    assert np.abs(g["dV"] - 256.0).max() <= tol, (g["dV"].min(), g["dV"].max())
    if d == 64:  # (1/sqrt(128) is no power of two: the rounding of dS would show)
        assert np.abs(g["dK"][0, 0, :, 32:64] - 256.0 * sign[:, None]).max() <= tol


def test_many_more_keys_than_queries():
    """Nk of ten times Nq: the partial sums' low halves have a region of the workspace of their own."""
    from paper_2506_16640_amd import synth
    from tests.parity_util import compare, oracle_run
    nq, nk = 384, 3900
    data = synth.make_inputs(B=1, H=2, n=nq, nk=nk, d=128, dtype="bf16", scale="query", seed=9)
    data["beta"] = np.broadcast_to(np.linspace(3.0, 0.02, nq, dtype=np.float32), (1, 2, nq)).copy()
    data["gamma"], data["delta"] = np.ones_like(data["beta"]), 0.0
    r = oracle_run(data, 1.5, causal=False)
    for use_saved in (False, True):
        g = gpu_run(data, 1.5, "bf16", causal=False, stats=True, use_saved=use_saved)
        st = g["stats"]
        print(use_saved, compare(g, r, label="many keys"), {k: v for k, v in st.items() if v})
        assert st["bwd_support"] > 0 and st["bwd_dkv_tiles"] > 0
