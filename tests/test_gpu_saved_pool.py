"""The pool of the `saved` buffer where it runs out: which query blocks keep their support lists for the backward follows
from the blocks' candidate counts, not from the order in which the workgroups run, and blocks whose supports are too
long for the backward's lists take no room from the others."""
import numpy as np
import pytest
import torch

from paper_2506_16640_amd import binding, synth
from tests.parity_util import compare, gpu_run, oracle_run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,H,n,d,dtype", [(4, 12, 1082, 64, "bf16"), (2, 16, 437, 128, "fp32"), (8, 48, 1400, 64, "bf16")])
def test_outputs_repeat_when_the_pool_runs_out(B, H, n, d, dtype):
    """alpha 1.25: six to twelve keys a row, so the pool of the size the library asks for (six a row) cannot hold every
    block's.  8 x 48 heads of eleven blocks: more than 64 blocks to a part of the pool.  The tiled and the list path
    round differently, so a block that takes the other one shows in dQ, dK and dV."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(5)
    t = torch.bfloat16 if dtype == "bf16" else torch.float32
    q, k, v, do = (torch.randn(B, H, n, d, generator=gen, device="cuda").to(t) for _ in range(4))
    beta, gamma = torch.linspace(0.6, 1.2, H, device="cuda"), torch.full((H,), 0.8, device="cuda")
    kw = dict(alpha=1.25, beta=beta, gamma=gamma, delta=1.0)
    saved = binding.new_saved(binding.make_params(q, k, 1.25, 1.0, True, beta, 0))
    first = None
    for _ in range(5):
        st = binding.new_stats()
        o, tau = binding.entmax_attn_fwd(q, k, v, saved=saved, **kw)
        res = (o, tau, *binding.entmax_attn_bwd(q, k, v, o, do, tau, saved=saved, stats=st, **kw))
        sd = binding.stats_dict(st)
        print(B, H, n, d, dtype, {a: b for a, b in sd.items() if b})
        assert sd["bwd_support"] > 0 and sd["bwd_dq_tiles"] > 0  # both paths at work
        if first is None:
            first, sd0 = [x.clone() for x in res], sd
        assert sd["bwd_support"] == sd0["bwd_support"]
        for name, a, b in zip(("O", "tau", "dQ", "dK", "dV", "dbeta", "dgamma"), first, res):
            assert torch.equal(a, b), name


def test_unusable_supports_take_no_room():
    """Every eighth head has four keys a row; the others' blocks all have half rows of 17 to 23 (more than the
    backward's lists hold) and ask for three times the pool: every block of the former keeps its lists."""
    H, n = 64, 512
    data = synth.make_inputs(B=1, H=H, n=n, nk=n, d=64, dtype="bf16", scale="head", seed=3)
    for x in ("Q", "K"):  # every head the same scores but for its scale
        data[x][:] = data[x][:, :1]
    data["beta"][:] = 1.0 / np.log(n)
    data["beta"][7::8] = 3.0 / np.log(n)
    data["gamma"][:], data["delta"] = 1.0, 0.0
    g = gpu_run(data, 1.5, "bf16", causal=False, stats=True, use_saved=True)
    r = oracle_run(data, 1.5, causal=False)
    st = g["stats"]
    print(compare(g, r, label="unusable supports"), {k: v for k, v in st.items() if v})
    assert st["fwd_sparse_blocks"] > 8 and st["bwd_dq_tiles"] > 0  # long rows are on the forward's lists and not on the backward's
    # (a key on the threshold may fall on either side)
    assert st["bwd_support"] >= 0.999 * r["support"][0, 7::8].sum(), (st["bwd_support"], r["support"][0, 7::8].sum())
