"""The backward's row kernel takes a block of 128 rows or a group of 32 per workgroup by the size of the launch: one call over many heads
against the same heads in two calls, which are below the line, and a few heads of each against the oracle."""
import numpy as np
import pytest
import torch

from paper_2506_16640_amd import binding, synth
from tests.parity_util import compare, oracle_run

pytestmark = pytest.mark.gpu


def _step(t, beta, gamma, alpha, heads):
    q, k, v, do = (x[heads] for x in t)
    kw = dict(alpha=alpha, beta=beta, gamma=gamma, delta=0.0, causal=True)
    saved = binding.new_saved(binding.make_params(q, k, alpha, 0.0, True, beta, 0))
    st = binding.new_stats()
    o, tau = binding.entmax_attn_fwd(q, k, v, saved=saved, **kw)
    grads = binding.entmax_attn_bwd(q, k, v, o, do, tau, saved=saved, stats=st, **kw)
    return (o, tau) + tuple(grads[:3]), grads[3], binding.stats_dict(st)


# (n 300: three blocks, the last one ragged; scale 1: some blocks' supports are too long for the backward's lists)
@pytest.mark.parametrize("n,batch,scale", [(300, 236, 1.0), (300, 236, 6.0), (130, 352, 3.0)])
@pytest.mark.parametrize("d,dtype", [(64, "bf16"), (128, "bf16"), (64, "fp32")])
def test_one_call_and_two(d, dtype, n, batch, scale):
    B, H, alpha = batch, 2, 1.5
    assert B * H * -(-n // 128) >= 1408 > B // 2 * H * -(-n // 128)
    small = synth.make_inputs(B=4, H=H, n=n, nk=n, d=d, dtype=dtype, scale="head", seed=n + d)
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    t = [torch.from_numpy(small[x]).cuda().to(tdt) for x in ("Q", "K", "V", "dO")]
    gen = torch.Generator(device="cuda")
    gen.manual_seed(3)
    more = [torch.randn(B - 4, H, n, d, generator=gen, device="cuda").to(tdt) for _ in t]
    t = [torch.cat([a, b]) for a, b in zip(t, more)]  # batches 0 .. 3 are those of the oracle
    beta, gamma = torch.full((H,), scale, device="cuda"), torch.zeros(H, device="cuda")
    one, dbeta, st = _step(t, beta, gamma, alpha, slice(0, B))
    a, db_a, st_a = _step(t, beta, gamma, alpha, slice(0, B // 2))
    b, db_b, st_b = _step(t, beta, gamma, alpha, slice(B // 2, B))
    print(d, dtype, n, scale, {k: (v, st_a[k] + st_b[k]) for k, v in st.items() if v})
    # rows are summed the same way; which blocks have room in `saved` follows from the size of the problem
    if st["bwd_support"] == st_a["bwd_support"] + st_b["bwd_support"]:
        for x, u, w, name in zip(one, a, b, ("O", "tau", "dQ", "dK", "dV")):
            if name in ("O", "tau", "dQ") or scale > 1.0:  # (keys of many entries: in the order of arrival)
                assert torch.equal(x, torch.cat([u, w])), name
    else:
        assert scale == 1.0
    assert abs(dbeta - db_a - db_b).max() <= 1e-3 * abs(dbeta).max() + 1e-4
    data = {x: small[x] for x in ("Q", "K", "V", "dO")}
    data.update(beta=beta.cpu().numpy(), gamma=gamma.cpu().numpy(), delta=0.0)
    r = oracle_run(data, alpha)
    g = {x: y[:4].float().cpu().numpy().astype(np.float64) for x, y in zip(("O", "tau", "dQ", "dK", "dV"), one)}
    compare(g, dict(r, dbeta=None, dgamma=None), label="%d %s %d %g" % (d, dtype, n, scale))
