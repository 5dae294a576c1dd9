"""The order of the forward's candidate lists, read back from the workspace: the sums over a list, and with them the last bits of the outputs,
follow it."""
import numpy as np
import pytest
import torch

from paper_2506_16640_amd import binding, synth

pytestmark = pytest.mark.gpu

CAP = 32  # entries of a half row


def _align(x):
    return (x + 255) // 256 * 256


@pytest.mark.parametrize("d,dtype", [(64, "bf16"), (128, "bf16"), (64, "fp32")])
@pytest.mark.parametrize("scale", [3.0, 5.0, 9.0])
def test_lists_hold_the_largest_groups_first(d, dtype, scale):
    """A lane's list takes its groups of eight keys in descending order of their largest score (or, where too many were above the bound to be
    remembered, all keys in their order), and the keys of a group in theirs."""
    B, H, n = 2, 3, 1300
    data = synth.make_inputs(B=B, H=H, n=n, nk=n, d=d, dtype=dtype, scale="none", seed=17)
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    q, k, v = (torch.from_numpy(data[x]).cuda().to(tdt) for x in ("Q", "K", "V"))
    prm = binding.make_params(q, k, 1.5, scale, True, None, 0)
    ws = torch.zeros(binding.workspace_bytes(prm, 0), dtype=torch.uint8, device="cuda")
    binding.entmax_attn_fwd(q, k, v, alpha=1.5, delta=scale, causal=True, workspace=ws)
    raw = ws.cpu().numpy()
    nqb, bh = (n + 127) // 128, B * H
    cand = _align(bh * d * nqb * 128 * (2 if dtype == "bf16" else 4))
    cnt_at = cand + _align(bh * nqb * 256 * CAP * 8)
    lists = raw[cand:cand + bh * nqb * 256 * CAP * 8].view(np.uint32).reshape(bh, nqb, 4, CAP, 64, 2)
    count = raw[cnt_at:cnt_at + bh * n * 2 * 4].view(np.int32).reshape(bh, n, 2)
    by_score, wraps = 0, 0
    for head in range(bh):
        for i in range(n):
            for half in range(2):
                m = count[head, i, half]
                if m < 2:
                    continue
                e = lists[head, i // 128, (i % 128) // 32, :m, 32 * half + i % 32]
                key, score = e[:, 0].astype(np.int64), e[:, 1].copy().view(np.float32)
                if (np.diff(key) > 0).all():
                    continue  # in the keys' order
                group = key // 16
                starts = np.flatnonzero(np.r_[True, np.diff(group) != 0])
                assert len(np.unique(group)) == len(starts), (head, i, half, key)
                assert (np.diff(key)[np.diff(group) == 0] > 0).all(), (head, i, half, key)
                most = np.maximum.reduceat(score, starts)
                # (two groups may change places where the sweep, which cuts mantissa bits off, sees their scores as one)
                assert (np.diff(most) <= 2.0 ** -12 * np.abs(most[:-1]) + 1e-5).all(), (head, i, half, key, score)
                by_score += 1
    print(d, dtype, scale, "lists in the order of scores:", by_score)
    assert by_score > 100
