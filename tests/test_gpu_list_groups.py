"""GPU parity of the forward's list kernels where their memory of a row's largest key groups ends: rows whose large scores lie
in fewer, as many and more groups than a lane keeps (8 for strong scales, 12 else), in so few lanes of a query block that their keys are looked at
one by one and in more, in short rows that are swept a second time at once; one and two query blocks per workgroup, with and
without distance bias.  Which way a case took is read from the counters: no block is the tiled kernel's, and the score tiles computed are the visible
ones where groups are rescored or lanes looked through, more where blocks are swept again.  The backward gets the forward's lists.  The bars are
the parity tests' (bf16 inputs, sums in fp32)."""
import numpy as np
import pytest

from paper_2506_16640_amd import synth
from tests.parity_util import compare, gpu_run, oracle_run

pytestmark = pytest.mark.gpu


def _data(n, d, dtype, scale, groups, rows, half, seed):
    """`groups` keys, each in a group of its own (8 keys of one lane half), point along a common direction that `rows` late queries carry."""
    data = synth.make_inputs(B=1, H=2, n=n, nk=n, d=d, dtype=dtype, scale="head", seed=seed)
    rng = np.random.default_rng(seed)
    data["beta"][:], data["gamma"][:], data["delta"] = (scale - 1.0) / np.log(n), 1.0, 1.0
    u = np.ones(d, dtype=np.float32)
    at = n - 140 - rng.choice(rows * 3, size=rows, replace=False)
    data["Q"][:, :, at] = data["Q"][:, :, at] * 0.125 + np.float32(16.0 / d) * u
    pick = rng.choice((n - 140 - rows * 3) // 16, size=groups, replace=False)  # 16 keys: a group of either half
    keys = 16 * pick + 8 * rng.integers(0, 2, size=groups) + 4 * half + rng.integers(0, 4, size=groups)
    data["K"][:, :, keys] = (2.0 + 0.0625 * rng.integers(0, 3, size=groups)).astype(np.float32)[:, None] * u
    if dtype == "bf16":  # both sides see the same bf16 values
        data["Q"][:] = synth.bf16_round(data["Q"])
    return data


def _check(data, alpha, dtype, label, swept_again=None, lists=True, **kw):
    g = gpu_run(data, alpha, dtype, use_saved=True, stats=True, **kw)
    kw.pop("path", None)
    r = oracle_run(data, alpha, **kw)
    st = {k: v for k, v in g["stats"].items() if v}
    print(label, compare(g, r, label=label), st)
    B, H, n, _ = data["Q"].shape
    assert not lists or st["fwd_sparse_blocks"] == B * H * ((n + 127) // 128), st
    if swept_again is not None:
        assert st["fwd_list_qk"] > st["fwd_tiles_visible"] if swept_again else st["fwd_list_qk"] == st["fwd_tiles_visible"], st


@pytest.mark.parametrize("d,dtype", [(64, "bf16"), (128, "bf16"), (64, "fp32"), (128, "fp32")])
@pytest.mark.parametrize("scale", [7.0, 4.0])
@pytest.mark.parametrize("groups", [7, 8, 9, 11, 12, 13, 20])
def test_groups_and_lanes(groups, scale, d, dtype):
    for rows in (1, 8, 9, 60):
        data = _data(704, d, dtype, scale, groups, rows, half=groups & 1, seed=groups + rows)
        # fewer groups than a lane keeps: rescored.  13 groups, a single row at the strong scale: its lane is looked through.  20 groups in 60 rows: swept
        swept_again = False if groups == 7 or (groups, rows, scale) == (13, 1, 7.0) else True if (groups, rows) == (20, 60) else None
        _check(data, 1.5, dtype, "groups %d rows %d scale %g d%d %s" % (groups, rows, scale, d, dtype), swept_again)


@pytest.mark.parametrize("alpha", [1.25, 1.7, 2.0])
def test_other_alphas(alpha):
    for groups, rows in ((8, 8), (13, 5), (20, 40)):
        _check(_data(704, 64, "bf16", 7.0, groups, rows, 0, seed=3), alpha, "bf16", "alpha %g groups %d rows %d" % (alpha, groups, rows))


@pytest.mark.parametrize("n", [620, 769, 1100])
def test_two_blocks_per_workgroup(n):
    for groups, rows, scale in ((8, 4, 7.0), (9, 4, 7.0), (12, 40, 4.0), (14, 3, 4.0), (20, 40, 7.0)):
        _check(_data(n, 64, "bf16", scale, groups, rows, 1, seed=n + groups), 1.5, "bf16", "two blocks n%d groups %d rows %d" % (n, groups, rows),
               True if (groups, rows) == (20, 40) else None, path=2)


@pytest.mark.parametrize("bias_mode,causal", [(0, True), (1, True), (0, False)])
@pytest.mark.parametrize("path", [0, 2])
def test_with_distance_bias(bias_mode, causal, path):
    slopes = np.array([0.0, 1.0 / 512], dtype=np.float32)
    for groups, rows in ((8, 3), (13, 6), (20, 40)):
        data = _data(900, 64, "bf16", 7.0, groups, rows, 0, seed=groups)
        _check(data, 1.5, "bf16", "bias m%d groups %d rows %d" % (bias_mode, groups, rows), {8: False, 13: None, 20: True}[groups], slopes=slopes, bias_mode=bias_mode, causal=causal, path=path)


def test_negative_scales_and_weak_short_rows():
    data = _data(704, 64, "bf16", 7.0, 13, 6, 0, seed=1)
    data["K"][:] = -data["K"]
    data["beta"][:], data["delta"] = -data["beta"], -1.0
    _check(data, 1.5, "bf16", "negative scale")
    for n in (97, 130, 260):  # short rows that keep a good part of their keys
        data = synth.make_inputs(B=2, H=2, n=n, nk=n, d=64, dtype="bf16", scale="none", seed=n)
        _check(data, 1.5, "bf16", "short rows n%d" % n, True, lists=n < 260)  # (of the longest a block overflows)


@pytest.mark.parametrize("d,dtype", [(64, "bf16"), (128, "bf16"), (64, "fp32"), (128, "fp32")])
@pytest.mark.parametrize("use_saved", [False, True])
def test_supports_of_every_length(use_saved, d, dtype):
    """The backward's row kernel takes eight entries of a row at a time: rows of 1 to 32 entries (16 per half row at most), uneven between
    the halves, next to each other; the last 128-row block is ragged."""
    n = 300
    data = synth.make_inputs(B=1, H=2, n=n, nk=n, d=d, dtype=dtype, scale="none", seed=d)
    # features 0 .. 31: every query in a class of its own feature, with as many keys of one and the same score far above
    # the rest (features 32 .. 47) as the class has; features 48 .. are the keys' alone, so that dQ is not zero
    data["Q"][..., :32] = data["Q"][..., 48:] = 0.0
    data["K"][..., :32] = 0.0
    free, lengths = list(range(n)), []
    while True:
        length = len(lengths) + 1
        first = min(length, 16) if length % 3 else length // 2  # of the first half row
        keys = [j for j in free if (j // 4) % 2 == 0][:first] + [j for j in free if (j // 4) % 2 == 1][:length - first]
        if len(keys) < length or length > 24:
            break
        free = [j for j in free if j not in keys]
        data["K"][:, :, keys, :48] = 0.0
        data["K"][:, :, keys, len(lengths)] = 5.0
        lengths.append(length)
    assert len(lengths) >= 18
    data["Q"][:, :, np.arange(n), np.arange(n) % len(lengths)] = 8.0
    data["delta"] = np.sqrt(d)  # (alpha-1) s = 20 against a spread of 2
    g = gpu_run(data, 1.5, dtype, causal=False, use_saved=use_saved, saved_factor=8, stats=True)
    r = oracle_run(data, 1.5, causal=False)
    counts = np.bincount(r["support"].astype(int).ravel(), minlength=len(lengths) + 1)
    print(counts, compare(g, r, label="lengths %s d%d %s" % (use_saved, d, dtype)), {k: v for k, v in g["stats"].items() if v})
    assert (counts[1:len(lengths) + 1] > 0).all() and g["stats"]["bwd_support"] == r["support"].sum()
