"""GPU parity of the decode shapes (a few query rows against a long key sequence, the regime of the
paper's long-context evaluation): the split-key kernels behind entmax_attn_fwd against the fp64 oracle.
Same bars as the other parity tests: max-abs 2e-2 on O, 1e-3 on tau, 5e-2 relative on gradients."""
import numpy as np
import pytest

from paper_2506_16640_amd import synth
from tests.parity_util import compare, gpu_run, oracle_run

pytestmark = pytest.mark.gpu


def _case(nq, nk, d, dtype, scale, seed, B=2, H=3):
    return synth.make_inputs(B=B, H=H, n=nq, nk=nk, d=d, dtype=dtype, scale=scale, seed=seed)


@pytest.mark.parametrize("nq,nk", [(1, 1), (1, 70), (1, 5000), (3, 1500), (8, 777), (8, 4133)])
@pytest.mark.parametrize("alpha", [1.5, 2.0, 1.25, 1.7])
def test_decode_forward(nq, nk, alpha):
    # key chunks of 512: 4133 and 5000 span several with a ragged last one; causal rows see nk - nq + i + 1 keys
    data = _case(nq, nk, 64, "bf16", "head", seed=11)
    g = gpu_run(data, alpha, "bf16", bwd=False)
    r = oracle_run(data, alpha, bwd=False)
    print(nq, nk, alpha, compare(g, r, bwd=False, label=f"decode {nq}x{nk} a{alpha}"))


@pytest.mark.parametrize("nq,nk,decode", [(9, 600, True), (15, 1000, True), (16, 1100, True), (17, 1100, True), (33, 2200, True), (64, 4133, True), (64, 4000, False),
                                          (65, 5000, False)])
def test_decode_more_rows_against_long_keys(nq, nk, decode):
    # up to 64 rows take the split-key kernels when the keys are at least 64 times as many; the tile counters
    # (which only the training kernels keep) tell which path ran
    data = _case(nq, nk, 64, "bf16", "head", seed=18, B=1, H=2)
    g = gpu_run(data, 1.5, "bf16", bwd=False, stats=True)
    r = oracle_run(data, 1.5, bwd=False)
    print(nq, nk, compare(g, r, bwd=False, label=f"decode {nq}x{nk}"))
    assert (g["stats"]["fwd_list_qk"] + g["stats"]["fwd_qk_max"] == 0) == decode


@pytest.mark.parametrize("d,dtype", [(64, "fp32"), (128, "bf16"), (128, "fp32")])
@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("nq", [5, 20])
def test_decode_dtypes_and_head_dims(d, dtype, causal, nq):
    data = _case(nq, 1300, d, dtype, "head", seed=12)
    g = gpu_run(data, 1.5, dtype, causal=causal, bwd=False)
    r = oracle_run(data, 1.5, causal=causal, bwd=False)
    print(d, dtype, causal, compare(g, r, bwd=False, label=f"decode d{d} {dtype}"))


@pytest.mark.parametrize("scale,logn_mode", [("none", 0), ("query", 0), ("query", 1), ("head", 1)])
def test_decode_scale_layouts(scale, logn_mode):
    data = _case(4, 900, 64, "bf16", scale, seed=13)
    g = gpu_run(data, 1.5, "bf16", logn_mode=logn_mode, bwd=False)
    r = oracle_run(data, 1.5, logn_mode=logn_mode, bwd=False)
    print(scale, logn_mode, compare(g, r, bwd=False, label=f"decode scale {scale} {logn_mode}"))


def test_decode_negative_and_zero_scale():
    data = _case(2, 600, 64, "bf16", "head", seed=14, B=1)
    data["beta"] = np.array([-0.8, 0.0, 0.5], dtype=np.float32)  # negative multiplier; scale = delta = 0; ordinary
    data["gamma"] = np.ones(3, dtype=np.float32)
    data["delta"] = 0.0
    g = gpu_run(data, 1.5, "bf16", bwd=False)
    r = oracle_run(data, 1.5, bwd=False)
    print(compare(g, r, bwd=False, label="decode neg/zero scale"))


@pytest.mark.parametrize("alpha", [1.5, 2.0, 1.25, 1.1])
def test_decode_long_supports(alpha):
    """Supports longer than the solver's in-LDS candidate list (4096 keys): zero queries give equal scores, so
    every visible key is in the support with p = 1/n_i, tau = -(n_i)^-(alpha-1) and O the mean of the values;
    the dense recipe (delta = 0, gamma = -1/2) keeps most of 6000 keys within reach of the threshold."""
    nq, nk = 3, 6000
    data = _case(nq, nk, 64, "bf16", "dense", seed=15, B=1, H=2)
    data["Q"][:, 0] = 0.0
    g = gpu_run(data, alpha, "bf16", bwd=False)
    r = oracle_run(data, alpha, bwd=False)
    print(alpha, compare(g, r, bwd=False, label=f"decode long a{alpha}"))
    for i in range(nq):
        n_i = nk - nq + i + 1
        assert abs(g["tau"][0, 0, i] + n_i ** -(alpha - 1.0)) < 1e-3
        np.testing.assert_allclose(g["O"][0, 0, i], data["V"][0, 0, :n_i].mean(axis=0), atol=2e-2)


def test_decode_rows_without_keys():
    # more query rows than keys under the causal mask: the first rows see nothing, O = 0 and tau = 0 there
    data = _case(6, 4, 64, "bf16", "head", seed=16, B=1, H=2)
    g = gpu_run(data, 1.5, "bf16", bwd=False)
    r = oracle_run(data, 1.5, bwd=False)
    print(compare(g, r, bwd=False, label="decode empty rows"))
    assert np.all(g["O"][:, :, :2] == 0.0)


@pytest.mark.parametrize("use_saved", [False, True])
def test_decode_forward_then_backward(use_saved):
    # the backward kernels take tau from the decode forward (with `saved`: told to use the tiled kernels)
    data = _case(8, 700, 64, "bf16", "head", seed=17)
    g = gpu_run(data, 1.5, "bf16", use_saved=use_saved)
    r = oracle_run(data, 1.5)
    print(use_saved, compare(g, r, label="decode fwd+bwd"))


@pytest.mark.parametrize("nq,nk", [(2, 31), (2, 32), (2, 33), (3, 511), (3, 513), (32, 2049), (33, 2113), (64, 6147)])
@pytest.mark.parametrize("rising", [False, True])
def test_decode_scores_left_out(nq, nk, rising):
    """The matrix-core score kernel writes a row's scores of a 32-key block only where they can matter.  Edges of the
    blocks, of the 512-key chunks and of the 32-row query blocks; `rising`: every later key scores higher, so every
    block is above the rows' largest score so far."""
    data = _case(nq, nk, 64, "bf16", "head", seed=19, B=1, H=2)
    if rising:
        data["Q"][...] = np.abs(data["Q"])
        data["K"][...] = np.linspace(0.05, 0.5, nk)[None, None, :, None]
        data["Q"], data["K"] = (synth.bf16_round(data[x]) for x in ("Q", "K"))
    g = gpu_run(data, 1.5, "bf16", bwd=False)
    r = oracle_run(data, 1.5, bwd=False)
    print(nq, nk, rising, compare(g, r, bwd=False, label=f"decode blocks {nq}x{nk}"))


@pytest.mark.parametrize("B,H,nq,nk,d,dtype", [
    (2, 192, 2, 2081, 64, "bf16"),   # 768 rows, four chunks to a workgroup and a last workgroup of one
    (4, 64, 5, 2300, 128, "bf16"),   # two chunks to a workgroup, 256 threads a row in the solve
    (1, 384, 33, 2112, 64, "bf16"),  # two 32-row query blocks, four chunks to a workgroup
    (1, 12, 64, 4133, 128, "bf16"),  # the same in wide heads, one chunk to a workgroup
    (2, 128, 16, 1100, 64, "fp32"),  # fp32 from 16 rows on
    (1, 3, 40, 2600, 128, "fp32"),
])
def test_decode_left_out_scores_are_never_read(B, H, nq, nk, d, dtype):
    """The workspace is full of large scores before the call: an unwritten score that is read would be the row's
    largest.  The rows' largest scores rise along most of the keys, so that a row's lanes and the waves of a workgroup
    keep raising the row's limit while others test against it."""
    data = _case(nq, nk, d, dtype, "head", seed=23, B=B, H=H)
    ramp = np.linspace(0.2, 1.0, nk, dtype=np.float32)[None, None, :, None]
    data["K"][...] = synth.bf16_round(data["K"] * ramp)
    _compare_on_a_poisoned_workspace(data, 1.5, dtype, f"decode poisoned {nq}x{nk} d{d} {dtype}")


def _compare_on_a_poisoned_workspace(data, alpha, dtype, label):
    import torch
    from paper_2506_16640_amd import binding
    from tests.parity_util import to_dev
    q, k, v = (to_dev(data[x], dtype) for x in ("Q", "K", "V"))
    beta, gamma = (None if data[x] is None else torch.from_numpy(data[x]).float().cuda() for x in ("beta", "gamma"))
    kw = dict(alpha=alpha, beta=beta, gamma=gamma, delta=data["delta"])
    ws = torch.empty(binding.workspace_bytes(binding.make_params(q, k, alpha, data["delta"], True, beta, 0), 0), dtype=torch.uint8,
                     device="cuda")
    r = oracle_run(data, alpha, bwd=False)
    for _ in range(3):
        ws.view(torch.float32).fill_(1e30)
        o, tau = binding.entmax_attn_fwd(q, k, v, workspace=ws, **kw)
        g = {"O": o.float().cpu().numpy().astype(np.float64), "tau": tau.cpu().numpy().astype(np.float64)}
        print(label, compare(g, r, bwd=False, label=label))
    return r


@pytest.mark.parametrize("nq,B,H", [(3, 1, 2), (5, 4, 26)])  # 6 rows (1024 threads each), 520 rows (512 threads)
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("near,alpha", [(60, 1.5), (300, 1.25), (1500, 2.0), (3800, 1.5), (5000, 1.5), (5000, 1.25), (5000, 1.7)])
def test_decode_long_lists(near, alpha, nq, B, H, d):
    """`near` keys with scores close together, the others far below and falling along the sequence, so that most of
    their blocks are not written: one wave's rows, lists in LDS, and rows of more than 4096 candidates, which are read
    again where they stand with the unwritten scores left out."""
    nk = 6200
    data = _case(nq, nk, d, "bf16", "none", seed=31, B=B, H=H)
    data["Q"] *= 0.25
    data["Q"][..., 0] = 4.0
    data["K"][:, :, :near, 0] = 0.0
    data["K"][:, :, near:, 0] = np.linspace(-24.0, -400.0, nk - near, dtype=np.float32) * (d / 64) ** 0.5
    data["Q"], data["K"] = (synth.bf16_round(data[x]) for x in ("Q", "K"))
    r = _compare_on_a_poisoned_workspace(data, alpha, "bf16", f"decode long lists {near} a{alpha} {nq}x{B}x{H} d{d}")
    assert r["support"].max() <= near


@pytest.mark.parametrize("nq", [1, 3])
@pytest.mark.parametrize("dtype", ["bf16", "fp32"])
@pytest.mark.parametrize("ties", [1, 100])
def test_decode_scores_too_large_for_a_unit_step(nq, dtype, ties):
    """(alpha-1) s = 2^26 for the largest keys: one less is the same fp32 number, no key lies above it, and the
    threshold is the largest score itself, to fp32 (2^-24 of it off the threshold in exact arithmetic).  With a score
    beyond fp32 it is infinite."""
    data = _case(nq, 700, 64, dtype, "none", seed=29, B=1, H=2)
    data["Q"][...], data["K"][...] = 0.0, 0.0
    data["Q"][..., 0] = 2.0 ** 12
    data["K"][:, :, 50:50 + ties, 0] = 2.0 ** 18
    g = gpu_run(data, 1.5, dtype, bwd=False)
    r = oracle_run(data, 1.5, bwd=False)
    assert np.abs(g["tau"] / r["tau"] - 1.0).max() <= 2.0 ** -24, (g["tau"], r["tau"])
    data["Q"][..., 0], data["K"][:, :, 50:50 + ties, 0] = 2.0 ** 100, 2.0 ** 100
    assert np.all(gpu_run(data, 1.5, dtype, bwd=False)["tau"] == np.inf)


@pytest.mark.parametrize("B,H,nq,nk", [(1, 2, 1, 6200), (1, 2, 4, 6200), (2, 66, 5, 1500)])
def test_decode_scores_of_some_hundreds(B, H, nq, nk):
    """(alpha-1) s of 200 to 500: the chunks' largest scores, kept to 16 bits, are one or two units too low, and the
    candidates are sifted from as many more."""
    data = _case(nq, nk, 64, "bf16", "head", seed=37, B=B, H=H)
    data["beta"][:], data["gamma"][:] = 25.0, 1.0
    g = gpu_run(data, 1.5, "bf16", bwd=False)
    r = oracle_run(data, 1.5, bwd=False)
    assert 200.0 < np.median(r["tau"]) and r["tau"].max() < 512.0
    # fp32 scores: the products' sums and the scale's logarithm and power err by a few 2^-24 each, 3e-6 of 512
    print(nq, nk, compare(g, r, bwd=False, tol_tau=2e-3, label=f"decode hundreds {nq}x{nk}"))
