"""GPU: what the attention kernels of any sequence length and head size keep of the arithmetic of a softmax taken
row by row: masked entries have no part in it, whatever they hold, and its weights are fp32."""
import numpy as np
import pytest

import zb_inputs
from zb_testlib import TOL, make_device_stage, make_oracle, rel_fro

pytestmark = pytest.mark.gpu

W = zb_inputs.Workload

SHAPES = [
    # dtype, hidden, heads, seq, mb_size      which kernel
    ("fp32", 128, 2, 100, 1),       # head size 64, four blocks of 32 rows, the last one cut
    ("fp32", 128, 4, 161, 2),       # head size 32, six blocks: a wave takes two
    ("bf16", 600, 8, 77, 1),        # head size 75, two 64-row tiles
    ("bf16", 128, 4, 130, 2),       # head size 32, two rows past two tiles
    ("bf16", 256, 2, 200, 1),       # head size 128
    ("bf16", 600, 8, 333, 1),       # from 256 tokens on two groups of waves take the tiles in turn: head size 75, forward
    ("bf16", 128, 4, 300, 1),       # head size 32, both ways
    ("bf16", 192, 4, 260, 1),       # 48
    ("bf16", 256, 2, 300, 1),       # 128, forward
]
# whole tiles: the kernels without edges
WHOLE = [
    ("bf16", 128, 2, 128, 1),       # head size 64, two groups of waves with one tile each
    ("bf16", 128, 2, 512, 1),       # eight tiles
    ("bf16", 192, 2, 128, 1),       # head size 96
    ("bf16", 256, 2, 384, 1),       # head size 128, six tiles
]
IDS = ["%s_h%d_a%d_s%d_b%d" % c for c in SHAPES + WHOLE]


def run_once(w, params, X, dY):
    import paper_2401_10241_amd as zb
    dev = make_device_stage(w, 1, pools=(1, 1, 1))
    dev.set_params(params)
    dev.begin_iteration(0, 1)
    dev.set_tensor(zb.T_INPUT_X, 0, 0, X)
    dev.set_tensor(zb.T_INPUT_DY, 0, 0, dY)
    dev.forward(0)
    dev.backward_input(0)
    dev.synchronize()
    return dev


@pytest.mark.parametrize("low,live", [((32, 64), 0), ((0, 64), 64), ((64, 128), 0)],
                         ids=["second_block", "first_blocks", "second_tile"])
@pytest.mark.parametrize("shape", SHAPES + WHOLE, ids=IDS)
def test_scores_of_minus_infinity_have_no_weight(shape, low, live):
    # feature 0 of a token is the sign of its scores with every query (1e38 and more, an infinity in fp32): tokens
    # `low` get -inf, the others exactly 0.  From query `live` on there is a finite score, and those rows are
    # softmaxes over the other keys; in fp64 the oracle has weights of exp(-1e38) = 0 there
    import paper_2401_10241_amd as zb
    dtype, hidden, heads, seq, b = shape
    w = W("low", dtype, 1, hidden, heads, 4 * hidden, seq, b, 4, 0, 1, "H1", seed=59)
    params = zb_inputs.stage_params(w)
    d = hidden // heads
    P = params[0]
    P["wqkv"][:, :2 * hidden] = 0.0
    P["bqkv"][:2 * hidden] = 0.0
    P["bqkv"][0:hidden:d] = 2.0 ** 64            # q of every head: one column
    P["wqkv"][0, hidden:2 * hidden:d] = 2.0 ** 70  # k: that column is feature 0
    X = np.where(np.arange(hidden) % 2 == 0, 1.0, -1.0) * np.ones((seq * b, 1))
    X[:, :2] = 0.0                               # rows of mean zero: feature 0 stays exactly 0 in the LayerNorm
    X[:, 2:] *= 1.0 + 0.25 * (np.arange(seq * b)[:, None] % 3)
    for i in range(b):
        X[i * seq + low[0]:i * seq + min(low[1], seq), 0] = -1.0
        X[i * seq + low[0]:i * seq + min(low[1], seq), 1] = 1.0
    X = X.astype(np.float32)
    orc = make_oracle(w, params)
    orc.begin_iteration(1)
    orc.set_input(0, X)
    orc.forward(0)
    dev = run_once(w, params, X, np.zeros_like(X))
    y, dx = dev.get_tensor(zb.T_OUTPUT_Y, 0, 0), dev.get_tensor(zb.T_OUTPUT_DX, 0, 0)
    dev.close()
    keep = np.concatenate([np.arange(i * seq + live, (i + 1) * seq) for i in range(b)])
    assert np.isfinite(y[keep]).all()
    assert live or np.isfinite(dx).all()         # the backward's weights are made from the log-sum-exp
    assert rel_fro(y[keep], np.asarray(orc.Y[0])[keep]) <= TOL[dtype]


@pytest.mark.parametrize("shape", SHAPES, ids=IDS[:len(SHAPES)])
@pytest.mark.parametrize("bad", [float("nan"), float("inf")], ids=["nan", "inf"])
def test_a_token_that_is_not_finite_stays_causal(shape, bad):
    import paper_2401_10241_amd as zb
    dtype, hidden, heads, seq, b = shape
    w = W("causal", dtype, 1, hidden, heads, 4 * hidden, seq, b, 4, 0, 1, "H1", seed=53)
    params = zb_inputs.stage_params(w)
    X = zb_inputs.stage_input(w, 0, 0)
    dY = zb_inputs.upstream_grad(w, 0, 0)
    dev = run_once(w, params, X, dY)
    y0 = dev.get_tensor(zb.T_OUTPUT_Y, 0, 0).copy()
    dx0 = dev.get_tensor(zb.T_OUTPUT_DX, 0, 0).copy()
    dev.close()
    for t in (0, 20, seq - 1) + ((70, 140) if seq > 256 else ()):   # a token of the first sample; in tiles of both groups
        # in the forward only tokens t .. seq-1 of its sample may see it
        Xb = X.copy()
        Xb[t, 3] = bad
        dev = run_once(w, params, Xb, dY)
        y = dev.get_tensor(zb.T_OUTPUT_Y, 0, 0)
        dev.close()
        keep = np.r_[0:t, seq:seq * b]
        assert np.isfinite(y[keep]).all(), f"Y before token {t} is not finite"
        assert rel_fro(y[keep], y0[keep]) <= TOL[dtype]
        assert not np.isfinite(y[t]).any() and not np.isfinite(y[t:seq]).all(axis=1).any()
        # in the backward only tokens 0 .. t may
        dYb = dY.copy()
        dYb[t, 3] = bad
        dev = run_once(w, params, X, dYb)
        dx = dev.get_tensor(zb.T_OUTPUT_DX, 0, 0)
        dev.close()
        keep = np.r_[t + 1:seq * b]
        assert np.isfinite(dx[keep]).all(), f"dX after token {t} is not finite"
        assert rel_fro(dx[keep], dx0[keep]) <= TOL[dtype]
        assert not np.isfinite(dx[:t + 1]).all(axis=1).any()


def bf16_half_ulp(x):
    return 2.0 ** (np.floor(np.log2(np.maximum(np.abs(x), 1e-38))) - 8)


@pytest.mark.parametrize("shape", [s for s in SHAPES if s[0] == "bf16"], ids=IDS[2:len(SHAPES)])
def test_probabilities_keep_24_bits_in_the_products(shape):
    # Every column of W_qkv picks one input feature and W_o is a permutation, so Q, K, V and dO are columns of the
    # stashed LayerNorm output and output gradient, exactly, and the attention's results have a reference in 64 bits
    # from the device's own operands.  Beyond the rounding of the stored bf16 value an fp32 softmax leaves on a weight
    # the roundings of the scaled score, the log-sum-exp (both below 8: 2^-22 each), the exponential and the sum, 2^-21
    # together, and on dP - D those of two sums, 2^-23 of their absolute terms.  Weights of 16 bits (a bf16 and its
    # bf16 remainder) exceed these bounds 1.4 to 5 times, weights of 8 bits hundreds of times.
    import paper_2401_10241_amd as zb
    _, hidden, heads, seq, b = shape
    w = W("bits", "bf16", 1, hidden, heads, 4 * hidden, seq, b, 4, 0, 1, "H1", seed=61)
    params = zb_inputs.stage_params(w)
    rng = np.random.default_rng(67)
    pick = np.concatenate([rng.permutation(hidden) for _ in range(3)])
    params[0]["wqkv"] = np.zeros((hidden, 3 * hidden), np.float32)
    params[0]["wqkv"][pick, np.arange(3 * hidden)] = 1.0
    perm = rng.permutation(hidden)
    params[0]["wo"] = np.zeros((hidden, hidden), np.float32)
    params[0]["wo"][np.arange(hidden), perm] = 1.0
    dev = run_once(w, params, zb_inputs.stage_input(w, 0, 0), zb_inputs.upstream_grad(w, 0, 0))
    cols = np.arange(hidden)
    qkv = dev.get_stash_columns(zb.S_QKV_IN, 0, 0, cols).astype(np.float64)[:, pick]
    do = dev.get_stash_columns(zb.S_PROJ_DOUT, 0, 0, cols).astype(np.float64)[:, perm]
    out = dev.get_stash_columns(zb.S_PROJ_IN, 0, 0, cols).astype(np.float64)
    dqkv = np.hstack([dev.get_stash_columns(zb.S_QKV_DOUT, 0, 0, cols + k * hidden) for k in range(3)]).astype(np.float64)
    dev.close()
    d = hidden // heads
    masked = np.triu(np.ones((seq, seq), bool), 1)
    worst = {}
    for i in range(b):
        rows = slice(i * seq, (i + 1) * seq)
        for hd in range(heads):
            c = [slice(k * hidden + hd * d, k * hidden + (hd + 1) * d) for k in range(3)]
            q, k, v, o, g = qkv[rows, c[0]], qkv[rows, c[1]], qkv[rows, c[2]], out[rows, c[0]], do[rows, c[0]]
            x = np.where(masked, -np.inf, q @ k.T / np.sqrt(d))
            assert np.abs(x[~masked]).max() < 8.0
            p = np.exp(x - x.max(axis=1, keepdims=True))
            p /= p.sum(axis=1, keepdims=True)
            ds = p * (g @ v.T - (g * o).sum(axis=1, keepdims=True))
            tds = 2.0 ** -21 * np.abs(ds) + 2.0 ** -23 * p * (np.abs(g) @ np.abs(v).T + np.abs(g * o).sum(axis=1, keepdims=True))
            for name, dev_, ref, bound in (
                    ("O", o, p @ v, 2.0 ** -21 * p @ np.abs(v)),
                    ("dQ", dqkv[rows, c[0]], ds @ k / np.sqrt(d), tds @ np.abs(k) / np.sqrt(d)),
                    ("dK", dqkv[rows, c[1]], ds.T @ q / np.sqrt(d), tds.T @ np.abs(q) / np.sqrt(d)),
                    ("dV", dqkv[rows, c[2]], p.T @ g, 2.0 ** -21 * p.T @ np.abs(g))):
                beyond = np.abs(dev_ - ref) - bf16_half_ulp(dev_)
                worst[name] = max(worst.get(name, 0.0), float((beyond / (bound + 1e-300)).max()))
    print(f"[{shape}] largest error beyond the stored value's rounding, of its bound: {worst}", flush=True)
    assert max(worst.values()) <= 1.0, worst


def test_fp32_sequence_beyond_the_grid_is_refused():
    # 2^20 tokens: two workgroups per 32 rows of the backward are one more than a grid's last dimension takes.  The
    # forward already refuses, so no pass runs on a sequence whose B could not be launched.
    import paper_2401_10241_amd as zb
    w = W("long", "fp32", 1, 8, 2, 8, 1 << 20, 1, 4, 0, 1, "H1", seed=71)
    dev = make_device_stage(w, 1, pools=(1, 1, 1), journal=False)
    dev.begin_iteration(0, 1)
    with pytest.raises(zb.ZbError) as e:
        dev.forward(0)
    assert e.value.status == zb.EDEVICE
    dev.close()
