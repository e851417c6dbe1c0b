"""GPU: what the attention kernels of any sequence length and head size keep of the arithmetic of a softmax taken
row by row: masked entries have no part in it, whatever they hold."""
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
]
IDS = ["%s_h%d_a%d_s%d_b%d" % c for c in SHAPES]


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


@pytest.mark.parametrize("low,live", [((32, 64), 0), ((0, 64), 64)], ids=["second_block", "first_blocks"])
@pytest.mark.parametrize("shape", SHAPES, ids=IDS)
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
        X[i * seq + low[0]:i * seq + low[1], 0] = -1.0
        X[i * seq + low[0]:i * seq + low[1], 1] = 1.0
    X = X.astype(np.float32)
    orc = make_oracle(w, params)
    orc.begin_iteration(1)
    orc.set_input(0, X)
    orc.forward(0)
    dev = run_once(w, params, X, np.zeros_like(X))
    y = dev.get_tensor(zb.T_OUTPUT_Y, 0, 0)
    dev.close()
    keep = np.concatenate([np.arange(i * seq + live, (i + 1) * seq) for i in range(b)])
    assert np.isfinite(y[keep]).all()
    assert rel_fro(y[keep], np.asarray(orc.Y[0])[keep]) <= TOL[dtype]


@pytest.mark.parametrize("shape", SHAPES, ids=IDS)
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
    for t in (0, 20, seq - 1):          # a token of the first sample
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
