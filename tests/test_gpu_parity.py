"""GPU parity: the HIP path (through the C ABI) against the CPU oracle on the same seeded inputs.
Tolerances: max relative Frobenius error 1e-4 (fp32), 2e-2 (bf16);
schedule order, rollback and accumulation determinism are bit-exact."""
import numpy as np
import pytest

import zb_inputs
from oracle import optimizer as O
from oracle.schedule import stage_order
from zb_testlib import (TOL, WORST_ELEM, check_delta_theta, check_second_moment, check_tensor, compare_grads, compare_outputs,
                        load_iteration, make_device_stage, make_oracle, rel_fro)
from oracle.stage import PARAM_ORDER

pytestmark = pytest.mark.gpu

W = zb_inputs.Workload


def run_and_compare(w, m=None, mbs_full=None):
    import paper_2401_10241_amd as zb
    m = m or w.m
    params = zb_inputs.stage_params(w)
    dev = make_device_stage(w, m)
    orc = make_oracle(w, params)
    dev.set_params(params)
    dev.begin_iteration(0, m)
    orc.begin_iteration(m)
    load_iteration(w, 0, m, dev, orc)
    dev.run_schedule(w.p, w.stage, m, w.kind)
    dev.synchronize()
    orc.run(stage_order(w.p, w.stage, m, w.kind))
    tol = TOL[w.dtype]
    e1 = compare_outputs(dev, orc, m, tol, mbs_full)
    e2 = compare_grads(dev, orc, tol)
    print(f"[{w.name}] worst rel-fro: outputs {e1:.2e}, grads {e2:.2e} (tol {tol}); largest entry error so far "
          f"{WORST_ELEM[0]:.2f} x the element-wise bound", flush=True)
    dev.close()
    return e1, e2


def test_c1_tiny_fp32_full():
    # workload c1: stage 0 of p=4, ZB-H1, m=8, fp32
    run_and_compare(zb_inputs.workload("c1"))


def test_small_bf16_mfma_shapes():
    # bf16, shapes that are multiples of the MFMA tiles, ZB-H2 order
    w = W("small_bf16", "bf16", 2, 256, 4, 1024, 128, 1, 4, 1, 6, "H2", seed=11)
    run_and_compare(w)


@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
def test_ragged_shapes(dtype):
    # nothing is a multiple of a tile: seq 80, hidden 72 (3 heads of 24), ffn 200, two sequences per microbatch
    w = W("ragged", dtype, 2, 72, 3, 200, 80, 2, 3, 1, 4, "H1", seed=5)
    run_and_compare(w)


def test_head_dim_96_and_single_microbatch():
    w = W("d96", "bf16", 1, 192, 2, 768, 64, 1, 2, 0, 1, "H2", seed=6)
    run_and_compare(w)


@pytest.mark.parametrize("d,heads,seq,b", [(128, 2, 256, 1), (96, 2, 256, 1), (64, 4, 384, 2), (128, 1, 512, 1),
                                           (128, 8, 384, 2), (128, 1, 128, 3), (128, 1, 640, 1), (96, 1, 1152, 1),
                                           (128, 2, 2048, 1)])
def test_mfma_attention_shapes(d, heads, seq, b):
    # several query/key tiles per head, diagonal tiles, every supported head size, two sequences per microbatch;
    # (128, 8, 384, 2) has a multiple of 8 heads (backward workgroups ordered per XCD) and an odd number of blocks;
    # then a single row block (each of the forward's two wave groups gets one key tile), 5 and 9 blocks, and 16
    # blocks of 2048 tokens (twice the workloads' sequence: 32 key tiles for the last row block)
    h = d * heads
    w = W(f"attn_d{d}_s{seq}", "bf16", 1, h, heads, 4 * h, seq, b, 2, 0, 2, "H1", seed=40 + d)
    run_and_compare(w)


def test_split_k_gemm_shapes():
    # few output tiles and a long contraction (hidden 2048, ffn 8192, 256 tokens): the N = hidden GEMMs
    # run as K slices plus a fix-up kernel
    w = W("splitk", "bf16", 1, 2048, 16, 8192, 256, 1, 2, 1, 2, "H1", seed=77)
    run_and_compare(w)


def test_tail_split_gemm_shapes():
    # 1024 tokens x ffn 16896: 4 x 66 tiles of 256 x 256, two tile columns more than one round over the 256
    # CUs; those columns run as K slices plus a fix-up kernel writing a column range of the output
    w = W("tailsplit", "bf16", 1, 2048, 16, 16896, 1024, 1, 2, 1, 1, "H1", seed=78)
    run_and_compare(w)


def test_accumulation_is_bitwise_identical_across_orders():
    import paper_2401_10241_amd as zb
    w = W("det", "bf16", 2, 256, 4, 1024, 128, 1, 4, 1, 8, "H1", seed=21)
    params = zb_inputs.stage_params(w)
    dev = make_device_stage(w, 8, pools=(8, 8, 8))
    dev.set_params(params)
    load_iteration(w, 0, 8, dev)
    results = []
    flat = [(0, k) for k in range(8)] + [(1, k) for k in range(8)] + [(2, k) for k in range(8)]
    for order in (zb.schedule_order(4, 1, 8, "H1"), zb.schedule_order(4, 3, 8, "H2"),
                  zb.schedule_order(8, 0, 8, "H2"), zb.schedule_order(4, 2, 8, "1F1B"), flat):
        dev.begin_iteration(0, 8)
        for c, k in order:
            (dev.forward, dev.backward_input, dev.backward_weight)[c](k)
        dev.synchronize()
        results.append((dev.get_tensor(zb.T_FLAT_GRADS).copy(),
                        [dev.get_tensor(zb.T_OUTPUT_DX, 0, k).copy() for k in range(8)]))
    for g, dxs in results[1:]:
        assert g.tobytes() == results[0][0].tobytes()
        for a, b in zip(dxs, results[0][1]):
            assert a.tobytes() == b.tobytes()
    assert np.abs(results[0][0]).max() > 0
    # What the library guarantees bit for bit is the sum taken in increasing microbatch order, which is the
    # order of W in every schedule of the paper (and of B, which carries the LayerNorm gradients).  An order
    # that runs the W passes in another microbatch sequence (legal: W_k only needs B_k) adds the same fp32
    # terms in another order: equal to rounding, not to the bit.
    shuffled = [(0, k) for k in range(8)] + [(1, k) for k in range(8)] + [(2, k) for k in (5, 2, 7, 0, 3, 6, 1, 4)]
    dev.begin_iteration(0, 8)
    dev.run_order(shuffled)
    dev.synchronize()
    g = dev.get_tensor(zb.T_FLAT_GRADS)
    assert rel_fro(g, results[0][0]) < 1e-6
    dev.close()


@pytest.mark.parametrize("shape", [(256, 4, 1024, 128), (72, 3, 200, 80)], ids=["whole_tiles", "edges"])
def test_grouped_w_has_the_bits_of_one_by_one_w(shape):
    # consecutive W passes of an order run as one grouped W: every gradient must keep every bit, whether the
    # kernel of whole tiles takes the shape (hidden 256) or the one with edges (hidden 72)
    import paper_2401_10241_amd as zb
    hidden, heads, ffn, seq = shape
    m = 6
    w = W("grp", "bf16", 2, hidden, heads, ffn, seq, 1, 4, 3, m, "H1", seed=23)
    params = zb_inputs.stage_params(w)
    order = zb.schedule_order(4, 3, m, "H1")          # ends in three consecutive W
    assert [c for c, _ in order[-3:]] == [2, 2, 2]
    results = []
    for mode in ("one by one", "run_schedule grouped", "explicit group", "run_schedule, grouping off"):
        dev = make_device_stage(w, m, pools=(m, m, m), **({"group_w": False} if mode.endswith("off") else {}))
        dev.set_params(params)
        dev.begin_iteration(0, m)
        load_iteration(w, 0, m, dev)
        if mode == "one by one":
            for c, k in order:
                (dev.forward, dev.backward_input, dev.backward_weight)[c](k)
        elif mode == "explicit group":
            for k in range(m):
                dev.forward(k)
                dev.backward_input(k)
            dev.backward_weight_group([0, 1])
            dev.backward_weight(2)
            dev.backward_weight_group([3, 4, 5])
            with pytest.raises(zb.ZbError) as e:
                dev.backward_weight_group([1, 2])      # already done
            assert e.value.status == zb.EORDER
        else:
            dev.run_schedule(4, 3, m, "H1")
        dev.synchronize()
        results.append(dev.get_tensor(zb.T_FLAT_GRADS).copy())
        dev.close()
    assert np.abs(results[0]).max() > 0
    for g in results[1:]:
        assert g.tobytes() == results[0].tobytes()


@pytest.mark.parametrize("shape", [(1024, 8, 4096, 256, 1, 2), (1024, 8, 4096, 128, 2, 4), (1024, 8, 4096, 128, 1, 4)],
                         ids=["h1024_s256", "h1024_s128_L2", "h1024_s128"])
def test_w_bits_do_not_depend_on_the_tiles(shape):
    # which tiles a W launch takes depends on tokens x microbatches and on the tiles of its layers: at 256 tokens one W
    # alone runs on 128-row tiles and two together on 256-row ones (192 of them); at 128 tokens the other way round with
    # one layer, and four together on 256-row ones again; with two layers (the single backward takes one at a time) too
    import paper_2401_10241_amd as zb
    hidden, heads, ffn, seq, layers, m = shape
    w = W("tiles", "bf16", layers, hidden, heads, ffn, seq, 1, 4, 2, m, "1F1B", seed=41)
    params = zb_inputs.stage_params(w)
    grads = []
    for mode in ("one by one", "two by two", "together", "fused"):
        dev = make_device_stage(w, m, pools=(m, m, m))
        dev.set_params(params)
        dev.begin_iteration(0, m)
        load_iteration(w, 0, m, dev)
        for k in range(m):
            dev.forward(k)
            if mode == "fused":
                dev.backward_fused(k)
            else:
                dev.backward_input(k)
        n = {"one by one": 1, "two by two": 2, "together": m, "fused": 0}[mode]
        for k in range(0, m, n) if n else ():
            dev.backward_weight_group(list(range(k, k + n))) if n > 1 else dev.backward_weight(k)
        dev.synchronize()
        grads.append(dev.get_tensor(zb.T_FLAT_GRADS).copy())
        dev.close()
    assert np.abs(grads[0]).max() > 0
    for g in grads[1:]:
        assert np.array_equal(g.view(np.uint32), grads[0].view(np.uint32))


@pytest.mark.parametrize("group", [2, 3])
def test_w_grouped_order_has_the_bits_of_the_plain_order(group):
    # the order with its steady-state W passes `group` at a time (zb_order_group_w) through zb_run_order: the W of
    # a parameter run in the same microbatch sequence, so every gradient and input gradient keeps every bit
    import paper_2401_10241_amd as zb
    m = 12
    w = W("pairw", "bf16", 2, 256, 4, 1024, 128, 1, 4, 1, m, "H1", seed=27)
    params = zb_inputs.stage_params(w)
    plain = zb.schedule_order(w.p, w.stage, m, "H1")
    paired = zb.order_group_w(plain, group)
    assert paired != plain and sorted(paired) == sorted(plain)
    assert sum(1 for i in range(len(paired) - 1) if paired[i][0] == 2 and paired[i + 1][0] == 2) >= 3
    results = []
    for ops in (plain, paired):
        pools = zb.order_stash_need(ops)
        dev = make_device_stage(w, m, pools=pools)
        dev.set_params(params)
        dev.begin_iteration(0, m)
        load_iteration(w, 0, m, dev)
        dev.run_order(ops)
        dev.synchronize()
        results.append((dev.get_tensor(zb.T_FLAT_GRADS).copy(),
                        [dev.get_tensor(zb.T_OUTPUT_DX, 0, k).copy() for k in range(m)]))
        dev.close()
    assert np.abs(results[0][0]).max() > 0
    assert results[0][0].tobytes() == results[1][0].tobytes()
    for a, b in zip(results[0][1], results[1][1]):
        assert a.tobytes() == b.tobytes()
    assert zb.order_stash_need(paired)[1] == zb.order_stash_need(plain)[1] + group - 1


def test_fused_backward_has_the_bits_of_b_then_w():
    # the traditional single backward (layer by layer: input gradient, then that layer's parameter
    # gradients) against B then W of the split, bit for bit, and against the oracle
    import paper_2401_10241_amd as zb
    m = 4
    w = W("fused", "bf16", 3, 256, 4, 1024, 128, 1, 4, 2, m, "H1", seed=29)
    params = zb_inputs.stage_params(w)
    order = zb.schedule_order(4, 2, m, "1F1B")
    results = []
    for mode in ("split", "fused calls", "run_schedule with fuse_bw"):
        dev = make_device_stage(w, m, pools=(m, m, m), **({"fuse_bw": True} if mode.startswith("run") else {}))
        dev.set_params(params)
        dev.begin_iteration(0, m)
        load_iteration(w, 0, m, dev)
        if mode == "split":
            for c, k in order:
                (dev.forward, dev.backward_input, dev.backward_weight)[c](k)
        elif mode == "fused calls":
            for c, k in order:
                if c == 0:
                    dev.forward(k)
                elif c == 1:
                    dev.backward_fused(k)
            with pytest.raises(zb.ZbError) as e:
                dev.backward_weight(0)                  # the fused call did W too
            assert e.value.status == zb.EORDER
        else:
            dev.run_schedule(4, 2, m, "1F1B")
        dev.synchronize()
        results.append((dev.get_tensor(zb.T_FLAT_GRADS).copy(),
                        [dev.get_tensor(zb.T_OUTPUT_DX, 0, k).copy() for k in range(m)]))
        if mode == "fused calls":
            orc = make_oracle(w, params)
            orc.begin_iteration(m)
            load_iteration(w, 0, m, orc=orc)
            orc.run(order)
            compare_outputs(dev, orc, m, TOL["bf16"])
            compare_grads(dev, orc, TOL["bf16"])
        dev.close()
    for g, dxs in results[1:]:
        assert g.tobytes() == results[0][0].tobytes()
        for a, b in zip(dxs, results[0][1]):
            assert a.tobytes() == b.tobytes()


def test_pass_order_is_enforced():
    import paper_2401_10241_amd as zb
    w = W("ord", "fp32", 1, 64, 2, 256, 32, 1, 2, 0, 2, "H1", seed=3)
    dev = make_device_stage(w, 2, pools=(1, 1, 1))
    dev.set_params(zb_inputs.stage_params(w))
    with pytest.raises(zb.ZbError) as e:
        dev.forward(0)
    assert e.value.status == zb.ESTATE          # no iteration begun
    dev.begin_iteration(0, 2)
    load_iteration(w, 0, 2, dev)
    for fn in (dev.backward_input, dev.backward_weight):
        with pytest.raises(zb.ZbError) as e:
            fn(0)
        assert e.value.status == zb.EORDER
    dev.forward(0)
    with pytest.raises(zb.ZbError) as e:
        dev.forward(0)
    assert e.value.status == zb.EORDER
    with pytest.raises(zb.ZbError) as e:
        dev.forward(1)
    assert e.value.status == zb.ENOMEM          # only one pending-B slot
    with pytest.raises(zb.ZbError) as e:
        dev.backward_weight(0)
    assert e.value.status == zb.EORDER
    dev.backward_input(0)
    dev.backward_weight(0)
    with pytest.raises(zb.ZbError) as e:
        dev.forward(2)
    assert e.value.status == zb.EINVAL
    dev.forward(1)
    dev.backward_input(1)
    dev.backward_weight(1)
    dev.synchronize()
    dev.close()


# ---------------------------------------------------------------------------------------------
# optimizer: post-validation outcomes, against the oracle's protocol and its synchronous result
# ---------------------------------------------------------------------------------------------
OPT_CASES = [
    # prev_sq, rest_sq, prev_nf, rest_nf, dY scale, nan, force, outcome
    (0.0, 0.0, False, False, 1e-3, False, False, O.COMMITTED),
    (0.0, 4.0, False, False, 1e-3, False, False, O.ROLLED_BACK_RECLIPPED),
    (0.0, 0.0, False, True, 1e-3, False, False, O.ROLLED_BACK_NONFINITE),
    (0.0, float("inf"), False, False, 1e-3, False, False, O.ROLLED_BACK_NONFINITE),
    (9.0, 0.0, False, False, 1e-3, False, False, O.DEFERRED_CLIPPED),
    (0.0, 0.0, False, False, 1.0, False, False, O.DEFERRED_CLIPPED),
    (9.0, 0.0, False, True, 1e-3, False, False, O.DEFERRED_SKIPPED),
    (0.0, 0.0, True, False, 1e-3, False, False, O.SKIPPED_LOCAL),
    (0.0, 0.0, False, False, 1e-3, True, False, O.SKIPPED_LOCAL),
    (0.0, 0.0, False, False, 1e-3, True, True, O.ROLLED_BACK_NONFINITE),
    (9.0, 0.0, False, False, 1e-3, False, True, O.ROLLED_BACK_RECLIPPED),
]


@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
def test_post_validated_optimizer_outcomes(dtype):
    import paper_2401_10241_amd as zb
    w = W("opt", dtype, 2, 128, 4, 512, 64, 1, 4, 1, 3, "H1", seed=31, lr=1e-3, clip=1.0)
    m = 3
    params = zb_inputs.stage_params(w)
    dev = make_device_stage(w, m)
    orc = make_oracle(w, params)
    dev.set_params(params)
    tol = TOL[dtype]
    for it, (prev_sq, rest_sq, prev_nf, rest_nf, scale, nan, force, want) in enumerate(OPT_CASES):
        dev.begin_iteration(it, m)
        orc.begin_iteration(m)
        for k in range(m):
            X = zb_inputs.stage_input(w, it, k)
            dY = zb_inputs.upstream_grad(w, it, k) * np.float32(scale)
            if dtype == "bf16":
                dY = zb_inputs.round_to_bf16(dY)
            if nan and k == 1:
                dY = dY.copy()
                dY[5, 7] = np.nan
            dev.set_tensor(zb.T_INPUT_X, 0, k, X)
            dev.set_tensor(zb.T_INPUT_DY, 0, k, dY)
            orc.set_input(k, X)
            orc.set_upstream_grad(k, dY)
        dev.run_schedule(w.p, w.stage, m, w.kind)
        orc.run(stage_order(w.p, w.stage, m, w.kind))
        before = [dev.get_tensor(x).copy() for x in (zb.T_FLAT_PARAMS, zb.T_FLAT_ADAM_M, zb.T_FLAT_ADAM_V)]
        theta_before = dev.get_group(zb.T_PARAM)
        ref_before = [{k: v.copy() for k, v in P.items()} for P in orc.master]
        rep = dev.optimizer_step_validated(prev_sq, rest_sq, prev_nf, rest_nf, force)
        ref = orc.optimizer_step(O.GlobalState(prev_sq, rest_sq, prev_nf, rest_nf, force))
        assert rep.outcome == want == ref.outcome, (it, rep.outcome_name)
        assert rep.t == ref.t and rep.stepped_optimistically == ref.stepped_optimistically
        after = [dev.get_tensor(x) for x in (zb.T_FLAT_PARAMS, zb.T_FLAT_ADAM_M, zb.T_FLAT_ADAM_V)]
        skipped = want in (O.SKIPPED_LOCAL, O.ROLLED_BACK_NONFINITE, O.DEFERRED_SKIPPED)
        if skipped:   # bit-identical to never having stepped
            for a, b in zip(after, before):
                assert a.tobytes() == b.tobytes(), f"case {it}: state changed although the iteration is skipped"
        else:
            assert after[0].tobytes() != before[0].tobytes()
            assert rel_fro(rep.local_sq, ref.local_sq) < (1e-6 if dtype == "fp32" else 5e-2)
            assert rep.global_norm == pytest.approx(ref.global_norm, rel=1e-5 if dtype == "fp32" else 3e-2)
            assert rep.clip_coef == pytest.approx(ref.clip_coef, rel=1e-5 if dtype == "fp32" else 3e-2)
        # state against the oracle's, tensor by tensor: the moments of all 12 tensors, the parameters of those
        # that do not start at zero, and (when a step was taken) the UPDATE of all 12
        groups = {base: dev.get_group(base) for base in (zb.T_PARAM, zb.T_ADAM_M, zb.T_ADAM_V)}
        for l in range(w.layers):
            for name in PARAM_ORDER:
                check_tensor(f"case {it} m {l} {name}", groups[zb.T_ADAM_M][l][name], orc.adam_m[l][name], tol, "fp32")
                check_second_moment(f"case {it} v {l} {name}", groups[zb.T_ADAM_V][l][name], orc.adam_v[l][name], tol)
                # Parameters that start at zero (biases, LayerNorm beta) are left out of the check of theta
                # itself: Adam's first update of such an element is lr times the SIGN of its gradient, so an
                # element whose gradient is smaller than the bf16 rounding noise flips by 2*lr whatever the
                # kernel does.  Their update is checked below on the entries whose gradient is not that small.
                if name in ("wqkv", "wo", "w1", "w2", "ln1_g", "ln2_g"):
                    check_tensor(f"case {it} theta {l} {name}", groups[zb.T_PARAM][l][name], orc.master[l][name], tol,
                                 "fp32")
                if not skipped:
                    check_delta_theta(f"case {it} update {l} {name}", theta_before[l][name],
                                      groups[zb.T_PARAM][l][name], ref_before[l][name], orc.master[l][name],
                                      orc.adam_v[l][name], max(tol, 1e-3))
    dev.close()


def test_rollback_then_redo_equals_direct_clipped_step_bitwise():
    """ROLLED_BACK_RECLIPPED must land on the same bits as DEFERRED_CLIPPED-style single clipped step."""
    import paper_2401_10241_amd as zb
    w = W("opt2", "bf16", 1, 128, 4, 512, 64, 1, 2, 0, 2, "H1", seed=32, lr=1e-3)
    params = zb_inputs.stage_params(w)
    finals = []
    for force in (True, False):
        dev = make_device_stage(w, 2)
        dev.set_params(params)
        dev.begin_iteration(0, 2)
        load_iteration(w, 0, 2, dev)
        dev.run_schedule(w.p, w.stage, 2, w.kind)
        # prev_sq = 9 makes the partial norm exceed the threshold: forced -> step, rollback, redo clipped;
        # not forced -> wait, one clipped step
        rep = dev.optimizer_step_validated(9.0, 0.0, False, False, force)
        assert rep.outcome == (O.ROLLED_BACK_RECLIPPED if force else O.DEFERRED_CLIPPED)
        finals.append([dev.get_tensor(x).copy() for x in (zb.T_FLAT_PARAMS, zb.T_FLAT_ADAM_M, zb.T_FLAT_ADAM_V)])
        if force:
            assert rep.alg1_mismatch_elems >= 0
        dev.close()
    for a, b in zip(*finals):
        assert a.tobytes() == b.tobytes()


def test_algorithm_1_rollback_without_journal_is_close_but_not_exact():
    import paper_2401_10241_amd as zb
    w = W("opt3", "fp32", 1, 128, 4, 512, 64, 1, 2, 0, 2, "H1", seed=33, lr=1e-3, clip=100.0)
    params = zb_inputs.stage_params(w)
    dev = make_device_stage(w, 2, journal=False)
    dev.set_params(params)
    for it in range(2):   # the first iteration commits so that m, v are non-zero
        dev.begin_iteration(it, 2)
        load_iteration(w, it, 2, dev)
        dev.run_schedule(w.p, w.stage, 2, w.kind)
        if it == 0:
            assert dev.optimizer_step_validated().outcome == O.COMMITTED
    before = [dev.get_tensor(x).copy() for x in (zb.T_FLAT_PARAMS, zb.T_FLAT_ADAM_M, zb.T_FLAT_ADAM_V)]
    rep = dev.optimizer_step_validated(0.0, 0.0, False, True, False)   # full state non-finite -> rollback
    assert rep.outcome == O.ROLLED_BACK_NONFINITE and rep.t == 1
    after = [dev.get_tensor(x) for x in (zb.T_FLAT_PARAMS, zb.T_FLAT_ADAM_M, zb.T_FLAT_ADAM_V)]
    assert rel_fro(after[0], before[0]) < 1e-6
    assert rel_fro(after[1], before[1]) < 1e-4
    assert rel_fro(after[2], before[2]) < 1e-4
    dev.close()


SWEEP = [
    # hidden, heads, ffn, seq, b, layers, dtype      which kernels the shape reaches
    (128, 2, 512, 64, 2, 2, "bf16"),      # head size 64, N = 384 / 128 not multiples of 256: GEMM tiles with edges
    (512, 4, 2048, 256, 1, 2, "bf16"),    # head size 128, 256 tokens: small GEMM tiles
    (768, 12, 3072, 128, 3, 1, "bf16"),   # head size 64, 384 tokens: small GEMM tiles
    (320, 4, 1280, 96, 1, 2, "bf16"),     # head size 80 and 96 tokens: attention with edges, mixed GEMMs
    (1024, 8, 4096, 200, 1, 1, "bf16"),   # head size 128 but a ragged sequence: attention with edges, 200-token GEMMs
    (384, 4, 1536, 192, 2, 1, "bf16"),    # head size 96
    (256, 2, 1024, 320, 1, 1, "fp32"),    # fp32 arithmetic everywhere
    (2048, 16, 8192, 512, 1, 1, "bf16"),  # 128 x 128 tiles, whole and in four slices
    (1536, 12, 6144, 256, 1, 1, "bf16"),  # wgrad on 128-row tiles, two workgroups per CU (288 tiles for FC1 / FC2)
    (768, 12, 16384, 128, 3, 1, "bf16"),  # 384 tokens, FC1 and its backward on 192 tiles of 128 x 256
    (512, 8, 24576, 128, 3, 1, "bf16"),   # the same on 288, two workgroups per CU
    (1536, 24, 1024, 128, 11, 1, "bf16"), # 1408 tokens, QKV on 198 tiles of 128 x 256
    (2304, 36, 1024, 128, 11, 1, "bf16"), # QKV on 594 of 128 x 128
]


@pytest.mark.parametrize("cfg", SWEEP, ids=lambda c: "h%d_a%d_f%d_s%d_b%d_L%d_%s" % c)
def test_shape_sweep(cfg):
    hidden, heads, ffn, seq, b, layers, dtype = cfg
    w = W("sweep", dtype, layers, hidden, heads, ffn, seq, b, 4, 1, 3, "H2", seed=101 + hidden + seq)
    run_and_compare(w)


EDGES = [
    # hidden, heads, ffn, seq, b, layers       what is cut where
    (600, 8, 1208, 77, 2, 2),     # head size 75 (odd: rows at 2-byte addresses), every width and the 154 tokens ragged
    (72, 3, 136, 33, 1, 2),       # head size 24, widths below one tile, one row past a 32-row block
    (400, 4, 1608, 130, 1, 1),    # head size 100; two rows past two 64-row tiles
    (96, 12, 264, 65, 3, 1),      # head size 8, the smallest the matrix-core kernels take
    (56, 8, 72, 50, 1, 1),        # head size 7, below it
    (256, 2, 1032, 129, 1, 1),    # head size 128, one row past a whole 128-row block
    (264, 3, 1024, 1, 1, 1),      # head size 88, a single token
    (1032, 8, 4104, 520, 2, 1),   # head size 129, above the matrix-core kernels; K cut into slices with a short last one
    (768, 12, 3072, 512, 1, 1),   # whole tiles of every kind, but too few of the large ones
]


@pytest.mark.parametrize("cfg", EDGES, ids=lambda c: "h%d_a%d_f%d_s%d_b%d_L%d" % c)
def test_edge_tiles(cfg):
    hidden, heads, ffn, seq, b, layers = cfg
    run_and_compare(W("edges", "bf16", layers, hidden, heads, ffn, seq, b, 4, 1, 3, "H2", seed=301 + hidden + seq))


@pytest.mark.parametrize("cfg", [
    # hidden, heads, ffn, seq, b       products of few steps of 32 k on the large tiles (the pipeline's fill and end)
    (64, 1, 2048, 64, 68),       # FC1 and FC2's backward: two steps on 128-row tiles, two workgroups per CU
    (128, 2, 2048, 64, 68),      # four
    (192, 3, 2048, 64, 68),      # six
    (64, 1, 2048, 64, 66),       # two, an odd number of tiles
    (256, 4, 24576, 64, 1),      # W: two steps on 256-row tiles
    (256, 4, 24576, 64, 2),      # four
    (256, 4, 24576, 64, 3),      # six on 128-row tiles, two workgroups per CU
    (256, 4, 17920, 64, 1),      # two
    (256, 4, 1024, 64, 5),       # ten on 128-row tiles, one per CU
], ids=lambda c: "h%d_a%d_f%d_s%d_b%d" % c)
def test_few_steps_of_the_large_tiles(cfg):
    hidden, heads, ffn, seq, b = cfg
    run_and_compare(W("few", "bf16", 1, hidden, heads, ffn, seq, b, 4, 1, 2, "H2", seed=601 + hidden + b))


@pytest.mark.parametrize("cfg", [
    # hidden, heads, ffn, seq, b       each tile of the products at about the fewest steps that reach it
    (512, 8, 64, 512, 11),       # QKV on 256 x 256 tiles, 16 steps of 32
    (1280, 20, 64, 64, 52),      # QKV's backward on them in three slices, 40
    (64, 1, 768, 64, 86),        # FC1 on 128 x 256 tiles, two
    (128, 2, 1280, 64, 52),      # four
    (192, 3, 1280, 64, 52),      # six
    (64, 1, 1280, 64, 104),      # the same with two workgroups per CU, two
    (128, 2, 832, 64, 40),       # FC1 on 128 x 128 tiles, two steps of 64
    (832, 13, 64, 64, 20),       # QKV's backward on them in three slices, thirteen
], ids=lambda c: "h%d_a%d_f%d_s%d_b%d" % c)
def test_products_on_each_tile(cfg):
    hidden, heads, ffn, seq, b = cfg
    run_and_compare(W("tiles", "bf16", 1, hidden, heads, ffn, seq, b, 4, 1, 1, "H1", seed=691 + hidden + b))


@pytest.mark.parametrize("steps", range(1, 8))
def test_few_steps_of_the_small_tiles(steps):
    # 1 to 7 steps of a ring of five stages, the last one cut: 64 k of the products, 32 tokens of W
    hidden = 64 * steps - 8
    run_and_compare(W("few_small", "bf16", 1, hidden, 8, 64 * steps + 8, 32 * steps - 3, 1, 4, 1, 2, "H2", seed=671 + steps))


@pytest.mark.parametrize("cfg", [
    # hidden, heads, ffn, seq, b       32-k blocks per wave (eight waves, four waves of the 64 x 64 tiles)
    (40, 1, 200, 33, 1),         # 16 x 16 tiles: two waves with a block; seven, the last one cut
    (264, 3, 520, 33, 1),        # two and one; three and two
    (776, 2, 1032, 17, 1),       # four and three; five and four
    (264, 3, 1032, 101, 5),      # 32 x 32 tiles: 17 x 9 and 17 x 33 of them, two and one blocks, five and four
    (520, 2, 40, 150, 2),        # 10 x 17, three and two
    (40, 1, 4104, 130, 4),       # 64 x 64 tiles: 9 x 65, two waves with a block
    (136, 1, 4104, 130, 4),      # two and one
], ids=lambda c: "h%d_a%d_f%d_s%d_b%d" % c)
def test_few_blocks_of_the_fp32_products(cfg):
    hidden, heads, ffn, seq, b = cfg
    run_and_compare(W("f32", "fp32", 1, hidden, heads, ffn, seq, b, 4, 1, 2, "H1", seed=731 + hidden + ffn))


@pytest.mark.parametrize("layers,cfg", [
    (9, (72, 3, 200, 33, 1)),     # 36 weight matrices: two launches transpose them; no side a multiple of 64
    (8, (64, 1, 128, 32, 1)),     # 32: one
    (1, (136, 1, 8, 16, 2)),      # the smallest ffn
], ids=lambda c: str(c))
def test_weights_are_transposed_after_a_step(layers, cfg):
    # the iteration after a step is bit for bit that of a stage that is given the stepped weights
    import paper_2401_10241_amd as zb
    hidden, heads, ffn, seq, b = cfg
    w = W("transposed", "bf16", layers, hidden, heads, ffn, seq, b, 4, 1, 2, "H1", seed=711 + hidden, lr=0.05)
    dev, other = make_device_stage(w), make_device_stage(w)
    dev.set_params(zb_inputs.stage_params(w))
    dev.begin_iteration(0, w.m)
    load_iteration(w, 0, w.m, dev)
    dev.run_schedule(w.p, w.stage, w.m, w.kind)
    dev.optimizer_step_validated(0.0, 0.0)
    other.set_params(dev.get_group(zb.T_PARAM))
    got = []
    for st in (dev, other):
        st.begin_iteration(1, w.m)
        load_iteration(w, 1, w.m, st)
        st.run_schedule(w.p, w.stage, w.m, w.kind)
        grads = st.get_group(zb.T_GRAD)
        got.append([st.get_tensor(zb.T_OUTPUT_DX, 0, k) for k in range(w.m)] + [g[n] for g in grads for n in sorted(g)])
        st.close()
    assert all(np.array_equal(a, c) for a, c in zip(*got))


@pytest.mark.parametrize("dtype,cfg", [
    ("bf16", (64, 1, 2048, 64, 68)),   # FC1 and FC2's backward on 256-row tiles
    ("bf16", (256, 4, 1032, 100, 1)),  # small tiles with edges
    ("fp32", (64, 1, 256, 64, 1)),
])
def test_gelu_over_its_range(dtype, cfg):
    # pre-activations from -60 to 60 (past the exponential's range on both sides), set through FC1's bias
    import paper_2401_10241_amd as zb
    hidden, heads, ffn, seq, b = cfg
    w = W("gelu", dtype, 1, hidden, heads, ffn, seq, b, 4, 1, 1, "H1", seed=651)
    params = zb_inputs.stage_params(w)
    params[0]["b1"] = np.linspace(-60.0, 60.0, ffn).astype(np.float32)
    dev, orc = make_device_stage(w, 1), make_oracle(w, params)
    dev.set_params(params)
    dev.begin_iteration(0, 1)
    orc.begin_iteration(1)
    load_iteration(w, 0, 1, dev, orc)
    dev.run_schedule(w.p, w.stage, 1, w.kind)
    orc.run(stage_order(w.p, w.stage, 1, w.kind))
    compare_outputs(dev, orc, 1, TOL[dtype], None)
    compare_grads(dev, orc, TOL[dtype])
    dev.close()


# products with the GELU in their epilogue: 256-row tiles, small tiles with edges, K slices and the launch that adds them
GELU_SHAPES = [(64, 1, 2048, 64, 68), (256, 4, 1032, 100, 1), (2048, 16, 256, 64, 1)]


def gelu_by_column(cfg, b1, dy):
    """G = gelu(b1) and dF = dG * gelu'(b1) of a bf16 stage, [tokens, ffn], as its epilogues make them: FC1's weights are
    zero, and W2 makes dG = dy[:, 0] + dy[:, 1] / 256 in every column, exactly (16 bits)."""
    import paper_2401_10241_amd as zb
    hidden, heads, ffn, seq, b = cfg
    w = W("gelu", "bf16", 1, hidden, heads, ffn, seq, b, 4, 1, 1, "H1", seed=653)
    params = zb_inputs.stage_params(w)
    params[0]["w1"][:] = 0.0
    params[0]["b1"] = b1.astype(np.float32)
    params[0]["w2"][:] = 0.0
    params[0]["w2"][:, 0] = 1.0
    params[0]["w2"][:, 1] = 2.0 ** -8
    dY = np.zeros((seq * b, hidden), np.float32)
    dY[:, :2] = dy
    dev = make_device_stage(w, 1)
    dev.set_params(params)
    dev.begin_iteration(0, 1)
    dev.set_tensor(zb.T_INPUT_X, 0, 0, zb_inputs.stage_input(w, 0, 0))
    dev.set_tensor(zb.T_INPUT_DY, 0, 0, dY)
    dev.forward(0)
    dev.backward_input(0)
    G, dF = (np.hstack([dev.get_stash_columns(what, 0, 0, np.arange(n, min(n + 32, ffn))) for n in range(0, ffn, 32)])
             for what in (zb.S_FC2_IN, zb.S_FC1_DOUT))
    y, dx = dev.get_tensor(zb.T_OUTPUT_Y, 0, 0), dev.get_tensor(zb.T_OUTPUT_DX, 0, 0)
    dev.close()
    assert np.isfinite(y).all() and np.isfinite(dx).all()
    return G, dF


@pytest.mark.parametrize("cfg", GELU_SHAPES, ids=lambda c: "h%d_a%d_f%d_s%d_b%d" % c)
def test_gelu_of_pre_activations_whose_cube_overflows(cfg):
    # finite pre-activations of any size: the GELU is x or 0 and its derivative 1 or 0.  x^3 leaves fp32 at 7e12, x^2 at 1.8e19
    hidden, heads, ffn, seq, b = cfg
    big = np.array([64.0, 2.0 ** 20, 2.0 ** 42, 2.0 ** 43, 2.0 ** 44, 2.0 ** 50, 2.0 ** 60, 2.0 ** 63], np.float32)
    x = np.resize(np.concatenate([big, -big]), ffn)
    dy = np.stack([2.0 ** (np.arange(seq * b) % 8), np.zeros(seq * b)], axis=1)
    G, dF = gelu_by_column(cfg, x, dy)
    assert np.array_equal(G, np.broadcast_to(np.maximum(x, 0.0), G.shape))
    assert np.array_equal(dF, np.outer(dy[:, 0], x > 0))


@pytest.mark.parametrize("cfg", GELU_SHAPES, ids=lambda c: "h%d_a%d_f%d_s%d_b%d" % c)
def test_gelu_and_its_derivative_keep_24_bits(cfg):
    # What is stored is a bf16, but where the exact value lies further from the middle of two bf16 than the fp32 value's
    # error, that error decides nothing.  For x >= 0 both are sums of a term and a smaller one: 2^-24 for the rounding of the
    # sum, as much for the smaller term's own, 2^-24 from the exponential (2^-23 of it, a quarter of which at most is in the
    # sum), and for dF one more for the product with dG: 2^-22 in all.  (The derivative with s (1 - s) from 1 - s is up to
    # 2e-6 off = 8 x 2^-22, one from an fp32 tanh 5.6e-7.)
    hidden, heads, ffn, seq, b = cfg
    rng = np.random.default_rng(659)
    grid = np.concatenate([np.float32(2.0) ** e * (1.0 + np.arange(128, dtype=np.float32) / 128) for e in range(-6, 4)])
    x = np.resize(rng.permutation(grid[grid < 12.0]), ffn)             # bf16 values: the backward reads the stored one
    dy = 1.0 + rng.integers(0, 128, (seq * b, 2)) / 128.0
    G, dF = gelu_by_column(cfg, x, dy)
    X = x.astype(np.longdouble)
    c, a = np.sqrt(2 / np.longdouble(np.pi)), np.longdouble("0.044715")
    w = 1 / (1 + np.exp(2 * c * (X + a * X ** 3)))
    slope = (1 - w) + 2 * X * w * (1 - w) * c * (1 + 3 * a * X ** 2)
    for name, got, want in (("G", G, np.broadcast_to((X * (1 - w)).astype(np.float64), G.shape)),
                            ("dF", dF, np.outer(dy[:, 0] + dy[:, 1] / 256, slope.astype(np.float64)))):
        half_ulp = 2.0 ** (np.floor(np.log2(got.astype(np.float64))) - 8)
        off = float((np.maximum(np.abs(got - want) - half_ulp, 0) / want).max())
        print(f"[{cfg}] {name}: {off * 2 ** 22:.2f} x 2^-22 beyond the stored value's rounding", flush=True)
        assert off <= 2.0 ** -22, (name, off)


@pytest.mark.parametrize("cfg", [
    # hidden, heads, ffn, seq, b       row blocks and groups of waves of the attention (128-row blocks of a launch)
    (256, 4, 512, 128, 3),       # head size 64, 12 whole blocks: 64 rows, two groups; the first blocks have one tile
    (256, 4, 512, 512, 9),       # 144 of them: 128 rows, two groups, both ways
    (256, 4, 512, 256, 20),      # 160 short ones: the backward with one group of 64 rows
    (120, 3, 248, 300, 16),      # head size 40, 144 blocks with edges: the backward with one group of 128 rows
    (80, 2, 160, 257, 2),        # five tiles, both ways with two groups of 64 rows
    (600, 8, 1208, 333, 1),      # head size 75, six tiles: the forward with two groups of 128
    (128, 4, 264, 300, 1),       # head size 32, both ways with two groups of 64
    (320, 5, 640, 128, 20),      # head size 64, 100 whole blocks of one row block each: the backward with one group
    (1200, 16, 408, 257, 6),     # head size 75, 288 blocks: one group
    (200, 2, 400, 260, 1),       # head size 100: the forward with two groups of 128
    (240, 2, 480, 321, 1),       # head size 120, six tiles
], ids=lambda c: "h%d_a%d_f%d_s%d_b%d" % c)
def test_attention_in_groups(cfg):
    hidden, heads, ffn, seq, b = cfg
    run_and_compare(W("groups", "bf16", 1, hidden, heads, ffn, seq, b, 4, 1, 1, "H1", seed=551 + hidden + seq))


@pytest.mark.parametrize("cfg", [
    # hidden, heads, ffn, seq, b       the attention's row blocks per workgroup that only many heads reach
    (256, 4, 512, 128, 128),     # head size 64, 512 whole blocks: 128 rows forward, 64 backward
    (512, 4, 512, 130, 44),      # head size 128, 352 blocks with edges: 64 rows forward and backward
    (72, 3, 136, 33, 64),        # head size 24, 192 blocks: 64 rows backward
    (120, 3, 248, 70, 64),       # head size 40, likewise
], ids=lambda c: "h%d_a%d_f%d_s%d_b%d" % c)
def test_attention_with_many_heads(cfg):
    hidden, heads, ffn, seq, b = cfg
    run_and_compare(W("many", "bf16", 1, hidden, heads, ffn, seq, b, 4, 1, 1, "H1", seed=501 + hidden))


@pytest.mark.parametrize("cfg", [
    (72, 3, 136, 33, 1, 2),      # widths and tokens cut every tile
    (512, 4, 2048, 300, 2, 1),   # 600 tokens ragged, FC1 on 1216 tiles of 32 x 32
    (256, 4, 3464, 300, 2, 1),   # the same with FC1 on tiles of 64 x 64 (2071 of 32 x 32 would be too many)
    (40, 5, 8, 5, 1, 1),         # contractions shorter than one wave's block of 32
    (160, 8, 320, 161, 1, 1),    # head size 20, six blocks of 32 rows (a wave takes two), the last one row long
    (384, 4, 768, 97, 2, 1),     # head size 96
    (200, 2, 400, 64, 1, 1),     # head size 100
    (152, 2, 304, 40, 1, 1),     # head size 76; 152 / 8 = 19 below
    (152, 8, 304, 40, 1, 1),     # head size 19: one wavefront per row
    (1024, 8, 4096, 17, 1, 1),   # gradients on the vector ALUs, bias sums in a launch of their own
], ids=lambda c: "h%d_a%d_f%d_s%d_b%d_L%d" % c)
def test_fp32_tiles(cfg):
    hidden, heads, ffn, seq, b, layers = cfg
    run_and_compare(W("fp32_tiles", "fp32", layers, hidden, heads, ffn, seq, b, 4, 1, 3, "H2", seed=401 + hidden + seq))


def test_fp32_grouped_w_has_the_bits_of_one_by_one_w():
    import paper_2401_10241_amd as zb
    w = W("grp32", "fp32", 2, 72, 3, 200, 50, 1, 4, 3, 6, "H1", seed=29)
    params = zb_inputs.stage_params(w)
    grads = []
    for group in (True, False):
        dev = make_device_stage(w, 6, group_w=group)
        dev.set_params(params)
        dev.begin_iteration(0, 6)
        load_iteration(w, 0, 6, dev)
        dev.run_schedule(4, 3, 6, "H1")   # ends in three consecutive W
        dev.synchronize()
        grads.append(dev.get_tensor(zb.T_FLAT_GRADS).copy())
        dev.close()
    assert np.abs(grads[0]).max() > 0 and grads[0].tobytes() == grads[1].tobytes()


@pytest.mark.parametrize("hidden,heads,ffn,seq,layers,groups", [
    (256, 4, 1024, 160, 2, (9, 1)),  # nine and more microbatches: one layer per W launch instead of both
    (256, 4, 1024, 128, 2, (9, 1)),  # the same at 128 tokens: four waves a tile
    (160, 5, 640, 160, 4, (5, 5)),   # five microbatches: three layers and one instead of all four
    (1024, 8, 4096, 17, 2, (9, 1)),  # gradients on the vector ALUs, bias sums in a launch of their own
], ids=["h256_s160_L2", "h256_s128_L2", "h160_s160_L4", "h1024_s17_L2"])
def test_fp32_w_bits_do_not_depend_on_the_layers_per_launch(hidden, heads, ffn, seq, layers, groups):
    # how many layers share a W launch follows from the number of microbatches and from the pass (the single
    # backward takes one layer at a time); at 160 tokens the waves of a workgroup split K unevenly
    import paper_2401_10241_amd as zb
    m = sum(groups)
    w = W("fp32_bits", "fp32", layers, hidden, heads, ffn, seq, 1, 4, 2, m, "1F1B", seed=37)
    params = zb_inputs.stage_params(w)
    grads = []
    for mode in ("one by one", "groups", "fused"):
        dev = make_device_stage(w, m, pools=(m, m, m))
        dev.set_params(params)
        dev.begin_iteration(0, m)
        load_iteration(w, 0, m, dev)
        for k in range(m):
            dev.forward(k)
            if mode == "fused":
                dev.backward_fused(k)
            else:
                dev.backward_input(k)
                if mode == "one by one":
                    dev.backward_weight(k)
        if mode == "groups":
            k = 0
            for n in groups:
                dev.backward_weight_group(list(range(k, k + n))) if n > 1 else dev.backward_weight(k)
                k += n
        dev.synchronize()
        grads.append(dev.get_tensor(zb.T_FLAT_GRADS).copy())
        dev.close()
    assert np.abs(grads[0]).max() > 0
    for g in grads[1:]:
        assert np.array_equal(g.view(np.uint32), grads[0].view(np.uint32))
