"""zb_grad_norm_static (the entry point for callers that cannot allocate) against the gradient-norm step
of zb_optimizer_step_validated, through the C ABI: two calls in a row, the second on a smaller input.

Both run the same fixed-order fp64 sums (one launch up to 2^22 values, three above), so for the same gradient vector
the sum of squares must agree bit for bit and the non-finite flag exactly; the flat gradient of a stage also has a
plain definition (sum of squares of its entries), checked in fp64 to 1e-12 relative."""
import numpy as np
import pytest

import zb_inputs
from zb_testlib import make_device_stage, load_iteration

pytestmark = pytest.mark.gpu


def _stage_gradients(hidden, layers, seed):
    """Runs a small fp32 iteration and returns (flat gradients, local_sq reported by the optimizer step)."""
    import paper_2401_10241_amd as zb
    w = zb_inputs.Workload("noalloc", "fp32", layers, hidden, 4, 4 * hidden, 64, 1, 2, 0, 2, "H1", seed=seed)
    dev = make_device_stage(w)
    dev.set_params(zb_inputs.stage_params(w))
    dev.begin_iteration(0, w.m)
    load_iteration(w, 0, w.m, dev=dev)
    dev.run_schedule(w.p, w.stage, w.m, w.kind)
    flat = dev.get_tensor(zb.T_FLAT_GRADS).copy()
    rep = dev.optimizer_step_validated(0.0, 0.0)
    dev.close()
    return flat, rep


def _static_norm(flat, stream):
    import torch
    import paper_2401_10241_amd as zb
    g = torch.from_numpy(flat).to("cuda:0")
    sq = torch.full((1,), -1.0, dtype=torch.float64, device="cuda:0")
    nf = torch.full((1,), -1, dtype=torch.int32, device="cuda:0")
    torch.cuda.synchronize()
    with torch.cuda.device(0):
        zb.binding.grad_norm_static(g.data_ptr(), g.numel(), sq.data_ptr(), nf.data_ptr(), stream.cuda_stream)
    stream.synchronize()
    return float(sq.item()), int(nf.item())


def test_static_grad_norm_matches_the_optimizer_step_twice_second_smaller():
    import torch
    stream = torch.cuda.Stream(device="cuda:0")
    big, rep_big = _stage_gradients(hidden=256, layers=2, seed=11)
    small, rep_small = _stage_gradients(hidden=128, layers=1, seed=12)
    assert small.size < big.size
    for flat, rep in ((big, rep_big), (small, rep_small)):   # second call: smaller input, same scratch array
        sq, nf = _static_norm(flat, stream)
        assert nf == 0
        assert sq == rep.local_sq, f"{sq!r} != {rep.local_sq!r}"          # same reduction order: same bits
        want = float(np.sum(flat.astype(np.float64) ** 2))
        assert abs(sq - want) <= 1e-12 * want
    # a NaN in the smaller input, after the larger call left its partials behind
    poisoned = small.copy()
    poisoned[poisoned.size // 3] = np.nan
    sq, nf = _static_norm(poisoned, stream)
    assert nf == 1 and np.isnan(sq)
    sq, nf = _static_norm(small, stream)
    assert nf == 0 and sq == rep_small.local_sq


def test_static_grad_norm_rejects_bad_sizes():
    import torch
    import paper_2401_10241_amd as zb
    g = torch.zeros(64, dtype=torch.float32, device="cuda:0")
    sq = torch.zeros(1, dtype=torch.float64, device="cuda:0")
    nf = torch.zeros(1, dtype=torch.int32, device="cuda:0")
    lib = zb.lib
    assert lib.zb_grad_norm_static(g.data_ptr(), 0, sq.data_ptr(), nf.data_ptr(), None) == zb.EINVAL
    assert lib.zb_grad_norm_static(g.data_ptr(), 62, sq.data_ptr(), nf.data_ptr(), None) == zb.EINVAL
    assert lib.zb_grad_norm_static(g.data_ptr(), zb.binding.GRAD_NORM_STATIC_MAX_FLOATS + 4, sq.data_ptr(),
                                   nf.data_ptr(), None) == zb.EINVAL
    assert lib.zb_grad_norm_static(None, 64, sq.data_ptr(), nf.data_ptr(), None) == zb.EINVAL
    assert lib.zb_grad_norm_static(g.data_ptr() + 4, 60, sq.data_ptr(), nf.data_ptr(), None) == zb.EINVAL


@pytest.mark.parametrize("n", [4, 1028, 16384, 16388, 1 << 20, (1 << 22) - 4, 1 << 22, (1 << 22) + 4])
def test_static_grad_norm_at_the_edges_of_its_workgroups(n):
    # one workgroup, two, the most that share a launch, and three launches; three times each, so that every call finds
    # what the one before left behind, with a value that is not finite in the last element of the second
    import torch
    stream = torch.cuda.Stream(device="cuda:0")
    rng = np.random.default_rng(n)
    flat = rng.standard_normal(n).astype(np.float32)
    want = float(np.sum(flat.astype(np.float64) ** 2))
    poisoned = flat.copy()
    poisoned[-1] = np.inf
    first, nf = _static_norm(flat, stream)
    assert nf == 0 and abs(first - want) <= 1e-12 * want   # fp64 sums of n <= 2^22 squares: n * 2^-53 at most
    sq, nf = _static_norm(poisoned, stream)
    assert nf == 1 and sq == np.inf
    again, nf = _static_norm(flat, stream)
    assert nf == 0 and again == first


def test_calls_that_overlap_leave_the_counters_at_zero():
    # Calls on two streams without order between them: their own results are not defined, but every workgroup counts once
    # and calls of one size share a counter that is taken modulo their workgroups, so the calls after them find it at zero.
    # More of them than counters, of sizes that finish in one launch (17, 3, 256, 1 and 2 workgroups) and one that does not;
    # then each size twice, once in a graph captured before the overlap and replayed after it.
    import torch
    import paper_2401_10241_amd as zb
    streams = [torch.cuda.Stream(device="cuda:0") for _ in range(2)]
    sizes = [17 * 16384 - 4, 3 * 16384, 1 << 22, 4, 16388, (1 << 22) + 4]
    g = torch.randn(max(sizes), generator=torch.Generator(device="cuda").manual_seed(3), device="cuda")
    sq = torch.zeros(3, dtype=torch.float64, device="cuda")
    nf = torch.zeros(3, dtype=torch.int32, device="cuda")

    def call(n, out, stream):
        zb.binding.grad_norm_static(g.data_ptr(), n, sq.data_ptr() + 8 * out, nf.data_ptr() + 4 * out, stream.cuda_stream)

    def result(out):
        torch.cuda.synchronize()
        got = float(sq[out].item()), int(nf[out].item())
        sq[out], nf[out] = -1.0, -1
        return got

    torch.cuda.synchronize()
    want, graphs = {}, {}
    for n in sizes:
        call(n, 2, streams[0])
        want[n] = result(2)
        assert want[n][1] == 0 and want[n][0] > 0
        graphs[n] = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graphs[n], stream=streams[0]):
            call(n, 2, streams[0])
        torch.cuda.synchronize()
    for k in range(300):
        for i, stream in enumerate(streams):
            call(sizes[(k * (i + 1)) % len(sizes)], i, stream)
    result(0), result(1)
    for n in sizes:
        call(n, 2, streams[1])
        assert result(2) == want[n], n
        graphs[n].replay()
        assert result(2) == want[n], n
