"""hb_batch_loss_static (the entry point that allocates nothing: its workspace is a static device
array of the library) against hb_batch_loss_async on a handle that holds the same parameters, and
against the fp64 oracle.  Two calls in a row share the workspace, the second with a smaller
input: nothing of the first call may leak into the second."""
import numpy as np
import pytest

import hb_inputs as hi
import oracle

pytestmark = pytest.mark.gpu

CASES = [
    # dims, act, loss, B of the first call, B of the second call
    ((54, 512, 512, 512, 512, 7), hi.ACT_SIGMOID, hi.LOSS_SOFTMAX_CE, 4096, 1000),   # fused narrow output layer
    ((70, 65, 129, 67, 2), hi.ACT_RELU, hi.LOSS_LOGISTIC, 321, 33),                 # ragged widths, 2-way logistic
    ((40, 72, 100), hi.ACT_RELU, hi.LOSS_SOFTMAX_CE, 500, 77),                      # wide output: general product + loss kernel
    ((33, 1), hi.ACT_SIGMOID, hi.LOSS_LOGISTIC, 130, 1),                            # no hidden layer
    # networks that fit a workgroup: one block of rows and several, the most layers, and more rows than that kernel takes
    ((54, 32, 7), hi.ACT_SIGMOID, hi.LOSS_SOFTMAX_CE, 2000, 64),
    ((20, 24, 24, 1), hi.ACT_RELU, hi.LOSS_LOGISTIC, 65, 16),
    ((8,) + (10,) * 15 + (4,), hi.ACT_SIGMOID, hi.LOSS_SOFTMAX_CE, 4097, 33),
    ((200, 60, 60, 10), hi.ACT_SIGMOID, hi.LOSS_SOFTMAX_CE, 8200, 300),
]


@pytest.mark.parametrize("dims,act,loss,B1,B2", CASES)
def test_static_loss_equals_handle_loss_on_two_calls_in_a_row(dims, act, loss, B1, B2):
    import torch
    import paper_2004_08771_amd as hb
    rng = np.random.default_rng(4242 + B1)
    params = hi.xavier_uniform_params(dims, rng, bias_scale=0.2)
    X = rng.standard_normal((B1, dims[0]), dtype=np.float32)
    if loss == hi.LOSS_SOFTMAX_CE:
        y = rng.integers(0, dims[-1], size=B1).astype(np.int32)
    else:
        y = (2 * rng.integers(0, 2, size=B1) - 1).astype(np.int32)
    dX, dy = torch.from_numpy(X).cuda(), torch.from_numpy(y).cuda()
    d_params = torch.from_numpy(params).cuda()
    m = hb.Model(dims, act, loss).configure(hb.HB_F32, B1)
    m.set_params(params)
    out = torch.full((2,), float("nan"), device="cuda")
    ref = torch.full((2,), float("nan"), device="cuda")
    # first call: the whole batch; second call: a smaller batch taken from the middle of it
    lo = (B1 - B2) // 2
    calls = [(dX, dy, B1), (dX[lo:lo + B2], dy[lo:lo + B2], B2)]
    for i, (x, t, B) in enumerate(calls):
        hb.batch_loss_static(dims, act, loss, d_params, x, t, B, out[i:i + 1])
    for i, (x, t, B) in enumerate(calls):
        m.batch_loss_async(x, t, B, ref[i:i + 1])
    torch.cuda.synchronize()
    m.destroy()
    got, want = out.cpu().numpy(), ref.cpu().numpy()
    assert np.array_equal(got, want), f"static {got} vs handle {want}"       # the same kernels: bit-identical
    assert np.array_equal(d_params.cpu().numpy(), params)                    # parameters are only read
    for i, (lo_, B) in enumerate([(0, B1), (lo, B2)]):
        l_ref = oracle.batch_loss(dims, act, loss, params, X[lo_:lo_ + B], y[lo_:lo_ + B])
        assert abs(got[i] - l_ref) <= 1e-4 * abs(l_ref), f"call {i}: {got[i]} vs oracle {l_ref}"


def test_static_loss_rejects_what_does_not_fit_and_bad_arguments():
    import torch
    import paper_2004_08771_amd as hb
    dims = (54, 512, 512, 512, 512, 7)
    p = torch.zeros(hi.num_params(dims), device="cuda")
    x = torch.zeros(16, 54, device="cuda")
    y = torch.zeros(16, dtype=torch.int32, device="cuda")
    out = torch.zeros(1, device="cuda")
    with pytest.raises(hb.HbError) as e:      # 16384 x 2056 floats = 135 MB of activations: beyond the workspace
        hb.batch_loss_static(dims, 0, 0, p, x, y, 16384, out)
    assert e.value.code == hb.HB_ERR_UNSUPPORTED
    for args in [(dims, 0, 0, None, x, y, 16, out), (dims, 0, 0, p, None, y, 16, out),
                 (dims, 0, 0, p, x, None, 16, out), (dims, 0, 0, p, x, y, 16, None),
                 (dims, 0, 0, p, x, y, 0, out), ((54,), 0, 0, p, x, y, 16, out),
                 (dims, 0, 0, p.data_ptr() + 4, x, y, 16, out)]:
        with pytest.raises(hb.HbError) as e:
            hb.batch_loss_static(*args)
        assert e.value.code == hb.HB_ERR_INVALID
    hb.batch_loss_static(dims, 0, 0, p, x, y, 16, out)     # zero weights: ln 7
    assert abs(float(out.cpu()[0]) - np.log(7.0)) < 1e-6


def test_static_loss_of_a_small_network_can_be_captured():
    """Kernels only: five replays with eager work of the caller's own between them, each equal to the eager result."""
    import torch
    import paper_2004_08771_amd as hb
    dims, B = (54, 32, 7), 300
    rng = np.random.default_rng(99)
    p = torch.from_numpy(hi.xavier_uniform_params(dims, rng, bias_scale=0.2)).cuda()
    X = torch.from_numpy(rng.standard_normal((B, dims[0]), dtype=np.float32)).cuda()
    y = torch.from_numpy(rng.integers(0, 5, size=B).astype(np.int32)).cuda()
    st = torch.cuda.Stream()
    out, want = torch.zeros(1, device="cuda"), torch.zeros(1, device="cuda")
    other = torch.ones(1 << 16, device="cuda")
    torch.cuda.synchronize()
    hb.batch_loss_static(dims, 0, 0, p, X, y, B, want, st.cuda_stream)
    st.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=st):
        hb.batch_loss_static(dims, 0, 0, p, X, y, B, out, st.cuda_stream)
    for k in range(5):
        out.zero_()
        hb.batch_loss_static((33, 40, 5), 1, 0, p, X, y, 64, other)  # another network in the same workspace
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert float(out) == float(want), k
