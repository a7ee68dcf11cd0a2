"""Parity of the HIP path (through the C ABI) with the fp64 CPU oracle on the same seeded
inputs.  Tolerances are the ones the task states: relative 1e-4 on the loss and on the
parameters after one step for fp32 (2e-2 for bf16 storage), per tensor, and the same bound on
the gradient itself (stricter: lr * g is small next to W).  Beside every relative-L2 bound an
element-wise one is asserted, and tensors whose entries are sums that cancel are judged against
the sum of the absolute values of their terms (tests/parity_checks.py)."""
import os

import numpy as np
import pytest

import hb_inputs as hi
import oracle
from oracle import matrix_form as mf
from parity_checks import RHO_BF16, assert_close
from relu_margin import keep_relu_units_off_the_kink

pytestmark = pytest.mark.gpu

TOL_F32 = 1e-4
# every gradient entry against the sum of the absolute values of its terms: fp32 products and
# sums contribute ~1e-7 of it per term, the fast exp / log / reciprocal of the epilogues ~1e-6
TOL_F32_TERMS = 1e-5
LOOP_ORACLE_WORK = 6e8     # batch x weights up to which the plain-loop oracle is the reference


def _torch():
    import torch
    return torch


def _work(dims, B):
    return B * sum(a * b for a, b in zip(dims[:-1], dims[1:]))


def oracle_grad(dims, act, loss, params, X, y):
    """(loss, gradient, per-entry sum of absolute terms).  The plain-loop oracle where it finishes
    in seconds, the matrix form (numpy matmul as a step) beyond; the sums of absolute terms always
    come from the matrix form."""
    l_m, g_m, scale = mf.batch_grad(dims, act, loss, params, X, y, with_error_scale=True)
    if _work(dims, y.size) > LOOP_ORACLE_WORK:
        return l_m, g_m, scale
    if isinstance(X, tuple):
        l, g = oracle.batch_grad_csr(dims, act, loss, params, X[0], X[1], X[2], y)
    else:
        l, g = oracle.batch_grad(dims, act, loss, params, X, y)
    return l, g, scale


# A ReLU unit whose pre-activation lies within EPS_Z x (the sum of the absolute values of its terms)
# of 0 may come out on or off depending on precision and summation order; the oracle then takes
# the decision the kernels took (read back through hb_model_get_activations), and every other
# decision of the kernels must be the oracle's own.  fp32 sums: a few 1e-7 per term.  bf16
# storage: a stored activation that rounds to the neighbouring bf16 value moves the next
# pre-activation by 2^-8 of one term.
EPS_Z_F32 = 1e-5
EPS_Z_BF16 = 2e-4


def relu_decisions(dims, params, X, gpu_acts, eps, store_bf16=False):
    """{l: boolean B x d_l} for mf.batch_grad(relu_on=...): the oracle's own decision [z > 0] where
    |z| >= eps x scale, the kernels' [A_l > 0] inside that band.  Asserts that outside the band the
    kernels decided as the oracle does.  Also returns the number of units inside the band and the
    number of those where the two sides differ."""
    pre, scales = [], []
    mf.forward(dims, hi.ACT_RELU, params, X, store_bf16, pre_activations=pre, pre_activation_scales=scales)
    relu_on, free_n, flipped_n = {}, 0, 0
    for l in range(1, len(dims) - 1):
        z, sc = pre[l - 1], scales[l - 1]
        free = np.abs(z) < eps * sc
        own, gpu = z > 0, gpu_acts[l] > 0
        wrong = (own != gpu) & ~free
        if wrong.any():
            i, j = np.argwhere(wrong)[np.argmax((np.abs(z) / sc)[wrong])]
            raise AssertionError(f"hidden layer {l}: {int(wrong.sum())} ReLU units switched differently from the "
                                 f"oracle although their pre-activation is not within rounding of 0; worst: row {i} "
                                 f"unit {j}, z = {z[i, j]:.3e}, sum of |terms| = {sc[i, j]:.3e}, kernel activation "
                                 f"{gpu_acts[l][i, j]:.3e}")
        relu_on[l] = np.where(free, gpu, own)
        free_n += int(free.sum())
        flipped_n += int((free & (own != gpu)).sum())
    return relu_on, free_n, flipped_n


def gpu_hidden_activations(m, dims, B):
    acts = {}
    for l in range(1, len(dims) - 1):
        acts[l] = np.empty((B, dims[l]), dtype=np.float32)
        m.get_activations(l, B, acts[l])
    return acts


def assert_close_per_tensor(dims, got, ref, tol, what, abs_floor=0.0):
    assert_close(dims, got, ref, tol, what, abs_floor=abs_floor)


def make_model(dims, act, loss, max_B, params):
    import paper_2004_08771_amd as hb
    m = hb.Model(dims, act, loss).configure(hb.HB_F32, max_B)
    assert m.num_params == params.size == hi.num_params(dims)
    m.set_params(np.ascontiguousarray(params, dtype=np.float32))
    return m


def gpu_grad_and_step(dims, act, loss, params, X, y, lr, max_B=None, want_acts=False):
    """(loss from batch_grad, grad, loss from batch_step, params after) on the GPU."""
    torch = _torch()
    B = X.shape[0]
    m = make_model(dims, act, loss, max_B or B, params)
    dX = torch.from_numpy(np.ascontiguousarray(X, dtype=np.float32)).cuda()
    dy = torch.from_numpy(np.ascontiguousarray(y, dtype=np.int32)).cuda()
    dg = torch.full((params.size,), float("nan"), dtype=torch.float32, device="cuda")
    lg = m.batch_grad(dX, dy, B, dg)
    acts = gpu_hidden_activations(m, dims, B) if want_acts else None
    before = np.empty(params.size, dtype=np.float32)
    m.get_params(before)
    assert np.array_equal(before, params.astype(np.float32)), "batch_grad must not touch the replica"
    lf = m.batch_loss(dX, dy, B)
    ls = m.batch_step(dX, dy, B, lr)
    after = np.empty(params.size, dtype=np.float32)
    m.get_params(after)
    m.destroy()
    if want_acts:
        return lg, dg.cpu().numpy(), lf, ls, after, acts
    return lg, dg.cpu().numpy(), lf, ls, after


def check_case(dims, act, loss, params, X, y, lr, max_B=None, tol=TOL_F32, condition_relu=True):
    """condition_relu (ReLU nets): True nudges bias entries until no hidden pre-activation of the
    batch is within rounding of 0, so that fp32 and fp64 take the same decisions; False leaves the
    inputs alone and lets the oracle take the kernels' decision for exactly the units whose
    pre-activation is within rounding of 0 (relu_decisions)."""
    relu = act == hi.ACT_RELU and len(dims) > 2
    if relu and condition_relu:
        params = keep_relu_units_off_the_kink(dims, params, X)
    stats = None
    if relu and not condition_relu:
        lg, g, lf, ls, after, acts = gpu_grad_and_step(dims, act, loss, params, X, y, lr, max_B, want_acts=True)
        relu_on, free_n, flipped_n = relu_decisions(dims, params, X, acts, EPS_Z_F32)
        l_ref, g_ref, scale = mf.batch_grad(dims, act, loss, params, X, y, with_error_scale=True, relu_on=relu_on)
        stats = (free_n, flipped_n)
    else:
        l_ref, g_ref, scale = oracle_grad(dims, act, loss, params, X, y)
        lg, g, lf, ls, after = gpu_grad_and_step(dims, act, loss, params, X, y, lr, max_B)
    p_ref = oracle.sgd_update(params, g_ref, lr)
    for name, v in (("batch_grad", lg), ("batch_loss", lf), ("batch_step", ls)):
        assert abs(v - l_ref) <= tol * max(abs(l_ref), 1e-12), f"{name} loss {v} vs {l_ref}"
    assert_close(dims, g, g_ref, tol, "gradient", scale=scale, tol_scale=TOL_F32_TERMS)
    assert_close(dims, after, p_ref, tol, "parameters after one step", scale=scale, tol_scale=TOL_F32_TERMS,
                 scale_factor=lr, ref_rounding=2.0 ** -23)
    return stats


def _problem(dims, loss, B, seed, bias_scale=0.3):
    rng = np.random.default_rng(seed)
    params = hi.xavier_uniform_params(dims, rng, bias_scale=bias_scale)
    X = rng.standard_normal((B, dims[0]), dtype=np.float32)
    if loss == hi.LOSS_SOFTMAX_CE:
        y = rng.integers(0, dims[-1], size=B).astype(np.int32)
    else:
        y = (2 * rng.integers(0, 2, size=B) - 1).astype(np.int32)
    return params, X, y


F32_KERNELS = ["small", "64", "128x64", "128", "64s", "64x32"]  # hb_plan_f32_kernel
BF16_KERNELS = ["refused", "dma", "128", "128s", "64", "64s"]  # hb_plan_bf16_kernel; S: shifted rows of X, B: batch-major


def check_plan(got, want):
    """The sizes of a case reach the kernels it names -- unless a tuning aid of the environment sends them elsewhere."""
    aids = ("HB_BF16_TILE", "HB_BF16_BMAJ", "HB_BF16_NO_PAIR", "HB_GEMM_SMALL_TILES", "HB_GEMM_SMALL_K", "HB_NO_PAIR")
    assert got == want or any(a in os.environ for a in aids), (got, want)
    return got == want


def f32_plan(dims, B):
    """"forward ...; backward pairs of layers 2 ...; weight gradient of layer 1" of a dense fp32 network."""
    from paper_2004_08771_amd import lib
    name = lambda product, l: F32_KERNELS[lib().hb_plan_f32_kernel(product, dims[l], dims[l - 1], B, B, None)]
    L = len(dims) - 1
    return "; ".join([" ".join(name(0, l) for l in range(1, L + 1)), " ".join(name(1, l) for l in range(2, L + 1)),
                      name(2, 1)])


def small_net_rows(dims, B):
    """Rows per workgroup of a dense fp32 network that fits one, 0: its layers run kernels of their own."""
    import ctypes
    from paper_2004_08771_amd import lib
    return lib().hb_plan_small_net((ctypes.c_int32 * len(dims))(*dims), len(dims), B)


def bf16_plan(dims, B):
    """"forward ...; backward-data of layers 2 ...; weight gradients" of a bf16 network, 16-byte aligned X."""
    from paper_2004_08771_amd import lib
    L = len(dims) - 1

    def name(product, l):
        v = lib().hb_plan_bf16_kernel(product, dims[l], dims[l - 1], B, (l == 1) + 2 * (l == L))
        slices = lib().hb_plan_bf16_dw_slices(dims[l], dims[l - 1], B, 0) if product == 2 else 1
        return (BF16_KERNELS[v & 15] + ("S" if v & 16 else "") + ("B" if v & 32 else "") +
                (f"/{slices}" if slices > 1 else ""))

    return "; ".join(" ".join(name(q, l) for l in range(2 if q == 1 else 1, L + 1)) for q in range(3))


def bf16_pairs(dims, B):
    """{layer: groups of wavefronts} of the weight gradients that share a launch with the next backward product."""
    import ctypes
    from paper_2004_08771_amd import lib
    arr = (ctypes.c_int32 * len(dims))(*dims)
    return {l: n for l in range(1, len(dims)) if (n := lib().hb_plan_bf16_pair(arr, len(dims), B, l))}


# ---------------------------------------------------------------- small shapes, every mode
SMALL = [
    # dims, act, loss, B   (ragged everything: odd widths, B not a tile multiple)
    ((54, 32, 7), hi.ACT_SIGMOID, hi.LOSS_SOFTMAX_CE, 64),
    ((5, 4, 3), hi.ACT_SIGMOID, hi.LOSS_SOFTMAX_CE, 3),
    ((5, 4, 3), hi.ACT_RELU, hi.LOSS_SOFTMAX_CE, 1),
    ((6, 5, 4, 1), hi.ACT_SIGMOID, hi.LOSS_LOGISTIC, 7),
    ((6, 5, 4, 2), hi.ACT_RELU, hi.LOSS_LOGISTIC, 9),
    ((33, 1), hi.ACT_SIGMOID, hi.LOSS_LOGISTIC, 130),          # no hidden layer
    ((33, 10), hi.ACT_SIGMOID, hi.LOSS_SOFTMAX_CE, 257),       # softmax regression
    ((70, 65, 129, 67, 5), hi.ACT_SIGMOID, hi.LOSS_SOFTMAX_CE, 193),
    ((70, 65, 129, 67, 2), hi.ACT_RELU, hi.LOSS_LOGISTIC, 321),
    ((100, 200, 100), hi.ACT_RELU, hi.LOSS_SOFTMAX_CE, 77),    # K = 100 softmax (> 64 lanes)
    ((40, 72, 1000), hi.ACT_RELU, hi.LOSS_SOFTMAX_CE, 50),     # K = 1000 softmax
    ((20, 24, 16), hi.ACT_SIGMOID, hi.LOSS_SOFTMAX_CE, 100),   # widest output of the fused output layer
    ((20, 24, 13), hi.ACT_RELU, hi.LOSS_SOFTMAX_CE, 37),
    ((90, 96, 3), hi.ACT_SIGMOID, hi.LOSS_SOFTMAX_CE, 1500),   # split-wavefront kernels, 3 batch slices
]


@pytest.mark.parametrize("dims,act,loss,B", SMALL)
def test_small_shapes_match_oracle(dims, act, loss, B):
    params, X, y = _problem(dims, loss, B, seed=100 + B + len(dims))
    check_case(dims, act, loss, params, X, y, lr=0.1)


# dense fp32 networks that fit a workgroup, with the rows of its blocks
SMALL_NETS = [
    # one workgroup: row blocks of 16, 32 and 64 rows, full and cut; widths of one block of 16 and one value more or less
    ((16, 15, 17, 16), hi.ACT_SIGMOID, hi.LOSS_SOFTMAX_CE, 16),
    ((1, 33, 1), hi.ACT_SIGMOID, hi.LOSS_LOGISTIC, 17),
    ((63, 48, 31, 2), hi.ACT_RELU, hi.LOSS_LOGISTIC, 32),
    ((54, 32, 7), hi.ACT_SIGMOID, hi.LOSS_SOFTMAX_CE, 33),
    ((65, 47, 3), hi.ACT_RELU, hi.LOSS_SOFTMAX_CE, 64),
    # several: the last with one row; the most of them, and the first size with blocks of 32 and 64 rows
    ((54, 32, 7), hi.ACT_SIGMOID, hi.LOSS_SOFTMAX_CE, 65),
    ((20, 24, 24, 1), hi.ACT_SIGMOID, hi.LOSS_LOGISTIC, 2048),
    ((33, 40, 12, 5), hi.ACT_RELU, hi.LOSS_SOFTMAX_CE, 2049),
    ((9, 17, 16), hi.ACT_SIGMOID, hi.LOSS_SOFTMAX_CE, 4097),
    # up to 64 rows in several blocks of 16: one row over, all of them
    ((64, 64, 64, 64, 5), hi.ACT_SIGMOID, hi.LOSS_SOFTMAX_CE, 33),
    ((100, 64, 64, 64, 64, 64, 4), hi.ACT_RELU, hi.LOSS_SOFTMAX_CE, 64),
    # the most layers; nearly the most parameters of two layers
    ((8,) + (10,) * 15 + (4,), hi.ACT_SIGMOID, hi.LOSS_SOFTMAX_CE, 50),
    ((80, 100, 4), hi.ACT_SIGMOID, hi.LOSS_SOFTMAX_CE, 100),
    # the most layers over several workgroups: every segment of the update kernel
    ((8,) + (10,) * 15 + (4,), hi.ACT_RELU, hi.LOSS_SOFTMAX_CE, 100),
]


@pytest.mark.parametrize("dims,act,loss,B", SMALL_NETS)
def test_networks_that_fit_a_workgroup(dims, act, loss, B):
    assert small_net_rows(dims, B) > 0
    params, X, y = _problem(dims, loss, B, seed=200 + B + len(dims))
    check_case(dims, act, loss, params, X, y, lr=0.1)
    # a smaller batch on the same handle, and rows of X at an odd address: as a handle of its own
    torch, n = _torch(), B // 2 + 1
    buf = torch.zeros(n * dims[0] + 1, device="cuda")
    buf[1:] = torch.from_numpy(X[:n].ravel().copy()).cuda()
    yd, out = torch.from_numpy(y[:n].copy()).cuda(), []
    for max_B, Xd in ((B, buf[1:]), (n, buf[1:].clone())):
        m = make_model(dims, act, loss, max_B, params)
        g = torch.empty(params.size, device="cuda")
        l = m.batch_grad(Xd, yd, n, g)
        out.append((l, g.cpu().numpy()))
        m.destroy()
    assert out[0][0] == out[1][0]
    np.testing.assert_array_equal(out[0][1], out[1][1])


@pytest.mark.parametrize("dims,B", [((480, 16, 2), 32), ((480, 16, 2), 100), ((54, 32, 7), 64), ((40, 33, 2), 2000)])
def test_networks_that_fit_a_workgroup_sum_in_short_chains(dims, B):
    """A_1 of positive rows and weights.  The result's own rounding is 2.5e-8 to 3.4e-8 rms; one running fp32 sum of n such
    terms adds 2^-24 sqrt(n) / 3 and more (n = 54: 1.1e-7 measured, 480: 2.9e-7), sums of sixteen terms that meet in a tree
    2^-24 / 2 at most.  The kernels of the single layers: 4.8e-8 to 5.8e-8."""
    torch, rng = _torch(), np.random.default_rng(5)
    params = rng.random(hi.num_params(dims), dtype=np.float32)
    X, y = rng.random((B, dims[0]), dtype=np.float32), rng.integers(0, 2, size=B).astype(np.int32)
    m = make_model(dims, hi.ACT_RELU, hi.LOSS_SOFTMAX_CE, B, params)
    m.batch_loss(torch.from_numpy(X).cuda(), torch.from_numpy(y).cuda(), B)
    got = gpu_hidden_activations(m, dims, B)[1]
    m.destroy()
    n = dims[0] * dims[1]
    z = X.astype(np.float64) @ params[:n].astype(np.float64).reshape(dims[1], dims[0]).T + params[n:n + dims[1]]
    err = np.sqrt(np.mean((got / z - 1.0) ** 2))
    assert err <= 7.5e-8, f"{err:.2e}"


@pytest.mark.parametrize("K", range(1, 17))
def test_every_width_of_the_fused_output_layer(K):
    """On networks that do not fit a workgroup, one block of rows and one more row."""
    dims, B = (600, 40, K), 9
    assert small_net_rows(dims, B) == 0
    params, X, y = _problem(dims, hi.LOSS_SOFTMAX_CE if K > 2 else hi.LOSS_LOGISTIC, B, seed=900 + K)
    check_case(dims, hi.ACT_SIGMOID, hi.LOSS_SOFTMAX_CE if K > 2 else hi.LOSS_LOGISTIC, params, X, y, lr=0.1)


WIDTHS = [1, 2, 3, 5, 7, 8, 13, 16, 17, 31, 32, 33, 54, 63, 64, 65, 96, 100, 127, 128, 129, 200, 256, 300, 512, 520]
BATCHES = [1, 2, 3, 7, 16, 31, 32, 33, 63, 64, 65, 100, 127, 128, 129, 200, 255, 256, 257, 500, 769, 1000,
           1025, 1500, 2047, 2048, 2049]


def random_dense_case(rng, max_work=3e8):
    """(dims, act, loss, B) around every tile size the kernels use (32, 64, 128, 256 outputs and
    rows; k-tiles of 32 and 64; batch slices of 512; 1 to 16 outputs for the fused output layer,
    more for the general one)."""
    nh = int(rng.integers(0, 4))
    dims = [int(rng.choice(WIDTHS))] + [int(rng.choice(WIDTHS[6:])) for _ in range(nh)]
    loss = int(rng.integers(0, 2))
    dims.append(int(rng.choice([1, 2])) if loss == hi.LOSS_LOGISTIC else int(rng.choice([2, 3, 7, 10, 16, 17, 40, 100])))
    act = int(rng.choice([hi.ACT_SIGMOID, hi.ACT_RELU]))
    B = int(rng.choice(BATCHES))
    work = _work(dims, B)
    if work > max_work:                      # keeps the oracle quick
        B = max(1, int(B * max_work / work))
    return tuple(dims), act, loss, B


def _run_sweep(n_cases, seed, one_case):
    """Runs one_case(rng, case) n_cases times; a case whose ReLU units cannot be moved off the kink
    (RuntimeError from the conditioning helper) is drawn again.  The first failure stops the sweep
    and names its case."""
    rng = np.random.default_rng(seed)
    done = redrawn = 0
    while done < n_cases:
        assert redrawn <= n_cases, "too many cases could not be conditioned"
        try:
            what = one_case(rng, done)
        except RuntimeError as e:
            if "off the kink" not in str(e):
                raise
            redrawn += 1
            continue
        except AssertionError as e:
            raise AssertionError(f"seed {seed}, case {done} ({redrawn} redrawn): {e}") from None
        done += 1


@pytest.mark.parametrize("seed", [3, 20200408, 77])
def test_random_shapes_match_oracle(seed):
    """Seeded sweeps over network shapes and batch sizes.  No seed is special: tensors whose
    entries are sums of cancelling terms (a bias gradient over two classes and two rows) are
    judged against the sum of the absolute values of their terms, not against their own size."""
    state = {}

    def one_case(rng, case):
        dims, act, loss, B = random_dense_case(rng)
        state["what"] = f"dims {dims} act {act} loss {loss} B {B}"
        params, X, y = _problem(dims, loss, B, seed=seed * 1000 + case)
        try:
            check_case(dims, act, loss, params, X, y, lr=0.1)
        except AssertionError as e:
            raise AssertionError(f"{state['what']}: {e}") from None

    _run_sweep(80, seed, one_case)


# ---------------------------------------------------------------- config 1, a whole epoch
def test_config1_one_epoch_of_64_steps():
    torch = _torch()
    cfg = hi.CONFIGS[1]
    X, y = hi.make_dense_dataset(1)
    params = hi.make_params(1)
    m = make_model(cfg.dims, cfg.activation, cfg.loss, cfg.batch, params)
    dX = torch.from_numpy(X).cuda()
    dy = torch.from_numpy(y).cuda()
    p_ref = params.astype(np.float64)
    for s in range(cfg.n_examples // cfg.batch):
        lo, hi_ = s * cfg.batch, (s + 1) * cfg.batch
        l_ref, p_ref = oracle.batch_step(cfg.dims, cfg.activation, cfg.loss, p_ref, X[lo:hi_], y[lo:hi_], cfg.lr)
        l_gpu = m.batch_step(dX[lo:hi_], dy[lo:hi_], cfg.batch, cfg.lr)
        assert abs(l_gpu - l_ref) <= TOL_F32 * abs(l_ref), f"step {s}: {l_gpu} vs {l_ref}"
    after = np.empty(params.size, dtype=np.float32)
    m.get_params(after)
    m.destroy()
    assert_close_per_tensor(cfg.dims, after, p_ref, TOL_F32, "parameters after one epoch")


# ---------------------------------------------------------------- config 2, batch ladder
@pytest.mark.parametrize("B", [16, 48, 256, 1000, 1100, 1999, 2048, 4096, 4097, 5793, 8192, 16384])
def test_config2_batch_sizes(B):
    """Algorithm 2's ladder (powers of two up to the largest batch the benchmark names) and ragged
    sizes a user-set alpha gives (5793 = 8192 / sqrt 2)."""
    cfg = hi.CONFIGS[2]
    X, y = hi.make_dense_dataset(2, 16384 + 123)
    params = hi.make_params(2, bias_scale=0.1)
    off = 123
    check_case(cfg.dims, cfg.activation, cfg.loss, params, X[off:off + B], y[off:off + B],
               lr=0.1 * B / 256, max_B=max(8192, B))


def test_config2_varying_batch_on_one_handle():
    """Adaptive Hogbatch hands the same worker a different B on every call."""
    torch = _torch()
    cfg = hi.CONFIGS[2]
    X, y = hi.make_dense_dataset(2, 4096)
    params = hi.make_params(2)
    m = make_model(cfg.dims, cfg.activation, cfg.loss, 2048, params)
    dX, dy = torch.from_numpy(X).cuda(), torch.from_numpy(y).cuda()
    p_ref = params.astype(np.float64)
    pos = 0
    for B in [2048, 1024, 512, 300, 128, 64, 20]:
        l_ref, p_ref = oracle.batch_step(cfg.dims, cfg.activation, cfg.loss, p_ref, X[pos:pos + B],
                                         y[pos:pos + B], 0.05)
        l_gpu = m.batch_step(dX[pos:pos + B], dy[pos:pos + B], B, 0.05)
        assert abs(l_gpu - l_ref) <= TOL_F32 * abs(l_ref), f"B={B}: {l_gpu} vs {l_ref}"
        pos += B
    after = np.empty(params.size, dtype=np.float32)
    m.get_params(after)
    m.destroy()
    assert_close_per_tensor(cfg.dims, after, p_ref, TOL_F32, "parameters after 7 steps")


# ---------------------------------------------------------------- config 3
@pytest.mark.parametrize("B", [333, 4096])
def test_config3(B):
    cfg = hi.CONFIGS[3]
    X, y = hi.make_dense_dataset(3, B)
    params = hi.make_params(3, bias_scale=0.05)
    check_case(cfg.dims, cfg.activation, cfg.loss, params, X, y, lr=cfg.lr)


def test_config3_relu_inputs_left_alone():
    """Config 3 at B = 4096 without nudging any bias: 12.6 M hidden pre-activations, some of them
    within fp32 rounding of 0.  Every unit the kernels switched differently from the fp64 oracle
    must be one of those (relu_decisions asserts it); with the kernels' decision taken for them,
    gradient and parameters meet the usual bounds."""
    cfg = hi.CONFIGS[3]
    X, y = hi.make_dense_dataset(3, 4096)
    params = hi.make_params(3, bias_scale=0.0)      # zero biases: pre-activations symmetric about the kink
    free_n, flipped_n = check_case(cfg.dims, cfg.activation, cfg.loss, params, X, y, lr=cfg.lr, condition_relu=False)
    assert free_n > 0, "no unit within rounding of the kink: the case does not test what it is meant to"
    assert free_n < 1e-3 * 4096 * 3072


@pytest.mark.parametrize("seed", [5])
def test_random_relu_shapes_with_inputs_left_alone(seed):
    """The fp32 sweep's generator, ReLU only, no conditioning of the inputs."""
    def one_case(rng, case):
        dims, act, loss, B = random_dense_case(rng)
        if len(dims) < 3:
            dims = (dims[0], 64, dims[-1])
        what = f"dims {dims} relu loss {loss} B {B}"
        params, X, y = _problem(dims, loss, B, seed=seed * 1000 + case)
        try:
            check_case(dims, hi.ACT_RELU, loss, params, X, y, lr=0.1, condition_relu=False)
        except AssertionError as e:
            raise AssertionError(f"{what}: {e}") from None

    _run_sweep(40, seed, one_case)


# ---------------------------------------------------------------- async variant + merge
@pytest.mark.parametrize("dims,B", [
    ((54, 512, 512, 512, 512, 512, 512, 2), 1000),            # the paper's covtype network: 6 x 512 hidden, 2 labels
    ((500, 512, 512, 512, 512, 512, 512, 512, 512, 983), 512),  # delicious-shaped: 8 x 512 hidden, 983 outputs
])
def test_paper_shaped_deep_nets(dims, B):
    """The networks of the paper's experiments (Table 2 / Section 7.1: 6 to 8 hidden layers of
    512 sigmoid units; the 983-way output takes the separate loss kernel instead of the fused
    narrow output layer) on synthetic data of their shapes."""
    params, X, y = _problem(dims, hi.LOSS_SOFTMAX_CE, B, seed=900 + len(dims), bias_scale=0.1)
    check_case(dims, hi.ACT_SIGMOID, hi.LOSS_SOFTMAX_CE, params, X, y, lr=0.1)


@pytest.mark.parametrize("dims", [(54, 64, 64, 7), (254, 64, 64, 7)])  # whole in a workgroup; layer by layer
def test_async_step_matches_sync_and_writes_device_loss(dims):
    torch = _torch()
    act, loss = hi.ACT_SIGMOID, hi.LOSS_SOFTMAX_CE
    assert (small_net_rows(dims, 500) > 0) == (dims[0] == 54)
    params, X, y = _problem(dims, loss, 500, seed=5)
    dX, dy = torch.from_numpy(X).cuda(), torch.from_numpy(y).cuda()
    a = make_model(dims, act, loss, 500, params)
    b = make_model(dims, act, loss, 500, params)
    d_loss = torch.zeros(3, dtype=torch.float32, device="cuda")
    for i in range(3):
        a.batch_step_async(dX, dy, 500, 0.2, d_loss[i:i + 1])
    torch.cuda.synchronize()
    sync_losses = [b.batch_step(dX, dy, 500, 0.2) for _ in range(3)]
    pa, pb = np.empty(params.size, np.float32), np.empty(params.size, np.float32)
    a.get_params(pa)
    b.get_params(pb)
    # forward-only loss, asynchronous and synchronous: same kernels, same value, replica untouched
    d_eval = torch.zeros(1, dtype=torch.float32, device="cuda")
    a.batch_loss_async(dX, dy, 500, d_eval)
    torch.cuda.synchronize()
    assert float(d_eval.cpu()[0]) == b.batch_loss(dX, dy, 500)
    pa2 = np.empty(params.size, np.float32)
    a.get_params(pa2)
    np.testing.assert_array_equal(pa2, pa)
    a.destroy()
    b.destroy()
    np.testing.assert_array_equal(d_loss.cpu().numpy(), np.array(sync_losses, dtype=np.float32))
    np.testing.assert_array_equal(pa, pb)   # fixed summation order: bit-identical reruns
    assert sync_losses[2] < sync_losses[0]


@pytest.mark.parametrize("w", [0.0, 1.0, 0.5, 0.25])
def test_model_merge_matches_oracle(w):
    dims = (54, 32, 7)
    rng = np.random.default_rng(17)
    D0 = hi.xavier_uniform_params(dims, rng, 0.2)
    H0 = hi.xavier_uniform_params(dims, rng, 0.2)
    m = make_model(dims, hi.ACT_SIGMOID, hi.LOSS_SOFTMAX_CE, 8, D0)
    H = H0.copy()
    m.model_merge(H, w)
    D = np.empty_like(D0)
    m.get_params(D)
    m.destroy()
    d_ref, h_ref = oracle.model_merge(D0, H0, w)
    if w in (0.0, 1.0):
        np.testing.assert_array_equal(D, d_ref.astype(np.float32))
        np.testing.assert_array_equal(H, h_ref.astype(np.float32))
    else:
        np.testing.assert_allclose(D, d_ref, rtol=1e-6, atol=1e-7)
        np.testing.assert_allclose(H, h_ref, rtol=1e-6, atol=1e-7)
    np.testing.assert_array_equal(D, H)


def test_merge_then_step_round_trip():
    """ExecuteWork on the GPU worker: replica <- global, step, global <- replica."""
    torch = _torch()
    cfg = hi.CONFIGS[1]
    X, y = hi.make_dense_dataset(1, 64)
    glob = hi.make_params(1, bias_scale=0.1)
    m = make_model(cfg.dims, cfg.activation, cfg.loss, 64, np.zeros_like(glob))
    host = glob.copy()
    m.model_merge(host, 0.0)
    l_gpu = m.batch_step(torch.from_numpy(X).cuda(), torch.from_numpy(y).cuda(), 64, 0.1)
    m.model_merge(host, 1.0)
    m.destroy()
    l_ref, p_ref = oracle.batch_step(cfg.dims, cfg.activation, cfg.loss, glob, X, y, 0.1)
    assert abs(l_gpu - l_ref) <= TOL_F32 * abs(l_ref)
    assert_close_per_tensor(cfg.dims, host, p_ref, TOL_F32, "global model after push")


def test_step_with_lr_zero_leaves_replica_bit_identical():
    torch = _torch()
    dims = (54, 48, 7)
    params, X, y = _problem(dims, hi.LOSS_SOFTMAX_CE, 100, seed=9)
    m = make_model(dims, hi.ACT_SIGMOID, hi.LOSS_SOFTMAX_CE, 100, params)
    m.batch_step(torch.from_numpy(X).cuda(), torch.from_numpy(y).cuda(), 100, 0.0)
    after = np.empty_like(params)
    m.get_params(after)
    m.destroy()
    np.testing.assert_array_equal(after, params)


def test_zero_weights_give_log_k_on_gpu():
    torch = _torch()
    import math
    dims = (54, 32, 7)
    _, X, y = _problem(dims, hi.LOSS_SOFTMAX_CE, 64, seed=2)
    m = make_model(dims, hi.ACT_SIGMOID, hi.LOSS_SOFTMAX_CE, 64, np.zeros(hi.num_params(dims), np.float32))
    l = m.batch_loss(torch.from_numpy(X).cuda(), torch.from_numpy(y).cuda(), 64)
    m.destroy()
    assert abs(l - math.log(7)) < 1e-6


def test_gpu_argument_errors():
    import paper_2004_08771_amd as hb
    torch = _torch()
    m = hb.Model((8, 4, 2)).configure(hb.HB_F32, 16)
    x = torch.zeros(16, 8, device="cuda")
    y = torch.zeros(16, dtype=torch.int32, device="cuda")
    for bad_B in (0, -1, 17):
        with pytest.raises(hb.HbError):
            m.batch_step(x, y, bad_B, 0.1)
    with pytest.raises(hb.HbError):
        m.batch_step(x, y, 4, float("nan"))
    with pytest.raises(hb.HbError):
        m.batch_step(None, y, 4, 0.1)
    with pytest.raises(hb.HbError):
        m.model_merge(np.zeros(m.num_params, np.float32), 1.5)
    with pytest.raises(hb.HbError):
        m.configure(hb.HB_F32, 16)
    m.destroy()


# ---------------------------------------------------------------- CSR first layer
def test_label_check_is_opt_in_and_catches_bad_labels():
    """HB_CHECK_LABELS=1 is read when the library sees its first batch call, so the check runs
    in a child process: good labels pass, a class index of d_L and a logistic label of 0 fail
    with HB_ERR_INVALID, and without the variable the same calls go through."""
    import os
    import subprocess
    import sys
    code = r"""
import sys, numpy as np, torch
sys.path.insert(0, %r)
import paper_2004_08771_amd as hb
X = torch.zeros(8, 5, device="cuda")
m = hb.Model((5, 4, 3), hb.HB_ACT_SIGMOID, hb.HB_LOSS_SOFTMAX_CE).configure(hb.HB_F32, 8)
good = torch.tensor([0, 1, 2, 0, 1, 2, 0, 1], dtype=torch.int32, device="cuda")
bad = good.clone(); bad[5] = 3
out = []
out.append(bool(np.isfinite(m.batch_loss(X, good, 8))))
try:
    m.batch_step(X, bad, 8, 0.1); out.append("no error")
except hb.HbError as e:
    out.append(e.code == hb.HB_ERR_INVALID)
lg = hb.Model((5, 1), hb.HB_ACT_SIGMOID, hb.HB_LOSS_LOGISTIC).configure(hb.HB_F32, 8)
pm = torch.tensor([1, -1, 1, -1, 1, -1, 1, -1], dtype=torch.int32, device="cuda")
out.append(bool(np.isfinite(lg.batch_loss(X, pm, 8))))
pm[0] = 0
try:
    lg.batch_loss(X, pm, 8); out.append("no error")
except hb.HbError as e:
    out.append(e.code == hb.HB_ERR_INVALID)
print("RESULT", out)
""" % os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    env = dict(os.environ, HB_CHECK_LABELS="1")
    r = subprocess.run([sys.executable, "-c", code], env=env, capture_output=True, text=True, timeout=300)
    assert "RESULT [True, True, True, True]" in r.stdout, r.stdout + r.stderr
    env.pop("HB_CHECK_LABELS")
    r = subprocess.run([sys.executable, "-c", code], env=env, capture_output=True, text=True, timeout=300)
    assert "RESULT [True, 'no error', True, 'no error']" in r.stdout, r.stdout + r.stderr


def test_index_check_is_opt_in_and_catches_malformed_csr_batches():
    """HB_CHECK_INDICES=1 (read at the first CSR call, hence the child process): a column index
    outside [0, d_0), a row pointer that decreases or does not end at nnz fail with HB_ERR_INVALID
    before any kernel dereferences them; a well-formed batch passes.  (Without the variable the
    indices are trusted, and the malformed batches are not run.)"""
    import os
    import subprocess
    import sys
    code = r"""
import sys, numpy as np, torch
sys.path.insert(0, %r)
import paper_2004_08771_amd as hb
m = hb.Model((50, 8, 2), hb.HB_ACT_RELU, hb.HB_LOSS_LOGISTIC).configure(hb.HB_F32, 8, True)
rp = torch.tensor([0, 2, 2, 5, 6], dtype=torch.int32, device="cuda")
ci = torch.tensor([3, 49, 0, 7, 7, 12], dtype=torch.int32, device="cuda")
va = torch.ones(6, device="cuda")
y = torch.tensor([1, -1, 1, -1], dtype=torch.int32, device="cuda")
out = [bool(np.isfinite(m.batch_step_csr(rp, ci, va, 6, y, 4, 0.1)))]
def refused(rp_, ci_, nnz):
    try:
        m.batch_loss_csr(rp_, ci_, va, nnz, y, 4)
        return "no error"
    except hb.HbError as e:
        return e.code == hb.HB_ERR_INVALID
bad = ci.clone(); bad[1] = 50
out.append(refused(rp, bad, 6))
bad = ci.clone(); bad[4] = -1
out.append(refused(rp, bad, 6))
out.append(refused(torch.tensor([0, 2, 1, 5, 6], dtype=torch.int32, device="cuda"), ci, 6))
out.append(refused(torch.tensor([0, 2, 2, 5, 5], dtype=torch.int32, device="cuda"), ci, 6))
out.append(refused(torch.tensor([1, 2, 2, 5, 6], dtype=torch.int32, device="cuda"), ci, 6))
out.append(bool(np.isfinite(m.batch_loss_csr(rp, ci, va, 6, y, 4))))
print("RESULT", out)
""" % os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    env = dict(os.environ, HB_CHECK_INDICES="1")
    r = subprocess.run([sys.executable, "-c", code], env=env, capture_output=True, text=True, timeout=300)
    assert "RESULT [True, True, True, True, True, True, True]" in r.stdout, r.stdout + r.stderr


def _csr_problem(dims, n_rows, seed, mean_nnz, max_nnz=256, bias_scale=0.2):
    rng = np.random.default_rng(seed)
    rp, ci, va = hi.zipf_csr(n_rows, dims[0], rng, mean_nnz=mean_nnz, max_nnz=max_nnz)
    y = hi.csr_pm1_labels(rp, ci, va, dims[0], rng)
    params = hi.xavier_uniform_params(dims, rng, bias_scale=bias_scale)
    return params, rp, ci, va, y


def check_csr_case(dims, act, loss, params, rp, ci, va, y, lr, tol=TOL_F32, helpers=None):
    import paper_2004_08771_amd as hb
    torch = _torch()
    B = y.size
    if act == hi.ACT_RELU:
        params = keep_relu_units_off_the_kink(dims, params, csr=(rp, ci, va))
    l_ref, g_ref, scale = oracle_grad(dims, act, loss, params, (rp, ci, va), y)
    p_ref = oracle.sgd_update(params, g_ref, lr)

    m = hb.Model(dims, act, loss).configure(hb.HB_F32, B, sparse_first_layer=True)
    m.set_params(params)
    back = np.empty_like(params)
    m.get_params(back)
    np.testing.assert_array_equal(back, params)  # transposed storage round-trips exactly
    d_rp, d_ci = torch.from_numpy(rp).cuda(), torch.from_numpy(ci).cuda()
    d_va, d_y = torch.from_numpy(va).cuda(), torch.from_numpy(y).cuda()
    d_g = torch.full((params.size,), float("nan"), dtype=torch.float32, device="cuda")
    lg = m.batch_grad_csr(d_rp, d_ci, d_va, ci.size, d_y, B, d_g)
    ll = m.batch_loss_csr(d_rp, d_ci, d_va, ci.size, d_y, B)
    d_l = torch.zeros(1, device="cuda")
    m.batch_loss_csr_async(d_rp, d_ci, d_va, ci.size, d_y, B, d_l)
    assert float(d_l.cpu()[0]) == ll
    m.get_params(back)
    np.testing.assert_array_equal(back, params)
    ls = m.batch_step_csr(d_rp, d_ci, d_va, ci.size, d_y, B, lr)
    after = np.empty_like(params)
    m.get_params(after)
    if helpers is not None:
        ran = csr_helper_launches(m, lambda: m.batch_step_csr(d_rp, d_ci, d_va, ci.size, d_y, B, lr))
        assert ran == helpers, ran
    m.destroy()

    for name, v in (("batch_grad_csr", lg), ("batch_loss_csr", ll), ("batch_step_csr", ls)):
        assert abs(v - l_ref) <= tol * abs(l_ref), f"{name} loss {v} vs {l_ref}"
    assert_close(dims, d_g.cpu().numpy(), g_ref, tol, "gradient", scale=scale, tol_scale=TOL_F32_TERMS)
    # a column that occurs in many rows is summed in parts (16 groups of one workgroup, or up to 32
    # atomic adds in the general kernel), each part rounded to fp32: a few units in the last place of W
    assert_close(dims, after, p_ref, tol, "parameters after one step", scale=scale, tol_scale=TOL_F32_TERMS,
                 scale_factor=lr, ref_rounding=2.0 ** -20)
    # weight columns that do not occur in the batch are bit-unchanged
    d0, d1 = dims[0], dims[1]
    untouched = np.setdiff1d(np.arange(d0), ci)
    W1_before = params[:d0 * d1].reshape(d1, d0)
    W1_after = after[:d0 * d1].reshape(d1, d0)
    assert np.array_equal(W1_after[:, untouched], W1_before[:, untouched])
    g1 = d_g.cpu().numpy()[:d0 * d1].reshape(d1, d0)
    assert not g1[:, untouched].any()


@pytest.mark.parametrize("dims,act,B,mean_nnz", [
    ((300, 16, 8, 2), hi.ACT_RELU, 40, 6),
    ((300, 16, 8, 2), hi.ACT_SIGMOID, 40, 6),
    ((1000, 130, 2), hi.ACT_RELU, 700, 30),          # d_1 not a multiple of 4; hot columns > 1 chunk
    ((500, 1), hi.ACT_SIGMOID, 300, 10),             # sparse logistic regression
    ((2000, 64, 64, 1), hi.ACT_RELU, 1, 12),         # B = 1
    # d_1 a multiple of 64: the kernels that give each XCD a 64-float slice of d_1 -- one slice shared
    # by all 8 XCDs (64), by 4 (128), by 2 (256), two slices per XCD (1024); ragged row / chunk groups.
    # (The forward kernel; the weight gradient's in the test of the four launches.)
    ((700, 64, 2), hi.ACT_SIGMOID, 333, 9),
    ((400, 128, 8, 2), hi.ACT_RELU, 100, 10),
    ((900, 256, 2), hi.ACT_RELU, 1001, 40),
    ((600, 1024, 2), hi.ACT_SIGMOID, 70, 12),
])
def test_csr_small_shapes_match_oracle(dims, act, B, mean_nnz):
    params, rp, ci, va, y = _csr_problem(dims, B, seed=300 + B, mean_nnz=mean_nnz)
    check_csr_case(dims, act, hi.LOSS_LOGISTIC, params, rp, ci, va, y, lr=0.1)


@pytest.mark.parametrize("dims,act,B,mean_nnz", [
    ((700, 64, 2), hi.ACT_SIGMOID, 333, 9),
    ((400, 128, 8, 2), hi.ACT_RELU, 100, 10),
    ((900, 256, 2), hi.ACT_RELU, 700, 25),
    ((600, 1024, 2), hi.ACT_SIGMOID, 70, 12),
    ((1000, 130, 2), hi.ACT_RELU, 700, 25),
    ((1000, 132, 2), hi.ACT_SIGMOID, 700, 25),
])
def test_csr_small_shapes_in_four_launches(monkeypatch, dims, act, B, mean_nnz):
    """The kernels of larger batches at sizes that one launch would take: the sliced weight gradient with 8, 4 and 2 XCDs to a
    slice and with two slices to an XCD, and the general one."""
    monkeypatch.setenv("HB_CSC_ONE", "0")
    params, rp, ci, va, y = _csr_problem(dims, B, seed=350 + B, mean_nnz=mean_nnz)
    assert B <= 1024 and ci.size <= 20480
    check_csr_case(dims, act, hi.LOSS_LOGISTIC, params, rp, ci, va, y, lr=0.1, helpers={1, 2, 3, 4, 5})


def test_csr_rows_with_unsorted_and_duplicate_columns():
    """The entries of a row may come in any order and may name a column more than once (their
    products add, in the forward sums and in the weight gradient)."""
    dims = (1000, 130, 64, 2)
    params, rp, ci, va, y = _csr_problem(dims, 700, seed=77, mean_nnz=30)
    rp2, ci2, va2 = hi.scramble_csr_rows(rp, ci, va, np.random.default_rng(78), dup_prob=0.3)
    assert rp2[-1] > rp[-1] and not np.array_equal(ci2[:rp2[1]], np.sort(ci2[:rp2[1]]))
    for act in (hi.ACT_RELU, hi.ACT_SIGMOID):
        check_csr_case(dims, act, hi.LOSS_LOGISTIC, params, rp2, ci2, va2, y, lr=0.1)
    # a row that is one column repeated many times, and a hot column named twice by every row
    rng = np.random.default_rng(79)
    B = 300
    rows_c = [np.full(40, 5, np.int32)] + [np.concatenate([[7, 7], rng.integers(0, 1000, 6)]).astype(np.int32)
                                            for _ in range(B - 1)]
    rp3 = np.concatenate([[0], np.cumsum([r.size for r in rows_c])]).astype(np.int32)
    ci3 = np.concatenate(rows_c)
    va3 = rng.standard_normal(ci3.size).astype(np.float32) * 0.3
    y3 = (2 * rng.integers(0, 2, size=B) - 1).astype(np.int32)
    check_csr_case(dims, hi.ACT_SIGMOID, hi.LOSS_LOGISTIC, params, rp3, ci3, va3, y3, lr=0.1)


@pytest.mark.parametrize("d1", [64, 36])
def test_csr_more_long_columns_than_workgroups_set_aside_for_them(d1):
    """Every one of 600 columns occurs in about a quarter of 1500 rows: more columns of over 128
    entries than the weight-gradient kernel has workgroups for long columns (it walks over the
    rest), in the sliced kernel (d_1 = 64) and in the general one (36)."""
    dims = (600, d1, 2)
    rng = np.random.default_rng(4100 + d1)
    B = 1500
    rows_c = [np.sort(rng.choice(600, size=int(rng.integers(130, 170)), replace=False)).astype(np.int32)
              for _ in range(B)]
    rp = np.concatenate([[0], np.cumsum([r.size for r in rows_c])]).astype(np.int32)
    ci = np.concatenate(rows_c)
    assert np.bincount(ci, minlength=600).min() > 128
    va = (rng.standard_normal(ci.size) * 0.1).astype(np.float32)
    y = (2 * rng.integers(0, 2, size=B) - 1).astype(np.int32)
    params = hi.xavier_uniform_params(dims, rng, bias_scale=0.2)
    check_csr_case(dims, hi.ACT_SIGMOID, hi.LOSS_LOGISTIC, params, rp, ci, va, y, lr=0.1)


def test_csr_weight_gradient_with_fewer_workgroups_than_pieces_of_work(monkeypatch):
    """The sliced weight-gradient kernel is launched with a bounded number of units and walks over
    its work with that stride; three units per slice make every unit take many pieces of each kind
    (long columns with their barriers first, then the others)."""
    monkeypatch.setenv("HB_DW_UNITS", "3")
    dims = (3000, 64, 2)
    params, rp, ci, va, y = _csr_problem(dims, 1200, seed=515, mean_nnz=40)
    counts = np.bincount(ci, minlength=dims[0])
    assert (counts > 1024).sum() >= 1 and (counts > 128).sum() >= 8 and ((counts > 16) & (counts <= 128)).sum() >= 100
    check_csr_case(dims, hi.ACT_SIGMOID, hi.LOSS_LOGISTIC, params, rp, ci, va, y, lr=0.1)


CSR_ONE_LAUNCH = [
    ((3, 8, 2), 5, 2),              # fewer columns than ranges of columns
    ((129, 320, 2), 1024, 18),      # ranges of two columns, the last of one; the most rows; columns of several parts
    ((20001, 64, 2), 300, 60),      # a wide range, columns of 1 .. 4 entries, ranges without any
    ((700, 33, 2), 400, 50),        # rows of delta_1 that are no float4: close to the most entries (20,480)
    ((400, 1028, 1), 130, 20),      # more than a float4 to a thread
    ((900, 256, 2), 400, 40),       # in four launches: slices of d_1 per XCD
]


@pytest.mark.parametrize("one", ["", "0"])
@pytest.mark.parametrize("dims,B,mean_nnz", CSR_ONE_LAUNCH)
def test_csr_batches_with_the_columns_built_in_one_launch_and_in_four(monkeypatch, dims, B, mean_nnz, one):
    monkeypatch.setenv("HB_CSC_ONE", one)
    params, rp, ci, va, y = _csr_problem(dims, B, seed=900 + B, mean_nnz=mean_nnz)
    assert B <= 1024 and ci.size <= 20480, ci.size
    rp, ci, va = hi.scramble_csr_rows(rp, ci, va, np.random.default_rng(B), dup_prob=0.0)
    check_csr_case(dims, hi.ACT_SIGMOID, hi.LOSS_LOGISTIC, params, rp, ci, va, y, lr=0.1,
                   helpers={2} if one == "" else {1, 2, 3, 4, 5})


def csr_helper_launches(m, step):
    """The helper kernels of a CSR step, by the number the profile gives them: {2} the columns in one launch, {1, 2, 3, 4, 5} in four."""
    m.profile_enable(True)
    step()
    stats = m.profile_read()
    m.profile_enable(False)
    return {s["layer"] for s in stats if s["kind"] == 7}


def csr_batch_on_gpu(rp, ci, va, y):
    torch = _torch()
    return [torch.from_numpy(rp).cuda(), torch.from_numpy(ci).cuda(), torch.from_numpy(va).cuda(), ci.size,
            torch.from_numpy(y).cuda(), y.size]


CSR_REPEATED = [
    # columns of one entry up to nearly one per row; values of delta_1 that are a float4 and that are none
    ((2003, 320, 64, 2), 701, 25),
    ((1000, 50, 10, 2), 400, 40),
    # entries named twice by a row, also those of the longest columns
    ((300, 128, 2), 500, 20),
]


@pytest.mark.parametrize("dims,B,mean_nnz", CSR_REPEATED)
def test_small_csr_steps_repeat_bit_for_bit(dims, B, mean_nnz):
    """A column's entries are added in the order of the batch and a weight is rounded once, so that the same steps give the
    same bits: a ReLU unit within rounding of zero is decided alike every time."""
    import paper_2004_08771_amd as hb
    torch = _torch()
    params, rp, ci, va, y = _csr_problem(dims, B, seed=500 + B, mean_nnz=mean_nnz)
    if dims[0] == 300:
        rp, ci, va = hi.scramble_csr_rows(rp, ci, va, np.random.default_rng(B), dup_prob=0.5)
    assert B <= 1024 and ci.size <= 20480 and np.bincount(ci).max() > 256
    batch, runs = csr_batch_on_gpu(rp, ci, va, y), []
    for _ in range(4):
        m = hb.Model(dims, hi.ACT_RELU, hi.LOSS_LOGISTIC).configure(hb.HB_F32, B, sparse_first_layer=True)
        m.set_params(params)
        assert csr_helper_launches(m, lambda: m.batch_step_csr(*batch, 0.05)) == {2}
        g = torch.full((params.size,), float("nan"), device="cuda")
        losses = [m.batch_step_csr(*batch, 0.05) for _ in range(5)] + [m.batch_grad_csr(*batch, g)]
        after = np.empty_like(params)
        m.get_params(after)
        m.destroy()
        runs.append((np.array(losses), after, g.cpu().numpy()))
    for losses, after, g in runs[1:]:
        np.testing.assert_array_equal(losses, runs[0][0])
        np.testing.assert_array_equal(after, runs[0][1])
        np.testing.assert_array_equal(g, runs[0][2])


@pytest.mark.parametrize("d1", [320, 50])
def test_small_csr_batches_with_infinite_deltas(d1):
    """Rows of the wrong class have a delta_1 of +inf (weights of 1e7 and 1e34), the others 0: a column of positive values sums to
    inf or to 0, and no entry past its end makes a NaN of it."""
    import paper_2004_08771_amd as hb
    torch = _torch()
    dims = (300, d1, 4, 2)
    _, rp, ci, va, _ = _csr_problem(dims, 400, seed=61, mean_nnz=30)
    rng = np.random.default_rng(62)
    y = np.where(rng.random(400) < 0.5, 1, -1).astype(np.int32)
    params = np.zeros(hi.num_params(dims), np.float32)
    for (w, b), fill in zip(hi.param_offsets(dims), (1e-7, 1e7, 1e34)):
        params[w:b] = fill
    w3 = hi.param_offsets(dims)[2][0]
    params[w3 + 4:w3 + 8] = -1e34  # the class of y = +1 (Section 7.1: labels -1, +1 are classes 0, 1) is never taken
    m = hb.Model(dims, hi.ACT_RELU, hi.LOSS_LOGISTIC).configure(hb.HB_F32, 400, sparse_first_layer=True)
    m.set_params(params)
    g = torch.full((params.size,), float("nan"), device="cuda")
    m.batch_grad_csr(*csr_batch_on_gpu(rp, ci, va, y), g)
    m.destroy()
    rows = np.repeat(np.arange(400), np.diff(rp))
    wrong = np.bincount(ci, weights=(y[rows] > 0).astype(float), minlength=300)
    assert wrong.max() > 128 and ((wrong > 0) & (wrong < 16)).any() and (wrong == 0).any()
    expect = np.tile(np.where(wrong > 0, np.inf, 0.0).astype(np.float32), (d1, 1))
    np.testing.assert_array_equal(g.cpu().numpy()[:300 * d1].reshape(d1, 300), expect)


@pytest.mark.parametrize("d1,helpers", [(2048, {2}), (2052, {2}), (2560, {1, 2, 3, 4, 5})])
def test_small_csr_batches_of_wide_rows(d1, helpers):
    """Rows of 2048 values and ones that no XCD gets whole slices of: in one launch, a row shared by several workgroups; wider
    rows in slices: in four."""
    dims = (150, d1, 2)
    params, rp, ci, va, y = _csr_problem(dims, 90, seed=d1, mean_nnz=12)
    check_csr_case(dims, hi.ACT_SIGMOID, hi.LOSS_LOGISTIC, params, rp, ci, va, y, lr=0.1, helpers=helpers)


def hottest_columns_first(ci, d0):
    """The columns renamed in the order of their number of entries, as in a vocabulary sorted by frequency."""
    name = np.empty(d0, np.int32)
    name[np.argsort(-np.bincount(ci, minlength=d0), kind="stable")] = np.arange(d0, dtype=np.int32)
    return name[ci]


@pytest.mark.parametrize("dims,B,mean_nnz", [((2003, 50, 10, 2), 701, 25), ((5003, 320, 2), 701, 25), ((5003, 701, 2), 300, 50)])
def test_small_csr_batches_with_the_hot_columns_side_by_side(dims, B, mean_nnz):
    """The column copy and the weight gradient take no longer where the long columns are neighbours: the same batch with its
    columns in random order and sorted by frequency, kernel times.  (By ranges of neighbouring columns: 2.0 to 5.6 times.)"""
    import paper_2004_08771_amd as hb
    params, rp, ci, va, y = _csr_problem(dims, B, seed=40 + B, mean_nnz=mean_nnz)
    by_rank = hottest_columns_first(ci, dims[0])
    assert B <= 1024 and ci.size <= 20480 and np.bincount(by_rank)[:8].min() > 128
    check_csr_case(dims, hi.ACT_SIGMOID, hi.LOSS_LOGISTIC, params, rp, by_rank, va, y, lr=0.1, helpers={2})
    m = hb.Model(dims, hi.ACT_SIGMOID, hi.LOSS_LOGISTIC).configure(hb.HB_F32, B, sparse_first_layer=True)
    m.set_params(params)

    def kernel_ms(columns):
        batch, times = csr_batch_on_gpu(rp, columns, va, y), []
        m.profile_enable(True)
        for _ in range(15):
            m.batch_step_csr(*batch, 0.01)
            times.append(sum(s["total_ms"] for s in m.profile_read()
                             if s["kind"] == 6 or (s["kind"] == 7 and s["layer"] == 2)))
        m.profile_enable(False)
        return float(np.median(times))

    apart, side_by_side = kernel_ms(ci), kernel_ms(by_rank)
    m.destroy()
    assert side_by_side <= 1.4 * apart, (side_by_side, apart)


def test_csr_steps_of_changing_size_on_one_handle():
    """Batches whose columns are built in one launch and in four, in turn: the arrays they leave differ in layout, and each step
    has to use its own.  After every step the parameters, and before it the ReLU decisions, are compared with the oracle's from
    the same parameters."""
    import paper_2004_08771_amd as hb
    dims, lr = (1500, 36, 24, 2), 0.1
    rng = np.random.default_rng(31)
    m = hb.Model(dims, hi.ACT_RELU, hi.LOSS_LOGISTIC).configure(hb.HB_F32, 1500, sparse_first_layer=True)
    params = hi.xavier_uniform_params(dims, rng, bias_scale=0.2)
    m.set_params(params)
    for B, mean_nnz in ((300, 30), (1500, 20), (17, 60), (1024, 15), (1025, 15), (700, 40), (600, 30)):
        rp, ci, va = hi.zipf_csr(B, dims[0], rng, mean_nnz=mean_nnz)
        y = hi.csr_pm1_labels(rp, ci, va, dims[0], rng)
        batch = csr_batch_on_gpu(rp, ci, va, y)
        m.batch_loss_csr(*batch)
        relu_on, _, _ = relu_decisions(dims, params, (rp, ci, va), gpu_hidden_activations(m, dims, B), EPS_Z_F32)
        l_ref, g_ref, scale = mf.batch_grad(dims, hi.ACT_RELU, hi.LOSS_LOGISTIC, params, (rp, ci, va), y, with_error_scale=True,
                                            relu_on=relu_on)
        loss = []
        helpers = csr_helper_launches(m, lambda: loss.append(m.batch_step_csr(*batch, lr)))
        assert helpers == ({2} if B <= 1024 and ci.size <= 20480 else {1, 2, 3, 4, 5})
        after = np.empty_like(params)
        m.get_params(after)
        assert abs(loss[0] - l_ref) <= TOL_F32 * abs(l_ref)
        assert_close(dims, after, oracle.sgd_update(params, g_ref, lr), TOL_F32, f"parameters after {B} rows", scale=scale,
                     tol_scale=TOL_F32_TERMS, scale_factor=lr, ref_rounding=2.0 ** -20)
        params = after
    m.destroy()


@pytest.mark.parametrize("seed", [11, 12])
def test_random_csr_shapes_match_oracle(seed):
    """Seeded sweep over CSR batches: input widths from 10 to 30,000 columns, 1 to 50 stored entries
    per row on average, every third case with unsorted rows and duplicate columns."""
    def one_case(rng, case):
        d0 = int(rng.choice([10, 50, 300, 1000, 5000, 20958, 30000]))
        nh = int(rng.integers(0, 3))
        dims = tuple([d0] + [int(rng.choice([4, 8, 16, 33, 64, 130, 256, 512])) for _ in range(nh)]
                     + [int(rng.choice([1, 2]))])
        B = int(rng.choice([1, 2, 7, 40, 64, 129, 300, 700, 1500, 3000]))
        mean_nnz = min(int(rng.choice([1, 3, 10, 30, 50])), d0)
        act = int(rng.choice([hi.ACT_SIGMOID, hi.ACT_RELU]))
        if B * dims[1] * mean_nnz > 4e7:
            B = max(1, int(4e7 / (dims[1] * mean_nnz)))
        what = f"dims {dims} act {act} B {B} mean_nnz {mean_nnz}"
        params, rp, ci, va, y = _csr_problem(dims, B, seed=seed * 1000 + case, mean_nnz=mean_nnz,
                                             max_nnz=min(256, d0))
        if case % 3 == 2:
            rp, ci, va = hi.scramble_csr_rows(rp, ci, va, rng)
            what += " scrambled"
        try:
            check_csr_case(dims, act, hi.LOSS_LOGISTIC, params, rp, ci, va, y, lr=0.1)
        except AssertionError as e:
            raise AssertionError(f"{what}: {e}") from None

    _run_sweep(40, seed, one_case)


def test_csr_empty_rows_and_empty_batch():
    import paper_2004_08771_amd as hb
    torch = _torch()
    dims = (50, 8, 2)
    params = hi.xavier_uniform_params(dims, np.random.default_rng(1), 0.2)
    rp = np.array([0, 0, 2, 2, 3, 3], dtype=np.int32)
    ci = np.array([1, 7, 3], dtype=np.int32)
    va = np.array([0.5, -1.5, 2.0], dtype=np.float32)
    y = np.array([1, -1, 1, -1, 1], dtype=np.int32)
    check_csr_case(dims, hi.ACT_SIGMOID, hi.LOSS_LOGISTIC, params, rp, ci, va, y, lr=0.3)
    # a batch without any non-zero: only the biases move
    rp0 = np.zeros(4, dtype=np.int32)
    y0 = np.array([1, -1, 1], dtype=np.int32)
    e_i, e_f = np.zeros(0, np.int32), np.zeros(0, np.float32)
    l_ref, p_ref = oracle.batch_step_csr(dims, hi.ACT_SIGMOID, hi.LOSS_LOGISTIC, params, rp0, e_i, e_f, y0, 0.3)
    m = hb.Model(dims, hi.ACT_SIGMOID, hi.LOSS_LOGISTIC).configure(hb.HB_F32, 8, True)
    m.set_params(params)
    l = m.batch_step_csr(torch.from_numpy(rp0).cuda(), None, None, 0, torch.from_numpy(y0).cuda(), 3, 0.3)
    after = np.empty_like(params)
    m.get_params(after)
    m.destroy()
    assert abs(l - l_ref) <= TOL_F32 * abs(l_ref)
    assert_close_per_tensor(dims, after, p_ref, TOL_F32, "parameters after an all-empty batch")


@pytest.mark.parametrize("B", [512, 8192])
def test_config4_csr(B):
    cfg = hi.CONFIGS[4]
    rp, ci, va, y = hi.make_csr_dataset(4, B)
    params = hi.make_params(4, bias_scale=0.05)
    check_csr_case(cfg.dims, cfg.activation, cfg.loss, params, rp, ci, va, y, lr=cfg.lr)


def test_csr_merge_round_trip():
    """set/get/merge see the flat out x in layout although layer 1 is stored transposed."""
    import paper_2004_08771_amd as hb
    dims = (300, 16, 2)
    rng = np.random.default_rng(4)
    D0 = hi.xavier_uniform_params(dims, rng, 0.2)
    H0 = hi.xavier_uniform_params(dims, rng, 0.2)
    for w in (0.0, 1.0, 0.5):
        m = hb.Model(dims, hi.ACT_RELU, hi.LOSS_LOGISTIC).configure(hb.HB_F32, 8, True)
        m.set_params(D0)
        H = H0.copy()
        m.model_merge(H, w)
        D = np.empty_like(D0)
        m.get_params(D)
        m.destroy()
        d_ref, h_ref = oracle.model_merge(D0, H0, w)
        np.testing.assert_allclose(D, d_ref, rtol=1e-6, atol=1e-7)
        np.testing.assert_allclose(H, h_ref, rtol=1e-6, atol=1e-7)
        np.testing.assert_array_equal(D, H)


def test_dense_and_csr_calls_are_not_interchangeable():
    import paper_2004_08771_amd as hb
    torch = _torch()
    x = torch.zeros(4, 8, device="cuda")
    y = torch.ones(4, dtype=torch.int32, device="cuda")
    rp = torch.zeros(5, dtype=torch.int32, device="cuda")
    dense = hb.Model((8, 4, 2), hb.HB_ACT_RELU, hb.HB_LOSS_LOGISTIC).configure(hb.HB_F32, 4)
    sparse = hb.Model((8, 4, 2), hb.HB_ACT_RELU, hb.HB_LOSS_LOGISTIC).configure(hb.HB_F32, 4, True)
    with pytest.raises(hb.HbError):
        dense.batch_step_csr(rp, None, None, 0, y, 4, 0.1)
    with pytest.raises(hb.HbError):
        sparse.batch_step(x, y, 4, 0.1)
    with pytest.raises(hb.HbError):
        sparse.batch_step_csr(rp, None, None, 5, y, 4, 0.1)   # nnz > 0 without arrays
    with pytest.raises(hb.HbError):
        sparse.batch_step_csr(rp, rp, x, 4 * 8 + 1, y, 4, 0.1)  # nnz > B * d_0
    dense.destroy()
    sparse.destroy()


# ---------------------------------------------------------------- bf16 mode
TOL_BF16 = 2e-2        # the task's bound: loss and parameters after one step
TOL_BF16_GRAD = 5e-3   # gradient against the oracle that rounds what the policy stores in bf16
# ... and every entry of it against the sum of the absolute values of its terms: what is left between
# the kernels and that oracle is fp32 against fp64 sums plus the few stored values that land on
# the other side of a bf16 rounding boundary (2^-8 of one term each)
TOL_BF16_TERMS = 1e-3


def oracle_grad_bf16(dims, act, loss, params, X, y):
    """The two references of the bf16 mode on bf16-rounded X and weights: (loss, gradient, sums of
    absolute terms) without any intermediate rounding, and (loss, gradient) with the hidden
    activations and deltas rounded where the policy stores them.  In a ReLU net the reference
    without rounding takes its derivative decisions where the kernels take them, on the STORED
    activation (bf16(max(z, 0)) > 0 under the storage policy): a decision is an integer, and both
    sides take it in the same precision; everything else in that reference is unrounded."""
    Wr = mf.round_weights_bf16(dims, params)
    Xr = mf.bf16_round(X).astype(np.float64)
    relu_on = None
    if act == hi.ACT_RELU and len(dims) > 2:
        stored = mf.forward(dims, act, Wr, Xr, store_bf16=True)
        relu_on = {l: stored[l] > 0 for l in range(1, len(dims) - 1)}
    l_ref, g_plain, scale = mf.batch_grad(dims, act, loss, Wr, Xr, y, with_error_scale=True, relu_on=relu_on)
    if _work(dims, y.size) > LOOP_ORACLE_WORK:
        l_st, g_st = mf.batch_grad(dims, act, loss, Wr, Xr, y, store_bf16=True)
    else:
        l_st, g_st = oracle.batch_grad_bf16_storage(dims, act, loss, params, X, y)
    return (l_ref, g_plain, scale), (l_st, g_st), (Wr, Xr)


def check_bf16_case(dims, act, loss, params, X, y, lr, check_loss_after=True, condition_relu=True):
    """Contract: loss and parameters after one step within 2e-2 of the fp64 oracle run on the
    bf16-rounded inputs (no intermediate rounding), and so is the gradient itself, per tensor.
    Diagnostic: the gradient against the oracle's bf16-storage variant (same rounding points as
    the kernels), much tighter; element-wise bounds beside both.
    condition_relu as in check_case; with False both oracle variants take the kernels' decision
    for the units whose pre-activation (under the storage policy) is within rounding of 0."""
    import paper_2004_08771_amd as hb
    torch = _torch()
    B = X.shape[0]
    relu = act == hi.ACT_RELU and len(dims) > 2
    if relu and condition_relu:
        # a stored activation that lands on the other side of a bf16 rounding boundary (fp32 vs
        # fp64 sums) moves the next layer's z by ~1e-4 of its scale: keep the kink further away
        params = keep_relu_units_off_the_kink(dims, params, X, tau=1e-3, bf16_storage=True)

    m = hb.Model(dims, act, loss).configure(hb.HB_BF16_F32MASTER, B)
    m.set_params(params)
    dX = torch.from_numpy(X).cuda().to(torch.bfloat16)
    dy = torch.from_numpy(y).cuda()
    dg = torch.full((params.size,), float("nan"), dtype=torch.float32, device="cuda")
    lg = m.batch_grad(dX, dy, B, dg)
    acts = gpu_hidden_activations(m, dims, B) if relu and not condition_relu else None
    before = np.empty_like(params)
    m.get_params(before)
    np.testing.assert_array_equal(before, params)
    lf = m.batch_loss(dX, dy, B)
    ls = m.batch_step(dX, dy, B, lr)
    after = np.empty_like(params)
    m.get_params(after)
    # the bf16 weight copies were refreshed by the step: a second loss uses the new weights
    l_after = m.batch_loss(dX, dy, B)
    m.destroy()
    g = dg.cpu().numpy()
    x_gpu = dX.float().cpu().numpy()
    del dX, dg

    stats = None
    if acts is None:
        (l_ref, g_plain, scale), (l_st, g_st), (Wr, Xr) = oracle_grad_bf16(dims, act, loss, params, X, y)
    else:
        Wr = mf.round_weights_bf16(dims, params)
        Xr = mf.bf16_round(X).astype(np.float64)
        relu_on, free_n, flipped_n = relu_decisions(dims, Wr, Xr, acts, EPS_Z_BF16, store_bf16=True)
        stats = (free_n, flipped_n)
        del acts
        l_st, g_st = mf.batch_grad(dims, act, loss, Wr, Xr, y, store_bf16=True, relu_on=relu_on)
        l_ref, g_plain, scale = mf.batch_grad(dims, act, loss, Wr, Xr, y, with_error_scale=True, relu_on=relu_on)
    assert np.array_equal(x_gpu, Xr), "torch's bf16 rounding of X differs from the oracle's"
    p_ref = oracle.sgd_update(params, g_plain, lr)          # update applies to the fp32 master

    for name, v in (("batch_grad", lg), ("batch_loss", lf), ("batch_step", ls)):
        assert abs(v - l_ref) <= TOL_BF16 * abs(l_ref), f"{name} loss {v} vs {l_ref}"
        assert abs(v - l_st) <= 1e-3 * abs(l_st), f"{name} loss {v} vs bf16-storage oracle {l_st}"
    assert_close(dims, after, p_ref, TOL_BF16, "parameters after one step", scale=scale, scale_factor=lr,
                 rho=RHO_BF16)
    assert_close(dims, g, g_plain, TOL_BF16, "gradient (oracle without intermediate rounding)", scale=scale,
                 rho=RHO_BF16)
    assert_close(dims, g, g_st, TOL_BF16_GRAD, "gradient (bf16-storage oracle)", scale=scale,
                 tol_scale=TOL_BF16_TERMS)
    if check_loss_after:
        l_after_ref = mf.batch_loss(dims, act, loss, mf.round_weights_bf16(dims, p_ref.astype(np.float32)), Xr, y)
        # against max(loss, 1): a step that overshoots (B = 1, |x|^2 = d_0) leaves a loss near 0, which
        # is a difference of logits and carries their absolute error, not a relative one
        assert abs(l_after - l_after_ref) <= TOL_BF16 * max(abs(l_after_ref), 1.0), \
            f"loss after the step {l_after} vs {l_after_ref} (the bf16 weight copies were not refreshed?)"
        assert l_after != ls, "the loss did not change after a step: the bf16 weight copies were not refreshed"
    return stats


def test_bf16_overshooting_step_on_one_row():
    """B = 1 without a hidden layer: one step with |x|^2 = 300 takes the loss from 2.85 to 1e-5.
    The gradient and the parameters are compared as everywhere; the loss after the step only
    against max(loss, 1)."""
    dims, loss, B = (300, 40), hi.LOSS_SOFTMAX_CE, 1
    params, X, y = _problem(dims, loss, B, seed=12002)
    check_bf16_case(dims, hi.ACT_RELU, loss, params, X, y, lr=0.05)


BF16_WIDE = [
    # the forward and backward-data products of the two 2050-wide layers take the LDS-direct 256 x 256 x 64
    # kernel (at least 128 tiles: 15 x 9) with a steady-state k loop: forward K = 520 and 2050 (8 and 32
    # k-tiles + tails), backward-data K = 2050 and 10 (tail only); the weight gradient of layer 2, K = B = 3700,
    # is split over the batch (operands batch-major: the row-major deltas and activations, a ragged last
    # k-tile in every slice); ragged edges in every dimension
    ((520, 2050, 2050, 10), hi.ACT_RELU, hi.LOSS_SOFTMAX_CE, 3700, "dma dma 64s; dma dma; 64B dmaB/3 64sB"),
    ((520, 2050, 2050, 10), hi.ACT_SIGMOID, hi.LOSS_SOFTMAX_CE, 3700, "dma dma 64s; dma dma; 64B dmaB/3 64sB"),
    # rows of X that are not 16-byte aligned (d_0 = 516): the first layer's weight gradient cannot
    # read X itself and takes the transposed copies of X and of D_1 (written by the transpose
    # kernel and by the backward-data epilogue of layer 2), split over the batch; layer 2 the row-major tensors
    ((516, 2050, 2050, 10), hi.ACT_RELU, hi.LOSS_SOFTMAX_CE, 5200, "128 dma 64s; dma dma; dma/5 dmaB/3 64sB"),
]


@pytest.mark.parametrize("dims,act,loss,B,plan", BF16_WIDE)
def test_bf16_wide_layers_with_many_k_tiles(dims, act, loss, B, plan):
    check_plan(bf16_plan(dims, B), plan)
    params, X, y = _problem(dims, loss, B, seed=600 + B + len(dims), bias_scale=0.1)
    stats = check_bf16_case(dims, act, loss, params, X, y, lr=0.1, condition_relu=False)
    if act == hi.ACT_RELU:
        free_n, flipped_n = stats
        assert 0 < free_n < 0.02 * B * (dims[1] + dims[2]), f"{free_n} units within rounding of the kink"


def test_bf16_more_tiles_than_compute_units_and_not_a_multiple():
    """5000 x 4096 outputs are 20 x 16 = 320 tiles of 256 x 256 on 256 compute units: the
    persistent LDS-direct kernel gives 64 workgroups two tiles and the others one, the last tile
    row is cut by the end of the batch (5000 = 19 x 256 + 136), and every workgroup that takes a
    second tile finds LDS as its first one left it."""
    dims, B = (264, 4096, 4096, 5), 5000
    params, X, y = _problem(dims, hi.LOSS_SOFTMAX_CE, B, seed=1234, bias_scale=0.1)
    check_bf16_case(dims, hi.ACT_RELU, hi.LOSS_SOFTMAX_CE, params, X, y, lr=0.1, condition_relu=False)


@pytest.mark.parametrize("B", [5, 37, 64, 100])
def test_bf16_batch_shorter_than_a_k_tile_in_the_batch_major_weight_gradient(B):
    """dW_2 is 2050 x 4096 (144 tiles of 256 x 256: the LDS-direct kernel with batch-major operands)
    and contracts over B rows: fewer than one k-tile of 64 (only the masked tail runs), exactly
    one, or one and a tail."""
    dims = (264, 4096, 2050, 5)
    params, X, y = _problem(dims, hi.LOSS_SOFTMAX_CE, B, seed=900 + B, bias_scale=0.1)
    check_bf16_case(dims, hi.ACT_RELU, hi.LOSS_SOFTMAX_CE, params, X, y, lr=0.05, condition_relu=False)


@pytest.mark.parametrize("B", [130, 259, 3841, 3842, 3843])
def test_bf16_relu_batch_edges_of_the_backward_data_epilogue(B):
    """The backward-data epilogue applies the ReLU decisions the forward epilogue left as bits, 16 per
    lane and 32 x 32 block of the activations; a block cut by the end of the batch or of a row is
    written and read under guards, and in the last group of four rows of a ragged batch one, two
    or three exist (B mod 4 = 1, 2, 3).  130 and 259 rows run the kernel of small tiles, 3841-3843 the
    LDS-direct 256 x 256 kernel (15 full tile rows and one row tile holding 1-3 rows), with
    2050 = 8 x 256 + 2 columns: ragged in both directions."""
    dims = (264, 2050, 520, 5)
    params, X, y = _problem(dims, hi.LOSS_SOFTMAX_CE, B, seed=700 + B, bias_scale=0.1)
    check_bf16_case(dims, hi.ACT_RELU, hi.LOSS_SOFTMAX_CE, params, X, y, lr=0.1, condition_relu=False)


@pytest.mark.parametrize("act", [hi.ACT_RELU, hi.ACT_SIGMOID])
def test_bf16_one_replica_through_changing_batch_sizes(act):
    """What Adaptive Hogbatch does to the GPU worker: ONE replica, configured for the largest batch,
    takes steps on batches of changing size.  The sizes move the weight gradients between the kernel of
    small tiles (one or two groups of wavefronts) and, at 6100 rows, the LDS-direct one split over the batch,
    and the other products between 64 x 64, 128 x 128 and LDS-direct tiles, so every step finds the buffers as
    another form left them.  Each step is compared with an oracle step from the replica's parameters
    before it (read back), so errors do not add up over the ladder."""
    import paper_2004_08771_amd as hb
    torch = _torch()
    dims, loss, lr = (264, 2050, 520, 5), hi.LOSS_SOFTMAX_CE, 0.1
    sizes = [300, 2500, 64, 6100, 1000, 4096, 2049, 1]
    plans = [bf16_plan(dims, B) for B in sizes]
    check_plan("dmaB/5" in plans[3] and "dma" in plans[5] and plans[1].startswith("128 64 ") and len(set(plans)) >= 5, True)
    rng = np.random.default_rng(4242 + act)
    params = hi.xavier_uniform_params(dims, rng, bias_scale=0.1)
    m = hb.Model(dims, act, loss).configure(hb.HB_BF16_F32MASTER, max(sizes))
    m.set_params(params)
    try:
        for step, B in enumerate(sizes):
            X = rng.standard_normal((B, dims[0]), dtype=np.float32)
            y = rng.integers(0, dims[-1], size=B).astype(np.int32)
            before = np.empty_like(params)
            m.get_params(before)
            dX = torch.from_numpy(X).cuda().to(torch.bfloat16)
            dy = torch.from_numpy(y).cuda()
            ls = m.batch_step(dX, dy, B, lr)
            after = np.empty_like(params)
            m.get_params(after)
            Wr = mf.round_weights_bf16(dims, before)
            Xr = mf.bf16_round(X).astype(np.float64)
            relu_on = None
            if act == hi.ACT_RELU:
                acts = gpu_hidden_activations(m, dims, B)
                relu_on, _, _ = relu_decisions(dims, Wr, Xr, acts, EPS_Z_BF16, store_bf16=True)
            l_ref, g_ref, scale = mf.batch_grad(dims, act, loss, Wr, Xr, y, with_error_scale=True, relu_on=relu_on)
            p_ref = oracle.sgd_update(before, g_ref, lr)
            what = f"step {step}, B = {B}"
            assert abs(ls - l_ref) <= TOL_BF16 * abs(l_ref), f"{what}: loss {ls} vs {l_ref}"
            assert_close(dims, after, p_ref, TOL_BF16, f"{what}: parameters after the step", scale=scale,
                         scale_factor=lr, rho=RHO_BF16)
            # the step itself, not only its sum with the old parameters: lr * g is small next to W
            assert_close(dims, (before.astype(np.float64) - after) / lr, g_ref, TOL_BF16, f"{what}: applied gradient",
                         scale=scale, rho=RHO_BF16)
    finally:
        m.destroy()


@pytest.mark.parametrize("seed", [21, 22])
def test_random_bf16_shapes_match_oracle(seed):
    """Seeded sweep of the bf16 mode over the same shape generator as the fp32 sweep."""
    def one_case(rng, case):
        dims, act, loss, B = random_dense_case(rng)
        what = f"dims {dims} act {act} loss {loss} B {B}"
        params, X, y = _problem(dims, loss, B, seed=seed * 1000 + case)
        try:
            check_bf16_case(dims, act, loss, params, X, y, lr=0.05)
        except AssertionError as e:
            raise AssertionError(f"{what}: {e}") from None

    _run_sweep(50, seed, one_case)


def test_config5_bf16_reduced_batch():
    cfg = hi.CONFIGS[5]
    B = 160                                   # one full 128-row tile and a ragged tail
    X, y = hi.make_dense_dataset(5, B)
    params = hi.make_params(5, bias_scale=0.02)
    check_bf16_case(cfg.dims, cfg.activation, cfg.loss, params, X, y, lr=cfg.lr)


@pytest.mark.parametrize("B", [2048, 16384])
def test_config5_bf16_at_size(B):
    """Config 5 (2048-4096-4096-4096-1000) at the batch sizes where all three products of the
    4096-wide layers run the LDS-direct kernel (B = 2048: 128 tiles of 256 x 256) and at the
    size the benchmark names (B = 16384), against the oracle in matrix form (4.25 TFLOP of fp64
    matmul at the full size: about a minute on the host's cores)."""
    cfg = hi.CONFIGS[5]
    X, y = hi.make_dense_dataset(5, B)
    params = hi.make_params(5, bias_scale=0.02)
    check_bf16_case(cfg.dims, cfg.activation, cfg.loss, params, X, y, lr=cfg.lr, check_loss_after=(B <= 2048),
                    condition_relu=False)


def test_config5_bf16_full_batch_equals_mean_of_sub_batches():
    """The mean over the batch is linear, and 1/B scaling by a power of two commutes with bf16
    rounding, so the gradient of the whole batch (B = 16384) must equal the mean of the gradients
    of its four quarters up to fp32 summation order: a consistency check of the batch split of the
    weight-gradient products, beside the oracle comparison above."""
    import paper_2004_08771_amd as hb
    torch = _torch()
    cfg = hi.CONFIGS[5]
    B, parts = cfg.batch, 4
    X, y = hi.make_dense_dataset(5, B)
    params = hi.make_params(5, bias_scale=0.02)
    m = hb.Model(cfg.dims, cfg.activation, cfg.loss).configure(hb.HB_BF16_F32MASTER, B)
    m.set_params(params)
    dX = torch.from_numpy(X).cuda().to(torch.bfloat16)
    dy = torch.from_numpy(y).cuda()
    g_full = torch.empty(params.size, dtype=torch.float32, device="cuda")
    l_full = m.batch_grad(dX, dy, B, g_full)
    g_sum = torch.zeros_like(g_full)
    g_part = torch.empty_like(g_full)
    l_sum, q = 0.0, B // parts
    for i in range(parts):
        l_sum += m.batch_grad(dX[i * q:(i + 1) * q], dy[i * q:(i + 1) * q], q, g_part)
        g_sum += g_part
    m.destroy()
    assert abs(l_full - l_sum / parts) <= 1e-5 * abs(l_full)
    assert abs(l_full - np.log(1000.0)) < 0.5          # random labels, small weights
    assert_close_per_tensor(cfg.dims, g_full.cpu().numpy(), (g_sum / parts).cpu().numpy(), 2e-3,
                            "full-batch gradient vs mean of quarter-batch gradients", abs_floor=1e-9)


@pytest.mark.parametrize("bf16,dims", [(False, (40, 96, 64, 5)), (True, (40, 96, 64, 5)),
                                       (False, (340, 96, 64, 5))])  # whole in a workgroup; bf16; layer by layer
def test_step_can_be_captured_in_a_graph_and_replays_like_eager_steps(bf16, dims):
    """hb_batch_step_async records kernels only (no memset or copy nodes, no allocation, no
    synchronisation), so a caller may capture it.  A captured step is replayed five times, with
    eager work and synchronisations of the caller's own in between; after every replay the
    replica equals, bit for bit, that of a second handle taking the same steps eagerly."""
    import paper_2004_08771_amd as hb
    torch = _torch()
    act, loss, B = hi.ACT_SIGMOID, hi.LOSS_SOFTMAX_CE, 200
    assert bf16 or (small_net_rows(dims, B) > 0) == (dims[0] == 40)
    rng = np.random.default_rng(77)
    X = rng.standard_normal((B, dims[0])).astype(np.float32)
    y = rng.integers(0, dims[-1], size=B).astype(np.int32)
    params = hi.xavier_uniform_params(dims, rng, bias_scale=0.1)
    dtype = hb.HB_BF16_F32MASTER if bf16 else hb.HB_F32
    st = torch.cuda.Stream()
    with torch.cuda.stream(st):
        dX = torch.from_numpy(X).cuda()
        if bf16:
            dX = dX.to(torch.bfloat16)
        dy = torch.from_numpy(y).cuda()
        dl_g, dl_e = torch.zeros(1, device="cuda"), torch.zeros(1, device="cuda")
        other = torch.ones(1 << 16, device="cuda")
    st.synchronize()
    eager = hb.Model(dims, act, loss).configure(dtype, B, stream=st.cuda_stream)
    graphed = hb.Model(dims, act, loss).configure(dtype, B, stream=st.cuda_stream)
    eager.set_params(params)
    graphed.set_params(params)
    graphed.batch_step_async(dX, dy, B, 0.0, dl_g)       # lr = 0: anything created lazily exists before the capture
    st.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=st):
        graphed.batch_step_async(dX, dy, B, 0.2, dl_g)
    pe, pg = np.empty_like(params), np.empty_like(params)
    graphed.get_params(pg)
    np.testing.assert_array_equal(pg, params)            # capturing ran nothing
    for k in range(5):
        g.replay()
        eager.batch_step_async(dX, dy, B, 0.2, dl_e)
        with torch.cuda.stream(st):
            other.mul_(1.0001)                           # the caller's own eager work between replays
        torch.cuda.synchronize()
        eager.get_params(pe)
        graphed.get_params(pg)
        np.testing.assert_array_equal(pg, pe, err_msg=f"replay {k}")
        assert float(dl_g.cpu()[0]) == float(dl_e.cpu()[0])
    assert not np.array_equal(pe, params)
    eager.destroy()
    graphed.destroy()



# ---------------------------------------------------------------- fp32 products as bf16 planes
F32_EDGES = [
    # contractions of a single partial k-tile (17, 31, 20, 33 = 32 + 1)
    ((31, 40, 33, 20), hi.ACT_SIGMOID, 17, "64 64 64; 128x64 128x64; 64"),
    # whole k-tiles forward, a lone partial one over the batch
    ((32, 64, 64, 17), hi.ACT_RELU, 31, "64 small small; small 128x64; 64"),
    # 64 x 64 by two groups backward, both operands cut, rows not 16-byte aligned
    ((100, 130, 65, 20), hi.ACT_SIGMOID, 2561, "small small small; 64s 64s; small"),
    # 64 x 64 by one group forward, four k-tiles, the partial one first
    ((100, 330, 290, 40), hi.ACT_SIGMOID, 2561, "64 64s small; 128x64 64s; small"),
    # the same backward; 128 x 64 forward
    ((97, 257, 129, 33), hi.ACT_RELU, 4099, "128x64 64s small; 64 64s; small"),
    # 128 x 128 backward, two values short of a 16-byte row
    ((129, 520, 514, 40), hi.ACT_SIGMOID, 8200, "128x64 64s small; 128 128x64; 128"),
    # 128 x 128 forward, rows and columns cut
    ((100, 500, 500, 40), hi.ACT_RELU, 8150, "128 128 small; 128 128x64; small"),
    # 64 x 64 by two groups: nine k-tiles, the partial one first
    ((265, 258, 257, 40), hi.ACT_SIGMOID, 1030, "small small small; 64s 64s; small"),
    # ten k-tiles, rows and columns cut
    ((300, 290, 270, 12), hi.ACT_RELU, 2100, "64s 64s small; 128x64 64s; 128"),
    # weight gradients on their own: 64 x 64, by two groups, 128 x 64
    ((1100, 100, 40), hi.ACT_SIGMOID, 2101, "small small; 64s; 64"),
    ((1020, 63, 40), hi.ACT_SIGMOID, 8201, "small 64; 64s; 64s"),
    ((100, 130, 40), hi.ACT_SIGMOID, 8201, "128x64 small; 64s; 128x64"),
]


F32_LONG_FORWARD = [
    # tiles of 64 x 32 by four groups: 17 k-tiles, the partial one first, and 9 more than a row of groups; rows and columns cut
    ((515, 546, 513, 4), hi.ACT_SIGMOID, 577, ["64x32", "64x32"]),
    # the other line: 128 tiles over less than 768
    ((512, 512, 4), hi.ACT_SIGMOID, 961, ["small"]),
    # whole k-tiles, one row in the second tile, a wide output
    ((512, 2560, 4), hi.ACT_RELU, 65, ["64x32"]),
    # the lines: 80 and 72 tiles, fp32 MFMAs; one row of tiles, however many; 156, but 312 of 64 x 32: 64 x 64 by two groups
    ((512, 512, 4), hi.ACT_SIGMOID, 577, ["64x32"]),
    ((512, 512, 4), hi.ACT_SIGMOID, 576, ["small"]),
    ((512, 5120, 4), hi.ACT_SIGMOID, 64, ["small"]),
    ((800, 768, 4), hi.ACT_SIGMOID, 800, ["64s"]),
]


@pytest.mark.parametrize("dims,act,B,kernels", F32_LONG_FORWARD)
def test_long_forward_products_of_few_tiles(dims, act, B, kernels):
    from paper_2004_08771_amd import lib
    got = [F32_KERNELS[lib().hb_plan_f32_kernel(0, dims[l], dims[l - 1], B, B, None)] for l in range(1, len(dims) - 1)]
    check_plan(got, kernels)
    params, X, y = _problem(dims, hi.LOSS_SOFTMAX_CE, B, seed=60 + B)
    check_case(dims, act, hi.LOSS_SOFTMAX_CE, params, X, y, lr=0.1, condition_relu=False)


F32_FEW_ROWS = [
    # the backward-data product's workgroups first (contraction 1100 against 17 rows) ...
    ((20, 1100, 1100, 3), hi.ACT_SIGMOID, 17, "64 small small; small 128x64; 128x64"),
    # ... also with 64 tiles of 64 x 64 (256 of 32 x 32); rows and columns cut
    ((20, 1020, 1100, 3), hi.ACT_RELU, 225, "64 small small; small 128x64; small"),
    # the weight gradient's first: as long a contraction
    ((20, 200, 300, 3), hi.ACT_SIGMOID, 301, "64 small small; small 64s; small"),
    # more than 2^24 weights and fewer than 64 rows: two launches
    ((3, 4100, 4100, 2), hi.ACT_SIGMOID, 5, "64 small small; small 128x64; 128x64"),
]


@pytest.mark.parametrize("dims,act,B,plan", F32_FEW_ROWS)
def test_backward_of_few_rows(dims, act, B, plan):
    """Both orders of the workgroups in the paired launch of small tiles, and the launch of the two products apart."""
    check_plan(f32_plan(dims, B), plan)
    params, X, y = _problem(dims, hi.LOSS_SOFTMAX_CE, B, seed=40 + B)
    check_case(dims, act, hi.LOSS_SOFTMAX_CE, params, X, y, lr=0.1, condition_relu=False)


@pytest.mark.parametrize("dims,act,B", [
    # 16 x 16 blocks; contractions of 2, 8 and 16 pieces of 32 and one value more; a wavefront to each block of dW (17 rows)
    ((65, 257, 513, 67, 4), hi.ACT_SIGMOID, 17),
    ((66, 255, 511, 64, 3), hi.ACT_RELU, 16),
    # dW by workgroups over 33 rows (wavefronts without any) and 100; 16 x 16 forward only, 32 x 32 backward
    ((64, 300, 70, 20), hi.ACT_SIGMOID, 33),
    ((90, 420, 300, 5), hi.ACT_RELU, 200),
    # 32 x 32 blocks throughout, more than one slice of the batch in dW_1
    ((300, 520, 610, 9), hi.ACT_SIGMOID, 523),
    # a wavefront to each of 1056 blocks over 40 rows
    ((70, 1000, 1030, 3), hi.ACT_RELU, 40),
])
def test_small_products_at_block_edges(dims, act, B):
    """Both block sizes of the small fp32 products and both forms of their weight gradient, rows and contractions cut."""
    params, X, y = _problem(dims, hi.LOSS_SOFTMAX_CE, B, seed=60 + B)
    check_case(dims, act, hi.LOSS_SOFTMAX_CE, params, X, y, lr=0.1, condition_relu=act == hi.ACT_RELU)


def f32_small_forms(dims, B):
    """"forward ...; backward pairs of layers 2 ...; weight gradient of layer 1": block, s: through LDS, w1 / w2: a wavefront
    to each block of the weight gradient over up to 64 / 128 rows; -: no small product."""
    from paper_2004_08771_amd import lib

    def name(product, l):
        v = lib().hb_plan_f32_small_form(product, dims[l], dims[l - 1], B, B)
        return f"{v & 63}{'s' if v & 64 else ''}{['', 'w1', 'w2'][v >> 7]}" if v else "-"

    L = len(dims) - 1
    return "; ".join([" ".join(name(0, l) for l in range(1, L + 1)), " ".join(name(1, l) for l in range(2, L + 1)), name(2, 1)])


F32_SMALL = [
    # pairs with 16 x 16 blocks: weight gradient by workgroups, by a wavefront to each block over 33 .. 64 and 65 .. 128 rows
    ((70, 300, 300, 40), hi.ACT_SIGMOID, 65, "16 16 16; 16 -; 32"),
    ((70, 700, 640, 40), hi.ACT_SIGMOID, 48, "16 16 16; 16w1 -; -"),
    ((70, 700, 640, 40), hi.ACT_RELU, 65, "16 16 16; 16w2 -; 32"),
    ((70, 700, 640, 40), hi.ACT_SIGMOID, 73, "16 16 16; 16w2 -; 32"),
    # the same with 32 x 32 blocks, at the most rows of each
    ((70, 600, 600, 40), hi.ACT_RELU, 130, "16 16 16; 32 -; 32"),
    ((70, 1040, 1040, 40), hi.ACT_SIGMOID, 64, "16 16 16; 32w1 -; 32"),
    ((70, 1040, 1040, 40), hi.ACT_RELU, 127, "32 32 16; 32w2 -; 32"),
    # the weight gradient of a first layer of 800 blocks on its own: 64 rows, 128 rows and one more
    ((1000, 800, 20), hi.ACT_SIGMOID, 64, "16 16; -; 32w1"),
    ((1000, 800, 20), hi.ACT_RELU, 128, "16 16; -; 32w2"),
    ((1000, 800, 20), hi.ACT_SIGMOID, 129, "16 16; -; 32"),
    # forward by 32 x 32 blocks straight from memory and through LDS
    ((70, 500, 500, 40), hi.ACT_SIGMOID, 300, "32 32 16; 32 -; 32"),
    ((70, 500, 500, 40), hi.ACT_RELU, 1000, "32s 32s 16; - -; 32"),
]


@pytest.mark.parametrize("dims,act,B,forms", F32_SMALL)
def test_forms_of_small_products(dims, act, B, forms):
    check_plan(f32_small_forms(dims, B), forms)
    params, X, y = _problem(dims, hi.LOSS_SOFTMAX_CE, B, seed=700 + B)
    check_case(dims, act, hi.LOSS_SOFTMAX_CE, params, X, y, lr=0.1, condition_relu=False)


def _padded(dims, wide, params, X):
    """The same ReLU network with zero columns of X or hidden units without weights up to `wide`."""
    P, off = [], 0
    for l in range(1, len(dims)):
        W, b = np.zeros((wide[l], wide[l - 1]), np.float32), np.zeros(wide[l], np.float32)
        n = dims[l] * dims[l - 1]
        W[:dims[l], :dims[l - 1]] = params[off:off + n].reshape(dims[l], dims[l - 1])
        b[:dims[l]] = params[off + n:off + n + dims[l]]
        off += n + dims[l]
        P += [W.ravel(), b]
    Xw = np.zeros((X.shape[0], wide[0]), np.float32)
    Xw[:, :dims[0]] = X
    return np.concatenate(P), Xw


SAME_SUMS = [
    # the weight gradient of layer 1 by workgroups, and by a wavefront to each block over 64 and over 100 rows
    ((512, 512, 40), (800, 512, 40), 64, "16 16; -; 32", "16 16; -; 32w1"),
    ((512, 512, 40), (1220, 512, 40), 100, "16 16; -; 32", "16 16; -; 32w2"),
    # 16 x 16 and 32 x 32 blocks of the backward-data product; the weight gradient of the same launch in both forms
    ((70, 512, 512, 40), (70, 804, 512, 40), 100, "16 16 16; 16 -; 32", "16 16 16; 32 -; 32"),
    ((70, 512, 512, 40), (70, 1300, 512, 40), 100, "16 16 16; 16 -; 32", "32 16 16; 32w2 -; 32"),
]


@pytest.mark.parametrize("dims,wide,B,forms,wide_forms", SAME_SUMS)
def test_forms_of_small_products_add_the_same_sums(dims, wide, B, forms, wide_forms):
    """Zeros added to a contraction change no sum, so both networks give the same gradient, bit for bit."""
    torch = _torch()
    if not (check_plan(f32_small_forms(dims, B), forms) and check_plan(f32_small_forms(wide, B), wide_forms)):
        pytest.skip("a tuning aid sends the products to other kernels")
    params, X, y = _problem(dims, hi.LOSS_SOFTMAX_CE, B, seed=800 + B)
    out = []
    for d, (p, x) in ((dims, (params, X)), (wide, _padded(dims, wide, params, X))):
        m = make_model(d, hi.ACT_RELU, hi.LOSS_SOFTMAX_CE, B, p)
        g = torch.empty(p.size, device="cuda")
        m.batch_grad(torch.from_numpy(x).cuda(), torch.from_numpy(y).cuda(), B, g)
        m.destroy()
        g, off, tensors = g.cpu().numpy(), 0, []
        for l in range(1, len(d)):
            n = d[l] * d[l - 1]
            tensors += [g[off:off + n].reshape(d[l], d[l - 1])[:dims[l], :dims[l - 1]], g[off + n:off + n + dims[l]]]
            off += n + d[l]
        out.append(tensors)
    for i, (a, b) in enumerate(zip(*out)):
        np.testing.assert_array_equal(a, b, err_msg=f"{'dW db'.split()[i % 2]}_{i // 2 + 1}")


def test_forward_forms_add_the_same_sums():
    """The first 100 rows in batches that take 16 x 16 blocks, 32 x 32 blocks and those through LDS."""
    torch = _torch()
    dims, forms = (70, 512, 512, 40), {100: "16", 300: "32", 1000: "32s"}
    params, X, y = _problem(dims, hi.LOSS_SOFTMAX_CE, 1000, seed=81)
    m = make_model(dims, hi.ACT_SIGMOID, hi.LOSS_SOFTMAX_CE, 1000, params)
    dX, dy, acts = torch.from_numpy(X).cuda(), torch.from_numpy(y).cuda(), []
    for B, form in forms.items():
        if not check_plan(f32_small_forms(dims, B).split()[:2], [form] * 2):
            pytest.skip("a tuning aid sends the products to other kernels")
        m.batch_loss(dX, dy, B)
        acts.append(gpu_hidden_activations(m, dims, 100))
    m.destroy()
    for a in acts[1:]:
        for l in (1, 2):
            np.testing.assert_array_equal(a[l], acts[0][l])


@pytest.mark.parametrize("dims,act,B,plan", F32_EDGES)
def test_split_plane_products_at_tile_edges(dims, act, B, plan):
    """Each tile shape of the large fp32 products with rows, columns and k-tiles cut by the end of
    the matrix, rows of every alignment."""
    check_plan(f32_plan(dims, B), plan)
    params, X, y = _problem(dims, hi.LOSS_SOFTMAX_CE, B, seed=B)
    check_case(dims, act, hi.LOSS_SOFTMAX_CE, params, X, y, lr=0.1, condition_relu=B < 100)


def _relu_gradient_in_64_bits(dims, params, X, y, on):
    """Gradient and hidden activations of a ReLU network with the softmax loss; `on` = {layer: mask}."""
    P, off = [], 0
    for a, b in zip(dims[:-1], dims[1:]):
        P.append(params[off:off + a * b].astype(np.float64).reshape(b, a))
        off += a * b
        P.append(params[off:off + b].astype(np.float64))
        off += b
    L = len(dims) - 1
    acts = [X.astype(np.float64)]
    for l in range(1, L + 1):
        z = acts[-1] @ P[2 * l - 2].T + P[2 * l - 1]
        acts.append(np.where(on[l], z, 0.0) if l < L else z)
    p = np.exp(acts[L] - acts[L].max(1, keepdims=True))
    p /= p.sum(1, keepdims=True)
    p[np.arange(y.size), y] -= 1.0
    d, grads = p / y.size, []
    for l in range(L, 0, -1):
        grads += [d.sum(0), (d.T @ acts[l - 1]).ravel()]
        if l > 1:
            d = np.where(on[l - 1], d @ P[2 * l - 2], 0.0)
    return np.concatenate(grads[::-1]), acts


@pytest.mark.parametrize("dims,B,plan", [
    ((300, 300, 290, 40), 2560, "64s 64s small; 128x64 64s; 128"),
    ((546, 515, 530, 40), 577, "64x32 64x32 small; 64s 64s; small"),
])
def test_split_plane_products_of_tiny_operands(dims, B, plan):
    """Operands down to 2^-126 keep all their bits in the three planes: weights of 2^-116 against inputs of 2^100
    (forward), activations of 2^-116 (forward and weight gradient), deltas of 2^-117 (weight gradient of layer 1, read
    M-major).  Without a scale the planes of 2^-116 hold about 18 bits (relative error 2e-6)."""
    check_plan(f32_plan(dims, B), plan)
    rng = np.random.default_rng(11)
    W = [rng.standard_normal((b, a)) * s for a, b, s in zip(dims[:-1], dims[1:], (2.0 ** -116, 2.0 ** -108, 0.1))]
    params = np.concatenate([np.concatenate([w.ravel(), np.zeros(w.shape[0])]) for w in W])
    params[-40:] = rng.standard_normal(40)
    params = params.astype(np.float32)
    X = (rng.standard_normal((B, dims[0])) * 2.0 ** 100).astype(np.float32)
    y = rng.integers(0, 40, size=B).astype(np.int32)
    _, g, _, _, _, acts = gpu_grad_and_step(dims, hi.ACT_RELU, hi.LOSS_SOFTMAX_CE, params, X, y, 0.0, want_acts=True)
    ref, ref_acts = _relu_gradient_in_64_bits(dims, params, X, y, {l: acts[l] > 0 for l in (1, 2)})
    for l in (1, 2):
        err = np.linalg.norm(acts[l] - ref_acts[l]) / np.linalg.norm(ref_acts[l])
        assert err <= 4e-7, f"activations of layer {l}: {err:.1e}"   # fp32 sums of 300 terms: 2.2e-7 (1.3e-7 measured)
    off = 0
    for l, (a, b) in enumerate(zip(dims[:-1], dims[1:]), 1):
        for name, n in (("dW", a * b), ("db", b)):
            r = ref[off:off + n]
            err = np.linalg.norm(g[off:off + n] - r) / np.linalg.norm(r)
            assert err <= 1e-6, f"{name}_{l}: {err:.1e}"   # the same and the fast exp of the loss: about 3e-7
            off += n


@pytest.mark.parametrize("K", [1, 2, 16, 17, 31, 32])
def test_split_plane_products_of_one_k_tile_are_exact_before_the_rounding(K):
    """A contraction of one k-tile has all eight products of planes that fp32 can tell from nothing: a sum of one product
    is the fp32 product (half a unit in the last place, 2^-24, and 2^-34 of it for x2 y2).  The six of longer contractions
    miss up to 2^-24 more, most for significands just above 1."""
    dims, B = (K, 330, 20), 2600
    check_plan(f32_plan(dims, B).split()[0], "64")
    rng = np.random.default_rng(K)
    W = (1.0 + 0.0039 * rng.random((330, K))).astype(np.float32)
    X = np.zeros((B, K), dtype=np.float32)
    X[np.arange(B), rng.integers(0, K, size=B)] = 1.0 + 0.0039 * rng.random(B)
    params = np.concatenate([W.ravel(), np.zeros(330 + 20 * 330 + 20, dtype=np.float32)])
    torch = _torch()
    m = make_model(dims, hi.ACT_RELU, hi.LOSS_SOFTMAX_CE, B, params)
    m.batch_loss(torch.from_numpy(X).cuda(), torch.zeros(B, dtype=torch.int32, device="cuda"), B)
    got = gpu_hidden_activations(m, dims, B)[1]
    m.destroy()
    ref = X.astype(np.float64) @ W.T.astype(np.float64)
    err = float(np.max(np.abs(got - ref) / ref))
    assert err <= 2.0 ** -24 * 1.01, f"{err:.2e}"


# every shape of the split-plane kernels, forward and backward; rows, columns and k-tiles cut
SPLIT_SIZES = [
    ((300, 330, 290, 40), 2561, "64s 64s small; 128x64 64s; 128"),
    ((100, 330, 290, 40), 2561, "64 64s small; 128x64 64s; small"),
    ((130, 257, 250, 40), 4099, "128x64 128x64 small; 128 128x64; small"),
    ((97, 257, 129, 33), 4099, "128x64 64s small; 64 64s; small"),
    ((100, 500, 500, 40), 8150, "128 128 small; 128 128x64; small"),
    ((546, 515, 530, 40), 577, "64x32 64x32 small; 64s 64s; small"),  # 64 x 32, four groups of wavefronts (forward)
]


@pytest.mark.parametrize("dims,B,plan", SPLIT_SIZES)
def test_split_plane_products_are_as_close_to_64_bits_as_fp32_ones(dims, B, plan):
    """Sums of up to 512 products: fp32 MFMAs are within 3e-7 (relative 2-norm), the planes within 1.3e-7; with the three
    largest of the six products of planes alone it would be 4.4e-6."""
    check_plan(f32_plan(dims, B), plan)
    params, X, y = _problem(dims, hi.LOSS_SOFTMAX_CE, B, seed=B + 1)
    _, g, _, _, _, acts = gpu_grad_and_step(dims, hi.ACT_RELU, hi.LOSS_SOFTMAX_CE, params, X, y, 0.0, want_acts=True)
    ref, ref_acts = _relu_gradient_in_64_bits(dims, params, X, y, {l: acts[l] > 0 for l in (1, 2)})
    for l in (1, 2):
        err = np.linalg.norm(acts[l] - ref_acts[l]) / np.linalg.norm(ref_acts[l])
        assert err <= 3e-7 * l, f"activations of layer {l}: {err:.1e}"
    off = 0
    for l, (a, b) in enumerate(zip(dims[:-1], dims[1:]), 1):
        r = ref[off:off + a * b]
        err = np.linalg.norm(g[off:off + a * b] - r) / np.linalg.norm(r)
        # up to three products forward and three backward, the loss's fast exponential and sums over the batch
        assert err <= 1.5e-6, f"dW_{l}: {err:.1e}"
        off += a * b + b


@pytest.mark.parametrize("dims,B,plan", SPLIT_SIZES)
def test_split_plane_products_of_huge_operands(dims, B, plan):
    """Operands of 2^104 and more have no finite planes and sums beyond 2^80 do not fit the scaled accumulators: those
    blocks are computed again with fp32 MFMAs.  Inputs of 2^105, weights of layer 2 of 2^106 and activations of
    2^99 send every product but the last layer's forward one there, with results that fp32 holds."""
    check_plan(f32_plan(dims, B), plan)
    rng = np.random.default_rng(B)
    scales = [2.0 ** -120, 2.0 ** 106, 2.0 ** -104]
    W = [rng.standard_normal((b, a)) * s for a, b, s in zip(dims[:-1], dims[1:], scales)]
    params = np.concatenate([np.concatenate([w.ravel(), np.zeros(w.shape[0])]) for w in W]).astype(np.float32)
    X = (rng.standard_normal((B, dims[0])) * 2.0 ** 105).astype(np.float32)
    y = rng.integers(0, dims[-1], size=B).astype(np.int32)
    _, g, _, _, _, acts = gpu_grad_and_step(dims, hi.ACT_RELU, hi.LOSS_SOFTMAX_CE, params, X, y, 0.0, want_acts=True)
    ref, ref_acts = _relu_gradient_in_64_bits(dims, params, X, y, {l: acts[l] > 0 for l in (1, 2)})
    for l in (1, 2):
        err = np.linalg.norm(acts[l].astype(np.float64) - ref_acts[l]) / np.linalg.norm(ref_acts[l])
        assert err <= 6e-7, f"activations of layer {l}: {err:.1e}"   # fp32 MFMAs: 2.9e-7 for 512 terms; two layers
    off = 0
    for l, (a, b) in enumerate(zip(dims[:-1], dims[1:]), 1):
        for name, n in (("dW", a * b), ("db", b)):
            r = ref[off:off + n]
            err = np.linalg.norm(g[off:off + n].astype(np.float64) - r) / np.linalg.norm(r)
            # the scores are sums of about 2^0 .. 2^3 whose rounding the softmax passes on; sums over the batch
            assert err <= 5e-6, f"{name}_{l}: {err:.1e}"
            off += n


@pytest.mark.parametrize("dims,B,plan", SPLIT_SIZES)
def test_split_plane_products_of_values_without_finite_planes(dims, B, plan):
    """An infinite or nearly largest fp32 input has no finite leading bf16 part, yet the product is
    what fp32 arithmetic gives: a saturated unit, not a NaN.  In the first and the last row tile (cut) and in the
    partial k-tile."""
    check_plan(f32_plan(dims, B), plan)
    params, X, y = _problem(dims, hi.LOSS_SOFTMAX_CE, B, seed=5)
    X[3, 7], X[B - 1, dims[0] - 1], X[B - 2, dims[0] - 2] = np.inf, -np.inf, 3.4e38
    torch = _torch()
    m = make_model(dims, hi.ACT_SIGMOID, hi.LOSS_SOFTMAX_CE, B, params)
    got = m.batch_loss(torch.from_numpy(X).cuda(), torch.from_numpy(y).cuda(), B)
    acts = gpu_hidden_activations(m, dims, B)
    m.destroy()
    with np.errstate(over="ignore"):
        ref = mf.batch_grad(dims, hi.ACT_SIGMOID, hi.LOSS_SOFTMAX_CE, params, X.astype(np.float64), y)[0]
    assert np.isfinite(ref) and abs(got - ref) <= TOL_F32 * abs(ref)
    for row in (3, B - 1, B - 2):
        assert set(np.unique(acts[1][row])) <= {0.0, 1.0}


@pytest.mark.parametrize("dims,B,plan", SPLIT_SIZES)
def test_split_plane_products_keep_a_nan_in_its_row(dims, B, plan):
    check_plan(f32_plan(dims, B), plan)
    torch = _torch()
    params, X, y = _problem(dims, hi.LOSS_SOFTMAX_CE, B, seed=7)
    m, acts = make_model(dims, hi.ACT_SIGMOID, hi.LOSS_SOFTMAX_CE, B, params), []
    dy = torch.from_numpy(y).cuda()
    for value in (X[B - 1, dims[0] - 1], np.nan):
        X[B - 1, dims[0] - 1] = value
        m.batch_loss_async(torch.from_numpy(X).cuda(), dy, B)
        acts.append(gpu_hidden_activations(m, dims, B))
    m.destroy()
    for l in (1, 2):
        assert np.isnan(acts[1][l][B - 1]).all()
        # the blocks with the NaN are the same planes or fp32 products of the same values: sums of up to 546 terms
        assert np.allclose(acts[1][l][:B - 1], acts[0][l][:B - 1], rtol=1e-5, atol=0)


def test_nan_operands_stay_nan_and_cost_no_second_product():
    """A NaN reaches exactly the results that depend on it (here one row of X, through two layers), and a run whose
    weights have become NaN is about as quick as any other: its products are not computed twice."""
    import paper_2004_08771_amd as hb
    torch = _torch()
    dims, B = (300, 512, 512, 512, 40), 4096
    params, X, y = _problem(dims, hi.LOSS_SOFTMAX_CE, B, seed=6)
    dX, dy = torch.from_numpy(X).cuda(), torch.from_numpy(y).cuda()
    bad = dX.clone()
    bad[1234, 17] = float("nan")
    m = make_model(dims, hi.ACT_SIGMOID, hi.LOSS_SOFTMAX_CE, B, params)
    m.batch_loss_async(dX, dy, B)
    clean = gpu_hidden_activations(m, dims, B)
    m.batch_loss_async(bad, dy, B)
    acts = gpu_hidden_activations(m, dims, B)
    m.destroy()
    for l in (1, 2, 3):
        assert np.isnan(acts[l][1234]).all()
        rest = np.arange(B) != 1234
        assert np.allclose(acts[l][rest], clean[l][rest], rtol=1e-5, atol=0)   # fp32 or split products of the same values
    us = {}
    for name, p in (("finite", params), ("nan", np.full_like(params, np.nan))):
        m = hb.Model(dims, hi.ACT_SIGMOID, hi.LOSS_SOFTMAX_CE).configure(hb.HB_F32, B, False,
                                                                        torch.cuda.current_stream().cuda_stream)
        m.set_params(p)
        times = []
        for i in range(40):
            ev = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
            ev[0].record()
            m.batch_step_async(dX, dy, B, 0.0)
            ev[1].record()
            times.append(ev)
        torch.cuda.synchronize()
        us[name] = sorted(a.elapsed_time(b) for a, b in times[20:])[5] * 1e3
        m.destroy()
    assert us["nan"] <= 2.0 * us["finite"], us    # 1.0 measured; 5 when every product was computed again


# ---------------------------------------------------------------- bf16 products of small tiles
BF16_SMALL_TILES = [
    # one partial k-tile over the batch, column pairs cut in the middle
    ((66, 65, 130, 3), hi.ACT_SIGMOID, 63, "64 64 64; 64 64; 64B 64B 64B"),
    # odd rows of X: shifted loads, transposed copies for dW_1
    ((65, 70, 5), hi.ACT_SIGMOID, 130, "64S 64; 64; 64 64B"),
    # contraction over the batch shared by two groups: 9 k-tiles and one row
    ((66, 129, 65, 2), hi.ACT_RELU, 577, "64 64 64; 64 64; 64sB 64sB 64sB"),
    # the same forward (514, 575) ...
    ((514, 575, 33), hi.ACT_SIGMOID, 200, "64s 64s; 64; 64B 64B"),
    # ... and backward-data (575)
    ((66, 300, 575, 33), hi.ACT_RELU, 200, "64 64 64s; 64s 64; 64B 64B 64B"),
    # one wavefront group each (more than 256 tiles) forward
    ((300, 1030, 2), hi.ACT_RELU, 1025, "64 64s; 64; 64sB 64sB"),
    # 13 x 17 tiles of 128 x 128, cut in both directions
    ((70, 2100, 2060, 9), hi.ACT_RELU, 1600, "128 128 64s; 128 128; 64sB 64B 64sB"),
    # the same for a weight gradient from the transposed copies (odd rows of X)
    ((1101, 3000, 2), hi.ACT_SIGMOID, 300, "64sS 64s; 64; 128 64B"),
]


@pytest.mark.parametrize("dims,act,B,plan", BF16_SMALL_TILES)
def test_bf16_small_tile_products_at_tile_edges(dims, act, B, plan):
    check_plan(bf16_plan(dims, B), plan)
    params, X, y = _problem(dims, hi.LOSS_SOFTMAX_CE, B, seed=300 + B, bias_scale=0.1)
    check_bf16_case(dims, act, hi.LOSS_SOFTMAX_CE, params, X, y, lr=0.1, condition_relu=False)


@pytest.mark.parametrize("d0,B", [(66, 64), (70, 65), (76, 128), (130, 129), (134, 1), (72, 640), (302, 641)])
def test_bf16_weight_gradient_of_rows_without_padding(d0, B):
    """The last columns of X's rows (2, 4 or 6 past a 16-byte piece) run on into the next row, the last batch row's must not:
    batches that end with a k-tile of 64 and one row later, by one group of wavefronts and by two."""
    dims = (d0, 70, 5)
    form = bf16_plan(dims, B).split("; ")[2].split()[0]
    check_plan(form, form if form in ("64B", "64sB") else "64B or 64sB")
    params, X, y = _problem(dims, hi.LOSS_SOFTMAX_CE, B, seed=500 + B + d0, bias_scale=0.1)
    check_bf16_case(dims, hi.ACT_SIGMOID, hi.LOSS_SOFTMAX_CE, params, X, y, lr=0.1, condition_relu=False)


@pytest.mark.parametrize("dims,act,B,plan", BF16_SMALL_TILES + [
    ((66, 129, 65, 70, 3), hi.ACT_SIGMOID, 200, "64 64 64 64; 64 64 64; 64B 64B 64B 64B"),
    ((34, 1700, 1700, 2), hi.ACT_RELU, 600, "64 64s 64s; 64s 64; 64sB 64B 64sB"),
])
def test_bf16_small_tile_products_each_in_a_launch_of_its_own(monkeypatch, dims, act, B, plan):
    """The backward products as they run where none can share a launch, in the kernels that hb_plan_bf16_kernel names."""
    monkeypatch.setenv("HB_BF16_NO_PAIR", "1")
    assert bf16_pairs(dims, B) == {}
    check_plan(bf16_plan(dims, B), plan)
    params, X, y = _problem(dims, hi.LOSS_SOFTMAX_CE, B, seed=310 + B, bias_scale=0.1)
    assert bf16_pair_launches(dims, act, X, y) == set()
    check_bf16_case(dims, act, hi.LOSS_SOFTMAX_CE, params, X, y, lr=0.1, condition_relu=False)


BF16_PAIRS = [
    # two layers: the two weight gradients share a launch, with the mean loss; a batch cut inside its second k-tile
    ((66, 129, 5), hi.ACT_RELU, 65, {2: 1}),
    # each weight gradient with the next backward-data product, one group of wavefronts; three deltas at once
    ((66, 129, 65, 70, 3), hi.ACT_SIGMOID, 200, {4: 1, 3: 1, 2: 1}),
    # two groups: nine k-tiles over the batch and one row
    ((66, 129, 65, 70, 3), hi.ACT_RELU, 577, {4: 2, 3: 2, 2: 2}),
    # 756 tiles over ten k-tiles: one group; the launch before it 298 tiles, the mean loss one of them: two
    ((34, 1700, 1700, 2), hi.ACT_RELU, 600, {3: 2, 2: 1}),
    # 550 tiles over 49 k-tiles: two groups
    ((34, 700, 700, 3), hi.ACT_SIGMOID, 3100, {3: 2, 2: 2}),
    # odd rows of X: dW_1 from transposed copies, in a launch of its own
    ((65, 70, 90, 5), hi.ACT_SIGMOID, 130, {3: 1}),
    # 16 x 16 tiles over eight k-tiles and 16 x 16 of the next product: the most for two groups; with a row more, one group
    ((34, 1024, 1024, 1024, 2), hi.ACT_SIGMOID, 1024, {4: 2, 3: 2, 2: 2}),
    ((34, 1024, 1024, 1024, 2), hi.ACT_SIGMOID, 1025, {4: 2, 3: 1, 2: 2}),
]


def bf16_pair_launches(dims, act, X, y):
    """The layers whose weight gradient shared a launch in one step."""
    import paper_2004_08771_amd as hb
    torch = _torch()
    m = hb.Model(dims, act, hi.LOSS_SOFTMAX_CE).configure(hb.HB_BF16_F32MASTER, y.size)
    m.set_params(np.zeros(hi.num_params(dims), np.float32))
    dX, dy = torch.from_numpy(X).cuda().to(torch.bfloat16), torch.from_numpy(y).cuda()
    m.profile_enable(True)
    m.batch_step(dX, dy, y.size, 0.1)
    ran = {s["layer"] for s in m.profile_read() if s["kind"] == 9}
    m.destroy()
    return ran


@pytest.mark.parametrize("dims,act,B,pairs", BF16_PAIRS)
def test_bf16_backward_products_that_share_a_launch(dims, act, B, pairs):
    params, X, y = _problem(dims, hi.LOSS_SOFTMAX_CE, B, seed=700 + B, bias_scale=0.1)
    check_plan(bf16_pairs(dims, B), pairs)
    check_plan(bf16_pair_launches(dims, act, X, y), set(pairs))
    check_bf16_case(dims, act, hi.LOSS_SOFTMAX_CE, params, X, y, lr=0.1, condition_relu=False)


BF16_SHORT = [
    # 17 x 17 tiles, one k-tile: forward, and backward-data of layer 2 (K = 40)
    ((54, 2060, 40, 3), hi.ACT_RELU, 2100, "128s 64s 64; 128s 64; 64sB 64sB 64sB"),
    # the same from odd rows
    ((63, 2060, 40, 3), hi.ACT_SIGMOID, 2100, "128sS 64s 64; 128s 64; 64s 64sB 64sB"),
    # 23 x 23 tiles, two k-tiles
    ((100, 2900, 3), hi.ACT_SIGMOID, 2900, "128s 64s; dma; 64sB 64sB"),
    # the same from odd rows, the partial one of 63
    ((127, 2900, 3), hi.ACT_RELU, 2900, "128sS 64s; dma; 64s 64sB"),
]


@pytest.mark.parametrize("dims,act,B,plan", BF16_SHORT)
def test_bf16_short_contractions_with_many_tiles(dims, act, B, plan):
    """Products of one or two k-tiles with more 128 x 128 tiles than compute units (and twice as many) run two
    workgroups per compute unit with two register sets."""
    check_plan(bf16_plan(dims, B), plan)
    params, X, y = _problem(dims, hi.LOSS_SOFTMAX_CE, B, seed=700 + dims[0], bias_scale=0.1)
    check_bf16_case(dims, act, hi.LOSS_SOFTMAX_CE, params, X, y, lr=0.1, condition_relu=False)


BF16_SHIFTED = [
    ((63, 70, 5), 130, 0, "64S"),        # one k-tile, element loads at its end
    ((65, 129, 3), 200, 0, "64S"),       # a whole k-tile and one value
    ((65, 129, 3), 200, 1, "64S"),       # the same from an odd address: other rows are the aligned ones
    ((64, 66, 3), 67, 1, "64"),          # even rows from an odd address, whole k-tiles: the last one is taken as a partial one
    ((577, 300, 2), 513, 0, "64sS"),     # two groups of wavefronts share ten k-tiles
    ((201, 1030, 2), 1921, 1, "64S"),    # 64 x 64 tiles, one group
    ((201, 2060, 2), 1601, 0, "128S"),   # 128 x 128 tiles, cut in both directions
]


@pytest.mark.parametrize("dims,B,at,first", BF16_SHIFTED)
def test_bf16_rows_of_X_that_are_not_4_byte_aligned(dims, B, at, first):
    """The forward product of layer 1 reads such rows as aligned dwords and shifts them: the activations
    are those of the same X in rows of even pitch (the layer's other operand and the sums are the same, the order of
    the k-tiles may not be: fp32 sums, then rounded to bf16)."""
    import paper_2004_08771_amd as hb
    check_plan(bf16_plan(dims, B).split()[0], first)
    torch = _torch()
    params, X, y = _problem(dims, hi.LOSS_SOFTMAX_CE, B, seed=B + at)
    flat = torch.zeros(X.size + 1, dtype=torch.bfloat16, device="cuda")
    dX = flat[at:at + X.size].view(X.shape)
    dX.copy_(torch.from_numpy(X))
    dy = torch.from_numpy(y).cuda()
    W = torch.from_numpy(params[:dims[0] * dims[1]].reshape(dims[1], dims[0])).to(torch.bfloat16).double()
    b = params[dims[0] * dims[1]:dims[0] * dims[1] + dims[1]].astype(np.float64)
    z = dX.cpu().double().numpy() @ W.numpy().T + b
    m = hb.Model(dims, hi.ACT_RELU, hi.LOSS_SOFTMAX_CE).configure(hb.HB_BF16_F32MASTER, B)
    m.set_params(params)
    m.batch_loss(dX, dy, B)
    got = gpu_hidden_activations(m, dims, B)[1]
    m.destroy()
    # half a bf16 unit in the last place: 2^-8 of a value with eight significand bits; fp32 rounding of sums of K terms
    # of about 1 / sqrt(K) each: far below 1e-5
    off = float(np.max(np.abs(got - np.maximum(z, 0)) - 2.0 ** -8 * np.abs(z)))
    assert off <= 1e-5, off
