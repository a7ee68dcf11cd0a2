"""The calls whose speed is measured: what a GPU worker has the library do.

A case names a kind of call and its sizes:

  train     `steps` asynchronous steps over successive batches, then the replica is read back to
            the host, as between two exchanges with the global model (dense fp32 or bf16)
  train_csr the same for a sparse first layer
  grad      hb_batch_grad of one batch: the gradient stays on the device
  eval      hb_worker_eval_loss: the loss over a host-resident dataset, in pieces
  epoch     hb_worker_run_epoch: one epoch over a host-resident dataset with the host model pushed
            to every `merge_every` steps

Networks, batch sizes and learning rates are those of this repository's configurations
(hb_inputs.CONFIGS) and of the range in which Algorithm 2 varies the batch (16 .. 8192, any value).
"""
import math

import numpy as np
import torch

import paper_2004_08771_amd as hb

TINY = "54-32-7"
COVTYPE = "54-512-512-512-512-7"
W8A = "300-1024-1024-1024-2"
REALSIM = "20958-512-512-512-2"
WIDE = "2048-4096-4096-4096-1000"
DELICIOUS = "500-512-512-512-512-512-512-512-512-983"


def _case(name, kind, dims, act, loss, batch, steps=1, dtype="f32", lr=0.05, **more):
    return dict({"name": name, "kind": kind, "dims": dims, "act": act, "loss": loss, "batch": batch, "steps": steps,
                 "dtype": dtype, "lr": lr}, **more)


def listed():
    return [
        # the smallest workload: 64 steps of 64 rows, nothing but launch latency
        _case("train-tiny-b64", "train", TINY, "sigmoid", "softmax", 64, steps=64, lr=0.1),
        # the smallest batch the adaptive scheduler assigns on the covtype network, one synchronous call
        _case("grad-covtype-b16", "grad", COVTYPE, "sigmoid", "softmax", 16),
        # a batch in the middle of the adaptive range, an odd size as Algorithm 2's rescaling gives
        _case("train-covtype-b1021", "train", COVTYPE, "sigmoid", "softmax", 1021, steps=16, lr=0.4),
        # the headline workload: 4096 rows of the covtype network, resident in HBM
        _case("train-covtype-b4096", "train", COVTYPE, "sigmoid", "softmax", 4096, steps=8, lr=1.6),
        # wide ReLU network with the logistic loss, a ragged batch
        _case("train-w8a-b3001", "train", W8A, "relu", "logistic", 3001, steps=4),
        # deep network with a wide (983-way) output
        _case("grad-delicious-b2048", "grad", DELICIOUS, "sigmoid", "softmax", 2048),
        # sparse input at the largest batch the paper uses
        _case("train-realsim-b8192", "train_csr", REALSIM, "relu", "logistic", 8192, steps=8, nnz=50),
        # sparse input with a hidden width that is not a power of two and a small odd batch
        _case("train-csr-b701", "train_csr", "8003-320-64-2", "relu", "softmax", 701, steps=16, nnz=30),
        # mixed precision: a moderate network at a ragged batch ...
        _case("train-bf16-w8a-b2047", "train", W8A, "relu", "logistic", 2047, steps=8, dtype="bf16"),
        # ... and the largest workload
        _case("train-bf16-wide-b16384", "train", WIDE, "relu", "softmax", 16384, steps=4, dtype="bf16", lr=0.01),
        # the evaluation at the end of an epoch (forward passes only), from page-locked host memory
        _case("eval-covtype-b8192", "eval", COVTYPE, "sigmoid", "softmax", 8192, rows=100003),
        # the worker's loop over host-resident rows with a push of the model every eighth step
        _case("epoch-covtype-b4096", "epoch", COVTYPE, "sigmoid", "softmax", 4096, lr=1.6, rows=32 * 4096 + 1000,
              merge_every=8),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case: networks of 1 .. 8 hidden layers, batches of 16 .. 8192 rows, any remainder."""
    kind = rng.choice(["train", "train", "train", "grad", "grad", "train_csr", "bf16", "eval", "epoch"])
    dtype, loss = "f32", rng.choice(["softmax", "softmax", "logistic"])
    act = rng.choice(["sigmoid", "relu"])
    hidden = _log_int(rng, 32, 1024)
    if rng.random() < 0.5:
        hidden = max(32, hidden // 32 * 32)
    depth = rng.randint(1, 8)
    out = rng.choice([1, 2]) if loss == "logistic" else _log_int(rng, 2, 1000)
    d0 = _log_int(rng, 32, 1024)
    if kind == "bf16":
        kind, dtype = rng.choice(["train", "grad"]), "bf16"
        hidden = _log_int(rng, 64, 4096)
        depth = rng.randint(1, 3)
        d0 = 8 * _log_int(rng, 4, 256)
    elif kind == "train_csr":
        d0 = _log_int(rng, 2000, 30000)
        depth = rng.randint(1, 3)
        out = rng.choice([1, 2]) if loss == "logistic" else _log_int(rng, 2, 16)
    if kind == "grad":
        # A ReLU unit whose sum lies within rounding of 0 is on or off depending on the order of that
        # sum, and a row of the gradient with it: no one value to compare with.  (The weights after a
        # few steps move by lr times that, so ReLU is in the other kinds.)
        act = "sigmoid"
    batch = _log_int(rng, 16, 8192)
    case = _case("", kind, "-".join(str(d) for d in [d0] + [hidden] * depth + [out]), act, loss, batch, dtype=dtype,
                 lr=0.02 if act == "relu" else 0.1)
    del case["name"]
    if kind == "train_csr":
        case["nnz"] = _log_int(rng, 5, 100)
    if kind in ("train", "train_csr"):
        case["steps"] = rng.choice([4, 8])
    if kind == "eval":
        case["rows"] = batch * rng.randint(4, 12) + rng.randint(0, batch - 1)
    if kind == "epoch":
        case["rows"] = batch * rng.randint(8, 16) + rng.randint(0, batch - 1)
        case["merge_every"] = rng.choice([1, 4, 8])
    # no dearer than the largest listed case of its precision
    most = 4e12 if dtype == "bf16" else 1.6e11
    flops = work(case)["flops"]
    if flops > most:
        shrink = most / flops
        case["batch"] = max(16, int(batch * shrink))
        if "rows" in case:
            case["rows"] = max(case["batch"], int(case["rows"] * shrink))
    return case


# --------------------------------------------------------------------------- inputs
def _dims(case):
    return [int(d) for d in case["dims"].split("-")]


def _n_batches(case):
    return case["steps"] if case["kind"] in ("train", "train_csr") else 1


def _rows(case):
    return case["rows"] if "rows" in case else case["batch"] * _n_batches(case)


def _generator(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed))


def _make_params(case, g):
    """Flat fp32 parameters [W_1, b_1, W_2, ...] on the GPU: Xavier-uniform weights, small biases."""
    dims, parts = _dims(case), []
    for d_in, d_out in zip(dims[:-1], dims[1:]):
        a = math.sqrt(6.0 / (d_in + d_out))
        parts.append((torch.rand(d_out * d_in, generator=g, device="cuda") * 2 - 1) * a)
        parts.append((torch.rand(d_out, generator=g, device="cuda") * 2 - 1) * 0.05)
    return torch.cat(parts)


def _make_labels(case, rows, g):
    if case["loss"] == "logistic":
        return torch.randint(0, 2, (rows,), generator=g, device="cuda", dtype=torch.int32) * 2 - 1
    return torch.randint(0, _dims(case)[-1], (rows,), generator=g, device="cuda", dtype=torch.int32)


def _make_dense(case, rows, g):
    """covtype-like rows for the 54-wide inputs (10 numeric columns, 44 rare indicators), else Gaussian rows;
    the logistic workloads have rows of unit length, as the text data they stand for."""
    d0 = _dims(case)[0]
    if d0 == 54:
        X = torch.rand(rows, d0, generator=g, device="cuda")
        X[:, 10:] = (X[:, 10:] < 0.1).float()
    else:
        X = torch.randn(rows, d0, generator=g, device="cuda")
        if case["loss"] == "logistic":
            X /= X.norm(dim=1, keepdim=True)
    return X.to(torch.bfloat16) if case["dtype"] == "bf16" else X


def _make_csr(case, rows, g):
    """About `nnz` entries a row, columns by a truncated Zipf law (ascending, merged), unit rows."""
    d0 = _dims(case)[0]
    per_row = torch.poisson(torch.full((rows,), float(case["nnz"]), device="cuda"), generator=g).clamp(1, 256).long()
    row = torch.repeat_interleave(torch.arange(rows, device="cuda"), per_row)
    cdf = torch.cumsum(1.0 / torch.arange(1, d0 + 1, device="cuda", dtype=torch.float64), 0)
    u = torch.rand(row.numel(), generator=g, device="cuda", dtype=torch.float64) * cdf[-1]
    rank = torch.searchsorted(cdf, u).clamp(max=d0 - 1)
    perm = torch.randperm(d0, generator=g, device="cuda")
    key = torch.unique(row * d0 + perm[rank])  # sorted: rows in order, columns ascending within
    row, col = key // d0, key % d0
    val = torch.exp(0.5 * torch.randn(key.numel(), generator=g, device="cuda"))
    norm = torch.zeros(rows, device="cuda").index_add_(0, row, val * val).sqrt_()
    val = val / norm[row]
    ptr = torch.zeros(rows + 1, dtype=torch.int64, device="cuda")
    ptr[1:] = torch.cumsum(torch.bincount(row, minlength=rows), 0)
    return ptr, col.to(torch.int32), val.float()


def _inputs(case, seed):
    g = _generator(seed)
    d = {"params": _make_params(case, g)}
    rows = _rows(case)
    if case["kind"] == "train_csr":
        d["ptr"], d["col"], d["val"] = _make_csr(case, rows, g)
    else:
        d["X"] = _make_dense(case, rows, g)
    d["y"] = _make_labels(case, rows, g)
    return d


_ACT = {"sigmoid": hb.HB_ACT_SIGMOID, "relu": hb.HB_ACT_RELU}
_LOSS = {"softmax": hb.HB_LOSS_SOFTMAX_CE, "logistic": hb.HB_LOSS_LOGISTIC}


def prepare(case, seed):
    d = _inputs(case, seed)
    kind, B = case["kind"], case["batch"]
    model = hb.Model(_dims(case), _ACT[case["act"]], _LOSS[case["loss"]])
    model.configure(hb.HB_BF16_F32MASTER if case["dtype"] == "bf16" else hb.HB_F32, B, kind == "train_csr",
                    torch.cuda.current_stream().cuda_stream)
    host = d["params"].cpu().pin_memory()
    model.set_params(host)
    s = {"case": dict(case), "model": model, "host": host}
    if kind in ("eval", "epoch"):
        s["X"], s["y"] = d["X"].cpu().pin_memory(), d["y"].cpu().pin_memory()
        if kind == "epoch":
            s["sched"] = hb.Sched(case["rows"], [B], [B], [B])
        return s
    n = _n_batches(case)
    s["y"] = [d["y"][i * B:(i + 1) * B] for i in range(n)]
    if kind == "train_csr":
        at = d["ptr"][::B].tolist()
        s["csr"] = [((d["ptr"][i * B:(i + 1) * B + 1] - at[i]).to(torch.int32), d["col"][at[i]:at[i + 1]],
                     d["val"][at[i]:at[i + 1]], at[i + 1] - at[i]) for i in range(n)]
    else:
        s["X"] = [d["X"][i * B:(i + 1) * B] for i in range(n)]
    if kind == "grad":
        s["grad"] = torch.empty(model.num_params, device="cuda")
    else:
        s["loss"] = torch.zeros(n, device="cuda")
        s["loss_at"] = [s["loss"][i:] for i in range(n)]
    return s


# --------------------------------------------------------------------------- one pass
def run(s):
    case, model = s["case"], s["model"]
    kind, B, lr = case["kind"], case["batch"], case["lr"]
    if kind == "grad":
        loss = model.batch_grad(s["X"][0], s["y"][0], B, s["grad"])
        return {"loss": loss, "grad": s["grad"]}
    if kind == "eval":
        return {"loss": model.worker_eval_loss(s["X"], s["y"], case["rows"], B)}
    if kind == "epoch":
        s["sched"].new_epoch()
        _, steps, loss_sum = model.worker_run_epoch(s["sched"], 0, s["X"], s["y"], lr / B, s["host"],
                                                    case["merge_every"], 1.0)
        return {"steps": steps, "loss_sum": loss_sum, "params": s["host"]}
    for i in range(case["steps"]):
        if kind == "train_csr":
            ptr, col, val, nnz = s["csr"][i]
            model.batch_step_csr_async(ptr, col, val, nnz, s["y"][i], B, lr, s["loss_at"][i])
        else:
            model.batch_step_async(s["X"][i], s["y"][i], B, lr, s["loss_at"][i])
    model.get_params(s["host"])
    return {"loss": s["loss"], "params": s["host"]}


# --------------------------------------------------------------------------- what a pass cannot do without
def work(case):
    dims, B, kind = _dims(case), case["batch"], case["kind"]
    weights = sum(a * b for a, b in zip(dims[:-1], dims[1:]))
    params = weights + sum(dims[1:])
    first = dims[0] * dims[1]
    if kind == "train_csr":
        steps, nnz = case["steps"], case["nnz"]
        entries = B * nnz
        touched = min(entries, dims[0]) * dims[1]  # only the weight columns of the batch are read and written
        flops = steps * B * (4.0 * nnz * dims[1] + 6.0 * (weights - first))
        step_bytes = 8.0 * entries + 8.0 * B + 8.0 * touched + 8.0 * (params - first)
        return {"bytes": steps * step_bytes + 4.0 * params, "flops": flops}
    item = 2.0 if case["dtype"] == "bf16" else 4.0
    batch_bytes = B * (item * dims[0] + 4.0)
    if kind == "eval":
        return {"bytes": case["rows"] * (item * dims[0] + 4.0) + 4.0 * params, "flops": 2.0 * case["rows"] * weights}
    steps = case["rows"] // B if kind == "epoch" else _n_batches(case)
    flops = steps * B * (6.0 * weights - 2.0 * first)
    if kind == "grad":
        return {"bytes": batch_bytes + 8.0 * params, "flops": flops}
    copies = -(-steps // case["merge_every"]) if kind == "epoch" else 1
    return {"bytes": steps * (batch_bytes + 8.0 * params) + 4.0 * params * copies, "flops": flops}


# Four times what was seen against 64 bits over the listed and 100 drawn cases.
def tolerance(case):
    if case["dtype"] == "bf16":
        return {"rel": 2e-2, "max": 0.12}
    return {"rel": 1e-5, "max": 2e-4}


# --------------------------------------------------------------------------- the same in 64 bits
def _split_params(flat, dims):
    out, off = [], 0
    for d_in, d_out in zip(dims[:-1], dims[1:]):
        W = flat[off:off + d_in * d_out].view(d_out, d_in)
        off += d_in * d_out
        out.append((W, flat[off:off + d_out]))
        off += d_out
    return out


def _forward(case, X, layers, stored):
    """Activations A_0 .. A_{L-1} and the scores; `stored` rounds what the bf16 mode keeps in bf16."""
    acts = [X]
    for i, (W, b) in enumerate(layers):
        z = acts[-1] @ stored(W).t() + b
        if i + 1 < len(layers):
            acts.append(torch.sigmoid(z) if case["act"] == "sigmoid" else z.clamp_min(0))
    return acts, z


def _loss_and_delta(case, z, y):
    B = z.shape[0]
    if case["loss"] == "logistic" and z.shape[1] == 1:
        m = z[:, 0] * y
        loss = torch.nn.functional.softplus(-m).mean()
        return loss, (-y * torch.sigmoid(-m) / B)[:, None]
    cls = ((y + 1) // 2 if case["loss"] == "logistic" else y).long()
    lp = torch.log_softmax(z, 1)
    d = lp.exp()
    d[torch.arange(B, device=z.device), cls] -= 1
    return -lp.gather(1, cls[:, None]).mean(), d / B


def _gradient(case, X, y, flat, stored):
    layers = _split_params(flat, _dims(case))
    acts, z = _forward(case, X, layers, stored)
    loss, delta = _loss_and_delta(case, z, y)
    grads = []
    for i in range(len(layers) - 1, -1, -1):
        grads += [delta.sum(0), (delta.t() @ acts[i]).reshape(-1)]
        if i:
            delta = delta @ stored(layers[i][0])
            delta = delta * (acts[i] * (1 - acts[i]) if case["act"] == "sigmoid" else (acts[i] > 0))
    return loss, torch.cat(grads[::-1])


def exact(case, seed):
    d = _inputs(case, seed)
    kind, B, lr = case["kind"], case["batch"], float(np.float32(case["lr"]))
    stored = (lambda W: W.to(torch.bfloat16).double()) if case["dtype"] == "bf16" else (lambda W: W)
    flat, y = d["params"].double(), d["y"]
    if kind == "train_csr":
        ptr, dims = d["ptr"], _dims(case)

        def batch(i):
            lo, hi = int(ptr[i * B]), int(ptr[(i + 1) * B])
            row = torch.repeat_interleave(torch.arange(B, device="cuda"), torch.diff(ptr[i * B:(i + 1) * B + 1]))
            X = torch.zeros(B, dims[0], device="cuda", dtype=torch.float64)
            X[row, d["col"][lo:hi].long()] = d["val"][lo:hi].double()
            return X
    else:
        def batch(i):
            return d["X"][i * B:(i + 1) * B].double()
    if kind == "eval":
        total, layers = 0.0, _split_params(flat, _dims(case))
        for at in range(0, case["rows"], B):
            _, z = _forward(case, d["X"][at:at + B].double(), layers, stored)
            total += float(_loss_and_delta(case, z, y[at:at + B])[0]) * z.shape[0]
        return {"loss": total / case["rows"]}
    if kind == "grad":
        loss, g = _gradient(case, batch(0), y, flat, stored)
        return {"loss": loss, "grad": g}
    steps = case["rows"] // B if kind == "epoch" else case["steps"]
    if kind == "epoch":
        lr = float(np.float32(np.float32(case["lr"] / B) * np.float32(B)))
    losses = []
    for i in range(steps):
        loss, g = _gradient(case, batch(i), y[i * B:(i + 1) * B], flat, stored)
        losses.append(loss)
        flat = flat - lr * g
    if kind == "epoch":
        return {"steps": steps, "loss_sum": float(torch.stack(losses).sum()), "params": flat.cpu()}
    return {"loss": torch.stack(losses), "params": flat.cpu()}
