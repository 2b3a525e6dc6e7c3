"""What a user of this framework has it do, as cases that can be timed and compared.

    listed()            the cases by name
    draw(rng)           one more case of the same ranges
    prepare(case, seed) inputs, context, schedule: what a program has in hand before the call
    run(state)          one pass through the public entry points, and its outputs
    exact(case, seed)   the same outputs from plain torch in 64 bits
    work(case)          bytes and operations the pass cannot do without
    tolerance(case)     how far another correct fp32 implementation may be off

Kinds of case
    pass   hop_step over a whole schedule (a training run: gradients, Reduce, Apply for every worker iteration)
    waves  hop_step wave by wave with gradients the caller owns (a program that computes its own gradients has to
           stop after every wave)
    mix    hop_mix: one stand-alone averaging of many replicas
    dense / static / csr   one stand-alone SVM minibatch gradient (hop_svm_grad_dense, its allocation-free form,
           hop_svm_grad_csr)
"""
import math

import numpy as np
import torch

from paper_1902_01064_amd import hop, inputs
from paper_1902_01064_amd.session import Session

DEV = "cuda:0"

# The numbers behind "cost" (draw() keeps below the dearest listed case): microseconds, order of magnitude only.
DEAREST_US = 250000.0


# ------------------------------------------------------------------------------------------- the cases ----
def _run_case(**over):
    """Defaults of a "pass" / "waves" case: the suite's learning rate, no options."""
    c = dict(kind="pass", graph="ring", N=16, s=2, b=0, delay="exp1", slow="", skip=False, weights="uniform", model="synth",
             d=1 << 16, rows=0, batch=0, nnz=0, zipf=1.1, loss="hinge", momentum=0.0, lam=1e-4, K=20, serial=False,
             replay=False)
    c.update(over)
    return c


def listed():
    return [
        # ---- stand-alone calls: one gradient or one averaging, where latency and launches count
        # the gradient of a narrow model inside a serving loop or a captured stream: the smallest call there is
        dict(name="static-64x1k", kind="static", d=1024, rows=4096, batch=64, loss="hinge"),
        # one minibatch gradient of the wide dense SVM (65536 features, 128 samples)
        dict(name="dense-128x64k", kind="dense", d=65536, rows=2048, batch=128, loss="log"),
        # one minibatch gradient of the sparse SVM (2^20 features, 64 non-zeros a row, 256 samples)
        dict(name="csr-256x1m", kind="csr", d=1 << 20, rows=32768, batch=256, nnz=64, zipf=1.1, loss="hinge"),
        # one averaging step of 16 replicas on a 4 x 4 torus, five vectors and a gradient each, ragged length
        dict(name="mix-16x1m", kind="mix", graph="torus", N=16, d=1_000_003, grad=True),
        # ---- whole training runs on the built-in SVMs
        # narrow dense model, lock-step ring of 4: two tiny kernels a wave, replayed as a graph
        _run_case(name="run-dense-1k", N=4, s=1, delay="none", model="dense", d=1024, rows=4096, batch=64, K=50,
                  replay=True),
        # wide dense model, ring of 16 with Exp(1) delays, one 4x straggler and skipping: bound by the minibatch rows
        _run_case(name="run-dense-64k", N=16, s=2, slow="4", skip=True, model="dense", d=65536, rows=1024, batch=128, K=30,
                  replay=True),
        # the paper's optimiser (log loss, momentum 0.9) and slow-downs (6x with probability 1/n) on the ring-based
        # graph, with a feature count that is no multiple of four; launched kernel by kernel
        _run_case(name="run-dense-odd", graph="ring_based", N=8, s=5, b=1, delay="bernoulli6", model="dense", d=30_011,
                  rows=1024, batch=100, loss="log", momentum=0.9, K=40),
        # sparse model on a 4 x 4 torus with staleness and a backup worker
        _run_case(name="run-csr-1m", graph="torus", N=16, s=3, b=1, model="csr", d=1 << 20, rows=8192, batch=256, nnz=64,
                  K=100, replay=True),
        # the largest sparse model: 64 workers, 2^24 features, 16 stragglers, skipping
        _run_case(name="run-csr-16m", graph="torus", N=64, s=8, b=2, slow="2345", skip=True, model="csr", d=1 << 24,
                  rows=8192, batch=512, nnz=128, zipf=1.05, K=30, replay=True),
        # ---- whole runs of the mixing workload (a stand-in for a large model: seeded gradients)
        # the benchmark's own workload: 32 workers, 25 M parameters, two 3x stragglers, skipping
        _run_case(name="run-mix-25m", graph="chords", N=32, s=4, b=1, delay="none", slow="33", skip=True,
                  weights="metropolis", d=25_000_000, lam=0.0, K=100),
        # the same method with the paper's momentum on its double ring, Exp(1) delays, ragged length
        _run_case(name="run-mix-momentum", graph="double_ring", N=16, s=5, b=1, delay="exp1", d=2_000_003, lam=0.0,
                  momentum=0.9, K=40),
        # ---- a program with gradients of its own: Reduce + Apply wave by wave
        _run_case(name="waves-external-4m", kind="waves", graph="torus", N=16, s=3, b=1, model="external", d=1 << 22,
                  lam=0.0, K=16),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _ragged(rng, v):
    """Half of the sizes as drawn (any remainder), half rounded to a multiple of 64."""
    return v if rng.random() < 0.5 else max(64, v // 64 * 64)


def draw(rng):
    kind = rng.choice(["static", "dense", "csr", "mix", "run", "run", "run", "run", "waves"])
    if kind in ("static", "dense"):
        d = _ragged(rng, _log(rng, 1000, 120000))
        return dict(kind=kind, d=d, rows=rng.choice([512, 2048]), batch=rng.choice([16, 50, 64, 128, 200]),
                    loss=rng.choice(["hinge", "log"]))
    if kind == "csr":
        d = _log(rng, 20000, 4 << 20)
        return dict(kind=kind, d=d, rows=rng.choice([4096, 16384]), batch=rng.choice([64, 200, 256, 512]),
                    nnz=rng.choice([16, 64, 128]), zipf=rng.choice([1.05, 1.1]), loss=rng.choice(["hinge", "log"]))
    graph, N = rng.choice([("ring", 4), ("ring", 16), ("torus", 16), ("chords", 32), ("ring_based", 8),
                           ("double_ring", 16), ("torus", 64)])
    if kind == "mix":
        return dict(kind="mix", graph=graph, N=N, d=_ragged(rng, _log(rng, 5000, 4_000_000)), grad=rng.random() < 0.7)
    least = min(len(l) for l in _graph(graph, N, 1))
    c = _run_case(graph=graph, N=N, s=rng.choice([1, 2, 4, 5]), b=rng.randrange(0, min(2, least)),
                  delay=rng.choice(["none", "exp1", "bernoulli6"]), slow=rng.choice(["", "4", "33"]),
                  skip=rng.random() < 0.5, weights=rng.choice(["uniform", "metropolis"]), K=rng.choice([10, 20, 40]),
                  replay=rng.random() < 0.5)
    if kind == "waves":
        d = _log(rng, 50000, 8 << 20) // 64 * 64
        c.update(kind="waves", model="external", d=d, lam=0.0, replay=False, momentum=rng.choice([0.0, 0.9]))
    else:
        c.update(momentum=rng.choice([0.0, 0.0, 0.9]), loss=rng.choice(["hinge", "log"]),
                 model=rng.choice(["dense", "csr", "synth", "synth"]), serial=rng.random() < 0.2)
        if c["model"] == "dense":
            c.update(d=_ragged(rng, _log(rng, 1000, 65536)), rows=512, batch=rng.choice([32, 64, 128]))
        elif c["model"] == "csr":
            c.update(d=_log(rng, 20000, 4 << 20), rows=4096, batch=rng.choice([64, 256]), nnz=rng.choice([16, 64]))
        else:
            c.update(d=_ragged(rng, _log(rng, 5000, 16_000_000)), lam=0.0, loss="hinge")
    # no dearer than the dearest listed case: shorten the run, then the vectors
    while _cost_us(c) > 0.8 * DEAREST_US and c["K"] > 10:
        c["K"] //= 2
    while _cost_us(c) > 0.8 * DEAREST_US or c["N"] * c["d"] > 3e8:
        c["d"] = c["d"] // 2 // 64 * 64
    return c


def _cost_us(c):
    rec = c["N"] * c["K"] * (2.0 if c["serial"] else 1.0)
    return rec * (8.0 + 4.0 * c["d"] * (9.0 + 2.0 * c["batch"] * (c["model"] == "dense")) / 4e6)


# ------------------------------------------------------------------------------------- schedules, data ----
def _graph(name, n, seed):
    if name == "ring":
        return inputs.ring(n)
    if name == "torus":
        side = int(round(math.sqrt(n)))
        return inputs.torus(side, side)
    if name == "chords":
        return inputs.ring_with_chords(n, 2, seed)
    if name == "ring_based":
        return inputs.ring_based(n)
    return inputs.double_ring(n)


def _config(case, seed):
    """The case as a configuration of the framework (inputs.config has the same keys)."""
    nb = _graph(case["graph"], case["N"], seed)
    W = (inputs.metropolis_weights if case["weights"] == "metropolis" else inputs.uniform_weights)(nb)
    mult = None
    if case["slow"]:
        mult = [1.0] * case["N"]
        factors = [float(f) for f in case["slow"]]
        count = case["N"] // 4 if len(factors) > 2 else len(factors)
        for p, w in enumerate(inputs.slow_workers(seed, case["N"], count)):
            mult[w] = factors[p % len(factors)]
    delay = {"none": inputs.DELAY_NONE, "exp1": inputs.DELAY_EXP1, "bernoulli6": inputs.DELAY_BERNOULLI6}[case["delay"]]
    return dict(name="case", in_nbrs=nb, W=W, N=case["N"], s=case["s"], b=case["b"], delay_kind=delay, mult=mult,
                skip_on=case["skip"], max_ig=0, max_skip=10, trigger=1, model=case["model"], d=case["d"],
                rows=case["rows"], batch=case["batch"], nnz=case["nnz"], zipf_a=case["zipf"],
                loss=1 if case["loss"] == "log" else 0, momentum=case["momentum"], serial=case["serial"], lr=0.01,
                lam=case["lam"], grad_var=1e-3, K=case["K"], seed=seed)


def _data(c):
    """Per-worker data sets on the GPU: dense (X, y), or csr (rowptr, col, val, y)."""
    if c["model"] not in ("dense", "csr"):
        return None
    ws = inputs.hidden_w(c["seed"], c["d"], DEV)
    if c["model"] == "dense":
        return [inputs.dense_svm_data(c["seed"], i, c["rows"], c["d"], ws, DEV) for i in range(c["N"])]
    return [inputs.csr_svm_data(c["seed"], i, c["rows"], c["d"], c["nnz"], c["zipf_a"], ws, DEV) for i in range(c["N"])]


def _external(c):
    gen = torch.Generator(device=DEV).manual_seed(c["seed"] + 5)
    return torch.randn(c["N"] * c["d"], generator=gen, device=DEV) * math.sqrt(c["grad_var"])


def _sample_ids(seed, batch, rows):
    r = np.random.default_rng(seed)
    return torch.from_numpy(r.integers(0, rows, size=batch).astype(np.int32)).to(DEV)


def _mix_inputs(case, seed):
    """Replicas of one model (a common vector, a few per cent of disagreement), a gradient each."""
    nb = _graph(case["graph"], case["N"], seed)
    W = inputs.metropolis_weights(nb)
    gen = torch.Generator(device=DEV).manual_seed(seed)
    base = torch.randn(case["d"], generator=gen, device=DEV) * 0.1
    src = [base + 0.005 * torch.randn(case["d"], generator=gen, device=DEV) for _ in nb]
    grad = [0.03 * torch.randn(case["d"], generator=gen, device=DEV) if case["grad"] else None for _ in nb]
    return nb, W, src, grad


# ----------------------------------------------------------------------------------------- prepare, run ----
class _Run:
    """A session with its schedule simulated; outputs are views of the rings (and velocities)."""

    def __init__(self, case, seed):
        c = self.c = _config(case, seed)
        self.sess = s = Session(c, DEV)
        p0 = inputs.initial_params(seed, c["d"], 0.01, DEV)
        data = _data(c)
        if c["model"] == "dense":
            s.set_dense([x for x, _ in data], [y for _, y in data])
        elif c["model"] == "csr":
            s.set_csr(data)
        elif c["model"] == "external":
            self.ext = _external(c)
            hop.hop_set_grad_source(s.ctx, hop.HOP_GRAD_EXTERNAL, 0.0, self.ext.data_ptr())
        else:
            hop.hop_set_grad_source(s.ctx, hop.HOP_GRAD_SYNTH, c["grad_var"])
        s.set_params(p0)
        s.simulate()
        if case["replay"]:
            hop.hop_use_graph(s.ctx, 1)
        per = s.D * s.stride
        self.out = [s.arena[i * per:(i + 1) * per] for i in range(c["N"])]
        if c["momentum"] > 0:
            self.out = [s.arena[:c["N"] * per], s.arena[s.arena.numel() - c["N"] * s.stride:]]
        self.waves = list(range(s.sched.n_waves)) if case["kind"] == "waves" else None

    def __del__(self):
        try:
            self.sess.close()
        except Exception:
            pass


def prepare(case, seed):
    if case["kind"] in ("pass", "waves"):
        return _Run(case, seed)
    stream = torch.cuda.current_stream().cuda_stream
    if case["kind"] == "mix":
        nb, W, src, grad = _mix_inputs(case, seed)
        out = [torch.zeros(case["d"], device=DEV) for _ in nb]
        jobs = [dict(out=out[i].data_ptr(), g=grad[i].data_ptr() if case["grad"] else None, eta=0.01,
                     src=[src[j].data_ptr() for j in [i] + list(l)], w=[float(W[j][i]) for j in [i] + list(l)])
                for i, l in enumerate(nb)]
        return dict(case=case, jobs=jobs, stream=stream, keep=(src, grad), out=out)
    c = dict(seed=seed, d=case["d"], rows=case["rows"], N=1, model="csr" if case["kind"] == "csr" else "dense",
             nnz=case.get("nnz", 0), zipf_a=case.get("zipf", 0.0))
    data = _data(c)[0]
    w = inputs.initial_params(seed, case["d"], 0.01, DEV)
    rows = _sample_ids(seed, case["batch"], case["rows"])
    g, coef = torch.zeros(case["d"], device=DEV), torch.zeros(case["batch"], device=DEV)
    scratch = torch.zeros(hop.hop_grad_scratch_floats(case["d"], case["batch"]), device=DEV)
    p = [t.data_ptr() for t in data]
    loss = 1 if case["loss"] == "log" else 0
    tail = (w.data_ptr(), rows.data_ptr(), case["batch"], case["d"], 1e-4, g.data_ptr(), coef.data_ptr())
    return dict(case=case, args=tuple(p) + tail, scratch=scratch, stream=stream, loss=loss, keep=(data, w, rows),
                out=[g, coef])


def run(state):
    if isinstance(state, _Run):
        s = state.sess
        if state.waves is None:
            hop.hop_step(s.ctx, s.sched)
        else:
            for w in state.waves:
                hop.hop_step(s.ctx, s.sched, w, w + 1)
        return state.out
    kind = state["case"]["kind"]
    if kind == "mix":
        hop.hop_mix(state["jobs"], state["case"]["d"], state["stream"])
    elif kind == "static":
        hop.hop_svm_grad_dense_static(*state["args"], state["stream"], state["loss"])
    elif kind == "dense":
        hop.hop_svm_grad_dense(*state["args"], state["scratch"].data_ptr(), state["stream"], state["loss"])
    else:
        hop.hop_svm_grad_csr(*state["args"], state["stream"], state["loss"])
    return state["out"]


# ------------------------------------------------------------------------------------------------ exact ----
def _loss_coef(y, dot, batch, loss):
    m = y * dot
    if loss == "log":
        return y / (batch * (1.0 + torch.exp(m)))
    return torch.where(m < 1.0, y, torch.zeros_like(y)) / batch


def _svm(data, w, ids, lam, loss):
    """(gradient, coefficients) of one minibatch in 64 bits."""
    ids = ids.long()
    y = data[-1][ids].double()
    lam = float(np.float32(lam))
    if len(data) == 2:
        x = data[0][ids].double()
        coef = _loss_coef(y, x @ w, len(ids), loss)
        return lam * w - coef @ x, coef
    nnz = data[1].numel() // (data[0].numel() - 1)
    col, val = data[1].view(-1, nnz)[ids].long(), data[2].view(-1, nnz)[ids].double()
    coef = _loss_coef(y, (val * w[col]).sum(1), len(ids), loss)
    return (lam * w).index_add_(0, col.reshape(-1), -(coef[:, None] * val).reshape(-1)), coef


_M64 = (1 << 64) - 1


def _split_mix(z):
    z = (z + 0x9E3779B97F4A7C15) & _M64
    z = ((z ^ (z >> 30)) * 0xBF58476D1CE4E5B9) & _M64
    z = ((z ^ (z >> 27)) * 0x94D049BB133111EB) & _M64
    return z ^ (z >> 31)


def _signed(v):
    return v - (1 << 32) if v >= 1 << 31 else v


def _lshr(x, n):
    return (x >> n) & ((1 << (32 - n)) - 1)


def _hash32(x):
    x = x ^ _lshr(x, 16)
    x = x * _signed(0x7FEB352D)
    x = x ^ _lshr(x, 15)
    x = x * _signed(0x846CA68B)
    return x ^ _lshr(x, 16)


def _byte_sum(x):
    x = (x & 0x00FF00FF) + (_lshr(x, 8) & 0x00FF00FF)
    return (x & 0xFFFF) + _lshr(x, 16)


def _synthetic(seed, worker, it, variance, cols):
    """The seeded gradient: the centred sum of 12 hashed bytes times one fp32 factor (whole numbers until then)."""
    def key(n):
        h = _split_mix(seed & _M64)
        for v in (6, worker, it, n):
            h = _split_mix(h ^ v)
        return h
    ka, kb = key(0), key(1)
    a = _hash32(cols ^ _signed(ka & 0xFFFFFFFF))
    b = _hash32(cols ^ _signed(ka >> 32))
    t = (a + ((b << 16) | _lshr(b, 16))) ^ _signed(kb & 0xFFFFFFFF)
    s = _byte_sum(a) + _byte_sum(b) + _byte_sum(t) - 1530
    return (s.float() * float(np.float32(math.sqrt(variance / 65535.0)))).double()


def exact(case, seed):
    if case["kind"] == "mix":
        nb, W, src, grad = _mix_inputs(case, seed)
        out = []
        for i, l in enumerate(nb):
            acc = sum(float(W[j][i]) * src[j].double() for j in [i] + list(l))
            out.append(acc - float(np.float32(0.01)) * grad[i].double() if case["grad"] else acc)
        return out
    if case["kind"] not in ("pass", "waves"):
        c = dict(seed=seed, d=case["d"], rows=case["rows"], N=1, model="csr" if case["kind"] == "csr" else "dense",
                 nnz=case.get("nnz", 0), zipf_a=case.get("zipf", 0.0))
        w = inputs.initial_params(seed, case["d"], 0.01, DEV).double()
        return list(_svm(_data(c)[0], w, _sample_ids(seed, case["batch"], case["rows"]), 1e-4, case["loss"]))
    # A whole run: every record of the schedule in its order.  The schedule (who averages what, with which weights,
    # on which samples) is the plan that the program holds before the call; the arithmetic is done here.
    c = _config(case, seed)
    opts = hop.make_opts(max_ig=c["max_ig"], skip_on=c["skip_on"], max_skip=c["max_skip"], trigger=c["trigger"], lr=c["lr"],
                         lam=c["lam"], batch=c["batch"], seed=seed, loss=c["loss"], momentum=c["momentum"],
                         serial=c["serial"])
    row_ptr, col = inputs.to_csr(c["in_nbrs"])
    ctx = hop.hop_init(row_ptr, col, c["W"], c["N"], c["d"], c["s"], c["b"], opts)
    for i in range(c["N"]):
        if c["rows"]:
            hop.hop_set_rows(ctx, i, c["rows"])
    sched = hop.hop_simulate(ctx, c["K"], c["delay_kind"], c["mult"])
    slots, stride = hop.hop_layout(c["d"], c["s"], opts)
    N, d = c["N"], c["d"]
    rings = torch.zeros(N, slots, stride, dtype=torch.float64, device=DEV)
    p0 = inputs.initial_params(seed, d, 0.01, DEV).double()
    rings[:, slots - 1 if c["serial"] else 0, :d] = p0
    vel = torch.zeros(N, stride, dtype=torch.float64, device=DEV) if c["momentum"] > 0 else None
    data = _data(c)
    ext = _external(c).view(N, d) if c["model"] == "external" else None
    cols = torch.arange(d, device=DEV, dtype=torch.int32) if c["model"] == "synth" else None
    eta, mu = float(np.float32(c["lr"])), float(np.float32(c["momentum"]))
    loss = case["loss"]
    for e in range(sched.n_records):
        i, kind = int(sched.worker[e]), int(sched.kind[e])
        a0, a1 = int(sched.src_begin[e]), int(sched.src_begin[e + 1])
        vecs = [rings[int(j), int(q), :d] for j, q in zip(sched.src_worker[a0:a1], sched.src_slot[a0:a1])]
        acc = vecs[0] * float(sched.src_weight[a0])
        for v, w in zip(vecs[1:], sched.src_weight[a0 + 1:a1]):
            acc.add_(v, alpha=float(w))
        if kind in (hop.HOP_STEP, hop.HOP_APPLY):
            if c["model"] == "synth":
                g = _synthetic(seed, i, int(sched.iter[e]), c["grad_var"], cols)
            elif c["model"] == "external":
                g = ext[i].double()
            else:
                ids = torch.from_numpy(np.array(sched.batch_rows[e])).to(DEV)
                g, _ = _svm(data[i], vecs[0], ids, c["lam"], loss)
            if vel is not None:
                g = vel[i, :d].mul_(mu).add_(g)
            acc.sub_(g, alpha=eta)
        rings[i, int(sched.out_slot[e]), :d] = acc
    sched.free()
    hop.hop_destroy(ctx)
    if vel is not None:
        return [rings.view(-1), vel.view(-1)]
    return [rings[i].reshape(-1) for i in range(N)]


# --------------------------------------------------------------------------------------- work, tolerance ----
def work(case):
    d = case["d"]
    if case["kind"] == "mix":
        nb = _graph(case["graph"], case["N"], 1)
        terms = sum(len(l) + 1 for l in nb) + (len(nb) if case["grad"] else 0)
        return dict(bytes=4.0 * d * len(nb) * (3 if case["grad"] else 2), flops=2.0 * d * terms)
    if case["kind"] in ("static", "dense"):
        rows = case["rows"] * (1.0 - (1.0 - 1.0 / case["rows"]) ** case["batch"])         # distinct samples
        return dict(bytes=4.0 * d * (rows + 2), flops=4.0 * case["batch"] * d)
    if case["kind"] == "csr":
        return dict(bytes=8.0 * case["batch"] * case["nnz"] + 8.0 * d, flops=4.0 * case["batch"] * case["nnz"] + d)
    # a run: parameters in, every ring slot out, the data of each minibatch once, about N K records of a mean degree
    nb = _graph(case["graph"], case["N"], 1)
    records = case["N"] * case["K"]
    degree = sum(len(l) for l in nb) / len(nb)
    opts = hop.make_opts(momentum=case["momentum"], serial=case["serial"])
    slots, _ = hop.hop_layout(d, case["s"], opts)
    nbytes = 4.0 * d * case["N"] * (1 + slots + (2 if case["momentum"] > 0 else 0))
    flops = 2.0 * d * records * (1 + degree)
    if case["model"] == "dense":
        nbytes += 4.0 * d * records * case["batch"]
        flops += 4.0 * d * records * case["batch"]
    elif case["model"] == "csr":
        nbytes += 8.0 * records * case["batch"] * case["nnz"]
        flops += 4.0 * records * case["batch"] * case["nnz"]
    elif case["model"] == "external":
        nbytes += 4.0 * d * case["N"]
        flops += 2.0 * d * records
    else:
        flops += 30.0 * d * records                                                       # the generator's own operations
    return dict(bytes=nbytes, flops=flops)


def tolerance(case):
    """About four times what the fp32 path is off from 64 bits (measured: stand-alone calls 0.4 to 1.4e-7, runs on
    dense vectors 1 to 5e-7, sparse runs 0.5 to 1.5e-6)."""
    if case["kind"] not in ("pass", "waves"):
        return {"rel": 1e-6}
    if case["model"] == "dense" and case["loss"] == "hinge":
        # a sample whose margin lies within rounding of 1 may fall on either side of the hinge: one flip moves a
        # replica by eta / B |x|, a thousandth of its norm
        return {"rel": 4e-3, "max": 0.2}
    if case["model"] in ("dense", "csr"):
        return {"rel": 6e-6}
    return {"rel": 2e-6}
