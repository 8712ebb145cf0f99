"""What a user of this framework has it do, as cases that can be timed and compared.

A case is one of the passes that the README shows, called as it shows them:

* ``single``  smat_simulate and smat_backward_accum of one flat tensor;
* ``step``    one simulated step of a tensor list through a Plan: the step's scale drawn, the
              per-tensor parameters set, simulate, switch, backward, switch back;
* ``graph``   the same step replayed from one captured HIP graph of the device-driven calls;
* ``optim``   the clipped fused optimizer step: the gradient norm, then AdamW fed from the gradient
              at the simulated weights;
* ``train``   one simulated step through SimulatedMergeTraining, gradients handed over as autograd
              leaves them, with the clipped fused update;
* ``merge``   an N-expert merge (Task Arithmetic, DARE) of a tensor list.

Lists are shaped like the decoders and the vision tower that the benchmark's workloads stand for.
The arrays of a list are views of one buffer per kind (what the case returns): each tensor on its
own 512-byte boundary as an allocator places it, or, with ``ranks`` > 0, the piece of a flat
parameter buffer that one rank of a sharded run holds, its tensors packed end to end.
"""
from __future__ import annotations

import math
import random

import numpy as np
import torch

import paper_2609_33437_amd as smat
from paper_2609_33437_amd.training import SimulatedMergeTraining

DEV = "cuda"
SEED = 0x5EED0001
STEP = 7            # the global step of a state's first pass
ALPHA_MIN = 0.2
LAM = 0.5
MAX_NORM = 1.0
ADAM = dict(lr=2e-5, beta1=0.9, beta2=0.999, eps=1e-8, weight_decay=1e-3)
NOISE = {"gaussian": smat.SMAT_NOISE_GAUSSIAN, "uniform": smat.SMAT_NOISE_UNIFORM,
         "laplace": smat.SMAT_NOISE_LAPLACE}
DTYPES = {"f32": torch.float32, "bf16": torch.bfloat16}
BYTES = {"f32": 4, "bf16": 2}

# A ragged list of odd sizes that the repository's tests use: (elements, whether it is masked).
MINI = [(3000, 1), (7, 0), (257 * 129, 1), (4096, 0), (64000, 0), (2048 * 257, 1), (1, 0), (5 * 65537, 1), (31, 0),
        (64 * 4096, 1)]


# ---------------------------------------------------------------- the cases
def _list(kind, name, **kw):
    """A list case: a decoder of `layers` blocks (width d, k/v width kv, SwiGLU ffn), an embedding of
    `vocab` rows and `vectors` small vectors between them (layers 0: the mini list)."""
    c = dict(kind=kind, name=name, layers=0, d=0, kv=0, ffn=0, vocab=0, vectors=0, ranks=0, base="bf16", buffer="bf16",
             grad="bf16", noise="gaussian", keep=0.5, sigma=1e-3, accumulate=True)
    c.update(kw)
    return c


GPT2 = dict(layers=12, d=768, kv=768, ffn=2048, vocab=50304, vectors=53)             # about 125M parameters
DECODER = dict(layers=28, d=1536, kv=256, ffn=8960, vocab=151936)                    # 1.54B parameters


def listed():
    return [
        # one flat tensor, the smallest call: launch and host latency count
        dict(kind="single", name="single_1m", n=1 << 20, base="f32", buffer="bf16", grad="f32", noise="gaussian",
             keep=0.5, sigma=1e-3),
        # a handful of odd-sized tensors (adapters, a head): ten tensors, 1.2M elements
        _list("step", "step_small_odd"),
        # one rank's piece of a flat parameter buffer over eight ranks: odd sizes packed end to end,
        # tensors that start inside a Philox group and off any vector boundary
        _list("step", "step_shard_packed", layers=12, d=1023, kv=341, ffn=2731, vocab=50257, ranks=8, noise="uniform"),
        # the 125M-shaped decoder, ordinary size
        _list("step", "step_125m", **GPT2, keep=0.4),
        # the same step from a captured graph
        _list("graph", "graph_125m", **GPT2, keep=0.4),
        # a vision tower with hundreds of small vectors in fp32, uniform noise (the method's default),
        # the simulated gradient the step's only one (written, not accumulated)
        _list("step", "step_vision_f32", layers=24, d=1024, kv=1024, ffn=2731, vocab=844, vectors=1236, base="f32",
              buffer="f32", grad="f32", noise="uniform", sigma=2e-3, accumulate=False),
        # the 1.5B-shaped decoder with a sparse mask, the largest step
        _list("step", "step_1p5b", **DECODER, keep=0.1),
        # the clipped optimizer step when an expert gradient is already there (both losses every step)
        _list("optim", "optim_125m_acc", **GPT2, accumulate=True),
        # the clipped optimizer step of periodic scheduling on the large decoder
        _list("optim", "optim_1p5b", **DECODER, accumulate=False),
        # the method in a training loop: a 110M decoder, clipped fused update
        _list("train", "train_110m", layers=6, d=1024, kv=1024, ffn=2816, vocab=32000, noise="uniform", sigma=2e-3),
        # seven experts merged by Task Arithmetic, large
        _list("merge", "merge_ta_1p5b", **DECODER, experts=7, keep=1.0),
        # seven experts with DARE masks, ordinary size
        _list("merge", "merge_dare_125m", **GPT2, experts=7, keep=0.7),
    ]


# The most bytes a drawn case may move: below those of the largest listed one.
MOST_BYTES = 25e9


def draw(rng: random.Random):
    """One more case: any of the passes, from 2^16 parameters up, its size spread over the logarithm."""
    kind = rng.choice(["single", "step", "step", "graph", "optim", "train", "merge"])
    dt = lambda: rng.choice(["bf16", "bf16", "f32"])  # noqa: E731
    base, grad, buffer = dt(), dt(), dt()
    noise = rng.choice(["uniform", "gaussian", "laplace", "none"])
    keep = rng.choice([1.0, 0.1, round(rng.uniform(0.1, 0.9), 3), 0.5])
    sigma = 0.0 if noise == "none" else rng.choice([1e-3, 2e-3])
    noise = "gaussian" if noise == "none" else noise
    accumulate = rng.random() < 0.5
    experts = rng.choice([2, 3, 7, 8])
    per = {"optim": 32.0, "train": 34.0, "merge": 4.0 * (experts + 2)}.get(kind, 24.0)
    top = {"single": 1 << 27, "train": 1 << 28}.get(kind, MOST_BYTES / per)
    params = math.exp(rng.uniform(math.log(1 << 16), math.log(top)))
    if kind == "single":
        n = int(params) | rng.choice([0, 1])
        return dict(kind=kind, n=n, base=base, buffer=buffer, grad=grad, noise=noise, keep=keep, sigma=sigma)
    # a decoder of about that many parameters: d from layers (2 d^2 + 2 d kv + 3 d ffn) + vocab d
    layers = rng.choice([1, 2, 4, 6] if kind == "train" else [1, 2, 6, 12, 24])
    group, wide, rows = rng.choice([1, 2, 4]), rng.uniform(2.5, 4.0), rng.uniform(4.0, 40.0)
    d = math.sqrt(params / (layers * (2 + 2 / group + 3 * wide) + rows))
    ranks = rng.choice([0, 2, 5, 8]) if kind in ("step", "graph", "optim") and rng.random() < 0.4 else 0
    if ranks and rng.random() < 0.5:
        d, odd = d * math.sqrt(ranks), 1          # widths as they come, one of them odd
    else:
        d, odd = d * math.sqrt(max(ranks, 1)), 8  # widths in eights
    fit = lambda x: max(8, int(x) // odd * odd) if odd > 1 else max(9, int(x)) | 1  # noqa: E731
    c = _list(kind, "", layers=layers, d=fit(d), kv=fit(d / group), ffn=fit(d * wide), vocab=fit(d * rows),
              vectors=rng.choice([0, 0, 50, 600]) if kind != "train" else 0, ranks=ranks, base=base, buffer=buffer,
              grad=grad, noise=noise, keep=keep, sigma=sigma, accumulate=accumulate)
    del c["name"]
    if kind == "merge":
        c["experts"] = experts
    return c


# ---------------------------------------------------------------- lists
def _tensors(case):
    """(tensor id, first element, elements, masked) of every tensor that the case's process holds."""
    if case["kind"] == "single":
        return [(0, 0, case["n"], True)]
    if not case["layers"]:
        whole = [(n, bool(m)) for n, m in MINI]
    else:
        d, kv, ffn, vocab = case["d"], case["kv"], case["ffn"], case["vocab"]
        whole = []
        for _ in range(case["layers"]):
            whole += [(d * d, True), (kv * d, True), (kv * d, True), (d * d, True), (ffn * d, True), (ffn * d, True),
                      (d * ffn, True), (d, False), (d, False)]
        whole += [(vocab * d, False), (d, False)]
        rng = random.Random(5)
        small = [int(math.exp(rng.uniform(math.log(32), math.log(8192)))) for _ in range(case["vectors"])]
        mixed, at = [], 0
        for i, t in enumerate(whole):             # the small vectors spread evenly through the list
            mixed.append(t)
            upto = (i + 1) * len(small) // len(whole)
            mixed += [(n, False) for n in small[at:upto]]
            at = upto
        whole = mixed
    whole = [(i, 0, n, m) for i, (n, m) in enumerate(whole)]
    if not case["ranks"]:
        return whole
    total = sum(n for _, _, n, _ in whole)
    size = -(-total // case["ranks"])
    a, b, at, out = size, min(2 * size, total), 0, []   # the second rank's piece
    for i, _, n, m in whole:
        lo, hi = max(a, at), min(b, at + n)
        if lo < hi:
            out.append((i, lo - at, hi - lo, m))
        at += n
    return out


def _places(case):
    """(each tensor's first element in its buffer, the buffer's elements)."""
    at, places = 0, []
    for _, _, n, _ in _tensors(case):
        places.append(at)
        at += n if case.get("ranks") else -(-n // 128) * 128 if case["buffer"] == "f32" else -(-n // 256) * 256
    return places, at


def _params(case):
    return sum(n for _, _, n, _ in _tensors(case))


class _Inputs:
    """The case's arrays: one buffer per kind and its per-tensor views."""

    def __init__(self, case, seed):
        self.case, self.tensors = case, _tensors(case)
        self.places, self.size = _places(case)
        self.gen = torch.Generator(DEV).manual_seed(seed)

    def views(self, flat):
        return [flat[p:p + n] for p, (_, _, n, _) in zip(self.places, self.tensors)]

    def normal(self, std, dtype):
        out = torch.empty(self.size, dtype=dtype, device=DEV)
        for a in range(0, self.size, 1 << 28):
            part = out[a:a + (1 << 28)]
            part.copy_(torch.randn(part.numel(), generator=self.gen, device=DEV).mul_(std))
        return out

    def near(self, base, std, dtype):
        """base plus normal noise: fine-tuned weights beside their base."""
        out = torch.empty(self.size, dtype=dtype, device=DEV)
        for a in range(0, self.size, 1 << 28):
            part = base[a:a + (1 << 28)]
            fresh = torch.randn(part.numel(), generator=self.gen, device=DEV).mul_(std)
            out[a:a + (1 << 28)].copy_(fresh.add_(part.float()))
        return out


def _inputs(case, seed):
    """The arrays that the case's pass reads, by kind."""
    x = _Inputs(case, seed)
    kind = case["kind"]
    x.base = x.normal(0.02, DTYPES[case["base"]])
    if kind == "merge":
        x.experts = [x.near(x.base, 1e-3, DTYPES[case["base"]]) for _ in range(case["experts"])]
        return x
    x.theta = x.near(x.base, 1e-3, torch.float32)
    x.grad = x.normal(1e-2, DTYPES[case["buffer"] if kind == "train" else case["grad"]])
    if kind == "optim" or kind == "train":
        x.m1 = x.normal(1e-3, torch.float32)
        x.m2 = x.normal(1e-3, torch.float32).square_()
    if kind in ("single", "step", "graph") or (kind == "optim" and case["accumulate"]):
        x.acc = x.normal(1e-3, torch.float32)
    return x


def _keeps(case):
    return [np.float32(case["keep"] if m else 1.0).item() for _, _, _, m in _tensors(case)]


def _records(case, s):
    return smat.op_params_array(len(_tensors(case)), s, _keeps(case), case["sigma"], 1, NOISE[case["noise"]])


def _terms(case):
    keep = case["keep"]
    return [dict(gamma=0.3, keep=keep, seed=100 + j, step=j) for j in range(case["experts"])]


# ---------------------------------------------------------------- one pass
def prepare(case, seed):
    x = _inputs(case, seed)
    kind = case["kind"]
    st = {"case": case, "x": x, "step": STEP}
    if kind == "merge":
        st["out"] = torch.zeros(x.size, dtype=DTYPES[case["buffer"]], device=DEV)
        st["plan"] = smat.MergePlan(x.views(x.base), x.views(st["out"]), [x.views(e) for e in x.experts])
        st["terms"] = _terms(case)
        return st
    if kind == "train":
        params = [torch.nn.Parameter(v) for v in x.views(x.theta)]
        opt = torch.optim.AdamW(params, lr=ADAM["lr"], betas=(ADAM["beta1"], ADAM["beta2"]), eps=ADAM["eps"],
                                weight_decay=ADAM["weight_decay"], fused=True)
        for p, a, b in zip(params, x.views(x.m1), x.views(x.m2)):   # a run under way
            opt.state[p] = dict(step=torch.tensor(10.0, device=DEV), exp_avg=a, exp_avg_sq=b)
        st["wrapper"] = SimulatedMergeTraining(
            params, x.views(x.base), _keeps(case), ALPHA_MIN, case["sigma"], period=1, lam=LAM, seed=SEED,
            noise_kind=NOISE[case["noise"]], buffer_dtype=DTYPES[case["buffer"]])
        st["opt"], st["params"], st["grads"] = opt, params, x.views(x.grad)
        return st
    st["out"] = torch.zeros(x.size, dtype=DTYPES[case["buffer"]], device=DEV)
    if kind == "single":
        st["args"] = [x.views(a)[0] for a in (x.theta, x.base, st["out"], x.grad, x.acc)]
        return st
    acc = x.views(x.acc) if hasattr(x, "acc") else None
    plan = smat.Plan(x.views(x.theta), x.views(st["out"]), x.views(x.base), x.views(x.grad), acc,
                     tensor_ids=[i for i, _, _, _ in x.tensors], elem_offsets=[o for _, o, _, _ in x.tensors])
    st["plan"] = plan
    st["keep"] = _keeps(case)
    if kind == "optim":
        plan.bind_adam_state(x.views(x.m1), x.views(x.m2))
        plan.set_params(_records(case, smat.scale_draw(SEED, STEP, ALPHA_MIN)))
        st["sumsq"] = torch.zeros(1, dtype=torch.float64, device=DEV)
        st["coef"] = torch.ones(1, device=DEV)
    if kind == "graph":
        plan.set_params(_records(case, 1.0))
        st["state"] = smat.StepState(SEED, STEP - 1, 1.0)
        torch.cuda.synchronize()
        st["graph"] = torch.cuda.CUDAGraph()
        with torch.cuda.graph(st["graph"]):
            st["state"].advance(ALPHA_MIN)
            plan.simulate_dev(st["state"])
            plan.backward_dev(st["state"], LAM, case["accumulate"])
    return st


def run(st):
    case, x, step = st["case"], st["x"], st["step"]
    kind = case["kind"]
    st["step"] = step + 1
    if kind == "merge":
        st["plan"].merge(st["terms"])
        return st["out"]
    if kind == "graph":
        st["graph"].replay()
        return st["out"], x.acc
    if kind == "train":
        w = st["wrapper"]
        w.begin(step)
        for p, g in zip(st["params"], st["grads"]):
            p.grad = g
        norm = w.end(st["opt"], fused=True, max_norm=MAX_NORM)
        return {"norm": norm, "theta": x.theta, "exp_avg": x.m1, "exp_avg_sq": x.m2, "simulated": list(w.buffers)}
    if kind == "single":
        p = dict(s=smat.scale_draw(SEED, step, ALPHA_MIN), keep=case["keep"], sigma=case["sigma"],
                 noise_kind=NOISE[case["noise"]])
        theta, base, out, grad, acc = st["args"]
        smat.smat_simulate(theta, base, out, p, SEED, step)
        smat.smat_backward_accum(grad, acc, p, LAM, SEED, step)
        return st["out"], x.acc
    plan = st["plan"]
    if kind == "optim":
        # a run's step count only rises: the moments are where this step left them
        plan.grad_norm(SEED, step, LAM, case["accumulate"], MAX_NORM, st["sumsq"], st["coef"])
        plan.adamw_fused(SEED, step, LAM, dict(ADAM, step=step + 4), accumulate=case["accumulate"],
                         grad_scale_dev=st["coef"])
        return {"sumsq": st["sumsq"], "coef": st["coef"], "theta": x.theta, "exp_avg": x.m1, "exp_avg_sq": x.m2}
    s = smat.scale_draw(SEED, step, ALPHA_MIN)
    plan.set_params(smat.op_params_array(plan.count, s, st["keep"], case["sigma"], 1, NOISE[case["noise"]]))
    plan.simulate(SEED, step)
    plan.switch_storage(smat.SMAT_SIMULATED)
    plan.backward(SEED, step, LAM, case["accumulate"])
    plan.switch_storage(smat.SMAT_EXPERT)
    return st["out"], x.acc


def work(case):
    """Bytes: each array that the pass reads and writes, once.  Flops: the per-element arithmetic."""
    n, kind = _params(case), case["kind"]
    if kind == "merge":
        per = BYTES[case["base"]] * (case["experts"] + 1) + BYTES[case["buffer"]]
        return {"bytes": n * per, "flops": n * 4 * case["experts"]}
    simulate = 4 + BYTES[case["base"]] + BYTES[case["buffer"]]
    grad = BYTES[case["buffer"] if kind == "train" else case["grad"]]
    accumulate = case.get("accumulate", True)
    if kind == "optim":
        return {"bytes": n * (24 + grad + (4 if accumulate else 0)), "flops": n * 18}
    if kind == "train":
        return {"bytes": n * (simulate + 24 + grad), "flops": n * 26}
    return {"bytes": n * (simulate + grad + (8 if accumulate else 4)), "flops": n * 10}


def tolerance(case):
    """fp32 results of another order of the same roundings differ by a few 1e-7 (elements near
    cancellation by more), sums and the update's quotient by a little more; a bf16 result may round
    the other way, one part in 128 of its value at most, in a few of a million elements."""
    bf16_out = case["buffer"] == "bf16" and case["kind"] != "optim"
    return {"rel": 2e-4, "max": 1.6e-2} if bf16_out else {"rel": 2e-6, "max": 1e-4}


# ---------------------------------------------------------------- the same in 64 bits
_M32 = 0xFFFFFFFF


def _philox(group, tensor, c3, seed):
    """The four words of Philox4x32-10 (Salmon et al., SC'11) at counter (group, tensor, c3)."""
    a, b = group & _M32, group >> 32
    c, d = torch.full_like(group, tensor), torch.full_like(group, c3)
    k0, k1 = seed & _M32, seed >> 32 & _M32
    for _ in range(10):
        p, q = a * 0xD2511F53, c * 0xCD9E8D57     # 64-bit products, wrapped into int64
        a, b, c, d = (q >> 32 & _M32) ^ b ^ k0, q & _M32, (p >> 32 & _M32) ^ d ^ k1, p & _M32
        k0, k1 = (k0 + 0x9E3779B9) & _M32, (k1 + 0xBB67AE85) & _M32
    return a, b, c, d


def _words(first, n, tensor, c3, seed):
    """The word of each element first .. first + n - 1 of a tensor."""
    lo = first >> 2
    group = torch.arange(lo, (first + n + 3) >> 2, dtype=torch.int64, device=DEV)
    w = torch.stack(_philox(group, tensor, c3, seed), dim=1).reshape(-1)
    return w[first - 4 * lo:first - 4 * lo + n]


def _unit(first, n, tensor, step, noise):
    """The unit noise of each element."""
    lo, c3 = first >> 2, 4 * step + 1
    group = torch.arange(lo, (first + n + 3) >> 2, dtype=torch.int64, device=DEV)
    w = _philox(group, tensor, c3, SEED)
    if noise == "gaussian":
        z = []
        for a, b in ((w[0], w[1]), (w[2], w[3])):
            r = torch.sqrt(-2.0 * torch.log(((a >> 8) + 1).double() * 2.0 ** -24))
            turn = 2.0 * math.pi * ((b >> 8).double() * 2.0 ** -24)
            z += [r * torch.cos(turn), r * torch.sin(turn)]
    else:
        u = [((a >> 8).double() + 0.5) * 2.0 ** -24 - 0.5 for a in w]
        if noise == "uniform":
            z = [math.sqrt(12.0) * v for v in u]
        else:
            z = [-torch.sign(v) * torch.log1p(-2.0 * v.abs()) / math.sqrt(2.0) for v in u]
    z = torch.stack(z, dim=1).reshape(-1)
    return z[first - 4 * lo:first - 4 * lo + n]


def _kept(first, n, tensor, step, seed, keep):
    if keep >= 1.0:
        return None
    return _words(first, n, tensor, 4 * step, seed) < math.floor(keep * 2.0 ** 32)


def _alpha(step):
    g = torch.zeros(1, dtype=torch.int64, device=DEV)
    u = (int(_philox(g, 0, 4 * step + 2, SEED)[0]) >> 8) * 2.0 ** -24
    low = float(np.float32(ALPHA_MIN))
    return float(np.float32(low + (1.0 - low) * u))


def _pieces(case):
    """(place in the buffer, first element, elements, tensor id, keep) in parts of at most 2^25 elements."""
    places, _ = _places(case)
    for p, (i, o, n, _), keep in zip(places, _tensors(case), _keeps(case)):
        for a in range(0, n, 1 << 25):
            yield p + a, o + a, min(n - a, 1 << 25), i, keep


def exact(case, seed):
    x, kind = _inputs(case, seed), case["kind"]
    fresh = lambda: torch.zeros(x.size, dtype=torch.float64, device=DEV)  # noqa: E731
    if kind == "merge":
        out = fresh()
        for at, first, n, tensor, _ in _pieces(case):
            cut = slice(at, at + n)
            base = x.base[cut].double()
            y = base.clone()
            for e, t in zip(x.experts, _terms(case)):
                keep = float(np.float32(t["keep"]))
                d = (e[cut].double() - base) * (float(np.float32(t["gamma"])) / keep)
                m = _kept(first, n, tensor, t["step"], t["seed"], keep)
                y += d if m is None else torch.where(m, d, 0.0)
            out[cut] = y
        return out
    step, sigma = STEP, float(np.float32(case["sigma"]))
    s = _alpha(step)
    simulated, grad = fresh() if kind != "optim" else None, fresh()
    if hasattr(x, "acc") and case.get("accumulate", True):
        grad.copy_(x.acc)
    for at, first, n, tensor, keep in _pieces(case):
        cut = slice(at, at + n)
        m, t = _kept(first, n, tensor, step, SEED, keep), s / keep
        if simulated is not None:
            base = x.base[cut].double()
            d = (x.theta[cut].double() - base) * t
            y = base + (d if m is None else torch.where(m, d, 0.0))
            if sigma > 0.0:
                y += sigma * _unit(first, n, tensor, step, case["noise"])
            simulated[cut] = y
        g = x.grad[cut].double() * (LAM * t)
        grad[cut] += g if m is None else torch.where(m, g, 0.0)
    if kind in ("single", "step", "graph"):
        if hasattr(x, "acc") and case.get("accumulate", True) is False:   # between the tensors nothing is written
            gap = torch.ones(x.size, dtype=torch.bool, device=DEV)
            for at, _, n, _, _ in _pieces(case):
                gap[at:at + n] = False
            grad = torch.where(gap, x.acc.double(), grad)
        return simulated, grad
    # the clipped AdamW update; what lies between the tensors stays as it was
    inside = torch.zeros(x.size, dtype=torch.bool, device=DEV)
    for at, _, n, _, _ in _pieces(case):
        inside[at:at + n] = True
    grad *= inside
    sumsq = grad.square().sum()
    coef = torch.clamp(MAX_NORM / (sumsq.sqrt() + 1e-6), max=1.0)
    h = {k: float(np.float32(v)) for k, v in ADAM.items()}
    count = 11
    grad *= coef
    m1 = torch.where(inside, x.m1.double() + (1 - h["beta1"]) * (grad - x.m1.double()), x.m1.double())
    m2 = torch.where(inside, h["beta2"] * x.m2.double() + (1 - h["beta2"]) * grad.square(), x.m2.double())
    root = m2.sqrt() / math.sqrt(1 - h["beta2"] ** count) + h["eps"]
    update = h["lr"] / (1 - h["beta1"] ** count) * m1 / root
    theta = torch.where(inside, x.theta.double() * (1 - h["lr"] * h["weight_decay"]) - update, x.theta.double())
    if kind == "optim":
        return {"sumsq": sumsq.reshape(1), "coef": coef.reshape(1), "theta": theta, "exp_avg": m1, "exp_avg_sq": m2}
    return {"norm": sumsq.sqrt().reshape(1), "theta": theta, "exp_avg": m1, "exp_avg_sq": m2,
            "simulated": x.views(simulated)}
