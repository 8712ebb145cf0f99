"""Tensors off every vector boundary: shards that start inside a Philox group, in buffers packed end to
end.  Each gives the bytes that the same elements have in the whole, aligned tensor (which the oracle
tests check), and nothing outside it is written: sizes around a quad, a tile of 256 and of 2,048 elements
and a chunk of 16,384, all four offsets within a group, all four element shifts of the pointers."""
import pytest
import torch

import paper_2609_33437_amd as smat
from helpers import bits

pytestmark = pytest.mark.gpu
DEV = "cuda"
DT = {"bf16": torch.bfloat16, "f32": torch.float32}
SIZES = (1, 2, 3, 4, 5, 7, 253, 256, 257, 1021, 2047, 2052, 16381, 16384, 16391)
SEED, STEP, LAM = 0xABCDEF0123, 5, 0.75
HP = dict(lr=1e-3, beta1=0.9, beta2=0.99, eps=1e-8, weight_decay=0.1, step=3)


def shards(sizes=SIZES, shifts=(0, 1, 2, 3)):
    """(place in sizes, first element in its tensor, elements, element shift of the buffers)"""
    return [(i, 4 * i + (i * 7 + s) % 4 + (256 if i % 3 == 2 else 0), n, s)
            for s in shifts for i, n in enumerate(sizes)]


def random(n, g, scale, dtype=torch.float32):
    return (torch.randn(n, device=DEV, generator=g) * scale).to(dtype)


class Packed:
    """Whole tensors, and the shards cut from them packed into one buffer per array: each shard begins
    `shift` elements past where the last one ended, and NaN fills what is between them."""

    def __init__(self, arrays, seed, cuts=None):
        g = torch.Generator(DEV).manual_seed(seed)
        self.cuts = cuts or shards()
        self.whole = {k: [random(o + n + 3, g, scale, dt) for _, o, n, _ in self.cuts]
                      for k, (scale, dt) in arrays.items()}
        size = sum(n + s for _, _, n, s in self.cuts) + 8
        self.flat = {k: torch.full((size,), float("nan"), dtype=dt, device=DEV) for k, (_, dt) in arrays.items()}
        self.part, self.inside = {}, torch.zeros(size, dtype=torch.bool, device=DEV)
        for k in arrays:
            at, self.part[k] = 1, []
            for w, (_, o, n, s) in zip(self.whole[k], self.cuts):
                at += s
                view = self.flat[k][at:at + n]
                view.copy_(w[o:o + n])
                self.part[k].append(view)
                self.inside[at:at + n] = True
                at += n
        self.offs = [o for _, o, _, _ in self.cuts]
        self.ids = list(range(len(self.cuts)))

    def check(self, *names):
        for k in names:
            for w, p, (_, o, n, s) in zip(self.whole[k], self.part[k], self.cuts):
                assert torch.equal(bits(p), bits(w[o:o + n])), (k, o, n, s)
            assert bool(self.flat[k][~self.inside].isnan().all()), f"{k}: written outside the shards"


def params(count, noise_kind, rescale=1):
    return [dict(s=0.6 + 0.01 * i, keep=(0.5, 1.0, 0.0, 0.2)[i % 4] if i % 5 else 0.7, sigma=1e-3 if i % 3 else 0.0,
                 rescale=rescale, noise_kind=noise_kind) for i in range(count)]


@pytest.mark.parametrize("t0,out,grad,noise", [("bf16", "bf16", "bf16", 0), ("f32", "bf16", "f32", 1),
                                               ("bf16", "f32", "f32", 2), ("f32", "f32", "bf16", 0)])
def test_list_passes(t0, out, grad, noise):
    x = Packed(dict(theta=(0.02, torch.float32), theta0=(0.02, DT[t0]), out=(1.0, DT[out]), gs=(1e-2, DT[grad]),
                    gt=(1e-3, torch.float32), m1=(1e-3, torch.float32), m2=(1e-3, torch.float32)), 3 + noise)
    for k in ("whole", "part"):
        for m in getattr(x, k)["m2"]:
            m.square_()
    prm = params(len(x.cuts), noise)
    for side, offs in ((x.whole, None), (x.part, x.offs)):
        with smat.Plan(side["theta"], side["out"], side["theta0"], side["gs"], side["gt"], tensor_ids=x.ids,
                       elem_offsets=offs) as plan:
            plan.set_params(prm)
            plan.simulate(SEED, STEP)
            plan.backward(SEED, STEP, LAM, True)
            plan.bind_adam_state(side["m1"], side["m2"])
            sumsq = torch.zeros(1, dtype=torch.float64, device=DEV)
            plan.grad_norm(SEED, STEP, LAM, True, sumsq=sumsq)
            plan.adamw_fused(SEED, STEP, LAM, HP, accumulate=True)
            plan.adamw_fused(SEED, STEP + 1, LAM, HP)
            torch.cuda.synchronize()
    x.check("out", "gt", "theta", "m1", "m2")
    # the norm of the shards, from their own gradients in 64 bits (the partial sums are fp32, of at most
    # 32 squares per lane and 64 lanes: relative error within 96 u)
    with smat.Plan(x.part["theta"], x.part["out"], x.part["theta0"], x.part["gs"], x.part["gt"], tensor_ids=x.ids,
                   elem_offsets=x.offs) as plan:
        plan.set_params(prm)
        sumsq = torch.zeros(1, dtype=torch.float64, device=DEV)
        plan.grad_norm(SEED, STEP, LAM, False, sumsq=sumsq)
        plan.backward(SEED, STEP, LAM, False)
        torch.cuda.synchronize()
        want = sum(float(t.double().square().sum()) for t in x.part["gt"])
    assert abs(float(sumsq) - want) <= 96 * 2.0 ** -24 * want


@pytest.mark.parametrize("grad", ["bf16", "f32"])
def test_list_passes_overwrite_and_device_driven(grad):
    x = Packed(dict(theta=(0.02, torch.float32), theta0=(0.02, torch.bfloat16), out=(1.0, torch.bfloat16),
                    gs=(1e-2, DT[grad]), gt=(1e-3, torch.float32), m1=(1e-3, torch.float32),
                    m2=(0.0, torch.float32)), 11)
    for side, offs in ((x.whole, None), (x.part, x.offs)):
        state, adam = smat.StepState(SEED, STEP, 0.5), smat.AdamStepState(1e-3, 2)
        with smat.Plan(side["theta"], side["out"], side["theta0"], side["gs"], side["gt"], tensor_ids=x.ids,
                       elem_offsets=offs) as plan:
            plan.set_params(params(len(x.cuts), 1))
            plan.bind_adam_state(side["m1"], side["m2"])
            plan.simulate_dev(state)
            plan.backward_dev(state, LAM, False)
            plan.adamw_fused_dev(state, adam, LAM, HP, accumulate=True)
            torch.cuda.synchronize()
    x.check("out", "gt", "theta", "m1", "m2")


@pytest.mark.parametrize("e_dt,out_dt", [("bf16", "bf16"), ("f32", "f32"), ("bf16", "f32"), ("f32", "bf16")])
@pytest.mark.parametrize("keep", [0.6, 1.0])
def test_merge(e_dt, out_dt, keep):
    nexp = 5
    arrays = dict({f"e{j}": (0.02, DT[e_dt]) for j in range(nexp)}, base=(0.02, DT[e_dt]), out=(1.0, DT[out_dt]))
    x = Packed(arrays, 21)
    terms = [dict(gamma=0.3, keep=0.0 if j == 3 and keep < 1 else keep, seed=40 + j, step=j) for j in range(nexp)]
    for side, offs in ((x.whole, None), (x.part, x.offs)):
        with smat.MergePlan(side["base"], side["out"], [side[f"e{j}"] for j in range(nexp)], tensor_ids=x.ids,
                            elem_offsets=offs) as plan:
            plan.merge(terms)
            torch.cuda.synchronize()
    x.check("out")


@pytest.mark.parametrize("cuts", [None, shards((131071, 131072, 300001), (1, 3))])  # one run and several of each XCD
def test_single_tensor_calls(cuts):
    x = Packed(dict(theta=(0.02, torch.float32), theta0=(0.02, torch.bfloat16), out=(1.0, torch.bfloat16),
                    gs=(1e-2, torch.bfloat16), gt=(1e-3, torch.float32), m1=(1e-3, torch.float32),
                    m2=(0.0, torch.float32), e=(0.02, torch.bfloat16), merged=(1.0, torch.bfloat16)), 31, cuts)
    for side, offs in ((x.whole, [0] * len(x.cuts)), (x.part, x.offs)):
        for i, p in enumerate(params(len(x.cuts), 0)):
            a = {k: v[i] for k, v in side.items()}
            smat.smat_simulate(a["theta"], a["theta0"], a["out"], p, SEED, STEP, i, offs[i])
            smat.smat_backward_accum(a["gs"], a["gt"], p, LAM, SEED, STEP, i, offs[i])
            smat.smat_adamw_fused(a["gs"], a["theta"], a["m1"], a["m2"], p, LAM, HP, SEED, STEP, i, offs[i],
                                  grad_acc=a["gt"])
            smat.smat_merge([a["e"]], a["theta0"], a["merged"], [dict(gamma=0.4, keep=0.5, seed=9)], i, offs[i])
    torch.cuda.synchronize()
    x.check("out", "gt", "theta", "m1", "m2", "merged")
