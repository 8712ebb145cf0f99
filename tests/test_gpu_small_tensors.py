"""Lists of many small tensors, whose remainders run in segments of 2,048 elements instead of chunks of
16,384: every pass over the list equals the single-tensor calls bit for bit, with and without large
tensors beside the small ones, the norm equals that of the gradient in 64 bits, and the device-driven
calls and the static simulate equal the plan's."""
import pytest
import torch

import paper_2609_33437_amd as smat
from helpers import bits

pytestmark = pytest.mark.gpu
DEV = "cuda"
SEED, STEP, LAM = 31, 4, 0.5
EDGES = (1, 5, 255, 256, 257, 2047, 2048, 2049, 4097, 6000, 14336, 14337, 16383, 16384, 16385, 18432, 18433)
HP = dict(lr=1e-3, beta1=0.9, beta2=0.99, eps=1e-8, weight_decay=0.01, step=3)


def arrays(sizes, std, seed, dtype=torch.float32):
    g = torch.Generator(DEV).manual_seed(seed)
    return [(torch.randn(n, device=DEV, generator=g) * std).to(dtype) for n in sizes]


def same(a, b):
    return all(torch.equal(bits(x), bits(y)) for x, y in zip(a, b))


# 510 tensors spare 15,000-30,000 of their blocks; with a 4M tensor beside 1,020 the segments still pay
LISTS = [(EDGES[:9] * 40, 0), (EDGES * 30, 0), (EDGES * 30, 6), ((4 * 2 ** 20 + 3,) + EDGES[:8] * 128, 0)]


def spared_blocks(sizes, offset):
    """One-quad blocks (256 elements) of a list's remainders that segments spare, of those that chunks take."""
    spans = [n + offset % 4 for n in sizes]
    rest = [s % 16384 for s in spans if s % 16384]
    return sum(64 - 8 * -(-r // 2048) for r in rest), sum(64 * -(-s // 16384) for s in spans)


@pytest.mark.parametrize("sizes,offset", LISTS)
def test_these_lists_are_split(sizes, offset):
    spared, blocks = spared_blocks(sizes, offset)
    assert spared >= 16384 and 8 * spared >= blocks


@pytest.mark.parametrize("sizes,offset", LISTS)
def test_list_equals_single_calls(sizes, offset):
    count = len(sizes)
    th, t0 = arrays(sizes, 0.02, 1), arrays(sizes, 0.02, 2, torch.bfloat16)
    gs, gt = arrays(sizes, 1e-2, 3, torch.bfloat16), arrays(sizes, 1e-3, 4)
    m1, m2 = arrays(sizes, 1e-3, 5), [x.square_() for x in arrays(sizes, 1e-3, 6)]
    out = [torch.full_like(x, float("nan")) for x in t0]
    prm = [dict(s=0.5, keep=(0.4, 1.0)[i % 2], sigma=1e-3 * (i % 3)) for i in range(count)]
    ref = [[x.clone() for x in a] for a in (th, gt, m1, m2, out)]
    terms = [dict(gamma=0.3, keep=0.6, seed=8), dict(gamma=0.2, seed=9)]
    merged, merged_ref = [torch.empty_like(x) for x in t0], [torch.empty_like(x) for x in t0]
    ex = [arrays(sizes, 0.02, 7 + j, torch.bfloat16) for j in range(2)]
    for i in range(count):
        smat.smat_simulate(ref[0][i], t0[i], ref[4][i], prm[i], SEED, STEP, i, offset)
        smat.smat_backward_accum(gs[i], ref[1][i], prm[i], LAM, SEED, STEP, i, offset)
        smat.smat_adamw_fused(gs[i], ref[0][i], ref[2][i], ref[3][i], prm[i], LAM, HP, SEED, STEP, i, offset)
        smat.smat_merge([e[i] for e in ex], t0[i], merged_ref[i], terms, i, offset)
    sumsq = torch.zeros(1, dtype=torch.float64, device=DEV)
    offs = [offset] * count
    with smat.Plan(th, out, t0, gs, gt, elem_offsets=offs) as plan:
        plan.set_params(prm)
        plan.bind_adam_state(m1, m2)
        plan.simulate(SEED, STEP)
        plan.backward_accum(SEED, STEP, LAM)
        plan.adamw_fused(SEED, STEP, LAM, HP)
        plan.grad_norm(SEED, STEP, LAM, False, sumsq=sumsq)
        torch.cuda.synchronize()
    assert all(same(a, b) for a, b in zip((th, gt, m1, m2, out), ref))
    with smat.MergePlan(t0, merged, ex, elem_offsets=offs) as plan:
        plan.merge(terms)
        torch.cuda.synchronize()
    assert same(merged, merged_ref)
    with smat.Plan(th, out, t0, gs, gt, elem_offsets=offs) as plan:
        plan.set_params(prm)
        plan.backward(SEED, STEP, LAM, False)
        torch.cuda.synchronize()
    zeros = [torch.zeros_like(g) for g in gt]
    for i in range(count):
        smat.smat_backward_accum(gs[i], zeros[i], prm[i], LAM, SEED, STEP, i, offset)
    torch.cuda.synchronize()
    assert same(gt, zeros)          # the overwriting backward, element by element
    want = sum(float(g.double().square().sum()) for g in gt)
    # fp32 partial sums of at most 32 squares per lane and 64 lanes
    assert abs(float(sumsq) - want) <= 96 * 2.0 ** -24 * want


@pytest.mark.parametrize("dt", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("sizes,offset", LISTS[1:])
def test_device_driven_calls_equal_the_host_driven_ones(sizes, offset, dt):
    count = len(sizes)
    state, adam_state = smat.StepState(SEED, STEP, 0.75), smat.AdamStepState(HP["lr"], HP["step"])
    offs = [offset] * count
    # 0.75 * 0.5 is exact, so the host-driven records hold the same s
    prm = [dict(s=0.5, keep=(0.4, 1.0, 0.05, 0.0)[i % 4], sigma=1e-3 * (i % 3), rescale=i % 2) for i in range(count)]
    got = []
    for device in (False, True):
        th, t0 = arrays(sizes, 0.02, 1), arrays(sizes, 0.02, 2, dt)
        gs, gt = arrays(sizes, 1e-2, 3, dt), arrays(sizes, 1e-3, 4)
        m1, m2 = arrays(sizes, 1e-3, 5), [x.square_() for x in arrays(sizes, 1e-3, 6)]
        out = [torch.full_like(x, float("nan")) for x in t0]
        sumsq = torch.zeros(2, dtype=torch.float64, device=DEV)
        with smat.Plan(th, out, t0, gs, gt, elem_offsets=offs) as plan:
            plan.set_params(prm if device else [dict(p, s=0.75 * p["s"]) for p in prm])
            plan.bind_adam_state(m1, m2)
            if device:
                plan.simulate_dev(state)
                plan.backward_dev(state, LAM)
                acc = [g.clone() for g in gt]
                for k in range(2):
                    plan.grad_norm_dev(state, LAM, bool(k), sumsq=sumsq[k:k + 1])
                    plan.adamw_fused_dev(state, adam_state, LAM, HP, accumulate=bool(k))
                plan.backward_dev(state, LAM, False)
            else:
                plan.simulate(SEED, STEP)
                plan.backward_accum(SEED, STEP, LAM)
                acc = [g.clone() for g in gt]
                for k in range(2):
                    plan.grad_norm(SEED, STEP, LAM, bool(k), sumsq=sumsq[k:k + 1])
                    plan.adamw_fused(SEED, STEP, LAM, HP, accumulate=bool(k))
                plan.backward(SEED, STEP, LAM, False)
            torch.cuda.synchronize()
        got.append((out, acc, gt, th, m1, m2, [sumsq]))
    for a, b in zip(*got):
        assert same(a, b)
