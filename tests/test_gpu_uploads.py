"""Per-step tables of lists of 1 to 1,025 tensors reach the kernels whole: list results equal the
single-tensor calls, which take their parameters as arguments.  Counts sit around the upload kernels'
256-thread blocks; repeated calls reuse both staging slots while earlier steps are still queued."""
import pytest
import torch

import paper_2609_33437_amd as smat
from helpers import bits

pytestmark = pytest.mark.gpu
DEV = "cuda"
SEED = 77


def arrays(count, std, seed, dtype=torch.float32):
    g = torch.Generator(DEV).manual_seed(seed)
    return list((torch.randn(count, 8, device=DEV, generator=g) * std).to(dtype))


@pytest.mark.parametrize("count", [1, 31, 64, 65, 257, 1025])
def test_parameters_and_gradient_tables(count):
    th, t0 = arrays(count, 0.02, 1), arrays(count, 0.02, 2, torch.bfloat16)
    out, gt = arrays(count, 1.0, 3, torch.bfloat16), arrays(count, 1e-3, 4)
    m1, m2 = arrays(count, 1e-3, 5), [x.square_() for x in arrays(count, 1e-3, 6)]
    hp = dict(lr=1e-3, beta1=0.9, beta2=0.99, eps=1e-8, weight_decay=0.0, step=2)
    rounds = [[dict(s=0.3 + 0.001 * i + 0.1 * k, keep=0.2 + 0.7 * i / count, sigma=1e-3 * (1 + k)) for i in range(count)]
              for k in range(4)]
    grads = [arrays(count, 1e-2, 10 + k, torch.bfloat16) for k in range(4)]
    want = []
    ref = [[x.clone() for x in a] for a in (th, gt, m1, m2)]
    for k, prm in enumerate(rounds):
        tilde = [torch.empty_like(o) for o in out]
        for i in range(count):
            smat.smat_simulate(ref[0][i], t0[i], tilde[i], prm[i], SEED, k, i)
            smat.smat_backward_accum(grads[k][i], ref[1][i], prm[i], 0.5, SEED, k, i)
            smat.smat_adamw_fused(grads[k][i], ref[0][i], ref[2][i], ref[3][i], prm[i], 0.5, hp, SEED, k, i)
        want.append(tilde)
    got = []
    with smat.Plan(th, out, t0, grads[0], gt) as plan:
        plan.bind_adam_state(m1, m2)
        for k, prm in enumerate(rounds):       # nothing waits between the rounds
            plan.set_params(prm)
            plan.set_grads(grad_sims=grads[k])
            plan.simulate(SEED, k)
            plan.backward_accum(SEED, k, 0.5)
            plan.adamw_fused(SEED, k, 0.5, hp)
            got.append(torch.stack(out))
        torch.cuda.synchronize()
    for k in range(4):
        assert torch.equal(bits(got[k]), bits(torch.stack(want[k]))), k
    for a, b in zip((th, gt, m1, m2), ref):
        assert torch.equal(bits(torch.stack(a)), bits(torch.stack(b)))


@pytest.mark.parametrize("count,nexp", [(1, 1), (85, 3), (64, 4), (257, 1), (300, 5)])
def test_merge_terms(count, nexp):
    t0, out = arrays(count, 0.02, 1, torch.bfloat16), arrays(count, 1.0, 2, torch.bfloat16)
    ex = [arrays(count, 0.02, 20 + j, torch.bfloat16) for j in range(nexp)]
    rounds = [[[dict(gamma=0.2 + 0.001 * i + 0.1 * k, keep=0.3 + 0.1 * j, seed=(1 << 40) * (j + 1) + i, step=k)
                for j in range(nexp)] for i in range(count)] for k in range(4)]
    got, want = [], []
    with smat.MergePlan(t0, out, ex) as plan:
        for terms in rounds:
            plan.merge(terms)
            got.append(torch.stack(out))
        torch.cuda.synchronize()
    for terms in rounds:
        o = [torch.empty_like(x) for x in out]
        for i in range(count):
            smat.smat_merge([e[i] for e in ex], t0[i], o[i], terms[i], i)
        want.append(torch.stack(o))
    torch.cuda.synchronize()
    for k in range(4):
        assert torch.equal(bits(got[k]), bits(want[k])), k
