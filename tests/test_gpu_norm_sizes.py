"""The gradient norm at the sizes where its reduction changes form: around whole tiles of 2,048 elements
(the unguarded path), one block's 1,024 partials, and the 8,192 partials from which two launches add
them; against the gradient in 64 bits, and the same bits on every call."""
import pytest
import torch

import paper_2609_33437_amd as smat

pytestmark = pytest.mark.gpu
DEV = "cuda"
TILE = 2048


@pytest.mark.parametrize("grad", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("accumulate", [False, True])
@pytest.mark.parametrize("n", [TILE - 1, TILE, TILE + 1, 1023 * TILE, 1024 * TILE + 5, 8191 * TILE + 3, 8192 * TILE,
                               8192 * TILE + 1])
def test_norm(n, grad, accumulate):
    g = torch.Generator(DEV).manual_seed(n)
    th, gt = torch.zeros(n, device=DEV), torch.randn(n, device=DEV, generator=g) * 1e-3
    out = torch.zeros(n, device=DEV, dtype=torch.bfloat16)
    gs = (torch.randn(n, device=DEV, generator=g) * 1e-2).to(grad)
    got = []
    want_g = gt.clone() if accumulate else torch.zeros_like(gt)
    p = dict(s=0.7, keep=0.5, sigma=0.0)
    smat.smat_backward_accum(gs, want_g, p, 0.5, 9, 3)
    with smat.Plan([th], [out], [out.clone()], [gs], [gt]) as plan:
        plan.set_params([p])
        for _ in range(2):
            sumsq, coef = torch.zeros(1, dtype=torch.float64, device=DEV), torch.zeros(1, device=DEV)
            plan.grad_norm(9, 3, 0.5, accumulate, 0.25, sumsq, coef)
            torch.cuda.synchronize()
            got.append((float(sumsq), float(coef)))
    assert got[0] == got[1]
    want = float(want_g.double().square().sum())
    # fp32 partial sums of at most 32 squares per lane and 64 lanes: relative error within 96 u
    assert abs(got[0][0] - want) <= 96 * 2.0 ** -24 * want
    assert abs(got[0][1] - min(1.0, 0.25 / (want ** 0.5 + 1e-6))) <= 1e-6
