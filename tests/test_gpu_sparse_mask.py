"""Keep probabilities below 1/8, where whole 64-byte sectors without a kept element are neither read nor
written: list and single-tensor results equal the same elements' in shards that start off a sector (the
path of every other tensor) bit for bit; dropped coordinates keep their bits whatever they and their
gradients hold; keep around the line and down to none kept."""
import pytest
import torch

import oracle
import paper_2609_33437_amd as smat
from helpers import bits, host
from tolerances import check_theta_tilde

pytestmark = pytest.mark.gpu
DEV = "cuda"
DT = {"bf16": torch.bfloat16, "f32": torch.float32}
SEED, STEP, LAM = 5, 9, 0.5


@pytest.mark.parametrize("keep", [1e-9, 0.002, 0.02, 0.1, 0.1249, 0.125, 0.1251])
@pytest.mark.parametrize("t0_dt,out_dt,g_dt", [("bf16", "bf16", "bf16"), ("f32", "f32", "f32"), ("f32", "bf16", "bf16")])
@pytest.mark.parametrize("n", [16, 255, 256, 1024 * 3 + 7, 70000])
def test_equals_shards_off_a_sector(keep, t0_dt, out_dt, g_dt, n):
    g = torch.Generator(DEV).manual_seed(n)
    randn = lambda s, dt: (torch.randn(n, device=DEV, generator=g) * s).to(dt)  # noqa: E731
    th, t0 = randn(0.02, torch.float32), randn(0.02, DT[t0_dt])
    gs, gt = randn(1e-2, DT[g_dt]), randn(1e-3, torch.float32)
    out = torch.full((n,), float("nan"), dtype=DT[out_dt], device=DEV)
    off = lambda x: torch.cat([x.new_zeros(5), x])[5:]  # noqa: E731  20 or 10 bytes past an allocation's start
    th_o, t0_o, gs_o, gt_o, out_o = (off(x) for x in (th, t0, gs, gt, out))
    for noise, sigma in ((0, 1e-3), (1, 1e-3), (2, 1e-3), (0, 0.0)):
        p = dict(s=0.6, keep=keep, sigma=sigma, noise_kind=noise)
        for a in ((th, t0, out, gs, gt), (th_o, t0_o, out_o, gs_o, gt_o)):
            with smat.Plan([a[0]], [a[2]], [a[1]], [a[3]], [a[4]], tensor_ids=[3]) as plan:
                plan.set_params([p])
                plan.simulate(SEED, STEP)
                plan.backward_accum(SEED, STEP, LAM)
                torch.cuda.synchronize()
        assert torch.equal(bits(out), bits(out_o)) and torch.equal(bits(gt), bits(gt_o))
        single = torch.full_like(out, float("nan"))
        smat.smat_simulate(th, t0, single, p, SEED, STEP, 3)
        torch.cuda.synchronize()
        assert torch.equal(bits(single), bits(out))
    # the last pass (no noise) against the oracle
    thn, t0n = host(th)[0], host(t0)[0]
    y, kept, eps = oracle.simulate_f64(thn, t0n, t0_dt, p, SEED, STEP, 3)
    t = kept * oracle.coefficient(0.6, keep, 1)
    ok, _ = check_theta_tilde(host(out)[0], out_dt, y, oracle.as_f64(thn, "f32"), oracle.as_f64(t0n, t0_dt), t, eps, 0.0)
    assert ok.all()


@pytest.mark.parametrize("keep", [0.02, 0.1])
def test_dropped_coordinates_keep_their_bits(keep):
    n = 1 << 16
    kept = torch.zeros(n, dtype=torch.uint8, device=DEV)
    p = dict(s=1.0, keep=keep, sigma=0.0)
    smat.smat_debug_draws(n, p, SEED, STEP, 1, kept=kept)
    gt = torch.randn(n, device=DEV)
    gs = torch.ones(n, device=DEV, dtype=torch.bfloat16)
    th, t0 = torch.randn(n, device=DEV), torch.randn(n, device=DEV)
    drop = kept == 0
    for x in (gt, gs, th):                      # NaN and infinities where nothing is kept
        x[drop] = float("nan")
        x[drop.nonzero()[::3, 0]] = float("inf")
    before, out = gt.clone(), torch.empty_like(t0)
    smat.smat_backward_accum(gs, gt, p, LAM, SEED, STEP, 1)
    smat.smat_simulate(th, t0, out, p, SEED, STEP, 1)
    torch.cuda.synchronize()
    assert torch.equal(bits(gt)[drop], bits(before)[drop])
    assert bool(gt[~drop].isfinite().all()) and not torch.equal(gt[~drop], before[~drop])
    assert torch.equal(out[drop], t0[drop]) and bool(out.isfinite().all())
