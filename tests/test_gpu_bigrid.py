"""GPU tests of jobs whose one-launch grid would hold more than 2^32 work-items, which a dispatch
cannot express (the count would wrap without an error): the launchers split them into several
launches.  A copy of 68.7 GB, a one-tensor backward of 17.2e9 elements, 4.3e9 raw Philox words, a list of
17.2e9 elements (1.05 million chunks) and a list of 8.4 million tensors (8.4 million segments behind three
chunks) are checked at the piece boundaries and at the end, against the oracle or the single-tensor calls,
and for having written every element.  (tests/test_table_pieces.py walks the same launches on the host, the
gradient norm's included, whose lists would have to be eight times larger.)"""
import ctypes

import numpy as np
import pytest
import torch

import oracle
import paper_2609_33437_amd as smat
from paper_2609_33437_amd import _lib
from helpers import host
from tolerances import check_grad, check_theta_tilde

pytestmark = pytest.mark.gpu
DEV = "cuda"
MAX_BLOCKS = 0xFFFFFFFF // 64          # one-wave blocks per launch
GIB = 1 << 30


def free_gib():
    torch.cuda.empty_cache()
    return torch.cuda.mem_get_info()[0] / GIB


def test_stream_copy_past_the_grid_limit():
    n16 = MAX_BLOCKS * 64 + 12345                       # 16-byte vectors: two launches
    if free_gib() < 2 * n16 * 16 / GIB + 8:
        pytest.skip("needs about 140 GB of free device memory")
    n = n16 * 4
    src = torch.empty(n, dtype=torch.float32, device=DEV)
    piece = 1 << 30
    for off in range(0, n, piece):                      # distinct values in every piece of the check
        src[off:off + piece] = torch.arange(off % 1000003, off % 1000003 + min(piece, n - off), device=DEV,
                                            dtype=torch.float32)
    dst = torch.zeros_like(src)
    smat.smat_stream_copy(src, dst)
    torch.cuda.synchronize()
    for off in range(0, n, piece):
        assert torch.equal(src[off:off + piece], dst[off:off + piece]), off
    del src, dst
    torch.cuda.empty_cache()


def test_backward_one_past_the_grid_limit():
    boundary = MAX_BLOCKS * 256                         # first element of the second launch
    n = boundary + 4099                                 # and a ragged tail
    if free_gib() < n * 6 / GIB + 8:
        pytest.skip("needs about 110 GB of free device memory")
    gen = torch.Generator(DEV).manual_seed(5)
    gs = torch.randn(n, device=DEV, dtype=torch.bfloat16, generator=gen)
    gt = torch.full((n,), 0.25, device=DEV, dtype=torch.float32)
    p = dict(s=0.6, keep=0.5, sigma=0.0, rescale=1)
    lam, seed, step, tid = 0.5, 77, 3, 9
    smat.smat_backward_accum(gs, gt, p, lam, seed, step, tid)
    torch.cuda.synchronize()
    for lo, hi in ((0, 4096), (boundary - 4096, boundary + 4096), (n - 4099, n)):
        gsn, gs_dt = host(gs[lo:hi])
        g_old = np.full(hi - lo, 0.25, dtype=np.float32)
        want = oracle.backward_accum(gsn, gs_dt, g_old, p, lam, seed, step, tid, lo)
        got = host(gt[lo:hi])[0]
        coef = oracle.coefficient(p["s"], p["keep"], p["rescale"])
        assert check_grad(got, want, g_old, np.abs(lam * coef * oracle.as_f64(gsn, gs_dt))).all(), lo
        assert (got != 0.25).any(), lo                  # the range was reached
    del gs, gt
    torch.cuda.empty_cache()


def test_debug_draws_past_the_grid_limit():
    boundary = (0xFFFFFFFF // 256) * 256               # 256-thread blocks: first element of the second launch
    n = boundary + 1029
    if free_gib() < n * 4 / GIB + 8:
        pytest.skip("needs about 25 GB of free device memory")
    words = torch.zeros(n, dtype=torch.int32, device=DEV)
    seed, step, tid, off = 12345, 6, 3, 1 << 33
    smat.smat_debug_draws(n, dict(s=1.0, keep=1.0, sigma=0.0), seed, step, tid, off, mask_words=words)
    torch.cuda.synchronize()
    for lo, hi in ((0, 1024), (boundary - 2048, boundary + 1029), (n - 1029, n)):
        want = oracle.element_words(seed, step, tid, off + lo, hi - lo, 0)
        got = words[lo:hi].cpu().numpy().view(np.uint32)
        np.testing.assert_array_equal(got, want, err_msg=str(lo))
    del words
    torch.cuda.empty_cache()


def _list_plan(theta, theta0, out, grad_sim, grad_theta, n):
    """A plan over tensors of n[i] elements at the given addresses, bf16 but for theta and grad_theta, built
    through the C ABI from one descriptor array (no per-tensor Python objects)."""
    count = len(n)
    desc = np.zeros(count, dtype=np.dtype([("theta", "<u8"), ("theta0", "<u8"), ("out", "<u8"), ("grad_sim", "<u8"),
                                           ("grad_theta", "<u8"), ("theta0_host", "<u8"), ("n", "<i8"),
                                           ("tensor_id", "<u4"), ("reserved", "<u4"), ("elem_offset", "<u8")]))
    assert desc.itemsize == ctypes.sizeof(_lib.smat_tensor_desc)
    desc["theta"], desc["theta0"], desc["out"], desc["grad_sim"], desc["grad_theta"] = \
        theta, theta0, out, grad_sim, grad_theta
    desc["n"] = n
    desc["tensor_id"] = np.arange(count, dtype=np.uint32)
    lib = smat.lib()
    plan = ctypes.c_void_p()
    st = lib.smat_plan_create(desc.ctypes.data_as(ctypes.POINTER(_lib.smat_tensor_desc)), count, _lib.SMAT_BF16,
                              _lib.SMAT_BF16, _lib.SMAT_BF16, 0, ctypes.byref(plan))
    assert st == 0, lib.smat_last_error()
    nb = ctypes.c_size_t()
    assert lib.smat_plan_workspace_bytes(plan, ctypes.byref(nb)) == 0
    ws = torch.empty(nb.value, dtype=torch.uint8, device=DEV)
    assert lib.smat_plan_bind_workspace(plan, ctypes.c_void_p(ws.data_ptr()), nb.value, None) == 0
    return plan, ws


def _set_params(plan, count, **fields):
    params = smat.op_params_array(count, **fields)
    assert smat.lib().smat_plan_set_params(plan, params.ctypes.data_as(ctypes.POINTER(_lib.smat_op_params)), None) == 0


def test_list_past_the_grid_limit():
    """16,400 tensors of 2^20 elements (64 chunks each), two launches at one quad per thread: the second one
    begins with the last chunk of tensor 16,383.  theta0 and g~ are one array for all tensors."""
    n, count = 1 << 20, 16400
    assert count * 64 > MAX_BLOCKS // 64 > 16383 * 64
    if free_gib() < count * n * 10 / GIB + 8:
        pytest.skip("needs about 180 GB of free device memory")
    gen = torch.Generator(DEV).manual_seed(7)
    th = torch.randn(count, n, device=DEV, generator=gen)
    t0 = torch.randn(n, device=DEV, generator=gen).to(torch.bfloat16)
    gs = (torch.randn(n, device=DEV, generator=gen) * 1e-2).to(torch.bfloat16)
    out = torch.full((count, n), float("nan"), device=DEV, dtype=torch.bfloat16)
    gt = torch.full((count, n), 0.25, device=DEV)
    i = np.arange(count, dtype=np.uint64)
    lib, seed, step, lam = smat.lib(), 31, 8, 0.5
    plan, ws = _list_plan(th.data_ptr() + i * (4 * n), t0.data_ptr(), out.data_ptr() + i * (2 * n), gs.data_ptr(),
                          gt.data_ptr() + i * (4 * n), np.full(count, n))
    try:
        _set_params(plan, count, s=0.7, keep=0.4, sigma=1e-2)
        assert lib.smat_simulate_multi(plan, seed, step, None) == 0
        assert lib.smat_backward_multi(plan, seed, step, lam, 1, None) == 0
        torch.cuda.synchronize()
    finally:
        assert lib.smat_plan_destroy(plan) == 0
    p = dict(s=float(np.float32(0.7)), keep=float(np.float32(0.4)), sigma=float(np.float32(1e-2)))
    for k in (0, 1, 8191, 16382, 16383, 16384, count - 1):
        o, g = torch.full_like(t0, float("nan")), torch.full((n,), 0.25, device=DEV)
        smat.smat_simulate(th[k], t0, o, p, seed, step, k)
        smat.smat_backward_accum(gs, g, p, lam, seed, step, k)
        torch.cuda.synchronize()
        assert torch.equal(out[k].view(torch.int16), o.view(torch.int16)), k
        assert torch.equal(gt[k].view(torch.int32), g.view(torch.int32)), k
    for k in range(0, count, 1025):                     # every element was written
        assert bool(torch.isfinite(out[k:k + 1025]).all()), k
        changed = (gt[k:k + 1025] != 0.25).sum(dim=1)
        assert bool((changed > n // 4).all()), k        # 0.4 of each tensor's, less what the addition rounds away
    del th, out, gt
    torch.cuda.empty_cache()


def test_list_of_eight_million_tensors():
    """One tensor of three chunks and 4 elements, then 8.4M of 4 elements, whose remainders run in segments:
    at one quad per thread one launch for the chunks and two for the segments, the second one from segment
    8,388,607 on (tensor 8,388,607).  The overwriting backward (two quads) and the norm take one launch."""
    count, head = 8_400_000, 3 * 16384
    cut = MAX_BLOCKS // 8                               # segments per launch at one quad per thread
    assert 0 < count - cut
    gen = torch.Generator(DEV).manual_seed(6)
    n = head + 4 * count
    th = torch.randn(n, device=DEV, generator=gen) * 0.02
    t0 = (th + torch.randn(n, device=DEV, generator=gen) * 1e-3).to(torch.bfloat16)
    out = torch.full((n,), float("nan"), device=DEV, dtype=torch.bfloat16)
    gs = (torch.randn(n, device=DEV, generator=gen) * 1e-2).to(torch.bfloat16)
    gt = torch.full((n,), float("nan"), device=DEV, dtype=torch.float32)
    acc = torch.full((n,), 0.25, device=DEV, dtype=torch.float32)
    first = np.arange(count, dtype=np.uint64) * 4       # each tensor's first element
    first[1:] += head
    lib, seed, step, lam = smat.lib(), 31, 8, 0.5
    size = np.full(count, 4)
    size[0] += head
    plan, ws = _list_plan(th.data_ptr() + first * 4, t0.data_ptr() + first * 2, out.data_ptr() + first * 2,
                          gs.data_ptr() + first * 2, acc.data_ptr() + first * 4, size)
    try:
        _set_params(plan, count, s=0.7, keep=0.4, sigma=1e-4)
        assert lib.smat_simulate_multi(plan, seed, step, None) == 0
        assert lib.smat_backward_multi(plan, seed, step, lam, 1, None) == 0
        accumulated = acc.clone()
        assert lib.smat_backward_multi(plan, seed, step, lam, 0, None) == 0      # overwrite: writes every element
        gt.copy_(acc)
        sumsq = torch.zeros(1, dtype=torch.float64, device=DEV)
        assert lib.smat_grad_norm_multi(plan, seed, step, lam, 0, 1.0, ctypes.c_void_p(sumsq.data_ptr()), None,
                                        None) == 0
        torch.cuda.synchronize()
    finally:
        assert lib.smat_plan_destroy(plan) == 0
    assert bool(torch.isfinite(out).all()) and bool(torch.isfinite(gt).all()) and not bool((gt == 0.25).any())
    # the norm covers the same gradient that the overwrite wrote, and so does the accumulation (one fused
    # multiply-add onto 0.25: half an ulp of 0.25 and of the product)
    ref = float((gt.double() ** 2).sum())
    assert abs(sumsq.item() - ref) <= 1e-5 * ref
    assert float((accumulated.double() - 0.25 - gt.double()).abs().max()) <= 2.0 ** -26 + 2.0 ** -24 * float(gt.abs().max())
    p = dict(s=float(np.float32(0.7)), keep=float(np.float32(0.4)), sigma=float(np.float32(1e-4)), rescale=1)
    picks = list(range(0, 40)) + list(range(cut - 40, cut + 40)) + list(range(count - 40, count))
    thn, t0n, outn, gsn, gtn = (host(x)[0] for x in (th, t0, out, gs, gt))
    for i in picks:
        e = slice(int(first[i]), int(first[i]) + int(size[i]))
        y, kept, eps = oracle.simulate_f64(thn[e], t0n[e], "bf16", p, seed, step, i)
        coef = np.where(kept, oracle.coefficient(p["s"], p["keep"], p["rescale"]), 0.0)
        ok, _ = check_theta_tilde(outn[e], "bf16", y, thn[e], oracle.as_f64(t0n[e], "bf16"), coef, eps, p["sigma"])
        assert ok.all(), i
        zeros = np.zeros(int(size[i]), np.float32)
        want = oracle.backward_accum(gsn[e], "bf16", zeros, p, lam, seed, step, i)
        incr = np.abs(lam * coef * oracle.as_f64(gsn[e], "bf16"))
        assert check_grad(gtn[e], want, zeros, incr).all(), i
