"""Vocabulary slabs on the GPU against the oracle, either side of the few-token rule: calls whose whole
vocabulary is one slab although it is far wider than the rule's width for many tokens, and calls of
more than 4096 tokens, whose vocabulary takes several slabs (the dH accumulators are added to slab by
slab, the last slab is ragged)."""
import numpy as np
import pytest

from oracle import lce_oracle as O
from paper_2605_21442_amd import binding as B
from paper_2605_21442_amd import workloads as WL
from tests import lce_testutil as U

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,d,v,mask,reduction,nslab", [
    (4400, 64, 50001, 0.3, "mean", 3), (4353, 192, 26000, 0.0, "sum", 2),
    (700, 128, 50001, 0.2, "mean", 1), (257, 264, 33000, 0.1, "none", 1), (1, 64, 100000, 0.0, "mean", 1)])
def test_slabs_match_the_oracle(n, d, v, mask, reduction, nslab):
    assert B.lce_plan_info(B.problem(n, d, v))["nslab"] == nslab
    inp = WL.custom(n, d, v, seed=n, mask_frac=mask, sigma_w=0.3, case_id=53)
    grad = np.random.default_rng(n).standard_normal(n).astype(np.float32) if reduction == "none" else 1.0
    print(f"case n={n} d={d} v={v} {reduction} slabs={nslab}", flush=True)
    h, w, t = U.to_device(inp)
    gpu = U.run_gpu(h, w, t, inp.ignore_index, reduction, grad)
    U.assert_parity(gpu, O.lce(inp.h_bits, inp.w_bits, inp.targets, inp.ignore_index, reduction,
                               grad.astype(np.float64) if reduction == "none" else 1.0))


@pytest.mark.parametrize("n,d,nv,parts", [(256, 512, 230, 8), (700, 264, 1, 8), (2048, 1024, 1536, 8), (2048, 2048, 1537, 6),
                                          (4096, 2048, 3072, 4), (4096, 2048, 4096, 5), (11008, 2048, 7000, 3)])
def test_split_dh_parts_match_the_oracle_blockwise(n, d, nv, parts):
    # the K parts a split dH launch takes follow from Nv; every 384 x 256 block of dH is compared
    from tests.test_bounds_cpu import dh_split_blocks
    from tests.test_gpu_dh_split import _inputs
    kz_max = B.lce_plan_info(B.problem(n, d, 1000))["dh_kz"]
    assert next(iter(dh_split_blocks(n, nv, d, kz_max)))[4] == parts
    inp, valid = _inputs(n, d, nv, seed=7)
    print(f"case n={n} d={d} nv={nv} parts={parts}", flush=True)
    h, w, t = U.to_device(inp)
    gpu = U.run_gpu(h, w, t, inp.ignore_index, "mean", 1.0)
    ref = O.lce(inp.h_bits, inp.w_bits, inp.targets, inp.ignore_index, "mean", 1.0)
    U.assert_parity(gpu, ref)
    dh, dh_ref = gpu["dH"][valid], ref["dH"][valid]
    for m0 in range(0, nv, 384):
        for d0 in range(0, d, 256):
            blk, rb = dh[m0:m0 + 384, d0:d0 + 256], dh_ref[m0:m0 + 384, d0:d0 + 256]
            assert np.linalg.norm(blk - rb) <= U.GRAD_REL_TOL * np.linalg.norm(rb), (m0, d0)


@pytest.mark.parametrize("n,d,v,accumulate", [(8448, 4352, 700, False), (8600, 5888, 700, True), (8832, 8448, 400, False),
                                              (300, 264, 1000, True), (500, 72, 26000, True),
                                              # dW's blocks first (420 valid tokens against a part of 376 ids), and
                                              # dH's (against 2500)
                                              (9000, 512, 3001, False), (9000, 512, 20000, False)])
def test_dh_and_dw_in_one_launch_or_two_match_the_oracle(n, d, v, accumulate):
    # either side of the rule (768 dH tiles), with and without the accumulating dW epilogue; most rows
    # ignored where the widths are large, so that the oracle stays quick
    import torch
    from paper_2605_21442_amd import autograd as A
    rng = np.random.default_rng([n, d])
    t = np.full(n, -100, dtype=np.int32)
    valid = rng.choice(n, size=min(n, 420), replace=False)
    t[valid] = rng.integers(0, v, size=len(valid), dtype=np.int32)
    inp = WL.custom(n, d, v, seed=9, sigma_w=0.05, target_override=t)
    print(f"case n={n} d={d} v={v} accumulate={accumulate}", flush=True)
    h, w, tt = U.to_device(inp)
    loss, lse, nv, _, ws = A.forward(h, w, tt, keep_workspace=True)
    base = torch.randn((v, d), generator=torch.Generator("cuda").manual_seed(1), device="cuda").mul_(1e-3).bfloat16()
    acc = base.clone() if accumulate else None
    dh, dw = A.backward(h, w, tt, lse, nv, torch.ones(1, device="cuda"), accumulate_into=acc, workspace=ws)
    ref = O.lce(inp.h_bits, inp.w_bits, inp.targets)
    want = ref["dW"] + (base.float().cpu().numpy() if accumulate else 0.0)
    assert abs(float(loss) - ref["loss"]) <= U.LOSS_ABS_TOL
    assert U.rel_fro(dh.float().cpu().numpy(), ref["dH"]) <= U.GRAD_REL_TOL
    assert U.rel_fro(dw.float().cpu().numpy(), want) <= U.GRAD_REL_TOL


@pytest.mark.parametrize("n,d,v", [(700, 264, 5000), (2048, 1024, 9000), (4400, 64, 50001), (12288, 2048, 500), (0, 64, 300)])
@pytest.mark.parametrize("frozen", ["weight", "hidden"])
def test_a_gradient_that_is_not_wanted_leaves_the_other_as_it_was(n, d, v, frozen):
    # a frozen head (or hidden states without a gradient): one contraction less, the other's bits the same
    import torch
    from paper_2605_21442_amd import linear_cross_entropy
    inp = WL.custom(n, d, v, seed=5, mask_frac=0.3, sigma_w=0.3, case_id=54)
    h, w, t = U.to_device(inp)
    print(f"case n={n} d={d} v={v} frozen={frozen}", flush=True)
    grads = {}
    for both in (True, False):
        x = h.clone().requires_grad_(both or frozen != "hidden")
        y = w.clone().requires_grad_(both or frozen != "weight")
        linear_cross_entropy(x, y, t).backward()
        grads[both] = (x.grad, y.grad)
    k = 0 if frozen == "weight" else 1
    assert grads[False][1 - k] is None
    assert torch.equal(grads[True][k].view(torch.int16), grads[False][k].view(torch.int16))


@pytest.mark.parametrize("n,d,v", [(700, 264, 20000), (300, 72, 9216), (520, 1000, 9217), (64, 8, 40000), (257, 56, 384), (300, 64, 40000),
                                   (64, 8, 200000)])
def test_ragged_widths_and_the_least_forward_workspace(n, d, v):
    # widths that are not a multiple of 64 on the 384 x 256 tiles (their last K slice masked), and the forward
    # of those and of narrow heads in the least workspace (groups of 24 tiles, a launch each, folded into running pairs): the losses agree
    # to fp32 rounding of the merge order
    import torch
    inp = WL.custom(n, d, v, seed=3, mask_frac=0.2, sigma_w=0.3, case_id=55)
    print(f"case n={n} d={d} v={v}", flush=True)
    h, w, t = U.to_device(inp)
    p = B.problem(n, d, v, reduction="none")
    info = B.lce_plan_info(p)
    rows = (v + 383) // 384
    rows = rows if rows <= 24 else 49
    least = info["o_pm"] + 2 * ((4 * rows * info["npad"] + 255) // 256 * 256) + 4 * info["npad"]
    ref = O.lce(inp.h_bits, inp.w_bits, inp.targets, reduction="none", grad=np.ones(n))
    out = []
    for nbytes in (info["fwd_bytes"], least):
        loss = torch.empty(n, dtype=torch.float32, device="cuda")
        lse = torch.empty(n, dtype=torch.float32, device="cuda")
        nv = torch.empty(1, dtype=torch.int32, device="cuda")
        ws = torch.full((nbytes + 256,), 0xFF, dtype=torch.uint8, device="cuda")
        B.lce_forward(p, h.data_ptr(), w.data_ptr(), t.data_ptr(), loss.data_ptr(), lse.data_ptr(), nv.data_ptr(), 0,
                      ws.data_ptr(), nbytes, torch.cuda.current_stream().cuda_stream)
        assert torch.all(ws[nbytes:] == 0xFF)
        assert np.max(np.abs(loss.cpu().numpy() - ref["loss"])) <= 2e-5 * max(1.0, np.max(np.abs(ref["lse"])))
        out.append(lse.cpu().numpy())
    assert np.max(np.abs(out[0] - out[1])) <= 1e-5 * max(1.0, np.max(np.abs(out[0])))
    gpu = U.run_gpu(h, w, t, inp.ignore_index, "none", np.ones(n, np.float32))
    U.assert_parity(gpu, ref)


@pytest.mark.parametrize("n,d,v", [(256, 64, 384 * 64), (255, 72, 384 * 64 + 1), (257, 64, 384 * 65 - 191), (1, 128, 384 * 33),
                                   (129, 64, 384 * 128), (128, 200, 192), (384, 64, 193), (300, 64, 384 * 129),
                                   (513, 64, 384 * 105), (640, 64, 384 * 110 + 200), (64, 1024, 5000),
                                   (100, 136, 384 * 150 + 7), (384, 64, 384 * 90), (385, 64, 384 * 90)])
@pytest.mark.parametrize("sigma", [0.05, 1.0])
def test_launches_whose_last_round_is_cut_match_the_oracle(n, d, v, sigma):
    # forward and G launches of 64, 65, 128 and 129 tiles (4, 2, 2 and 1 parts per tile), tails after whole rounds,
    # ids and tokens that end inside, at and before a part, last token tiles of 1, 100, 128 and 129 tokens (half as
    # wide up to 128); every token's loss and lse to fp32 rounding
    inp = WL.custom(n, d, v, seed=v % 1000 + n, mask_frac=0.0, sigma_w=sigma, case_id=56)
    g = np.random.default_rng(n).standard_normal(n).astype(np.float32)
    print(f"case n={n} d={d} v={v} sigma={sigma}", flush=True)
    h, w, t = U.to_device(inp)
    gpu = U.run_gpu(h, w, t, inp.ignore_index, "none", g)
    ref = O.lce(inp.h_bits, inp.w_bits, inp.targets, inp.ignore_index, "none", g.astype(np.float64))
    U.assert_parity(gpu, ref)
    scale = max(1.0, np.max(np.abs(ref["lse"])))
    assert np.max(np.abs(gpu["lse"] - ref["lse"])) <= 1e-5 * scale
    assert np.max(np.abs(gpu["loss"] - ref["loss"])) <= 2e-5 * scale


def _guarded(nbytes):
    """A workspace of nbytes between two runs of 0xFF that a call must leave as they are."""
    import torch
    buf = torch.full((nbytes + 8192,), 0xFF, dtype=torch.uint8, device="cuda")
    start = 256 * ((buf.data_ptr() + 4096 + 255) // 256) - buf.data_ptr()
    return buf, buf[start:start + nbytes], lambda: bool((buf[:start] == 0xFF).all() and (buf[start + nbytes:] == 0xFF).all())


@pytest.mark.parametrize("n,d,v,mask", [(700, 128, 50001, 0.2), (300, 264, 33000, 0.0), (2048, 1024, 30000, 0.25), (64, 64, 800, 0.0)])
def test_the_least_workspace_serves_forward_backward_and_optimizer_step(n, d, v, mask):
    # the rule's slabs and fewer K parts of dH in place of the few-token form, both passes in one buffer (reuse)
    import torch
    inp = WL.custom(n, d, v, seed=12, mask_frac=mask, sigma_w=0.3, case_id=57)
    print(f"case least n={n} d={d} v={v}", flush=True)
    h, w, t = U.to_device(inp)
    p, pb = B.problem(n, d, v), B.problem(n, d, v, flags=B.LCE_FLAG_REUSE_FORWARD)
    size = max(B.lce_workspace_size_least(p))
    buf, ws, whole = _guarded(size)
    s = torch.cuda.current_stream().cuda_stream
    f32 = lambda k: torch.empty(k, dtype=torch.float32, device="cuda")
    loss, lse, nv, g = f32(1), f32(n), torch.empty(1, dtype=torch.int32, device="cuda"), torch.ones(1, device="cuda")
    dh, dw, dh2 = torch.empty_like(h), torch.empty_like(w), torch.empty_like(h)
    B.lce_forward(p, h.data_ptr(), w.data_ptr(), t.data_ptr(), loss.data_ptr(), lse.data_ptr(), nv.data_ptr(), 0,
                  ws.data_ptr(), size, s)
    for q in (pb, p):
        B.lce_backward(q, h.data_ptr(), w.data_ptr(), t.data_ptr(), lse.data_ptr(), nv.data_ptr(), g.data_ptr(),
                       dh.data_ptr(), dw.data_ptr(), ws.data_ptr(), size, s)
        torch.cuda.synchronize()
        gpu = dict(loss=float(loss), lse=lse.cpu().numpy().astype(np.float64), n_valid=int(nv), status=0,
                   dH=dh.float().cpu().numpy().astype(np.float64), dW=dw.float().cpu().numpy().astype(np.float64))
        U.assert_parity(gpu, O.lce(inp.h_bits, inp.w_bits, inp.targets))
    w2, m, v2 = w.clone(), torch.zeros_like(w, dtype=torch.float32), torch.zeros_like(w, dtype=torch.float32)
    B.lce_backward_adamw(p, h.data_ptr(), w2.data_ptr(), t.data_ptr(), lse.data_ptr(), nv.data_ptr(), g.data_ptr(),
                         dh2.data_ptr(), m.data_ptr(), v2.data_ptr(), 0, B.adamw(1e-3, 0.9, 0.999, 1e-8, 0.01, 1),
                         ws.data_ptr(), size, s)
    torch.cuda.synchronize()
    assert torch.equal(dh.view(torch.int16), dh2.view(torch.int16))
    assert torch.equal(m, dw.float() * np.float32(1 - np.float64(np.float32(0.9))))
    assert whole()


@pytest.mark.parametrize("n,ds,dt,v,mask", [(300, 64, 128, 30000, 0.2), (513, 128, 200, 26001, 0.0), (40, 64, 64, 700, 0.0)])
def test_the_least_workspace_serves_the_distillation_calls(n, ds, dt, v, mask):
    import torch
    from oracle import kd_oracle as K
    inp = WL.kd_custom(n, ds, dt, v, seed=13, mask_frac=mask)
    print(f"case kd least n={n} ds={ds} dt={dt} v={v}", flush=True)
    bf = lambda b: torch.from_numpy(b.view(np.int16)).view(torch.bfloat16).cuda()
    hs, ws, ht, wt, t = bf(inp.hs_bits), bf(inp.ws_bits), bf(inp.ht_bits), bf(inp.wt_bits), torch.from_numpy(inp.targets).cuda()
    p = B.kd_problem(n, ds, dt, v, temperature=2.0, target_bytes=t.element_size())
    ref = K.kd_bits(inp.hs_bits, inp.ws_bits, inp.ht_bits, inp.wt_bits, inp.targets, temperature=2.0)
    fb, bb = B.lce_kd_workspace_size_least(p)
    s = torch.cuda.current_stream().cuda_stream
    ptrs = [x.data_ptr() for x in (hs, ws, ht, wt, t)]
    g = torch.ones(1, device="cuda")
    got = []
    for fused in (False, True):
        loss, lse_s, lse_t = (torch.empty(k, dtype=torch.float32, device="cuda") for k in (1, n, n))
        nv, st = (torch.empty(1, dtype=torch.int32, device="cuda") for _ in range(2))
        dh, dw = torch.empty_like(hs), torch.empty_like(ws)
        fbuf, fws, fwhole = _guarded(fb)
        bbuf, bws, bwhole = _guarded(bb)
        if fused:
            B.lce_kd_forward_backward(p, *ptrs, g.data_ptr(), loss.data_ptr(), lse_s.data_ptr(), lse_t.data_ptr(),
                                      nv.data_ptr(), st.data_ptr(), dh.data_ptr(), dw.data_ptr(), bws.data_ptr(), bb, s)
        else:
            B.lce_kd_forward(p, *ptrs, loss.data_ptr(), lse_s.data_ptr(), lse_t.data_ptr(), nv.data_ptr(), st.data_ptr(),
                             fws.data_ptr(), fb, s)
            B.lce_kd_backward(p, *ptrs, lse_s.data_ptr(), lse_t.data_ptr(), nv.data_ptr(), g.data_ptr(), dh.data_ptr(),
                              dw.data_ptr(), bws.data_ptr(), bb, s)
        torch.cuda.synchronize()
        assert fwhole() and bwhole()
        assert abs(float(loss) - ref["loss"]) <= U.LOSS_ABS_TOL
        for x, k in ((dh, "dHs"), (dw, "dWs")):
            assert U.rel_fro(x.float().cpu().numpy(), ref[k]) <= U.GRAD_REL_TOL, k
        got.append((loss, lse_s, lse_t, dh.view(torch.int16), dw.view(torch.int16)))
    assert all(torch.equal(a, b) for a, b in zip(*got))       # one call or two, the same bits


def test_a_device_without_room_for_the_wide_slabs_takes_the_least_workspace(monkeypatch):
    # a cap on the process's memory between the two sizes: forward and backward run in the smaller one
    import torch
    from paper_2605_21442_amd import autograd as A, linear_cross_entropy, linear_kd_loss
    n, d, v = 2048, 512, 100000
    p = B.problem(n, d, v, target_bytes=8)
    big, least = max(B.lce_workspace_size(p)), max(B.lce_workspace_size_least(p))
    assert big > 3 * least // 2
    real, asked = torch.empty, []

    def empty(*size, **kw):
        if kw.get("dtype") is torch.uint8:
            asked.append(size[0])
            if size[0] > (big + least) // 2:
                raise torch.OutOfMemoryError("no room")
        return real(*size, **kw)

    inp = WL.custom(n, d, v, seed=14, mask_frac=0.25, sigma_w=0.1, case_id=58)
    h, w, t = U.to_device(inp, target_dtype=torch.int64)
    grads = []
    for tight in (False, True):
        if tight:
            monkeypatch.setattr(A.torch, "empty", empty)
        x, y = h.clone().requires_grad_(True), w.clone().requires_grad_(True)
        linear_cross_entropy(x, y, t).backward()
        kd = linear_kd_loss(x, y, h[:, :64], w[:, :64], t)
        grads.append([x.grad.float(), y.grad.float(), *(g.float() for g in torch.autograd.grad(kd, (x, y)))])
    monkeypatch.undo()
    assert asked[0] == big and asked[1] == least
    for a, b in zip(*grads):
        assert float((a - b).norm() / a.norm()) <= 1e-3 and bool(torch.isfinite(b).all())


@pytest.mark.parametrize("n,d,v,nv", [(16385, 64, 3000, 1), (16385, 64, 3000, 700), (17000, 200, 49000, 64), (16500, 1536, 2000, 65),
                                      (16384, 64, 3000, 700), (16385, 1544, 2000, 65), (16385, 64, 60001, 63)])
def test_both_widths_of_the_partials_merge_match_the_oracle(n, d, v, nv):
    # 64 tokens a workgroup from 16385 tokens on, up to 1536 wide, and 16 just outside; 1 to 65 valid tokens, and
    # the least workspace's running pairs folded in first
    import torch
    rng = np.random.default_rng([n, d, nv])
    t = np.full(n, -100, dtype=np.int32)
    rows = np.sort(rng.choice(n, size=nv, replace=False))
    t[rows] = rng.integers(0, v, size=nv, dtype=np.int32)
    inp = WL.custom(n, d, v, seed=15, sigma_w=0.2, target_override=t)
    print(f"case merge n={n} d={d} v={v} nv={nv}", flush=True)
    h, w, tt = U.to_device(inp)
    ref = O.lce(inp.h_bits, inp.w_bits, inp.targets, reduction="none", grad=np.ones(n))
    p = B.problem(n, d, v, reduction="none")
    scale = max(1.0, np.max(np.abs(ref["lse"])))
    for nbytes in (B.lce_workspace_size(p)[0], B.lce_workspace_size_least(p)[0]):
        loss, lse = (torch.full((n,), float("nan"), dtype=torch.float32, device="cuda") for _ in range(2))
        cnt = torch.empty(1, dtype=torch.int32, device="cuda")
        ws = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
        B.lce_forward(p, h.data_ptr(), w.data_ptr(), tt.data_ptr(), loss.data_ptr(), lse.data_ptr(), cnt.data_ptr(), 0,
                      ws.data_ptr(), nbytes, torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
        assert int(cnt) == nv
        assert np.max(np.abs(lse.cpu().numpy() - ref["lse"])) <= 1e-5 * scale
        assert np.max(np.abs(loss.cpu().numpy() - ref["loss"])) <= 2e-5 * scale
