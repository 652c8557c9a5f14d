"""GPU parity of the expert-parallel share (moe_experts_fwd / moe_experts_bwd)
against the oracle at small sizes: ragged and empty experts, rows left over
past the counts, and counts that overflow the row capacity (rows past the
capacity are dropped: never read, computed or written)."""
import numpy as np
import pytest

import workloads
from oracle import moe_oracle as O
from tests.parity import assert_close, dev_bf16, host

pytestmark = pytest.mark.gpu


def run(rows, H, E, F, counts, seed, dw_fp32=False):
    import torch
    import paper_2608_00916_amd as moe
    s = np.random.SeedSequence(seed).spawn(5)
    xp = workloads.normal_bf16(s[0], (rows, H), 1.0)
    wg = workloads.normal_bf16(s[1], (E, H, F), 0.02)
    wu = workloads.normal_bf16(s[2], (E, H, F), 0.02)
    wd = workloads.normal_bf16(s[3], (E, F, H), 0.02)
    d_o = workloads.normal_bf16(s[4], (rows, H), 1.0)
    counts = np.asarray(counts, dtype=np.int32)
    print(f"GPU experts rows={rows} H={H} E={E} F={F} counts={counts.tolist()}", flush=True)
    ex = moe.MoEExperts(rows, H, E, F, dw_fp32=dw_fp32)
    # sentinel in the output rows that must stay untouched
    ex.o.fill_(7.0)
    ex.dxp.fill_(7.0)
    t = {n: dev_bf16(a) for n, a in (("xp", xp), ("wg", wg), ("wu", wu), ("wd", wd), ("d_o", d_o))}
    ex.forward(t["xp"], torch.from_numpy(counts).cuda(), t["wg"], t["wu"], t["wd"])
    ex.backward(t["xp"], t["wg"], t["wu"], t["wd"], t["d_o"])
    torch.cuda.synchronize()
    # rows beyond the capacity are dropped: the definition restricted to the first `rows` rows
    used = np.minimum(np.cumsum(counts), rows)
    eff = np.diff(np.concatenate([[0], used]))
    R = int(used[-1])
    w = {n: O.widen_bf16(a) for n, a in (("xp", xp), ("wg", wg), ("wu", wu), ("wd", wd), ("d_o", d_o))}
    f = O.experts_share_forward(w["xp"][:R], eff, w["wg"], w["wu"], w["wd"])
    b = O.experts_share_backward(w["xp"][:R], eff, w["wg"], w["wu"], w["wd"], f, w["d_o"][:R])
    o = host(ex.o)
    dxp = host(ex.dxp)
    assert np.array_equal(host(ex.views["offsets"]), f["offsets"])
    if R:
        assert_close("o", o[:R], f["O"])
        assert_close("dxp", dxp[:R], b["dxp"])
    assert np.all(o[R:] == 7.0) and np.all(dxp[R:] == 7.0), "rows past the counts were written"
    tol = 5e-3 if dw_fp32 else 2e-2
    for n, got in (("dw_gate", ex.dw_gate), ("dw_up", ex.dw_up), ("dw_down", ex.dw_down)):
        got = host(got)
        for e in range(E):
            if eff[e] == 0:
                assert np.all(got[e] == 0), f"{n}[{e}] of an empty expert"
            else:
                assert_close(f"{n}[{e}]", got[e], b[n][e], tol)


def test_ragged_and_empty_experts():
    run(700, 256, 6, 128, [130, 0, 257, 1, 0, 300], seed=1)


def test_rows_left_over():
    run(600, 128, 4, 256, [100, 0, 200, 50], seed=2)


def test_counts_overflow_capacity():
    run(300, 128, 4, 128, [200, 150, 100, 0], seed=3)


def test_fp32_weight_grads():
    run(512, 256, 3, 128, [200, 150, 162], seed=4, dw_fp32=True)


def test_recompute_is_bit_identical():
    """The experts path with MOE_F_RECOMPUTE matches the run that kept G and U
    bit for bit."""
    import torch
    import paper_2608_00916_amd as moe
    rows, H, E, F = 700, 256, 6, 256
    counts = np.array([130, 0, 257, 1, 0, 300], dtype=np.int32)
    s = np.random.SeedSequence(5).spawn(5)
    t = {n: dev_bf16(workloads.normal_bf16(q, shape, std)) for n, q, shape, std in (
        ("xp", s[0], (rows, H), 1.0), ("wg", s[1], (E, H, F), 0.02), ("wu", s[2], (E, H, F), 0.02),
        ("wd", s[3], (E, F, H), 0.02), ("d_o", s[4], (rows, H), 1.0))}
    print(f"GPU experts recompute rows={rows} H={H} E={E} F={F}", flush=True)
    c = torch.from_numpy(counts).cuda()
    outs = []
    for recompute in (False, True):
        ex = moe.MoEExperts(rows, H, E, F, recompute=recompute)
        ex.o.zero_()
        ex.dxp.zero_()
        ex.forward(t["xp"], c, t["wg"], t["wu"], t["wd"])
        ex.backward(t["xp"], t["wg"], t["wu"], t["wd"], t["d_o"])
        torch.cuda.synchronize()
        outs.append({n: host(getattr(ex, n)) for n in ("o", "dxp", "dw_gate", "dw_up", "dw_down")})
        outs[-1]["a"] = host(ex.views["a"][:int(counts.sum())])  # rows past the counts are undefined
        if recompute:
            assert ex.views["g"] is None and ex.views["u"] is None
    for n in outs[0]:
        assert np.array_equal(outs[0][n], outs[1][n]), n


def tall_flags(ex):
    """Whether the down and the gate/up weight gradients of the last backward
    ran on 256-row tiles.  The schedule is the last region of the experts'
    workspace: the experts in their order, 2 x 9 tile bounds, the two flags."""
    n = ex.d.E + 2 * 9 + 2
    start = ex.ws.numel() - -(-n * 4 // 256) * 256
    plan = ex.ws[start:start + n * 4].cpu().numpy().view(np.int32)
    assert np.array_equal(np.sort(plan[:ex.d.E]), np.arange(ex.d.E)), "not the schedule"
    return bool(plan[-2]), bool(plan[-1])


def test_tall_weight_gradient_tiles():
    """Enough tiles for the 256-row weight-gradient tiles, with rows per expert
    around their 32-row steps, down to none and up to more steps (14) than a
    staged tile has drain calls (12): parity with the oracle on one expert of
    each count, and every expert's gradients bitwise those of a run whose one
    long expert sends the plan to the 128-row tiles (both sum the rows in the
    same order).  The plan's flags say which tiles either run took."""
    import torch
    import paper_2608_00916_amd as moe
    E, H, F = 256, 512, 512
    kinds = [0, 1, 31, 32, 33, 63, 64, 65, 95, 96, 97, 200, 385, 416, 417, 417]
    counts = np.array(kinds * (E // len(kinds)), dtype=np.int32)
    counts[-1] = 40
    rows = int(counts.sum()) + 8192
    g = torch.Generator(device="cuda")
    g.manual_seed(7)
    t = {n: torch.empty(shape, dtype=torch.bfloat16, device="cuda").normal_(0.0, std, generator=g) for n, shape, std in (
        ("xp", (rows, H), 1.0), ("wg", (E, H, F), 0.02), ("wu", (E, H, F), 0.02), ("wd", (E, F, H), 0.02),
        ("d_o", (rows, H), 1.0))}
    ex = moe.MoEExperts(rows, H, E, F)
    grads = []
    for last, tall in ((40, True), (40 + 8192, False)):
        c = counts.copy()
        c[-1] = last
        print(f"GPU experts tall rows={int(c.sum())} H={H} E={E} F={F} last={last}", flush=True)
        ex.forward(t["xp"], torch.from_numpy(c).cuda(), t["wg"], t["wu"], t["wd"])
        ex.backward(t["xp"], t["wg"], t["wu"], t["wd"], t["d_o"])
        torch.cuda.synchronize()
        assert tall_flags(ex) == (tall, tall)
        grads.append([w.clone() for w in (ex.dw_gate, ex.dw_up, ex.dw_down)])
    for a, b in zip(*grads):
        assert torch.equal(a[:-1], b[:-1])
        assert not torch.equal(a[-1], b[-1])
    ends = np.cumsum(counts)
    for e in range(len(kinds)):
        n = int(counts[e])
        if n == 0:
            assert not any(w[e].any() for w in grads[0])
            continue
        sl = slice(int(ends[e]) - n, int(ends[e]))
        w = {m: host(v[e:e + 1]) for m, v in t.items() if m in ("wg", "wu", "wd")}
        x, d_o = host(t["xp"][sl]), host(t["d_o"][sl])
        one = np.array([n])
        f = O.experts_share_forward(x, one, w["wg"], w["wu"], w["wd"])
        b = O.experts_share_backward(x, one, w["wg"], w["wu"], w["wd"], f, d_o)
        for m, got in zip(("dw_gate", "dw_up", "dw_down"), grads[0]):
            assert_close(f"{m}[{e}]", host(got[e]), b[m][0], 2e-2)


@pytest.mark.parametrize("H,n,flags", [
    (1536, 0, (False, False)), (1536, 2, (False, False)), (1536, 3, (True, True)), (1536, 24, (True, True)),
    (1536, 25, (False, False)), (1536, 41, (False, False)), (1536, 42, (True, True)), (1024, 24, (False, True)),
    (1024, 25, (False, False)), (1024, 47, (False, True)), (1024, 48, (True, True))])
def test_tall_tiles_follow_rows_per_expert(H, n, flags):
    """The plan takes 256-row tiles for a mean of 3 to 24 rows per expert and
    from 42 on, with fewer than 12 of them per workgroup from 48 on only (E = 256,
    F = 512: down and gate/up have 12 and 24 of them at H = 1536, 8 and 16 at
    H = 1024)."""
    import torch
    import paper_2608_00916_amd as moe
    E, F = 256, 512
    print(f"GPU experts tall rule H={H} E={E} F={F} n={n}", flush=True)
    rows = E * n + 1
    w = [torch.zeros(E, a, b, dtype=torch.bfloat16, device="cuda") for a, b in ((H, F), (H, F), (F, H))]
    x = torch.zeros(rows, H, dtype=torch.bfloat16, device="cuda")
    ex = moe.MoEExperts(rows, H, E, F)
    ex.forward(x, torch.full((E,), n, dtype=torch.int32, device="cuda"), *w)
    ex.backward(x, *w, x)
    torch.cuda.synchronize()
    assert tall_flags(ex) == flags
