"""Short calls on the GPU (query tiles of 128 (row, head) pairs, their keys dealt to several workgroups, steps
joined in one launch) against the oracle, at the sizes where tiles, shares and segment lists end."""
import ctypes as C

import numpy as np
import pytest
import torch

from paper_2509_26541_amd import workloads as wl
from tests.helpers import max_abs, oracle_grads, oracle_rows

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def tb():
    assert torch.cuda.is_available(), "GPU tests need an MI355X"
    from paper_2509_26541_amd import binding
    return binding


# name, N, rank, S, Hq, Hkv, d, dtype, mask
EDGES = [
    ("one_row_g3", 4, 3, 4, 3, 1, 128, "fp32", wl.FULL),                      # L = 1, three heads to a KV head
    ("tile_minus_1", 4, 1, 4 * 127, 1, 1, 64, "fp32", wl.FULL),
    ("tile", 8, 2, 16 * 128, 2, 2, 128, "fp32", wl.ZIGZAG_CAUSAL),
    ("tile_plus_1_g3", 8, 5, 16 * 43, 6, 2, 64, "fp32", wl.ZIGZAG_CAUSAL),   # 43 x 3 = 129 pairs
    ("tile_bf16_g8", 8, 0, 16 * 16, 8, 1, 128, "bf16", wl.ZIGZAG_CAUSAL),    # 16 x 8 = 128 pairs, the fewest keys
    ("tile_plus_bf16", 8, 7, 16 * 129, 2, 2, 64, "bf16", wl.ZIGZAG_CAUSAL),
    ("many_shares", 4, 2, 4 * 1031, 1, 1, 128, "bf16", wl.FULL),             # 32 shares of a prime number of keys
    ("many_shares_fp32", 8, 6, 16 * 257, 1, 1, 64, "fp32", wl.ZIGZAG_CAUSAL),
    ("small_pieces", 16, 11, 32 * 64, 4, 2, 64, "bf16", wl.ZIGZAG_CAUSAL),   # sub-chunks of four keys
    ("small_pieces_fp32", 16, 15, 32 * 31, 2, 1, 128, "fp32", wl.ZIGZAG_CAUSAL),
    ("many_ranks", 32, 17, 64 * 33, 2, 1, 64, "fp32", wl.ZIGZAG_CAUSAL),     # sub-chunks of one key
]


@pytest.mark.parametrize("case", EDGES, ids=[c[0] for c in EDGES])
def test_short_calls_all_rows(tb, case):
    name, n, rank, S, Hq, Hkv, d, dtype, mode = case
    w = wl.Workload(name, n, rank, S, Hq, Hkv, d, dtype, mode, seed=wl.BASE_SEED + 8000 + S)
    q, k, v = wl.make_qkv(w)
    qd, kd, vd = q.cuda(), k.cuda(), v.cuda()
    s = tb.tasp_schedule(n, rank)
    rows = list(range(w.L))
    ref_o, ref_l = oracle_rows(w, q, k, v, rows)
    tol_o, tol_l = (2e-2, 1e-3) if dtype == "bf16" else (1e-4, 1e-4)
    for fuse in (False, True):
        plan = tb.ChunkAttnPlan(s, qd, kd, vd, mode, fuse_merge=fuse)
        least = tb.lib.tasp_chunk_attn_workspace_bytes(s.handle, C.byref(plan.args))
        assert least <= plan.args.workspace_bytes <= max(least, tb.STATIC_SCRATCH_BYTES)
        # with room for every share, and with the least workspace the call takes
        for nbytes in {plan.args.workspace_bytes, least}:
            plan.args.workspace_bytes = nbytes
            plan.out.fill_(float("nan"))
            out, lse = plan.run()
            torch.cuda.synchronize()
            eo, el = max_abs(out.float().cpu().numpy(), ref_o), max_abs(lse.cpu().numpy(), ref_l)
            assert eo <= tol_o and el <= tol_l, (name, fuse, nbytes, eo, el)


@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
@pytest.mark.parametrize("d", [64, 128])
def test_steps_of_many_segments(tb, d, dtype):
    """Steps by themselves, the most segments a query block can have (31 rings, two each) and most of them of one key: every row
    of the pairs of all steps, merged."""
    n, rank, S, Hq, Hkv = 32, 17, 64 * 33, 2, 1
    w = wl.Workload("many_segments", n, rank, S, Hq, Hkv, d, dtype, wl.ZIGZAG_CAUSAL, seed=wl.BASE_SEED + 8300 + d)
    q, k, v = wl.make_qkv(w)
    s = tb.tasp_schedule(n, rank)
    ref_o, ref_l = oracle_rows(w, q, k, v, list(range(w.L)))
    parts = [tb.tasp_step_attn(q.cuda(), k.cuda(), v.cuda(), s, w.mask_mode, i) for i in range(n)]
    o, lse = tb.tasp_lse_merge_many([o for o, _ in parts], [l for _, l in parts])
    tol_o, tol_l = (2e-2, 1e-3) if dtype == "bf16" else (1e-4, 1e-4)
    assert max_abs(o.cpu().numpy(), ref_o) <= tol_o and max_abs(lse.cpu().numpy(), ref_l) <= tol_l


def test_fp32_fused_merge_leaves_an_unaligned_workspace_alone(tb):
    """fp32 with the merge folded in needs no workspace, so its pointer is not checked: shares of the keys, which
    would use it, are only planned where it is aligned."""
    w = wl.Workload("unaligned", 4, 1, 1024, 4, 4, 64, "fp32", wl.FULL, seed=wl.BASE_SEED + 8400)
    q, k, v = wl.make_qkv(w)
    plan = tb.ChunkAttnPlan(tb.tasp_schedule(4, 1), q.cuda(), k.cuda(), v.cuda(), w.mask_mode, fuse_merge=True)
    assert tb.lib.tasp_chunk_attn_workspace_bytes(plan.schedule.handle, C.byref(plan.args)) == 0
    assert plan.args.workspace_bytes > 256
    plan.workspace.fill_(77)
    plan.args.workspace += 4
    plan.args.workspace_bytes -= 4
    out, lse = plan.run()
    torch.cuda.synchronize()
    rows = list(range(w.L))
    ref_o, ref_l = oracle_rows(w, q, k, v, rows)
    assert max_abs(out.cpu().numpy(), ref_o) <= 1e-4 and max_abs(lse.cpu().numpy(), ref_l) <= 1e-4
    assert bool((plan.workspace == 77).all())


@pytest.mark.parametrize("shape", [(4, 1, 4 * 256, 4, 4, 64, wl.FULL), (8, 3, 16 * 257, 4, 1, 128, wl.ZIGZAG_CAUSAL)], ids=["d64", "d128_ragged"])
def test_fp32_static_calls_overlap(tb, shape):
    """fp32 with the merge folded in needs no workspace: static calls of it leave the library's array alone and may run on
    several streams at once, and they give the bits of the call whose shares go through a workspace."""
    n, rank, S, Hq, Hkv, d, mask = shape
    s = tb.tasp_schedule(n, rank)
    w = [wl.Workload("static_overlap", n, rank, S, Hq, Hkv, d, "fp32", mask, seed=wl.BASE_SEED + 8900 + i) for i in range(2)]
    x = [[t.cuda() for t in wl.make_qkv(i)] for i in w]
    ref = [[t.clone() for t in tb.tasp_chunk_attn(*i, s, mask, fuse_merge=True)] for i in x]
    assert tb.ChunkAttnPlan(s, *x[0], mask, fuse_merge=True).profile().other_launches == 1       # shares are dealt
    got = [[torch.empty_like(i[0]), torch.empty(i[0].shape[:-1], device="cuda")] for i in x]
    streams = [torch.cuda.Stream() for _ in x]
    torch.cuda.synchronize()
    for _ in range(20):
        for i in range(2):
            with torch.cuda.stream(streams[i]):
                tb.tasp_chunk_attn_static(*x[i], *got[i], s, mask, fuse_merge=True)
        torch.cuda.synchronize()
        for i in range(2):
            assert torch.equal(got[i][0], ref[i][0]) and torch.equal(got[i][1], ref[i][1])


@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
@pytest.mark.parametrize("heads", [(4, 4, 64), (8, 2, 128)], ids=["4x64", "8/2x128"])
def test_a_row_of_nan_scores_stays_nan(tb, dtype, heads):
    """NaN in a query row makes its output NaN, also where the pairs of several shares are added up; other rows
    are what they are without it, but for the rounding behind their running maximum, which 32 rows raise together."""
    Hq, Hkv, d = heads
    w = wl.Workload("nan_row", 4, 1, 4096, Hq, Hkv, d, dtype, wl.FULL, seed=wl.BASE_SEED + 8450 + d)
    q, k, v = (t.cuda() for t in wl.make_qkv(w))
    bad = q.clone()
    bad[5, 1] = float("nan")
    for fuse_steps in (False, True):
        plan = tb.ChunkAttnPlan(tb.tasp_schedule(4, 1), q, k, v, w.mask_mode, fuse_merge=True, fuse_steps=fuse_steps)
        clean = [t.clone() for t in plan.run()]
        prof = plan.profile()
        assert prof.attn_launches == 1 and prof.other_launches >= 1          # joined steps, and a launch that adds shares up
        out, lse = tb.tasp_chunk_attn(bad, k, v, plan.schedule, w.mask_mode, fuse_merge=True, fuse_steps=fuse_steps)
        assert bool(out[5, 1].isnan().all())
        out[5, 1], lse[5, 1] = clean[0][5, 1], clean[1][5, 1]
        assert float((out.float() - clean[0].float()).abs().max()) <= (2e-2 if dtype == "bf16" else 1e-5)
        assert float((lse - clean[1]).abs().max()) <= 1e-5


BWD_FP32 = [
    # name, N, rank, S, Hq, Hkv, d, mask
    ("one_row_g3", 4, 3, 4, 3, 1, 128, wl.FULL),
    ("tile_minus_1", 4, 1, 4 * 63, 1, 1, 128, wl.FULL),
    ("tile", 8, 2, 16 * 64, 2, 2, 64, wl.ZIGZAG_CAUSAL),
    ("tile_plus_1_g5", 8, 7, 16 * 13, 5, 1, 128, wl.ZIGZAG_CAUSAL),          # 13 x 5 = 65 pairs
    ("shares", 12, 4, 24 * 101, 6, 3, 64, wl.ZIGZAG_CAUSAL),                 # keys no multiple of anything
    ("not_joined", 4, 0, 8 * 2056, 1, 1, 64, wl.ZIGZAG_CAUSAL),              # 4 112 local rows: step by step
]


@pytest.mark.parametrize("case", BWD_FP32, ids=[c[0] for c in BWD_FP32])
def test_fp32_backward_every_element(tb, case):
    name, n, rank, S, Hq, Hkv, d, mode = case
    w = wl.Workload(name, n, rank, S, Hq, Hkv, d, "fp32", mode, seed=wl.BASE_SEED + 8500 + S)
    q, k, v = wl.make_qkv(w)
    do = wl.make_dout(w)
    s = tb.tasp_schedule(n, rank)
    qd, kd, vd, dod = q.cuda(), k.cuda(), v.cuda(), do.cuda()
    out, lse = tb.tasp_chunk_attn(qd, kd, vd, s, mode)
    ref = oracle_grads(w, q, k, v, do)
    plan = tb.ChunkAttnBwdPlan(s, qd, kd, vd, out, lse, dod, mode)
    least = tb.lib.tasp_chunk_attn_bwd_workspace_bytes(s.handle, C.byref(plan.args))
    for nbytes in {plan.args.workspace_bytes, least}:
        plan.args.workspace_bytes = nbytes
        for t in (plan.dq, plan.dk, plan.dv):
            t.fill_(float("nan"))
        got = plan.run()
        torch.cuda.synchronize()
        for nm, g, r in zip(("dq", "dk", "dv"), got, ref):
            err = float(np.abs(g.cpu().numpy().astype(np.float64) - r).max())
            assert err <= 1e-4 * max(1.0, float(np.abs(r).max())), (name, nm, nbytes, err)


@pytest.mark.parametrize("shape", [(16, 7, 16384, 12, 12, 64), (4, 0, 20480, 2, 1, 128)], ids=["16k_d64", "20k_d128"])
def test_fp32_dq_error_does_not_grow_with_the_keys(tb, shape):
    """dq of many keys against 64 bits, from out and lse that are exact but for their last rounding.  Bound: 7.5e-7, what
    sums over the lanes of a wavefront reach on these inputs (d = 64; 1.4e-6 for d = 128); one chain of additions per
    share of the keys has 1.0e-6 to 1.05e-6, the two levels of sums 4.7e-7."""
    n, rank, S, Hq, Hkv, d = shape
    w = wl.Workload("dq_error", n, rank, S, Hq, Hkv, d, "fp32", wl.FULL, seed=wl.BASE_SEED + 8600 + d)
    q, k, v = (t.cuda() for t in wl.make_qkv(w))
    do = wl.make_dout(w).cuda()
    out, lse = torch.empty_like(q), torch.empty(q.shape[:-1], device="cuda")
    ref = torch.empty(q.shape, dtype=torch.float64, device="cuda")
    for h in range(Hq):
        kh, vh, g = k[:, h * Hkv // Hq].double(), v[:, h * Hkv // Hq].double(), do[:, h].double()
        s = q[:, h].double() @ kh.t() / d ** 0.5
        l = torch.logsumexp(s, 1, keepdim=True)
        p = torch.exp(s - l)
        o = p @ vh
        out[:, h], lse[:, h] = o, l[:, 0]
        ref[:, h] = (p * (g @ vh.t() - (g * o).sum(1, keepdim=True))) @ kh / d ** 0.5
    dq = tb.tasp_chunk_attn_bwd(q, k, v, out, lse, do, tb.tasp_schedule(n, rank), w.mask_mode)[0]
    assert float((dq.double() - ref).norm() / ref.norm()) <= 7.5e-7


BWD_BF16 = [
    # name, N, rank, S, Hq, Hkv, d, mask, fuse_steps
    ("one_row", 4, 2, 4, 2, 1, 128, wl.FULL, False),
    ("tile_minus_1", 4, 1, 4 * 127, 2, 1, 64, wl.FULL, True),
    ("shares_and_heads", 8, 3, 16 * 129, 4, 1, 128, wl.ZIGZAG_CAUSAL, False),       # dq keys and dk/dv query tiles dealt out
    ("shares_and_heads_listed", 16, 9, 32 * 65, 4, 2, 64, wl.ZIGZAG_CAUSAL, True),  # the lists of the steps in device memory
    ("joined_edge", 4, 0, 4 * 4096, 2, 1, 64, wl.FULL, False),                      # the most local rows whose steps are joined
    ("not_joined", 4, 3, 4 * 4097, 2, 1, 64, wl.FULL, False),
]


@pytest.mark.parametrize("case", BWD_BF16, ids=[c[0] for c in BWD_BF16])
def test_bf16_backward_every_element(tb, case):
    name, n, rank, S, Hq, Hkv, d, mode, fuse_steps = case
    w = wl.Workload(name, n, rank, S, Hq, Hkv, d, "bf16", mode, seed=wl.BASE_SEED + 8700 + S)
    q, k, v = wl.make_qkv(w)
    do = wl.make_dout(w)
    s = tb.tasp_schedule(n, rank)
    qd, kd, vd, dod = q.cuda(), k.cuda(), v.cuda(), do.cuda()
    out, lse = tb.tasp_chunk_attn(qd, kd, vd, s, mode)
    keep = list(range(w.L)) if w.L <= 512 else wl.sample_rows(w, 64)          # rows with an upstream gradient
    sparse = torch.zeros_like(do)
    sparse[keep] = do[keep]
    ref = oracle_grads(w, q, k, v, do, rows=keep, out=out.cpu())
    plan = tb.ChunkAttnBwdPlan(s, qd, kd, vd, out, lse, sparse.cuda(), mode, fuse_steps=fuse_steps)
    least = tb.lib.tasp_chunk_attn_bwd_workspace_bytes(s.handle, C.byref(plan.args))
    for nbytes in {plan.args.workspace_bytes, least}:
        plan.args.workspace_bytes = nbytes
        for t in (plan.dq, plan.dk, plan.dv):
            t.fill_(float("nan"))
        dq, dk, dv = plan.run()
        torch.cuda.synchronize()
        assert bool(torch.isfinite(dq.float()).all())
        for nm, g, r in zip(("dq", "dk", "dv"), (dq[keep], dk, dv), ref):
            err = np.abs(g.float().cpu().numpy().astype(np.float64) - r)
            worst = float((err / (np.abs(r) / 128 + np.abs(r).max() / 256 + 1e-30)).max())
            assert worst <= 1.0, (name, nm, nbytes, worst)


NOT_FINITE = [
    # name, N, rank, S, Hq, Hkv, d
    ("shares", 8, 3, 16 * 75, 4, 2, 64),
    ("tile_edges", 4, 1, 8 * 97, 3, 1, 128),
    ("many_ranks", 32, 17, 64 * 33, 2, 1, 64),
]


@pytest.mark.parametrize("case", NOT_FINITE, ids=[c[0] for c in NOT_FINITE])
def test_fp32_what_is_not_seen_has_no_part(tb, case):
    """Infinities and NaN reach only the rows and keys of the pairs that the mask leaves."""
    from oracle import schedule as sch
    name, n, rank, S, Hq, Hkv, d = case
    w = wl.Workload(name, n, rank, S, Hq, Hkv, d, "fp32", wl.ZIGZAG_CAUSAL, seed=wl.BASE_SEED + 9100 + S)
    q, k, v = wl.make_qkv(w)
    do = wl.make_dout(w)
    pos = np.asarray(sch.local_positions(n, rank, S, wl.ZIGZAG_CAUSAL))
    s = tb.tasp_schedule(n, rank)
    half = S // (2 * n)
    t1, t2 = int(pos[half + half // 3]), int(pos[half // 2])                 # in a diagonal tile of each query block
    kp, vp = k.clone(), v.clone()
    vp[t1], vp[t2, :, 1] = float("nan"), float("inf")
    kp[S - 1, :, 0] = float("nan")                                           # seen by the last row of all only, if by one here
    ref_o, ref_l = oracle_rows(w, q, k, v, range(w.L))
    seen_v = pos >= min(t1, t2)
    seen_k = pos >= S - 1
    for fuse in (False, True):
        out, lse = tb.tasp_chunk_attn(q.cuda(), kp.cuda(), vp.cuda(), s, w.mask_mode, fuse_merge=fuse)
        out, lse = out.cpu().numpy(), lse.cpu().numpy()
        assert max_abs(out[~seen_v], ref_o[~seen_v]) <= 1e-4, (name, fuse)
        assert max_abs(lse[~seen_k], ref_l[~seen_k]) <= 1e-4, (name, fuse)
        assert not np.isfinite(out[seen_v]).all(axis=-1).any()
        assert np.isposinf(out[(pos >= t2) & (pos < t1)][..., 1]).all()

    # backward: the same keys, an upstream gradient that overflowed, and a row that saw no key
    out, lse = tb.tasp_chunk_attn(q.cuda(), k.cuda(), v.cuda(), s, w.mask_mode)
    r_inf, r_dead = half // 4, half + half // 2
    clean = do.clone()
    clean[[r_inf, r_dead]] = 0.0
    ref = oracle_grads(w, q, k, v, clean)
    do[r_inf] = float("inf")
    out[r_dead], lse[r_dead] = float("nan"), float("-inf")
    kp[t2] = float("nan")
    dq, dk, dv = (g.cpu().numpy() for g in tb.tasp_chunk_attn_bwd(q.cuda(), kp.cuda(), vp.cuda(), out, lse, do.cuda(), s, w.mask_mode))
    keys = np.arange(S)
    rows = (pos < min(t1, t2)) & (np.arange(w.L) != r_inf)
    rows[r_dead] = True
    cols = (keys > pos[r_inf]) & ~np.isin(keys, (t1, t2, S - 1))
    for nm, g, r, at in (("dq", dq, ref[0], rows), ("dk", dk, ref[1], cols), ("dv", dv, ref[2], cols)):
        err = float(np.abs(g[at].astype(np.float64) - r[at]).max())
        assert err <= 1e-4 * max(1.0, float(np.abs(r).max())), (name, nm, err)
    assert not np.isfinite(dv[: pos[r_inf] + 1]).any()


@pytest.mark.parametrize("heads", [(2, 2, 64), (6, 2, 128)], ids=["2x64", "6/2x128"])
def test_fp32_one_nan_at_any_place_of_a_tile(tb, heads):
    """A NaN in one V row, then in one upstream gradient, at places all over the tiles (diagonal or not, either half of
    one): what does not see it is what it is without it, what sees it is NaN."""
    from oracle import schedule as sch
    Hq, Hkv, d = heads
    w = wl.Workload("nan_place", 4, 2, 8 * 150, Hq, Hkv, d, "fp32", wl.ZIGZAG_CAUSAL, seed=wl.BASE_SEED + 9400 + d)
    q, k, v = (t.cuda() for t in wl.make_qkv(w))
    do = wl.make_dout(w).cuda()
    s = tb.tasp_schedule(w.n_ranks, w.rank)
    pos = torch.as_tensor(np.asarray(sch.local_positions(w.n_ranks, w.rank, w.S, w.mask_mode))).cuda()
    out, lse = (t.clone() for t in tb.tasp_chunk_attn(q, k, v, s, w.mask_mode))
    dq, dk, dv = (t.clone() for t in tb.tasp_chunk_attn_bwd(q, k, v, out, lse, do, s, w.mask_mode))
    keys = torch.arange(w.S, device="cuda")
    for row in range(3, w.L, 29):
        t = int(pos[row])
        bad = v.clone()
        bad[t] = float("nan")
        o, l = tb.tasp_chunk_attn(q, k, bad, s, w.mask_mode)
        gq = tb.tasp_chunk_attn_bwd(q, k, bad, out, lse, do, s, w.mask_mode)[0]
        sees = pos >= t
        assert bool(o[sees].isnan().all()) and bool(gq[sees].isnan().all()), t
        assert float((o[~sees] - out[~sees]).abs().max()) <= 1e-5 and float((gq[~sees] - dq[~sees]).abs().max()) <= 1e-4, t
        assert float((l - lse).abs().max()) <= 1e-5, t
        bad = do.clone()
        bad[row] = float("nan")
        _, gk, gv = tb.tasp_chunk_attn_bwd(q, k, v, out, lse, bad, s, w.mask_mode)
        seen = keys <= t
        assert bool(gk[seen].isnan().all()) and bool(gv[seen].isnan().all()), t
        assert float((gk[~seen] - dk[~seen]).abs().max()) <= 1e-4 and float((gv[~seen] - dv[~seen]).abs().max()) <= 1e-4, t


def test_fp32_values_that_are_not_finite_cost_little(tb):
    """Nearly all rows that see a NaN or infinity take the ordinary way: a call with one in a key or row that every other one
    meets, and one with nothing but NaN, take less than six times a clean one (each row by itself: hundreds of times)."""
    w = wl.Workload("not_finite_time", 8, 3, 16384, 4, 4, 64, "fp32", wl.ZIGZAG_CAUSAL, seed=wl.BASE_SEED + 9500)
    q, k, v = (t.cuda() for t in wl.make_qkv(w))
    do = wl.make_dout(w).cuda()
    s = tb.tasp_schedule(w.n_ranks, w.rank)
    out, lse = (t.clone() for t in tb.tasp_chunk_attn(q, k, v, s, w.mask_mode))

    def best_ms(f):
        times = []
        for _ in range(4):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            f()
            b.record()
            torch.cuda.synchronize()
            times.append(a.elapsed_time(b))
        return min(times)

    def times(q, k, v, out, lse, do):
        fwd = tb.ChunkAttnPlan(s, q, k, v, w.mask_mode)
        bwd = tb.ChunkAttnBwdPlan(s, q, k, v, out, lse, do, w.mask_mode)
        return best_ms(fwd.run), best_ms(bwd.run)

    clean = times(q, k, v, out, lse, do)
    first = v.clone()
    first[0] = float("inf")
    dead_o, dead_l, dead_q = out.clone(), lse.clone(), q.clone()
    dead_q[-1], dead_o[-1], dead_l[-1] = float("nan"), float("nan"), float("-inf")           # the forward's result for a NaN row
    every = [torch.full_like(t, float("nan")) for t in (q, k, v, out, lse, do)]
    for name, args in (("first key", (q, k, first, out, lse, do)), ("last row", (dead_q, k, v, dead_o, dead_l, do)), ("all", every)):
        got = times(*args)
        print(name, clean, got, flush=True)
        assert got[0] <= 6 * clean[0] and got[1] <= 6 * clean[1], (name, clean, got)
