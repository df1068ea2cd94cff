"""fp32 forward on inputs of a wide range: between the columns of Q, K and V, between rows next to each other and between runs of
rows.  Every product of two floats has the accuracy of fp32 whatever stands beside it, so the bounds are those of fp32 sums:
2e-6 for every single column of the output (about 4 times what these sizes show), 1e-5 for the log-sum-exp."""
import math

import pytest
import torch

from paper_2509_26541_amd import workloads as wl
from tests.test_gpu_fp32_halves import inputs, positions, reference, rel

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def tb():
    assert torch.cuda.is_available(), "GPU tests need an MI355X"
    from paper_2509_26541_amd import binding
    return binding


N, RANK, S, H = 4, 1, 8 * 300, 2
SHAPES = [(64, wl.FULL), (64, wl.ZIGZAG_CAUSAL), (128, wl.FULL), (128, wl.ZIGZAG_CAUSAL)]
IDS = ["%d-%s" % (d, "full" if m == wl.FULL else "zigzag") for d, m in SHAPES]


def check(tb, q, k, v, mask, what, floor=0.0):
    """Relative error of every output column and of the lse; `floor`: absolute error of an element that is let pass."""
    out, lse = tb.tasp_chunk_attn(q, k, v, tb.tasp_schedule(N, RANK), mask, fuse_merge=True)
    ref_o, ref_l = reference(q, k, v, positions(N, RANK, S, mask))
    err, size = (out.double() - ref_o).norm(dim=0), ref_o.norm(dim=0)
    worst = float(((err - floor * len(out) ** 0.5).clamp(min=0) / size).max())
    assert worst <= 2e-6 and float((lse.double() - ref_l).abs().max()) <= 1e-5, (what, worst, float((lse.double() - ref_l).abs().max()))


@pytest.mark.parametrize("d,mask", SHAPES, ids=IDS)
def test_a_large_column_of_v(tb, d, mask):
    for b in (20, 24, 30, 41, 100, -30, -100):
        q, k, v = inputs(N, S, H, H, d, 21)
        v[:, :, 5] *= 2.0 ** b
        check(tb, q, k, v, mask, b)


@pytest.mark.parametrize("d,mask", SHAPES, ids=IDS)
def test_columns_of_q_against_k(tb, d, mask):
    for r in (20, 30, 40, 60, -40, -60):
        q, k, v = inputs(N, S, H, H, d, 22)
        q[:, :, 3] *= 2.0 ** r
        k[:, :, 3] *= 2.0 ** -r
        check(tb, q, k, v, mask, r)


@pytest.mark.parametrize("d,mask", SHAPES, ids=IDS)
def test_large_rows_of_v_with_small_weight(tb, d, mask):
    """Every other run of 64 keys 2^r larger, its weights 2^-(r + 10)."""
    run = (torch.arange(S, device="cuda") // 64) % 2 == 1
    for r in (20, 24, 30, 60):
        q, k, v = inputs(N, S, H, H, d, 23)
        q[:, :, 0] = 1.0
        k[run, :, 0] = -(r + 10) * math.log(2.0) * d ** 0.5
        v[run] *= 2.0 ** r
        check(tb, q, k, v, mask, r)


@pytest.mark.parametrize("d,mask", SHAPES, ids=IDS)
def test_huge_rows_of_v_without_weight(tb, d, mask):
    for b in (90, 104, 120):
        q, k, v = inputs(N, S, H, H, d, 24)
        q[:, :, 0] = q[:, :, 0].abs() + 1.0
        k[32:64, :, 0] = -3000.0
        v[32:64] *= 2.0 ** b
        check(tb, q, k, v, mask, b)


@pytest.mark.parametrize("d,mask", SHAPES, ids=IDS)
def test_tiny_values(tb, d, mask):
    """V down to the smallest normal floats; what is below 2^-126 in the output has its spacing of 2^-149.  K and Q that small give
    scores of zero."""
    for b in (-98, -100, -110, -120, -124):
        q, k, v = inputs(N, S, H, H, d, 25)
        check(tb, q, k, v * 2.0 ** b, mask, ("v", b), floor=2.0 ** -149)
    v[:, :, 7] *= 2.0 ** -124
    check(tb, q, k, v, mask, "a column of v", floor=2.0 ** -149)
    q, k, v = inputs(N, S, H, H, d, 25)
    v = v.abs()                              # (the mean of them all: of both signs it would be small against the rounding of the sums)
    check(tb, q, k * 2.0 ** -110, v, mask, "k")
    check(tb, q * 2.0 ** -118, k, v, mask, "q")


@pytest.mark.parametrize("d,mask", SHAPES, ids=IDS)
def test_rows_of_different_size_side_by_side(tb, d, mask):
    """One row in four nearly zero; one in 64 very large."""
    at = torch.arange(S, device="cuda")
    q, k, v = inputs(N, S, H, H, d, 26)
    k[at % 4 == 1] *= 1e-9
    v[at % 4 == 1] *= 1e-9
    check(tb, q, k, v, mask, "one in four nearly zero")
    q, k, v = inputs(N, S, H, H, d, 27)
    v[at % 64 == 5] *= 2.0 ** 20
    check(tb, q, k, v, mask, "one in 64 very large")


@pytest.mark.parametrize("d,mask", SHAPES, ids=IDS)
def test_gradients_behind_such_a_forward(tb, d, mask):
    """The backward pass takes out and lse from the forward: with a column of Q 2^30 times as large, K's as much smaller, the
    probabilities still add up to one.  Bound: fp32 sums, 1e-5 of every tensor."""
    n, rank, size = 4, 1, 8 * 100
    q, k, v = inputs(n, size, 1, 1, d, 34)
    q[:, :, 3] *= 2.0 ** 30
    k[:, :, 3] *= 2.0 ** -30
    do = inputs(n, size, 1, 1, d, 35)[0]
    s = tb.tasp_schedule(n, rank)
    out, lse = tb.tasp_chunk_attn(q, k, v, s, mask, fuse_merge=True)
    got = tb.tasp_chunk_attn_bwd(q, k, v, out, lse, do, s, mask)
    x, y, z, g = q[:, 0].double(), k[:, 0].double(), v[:, 0].double(), do[:, 0].double()
    pos = positions(n, rank, size, mask)
    p = torch.softmax((x @ y.T / d ** 0.5).masked_fill(torch.arange(size, device="cuda")[None, :] > pos[:, None], -math.inf), 1)
    ds = p * (g @ z.T - (g * (p @ z)).sum(1, keepdim=True)) / d ** 0.5
    for name, a, b in zip(("dq", "dk", "dv"), got, (ds @ y, ds.T @ x, p.T @ g)):
        err, ref = (a[:, 0].double() - b).norm(dim=0), b.norm(dim=0)
        assert float((err / ref).max()) <= 1e-5, (name, float((err / ref).max()))


@pytest.mark.parametrize("d,mask", SHAPES, ids=IDS)
def test_scores_that_overflow_downwards(tb, d, mask):
    """Keys whose scores are below the smallest float have no weight, whichever sign the smaller products of their pieces have."""
    for big, far in ((1e14, -1.2345678e30), (1e14, -1.2378901e30), (3e30, -7.654321e24), (1e-3, -2.9e31)):
        q, k, v = inputs(N, S, H, H, d, 33)
        q[:, :, 0] = big * (1.0 + 0.1 * torch.rand(q.shape[:2], device="cuda"))
        k[:, :, 0] /= big
        gone = torch.tensor([0, 5, 6, 7, 37, 700, 1500, S - 1], device="cuda")
        k[gone, :, 0] = far
        kf = k.clone()
        kf[gone, :, 0] = -1e6 / big
        out, lse = tb.tasp_chunk_attn(q, k, v, tb.tasp_schedule(N, RANK), mask, fuse_merge=True)
        ref_o, ref_l = reference(q, kf, v, positions(N, RANK, S, mask))
        assert rel(out, ref_o) <= 2e-6 and float((lse.double() - ref_l).abs().max()) <= 1e-5, (big, far)


def long_error(tb, S, n, d, fuse_steps):
    """Errors of 512 rows of one head, no mask, over the output's root mean square."""
    q, k, v = inputs(n, S, 1, 1, d, 29)
    out, _ = tb.tasp_chunk_attn(q, k, v, tb.tasp_schedule(n, 3), wl.FULL, fuse_merge=True, fuse_steps=fuse_steps)
    pick = torch.linspace(0, S // n - 1, 512).long().cuda()
    ref = torch.cat([reference(q[rows], k, v, torch.full((64,), S, device="cuda"))[0] for rows in pick.split(64)])
    return (out[pick].double() - ref) / ref.pow(2).mean().sqrt()


@pytest.mark.parametrize("fuse_steps", [False, True], ids=["steps", "joined"])
@pytest.mark.parametrize("d", [64, 128])
def test_sums_are_not_biased(tb, d, fuse_steps):
    """The matrix pipe cuts sums off downwards; over many keys that may not add up.  65 536 errors of 8e-7 have a mean within 1e-8
    (three deviations); ten times that for the columns' and rows' common parts."""
    err = long_error(tb, 131072, 16, d, fuse_steps)
    assert abs(float(err.mean())) <= 1e-7, float(err.mean())


@pytest.mark.parametrize("fuse_steps", [False, True], ids=["steps", "joined"])
@pytest.mark.parametrize("d", [64, 128])
def test_error_does_not_grow_with_the_keys(tb, d, fuse_steps):
    """524 288 keys.  fp32 matrix instructions with two sets of sums show 9.7e-7 (joined) and 8.1e-7 (steps)."""
    err = long_error(tb, 524288, 16, d, fuse_steps)
    assert float(err.pow(2).mean().sqrt()) <= 9e-7, float(err.pow(2).mean().sqrt())


@pytest.mark.parametrize("fuse_merge", [False, True], ids=["merge_kernel", "folded"])
@pytest.mark.parametrize("n,rank,S,mask", [(4, 2, 4 * 16385, wl.FULL), (4, 1, 8 * 8200, wl.ZIGZAG_CAUSAL), (4, 3, 4 * 40000, wl.FULL)],
                         ids=["one_more", "zigzag", "three_rounds"])
def test_steps_whose_sums_go_through_memory(tb, n, rank, S, mask, fuse_merge):
    """Steps of a few more than 512 tiles of 32 keys, by themselves and folded into the running pair; rows of Q that are
    done again at the end: with an infinity (keeps to itself), and with values beyond 2^104."""
    q, k, v = inputs(n, S, 2, 1, 128, 30)
    k[:, :, 0] *= 2.0 ** -107
    q[5, 0] = 0.0
    q[5, 0, 0] = 2.0 ** 110
    pos = positions(n, rank, S, mask)
    s = tb.tasp_schedule(n, rank)
    L = S // n
    pick = torch.cat([torch.arange(0, 40), torch.arange(L // 2 - 20, L // 2 + 20), torch.arange(L - 40, L)]).cuda()
    ref_o, ref_l = reference(q[pick], k, v, pos[pick])

    def near(out, lse, rows):
        return rel(out[pick][rows], ref_o[rows]) <= 2e-6 and float((lse[pick][rows].double() - ref_l[rows]).abs().max()) <= 1e-5

    every = torch.ones(len(pick), dtype=torch.bool, device="cuda")
    out, lse = tb.tasp_chunk_attn(q, k, v, s, mask, fuse_merge=fuse_merge)
    assert near(out, lse, every)
    if fuse_merge:
        parts = [tb.tasp_step_attn(q, k, v, s, mask, i) for i in range(n)]
        assert near(*tb.tasp_lse_merge_many([o for o, _ in parts], [l for _, l in parts]), every)
        q[L - 3, 1, 0] = float("inf")
        out, lse = tb.tasp_chunk_attn(q, k, v, s, mask, fuse_merge=True)
        assert near(out, lse, every & (pick != L - 3))
        assert bool(out[L - 3, 1].isnan().all()) and float(lse[L - 3, 1]) == -float("inf")
        assert rel(out[L - 3, 0], ref_o[pick == L - 3][0, 0]) <= 2e-6


@pytest.mark.parametrize("n,S,heads,mask", [(16, 65536, (2, 1), wl.ZIGZAG_CAUSAL), (8, 40960, (64, 8), wl.ZIGZAG_CAUSAL), (32, 131072, (8, 2), wl.FULL)],
                         ids=["short_shares", "one_run", "long_shares"])
def test_many_keys_in_one_launch(tb, n, S, heads, mask):
    """Sums that go through memory at the place of the result and of a share's pair, and shares taken in turn."""
    q, k, v = inputs(n, S, *heads, 128, 31)
    s = tb.tasp_schedule(n, 1)
    fuse_steps = S // n > 4096
    out, lse = tb.tasp_chunk_attn(q, k, v, s, mask, fuse_merge=True, fuse_steps=fuse_steps)
    pick = torch.linspace(0, S // n - 1, 48).long().cuda()
    ref_o, ref_l = reference(q[pick, :2], k[:, :1], v[:, :1], positions(n, 1, S, mask)[pick])
    assert rel(out[pick, :2], ref_o) <= 2e-6 and float((lse[pick, :2].double() - ref_l).abs().max()) <= 1e-5
    if not fuse_steps:
        out2, lse2 = torch.empty_like(out), torch.empty_like(lse)
        tb.tasp_chunk_attn_static(q, k, v, out2, lse2, s, mask, fuse_merge=True, fuse_steps=False)
        assert rel(out2[pick, :2], ref_o) <= 2e-6 and float((lse2[pick, :2].double() - ref_l).abs().max()) <= 1e-5
        assert S == 131072 or (torch.equal(out, out2) and torch.equal(lse, lse2))


@pytest.mark.parametrize("fuse_steps", [False, True], ids=["steps", "joined"])
@pytest.mark.parametrize("d,mask", SHAPES, ids=IDS)
def test_keys_left_to_the_end_among_many(tb, d, mask, fuse_steps):
    """More than 512 tiles of 32 keys to a row: values beyond 2^104 without weight and with one that counts, an infinite K that
    no row gives weight, a NaN in V in a tile that not all rows see.  Bound: the weight that counts is exp(-95 ln 2 = -66), and a dot
    product of that size has been rounded some 32 times: 66 sqrt(32) 2^-24 / sqrt(3) = 1.3e-5 for the weight, times three."""
    n, rank, size = 4, 1, 8 * 10241
    q, k, v = inputs(n, size, 1, 1, d, 32)
    pos = positions(n, rank, size, mask)
    q[:, :, 0] = 1.0
    gone = torch.tensor([0, 31, 32, 5000, 5001, 5002, 5003, 5004, 9000, 20480, 30000, size - 1], device="cuda")
    k[gone, :, 0] = -float("inf")
    v[gone] *= 2.0 ** 110
    k[[7000, 7007], :, 0] = -95 * math.log(2.0) * d ** 0.5
    v[[7000, 7007]] *= 2.0 ** 105
    kf, vf = k.clone(), v.clone()
    kf[gone, :, 0] = -1e6
    vf[gone] = 0.0
    L = size // n
    pick = torch.cat([torch.arange(0, 40), torch.arange(L // 2 - 20, L // 2 + 20), torch.arange(L - 40, L)]).cuda()
    at = int(pos[20]) if mask else size - 5              # seen by some of the rows of a tile, or by all
    v[at, 0, 3] = float("nan")
    vf[at, 0, 3] = 0.0
    ref_o, ref_l = reference(q[pick], kf, vf, pos[pick])
    out, lse = tb.tasp_chunk_attn(q, k, v, tb.tasp_schedule(n, rank), mask, fuse_merge=True, fuse_steps=fuse_steps)
    sees = pos >= at
    assert bool(out[sees, 0, 3].isnan().all()) and not bool(out[~sees].isnan().any())
    out = out[pick].clone()
    out[sees[pick], 0, 3] = ref_o[sees[pick], 0, 3].float()
    assert rel(out, ref_o) <= 4e-5 and float((lse[pick].double() - ref_l).abs().max()) <= 1e-5


@pytest.mark.parametrize("heads", [(4, 4, 64), (16, 4, 128)], ids=["4x64", "16/4x128"])
def test_the_range_costs_no_time(tb, heads):
    """Rows nearly zero or very large, and columns that are: no slower than without (a quarter is for the noise of single calls)."""
    hq, hkv, d = heads
    s = tb.tasp_schedule(8, 2)
    q, k, v = inputs(8, 8192, hq, hkv, d, 28)
    at = torch.arange(8192, device="cuda")

    def best_ms(k, v):
        plan = tb.ChunkAttnPlan(s, q, k, v, wl.ZIGZAG_CAUSAL)
        times = []
        for _ in range(8):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            plan.run()
            b.record()
            torch.cuda.synchronize()
            times.append(a.elapsed_time(b))
        return min(times)

    clean = best_ms(k, v)
    tiny, large, column = v.clone(), v.clone(), v.clone()
    tiny[at % 4 == 1] *= 1e-9
    large[at % 64 == 5] *= 2.0 ** 20
    column[:, :, 5] *= 2.0 ** 40
    for name, x in (("tiny", tiny), ("large", large), ("column", column)):
        got = best_ms(k, x)
        print(name, clean, got, flush=True)
        assert got <= 1.25 * clean + 0.005, (name, clean, got)
    # key by key: one in 64 with an infinity twice a clean call, a row of Q that is done again no longer than its first keys
    # take (it is NaN with the first of them)
    some = v.clone()
    some[at % 64 == 5] = float("inf")
    got = best_ms(k, some)
    print("one in 64 infinite", clean, got, flush=True)
    assert got <= 2 * clean, (clean, got)
    q[7] = float("inf")
    got = best_ms(k, v)
    print("a row of Q infinite", clean, got, flush=True)
    assert got <= 2 * clean, (clean, got)
