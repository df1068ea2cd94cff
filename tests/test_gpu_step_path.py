"""Forward calls that run step by step (more than 4 096 local rows, all steps not asked for in one launch; fp32: four ranks with up to 8 192
rows), with half-chunks that no tile divides: the partial pair of a step written and merged by the merge kernel, and folded in by the attention kernel.
Sampled rows against the oracle; the number of launches shows which path ran."""
import numpy as np
import pytest
import torch

from paper_2509_26541_amd import workloads as wl
from tests.helpers import max_abs, oracle_rows

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def tb():
    assert torch.cuda.is_available(), "GPU tests need an MI355X"
    from paper_2509_26541_amd import binding
    return binding


CASES = [
    # name, N, rank, S, Hq, Hkv, d, dtype, mask, batch
    ("d128_grouped", 4, 1, 8 * 2051, 4, 2, 128, "bf16", wl.ZIGZAG_CAUSAL, 1),
    ("d128_full", 4, 3, 4 * 4099, 3, 1, 128, "bf16", wl.FULL, 1),
    ("d64_twelve_wavefronts", 4, 2, 8 * 2051, 2, 1, 64, "bf16", wl.ZIGZAG_CAUSAL, 1),     # 2 051 rows fill 384-row tiles as well as 256-row ones
    ("d64_eight_wavefronts", 4, 0, 8 * 2310, 2, 2, 64, "bf16", wl.ZIGZAG_CAUSAL, 1),      # 2 310 rows do not
    ("d128_batch", 4, 2, 8 * 2049, 2, 1, 128, "bf16", wl.ZIGZAG_CAUSAL, 2),
    ("fp32_d64", 4, 1, 8 * 2051, 2, 1, 64, "fp32", wl.ZIGZAG_CAUSAL, 1),
    ("fp32_d128_full", 4, 2, 4 * 4097, 1, 1, 128, "fp32", wl.FULL, 1),
]


@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_step_by_step(tb, case):
    name, n, rank, S, Hq, Hkv, d, dtype, mode, B = case
    ws = [wl.Workload(name, n, rank, S, Hq, Hkv, d, dtype, mode, seed=wl.BASE_SEED + 9600 + S + b) for b in range(B)]
    qkv = [wl.make_qkv(w) for w in ws]
    q, k, v = ((torch.stack([x[i] for x in qkv]) if B > 1 else qkv[0][i]).cuda() for i in range(3))
    s = tb.tasp_schedule(n, rank)
    w = ws[0]
    half = w.L // 2
    rows = sorted(set(wl.sample_rows(w, 48)) | {0, 255, 256, 383, 384, half - 1, half, half + 255, half + 256, w.L - 1})
    refs = [oracle_rows(ws[b], *qkv[b], rows) for b in range(B)]
    tol_o, tol_l = (2e-2, 1e-3) if dtype == "bf16" else (1e-4, 1e-4)

    def check(out, lse):
        for b in range(B):
            o, l = (out[b], lse[b]) if B > 1 else (out, lse)
            assert bool(torch.isfinite(l).all()) and bool(torch.isfinite(o.float()).all())
            eo, el = max_abs(o[rows].float().cpu().numpy(), refs[b][0]), max_abs(l[rows].cpu().numpy(), refs[b][1])
            assert eo <= tol_o and el <= tol_l, (name, b, eo, el)

    for fuse in (False, True):
        plan = tb.ChunkAttnPlan(s, q, k, v, mode, fuse_merge=fuse)
        prof = plan.profile()
        assert prof.attn_launches == n and (prof.merge_launches > 0) == (not fuse), (name, fuse, prof.attn_launches, prof.merge_launches)
        plan.out.fill_(float("nan"))
        plan.lse.fill_(float("nan"))
        out, lse = plan.run()
        torch.cuda.synchronize()
        check(out, lse)
    # all steps in one launch (of the kernel for few query tiles), against the oracle and against the pairs of the steps
    # merged at the end
    one = tb.ChunkAttnPlan(s, q, k, v, mode, fuse_steps=True)
    assert one.profile().attn_launches == 1
    out, lse = one.run()
    torch.cuda.synchronize()
    check(out, lse)
    parts = [tb.tasp_step_attn(q, k, v, s, mode, i) for i in range(n)]
    flat = [(o.reshape(-1, Hq, d), l.reshape(-1, Hq)) for o, l in parts]
    o_m, l_m = tb.tasp_lse_merge_many([o for o, _ in flat], [l for _, l in flat])
    torch.cuda.synchronize()
    check(o_m.reshape(out.shape), l_m.reshape(lse.shape))
    assert float((o_m.reshape(out.shape) - out.float()).abs().max()) <= 2 * tol_o and float((l_m.reshape(lse.shape) - lse).abs().max()) <= 2 * tol_l


def test_persistent_workgroups_against_the_steps(tb):
    """All steps in one launch of the large kernel at d = 64 with eight wavefronts, whose workgroups are persistent, against the
    pairs of the same kernel's single steps merged at the end (every row), and against the oracle (sampled rows of one sequence)."""
    B, n, rank, S, H, d = 6, 4, 0, 8 * 2310, 8, 64
    w = wl.Workload("persistent", n, rank, S, H, H, d, "bf16", wl.ZIGZAG_CAUSAL, seed=wl.BASE_SEED + 9700)
    q, k, v = (torch.stack([t] * B).cuda() for t in wl.make_qkv(w))
    for b in range(1, B):                             # other values of the same distribution
        for t in (q, k, v):
            t[b] = t[0].roll(b * 977, dims=0)
    s = tb.tasp_schedule(n, rank)
    one = tb.ChunkAttnPlan(s, q, k, v, w.mask_mode, fuse_steps=True)
    prof = one.profile()
    assert prof.attn_launches == 1 and prof.other_launches == 0        # no shares: not the kernel for few query tiles
    out, lse = one.run()
    parts = [tb.tasp_step_attn(q, k, v, s, w.mask_mode, i) for i in range(n)]
    o_m, l_m = tb.tasp_lse_merge_many([o.reshape(-1, H, d) for o, _ in parts], [l.reshape(-1, H) for _, l in parts])
    torch.cuda.synchronize()
    assert float((o_m.reshape(out.shape) - out.float()).abs().max()) <= 4e-2 and float((l_m.reshape(lse.shape) - lse).abs().max()) <= 2e-3
    rows = wl.sample_rows(w, 24)
    ref_o, ref_l = oracle_rows(w, q[0].cpu(), k[0].cpu(), v[0].cpu(), rows)
    assert max_abs(out[0][rows].float().cpu().numpy(), ref_o) <= 2e-2 and max_abs(lse[0][rows].cpu().numpy(), ref_l) <= 1e-3


# name, S, Hq, Hkv, d, k_scale, share of outlier keys; eight ranks, causal, more than 4 096 local rows
PRECISION = [
    ("d128_k2", 49152, 4, 4, 128, 2.0, 0.0),
    ("d64_k2", 49152, 4, 4, 64, 2.0, 0.0),
    ("d128_grouped_outliers", 65536, 4, 1, 128, 1.0, 0.01),
]


@pytest.mark.parametrize("case", PRECISION, ids=[c[0] for c in PRECISION])
def test_a_call_is_as_close_to_64_bits_as_its_steps(tb, case):
    """A bf16 call that does not ask for joined steps, against 64 bits, and the pairs of its single steps merged in fp32 and rounded once: a
    joined launch has one division for all keys, where each step has its own, and was 2 to 3 % further off on these inputs.  Running
    outputs are added up in another order than the pairs are: half a per cent for that."""
    name, S, Hq, Hkv, d, k_scale, outliers = case
    n, rank = 8, 3
    w = wl.Workload("precision_" + name, n, rank, S, Hq, Hkv, d, "bf16", wl.ZIGZAG_CAUSAL, k_scale=k_scale, outlier_frac=outliers, seed=wl.BASE_SEED + 9800 + d)
    q, k, v = (x.cuda() for x in wl.make_qkv(w))
    s = tb.tasp_schedule(n, rank)
    parts = [tb.tasp_step_attn(q, k, v, s, w.mask_mode, i) for i in range(n)]
    steps = tb.tasp_lse_merge_many([o for o, _ in parts], [l for _, l in parts])[0].to(torch.bfloat16)
    half = S // (2 * n)
    rows = torch.arange(0, w.L, 4, device="cuda")
    pos = torch.where(rows < half, rank * half + rows, S - (rank + 1) * half + rows - half)
    exact = torch.empty((len(rows), Hq, d), dtype=torch.float64, device="cuda")
    for h in range(Hq):
        kh, vh = k[:, h * Hkv // Hq].double(), v[:, h * Hkv // Hq].double()
        for i in range(0, len(rows), 512):
            x = q[rows[i:i + 512], h].double() @ kh.T / d ** 0.5
            x.masked_fill_(torch.arange(S, device="cuda")[None] > pos[i:i + 512, None], float("-inf"))
            exact[i:i + 512, h] = torch.softmax(x, -1) @ vh
    error = lambda o: ((o[rows].double() - exact).norm() / exact.norm()).item()
    bound = 1.005 * error(steps)
    for fuse_merge in (False, True):
        got = error(tb.tasp_chunk_attn(q, k, v, s, w.mask_mode, fuse_merge=fuse_merge)[0])
        assert got <= bound, (name, fuse_merge, got, bound)
