"""Joined steps of bf16 calls with few query tiles (csrc/attn_run.hip): the generated code around its hand-placed waits and which of the
shapes below take it, with how many shares (CPU), and every row against the oracle at the edges of its tiles, shares and key counts (GPU)."""
import os
import shutil

import pytest
import torch

from paper_2509_26541_amd import workloads as wl
from tests import asm_checks, test_plan
from tests.helpers import max_abs, oracle_rows


# ---------------------------------------------------------------- the generated code
def result_hazards(instructions, need=12):
    """Instructions that touch the result of a matrix instruction before it is there.  The kernel's matrix instructions are inline
    assembly, so the compiler does not place the wait states (12) between one and a vector or LDS instruction on its registers.  Along every
    path: another matrix instruction in between counts four (it is issued eight later), s_nop N counts N + 1, all else one."""
    blocks = asm_checks._blocks(instructions)
    entry = [None] * len(blocks)
    entry[0] = {}
    bad = set()

    def walk(block, age, report):
        age = dict(age)
        for line, s in block["ins"]:
            op = s.split()[0]
            matrix = op.startswith("v_mfma")
            if not matrix and report and asm_checks._regs(s[len(op):]) & set(age):
                bad.add((line, s))
            step = 4 if matrix else int(s.split()[1]) + 1 if op == "s_nop" else 1
            age = {r: a + step for r, a in age.items() if a + step < need}
            if matrix:
                age.update((r, 0) for r in asm_checks._regs(s[len(op):].split(",")[0]))
        return age

    work = [0]
    while work:
        k = work.pop()
        out = walk(blocks[k], entry[k], False)
        for n in blocks[k]["succ"]:
            old = entry[n]
            new = dict(out) if old is None else {**old, **{r: min(a, old.get(r, a)) for r, a in out.items()}}
            if new != old:
                entry[n] = new
                work.append(n)
    for k, block in enumerate(blocks):
        if entry[k] is not None:
            walk(block, entry[k], True)
    return sorted(bad)


def unbounded_offsets(instructions):
    """Direct loads whose scalar offset is not the result of a minimum (with the descriptor's records: the range check takes their
    difference, which must not be below zero)."""
    bad = []
    for i, (line, s) in enumerate(instructions):
        if not s.startswith("buffer_load_dwordx4"):
            continue
        offset = s.split(",")[2].split()[0]
        writer = next((t for _, t in reversed(instructions[:i]) if not t.endswith(":") and t.split()[1:2] == [offset + ","]), "")
        if not writer.startswith("s_min_u32"):
            bad.append((line, s, writer))
    return bad


def test_offset_checker_flags_a_planted_sum():
    load = "buffer_load_dwordx4 v1, s[0:3], s9 offen lds"
    assert unbounded_offsets([(1, "s_add_i32 s9, s8, s7"), (2, "s_min_u32 s9, s9, s6"), (3, load)]) == []
    assert [b[0] for b in unbounded_offsets([(1, "s_min_u32 s9, s8, s6"), (2, "s_add_i32 s9, s9, s7"), (3, load)])] == [3]


def test_hazard_checker_flags_a_planted_copy():
    mfma = "v_mfma_f32_32x32x16_bf16 v[0:15], v[16:19], v[20:23], v[0:15]"
    assert [b[0] for b in result_hazards([(1, mfma), (2, "v_mov_b32_e32 v30, v15")])] == [2]
    assert result_hazards([(1, mfma), (2, "s_nop 15"), (3, "v_mov_b32_e32 v30, v15")]) == []
    assert result_hazards([(1, mfma), (2, mfma)]) == []                                     # dependent matrix instructions need none
    loop = [(1, ".L:"), (2, "v_mov_b32_e32 v30, v15"), (3, "s_nop 15"), (4, mfma), (5, "s_cbranch_scc1 .L"), (6, "s_endpgm")]
    assert [b[0] for b in result_hazards(loop)] == [2]                                      # across the loop's end


@pytest.mark.skipif(shutil.which(os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")) is None, reason="hipcc not found")
def test_generated_code(tmp_path):
    """Nothing is kept in scratch and no vector register elsewhere (at d = 128 scalar ones are, in a vector register, where a tile's elements are
    masked), no register of an LDS read in flight is touched, no matrix result is read too early, every direct load has its descriptor and
    offset in scalar registers."""
    asm = asm_checks.compile_to_asm("attn_run.hip", str(tmp_path / "attn_run.s"))
    ks = {n: i for n, i in asm_checks.kernels(asm).items() if "attn_run_kernel" in n}
    assert len(ks) == 2, list(ks)
    assert all(spills == 0 and scratch == 0 for n, spills, scratch in asm_checks.spill_report(asm) if n in ks)
    for name, ins in ks.items():
        assert asm_checks.in_flight_violations(ins) == [], name
        assert result_hazards(ins) == [], name
        loads = [s for _, s in ins if s.startswith("buffer_load_dwordx4")]
        assert len(loads) >= 8 and all(s.endswith("offen lds") and ", s[" in s for s in loads), (name, loads[:2])
        assert unbounded_offsets(ins) == [], name


# ---------------------------------------------------------------- against the oracle
# name, N, rank, S, Hq, Hkv, d, mask, batch, (shares, tiles of 64 keys of the longest) of each block of rows.  Rows of a block times heads of
# a group: around 128 and 32; keys: around one and two tiles and even and odd counts of them; several shares, with keys and without.
CASES = [
    ("one_tile_of_keys", 4, 0, 8 * 8, 2, 1, 64, wl.ZIGZAG_CAUSAL, 1, ((1, 1), (1, 1))),
    ("two_tiles_of_keys_less_one", 4, 1, 4 * 31, 1, 1, 128, wl.FULL, 1, ((1, 2),)),
    ("two_tiles_and_one", 4, 3, 4 * 33, 3, 1, 64, wl.FULL, 2, ((1, 3),)),
    ("strip_and_one", 4, 2, 8 * 33, 1, 1, 128, wl.ZIGZAG_CAUSAL, 1, ((4, 1), (2, 1))),                # 33 rows: a strip with one
    ("tile_g3", 8, 5, 16 * 43, 6, 2, 128, wl.ZIGZAG_CAUSAL, 1, ((8, 1), (5, 1))),                     # 129 rows of pairs
    ("odd_tiles", 8, 3, 16 * 75, 4, 4, 64, wl.ZIGZAG_CAUSAL, 16, ((3, 6), (1, 5))),                   # last tile full, odd number of tiles in a share
    ("even_tiles", 8, 3, 16 * 83, 4, 4, 64, wl.ZIGZAG_CAUSAL, 4, ((9, 2), (3, 2))),
    ("no_shares", 8, 3, 16 * 75, 20, 20, 64, wl.ZIGZAG_CAUSAL, 20, ((1, 16), (1, 5))),
    ("no_shares_d128", 8, 6, 16 * 67, 16, 8, 128, wl.ZIGZAG_CAUSAL, 12, ((1, 11), (1, 8))),
    ("long_shares", 8, 7, 16 * 300, 1, 1, 64, wl.FULL, 40, ((2, 38),)),
    # the sum of probabilities in two levels: the first 64 tiles, and 128, are put by, with an odd and an even number left
    ("more_than_64_tiles", 8, 7, 16 * 292, 4, 4, 64, wl.FULL, 40, ((1, 73),)),
    ("more_than_64_tiles_d128", 8, 2, 16 * 296, 4, 4, 128, wl.FULL, 24, ((1, 74),)),
    ("more_than_128_tiles", 8, 7, 16 * 520, 4, 4, 64, wl.FULL, 24, ((1, 130),)),
    ("more_than_128_tiles_d128", 8, 0, 16 * 524, 8, 4, 128, wl.FULL, 12, ((1, 131),)),
]


# N, S, Hq, Hkv, d, sequences: key counts with one row in the last tile, just below and above one, two and three tiles, and shares
TAILS = [(4, 4, 2, 1, 64, 1), (4, 4, 2, 1, 128, 1), (4, 60, 2, 1, 128, 1), (4, 68, 2, 1, 64, 1), (4, 68, 2, 2, 128, 1), (4, 124, 2, 2, 64, 1), (4, 132, 2, 1, 64, 1),
         (4, 132, 2, 1, 128, 1), (4, 2404, 2, 1, 64, 1), (4, 2404, 2, 1, 128, 1), (4, 68, 2, 1, 128, 2), (4, 196, 2, 2, 64, 2)]

WHICH = r"""
int main() {
  int n, rank, S, hq, hkv, d, mask, batch;
  while (std::scanf("%d %d %d %d %d %d %d %d", &n, &rank, &S, &hq, &hkv, &d, &mask, &batch) == 8) {
    tasp_schedule_t* s = nullptr;
    if (tasp_schedule_create(n, rank, &s) != TASP_OK) return 2;
    tasp_attn_args a{};
    a.q = a.k = a.v = a.out = a.workspace = reinterpret_cast<void*>(256);
    a.lse = reinterpret_cast<float*>(256);
    a.S = S; a.Hq = hq; a.Hkv = hkv; a.d = d; a.batch = batch; a.dtype = TASP_DTYPE_BF16; a.mask_mode = mask; a.fuse_steps = 1;
    a.workspace_bytes = tasp_chunk_attn_best_workspace_bytes(s, &a);
    g = {};
    if (tasp_chunk_attn(s, &a, nullptr) != TASP_OK) return 3;
    std::printf("%d", g.tile == 1 && g.large == 0 && tasp::attn_run_takes(g.last, d));
    for (int t = 0; t < g.last.n_tasks; ++t) {
      const int keys = mask ? g.last.task[t].q_pos0 + g.last.task[t].n_q : S, ns = g.last.n_split[t];
      std::printf(" %d %d", ns, ((keys + ns - 1) / ns + 63) / 64);
    }
    std::printf("\n");
    tasp_schedule_destroy(s);
  }
  return 0;
}
"""


@pytest.mark.skipif(shutil.which(os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")) is None, reason="hipcc not found")
def test_the_shapes_below_take_this_kernel(tmp_path):
    """The planner, compiled for the host: kernel, shares and tiles of the longest share for every shape that is run on the GPU below."""
    shapes = [c[1:9] for c in CASES] + [(n, 1, S, Hq, Hkv, d, wl.FULL, B) for n, S, Hq, Hkv, d, B in TAILS]
    lines = test_plan.run_planner(tmp_path, WHICH, "\n".join(" ".join(str(int(x)) for x in c) for c in shapes)).split("\n")
    for i, c in enumerate(shapes):
        got = [int(x) for x in lines[i].split()]
        assert got[0] == 1, c
        if i < len(CASES):
            assert got[1:] == [x for t in CASES[i][9] for x in t], (CASES[i][0], got)


@pytest.mark.gpu
@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_joined_steps_all_rows(case):
    from paper_2509_26541_amd import binding as tb
    name, n, rank, S, Hq, Hkv, d, mode, B, _ = case
    ws = [wl.Workload(name, n, rank, S, Hq, Hkv, d, "bf16", mode, seed=wl.BASE_SEED + 9900 + S + b) for b in range(min(B, 2))]
    qkv = [wl.make_qkv(w) for w in ws]
    q, k, v = ((torch.stack([qkv[b % 2][i] for b in range(B)]) if B > 1 else qkv[0][i]).cuda() for i in range(3))
    plan = tb.ChunkAttnPlan(tb.tasp_schedule(n, rank), q, k, v, mode, fuse_steps=True)
    assert plan.profile().attn_launches == 1
    plan.out.fill_(float("nan"))
    plan.lse.fill_(float("nan"))
    out, lse = plan.run()
    first = out.clone()
    plan.run()
    torch.cuda.synchronize()
    assert torch.equal(first, out)
    rows = list(range(ws[0].L)) if ws[0].L <= 300 else wl.sample_rows(ws[0], 64)
    for b in range(len(ws)):
        o, l = (out[b], lse[b]) if B > 1 else (out, lse)
        ref_o, ref_l = oracle_rows(ws[b], *qkv[b], rows)
        assert max_abs(o[rows].float().cpu().numpy(), ref_o) <= 2e-2 and max_abs(l[rows].cpu().numpy(), ref_l) <= 1e-3, name
        # P and the output are rounded to bf16 (2^-9 each, random): four times what that leaves of the output's norm, where a tile
        # that is only partly added up (a matrix result read too early) shows and an element of the output does not
        err = ((o[rows].double().cpu() - torch.from_numpy(ref_o)).norm() / torch.from_numpy(ref_o).norm()).item()
        assert err <= 4 * 2.0 ** -9, (name, b, err)
    for b in range(2, B):                              # the same sequences again
        assert torch.equal(out[b], out[b % 2]) and torch.equal(lse[b], lse[b % 2])


@pytest.mark.gpu
@pytest.mark.parametrize("case", TAILS, ids=["S%d_d%d_batch%d" % (c[1], c[4], c[5]) for c in TAILS])
def test_what_lies_behind_the_last_key_is_not_seen(case):
    """K and V are the front of larger arrays, or the first of two sequences, and what follows is NaN: the rows of a tile behind the last key
    come as zeros (a probability of zero times NaN would be NaN), so the result has the bits of one with zeros there."""
    from paper_2509_26541_amd import binding as tb
    n, S, Hq, Hkv, d, B = case
    gen = torch.Generator(device="cuda").manual_seed(wl.BASE_SEED + 9990 + S + d)
    draw = lambda rows, heads: torch.randn((rows, heads, d), generator=gen, device="cuda").to(torch.bfloat16)
    q, k, v = draw(S // n, Hq), draw(S, Hkv), draw(S, Hkv)
    results = []
    for tail in (0.0, float("nan")):
        if B == 1:
            kt, vt = (torch.cat([t, torch.full((512, Hkv, d), tail, device="cuda", dtype=t.dtype)])[:S] for t in (k, v))
            qt = q
        else:
            kt, vt = (torch.stack([t, torch.full_like(t, tail)]) for t in (k, v))
            qt = torch.stack([q, q])
        plan = tb.ChunkAttnPlan(tb.tasp_schedule(n, 1), qt, kt, vt, wl.FULL, fuse_steps=True)
        plan.out.fill_(float("nan"))
        plan.lse.fill_(float("nan"))
        out, lse = plan.run()
        torch.cuda.synchronize()
        results.append((out, lse) if B == 1 else (out[0], lse[0]))
    assert all(bool(torch.isfinite(x.float()).all()) for x in results[1])
    assert torch.equal(results[0][0], results[1][0]) and torch.equal(results[0][1], results[1][1])
