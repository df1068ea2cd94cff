"""Joined steps of bf16 calls with few query tiles (csrc/attn_run.hip): the generated code around its hand-placed waits (CPU), and
every row against the oracle at the edges of its tiles, shares and key counts (GPU)."""
import os
import shutil

import pytest
import torch

from paper_2509_26541_amd import workloads as wl
from tests import asm_checks
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


def test_hazard_checker_flags_a_planted_copy():
    mfma = "v_mfma_f32_32x32x16_bf16 v[0:15], v[16:19], v[20:23], v[0:15]"
    assert [b[0] for b in result_hazards([(1, mfma), (2, "v_mov_b32_e32 v30, v15")])] == [2]
    assert result_hazards([(1, mfma), (2, "s_nop 15"), (3, "v_mov_b32_e32 v30, v15")]) == []
    assert result_hazards([(1, mfma), (2, mfma)]) == []                                     # dependent matrix instructions need none
    loop = [(1, ".L:"), (2, "v_mov_b32_e32 v30, v15"), (3, "s_nop 15"), (4, mfma), (5, "s_cbranch_scc1 .L"), (6, "s_endpgm")]
    assert [b[0] for b in result_hazards(loop)] == [2]                                      # across the loop's end


@pytest.mark.skipif(shutil.which(os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")) is None, reason="hipcc not found")
def test_generated_code(tmp_path):
    """No spills, no register of an LDS read in flight is touched, no matrix result is read too early, every direct load has its
    descriptor and offset in scalar registers."""
    asm = asm_checks.compile_to_asm("attn_run.hip", str(tmp_path / "attn_run.s"))
    ks = {n: i for n, i in asm_checks.kernels(asm).items() if "attn_run_kernel" in n}
    assert len(ks) == 2, list(ks)
    assert all(spills == 0 and scratch == 0 for n, spills, scratch in asm_checks.spill_report(asm) if n in ks)
    for name, ins in ks.items():
        assert asm_checks.in_flight_violations(ins) == [], name
        assert result_hazards(ins) == [], name
        loads = [s for _, s in ins if s.startswith("buffer_load_dwordx4")]
        assert len(loads) >= 8 and all(s.endswith("offen lds") and ", s[" in s for s in loads), (name, loads[:2])


# ---------------------------------------------------------------- against the oracle
# name, N, rank, S, Hq, Hkv, d, mask, batch.  Rows of a block times heads of a group: around 128 and 32; keys: around one and two
# tiles of 64 and even and odd counts of them; several shares, with keys and without.
CASES = [
    ("one_tile_of_keys", 4, 0, 8 * 8, 2, 1, 64, wl.ZIGZAG_CAUSAL, 1),
    ("two_tiles_of_keys_less_one", 4, 1, 4 * 31, 1, 1, 128, wl.FULL, 1),
    ("two_tiles_and_one", 4, 3, 4 * 33, 3, 1, 64, wl.FULL, 2),
    ("strip_and_one", 4, 2, 8 * 33, 1, 1, 128, wl.ZIGZAG_CAUSAL, 1),                # 33 rows: a strip with one
    ("tile_g3", 8, 5, 16 * 43, 6, 2, 128, wl.ZIGZAG_CAUSAL, 1),                     # 129 rows of pairs
    ("odd_tiles", 8, 3, 16 * 75, 4, 4, 64, wl.ZIGZAG_CAUSAL, 16),                   # last tile full, odd number of tiles in a share
    ("even_tiles", 8, 3, 16 * 83, 4, 4, 64, wl.ZIGZAG_CAUSAL, 4),
    ("no_shares", 8, 3, 16 * 75, 20, 20, 64, wl.ZIGZAG_CAUSAL, 20),
    ("no_shares_d128", 8, 6, 16 * 67, 16, 8, 128, wl.ZIGZAG_CAUSAL, 12),
    ("more_than_64_tiles", 8, 7, 16 * 300, 1, 1, 64, wl.FULL, 40),                  # the sum of probabilities in two levels
]


@pytest.mark.gpu
@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_joined_steps_all_rows(case):
    from paper_2509_26541_amd import binding as tb
    name, n, rank, S, Hq, Hkv, d, mode, B = case
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
