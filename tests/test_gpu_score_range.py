"""bf16 forward: one key far above all others, in either half of the eight keys that the two lane halves of a wavefront share
(the running maximum has to come from both)."""
import pytest
import torch

from paper_2509_26541_amd import workloads as wl
from tests.helpers import max_abs, oracle_rows

pytestmark = pytest.mark.gpu

# name, N, rank, S, Hq, Hkv, d, mask, fuse_steps: single steps and joined ones of the large kernel (d = 64: eight and twelve wavefronts), and
# joined steps with few query tiles
CASES = [
    ("steps_d128", 4, 1, 4 * 4104, 2, 1, 128, wl.FULL, False),
    ("steps_d64_twelve_wavefronts", 4, 2, 8 * 2051, 2, 1, 64, wl.ZIGZAG_CAUSAL, False),
    ("steps_d64_eight_wavefronts", 4, 0, 8 * 2310, 2, 2, 64, wl.ZIGZAG_CAUSAL, False),
    ("joined_d128", 4, 1, 4 * 4096, 32, 8, 128, wl.FULL, True),
    ("few_rows_d128", 8, 3, 16 * 64, 4, 1, 128, wl.FULL, True),
    ("few_rows_d64", 8, 3, 16 * 64, 4, 4, 64, wl.FULL, True),
]


@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_one_dominant_key_at_every_place(case):
    from paper_2509_26541_amd import binding as tb
    name, n, rank, S, Hq, Hkv, d, mode, fuse = case
    w = wl.Workload(name, n, rank, S, Hq, Hkv, d, "bf16", mode, seed=wl.BASE_SEED + 9950 + d)
    q, k0, v = wl.make_qkv(w)
    q = q + 4.0
    s = tb.tasp_schedule(n, rank)
    rows = wl.sample_rows(w, 8)
    qd, vd = q.cuda(), v.cuda()
    for at in range(500, 508):
        k = k0.clone()
        k[at] = 5.0 if d == 64 else 3.5                       # a score of about 160, 230 in base two: exp2 of it leaves fp32 against any other maximum
        out, lse = tb.tasp_chunk_attn(qd, k.cuda(), vd, s, mode, fuse_merge=True, fuse_steps=fuse)
        torch.cuda.synchronize()
        assert bool(torch.isfinite(out.float()).all()) and bool(torch.isfinite(lse).all()), (name, at)
        ref_o, ref_l = oracle_rows(w, q, k, v, rows)
        assert max_abs(out[rows].float().cpu().numpy(), ref_o) <= 2e-2 and max_abs(lse[rows].cpu().numpy(), ref_l) <= 1e-3, (name, at)
