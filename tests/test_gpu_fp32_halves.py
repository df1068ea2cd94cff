"""fp32 forward products formed on the 16-bit matrix pipe: edges of tiles, magnitudes, infinities and NaN.  The reference is the
softmax in 64 bits, on the GPU; scaling by powers of two has to give the same bits scaled."""
import numpy as np
import pytest
import torch

from paper_2509_26541_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def tb():
    assert torch.cuda.is_available(), "GPU tests need an MI355X"
    from paper_2509_26541_amd import binding
    return binding


def inputs(n, S, Hq, Hkv, d, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return [torch.empty((rows, h, d), device="cuda").normal_(generator=g) for rows, h in ((S // n, Hq), (S, Hkv), (S, Hkv))]


def positions(n, rank, S, mask):
    if mask == wl.FULL:
        return torch.full((S // n,), S, device="cuda")
    h = S // (2 * n)
    return torch.cat([torch.arange(rank * h, rank * h + h), torch.arange(S - (rank + 1) * h, S - rank * h)]).cuda()


def reference(q, k, v, pos):
    q, k, v = q.double(), k.double(), v.double()
    G = q.shape[1] // k.shape[1]
    out, lse = torch.empty_like(q), torch.empty(q.shape[:2], dtype=torch.float64, device="cuda")
    hidden = torch.arange(k.shape[0], device="cuda")[None, :] > pos[:, None]
    for h in range(q.shape[1]):
        s = (q[:, h] @ k[:, h // G].T / q.shape[2] ** 0.5).masked_fill(hidden, -np.inf)
        lse[:, h] = torch.logsumexp(s, 1)
        out[:, h] = torch.exp(s - lse[:, h:h + 1]) @ v[:, h // G]
    return out, lse


def rel(a, b):
    return float((a.double() - b).norm() / b.norm())


# n, rank, S, Hq, Hkv, d, mask: rows around the 256 (d = 128) and 128 (d = 64) of a query tile, keys around the 32 of a key tile
EDGES = [
    (4, 0, 8, 1, 1, 64, wl.FULL), (4, 3, 8, 1, 1, 128, wl.ZIGZAG_CAUSAL), (4, 1, 4 * 8, 2, 1, 64, wl.FULL), (4, 1, 8 * 4, 4, 2, 128, wl.ZIGZAG_CAUSAL),
    (4, 1, 4 * 255, 1, 1, 128, wl.FULL), (4, 2, 4 * 257, 1, 1, 128, wl.FULL), (4, 1, 8 * 129, 2, 1, 128, wl.ZIGZAG_CAUSAL),
    (4, 1, 4 * 127, 3, 1, 64, wl.FULL), (4, 2, 4 * 129, 1, 1, 64, wl.FULL), (8, 5, 16 * 65, 2, 2, 64, wl.ZIGZAG_CAUSAL),
    (8, 7, 16 * 33, 20, 20, 64, wl.ZIGZAG_CAUSAL), (16, 9, 16 * 511, 4, 1, 128, wl.FULL),
]


@pytest.mark.parametrize("case", EDGES, ids=["-".join(map(str, c)) for c in EDGES])
def test_edges_and_magnitudes(tb, case):
    """Sums of fp32 products err by about sqrt(terms) 2^-24 of their terms; 4 times the 5e-7 that these sizes show."""
    n, rank, S, Hq, Hkv, d, mask = case
    q, k, v = inputs(n, S, Hq, Hkv, d, 11 + S)
    s = tb.tasp_schedule(n, rank)
    out, lse = tb.tasp_chunk_attn(q, k, v, s, mask, fuse_merge=True)
    ref_o, ref_l = reference(q, k, v, positions(n, rank, S, mask))
    assert rel(out, ref_o) <= 2e-6 and float((lse.double() - ref_l).abs().max()) <= 1e-5
    # powers of two: the same bits, scaled (the scores are the same numbers)
    for a, b in ((60, 50), (-70, -80), (-40, 100)):
        out2, lse2 = tb.tasp_chunk_attn(q * 2.0 ** a, k * 2.0 ** -a, v * 2.0 ** b, s, mask, fuse_merge=True)
        assert torch.equal(out2, out * 2.0 ** b) and torch.equal(lse2, lse), (a, b)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("mask", [wl.FULL, wl.ZIGZAG_CAUSAL])
def test_keys_of_very_different_size(tb, d, mask):
    """V rows 2^30 and 2^60 times as large as their neighbours, next to them, a tile away and behind the rows that see them, all with
    scores that give them no weight: the others count as if these were not there.  And V in pieces that differ by up to
    2^12, where no piece may be lost."""
    n, rank, S, H = 4, 1, 8 * 300, 2
    q, k, v = inputs(n, S, H, H, d, 5)
    pos = positions(n, rank, S, mask)
    s = tb.tasp_schedule(n, rank)
    q[:, :, 0] = q[:, :, 0].abs() + 1.0
    big = torch.tensor([3, 70, 71, 340, 350, 601, 1500, S - 700, S - 1], device="cuda")
    k[big, :, 0] = -3000.0
    v[big] *= 2.0 ** 30
    v[big[::2]] *= 2.0 ** 30
    out, lse = tb.tasp_chunk_attn(q, k, v, s, mask, fuse_merge=True)
    ref_o, ref_l = reference(q, k, v, pos)
    assert rel(out, ref_o) <= 2e-6 and float((lse.double() - ref_l).abs().max()) <= 1e-5
    q, k, v = inputs(n, S, H, H, d, 6)
    size = torch.tensor([0, 3, 6, 2, 5, -3, -6, 1], device="cuda")
    v *= (2.0 ** size[(torch.arange(S, device="cuda") // 4) % 8])[:, None, None]
    q[:, :, 0] = 4.0                                         # weight on one size at a time, by the query
    for at in range(8):
        kk = k.clone()
        kk[:, :, 0] += 40.0 * ((torch.arange(S, device="cuda") // 4) % 8 == at)[:, None]
        out, lse = tb.tasp_chunk_attn(q, kk, v, s, mask, fuse_merge=True)
        ref_o, ref_l = reference(q, kk, v, pos)
        assert rel(out, ref_o) <= 6e-6, (at, rel(out, ref_o))      # (scores of about 30: fp32 products and sums give 4.2e-6)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("mask", [wl.FULL, wl.ZIGZAG_CAUSAL])
def test_infinities_and_nan(tb, d, mask):
    """Keys at minus infinity count as if they were not there, an infinite V makes its column infinite (NaN with both signs) for
    the rows that see it and leaves the others, a query row with an infinity is NaN by itself, and so is one with a NaN."""
    n, rank, S, H = 4, 2, 8 * 200, 2
    q, k, v = inputs(n, S, H, H, d, 9)
    pos = positions(n, rank, S, mask)
    s = tb.tasp_schedule(n, rank)
    q[:, :, 0] = q[:, :, 0].abs() + 0.5
    gone = torch.tensor([0, 37, 38, 400, 599, 600, S - 1], device="cuda")
    k[gone, :, 0] = -np.inf
    kf = k.clone()
    kf[gone, :, 0] = -1e6
    out, lse = tb.tasp_chunk_attn(q, k, v, s, mask, fuse_merge=True)
    ref_o, ref_l = reference(q, kf, v, pos)
    assert rel(out, ref_o) <= 2e-6 and float((lse.double() - ref_l).abs().max()) <= 1e-5
    k = kf
    v[410, 0, 3] = np.inf
    v[500, 1, 5] = -np.inf
    v[1020, 1, 7] = np.nan
    q[11, 0, 2] = np.inf
    q[13, 1, 2] = np.nan
    vf, qf = v.clone(), q.clone()
    vf[410, 0, 3] = vf[500, 1, 5] = vf[1020, 1, 7] = 0.0
    qf[11, 0, 2] = qf[13, 1, 2] = 0.0
    out, lse = tb.tasp_chunk_attn(q, k, v, s, mask, fuse_merge=True)
    ref_o, ref_l = reference(qf, k, vf, pos)
    seen = lambda key: pos >= key
    assert bool(out[11, 0].isnan().all()) and bool(out[13, 1].isnan().all()) and float(lse[11, 0]) == float(lse[13, 1]) == -np.inf
    rows = torch.arange(S // n, device="cuda")
    for head, col, key, what in ((0, 3, 410, np.inf), (1, 5, 500, -np.inf), (1, 7, 1020, np.nan)):
        here = seen(key) & (rows != 11 if head == 0 else rows != 13)
        x = out[here, head, col]
        assert bool(x.isnan().all() if np.isnan(what) else (x == what).all()), (head, col)
        out[here, head, col] = ref_o[here, head, col].float()
    out[11, 0], out[13, 1], lse[11, 0], lse[13, 1] = ref_o[11, 0].float(), ref_o[13, 1].float(), ref_l[11, 0].float(), ref_l[13, 1].float()
    assert rel(out, ref_o) <= 2e-6 and float((lse.double() - ref_l).abs().max()) <= 1e-5
