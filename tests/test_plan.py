"""How a call is cut follows from its shape: kernel, shares and partial sums are the same with the workspace that the
library reports for it and with a larger one, such as the array of the static call; and which kernel a step takes.
The planner of csrc/api.hip, compiled for the host.  CPU only."""
import os
import shutil
import subprocess

import pytest

from tests import asm_checks

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
pytestmark = pytest.mark.skipif(shutil.which(HIPCC) is None, reason="hipcc not found")

STUBS = r"""
#include "api.hip"
#include <cstdio>
#include <random>

struct Launched { int large, tile, serial, combine; tasp::AttnLaunch last; };
static Launched g;                                // what the forward launches would have been
static int g_dq, g_dkv, g_bwd_fp32;               // and the backward's

namespace tasp {   // launches: none is made here
hipError_t launch_attn_bf16(const AttnLaunch& p, int, hipStream_t) { ++g.large; g.last = p; return hipSuccess; }
hipError_t launch_attn_tile(const AttnLaunch& p, int, bool, bool serial, hipStream_t) { ++g.tile; g.serial += serial; g.last = p; return hipSuccess; }
hipError_t launch_combine(const AttnLaunch&, int, bool, hipStream_t) { ++g.combine; return hipSuccess; }
hipError_t launch_merge(float*, float*, const float*, const float*, int64_t, int64_t, int32_t, int32_t, int32_t, int64_t, hipStream_t) { return hipSuccess; }
hipError_t launch_fill_empty(float*, float*, int64_t, int64_t, int32_t, int32_t, int32_t, int64_t, hipStream_t) { return hipSuccess; }
hipError_t launch_cast_bf16(const float*, void*, int64_t, hipStream_t) { return hipSuccess; }
hipError_t launch_write_i32(int32_t*, const int32_t*, int64_t, hipStream_t) { return hipSuccess; }
hipError_t launch_bwd_dq_bf16(const BwdLaunch&, int, hipStream_t) { ++g_dq; return hipSuccess; }
hipError_t launch_bwd_dkv_bf16(const BwdLaunch&, int, hipStream_t) { ++g_dkv; return hipSuccess; }
hipError_t launch_bwd_dkv_reduce(const BwdLaunch&, int, hipStream_t) { return hipSuccess; }
int64_t bwd_dkv_workgroups(const BwdLaunch& p, int d) {
  const int bs = d == 128 ? 256 : 128;
  return (static_cast<int64_t>(p.rng_vbeg[p.n_rng]) + bs - 1) / bs * p.Hkv * p.batch;
}
int bwd_dkv_resident_workgroups(int d) { return d == 128 ? 256 : 768; }
hipError_t launch_bwd_delta_bf16(const void*, const void*, const float*, float*, float*, float, int64_t, int, hipStream_t) { return hipSuccess; }
hipError_t launch_zero_f32(float*, int64_t, hipStream_t) { return hipSuccess; }
hipError_t launch_bwd_fp32(const BwdLaunch&, int, bool, bool, hipStream_t) { ++g_bwd_fp32; return hipSuccess; }
hipError_t launch_bwd_sum(const float*, int64_t, int, void*, bool, int64_t, hipStream_t) { return hipSuccess; }
hipError_t launch_bwd_delta_fp32(const void*, const void*, float*, int64_t, int, hipStream_t) { return hipSuccess; }
}
"""

PLANS = r"""
struct Plan { bool ok, tile; int n0, n1, kv; size_t bytes; };

static Plan forward(const tasp_schedule_t* s, tasp_attn_args a, size_t ws) {     // ws = 0: as much as is reported for the call
  JoinedSteps js{};
  Shape sh;
  if (validate(s, &a, &sh) != TASP_OK || join_steps(s, &a, &js) != TASP_OK) return {};
  const FwdPlan p = plan_forward(&a, js, tasp_chunk_attn_workspace_bytes(s, &a), ws ? ws : tasp_chunk_attn_best_workspace_bytes(s, &a));
  return {true, p.tile, p.n_split[0], p.n_split[1], 0, p.part_bytes};
}
static Plan forward_none(const tasp_schedule_t* s, tasp_attn_args a) {     // without a workspace: the shares are taken in turn
  JoinedSteps js{};
  Shape sh;
  if (validate(s, &a, &sh) != TASP_OK || join_steps(s, &a, &js) != TASP_OK) return {};
  const FwdPlan p = plan_forward(&a, js, 0, 0);
  if (p.part_bytes > 0 || p.serial != (p.n_split[0] > 1 || p.n_split[1] > 1)) return {};
  return {true, p.tile, p.n_split[0], p.n_split[1], 0, 0};
}
static Plan backward(const tasp_schedule_t* s, tasp_attn_bwd_args b, size_t ws) {
  JoinedSteps js{};
  tasp_attn_args a;
  Shape sh;
  tasp::BwdLaunch bp{};
  if (validate_bwd(s, &b, &a, &sh) != TASP_OK || build_bwd_joined(s, &b, &a, &bp, &js) != TASP_OK) return {};
  const size_t used = ws ? ws : tasp_chunk_attn_bwd_best_workspace_bytes(s, &b);
  const BwdPlan p = plan_backward(&b, sh, bp, js.segments() > static_cast<size_t>(tasp::kPoolSeg) ? kFusedTableBytes : 0, used);
  if (plan_bytes(p, &b, sh) > used) std::printf("backward plan of %zu bytes in %zu\n", plan_bytes(p, &b, sh), used);
  return {plan_bytes(p, &b, sh) <= used, false, p.n_split, 0, p.kv_split, plan_bytes(p, &b, sh)};
}
static bool same(const Plan& x, const Plan& y) { return x.ok == y.ok && x.tile == y.tile && x.n0 == y.n0 && x.n1 == y.n1 && x.kv == y.kv; }
"""

PLAN = PLANS + r"""
int main() {
  std::mt19937 rng(5);
  auto pick = [&](std::initializer_list<int> l) { return l.begin()[rng() % l.size()]; };
  const size_t fixed = TASP_STATIC_SCRATCH_BYTES;
  int bad = 0, fwd = 0, bwd = 0, shared = 0;
  auto report = [&](const char* what, const tasp_attn_args& a, int n, const Plan& x, const Plan& y) {
    if (bad++ < 10)
      std::printf("%s: n=%d S=%lld %d/%d d=%d dtype=%d mask=%d batch=%d fuse_steps=%d: tile %d shares %d %d kv %d, not %d %d %d %d\n", what, n, (long long)a.S, a.Hq, a.Hkv,
                  a.d, a.dtype, a.mask_mode, a.batch, a.fuse_steps, x.tile, x.n0, x.n1, x.kv, y.tile, y.n0, y.n1, y.kv);
  };
  for (int i = 0; i < 12000; ++i) {
    const int n = pick({4, 8, 8, 12, 16}), r = static_cast<int>(rng() % n);
    tasp_schedule_t* s = nullptr;
    if (tasp_schedule_create(n, r, &s) != TASP_OK) return 2;
    tasp_attn_args a{};
    a.q = a.k = a.v = a.out = reinterpret_cast<void*>(256);
    a.d = pick({64, 128});
    a.Hkv = pick({1, 1, 2, 3, 4, 8, 12, 20});
    a.Hq = a.Hkv * pick({1, 1, 2, 3, 4, 8});
    a.dtype = pick({TASP_DTYPE_FP32, TASP_DTYPE_BF16, TASP_DTYPE_BF16});
    a.mask_mode = pick({TASP_MASK_FULL, TASP_MASK_ZIGZAG_CAUSAL, TASP_MASK_ZIGZAG_CAUSAL});
    a.fuse_merge = pick({0, 1});
    a.fuse_steps = pick({0, 1});
    a.batch = pick({1, 1, 2, 3, 4, 16});
    const int64_t rows = 2 << (rng() % 11);                            // up to 4096 local rows
    a.S = n * (rows + 2 * (rng() % (rows / 2 + 1)));
    if (a.S > n * kJoinRows) a.S = n * kJoinRows;
    const size_t need = tasp_chunk_attn_workspace_bytes(s, &a);
    const Plan best = forward(s, a, 0);
    if (best.ok && need <= fixed) {
      ++fwd;
      shared += best.n0 > 1 || best.n1 > 1;
      const Plan st = need > 0 ? forward(s, a, fixed) : forward_none(s, a);        // what the static call brings
      if (!same(best, st)) report("forward, static", a, n, best, st);
      const Plan least = forward(s, a, std::max<size_t>(need, 1));
      if (least.ok && least.bytes > std::max<size_t>(need, 1)) report("forward, least", a, n, least, least);
      if (best.bytes > std::max(tasp_chunk_attn_best_workspace_bytes(s, &a), need)) report("forward, bytes", a, n, best, best);
    }
    tasp_attn_bwd_args b{};
    b.q = b.k = b.v = b.out = b.dout = b.dq = b.dk = b.dv = reinterpret_cast<void*>(256);
    b.lse = reinterpret_cast<float*>(256);
    b.S = a.S; b.Hq = a.Hq; b.Hkv = a.Hkv; b.d = a.d; b.dtype = a.dtype; b.mask_mode = a.mask_mode; b.batch = a.batch;
    b.fuse_steps = a.dtype == TASP_DTYPE_BF16 ? a.fuse_steps : 0;
    const Plan bb = backward(s, b, 0);
    if (bb.ok) {
      ++bwd;
      const Plan more = backward(s, b, std::max(fixed, tasp_chunk_attn_bwd_workspace_bytes(s, &b)));
      if (!same(bb, more)) report("backward, room", a, n, bb, more);
      backward(s, b, tasp_chunk_attn_bwd_workspace_bytes(s, &b));      // the least: within it
    }
    tasp_schedule_destroy(s);
  }
  std::printf("%d forward (%d with shares), %d backward, %d differ\n", fwd, shared, bwd, bad);
  return bad != 0 || fwd < 8000 || shared < 2000 || bwd < 8000;
}
"""

# With more than kJoinRows local rows: fp32 calls and the backward pass.
PLAN_LONG = PLANS + r"""
int main() {
  std::mt19937 rng(6);
  auto pick = [&](std::initializer_list<int> l) { return l.begin()[rng() % l.size()]; };
  const size_t fixed = TASP_STATIC_SCRATCH_BYTES;
  int bad = 0, fwd = 0, bwd = 0, shared = 0, split = 0;
  for (int i = 0; i < 4000; ++i) {
    const int n = pick({4, 8, 8, 12, 16}), r = static_cast<int>(rng() % n);
    tasp_schedule_t* s = nullptr;
    if (tasp_schedule_create(n, r, &s) != TASP_OK) return 2;
    tasp_attn_args a{};
    a.q = a.k = a.v = a.out = reinterpret_cast<void*>(256);
    a.d = pick({64, 128});
    a.Hkv = pick({1, 1, 2, 3, 4, 8});
    a.Hq = a.Hkv * pick({1, 1, 2, 4, 8});
    a.mask_mode = pick({TASP_MASK_FULL, TASP_MASK_ZIGZAG_CAUSAL});
    a.fuse_merge = pick({0, 1});
    a.batch = pick({1, 1, 2, 4});
    const int64_t rows = kJoinRows << (rng() % 3);
    a.S = n * (rows + 2 * (1 + rng() % (rows / 2)));                   // 4 098 to 32 768 local rows
    auto report = [&](const char* what, const Plan& x, const Plan& y) {
      if (bad++ < 10)
        std::printf("%s: n=%d S=%lld %d/%d d=%d dtype=%d mask=%d batch=%d fuse_merge=%d: tile %d shares %d %d kv %d, not %d %d %d %d\n", what, n, (long long)a.S, a.Hq, a.Hkv,
                    a.d, a.dtype, a.mask_mode, a.batch, a.fuse_merge, x.tile, x.n0, x.n1, x.kv, y.tile, y.n0, y.n1, y.kv);
    };
    a.dtype = TASP_DTYPE_FP32;
    const size_t need = tasp_chunk_attn_workspace_bytes(s, &a);
    if (joins(s, &a) && need <= fixed) {
      const Plan best = forward(s, a, 0);
      ++fwd;
      shared += best.n0 > 1 || best.n1 > 1;
      if (need > 0) {
        const Plan st = forward(s, a, fixed);
        if (!same(best, st)) report("forward, static", best, st);
      } else {                       // in turn: as many, or as many more as one set of sums asks for (d = 128)
        const Plan st = forward_none(s, a);
        const int least = a.d == 128 ? static_cast<int>((a.S + tasp::kSumTiles * 32 - 1) / (tasp::kSumTiles * 32)) : 1;
        if (!st.ok || st.tile != best.tile || st.n0 < best.n0 || st.n1 < best.n1 || st.n0 > std::max(best.n0, least) || st.n1 > std::max(best.n1, least)) report("forward, in turn", best, st);
      }
      if (best.bytes > std::max(tasp_chunk_attn_best_workspace_bytes(s, &a), need)) report("forward, bytes", best, best);
      const Plan few = forward(s, a, std::max<size_t>(need, 1));
      if (few.ok && few.bytes > std::max<size_t>(need, 1)) report("forward, least", few, few);
    }
    for (int dtype : {TASP_DTYPE_FP32, TASP_DTYPE_BF16}) {
      a.dtype = dtype;
      if (!joins(s, &a, true)) continue;
      tasp_attn_bwd_args b{};
      b.q = b.k = b.v = b.out = b.dout = b.dq = b.dk = b.dv = reinterpret_cast<void*>(256);
      b.lse = reinterpret_cast<float*>(256);
      b.S = a.S; b.Hq = a.Hq; b.Hkv = a.Hkv; b.d = a.d; b.dtype = dtype; b.mask_mode = a.mask_mode; b.batch = a.batch;
      const Plan bb = backward(s, b, 0);
      if (!bb.ok) { report("backward, refused", bb, bb); continue; }
      ++bwd;
      split += bb.n0 > 1 || bb.kv > 0;
      const Plan more = backward(s, b, std::max(fixed, tasp_chunk_attn_bwd_workspace_bytes(s, &b)));
      if (!same(bb, more)) report("backward, room", bb, more);
      if (!backward(s, b, tasp_chunk_attn_bwd_workspace_bytes(s, &b)).ok) report("backward, least", bb, bb);
    }
    tasp_schedule_destroy(s);
  }
  std::printf("%d forward (%d with shares), %d backward (%d split), %d differ\n", fwd, shared, bwd, split, bad);
  return bad != 0 || fwd < 1200 || shared < 300 || bwd < 5000 || split < 300;
}
"""


STEPS = r"""
// n, rank, rows, heads, KV heads, d, mask, us a step with the large and with the small kernel
struct Case { int n, rank, rows, hq, hkv, d, mask; double large, small; };
static const Case kCases[] = {
  {8, 6, 3320, 16, 2, 128, 0, 94.3, 113.7}, {8, 0, 2974, 32, 4, 128, 1, 94.9, 104.9}, {4, 0, 3884, 32, 8, 128, 1, 138.1, 149.5},
  {4, 1, 4096, 8, 8, 128, 0, 89.0, 92.0}, {4, 2, 3072, 12, 12, 64, 0, 65.7, 68.2},
  {8, 1, 872, 12, 12, 64, 1, 26.9, 18.5}, {8, 2, 446, 16, 2, 128, 1, 26.9, 15.8}, {12, 7, 3248, 1, 1, 64, 1, 47.9, 40.0},
  {8, 0, 1330, 64, 8, 128, 0, 96.9, 81.9}, {16, 4, 1970, 8, 1, 128, 1, 62.7, 43.9},
};

int main() {
  int bad = 0;
  for (const Case& c : kCases) {
    tasp_schedule_t* s = nullptr;
    if (tasp_schedule_create(c.n, c.rank, &s) != TASP_OK) return 2;
    tasp_attn_args a{};
    a.q = a.k = a.v = reinterpret_cast<void*>(256);
    a.S = static_cast<int64_t>(c.rows) * c.n; a.Hq = c.hq; a.Hkv = c.hkv; a.d = c.d;
    a.dtype = TASP_DTYPE_BF16; a.mask_mode = c.mask ? TASP_MASK_ZIGZAG_CAUSAL : TASP_MASK_FULL;
    g = {};
    for (int i = 1; i < c.n; ++i)       // (step 0, with the diagonal, is another launch than the others)
      if (tasp_step_attn(s, &a, i, reinterpret_cast<float*>(256), reinterpret_cast<float*>(256), nullptr) != TASP_OK) return 3;
    std::printf("%d rows, %d/%d heads of %d: large %d, small %d\n", c.rows, c.hq, c.hkv, c.d, g.large, g.tile);
    bad += (c.large < c.small ? g.tile : g.large) != 0;
    tasp_schedule_destroy(s);
  }
  return bad;
}
"""


STATIC = r"""
// The static call of shapes that need no workspace: it succeeds without a GPU, so it does not ask for the array's address, and
// the launch has the shares of the other calls but no place for pairs of them.
int main() {
  tasp_schedule_t* s = nullptr;
  if (tasp_schedule_create(8, 3, &s) != TASP_OK) return 2;
  int shared = 0;
  for (int d : {64, 128})
    for (int rows : {2, 70, 256, 1024, 4096}) {
      tasp_attn_args a{};
      a.q = a.k = a.v = a.out = reinterpret_cast<void*>(256);
      a.lse = reinterpret_cast<float*>(256);
      a.S = 8 * rows; a.Hq = 4; a.Hkv = 2; a.d = d; a.dtype = TASP_DTYPE_FP32; a.mask_mode = TASP_MASK_ZIGZAG_CAUSAL; a.fuse_merge = 1;
      if (tasp_chunk_attn_workspace_bytes(s, &a) != 0) return 3;
      g = {};
      if (tasp_chunk_attn_static(s, &a, nullptr) != TASP_OK) return 4;
      const Launched st = g;
      if (st.tile != 1 || st.combine != 0 || st.last.part_o[0] != nullptr || st.last.part_o[1] != nullptr) return 5;
      g = {};
      a.workspace = reinterpret_cast<void*>(256);
      a.workspace_bytes = tasp_chunk_attn_best_workspace_bytes(s, &a);
      if (tasp_chunk_attn(s, &a, nullptr) != TASP_OK || g.serial != 0) return 6;
      for (int t = 0; t < 2; ++t)
        if (g.last.n_split[t] != st.last.n_split[t]) return 7;
      shared += g.combine;
    }
  return shared >= 6 ? 0 : 8;
}
"""


PATHS = r"""
// n, rank, sequence length, heads, KV heads, d, mask, batch: shapes whose steps are tested one by one and joined
struct Path { int n, rank, S, hq, hkv, d, mask, batch; };
static const Path kPaths[] = {
  {4, 1, 8 * 2051, 4, 2, 128, 1, 1}, {4, 3, 4 * 4099, 3, 1, 128, 0, 1}, {4, 2, 8 * 2051, 2, 1, 64, 1, 1}, {4, 0, 8 * 2310, 2, 2, 64, 1, 1}, {4, 2, 8 * 2049, 2, 1, 128, 1, 2},
  {4, 0, 8 * 2310, 8, 8, 64, 1, 6},
};

int main() {
  for (const Path& c : kPaths) {
    tasp_schedule_t* s = nullptr;
    if (tasp_schedule_create(c.n, c.rank, &s) != TASP_OK) return 2;
    tasp_attn_args a{};
    a.q = a.k = a.v = a.out = a.workspace = reinterpret_cast<void*>(256);
    a.lse = reinterpret_cast<float*>(256);
    a.workspace_bytes = size_t{1} << 40;
    a.S = c.S; a.Hq = c.hq; a.Hkv = c.hkv; a.d = c.d; a.batch = c.batch;
    a.dtype = TASP_DTYPE_BF16; a.mask_mode = c.mask ? TASP_MASK_ZIGZAG_CAUSAL : TASP_MASK_FULL;
    for (int fuse : {0, 1}) {
      g = {};
      a.fuse_merge = fuse;
      if (tasp_chunk_attn(s, &a, nullptr) != TASP_OK || g.large != c.n || g.tile != 0) return 3;      // the large kernel, step by step
    }
    g = {};
    a.fuse_steps = 1;
    if (tasp_chunk_attn(s, &a, nullptr) != TASP_OK) return 4;
    std::printf("S %d, d %d: joined by the %s kernel\n", c.S, c.d, g.large ? "large" : "small");
    tasp_schedule_destroy(s);
  }
  return 0;
}
"""


JOINS = r"""
// n, sequence length, heads, KV heads, d, launches of a call that does not ask for joined steps: bf16 forward, fp32 forward, backward
struct Join { int n, S, hq, hkv, d, bf16, fp32, bwd; };
static const Join kJoins[] = {
  {8, 8 * 4096, 8, 2, 128, 1, 1, 1}, {8, 8 * 4098, 8, 2, 128, 8, 1, 1}, {8, 131072, 32, 8, 128, 8, 1, 1}, {16, 16 * 4100, 20, 20, 64, 16, 1, 1},
  {12, 12 * 6000, 4, 1, 64, 12, 1, 1}, {8, 430080, 4, 4, 64, 8, 1, 1}, {4, 4 * 8194, 4, 4, 128, 4, 1, 1}, {4, 4 * 8192, 4, 4, 128, 4, 4, 4}, {4, 4 * 4098, 2, 1, 64, 4, 4, 4},
};

int main() {
  int bad = 0;
  for (const Join& c : kJoins) {
    tasp_schedule_t* s = nullptr;
    if (tasp_schedule_create(c.n, 1, &s) != TASP_OK) return 2;
    for (int mask : {TASP_MASK_FULL, TASP_MASK_ZIGZAG_CAUSAL})
      for (int dtype : {TASP_DTYPE_BF16, TASP_DTYPE_FP32}) {
        tasp_attn_args a{};
        a.q = a.k = a.v = a.out = a.workspace = reinterpret_cast<void*>(256);
        a.lse = reinterpret_cast<float*>(256);
        a.workspace_bytes = size_t{1} << 40;
        a.S = c.S; a.Hq = c.hq; a.Hkv = c.hkv; a.d = c.d; a.dtype = dtype; a.mask_mode = mask;
        for (int fuse_merge : {0, 1})
          for (int fuse_steps : {0, 1}) {
            a.fuse_merge = fuse_merge; a.fuse_steps = fuse_steps;
            g = {};
            if (tasp_chunk_attn(s, &a, nullptr) != TASP_OK) return 3;
            const int want = fuse_steps ? 1 : dtype == TASP_DTYPE_BF16 ? c.bf16 : c.fp32;
            if (g.large + g.tile != want && bad++ < 10)
              std::printf("forward, n %d, S %d, d %d, dtype %d, mask %d, fuse_merge %d, fuse_steps %d: %d launches\n", c.n, c.S, c.d, dtype, mask, fuse_merge, fuse_steps, g.large + g.tile);
          }
        tasp_attn_bwd_args b{};
        b.q = b.k = b.v = b.out = b.dout = b.dq = b.dk = b.dv = b.workspace = reinterpret_cast<void*>(256);
        b.lse = reinterpret_cast<float*>(256);
        b.workspace_bytes = size_t{1} << 40;
        b.S = c.S; b.Hq = c.hq; b.Hkv = c.hkv; b.d = c.d; b.dtype = dtype; b.mask_mode = mask;
        g_dq = g_dkv = g_bwd_fp32 = 0;
        if (tasp_chunk_attn_bwd(s, &b, nullptr) != TASP_OK) return 4;
        const bool bf16 = dtype == TASP_DTYPE_BF16;
        if ((g_dq != (bf16 ? c.bwd : 0) || g_dkv != g_dq || g_bwd_fp32 != (bf16 ? 0 : c.bwd)) && bad++ < 10)
          std::printf("backward, n %d, S %d, d %d, dtype %d, mask %d: %d, %d, %d launches\n", c.n, c.S, c.d, dtype, mask, g_dq, g_dkv, g_bwd_fp32);
      }
    tasp_schedule_destroy(s);
  }
  return bad;
}
"""


FEW_SHARES = r"""
// 16 ranks of two nodes, 20 heads of 64, 104 832 tokens, all steps in one launch: 2.73 ms with the small kernel and no
// shares, 3.30 with the large one.  The small one it is, whoever brings the workspace.
int main() {
  tasp_schedule_t* s = nullptr;
  if (tasp_schedule_create_multinode(8, 2, 12, &s) != TASP_OK) return 2;
  tasp_attn_args a{};
  a.q = a.k = a.v = a.out = a.workspace = reinterpret_cast<void*>(256);
  a.lse = reinterpret_cast<float*>(256);
  a.S = 104832; a.Hq = a.Hkv = 20; a.d = 64; a.dtype = TASP_DTYPE_BF16; a.mask_mode = TASP_MASK_ZIGZAG_CAUSAL; a.fuse_steps = 1;
  for (size_t bytes : {tasp_chunk_attn_workspace_bytes(s, &a), tasp_chunk_attn_best_workspace_bytes(s, &a), static_cast<size_t>(TASP_STATIC_SCRATCH_BYTES)}) {
    a.workspace_bytes = bytes;
    g = {};
    if (tasp_chunk_attn(s, &a, nullptr) != TASP_OK) return 3;
    std::printf("%zu bytes: large %d, small %d with %d and %d shares\n", bytes, g.large, g.tile, g.last.n_split[0], g.last.n_split[1]);
    if (g.tile != 1) return 4;
  }
  return 0;
}
"""


MAKESPAN = r"""
// Each workgroup to the slot that is free first, the longer kind first.
static double deal(int n0, double l0, int n1, double l1, int slots) {
  std::vector<double> done(slots, 0.0);
  if (l0 < l1) { std::swap(n0, n1); std::swap(l0, l1); }
  for (int i = 0; i < n0 + n1; ++i) *std::min_element(done.begin(), done.end()) += i < n0 ? l0 : l1;
  return *std::max_element(done.begin(), done.end());
}
int main() {
  std::mt19937 rng(1);
  auto upto = [&](int n) { return static_cast<int>(rng() % (n + 1)); };
  double worst = 0;
  for (int i = 0; i < 200000; ++i) {
    const int slots = 1 + upto(11), n0 = 1 + upto(5 * slots), n1 = i % 5 == 0 ? 0 : upto(8 * slots);
    const double l0 = 1 + upto(39), l1 = n1 == 0 ? 0 : 1 + upto(39);
    const double want = deal(n0, l0, n1, l1, slots), got = makespan(n0, l0, n1, l1, slots), gap = std::abs(got - want) / want;
    if (gap > worst) { worst = gap; std::printf("%d of %g, %d of %g, %d slots: %g, dealt one by one %g\n", n0, l0, n1, l1, slots, got, want); }
  }
  return worst > 1e-12 ? 3 : 0;
}
"""


def run_planner(tmp_path, program, text=""):
    """What `program` prints, compiled with the planner for the host, given `text`; it has to end with 0."""
    src, exe = tmp_path / "plan.cpp", tmp_path / "plan"
    src.write_text(STUBS + program)
    subprocess.run([HIPCC, "--offload-arch=gfx950", "-O1", "-std=c++17", "-I" + os.path.join(asm_checks.ROOT, "include"), "-I" + asm_checks.CSRC,
                    "-x", "hip", str(src), os.path.join(asm_checks.CSRC, "schedule.cpp"), "-o", str(exe)], check=True, capture_output=True, text=True)
    res = subprocess.run([str(exe)], input=text, capture_output=True, text=True, timeout=300)
    assert res.returncode == 0, res.stdout
    return res.stdout


def _run(tmp_path, program):
    run_planner(tmp_path, program)


def test_plan_follows_from_the_shape(tmp_path):
    _run(tmp_path, PLAN)


def test_plan_follows_from_the_shape_with_many_rows(tmp_path):
    """The same where the library joins the steps of calls with more than 4 096 local rows."""
    print(run_planner(tmp_path, PLAN_LONG))


def test_a_step_takes_the_faster_kernel(tmp_path):
    """Shapes timed with either kernel, per step."""
    _run(tmp_path, STEPS)


def test_static_calls_without_need_leave_the_array_alone(tmp_path):
    _run(tmp_path, STATIC)


def test_more_than_4096_rows_run_step_by_step(tmp_path):
    """The shapes of tests/test_gpu_step_path.py take the large kernel, a launch per step."""
    _run(tmp_path, PATHS)


def test_which_calls_have_their_steps_joined(tmp_path):
    """bf16 forward calls with more than 4 096 local rows run step by step, whatever the number of ranks, unless asked otherwise."""
    _run(tmp_path, JOINS)


def test_a_joined_call_takes_the_faster_kernel_without_shares(tmp_path):
    _run(tmp_path, FEW_SHARES)


def test_when_the_last_workgroup_is_done(tmp_path):
    """The formula by which shares are weighed, against dealing workgroup by workgroup."""
    _run(tmp_path, MAKESPAN)
