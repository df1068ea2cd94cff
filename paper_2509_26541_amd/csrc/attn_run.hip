// Blockwise attention of joined steps, bf16: 128 (row, query head of the group) pairs per workgroup, all keys by position.
//
// The same cut of the work as attn_tile_kernel: a tile's rows are packed over the heads of a group, and n_split workgroups
// each take an equal run of the tile's visible keys.  Over joined steps the keys are one run of positions, so there is no list
// to walk: the loader is a scalar offset per load, and the loop is pipelined by hand like that of the large kernel
// (attn_bf16.hip).  With 32 (d = 64) and 64 KiB (d = 128) of LDS and 162 and 213 registers three and two workgroups share a CU;
// they are at different places in their loops, so one's set-up, barrier and epilogue are filled by the others' work, where the
// large kernel has a CU to itself.
//
// What bounds it: the vector issue port.  Per 64-key tile and wavefront 106 vector instructions, 33 exponentials and 16 (d = 64) or
// 32 matrix instructions; attn_tile_kernel, whose loop serves single steps, takes 138 and some 70 scalar ones and branches.  Whole
// calls, against that kernel and against the large one:
//   16 ranks, 24 heads over 8 of 128, 2 086 of 33 376 tokens, causal, batch 2: 771 us, 845, 1 050 (large: 23 % of its rows are padding);
//   20 heads of 64, 384 of 3 072 tokens, causal, batch 128: 628 us, 664, 1 000;
//   12 heads of 64, 12 500 of 100 000 tokens, causal, batch 2: 4.37 ms, large 5.28 (256-row tiles);
//   32 heads over 8 of 128, 4 096 of 32 768 tokens, causal: 935 us, large 900: there 256 rows share a tile's fetch, and nothing is padded.
// Measured and not kept: six and three wavefronts to a workgroup at d = 64 (192 and 96 rows: they do not spread evenly over four
// SIMDs, 10 to 25 % slower); wavefronts without rows that leave at once instead of fetching (no gain); fetches all at the start of
// a body (1 % slower at d = 128).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <climits>

#include "gfx950.hpp"
#include "internal.hpp"
#include "pipeline.hpp"

namespace tasp {
namespace {

template <int D>
struct RunCfg {
  static constexpr int BM = tile_rows(false, D), NW = BM / 32, NTHREADS = 64 * NW;
  static constexpr int BT = 64;                         // keys per tile
  static constexpr int RB = 2 * D;                      // bytes of a row
  static constexpr int UNITS = RB / 16;                 // 16-byte units of it
  static constexpr int RPW = 64 / UNITS, RPP = NW * RPW, PASSES = BT / RPP;     // rows to a wavefront's load, to a pass of all; loads to a tile
  static constexpr int RPL = 16 / UNITS;                // rows per 256-byte bank line
  static constexpr int TILE_BYTES = BT * RB;
  static constexpr int NDB = D / 32, NJ = D / 16;
  static_assert(RPP % 16 == 0, "the swizzle of a thread's rows does not depend on the pass");
  __device__ static int swz_k(int r, int u) { return u ^ ((r / RPL) % UNITS); }
  __device__ static int swz_v(int r, int u) { return u ^ (4 * ((r / RPL) % (UNITS / 4))); }
};

// One block of query rows of a launch (AttnTask), and how its keys are dealt.
struct RunTask {
  int32_t q_row0, n_q, q_pos0, rows, tiles;     // rows: (row, head of the group) pairs
  int32_t n_split;
  Divider split;
  float* part_o;
  float* part_lse;
};
// What the kernel needs of an AttnLaunch, with every division prepared.
struct RunLaunch {
  const void* q;
  const void* k;
  const void* v;
  void* out;
  float* lse;
  int64_t q_bstride, kv_bstride, lse_bstride;
  int32_t Hq, Hkv, G, causal, n_keys, batch;
  float scale_log2e;
  int32_t items0;                               // work items of a unit (sequence, KV head) that belong to the first task
  XcdMap map;
  Divider by_kv_heads, by_group;
  RunTask task[kMaxTasks];
};

template <int D>
__global__ __launch_bounds__(RunCfg<D>::NTHREADS, D == 64 ? 3 : 2) void attn_run_kernel(const RunLaunch p) {
  using C = RunCfg<D>;
  constexpr int BM = C::BM, NW = C::NW, BT = C::BT, NDB = C::NDB, NJ = C::NJ;
  __shared__ __attribute__((aligned(16))) unsigned char smem[4 * C::TILE_BYTES];      // two K tiles, two V tiles

  const int thread = threadIdx.x, wave_u = __builtin_amdgcn_readfirstlane(thread >> 6);
  const int lane = thread & 63, h = lane >> 5, lq = lane & 31;
  // ---- which (sequence, KV head) and which item of it
  int unit, item;
  if (!xcd_item(p.map, blockIdx.x, unit, item)) return;
  const int bi = divide(unit, p.by_kv_heads), g = unit - bi * p.Hkv;
  const bool second = item >= p.items0;
  const RunTask& T = p.task[second ? 1 : 0];
  const int rem = item - (second ? p.items0 : 0), tile_up = divide(rem, T.split), share = rem - tile_up * T.n_split, ns = T.n_split;
  // under the causal mask the later tiles of a block see more keys: they start first
  const int tile = p.causal ? T.tiles - 1 - tile_up : tile_up;
  // The strip of 32 rows a wavefront takes moves with the work item: wavefront i of a workgroup runs on
  // SIMD i, and tiles with few rows left leave strips without work.
  const int strip = (wave_u + item) % NW, left = T.rows - tile * BM;
  const int m = tile * BM + strip * 32 + lq, mc = min(m, T.rows - 1), q_row = divide(mc, p.by_group);
  const bool q_valid = m < T.rows;
  const int64_t q_idx = static_cast<int64_t>(T.q_row0 + q_row) * p.Hq + g * p.G + mc - q_row * p.G;
  const int q_last = T.q_pos0 + divide(tile * BM + min(left, BM) - 1, p.by_group);
  const int q_first = p.causal ? T.q_pos0 + static_cast<int>(divide(tile * BM, p.by_group)) : INT_MAX - 1;   // a key at or before it is seen by every row

  // ---- the keys: n_keys of them from goff on
  int n_keys = p.causal ? q_last + 1 : p.n_keys, goff = 0;
  if (ns > 1) {
    const int chunk = (static_cast<int>(divide(n_keys + ns - 1, T.split)) + BT - 1) / BT * BT;
    goff = share * chunk;
    n_keys = max(0, min(n_keys - goff, chunk));
  }
  const int n_tiles = (n_keys + BT - 1) / BT, first_masked = min(n_keys, max(q_first + 1 - goff, 0)) / BT;      // tiles from first_masked on take the element-wise mask

  // ---- loader
  const unsigned row_bytes = static_cast<unsigned>(p.Hkv) * C::RB;
  const int64_t head0 = (bi * p.kv_bstride + static_cast<int64_t>(g) * D) * 2 + static_cast<int64_t>(goff) * row_bytes;
  const unsigned records = n_keys > 0 ? static_cast<unsigned>(n_keys - 1) * row_bytes + C::RB : 0u;
  // Records end with the share's last key: what is fetched behind it, in the last tile and by the fetches that run ahead, comes
  // as zeros.  The range check of a raw buffer is "vector offset >= records - scalar offset", so a scalar offset stops at the
  // records' end: beyond it the difference would be below zero.  (Before that, offsets stay below 2^32, see attn_run_takes.)
  const u32x4 k_buf = raw_buffer(static_cast<const unsigned char*>(p.k) + head0, records), v_buf = raw_buffer(static_cast<const unsigned char*>(p.v) + head0, records);
  const int fr = C::RPW * wave_u + lane / C::UNITS, fu = lane % C::UNITS;
  const unsigned lane_row = static_cast<unsigned>(lane / C::UNITS) * row_bytes;
  const unsigned k_lane = lane_row + C::swz_k(fr, fu) * 16, v_lane = lane_row + C::swz_v(fr, fu) * 16;
  // tile u of K or V to stage st; rows past the end come as zeros
  auto fetch = [&](auto vv, int u, int st) __attribute__((always_inline)) {
    constexpr bool V = decltype(vv)::value;
    unsigned char* const dst = smem + (V ? 2 * C::TILE_BYTES : 0) + st * C::TILE_BYTES + wave_u * 1024;
    const unsigned at = static_cast<unsigned>(u * BT + C::RPW * wave_u) * row_bytes;
#pragma unroll
    for (int i = 0; i < C::PASSES; ++i) buffer_to_lds_16<true>(V ? v_buf : k_buf, min(at + i * C::RPP * row_bytes, records), V ? v_lane : k_lane, dst + i * C::NTHREADS * 16);
  };
  constexpr std::false_type K{};
  constexpr std::true_type V{};
  fetch(K, 0, 0);
  fetch(K, 1, 1);
  fetch(V, 0, 0);
  u32x4 qf[NJ];
  {
    const u32x4* src = reinterpret_cast<const u32x4*>(static_cast<const __bf16*>(p.q) + bi * p.q_bstride + q_idx * D) + h;
#pragma unroll
    for (int j = 0; j < NJ; ++j) qf[j] = src[2 * j];
  }
  const int last_pos = min(p.causal ? T.q_pos0 + q_row : INT_MAX - 1, goff + n_keys - 1);      // the lane's row sees the keys up to it

  const unsigned smem_lds = static_cast<unsigned>(reinterpret_cast<size_t>((lds_void_ptr)smem));
  const unsigned k_adr = lq * C::RB + C::swz_k(lq, h) * 16;          // unit 2 j + h sits at k_adr ^ 32 j
  unsigned ka[NJ], va[NDB];
#pragma unroll
  for (int j = 0; j < NJ; ++j) ka[j] = smem_lds + (k_adr ^ (32 * j));
  {
    const int ga = lane >> 4, jj = lane & 15;
    const int vrow = 4 * (ga >> 1) + (jj >> 2);
#pragma unroll
    for (int db = 0; db < NDB; ++db) va[db] = smem_lds + vrow * C::RB + C::swz_v(vrow, 4 * db + 2 * (ga & 1) + ((jj & 3) >> 1)) * 16 + 8 * (jj & 1);
  }
  f32x16 o[NDB];
#pragma unroll
  for (int db = 0; db < NDB; ++db) o[db] = zero16();
  // running max (exp2 domain), this lane's sum in two levels (up to 64 tiles, everything before) and what rounding added to the largest
  // probabilities: as in the large kernel
  float m_run = kNegBig, m_raise = kNegBig, l_run = 0.f, l_lo = 0.f, r_fix = 0.f, mx = kNegBig;
  const float c = p.scale_log2e;

  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
#pragma unroll
  for (int j = 0; j < NJ; ++j) asm volatile("" : "+v"(qf[j]));
  __syncthreads();
  if (strip * 32 >= left) {            // no rows: fetches only, with the barriers of the others
    if (n_tiles > 1) __syncthreads();
    for (int t = 0; t + 1 < n_tiles; ++t) {
      fetch(K, t + 2, t & 1);
      fetch(V, t + 1, (t + 1) & 1);
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      __syncthreads();
    }
    return;
  }
  constexpr int NF = 2 * NJ, NV = 4 * NDB, PD = 4;
  f32x16 Sa[2], Sb[2];
  // The operand fragments of a body as one stream, read PD ahead: NF of K of the next tile, then NV of V^T of this one (of two reads
  // each).  One wait serves an even fragment and the odd one behind it.
  u32x4 fk[PD];
  u32x2 fl[PD], fh[PD];
  auto read = [&](auto ff, auto sk, auto sv) __attribute__((always_inline)) {
    constexpr int F = decltype(ff)::value;
    if constexpr (F < NF) {
      lds_read_b128<F % 2 * 32 * C::RB + decltype(sk)::value * C::TILE_BYTES>(fk[F % PD], ka[F / 2]);
    } else if constexpr (F < NF + NV) {
      constexpr int FV = F - NF, AT = (2 + decltype(sv)::value) * C::TILE_BYTES + FV / NDB * 16 * C::RB;
      lds_read_tr_b64<AT>(fl[F % PD], va[FV % NDB]);
      lds_read_tr_b64<AT + 8 * C::RB>(fh[F % PD], va[FV % NDB]);
    }
  };
  // LDS instructions younger than those of fragments f and f + 1 when f is needed (`end`: fragments of the stream)
  auto younger = [](int f, int end) constexpr {
    if (f % 2 != 0) return -1;
    int n = 0;
    for (int r = f + 2; r < f + PD && r < end; ++r) n += r < NF ? 1 : 2;
    return n;
  };
  auto v_fragment = [&](auto ff) __attribute__((always_inline)) { constexpr int F = decltype(ff)::value % PD; return u32x4{fl[F][0], fl[F][1], fh[F][0], fh[F][1]}; };
  static_assert(NF % PD == 0 && NF % 2 == 0 && NV % 2 == 0 && PD % 2 == 0 && 4 * C::TILE_BYTES <= 65536, "");
  auto mask = [&](int t, f32x16 (&S)[2]) __attribute__((always_inline)) {
    if (__builtin_expect(t < first_masked, 1)) return;
    const int at = goff + t * BT + 4 * h;
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
      for (int i = 0; i < 16; ++i)
        if (at + 32 * kb + 8 * (i / 4) + i % 4 > last_pos) S[kb][i] = -__builtin_inff();
  };
  auto max_step = [&](auto ii, f32x16 (&S)[2]) __attribute__((always_inline)) {      // scores 2 I, 2 I + 1 of the 32 a lane holds
    constexpr int I = decltype(ii)::value;
    const float a = S[I / 8][2 * I % 16], b = S[I / 8][2 * I % 16 + 1];
    mx = I == 0 ? fmaxf(a, b) : fmaxf(fmaxf(mx, a), b);
  };
  u32x4 pf[4];
  float late[2], sum[4];
  auto exp_one = [&](auto ee, f32x16 (&S)[2]) __attribute__((always_inline)) {
    constexpr int E = decltype(ee)::value;
    const float x = fast_exp2(__builtin_fmaf(S[E / 16][E % 16], c, -m_run));
    sum[E % 4] = E < 4 ? x : sum[E % 4] + x;
    asm volatile("" : "+v"(sum[E % 4]));           // (here, not in a later block)
    late[E % 2] = x;
    if constexpr (E % 2 == 1) {
      const bf16x2 pk = {static_cast<__bf16>(late[0]), static_cast<__bf16>(late[1])};
      unsigned u = __builtin_bit_cast(unsigned, pk);
      asm volatile("" : "+v"(u));
      pf[E / 8][E % 8 / 2] = u;
    }
  };
  auto exps = [&](auto lo, auto hi, f32x16 (&S)[2]) __attribute__((always_inline)) {
    constexpr int LO = decltype(lo)::value;
    static_for<decltype(hi)::value - LO>([&](auto i) __attribute__((always_inline)) { exp_one(std::integral_constant<int, LO + decltype(i)::value>{}, S); });
  };
  // a tile's probabilities are summed for themselves and then added to the sum, so that this is rounded once a tile
  auto add_up = [&]() __attribute__((always_inline)) {
    l_lo += (sum[0] + sum[1]) + (sum[2] + sum[3]);
    asm volatile("" : "+v"(l_lo));
  };
  // the output can be read by vector instructions from here on
  auto fence_o = [&]() __attribute__((always_inline)) {
    if constexpr (NDB == 2) asm volatile("s_nop 15\n\ts_nop 3" : "+v"(o[0]), "+v"(o[1]));
    else asm volatile("s_nop 15\n\ts_nop 3" : "+v"(o[0]), "+v"(o[1]), "+v"(o[NDB - 2]), "+v"(o[NDB - 1]));
  };
  // Before the probabilities of a tile whose maxima are in mx: raises the running max where it grew by more than the gap (a lane
  // tests the scores it holds; a row has grown iff one of its two lanes has), and takes down what rounding adds to the largest of them.
  auto raise = [&]() __attribute__((always_inline)) {
    if (__builtin_amdgcn_ballot_w64(mx * c > m_raise) != 0) {
      const float m_new = fmaxf(m_run, max_of_halves(mx) * c);     // both halves of a row agree
      const float alpha = fast_exp2(m_run - m_new);
      m_run = m_new;
      m_raise = m_new + kRescaleGap;
      fence_o();
      l_run *= alpha; l_lo *= alpha; r_fix *= alpha;
#pragma unroll
      for (int db = 0; db < NDB; ++db) {
        o[db] *= alpha;
        asm volatile("s_nop 1" : "+v"(o[db]));
      }
    }
    const float p_top = fast_exp2(__builtin_fmaf(mx, c, -m_run));
    r_fix += static_cast<float>(static_cast<__bf16>(p_top)) - p_top;
  };
  // Exponentials are dealt out to the matrix instructions as in the large kernel: PRE before the first, up to EK beside the scores,
  // the rest beside the first VE of the second product; the maxima of the next tile from its instruction VS on.
  constexpr int PRE = 2, EK = 20, VE = 3 * NV / 4, VS = NV / 4;
  // Tile t (stage t % 2): scores of tile t + 1 beside the first probabilities of S, then the second product beside the others and
  // the maxima of S_next.  The fetches go to what body t - 1 has left, and have this body's time: everybody has passed its
  // barrier, and they are waited for before the next.
  auto body = [&](auto ss, int t, f32x16 (&S)[2], f32x16 (&S_next)[2]) __attribute__((always_inline)) {
    constexpr int ST = decltype(ss)::value;
    constexpr std::integral_constant<int, ST ^ 1> sk{};
    static_for<PD>([&](auto f) __attribute__((always_inline)) { read(f, sk, ss); });
    __builtin_amdgcn_sched_barrier(0);
    raise();
    exps(std::integral_constant<int, 0>{}, std::integral_constant<int, PRE>{}, S);
    __builtin_amdgcn_sched_barrier(0);
    static_for<NF>([&](auto ff) __attribute__((always_inline)) {
      constexpr int F = decltype(ff)::value, ks = F / 2, kb = F % 2;
      if constexpr (ks == 0) mfma_s_first<false, younger(F, NF + NV)>(S_next[kb], fk[F % PD], qf[ks]);
      else mfma_s<false, younger(F, NF + NV)>(S_next[kb], fk[F % PD], qf[ks]);
      read(std::integral_constant<int, F + PD>{}, sk, ss);
      exps(std::integral_constant<int, PRE + (EK - PRE) * F / NF>{}, std::integral_constant<int, PRE + (EK - PRE) * (F + 1) / NF>{}, S);
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (F == 1) fetch(K, t + 2, ST);
      if constexpr (F == NF / 2 + 1) fetch(V, t + 1, ST ^ 1);
    });
    static_for<NV>([&](auto ff) __attribute__((always_inline)) {
      constexpr int F = decltype(ff)::value, gg = F / NDB, db = F % NDB;
      if constexpr (F == VS) { fence_s(S_next[0], S_next[1]); mask(t + 1, S_next); }
      if constexpr (db == 0) fence_p(pf[gg]);
      mfma_s<false, younger(NF + F, NF + NV)>(o[db], v_fragment(std::integral_constant<int, NF + F>{}), pf[gg]);
      read(std::integral_constant<int, NF + F + PD>{}, sk, ss);
      if constexpr (F < VE) exps(std::integral_constant<int, EK + (32 - EK) * F / VE>{}, std::integral_constant<int, EK + (32 - EK) * (F + 1) / VE>{}, S);
      if constexpr (F == VE) add_up();
      if constexpr (F >= VS) {
        constexpr int lo = 16 * (F - VS) / (NV - VS), hi = 16 * (F + 1 - VS) / (NV - VS);
        static_for<hi - lo>([&](auto i) __attribute__((always_inline)) { max_step(std::integral_constant<int, lo + decltype(i)::value>{}, S_next); });
      }
      __builtin_amdgcn_sched_barrier(0);
    });
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
  };
  // The last tile.
  auto tail = [&](auto ss, f32x16 (&S)[2]) __attribute__((always_inline)) {
    static_for<PD>([&](auto f) __attribute__((always_inline)) { read(std::integral_constant<int, NF + decltype(f)::value>{}, ss, ss); });
    __builtin_amdgcn_sched_barrier(0);
    raise();
    exps(std::integral_constant<int, 0>{}, std::integral_constant<int, 8>{}, S);
    __builtin_amdgcn_sched_barrier(0);
    static_for<NV>([&](auto ff) __attribute__((always_inline)) {
      constexpr int F = decltype(ff)::value, gg = F / NDB, db = F % NDB;
      if constexpr (db == 0) fence_p(pf[gg]);
      mfma_s<false, younger(NF + F, NF + NV)>(o[db], v_fragment(std::integral_constant<int, NF + F>{}), pf[gg]);
      read(std::integral_constant<int, NF + F + PD>{}, ss, ss);
      if constexpr (gg < 3) exps(std::integral_constant<int, 8 + 8 * F / NDB>{}, std::integral_constant<int, 8 + 8 * (F + 1) / NDB>{}, S);
      __builtin_amdgcn_sched_barrier(0);
    });
    add_up();
    fence_o();               // (here: the compiler may copy registers where the ways join)
  };
  constexpr std::integral_constant<int, 0> stage0{};
  constexpr std::integral_constant<int, 1> stage1{};
  if (n_tiles > 0) {
    static_for<PD>([&](auto f) __attribute__((always_inline)) { read(f, stage0, stage0); });
    static_for<NF>([&](auto ff) __attribute__((always_inline)) {
      constexpr int F = decltype(ff)::value, ks = F / 2, kb = F % 2;
      if constexpr (ks == 0) mfma_s_first<false, younger(F, NF)>(Sa[kb], fk[F % PD], qf[ks]);
      else mfma_s<false, younger(F, NF)>(Sa[kb], fk[F % PD], qf[ks]);
      if constexpr (F + PD < NF) read(std::integral_constant<int, F + PD>{}, stage0, stage0);
    });
    fence_s(Sa[0], Sa[1]);
    mask(0, Sa);
    static_for<16>([&](auto i) __attribute__((always_inline)) { max_step(i, Sa); });
    if (n_tiles > 1) __syncthreads();          // everybody has read K(0)
    int t = 0;
    for (; t + 2 < n_tiles; t += 2) {
      body(stage0, t, Sa, Sb);
      body(stage1, t + 1, Sb, Sa);
      if ((t & 62) == 62) { l_run += l_lo; l_lo = 0.f; }
    }
    if (t + 1 < n_tiles) {             // (a second way out of the loop would make the compiler copy the output in every round)
      body(stage0, t, Sa, Sb);
      Sa[0] = Sb[0];
      Sa[1] = Sb[1];
#pragma unroll
      for (int db = 0; db < NDB; ++db) va[db] += C::TILE_BYTES;
    }
    tail(stage0, Sa);
  }
  // ---- epilogue
  const float l_mine = l_run + l_lo;
  const float l_tot = l_mine + __shfl_xor(l_mine, 32), r_tot = l_tot + (r_fix + __shfl_xor(r_fix, 32));
  const bool seen = l_tot > 0.f;
  const float wb = seen && r_tot > 0.f ? 1.f / r_tot : 0.f;
  const float lse = seen ? (m_run + __builtin_amdgcn_logf(l_tot)) * kLn2 : -__builtin_inff();
  if (!q_valid) return;
  if (ns > 1) {
    const int64_t rh = (static_cast<int64_t>(share) * p.batch + bi) * T.n_q * p.Hq + q_idx - static_cast<int64_t>(T.q_row0) * p.Hq;
    float* const od = T.part_o + rh * D + 4 * h;
#pragma unroll
    for (int db = 0; db < NDB; ++db)
#pragma unroll
      for (int i4 = 0; i4 < 4; ++i4) {
        f32x4 x;
#pragma unroll
        for (int e = 0; e < 4; ++e) x[e] = o[db][4 * i4 + e] * wb;
        *reinterpret_cast<f32x4*>(od + 32 * db + 8 * i4) = x;
      }
    if (h == 0) T.part_lse[rh] = lse;
  } else {
    __bf16* const od = static_cast<__bf16*>(p.out) + bi * p.q_bstride + q_idx * D + 4 * h;
#pragma unroll
    for (int db = 0; db < NDB; ++db)
#pragma unroll
      for (int i4 = 0; i4 < 4; ++i4) {
        bf16x4 y;
#pragma unroll
        for (int e = 0; e < 4; ++e) y[e] = static_cast<__bf16>(o[db][4 * i4 + e] * wb);
        *reinterpret_cast<bf16x4*>(od + 32 * db + 8 * i4) = y;
      }
    if (h == 0) p.lse[bi * p.lse_bstride + q_idx] = lse;
  }
}

template <int D>
hipError_t launch_variant(const AttnLaunch& p, hipStream_t stream) {
  constexpr int BM = RunCfg<D>::BM;
  RunLaunch r{};
  r.q = p.q; r.k = p.k; r.v = p.v; r.out = p.out_final; r.lse = p.lse_dst;
  r.q_bstride = p.q_bstride; r.kv_bstride = p.kv_bstride; r.lse_bstride = p.lse_bstride;
  r.Hq = p.Hq; r.Hkv = p.Hkv; r.G = p.Hq / p.Hkv;
  r.causal = p.causal; r.n_keys = p.last_key + 1; r.batch = p.batch;
  r.scale_log2e = p.scale * kLog2e;
  int64_t per_unit = 0;
  for (int t = 0; t < p.n_tasks; ++t) {
    const int64_t rows = static_cast<int64_t>(p.task[t].n_q) * r.G, tiles = (rows + BM - 1) / BM;
    if (rows > INT_MAX - BM || p.n_split[t] < 1) return hipErrorInvalidValue;
    if (t == 0) r.items0 = static_cast<int32_t>(std::min<int64_t>(tiles * p.n_split[0], INT_MAX));
    per_unit += tiles * p.n_split[t];
    r.task[t] = {p.task[t].q_row0, p.task[t].n_q, p.task[t].q_pos0, static_cast<int32_t>(rows), static_cast<int32_t>(tiles), p.n_split[t],
                 make_divider(static_cast<uint32_t>(p.n_split[t])), p.part_o[t], p.part_lse[t]};
  }
  const int64_t units = static_cast<int64_t>(p.batch) * p.Hkv;
  if (per_unit == 0 || units == 0) return hipSuccess;
  if (per_unit * units > INT_MAX) return hipErrorInvalidValue;
  const int64_t blocks = xcd_balanced_blocks(units, per_unit);
  if (blocks > INT_MAX) return hipErrorInvalidValue;
  r.map = make_xcd_map(static_cast<int32_t>(units), static_cast<int32_t>(per_unit), xcd_window(D == 64 ? 96 : 64, static_cast<int>(per_unit)));
  r.by_kv_heads = make_divider(static_cast<uint32_t>(r.Hkv));
  r.by_group = make_divider(static_cast<uint32_t>(r.G));
  return TASP_LAUNCH((attn_run_kernel<D>), dim3(static_cast<unsigned>(blocks)), dim3(RunCfg<D>::NTHREADS), stream, r);
}

}  // namespace

hipError_t launch_attn_run(const AttnLaunch& p, int d, hipStream_t stream) {
  if (!attn_run_takes(p, d)) return hipErrorInvalidValue;
  return d == 64 ? launch_variant<64>(p, stream) : launch_variant<128>(p, stream);
}

}  // namespace tasp
