// Backward pass for fp32 inputs on the fp32 matrix pipe (v_mfma_f32_32x32x2_f32: full fp32 products
// and sums).  The formulas are those of the bf16 kernels:
//   p = exp(scale q.k - lse),  ds = p (dout.v - delta),  dq += scale ds k,  dk += scale ds q,  dv += p dout.
//
// One launch holds two kinds of workgroups, which do not depend on each other:
//   dq:   X = (Q, dout) of 64 (local row, query head of the group) pairs, Y = (K, V) of the keys they see;
//         the keys are dealt to n_split workgroups, whose sums launch_bwd_sum adds up in order;
//   dkv:  X = (K, V) of 64 keys, Y = (Q, dout) of every (local row, head) pair that sees one of them.
// Both form  T1 = Y1 X1^T,  T2 = Y2 X2^T  (scores and dout.v, one X row per lane column),  p and ds from
// them in registers, and  acc1 += Y1^T ds  (dkv: also  acc2 += Y2^T p),  where the score registers are
// the B operand as they stand.  A workgroup is 2 x 2 wavefronts: 32 X rows each, and each half of the
// 64-row Y tile, so that short calls have twice the workgroups that four strips of X rows would give;
// the two halves' sums are added through LDS at the end.  Y tiles arrive by direct global->LDS loads in
// two stages; a tile is read row-wise (T1, T2) and whole rows at a time (acc), swizzled for the former.
//
// What bounds it: the matrix pipe, 64 cycles an instruction, which leaves the issue slots for the rest,
// and in short calls the unequal work of the dk/dv workgroups under the causal mask.  Measured, whole
// call: 8 heads of 64, 514 of 6 168 tokens, causal, 144 us against 5 010 with a wavefront per row.
#include <hip/hip_runtime.h>

#include <climits>

#include "gfx950.hpp"
#include "internal.hpp"
#include "pipeline.hpp"

namespace tasp {
namespace {

constexpr int BX = 64, BT = 64;          // X rows of a workgroup, Y rows of a tile
constexpr int NTHREADS = 256;

template <int D>
struct FCfg {
  static constexpr int RB = 4 * D, UNITS = D / 4;
  static constexpr int RPP = NTHREADS / UNITS, PASSES = BT / RPP;
  static constexpr int TILE_BYTES = BT * RB, STAGE_BYTES = 2 * TILE_BYTES;
  static constexpr int NJ = UNITS / 2, NDB = D / 32;
};

__device__ inline f32x16 mfma(float a, float b, f32x16 c) { return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0); }

__device__ inline float wave_sum(float x) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) x += __shfl_xor(x, o);
  return x;
}

// Columns of register quad Q of an accumulator set (block c, row i of block = column NDB i + c).
template <int NDB, int Q>
__device__ inline int quad(const f32x16 (&o)[NDB], int h, f32x4& x) {
  if constexpr (NDB == 4) {
    x = f32x4{o[0][Q], o[1][Q], o[2][Q], o[3][Q]};
    return 4 * (8 * (Q / 4) + 4 * h + Q % 4);
  } else {
    x = f32x4{o[0][2 * Q], o[1][2 * Q], o[0][2 * Q + 1], o[1][2 * Q + 1]};
    return 2 * (8 * (2 * Q / 4) + 4 * h + (2 * Q) % 4);
  }
}

template <int D, bool DKV>
__device__ __forceinline__ void bwd_tile(const BwdLaunch& p, int block, unsigned char* smem) {
  using C = FCfg<D>;
  constexpr int NJ = C::NJ, NDB = C::NDB, NACC = DKV ? 2 : 1;
  __shared__ __attribute__((aligned(16))) int s_pos[2][BT];      // position of every Y row: key (INT_MAX: none) or query (-1: none)
  __shared__ __attribute__((aligned(256))) float s_lse[2][BT];   // dkv: of the tile's rows
  __shared__ __attribute__((aligned(256))) float s_del[2][BT];
  __shared__ __attribute__((aligned(16))) int s_msk[2][4];       // per wavefront: it fetched a row that takes the element-wise mask
  __shared__ int s_odd[4];                                       // per strip of X rows and half: it left tiles out
  __shared__ int e_vbeg[kMaxSeg + 1], e_goff[kMaxSeg], e_n;      // dq: effective segments of this share of the keys

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, h = lane >> 5, lq = lane & 31;
  // strip of X rows and half of the Y tile, dealt differently in neighbouring workgroups: wavefront i runs on
  // SIMD i, and strips and halves without rows are left out
  const int xs = (wave ^ block) & 1, yg = (wave >> 1 ^ block >> 1) & 1;
  const int G = p.Hq / p.Hkv;
  const Divider group = p.group;
  const int64_t q_pitch = static_cast<int64_t>(p.Hq) * C::RB, k_pitch = static_cast<int64_t>(p.Hkv) * C::RB;

  // ---- the workgroup's X rows
  int bi, g, tsk = 0, share = 0, x_pos, x_lo = 0, x_hi = 0;      // position of the lane's X row, of the first and the last one
  bool x_valid, idle;                                            // idle: no X row of the strip exists
  int64_t x_off;                                                 // byte offset of the lane's X row
  int64_t row_idx = 0;                                           // dq: (row, head) index of it
  if constexpr (!DKV) {
    const int m0 = p.task[0].n_q * G, m1 = p.n_tasks > 1 ? p.task[1].n_q * G : 0;
    const int tiles0 = (m0 + BX - 1) / BX, tiles1 = (m1 + BX - 1) / BX;
    const int per_g = (tiles0 + tiles1) * p.n_split;
    const int w = xcd_balanced(block, p.batch * p.Hkv, per_g);
    if (w < 0) return;
    const int bg = w / per_g;
    int rem = w - bg * per_g;
    bi = bg / p.Hkv; g = bg - bi * p.Hkv;
    tsk = rem >= tiles0 * p.n_split ? 1 : 0;
    if (tsk) rem -= tiles0 * p.n_split;
    share = rem % p.n_split;
    const int tile = p.causal ? (tsk ? tiles1 : tiles0) - 1 - rem / p.n_split : rem / p.n_split;   // more keys first
    const int m_all = tsk ? m1 : m0, m = tile * BX + xs * 32 + lq;
    x_valid = m < m_all;
    idle = tile * BX + xs * 32 >= m_all;
    const int mc = x_valid ? m : m_all - 1, row = mc / G, hq = g * G + mc - row * G;
    const int pos0 = p.task[tsk].q_pos0;
    x_pos = p.causal ? pos0 + row : INT_MAX - 1;
    x_lo = p.causal ? pos0 + tile * BX / G : INT_MAX - 1;
    x_hi = pos0 + (min(tile * BX + BX, m_all) - 1) / G;
    row_idx = bi * p.lse_bstride + static_cast<int64_t>(p.task[tsk].q_row0 + row) * p.Hq + hq;
    x_off = (bi * p.q_bstride + (static_cast<int64_t>(p.task[tsk].q_row0 + row) * p.Hq + hq) * D) * 4;
  } else {
    const int total = p.rng_vbeg[p.n_rng], tiles = (total + BX - 1) / BX;
    const int w = xcd_balanced(block, p.batch * p.Hkv, tiles);
    if (w < 0) return;
    const int bg = w / tiles, v0 = (w - bg * tiles) * BX;         // ranges come by position: under the mask by falling work
    bi = bg / p.Hkv; g = bg - bi * p.Hkv;
    auto token_of = [&](int v) __attribute__((always_inline)) {
      int t = 0;
      for (int j = 0; j < p.n_rng; ++j)
        if (v >= p.rng_vbeg[j] && v < p.rng_vbeg[j + 1]) t = p.rng_start[j] + (v - p.rng_vbeg[j]);
      return t;
    };
    const int v = v0 + xs * 32 + lq;
    x_valid = v < total;
    idle = v0 + xs * 32 >= total;
    x_pos = token_of(x_valid ? v : total - 1);
    x_lo = token_of(v0);
    x_hi = token_of(min(v0 + BX, total) - 1);
    x_off = (bi * p.kv_bstride + (static_cast<int64_t>(x_pos) * p.Hkv + g) * D) * 4;
  }
  u32x4 x1[NJ], x2[NJ];                                          // B operands: 16-byte units 2 j + h of the lane's rows
  {
    const u32x4* s1 = reinterpret_cast<const u32x4*>(static_cast<const unsigned char*>(DKV ? p.k : p.q) + x_off) + h;
    const u32x4* s2 = reinterpret_cast<const u32x4*>(static_cast<const unsigned char*>(DKV ? p.v : p.dout) + x_off) + h;
#pragma unroll
    for (int j = 0; j < NJ; ++j) { x1[j] = s1[2 * j]; x2[j] = s2[2 * j]; }
  }
  // a row that saw no key (lse = -inf) contributes nothing: exp2(-inf) = 0
  auto neg_lse2 = [](float l) __attribute__((always_inline)) { return l > -__builtin_inff() ? -l * kLog2e : -__builtin_inff(); };
  // exp2 of what rounding took from -lse log2(e), the same for every p of a row, less one
  auto lse2_rest = [](float l, float nl2) __attribute__((always_inline)) { return l > -__builtin_inff() ? __builtin_fmaf(-l, kLog2e, -nl2) * kLn2 : 0.f; };
  float x_nl = 0.f, x_del = 0.f, x_rest = 0.f;
  if constexpr (!DKV) { x_nl = neg_lse2(p.lse[row_idx]); x_rest = lse2_rest(p.lse[row_idx], x_nl); x_del = p.delta[row_idx]; }

  // ---- the Y rows: dq a share of the visible keys, dkv the pairs (row, head) of both query blocks from
  // the first row that sees the first key on
  int n_y, y_first[kMaxTasks] = {0, 0}, y_cnt0 = 0;              // dkv: first pair of each block, pairs of the first block
  if constexpr (!DKV) {
    if (wave == 0) {                                             // kMaxSeg = 64 segments at most: one per lane
      const AttnTask& T = p.task[tsk];
      int a = 0, len = 0;
      if (lane < T.n_seg) {
        a = p.pool[2 * (T.seg0 + lane)];
        const int e = p.pool[2 * (T.seg0 + lane) + 1];
        len = max(0, (p.causal ? min(e, x_hi + 1) : e) - a);
      }
      int sl = len;
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) { const int t = __shfl_up(sl, o); if (lane >= o) sl += t; }
      const int total = __shfl(sl, 63);
      const int chunk = ((total + p.n_split - 1) / p.n_split + BT - 1) / BT * BT, lo = share * chunk, hi = min(lo + chunk, total);
      const int beg = sl - len, cb = max(beg, lo), ce = min(sl, hi);
      const unsigned long long has = __builtin_amdgcn_ballot_w64(ce > cb);
      if (ce > cb) {
        const int idx = __builtin_popcountll(has & ((1ull << lane) - 1));
        e_vbeg[idx] = cb - lo;
        e_goff[idx] = a + (cb - beg) - (cb - lo);
      }
      if (lane == 0) { e_n = __builtin_popcountll(has); e_vbeg[e_n] = max(0, hi - lo); }
    }
    __syncthreads();
    n_y = e_vbeg[e_n];
  } else {
    n_y = 0;
#pragma unroll
    for (int b = 0; b < kMaxTasks; ++b) {
      if (b >= p.n_blk) break;
      y_first[b] = (p.causal ? min(max(0, x_lo - p.blk[b].pos0), p.blk[b].n) : 0) * G;
      const int cnt = p.blk[b].n * G - y_first[b];
      if (b == 0) y_cnt0 = cnt;
      n_y += cnt;
    }
  }
  const int n_tiles = (n_y + BT - 1) / BT;

  const int fr = tid / C::UNITS, fu = tid % C::UNITS;
  const int wave_u = __builtin_amdgcn_readfirstlane(wave);
  const unsigned char* Y1 = static_cast<const unsigned char*>(DKV ? p.q : p.k) + (DKV ? bi * p.q_bstride : bi * p.kv_bstride + static_cast<int64_t>(g) * D) * 4;
  const unsigned char* Y2 = static_cast<const unsigned char*>(DKV ? p.dout : p.v) + (DKV ? bi * p.q_bstride : bi * p.kv_bstride + static_cast<int64_t>(g) * D) * 4;
  int seg_j = -1, seg_end = 0, seg_off = 0;                      // dq: the segment of the thread's last row
  // (in registers: a choice between two kernel arguments would become a load, and the wait for it would be one
  // for the tile fetch in flight)
  int row0_a = p.blk[0].row0, row0_b = p.blk[1].row0, pos0_a = p.blk[0].pos0, pos0_b = p.blk[1].pos0;
  asm volatile("" : "+s"(row0_a), "+s"(row0_b), "+s"(pos0_a), "+s"(pos0_b));
  // dkv: pair v of the stream -> local row, head (v >= n_y: row 0 and position -1)
  auto y_row = [&](int v, int& pos, int& hh) __attribute__((always_inline)) {
    const bool second = v >= y_cnt0;
    const int m = second ? y_first[1] + v - y_cnt0 : y_first[0] + v;
    const int r = static_cast<int>(divide(static_cast<uint32_t>(m), group));   // exact up to INT_MAX (a float estimate with one correction is not)
    hh = m - r * G;
    if (v >= n_y) { pos = -1; hh = 0; return 0; }
    pos = p.causal ? (second ? pos0_b : pos0_a) + r : INT_MAX - 1;
    return (second ? row0_b : row0_a) + r;
  };
  auto fetch = [&](int t, int stage) __attribute__((always_inline)) {
    unsigned char* dst = smem + stage * C::STAGE_BYTES + wave_u * 1024;
    bool mask = false;
#pragma unroll
    for (int i = 0; i < C::PASSES; ++i) {
      const int r = fr + C::RPP * i, v = t * BT + r;
      int pos;
      int64_t src;
      if constexpr (!DKV) {
        if (v >= seg_end) {                                      // a thread's rows only move forward
          while (seg_j < e_n && v >= seg_end) { ++seg_j; seg_end = seg_j < e_n ? e_vbeg[seg_j + 1] : INT_MAX; }
          seg_off = seg_j < e_n ? e_goff[seg_j] : 0;
        }
        pos = seg_j < e_n ? v + seg_off : INT_MAX;
        mask |= pos > x_lo;
        src = (pos == INT_MAX ? 0 : pos) * k_pitch;
      } else {
        int hh;
        const int row = y_row(v, pos, hh);
        mask |= pos < x_hi;
        src = row * q_pitch + static_cast<int64_t>(g * G + hh) * C::RB;
      }
      if (fu == 0) s_pos[stage][r] = pos;
      const int col = (fu ^ (r % 16)) * 16;
      global_to_lds_16_far(Y1 + src + col, dst + i * NTHREADS * 16);
      global_to_lds_16_far(Y2 + src + col, dst + C::TILE_BYTES + i * NTHREADS * 16);
    }
    if constexpr (DKV) {
      if (wave_u == 0) {
        int pos, hh;
        const int row = y_row(t * BT + lane, pos, hh);
        const unsigned off = static_cast<unsigned>((static_cast<int64_t>(row) * p.Hq + g * G + hh) * 4);
        global_to_lds_4<true>(reinterpret_cast<const unsigned char*>(p.lse + bi * p.lse_bstride), off, reinterpret_cast<unsigned char*>(&s_lse[stage][0]));
        global_to_lds_4<true>(reinterpret_cast<const unsigned char*>(p.delta + bi * p.lse_bstride), off, reinterpret_cast<unsigned char*>(&s_del[stage][0]));
      }
    }
    const bool any = __builtin_amdgcn_ballot_w64(mask) != 0;
    if (lane == 0) s_msk[stage][wave] = any ? 1 : 0;
  };

  // ---- LDS read addresses inside a stage: row-wise unit 2 j + h of row 32 yg + lq at r_adr ^ 32 j;
  // whole rows: piece lq of row 32 yg + 4 h (+ 8 (r / 4) + r % 4), the swizzle's remaining bits as an XOR
  const int r_adr = (32 * yg + lq) * C::RB + ((h ^ (lq % 16)) * 16);
  const int w_row = (32 * yg + 4 * h) * C::RB;
  const int w_col = NDB == 4 ? (lq ^ (4 * h)) * 16 : ((lq / 2) ^ (4 * h)) * 16 + (lq % 2) * 8;

  f32x16 acc[NACC][NDB];
#pragma unroll
  for (int a = 0; a < NACC; ++a)
#pragma unroll
    for (int db = 0; db < NDB; ++db) acc[a][db] = zero16();
  // dq: what FLUSH tiles have added goes to a second set of sums, so that the error of the chain of additions does not
  // grow with the number of keys.  Relative error of dq, 12 heads of 64, 16 384 tokens of 16 ranks, no mask: 1.05e-6
  // with one set, 5.2e-7 with 8 tiles, 4.7e-7 with 2 (sums over a wavefront's lanes: 7.5e-7); 8 heads, 6 168 tokens: 145 us with either.
  constexpr int FLUSH = 2;
  f32x16 q_sum[DKV ? 1 : NDB];
#pragma unroll
  for (int db = 0; db < (DKV ? 1 : NDB); ++db) q_sum[db] = zero16();
  // Pairs that the mask leaves out, and in the dk/dv workgroups those of query rows that saw no key, have p = 0 and ds = 0.
  // An infinity or NaN of such a Y row would come to the X row as 0 times that: half tiles with such pairs and such
  // a row are left out (a wavefront decides for its own) and added to the stored rows at the end, row by row.
  bool odd_tiles = false;
  const float c = p.scale * kLog2e;

  if (n_tiles > 0) fetch(0, 0);
#pragma unroll
  for (int j = 0; j < NJ; ++j) asm volatile("" : "+v"(x1[j]), "+v"(x2[j]));   // landed before the loop
  asm volatile("" : "+v"(x_nl), "+v"(x_del));
  for (int t = 0; t < n_tiles; ++t) {
    const int stage = t & 1;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();                 // tile t is complete; nobody reads the other stage any more
    if (t + 1 < n_tiles) fetch(t + 1, stage ^ 1);    // (dealt out between the matrix instructions it spills at d = 128)
    if (idle || t * BT + 32 * yg >= n_y) continue;
    const unsigned char* st1 = smem + stage * C::STAGE_BYTES;
    const unsigned char* st2 = st1 + C::TILE_BYTES;
    // some pair of the half tile has no part (the mask, or a query row that saw no key)
    const i32x4 mk = *reinterpret_cast<const i32x4*>(&s_msk[stage][0]);
    bool apart = __builtin_amdgcn_readfirstlane(mk[0] | mk[1] | mk[2] | mk[3]) != 0;
    if constexpr (DKV) apart |= __builtin_amdgcn_ballot_w64(s_lse[stage][32 * yg + lq] == -__builtin_inff()) != 0;
    // formed where they are used: held across the loop the fragment addresses are registers too many at d = 64
    int rw = r_adr, wc = w_col;
    asm volatile("" : "+v"(rw), "+v"(wc));
    if (apart) {                     // see odd_tiles (looked at here, where few registers are taken)
      float z = DKV ? s_del[stage][32 * yg + lq] * 0.f : 0.f;
#pragma unroll 4
      for (int r = 0; r < 16; ++r) {
        const int at = w_row + (8 * (r / 4) + r % 4) * C::RB + (wc ^ ((8 * (r / 4 % 2) + r % 4) * 16));
        z = add_zero_times<NDB>(st1 + at, z);
        if constexpr (DKV) z = add_zero_times<NDB>(st2 + at, z);
      }
      if (__builtin_amdgcn_ballot_w64(!(z == 0.f)) != 0) { odd_tiles = true; continue; }
    }
    // The matrix instructions as four streams, their A operands read from LDS one or two steps ahead, and the
    // vector work in the shadow of the ones that do not need it: p beside T2, ds beside acc2 (dq: beside acc1,
    // one row ahead).  Left to itself it stood between the streams, where a lone wavefront's matrix pipe is idle
    // (71 % busy at d = 128; this order: see the head of the file).
    // Scores as NP, dout.v as NE chains (more spill), added up where they are used: the error of one
    // long chain was larger than that of sums over a wavefront's lanes (8 heads of 128, 600 of 4 800 tokens: dk 1.29e-6
    // against 1.15e-6; so 1.08e-6, with the rest of lse below; 2 to 4 % of the time).
    constexpr int NP = D / 32, NE = 2;
    f32x16 P = zero16(), E = zero16(), Pc[NP - 1], Ec[NE - 1];
#pragma unroll
    for (int i = 0; i < NP - 1; ++i) Pc[i] = zero16();
#pragma unroll
    for (int i = 0; i < NE - 1; ++i) Ec[i] = zero16();
    auto sum_of = [](const f32x16& x, const auto& more, int r) __attribute__((always_inline)) {
      if constexpr (sizeof(more) == sizeof(x)) return x[r] + more[0][r];
      else return (x[r] + more[0][r]) + (more[1][r] + more[2][r]);
    };
    f32x4 fr_[2];
    auto read_row = [&](auto jj) __attribute__((always_inline)) {              // stream of T1, then of T2
      constexpr int J = decltype(jj)::value;
      fr_[J % 2] = *reinterpret_cast<const f32x4*>((J < NJ ? st1 : st2) + (rw ^ (32 * (J % NJ))));
    };
    f32x4 nl = {0.f, 0.f, 0.f, 0.f};
    static_for<2>(read_row);
    __builtin_amdgcn_sched_barrier(0);
    static_for<2 * NJ>([&](auto jj) __attribute__((always_inline)) {
      constexpr int J = decltype(jj)::value, j = J % NJ;
      const f32x4 a = fr_[J % 2], x = __builtin_bit_cast(f32x4, J < NJ ? x1[j] : x2[j]);
      if constexpr (J < NJ) {
#pragma unroll
        for (int e = 0; e < 4; ++e) { f32x16& to = e % NP ? Pc[e % NP - 1] : P; to = mfma(a[e], x[e], to); }
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) { f32x16& to = e % NE ? Ec[e % NE - 1] : E; to = mfma(a[e], x[e], to); }
      }
      if constexpr (J + 2 < 2 * NJ) read_row(std::integral_constant<int, J + 2>{});
      if constexpr (J > NJ) {
#pragma unroll
        for (int r = (J - NJ - 1) * (16 / NJ); r < (J - NJ) * (16 / NJ); ++r) {
          P[r] = __builtin_amdgcn_exp2f(P[r]);
          if constexpr (DKV) P[r] = __builtin_fmaf(P[r], Pc[0][r], P[r]);
        }
      }
      if constexpr (J >= NJ) {
#pragma unroll
        for (int r = (J - NJ) * (16 / NJ); r < (J - NJ + 1) * (16 / NJ); ++r) {
          const float nl2 = DKV ? neg_lse2(nl[r % 4]) : x_nl;
          P[r] = __builtin_fmaf(sum_of(P, Pc, r), c, nl2);
          if constexpr (DKV) Pc[0][r] = lse2_rest(nl[r % 4], nl2);
        }
      }
      if constexpr (DKV && J >= NJ - 1 && (J + 1 - NJ) * (16 / NJ) % 4 == 0 && J + 1 < 2 * NJ)     // lse of the four rows that come next
        nl = *reinterpret_cast<const f32x4*>(&s_lse[stage][32 * yg + 8 * ((J + 1 - NJ) * (16 / NJ) / 4) + 4 * h]);
      __builtin_amdgcn_sched_barrier(0);
    });
#pragma unroll
    for (int r = 16 - 16 / NJ; r < 16; ++r) {
      P[r] = __builtin_amdgcn_exp2f(P[r]);
      if constexpr (DKV) P[r] = __builtin_fmaf(P[r], Pc[0][r], P[r]);
    }
    if (apart) {
#pragma unroll
      for (int i4 = 0; i4 < 4; ++i4) {
        const i32x4 ps = *reinterpret_cast<const i32x4*>(&s_pos[stage][32 * yg + 8 * i4 + 4 * h]);
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (DKV ? x_pos > ps[e] : ps[e] > x_pos) {
            P[4 * i4 + e] = 0.f;
            E[4 * i4 + e] = 0.f;                 // (an infinity from finite factors as well)
            for (f32x16& x : Ec) x[4 * i4 + e] = 0.f;
          }
      }
    }
    struct Piece { float v[NDB]; };
    Piece piece[2];
    auto read_piece = [&](auto kk) __attribute__((always_inline)) {            // stream of acc2 (dkv), then of acc1
      constexpr int K = decltype(kk)::value, r = K % 16;
      const unsigned char* at = (DKV && K < 16 ? st2 : st1) + w_row + (8 * (r / 4) + r % 4) * C::RB + (wc ^ ((8 * (r / 4 % 2) + r % 4) * 16));
      if constexpr (NDB == 4) {
        const f32x4 v = *reinterpret_cast<const f32x4*>(at);
#pragma unroll
        for (int e = 0; e < 4; ++e) piece[K % 2].v[e] = v[e];
      } else {
        const f32x2 v = *reinterpret_cast<const f32x2*>(at);
        piece[K % 2].v[0] = v[0]; piece[K % 2].v[1] = v[1];
      }
    };
    f32x4 dl = {0.f, 0.f, 0.f, 0.f};
    static_for<2>(read_piece);
    if constexpr (DKV) dl = *reinterpret_cast<const f32x4*>(&s_del[stage][32 * yg + 4 * h]);
    else E[0] = P[0] * (sum_of(E, Ec, 0) - x_del);
    __builtin_amdgcn_sched_barrier(0);
    static_for<16 * NACC>([&](auto kk) __attribute__((always_inline)) {
      constexpr int K = decltype(kk)::value, r = K % 16, A = DKV && K < 16 ? 1 : 0;
      const Piece y = piece[K % 2];
#pragma unroll
      for (int db = 0; db < NDB; ++db) acc[A * (NACC - 1)][db] = mfma(y.v[db], A ? P[r] : E[r], acc[A * (NACC - 1)][db]);
      if constexpr (K + 2 < 16 * NACC) read_piece(std::integral_constant<int, K + 2>{});
      if constexpr (DKV) {
        if constexpr (K < 16) E[r] = P[r] * (sum_of(E, Ec, r) - dl[r % 4]);
        if constexpr (K < 15 && r % 4 == 3) dl = *reinterpret_cast<const f32x4*>(&s_del[stage][32 * yg + 8 * ((r + 1) / 4) + 4 * h]);
      } else if constexpr (K < 15) {
        E[r + 1] = P[r + 1] * (sum_of(E, Ec, r + 1) - x_del);
      }
      __builtin_amdgcn_sched_barrier(0);
    });
    if constexpr (!DKV) {
      if (t % FLUSH == FLUSH - 1) {
#pragma unroll
        for (int db = 0; db < NDB; ++db) { q_sum[db] += acc[0][db]; acc[0][db] = zero16(); }
      }
    }
  }
  if constexpr (!DKV) {
#pragma unroll
    for (int db = 0; db < NDB; ++db) acc[0][db] += q_sum[db];
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();                   // the stages are free: the second half of the Y rows hands its sums over

  f32x4* hand = reinterpret_cast<f32x4*>(smem) + xs * (NACC * NDB * 4 * 64) + lane;
  if (lane == 0) s_odd[2 * xs + yg] = odd_tiles ? 1 : 0;
  if (yg == 1) {
#pragma unroll
    for (int a = 0; a < NACC; ++a)
#pragma unroll
      for (int db = 0; db < NDB; ++db)
#pragma unroll
        for (int i4 = 0; i4 < 4; ++i4)
          hand[((a * NDB + db) * 4 + i4) * 64] = f32x4{acc[a][db][4 * i4], acc[a][db][4 * i4 + 1], acc[a][db][4 * i4 + 2], acc[a][db][4 * i4 + 3]};
  }
  __syncthreads();
  if (yg == 1) return;
#pragma unroll
  for (int a = 0; a < NACC; ++a)
#pragma unroll
    for (int db = 0; db < NDB; ++db)
#pragma unroll
      for (int i4 = 0; i4 < 4; ++i4) {
        const f32x4 o = hand[((a * NDB + db) * 4 + i4) * 64];
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[a][db][4 * i4 + e] += o[e];
      }
  if (!x_valid) {
    // nothing
  } else if constexpr (DKV) {
    float* dk = reinterpret_cast<float*>(static_cast<unsigned char*>(p.dk) + x_off);
    float* dv = reinterpret_cast<float*>(static_cast<unsigned char*>(p.dv) + x_off);
    static_for<D / 8>([&](auto qq) __attribute__((always_inline)) {
      f32x4 a, b;
      const int col = quad<NDB, decltype(qq)::value>(acc[0], h, a);
      quad<NDB, decltype(qq)::value>(acc[NACC - 1], h, b);
#pragma unroll
      for (int e = 0; e < 4; ++e) a[e] *= p.scale;
      *reinterpret_cast<f32x4*>(dk + col) = a;
      *reinterpret_cast<f32x4*>(dv + col) = b;
    });
  } else {
    float* dq = (p.n_split > 1 ? p.part_dq + share * p.part_stride : p.dq_acc) + x_off / 4;
    static_for<D / 8>([&](auto qq) __attribute__((always_inline)) {
      f32x4 a;
      const int col = quad<NDB, decltype(qq)::value>(acc[0], h, a);
      f32x4 old = {0.f, 0.f, 0.f, 0.f};
      if (p.accumulate) old = *reinterpret_cast<const f32x4*>(dq + col);
#pragma unroll
      for (int e = 0; e < 4; ++e) a[e] = x_nl == -__builtin_inff() ? old[e] : __builtin_fmaf(__builtin_fmaf(a[e], x_rest, a[e]), p.scale, old[e]);     // (a row that saw no key: 0)
      *reinterpret_cast<f32x4*>(dq + col) = a;
    });
  }
  if (__builtin_amdgcn_readfirstlane(s_odd[2 * xs] | s_odd[2 * xs + 1]) == 0) return;

  // The half tiles that were left out: an X row after the other, a pair at a time, added to the rows stored above.  As
  // slow as it is rare.
  __threadfence_block();
  const float* const f1 = reinterpret_cast<const float*>(Y1);
  const float* const f2 = reinterpret_cast<const float*>(Y2);
  constexpr int CPL = D / 64;
  // position, and offset in floats from Y1 and Y2, of row v of the stream; dkv: and of its lse and delta
  auto y_at = [&](int v, int& pos, int64_t& at) __attribute__((always_inline)) {
    at = 0;
    if constexpr (!DKV) {
      pos = INT_MAX;
      for (int j = 0; j < e_n; ++j)
        if (v >= e_vbeg[j] && v < e_vbeg[j + 1]) pos = v + e_goff[j];
      return (pos == INT_MAX ? 0 : pos) * (k_pitch / 4);
    } else {
      int hh;
      const int row = y_row(v, pos, hh);
      at = bi * p.lse_bstride + static_cast<int64_t>(row) * p.Hq + g * G + hh;
      return row * (q_pitch / 4) + static_cast<int64_t>(g * G + hh) * D;
    }
  };
#pragma unroll 1
  for (int t = 0; t < n_tiles; ++t) {
    int pos;
    int64_t at;
    const int64_t mine = y_at(t * BT + lane, pos, at);
    const bool masked = __builtin_amdgcn_ballot_w64(DKV ? pos < x_hi : pos > x_lo) != 0;
    const unsigned long long no_key = __builtin_amdgcn_ballot_w64(DKV && p.lse[at] == -__builtin_inff());
    if (!masked && no_key == 0) continue;
    float z = DKV ? p.delta[at] * 0.f : 0.f;
#pragma unroll 1
    for (int e = 0; e < D; ++e) {
      z = __builtin_fmaf(f1[mine + e], 0.f, z);
      if constexpr (DKV) z = __builtin_fmaf(f2[mine + e], 0.f, z);
    }
    const unsigned long long odd = __builtin_amdgcn_ballot_w64(!(z == 0.f));
#pragma unroll 1
    for (int half = 0; half < 2; ++half) {
      if (static_cast<unsigned>(odd >> 32 * half) == 0 || !(masked || static_cast<unsigned>(no_key >> 32 * half) != 0)) continue;
      const int v_end = min(t * BT + 32 * half + 32, n_y);
#pragma unroll 1
      for (int src = 0; src < 32; ++src) {
        if (__shfl(x_valid ? 1 : 0, src) == 0) break;
        const int pos_a = __shfl(x_pos, src);
        const int64_t xo = (static_cast<int64_t>(__shfl(static_cast<int>(x_off >> 32), src)) << 32 | static_cast<unsigned>(__shfl(static_cast<int>(x_off), src))) / 4 + lane;
        const float nl_a = __shfl(x_nl, src), rest_a = __shfl(x_rest, src), del_a = __shfl(x_del, src);
        float xa[CPL], xb[CPL], sa[CPL], sb[CPL];
#pragma unroll
        for (int e = 0; e < CPL; ++e) {
          xa[e] = static_cast<const float*>(DKV ? p.k : p.q)[xo + 64 * e];
          xb[e] = static_cast<const float*>(DKV ? p.v : p.dout)[xo + 64 * e];
          sa[e] = sb[e] = 0.f;
        }
#pragma unroll 1
        for (int v = t * BT + 32 * half; v < v_end; ++v) {
          const int64_t y = y_at(v, pos, at) + lane;
          const float l = DKV ? p.lse[at] : 0.f, nl = DKV ? neg_lse2(l) : nl_a;
          if ((DKV ? pos_a > pos : pos > pos_a) || nl == -__builtin_inff()) continue;
          float ya[CPL], yb[CPL], s1 = 0.f, s2 = 0.f;
#pragma unroll
          for (int e = 0; e < CPL; ++e) {
            ya[e] = f1[y + 64 * e];
            yb[e] = f2[y + 64 * e];
            s1 = __builtin_fmaf(xa[e], ya[e], s1);
            s2 = __builtin_fmaf(xb[e], yb[e], s2);
          }
          float pr = __builtin_amdgcn_exp2f(__builtin_fmaf(wave_sum(s1), c, nl));
          pr = __builtin_fmaf(pr, DKV ? lse2_rest(l, nl) : rest_a, pr);
          const float ds = pr * (wave_sum(s2) - (DKV ? p.delta[at] : del_a));
#pragma unroll
          for (int e = 0; e < CPL; ++e) {
            sa[e] = __builtin_fmaf(ds, ya[e], sa[e]);
            sb[e] = __builtin_fmaf(pr, yb[e], sb[e]);
          }
        }
        float* const d1 = (DKV ? static_cast<float*>(p.dk) : p.n_split > 1 ? p.part_dq + share * p.part_stride : p.dq_acc) + xo;
#pragma unroll
        for (int e = 0; e < CPL; ++e) {
          d1[64 * e] = __builtin_fmaf(sa[e], p.scale, d1[64 * e]);
          if constexpr (DKV) static_cast<float*>(p.dv)[xo + 64 * e] += sb[e];
        }
      }
    }
  }
}

// d = 128 needs more than 256 registers (two stationary and two accumulated operands of 64 each): one
// wavefront per SIMD, whose instructions the 64-cycle matrix instructions hide.
template <int D>
__global__ __launch_bounds__(NTHREADS, D == 64 ? 2 : 1) void bwd_fp32_kernel(const BwdLaunch p, int n_dq) {
  __shared__ __attribute__((aligned(16))) unsigned char smem[2 * FCfg<D>::STAGE_BYTES];
  if (static_cast<int>(blockIdx.x) < n_dq) bwd_tile<D, false>(p, blockIdx.x, smem);
  else bwd_tile<D, true>(p, blockIdx.x - n_dq, smem);
}

template <int D>
__global__ __launch_bounds__(256) void bwd_delta_fp32_kernel(const float* __restrict__ out, const float* __restrict__ dout,
                                                             float* __restrict__ delta, int64_t n_rows) {
  constexpr int LPR = D / 4;                     // lanes per (row, head)
  const int64_t idx = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x, row = idx / LPR;
  float s = 0.f;
  if (row < n_rows) {
    const f32x4 a = *reinterpret_cast<const f32x4*>(out + 4 * idx), b = *reinterpret_cast<const f32x4*>(dout + 4 * idx);
#pragma unroll
    for (int e = 0; e < 4; ++e) s = __builtin_fmaf(a[e], b[e], s);
  }
#pragma unroll
  for (int m = LPR / 2; m >= 1; m >>= 1) s += __shfl_xor(s, m);
  if (row < n_rows && idx - row * LPR == 0) delta[row] = s;
}

// dst = sum of the n arrays of n4 x 4 floats, one behind the other, in order
template <typename T>
__global__ __launch_bounds__(256) void bwd_sum_kernel(const float* __restrict__ parts, int64_t stride, int n, T* __restrict__ dst, int64_t n4) {
  const int64_t i = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
  if (i >= n4) return;
  f32x4 s = *reinterpret_cast<const f32x4*>(parts + 4 * i);
#pragma unroll 4
  for (int k = 1; k < n; ++k) {
    const f32x4 x = *reinterpret_cast<const f32x4*>(parts + k * stride + 4 * i);
#pragma unroll
    for (int e = 0; e < 4; ++e) s[e] += x[e];
  }
  if constexpr (sizeof(T) == 4) {
    *reinterpret_cast<f32x4*>(dst + 4 * i) = s;
  } else {
    bf16x4 r;
#pragma unroll
    for (int e = 0; e < 4; ++e) r[e] = static_cast<__bf16>(s[e]);
    *reinterpret_cast<bf16x4*>(dst + 4 * i) = r;
  }
}

}  // namespace

hipError_t launch_bwd_fp32(const BwdLaunch& p, int d, bool dq, bool dkv, hipStream_t stream) {
  const int64_t units = static_cast<int64_t>(p.batch) * p.Hkv, G = p.Hq / p.Hkv;
  int64_t n_dq = 0, n_dkv = 0;
  if (dq) {
    int64_t per_g = 0;
    for (int t = 0; t < p.n_tasks; ++t) {
      if (p.task[t].n_q * G > INT_MAX - BX) return hipErrorInvalidValue;
      per_g += (p.task[t].n_q * G + BX - 1) / BX * p.n_split;
    }
    if (per_g * units > INT_MAX) return hipErrorInvalidValue;
    n_dq = per_g > 0 ? xcd_balanced_blocks(units, per_g) : 0;      // a multiple of 8: the XCD of a block does not move
  }
  if (dkv) {
    const int64_t tiles = (static_cast<int64_t>(p.rng_vbeg[p.n_rng]) + BX - 1) / BX;
    for (int b = 0; b < p.n_blk; ++b)
      if (p.blk[b].n * G * p.n_blk > INT_MAX - BT) return hipErrorInvalidValue;
    if (tiles * units > INT_MAX) return hipErrorInvalidValue;
    n_dkv = tiles > 0 ? xcd_balanced_blocks(units, tiles) : 0;
  }
  if (n_dq + n_dkv == 0) return hipSuccess;
  if (n_dq + n_dkv > INT_MAX) return hipErrorInvalidValue;
  const dim3 grid(static_cast<unsigned>(n_dq + n_dkv));
  if (d == 128) return TASP_LAUNCH((bwd_fp32_kernel<128>), grid, dim3(NTHREADS), stream, p, static_cast<int>(n_dq));
  if (d == 64) return TASP_LAUNCH((bwd_fp32_kernel<64>), grid, dim3(NTHREADS), stream, p, static_cast<int>(n_dq));
  return hipErrorInvalidValue;
}

hipError_t launch_bwd_sum(const float* parts, int64_t stride, int n, void* dst, bool bf16, int64_t n_elems, hipStream_t stream) {
  const int64_t blocks = (n_elems / 4 + 255) / 256;
  if (blocks == 0) return hipSuccess;
  if (blocks > INT_MAX) return hipErrorInvalidValue;
  const dim3 grid(static_cast<unsigned>(blocks));
  if (bf16) return TASP_LAUNCH((bwd_sum_kernel<__bf16>), grid, dim3(256), stream, parts, stride, n, static_cast<__bf16*>(dst), n_elems / 4);
  return TASP_LAUNCH((bwd_sum_kernel<float>), grid, dim3(256), stream, parts, stride, n, static_cast<float*>(dst), n_elems / 4);
}

hipError_t launch_bwd_delta_fp32(const void* out, const void* dout, float* delta, int64_t n_rows, int d,
                                 hipStream_t stream) {
  if (n_rows == 0) return hipSuccess;
  const int64_t blocks = (n_rows * (d / 4) + 255) / 256;
  if (blocks > INT_MAX) return hipErrorInvalidValue;
  const float* o = static_cast<const float*>(out);
  const float* g = static_cast<const float*>(dout);
  if (d == 128) return TASP_LAUNCH((bwd_delta_fp32_kernel<128>), dim3(static_cast<unsigned>(blocks)), dim3(256), stream, o, g, delta, n_rows);
  if (d == 64) return TASP_LAUNCH((bwd_delta_fp32_kernel<64>), dim3(static_cast<unsigned>(blocks)), dim3(256), stream, o, g, delta, n_rows);
  return hipErrorInvalidValue;
}

}  // namespace tasp
