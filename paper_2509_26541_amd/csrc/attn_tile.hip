// Blockwise attention for fp32 inputs of any size and for short bf16 calls: 128 query rows (fp32 with d = 128: 256) per
// workgroup, the keys of a query tile dealt to as many workgroups as it takes to fill the chip.
//
// The large bf16 kernel (attn_bf16.hip) gives a workgroup 256 rows of one head and all its keys; a
// call with a few hundred local rows then runs on a few dozen of the 256 CUs and a workgroup's chain
// of key tiles is the length of the call.  Here the rows of a query tile are (local row, query head
// of the group) pairs, so that grouped heads fill tiles and share K/V, and n_split workgroups each
// take an equal run of the tile's visible keys; launch_combine adds the partial pairs up.
//
// Per wavefront 32 of the tile's rows, S^T = K Q^T and O^T = V^T P^T with v_mfma_f32_32x32x16: one query per lane
// column, so the softmax is in-lane but for one exchange, and the score registers are the B operand of the second
// product as they stand; V through the transposing LDS read, K and V tiles by direct global->LDS loads.
//
// fp32 products are formed from two 16-bit floats each (v_mfma_f32_32x32x16_f16, three for one product; see the loop): a
// matrix instruction of that kind does in 32 cycles what eight fp32 ones do in 512.  The rows of K and V are split where
// they were fetched, in LDS and by the wavefront that fetched them, one tile ahead.  Eight wavefronts share a tile at d = 128:
// with four, a wavefront to a SIMD, twice the splitting and accumulators moved about, 16 heads of 128 took 797 us, not 506.
//
// Joined steps take the keys by position (a tile is a run of neighbouring keys: nothing to look up, the addresses are
// scalar), a step by itself walks its segments.
//
// What bounds it: the issue slots.  fp32 d = 128: 360 vector and 48 matrix instructions for 32 rows by 32 keys, 3 300 cycles of a
// SIMD of which the matrix pipe is busy 1 536; bf16 1 330 of the 1 450 cycles a SIMD takes for 32 rows by 64 keys at
// d = 64; in the shortest calls the launch, the set-up and the latency of the first tiles.  Measured, whole calls:
//   fp32, 16 heads of 128, 2 048 of 16 384 tokens, causal: 0.48 ms (287 TFLOP/s of products of floats) against 1.13 ms with
//     fp32 matrix instructions (their floor is 0.90); error of the output against 64 bits, 2 heads of 128, 5 120 of
//     20 480 tokens: 4.4e-7 against 5.8e-7; no mask, 2 heads of 64, 8 192 of 32 768: 5.3e-7 against 5.8e-7;
//   fp32, 4 heads of 64, 256 of 1 024 tokens: 16 us;
//   bf16, 8 heads of 128, 512 of 4 096 tokens: 23 us against 117 with the large kernel on 16 CUs;
//   bf16, 128 sequences of 3 072 tokens, 20 heads of 64: 0.70 ms (0.72 with the sub-chunks in their order of arrival,
//     0.91 with the large kernel, which pads 192 rows to 256).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <climits>

#include "gfx950.hpp"
#include "internal.hpp"

namespace tasp {
namespace {

constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;
constexpr float kRescaleGap = 8.0f;      // the running max is only raised when it grew by more than 2^8
constexpr float kRescaleGapF32 = 2.0f;   // fp32: 2^2, the probabilities go to 16-bit floats (below 2^16) scaled by 2^kProbExp
constexpr int kProbExp = 13;
constexpr int kSpread = 16;              // fp32: exponents that the rows of a piece of K or V may be apart
constexpr float kNegBig = -1.0e30f;
constexpr int CHUNK = 512;               // keys located at a time
constexpr int RUNS = 512;                // fp32: entries of the table of tiles with something left to the end

template <typename T, int D>
struct TCfg {
  static constexpr bool F32 = sizeof(T) == 4;
  static constexpr int BM = tile_rows(F32, D);          // rows per workgroup, 32 to a wavefront
  static constexpr int NW = BM / 32, NTHREADS = 64 * NW;
  static constexpr int BT = F32 ? 32 : 64;              // keys per tile
  static constexpr int NKB = BT / 32;                   // 32-key blocks
  static constexpr int RB = D * static_cast<int>(sizeof(T));   // bytes of a row
  static constexpr int UNITS = RB / 16;                 // 16-byte units per row
  static constexpr int RPP = NTHREADS / UNITS;          // rows filled per pass
  static constexpr int PASSES = BT / RPP;
  static constexpr int OWN = BT / NW;                   // fp32: rows of a tile that a wavefront fetches and converts, a pair of units a lane
  static constexpr int TILE_BYTES = BT * RB;
  static constexpr int STAGE_BYTES = 2 * TILE_BYTES;    // K tile, V tile
  static constexpr int STAGES = F32 ? 3 : 2;
  static constexpr int RPL = UNITS >= 16 ? 1 : 16 / UNITS;   // rows per 256-byte bank line
  static constexpr int NDB = D / 32;                    // 32-column blocks of O^T
  // bf16: physical unit of logical unit u of row r.  K is read row-wise (32 lanes, one row each, the same
  // unit): neighbouring bank lines differ.  V through the transposing read (4 rows, 2 units).
  __device__ static int swz_k(int r, int u) { return u ^ ((r / RPL) % (UNITS < 16 ? UNITS : 16)); }
  __device__ static int swz_v(int r, int u) { return u ^ (4 * ((r / RPL) % (UNITS / 4))); }
  // fp32: eight columns are two 16-byte units, fetched as eight floats and turned in place into the high halves
  // (unit 0 of the pair) and the low halves (unit 1) of their split.  Pair c of row r sits at pair c ^ x of the
  // row, its units swapped where y is 1: the fragment reads (K: 16 rows, one pair, one unit; V: 4 rows, 4 pairs,
  // one unit) and those of the conversion (neighbouring pairs, one unit) all meet 16 units of a 256-byte line.
  __device__ static int pair_x(bool v, int r) { return v ? 4 * (r & 1) : r & 7; }
  __device__ static int pair_y(bool v, int r, int pair) { return ((v ? r >> 1 : r >> 3) ^ (D == 128 ? pair >> 3 : r)) & 1; }   // pair: the physical one
};

__device__ inline float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }
__device__ inline f32x16 zero16() {
  f32x16 z;
#pragma unroll
  for (int i = 0; i < 16; ++i) z[i] = 0.f;
  return z;
}
// Eight floats times sa and sb (powers of two, for four each) as two sets of eight 16-bit floats, hi + lo = s x to 22 bits and a sign.  In one
// piece of assembly: one instruction for each half (scaled, subtracted, rounded once and packed; the compiler takes
// three for both).  Instructions that write half a register stand four apart from those that read it.
__device__ __forceinline__ void split8(const f32x4& a, const f32x4& b, float sa, float sb, u32x4& hi, u32x4& lo) {
  unsigned h0, h1, h2, h3, l0, l1, l2, l3;
  asm("v_fma_mixlo_f16 %0, %8, %16, 0\n\tv_fma_mixlo_f16 %1, %10, %16, 0\n\tv_fma_mixlo_f16 %2, %12, %17, 0\n\tv_fma_mixlo_f16 %3, %14, %17, 0\n\t"
      "v_fma_mixhi_f16 %0, %9, %16, 0\n\tv_fma_mixhi_f16 %1, %11, %16, 0\n\tv_fma_mixhi_f16 %2, %13, %17, 0\n\tv_fma_mixhi_f16 %3, %15, %17, 0\n\t"
      "v_fma_mixlo_f16 %4, %8, %16, -%0 op_sel_hi:[0,0,1]\n\tv_fma_mixlo_f16 %5, %10, %16, -%1 op_sel_hi:[0,0,1]\n\t"
      "v_fma_mixlo_f16 %6, %12, %17, -%2 op_sel_hi:[0,0,1]\n\tv_fma_mixlo_f16 %7, %14, %17, -%3 op_sel_hi:[0,0,1]\n\t"
      "v_fma_mixhi_f16 %4, %9, %16, -%0 op_sel:[0,0,1] op_sel_hi:[0,0,1]\n\tv_fma_mixhi_f16 %5, %11, %16, -%1 op_sel:[0,0,1] op_sel_hi:[0,0,1]\n\t"
      "v_fma_mixhi_f16 %6, %13, %17, -%2 op_sel:[0,0,1] op_sel_hi:[0,0,1]\n\tv_fma_mixhi_f16 %7, %15, %17, -%3 op_sel:[0,0,1] op_sel_hi:[0,0,1]"
      : "=&v"(h0), "=&v"(h1), "=&v"(h2), "=&v"(h3), "=&v"(l0), "=&v"(l1), "=&v"(l2), "=&v"(l3)
      : "v"(a[0]), "v"(a[1]), "v"(a[2]), "v"(a[3]), "v"(b[0]), "v"(b[1]), "v"(b[2]), "v"(b[3]), "v"(sa), "v"(sb));
  hi = u32x4{h0, h1, h2, h3};
  lo = u32x4{l0, l1, l2, l3};
}
__device__ inline f32x16 mfma_f16(const u32x4& a, const u32x4& b, const f32x16& c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
}
// The largest |x| of eight floats, NaN passed over unless there is nothing else, and m.
__device__ __forceinline__ float abs_max3(float m, float a, float b) {     // (as assembly: the compiler would quiet every input first)
  float r;
  asm("v_max3_f32 %0, %1, abs(%2), abs(%3)" : "=v"(r) : "v"(m), "v"(a), "v"(b));
  return r;
}
__device__ __forceinline__ float abs_max8(const f32x4& a, const f32x4& b, float m) {
  m = abs_max3(abs_max3(m, a[0], a[1]), a[2], a[3]);
  return abs_max3(abs_max3(m, b[0], b[1]), b[2], b[3]);
}
// Exponents, 2^e <= max < 2^(e + 1) and not below kLeastExp, 128 for an infinity, of the largest row of a wavefront's lanes and
// of the smallest one that is not all zeros (127 if all are); W lanes to a row, x their maxima as integers (>= 0: ordered like
// the floats).  Leaves the maximum of every row in its last lane.
constexpr int kLeastExp = -100;
template <int CTRL>
__device__ __forceinline__ int dpp_max(int x) { return max(x, __builtin_amdgcn_update_dpp(0, x, CTRL, 15, 15, true)); }
template <int W>
__device__ __forceinline__ void row_exps(int& x, int& most, int& least) {
  x = dpp_max<0x111>(x);                                 // shifts inside 16 lanes
  x = dpp_max<0x112>(x);
  x = dpp_max<0x114>(x);
  int lo, hi = x;
  if constexpr (W == 16) {
    hi = x = dpp_max<0x118>(x);
    lo = x - 1;
  } else {
    lo = x - 1;                                          // (zero: the largest of all, as an unsigned number)
    hi = dpp_max<0x118>(x);
    lo = static_cast<int>(min(static_cast<unsigned>(lo), static_cast<unsigned>(__builtin_amdgcn_update_dpp(lo, lo, 0x118, 15, 15, false))));
  }
  auto at = [](int v, int l) { return static_cast<unsigned>(__builtin_amdgcn_readlane(v, l)); };
  const unsigned m = max(max(at(hi, 15), at(hi, 31)), max(at(hi, 47), at(hi, 63)));
  const unsigned n = min(min(at(lo, 15), at(lo, 31)), min(at(lo, 47), at(lo, 63)));
  most = max(static_cast<int>(m >> 23) - 127, kLeastExp);
  least = max(min(static_cast<int>(n >> 23) - 127, 127), kLeastExp);
}
__device__ __forceinline__ float pow2(int e) { return __builtin_bit_cast(float, (e + 127) << 23); }     // -126 .. 127
__device__ inline bf16x8 lds_tr8(const unsigned char* lo, const unsigned char* hi) {
  const s16x4 a = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)(lds_void_ptr)const_cast<unsigned char*>(lo));
  const s16x4 b = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)(lds_void_ptr)const_cast<unsigned char*>(hi));
  return __builtin_bit_cast(bf16x8, __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7));
}

// One more (normalised) pair into running sums that are kept unnormalised against their running maximum: the sums are
// multiplied by r, the pair's outputs by w.  Where no share so far saw a key all weights are 0, and so are the outputs unless
// they are NaN (a row of NaN scores has lse = -inf and NaN outputs), which 0 times them keeps.
__device__ inline void fold(float lse, float& mx, float& den, float& r, float& w) {
  const float m = fmaxf(mx, lse), ref = m == -__builtin_inff() ? 0.f : m;
  r = __expf(mx - ref);
  w = __expf(lse - ref);
  den = __builtin_fmaf(den, r, w);
  mx = m;
}

// SERIAL (fp32): a workgroup takes all shares of its tile one after the other and folds their pairs in the output
// itself, as combine_kernel does from memory: the same bits without a workspace.
template <typename T, int D, bool SERIAL>
__global__ __launch_bounds__((TCfg<T, D>::NTHREADS), (D == 64 && !TCfg<T, D>::F32 ? 3 : 2)) void attn_tile_kernel(const AttnLaunch p) {
  using C = TCfg<T, D>;
  constexpr bool F32 = C::F32;
  constexpr int BM = C::BM, NTHREADS = C::NTHREADS, NW = C::NW;
  constexpr int BT = C::BT, NKB = C::NKB, NDB = C::NDB, NJ = C::UNITS / 2;
  __shared__ __attribute__((aligned(16))) unsigned char smem[C::STAGES * C::STAGE_BYTES];
  // fp32: per four rows of a tile (rows 8 i + 4 h ..: entry 4 h + i) the power of two below their largest |K| (less 14) and
  // |V|.  Where a wavefront found infinities: s_vx is infinite, the power is in s_vt, the rows it cleared are in s_bad;
  // s_odd marks the runs of `run` tiles that hold keys to be added at the end.
  __shared__ __attribute__((aligned(16))) float s_kx[C::STAGES][F32 ? 8 : 1], s_vx[C::STAGES][F32 ? 8 : 1], s_vt[C::STAGES][F32 ? 8 : 1];
  __shared__ int s_bad[C::STAGES][NW], s_odd[F32 ? RUNS : 1];
  // One step's launch: global positions of the keys (INT_MAX: none), whether a wavefront fetched a key that some row of the
  // tile must not see, and the effective segments of the tile.
  __shared__ __attribute__((aligned(16))) int s_tok[2 * CHUNK];
  __shared__ __attribute__((aligned(16))) int s_msk[C::STAGES][NW];
  __shared__ int e_vbeg[kMaxSeg + 1];      // start in their concatenation
  __shared__ int e_goff[kMaxSeg];          //   global position minus that
  __shared__ int e_n;
  __shared__ float s_all[SERIAL ? 2 : 1][SERIAL ? NTHREADS : 1];     // SERIAL: running maximum and sum of the shares so far

  const int thread = threadIdx.x, wave_u = __builtin_amdgcn_readfirstlane(thread >> 6);

  // What the set-up needs of the kernel arguments is asked for here, in one go and at fixed places: they
  // come from far (a first dependent read of them costs about as much as a tile).
  const AttnTask t0 = p.task[0], t1 = p.task[1];
  const bool linear = p.all_steps != 0;    // the keys of a tile are one run of positions, from the first key on
  int pair0[2] = {0, 0}, pair1[2] = {0, 0};
  if (!linear) {
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      pair0[e] = p.pool[2 * min(t0.seg0 + (thread & 63), kPoolSeg - 1) + e];
      pair1[e] = p.pool[2 * min(t1.seg0 + (thread & 63), kPoolSeg - 1) + e];
    }
  }

  // ---- which (sequence, KV head, task, row tile, share of the keys)
  const int G = p.Hq / p.Hkv;
  const int m0 = t0.n_q * G, m1 = p.n_tasks > 1 ? t1.n_q * G : 0;
  const int tiles0 = (m0 + BM - 1) / BM, tiles1 = (m1 + BM - 1) / BM;
  const int items0 = tiles0 * (SERIAL ? 1 : p.n_split[0]), per_g = items0 + tiles1 * (SERIAL ? 1 : p.n_split[1]);
  const int w_all = xcd_balanced(blockIdx.x, p.batch * p.Hkv, per_g, xcd_window(F32 ? (D == 64 ? 64 : 32) : D == 64 ? 96 : 64, per_g));
  if (w_all < 0) return;
  const int bg = w_all / per_g;
  int rem = w_all - bg * per_g;
  const int bi = bg / p.Hkv, g = bg - bi * p.Hkv;
  const bool second = rem >= items0;
  if (second) rem -= items0;
  const int ns = second ? p.n_split[1] : p.n_split[0];
  const int per_share = SERIAL ? 1 : ns;
  int share = rem % per_share;
  // under the causal mask the later tiles of a block see more keys: they start first
  const int tile = p.causal ? (second ? tiles1 : tiles0) - 1 - rem / per_share : rem / per_share;
  const int q_row0 = second ? t1.q_row0 : t0.q_row0, q_pos0 = second ? t1.q_pos0 : t0.q_pos0;
  const int n_seg = second ? t1.n_seg : t0.n_seg;
  const int m_all = second ? m1 : m0;
  // The strip of 32 rows a wavefront takes moves with the work item: wavefront i of a workgroup runs on
  // SIMD i, and tiles with few rows left leave strips without work.
  const int strip = (wave_u + w_all) % NW;
  // the lane's row: (local row of the task, query head), its index among the call's (row, head) pairs of the sequence, whether it exists
  struct Row { int row; int64_t idx; bool valid; };
  auto row_of = [&](int column) __attribute__((always_inline)) {
    const int m = tile * BM + strip * 32 + column, mc = min(m, m_all - 1), row = mc / G;
    return Row{row, static_cast<int64_t>(q_row0 + row) * p.Hq + g * G + mc - row * G, m < m_all};
  };
  const Row mine = row_of(thread & 31);
  const int q_pos = p.causal ? q_pos0 + mine.row : INT_MAX - 1;
  const int q_last = q_pos0 + (min(tile * BM + BM, m_all) - 1) / G;
  const int q_first = p.causal ? q_pos0 + tile * BM / G : INT_MAX - 1;   // a key at or before it is seen by every row

  // ---- Q fragments (B operand), bf16: 16-byte units 2 j + h of the lane's row; fp32: units 4 j + 2 h and the one behind it,
  // later the high and the low halves of these eight columns
  u32x4 qf[NJ];
  {
    const u32x4* src = reinterpret_cast<const u32x4*>(static_cast<const T*>(p.q) + bi * p.q_bstride + mine.idx * D) + (thread >> 5 & 1) * (F32 ? 2 : 1);
#pragma unroll
    for (int j = 0; j < NJ; ++j) qf[j] = src[F32 ? 4 * (j / 2) + j % 2 : 2 * j];
  }
  float cq = p.scale * kLog2e;          // fp32: times the power of two that the row was divided by
  bool q_inf = false;                   // fp32: the row holds an infinity

  auto split_q = [&]() __attribute__((always_inline)) {            // fp32: Q to halves
    constexpr int KS = D / 16;
    float m = 0.f;
#pragma unroll
    for (int j = 0; j < KS; ++j) m = abs_max8(__builtin_bit_cast(f32x4, qf[2 * j]), __builtin_bit_cast(f32x4, qf[2 * j + 1]), m);
    m = fmaxf(m, __shfl_xor(m, 32));
    q_inf = m == __builtin_inff();
    if (q_inf) m = 0.f;
    const int e = max((__builtin_bit_cast(int, m) >> 23) - 127, kLeastExp);
    const float s = q_inf ? 0.f : pow2(14 - e);            // (NaN: what comes of infinities is thrown away)
#pragma unroll
    for (int j = 0; j < KS; ++j) split8(__builtin_bit_cast(f32x4, qf[2 * j]), __builtin_bit_cast(f32x4, qf[2 * j + 1]), s, s, qf[2 * j], qf[2 * j + 1]);
    cq *= pow2(e - 14);
  };
  if constexpr (F32 && SERIAL) split_q();

  for (int round = 0; SERIAL ? round < ns : round == 0; ++round) {
  int tid = thread;
  if constexpr (SERIAL) {
    share = round;
    asm volatile("" : "+v"(tid));        // (what follows from it is formed in every round, not kept across the epilogue of the one before)
    if (round > 0) __syncthreads();      // nobody reads the tiles of the share before any more
  }
  const int lane = tid & 63, wave = tid >> 6, h = lane >> 5, lq = lane & 31;
  if constexpr (F32)
    for (int i = tid; i < RUNS; i += NTHREADS) s_odd[i] = 0;
  // ---- the keys.  Joined steps: over them every key of the sequence comes once, so this workgroup's share is a run of
  // positions, n_keys of them from goff on.
  int n_keys, goff = 0, n_eff = 1;
  if (SERIAL || linear) {
    n_keys = p.causal ? q_last + 1 : p.last_key + 1;
    if (ns > 1) {
      const int chunk = ((n_keys + ns - 1) / ns + BT - 1) / BT * BT;
      goff = share * chunk;
      n_keys = max(0, min(n_keys - goff, chunk));
    }
  } else {
    // One step: what the mask leaves of its segments (at most one to a lane) for this tile, laid end to end.
    if (wave == 0) {
      const int a = second ? pair1[0] : pair0[0], e = second ? pair1[1] : pair0[1];
      const int len = lane < n_seg ? max(0, (p.causal ? min(e, q_last + 1) : e) - a) : 0;
      int sl = len;                               // inclusive scan of the lengths
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) { const int t = __shfl_up(sl, o); if (lane >= o) sl += t; }
      const unsigned long long has = __builtin_amdgcn_ballot_w64(len > 0);
      if (len > 0) {
        const int idx = __builtin_popcountll(has & ((1ull << lane) - 1));
        e_vbeg[idx] = sl - len;
        e_goff[idx] = a - (sl - len);
      }
      if (lane == 63) { e_n = __builtin_popcountll(has); e_vbeg[__builtin_popcountll(has)] = sl; }
    }
    __syncthreads();
    n_eff = e_n;
    n_keys = e_vbeg[n_eff];
  }
  const int n_tiles = (n_keys + BT - 1) / BT;
  static_assert(kMaxSeg <= 64, "");

  // ---- positions of the keys of a step, looked up for CHUNK of them at a time: chunk c in half c % 2 of s_tok.
  // With sub-chunks of a few dozen keys most tiles cross a segment boundary; a search per tile and
  // row cost more than the tile's exponentials.
  auto find = [&](int v) __attribute__((always_inline)) {
    int lo = 0, n = n_eff;                                          // the last segment that begins at or before v
    while (n > 1) {
      const int half = n >> 1;
      if (e_vbeg[lo + half] <= v) lo += half;
      n -= half;
    }
    return v < n_keys ? v + e_goff[lo] : INT_MAX;
  };
  auto locate = [&](int chunk) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < CHUNK / NTHREADS; ++i) s_tok[(chunk & 1) * CHUNK + i * NTHREADS + tid] = find(chunk * CHUNK + i * NTHREADS + tid);
  };

  // ---- loader, bf16: this thread fills rows fr + RPP i, physical unit fu of the K and the V tile.  fp32: a
  // wavefront fills the rows that it will convert itself, OWN wave + RPW i.
  constexpr int RPW = 64 / C::UNITS, PASSES = F32 ? C::OWN / RPW : C::PASSES;
  const int fu = tid % C::UNITS;
  auto fill_row = [&](int i, int ln) __attribute__((always_inline)) { return (F32 ? C::OWN * wave_u + RPW * i : RPW * wave_u + C::RPP * i) + ln / C::UNITS; };
  auto column = [&](bool v, int r) __attribute__((always_inline)) {                              // what goes to physical unit fu of row r
    if constexpr (F32) return (2 * (fu / 2 ^ C::pair_x(v, r)) + (fu % 2 ^ C::pair_y(v, r, fu / 2))) * 16;
    else return (v ? C::swz_v(r, fu) : C::swz_k(r, fu)) * 16;
  };
  const unsigned row_bytes = static_cast<unsigned>(p.Hkv) * C::RB;
  const int64_t head0 = (bi * p.kv_bstride + static_cast<int64_t>(g) * D) * static_cast<int64_t>(sizeof(T));
  const unsigned char* Kg = static_cast<const unsigned char*>(p.k) + head0;
  const unsigned char* Vg = static_cast<const unsigned char*>(p.v) + head0;
  const u32x4 k_buf = raw_buffer(Kg), v_buf = raw_buffer(Vg);
  const unsigned k_col = column(false, fill_row(0, lane)), v_col = column(true, fill_row(0, lane));
  static_assert(!F32 || PASSES == 2, "");
  static_assert(F32 || (C::RPP % 16 == 0), "the swizzle of a thread's rows does not depend on the pass");
  // Rows past the end are masked.  A step fetches the first key for them: every row sees that one, so nothing it holds
  // reaches a row that it should not (0 times infinity).  A run of positions fetches its last key, whose products the tile has anyway.
  auto fetch = [&](int t, int stage) __attribute__((always_inline)) {
    unsigned char* dst = smem + stage * C::STAGE_BYTES + wave_u * (F32 ? C::OWN * C::RB : 1024);
    constexpr int PASS_BYTES = F32 ? 1024 : NTHREADS * 16;
    // fp32: the columns of a later pass are those of the first but for a bit (pair_x of K and, at d = 128, pair_y of V);
    // formed here, not held in registers across the loop
    unsigned ck = k_col, cv = v_col;
    int ln = lane;
    if constexpr (F32) asm volatile("" : "+v"(ck), "+v"(cv), "+v"(ln));
    auto k_of = [&](int i) __attribute__((always_inline)) { return F32 ? ck ^ (32u * RPW * i) : ck; };
    auto v_of = [&](int i) __attribute__((always_inline)) { return F32 ? cv ^ (D == 128 ? 16u * i : 0u) : cv; };
    if (linear) {
      // RPW neighbouring rows to a load: their common base is scalar
#pragma unroll
      for (int i = 0; i < PASSES; ++i) {
        const int first = t * BT + (F32 ? C::OWN * wave_u + RPW * i : RPW * wave_u + C::RPP * i);
        unsigned more = static_cast<unsigned>(ln / C::UNITS) * row_bytes;
        int base = first;
        if ((t + 1) * BT > n_keys) {
          base = min(first, n_keys - 1);
          more = static_cast<unsigned>(min(first + ln / C::UNITS, n_keys - 1) - base) * row_bytes;
        }
        base += goff;
        if constexpr (F32) {                                        // tensors may exceed what a 32-bit offset reaches
          const unsigned long long at = static_cast<unsigned long long>(static_cast<unsigned>(base)) * row_bytes;
          global_to_lds_16<true>(Kg + at, more + k_of(i), dst + i * PASS_BYTES);
          global_to_lds_16<true>(Vg + at, more + v_of(i), dst + C::TILE_BYTES + i * PASS_BYTES);
        } else {
          const unsigned at = static_cast<unsigned>(base) * row_bytes;
          buffer_to_lds_16<true>(k_buf, at, more + k_of(i), dst + i * PASS_BYTES);
          buffer_to_lds_16<true>(v_buf, at, more + v_of(i), dst + C::TILE_BYTES + i * PASS_BYTES);
        }
      }
      return;
    }
    int tok[PASSES], last = -1;
#pragma unroll
    for (int i = 0; i < PASSES; ++i) tok[i] = s_tok[(t * BT + fill_row(i, ln)) & (2 * CHUNK - 1)];     // one round trip for all passes
#pragma unroll
    for (int i = 0; i < PASSES; ++i) {
      last = max(last, tok[i]);
      const unsigned key = tok[i] == INT_MAX ? 0u : static_cast<unsigned>(tok[i]);
      if constexpr (F32) {
        const unsigned long long at = static_cast<unsigned long long>(key) * row_bytes;
        global_to_lds_16_far(Kg + (at + k_of(i)), dst + i * PASS_BYTES);
        global_to_lds_16_far(Vg + (at + v_of(i)), dst + C::TILE_BYTES + i * PASS_BYTES);
      } else {                                                      // both factors are below 2^24 (host check)
        const unsigned off = __umul24(key, row_bytes);
        buffer_to_lds_16<true>(k_buf, 0u, off + k_of(i), dst + i * PASS_BYTES);
        buffer_to_lds_16<true>(v_buf, 0u, off + v_of(i), dst + C::TILE_BYTES + i * PASS_BYTES);
      }
    }
    const bool any = __builtin_amdgcn_ballot_w64(last > q_first) != 0;
    if (lane == 0) s_msk[stage][wave] = any ? 1 : 0;
  };
  // whether tile t takes the element-wise mask; and the mask: keys 32 kb + 8 (i / 4) + 4 h + i % 4 of the tile
  auto is_masked = [&](int t, int stage) __attribute__((always_inline)) {
    if (linear) return (t + 1) * BT > n_keys || goff + (t + 1) * BT - 1 > q_first;
    int mk = 0;
#pragma unroll
    for (int i = 0; i < NW / 4; ++i) {
      const i32x4 m4 = *reinterpret_cast<const i32x4*>(&s_msk[stage][4 * i]);
      mk |= m4[0] | m4[1] | m4[2] | m4[3];
    }
    return __builtin_amdgcn_readfirstlane(mk) != 0;
  };
  auto mask_block = [&](int t, int kb, f32x16& S) __attribute__((always_inline)) {
    const int* tok = &s_tok[((t * BT) & (2 * CHUNK - 1)) + 32 * kb + 4 * h];
    const int last = linear ? min(q_pos, goff + n_keys - 1) : q_pos, at = goff + t * BT + 32 * kb + 4 * h;
#pragma unroll
    for (int i4 = 0; i4 < 4; ++i4) {
      i32x4 tk = {at + 8 * i4, at + 8 * i4 + 1, at + 8 * i4 + 2, at + 8 * i4 + 3};
      if (!linear) tk = *reinterpret_cast<const i32x4*>(tok + 8 * i4);
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (tk[e] > last) S[4 * i4 + e] = -__builtin_inff();
    }
  };

  // ---- LDS read addresses inside a stage
  // K: bf16 unit 2 j + h sits at k_adr ^ 32 j; fp32 pair 2 j + h at k_adr ^ 64 j (d = 128: ^ 16 from pair 8 on), the low halves ^ 16
  const int k_adr = lq * C::RB + (F32 ? 32 * (h ^ C::pair_x(false, lq)) + 16 * C::pair_y(false, lq, h ^ C::pair_x(false, lq)) : C::swz_k(lq, h) * 16);
  // V: as in the large kernel; fp32 the high halves of block db at v_adr[0] ^ 128 db (^ 16 from block 2 on), the low halves ^ 16
  int v_adr[F32 ? 1 : NDB];
  {
    const int ga = lane >> 4, jj = lane & 15;
    const int vrow = 4 * (ga >> 1) + (jj >> 2);
#pragma unroll
    for (int db = 0; db < (F32 ? 1 : NDB); ++db) {
      const int u = 4 * db + 2 * (ga & 1) + ((jj & 3) >> 1), pair = u ^ C::pair_x(true, vrow);
      v_adr[db] = C::TILE_BYTES + vrow * C::RB + (F32 ? 32 * pair + 16 * C::pair_y(true, vrow, pair) : C::swz_v(vrow, u) * 16) + 8 * (jj & 1);
    }
  }

  f32x16 o[NDB];
#pragma unroll
  for (int db = 0; db < NDB; ++db) o[db] = zero16();
  // running max (exp2 domain), sum in two levels (the last 64 tiles, everything before: one fp32
  // accumulator would swallow the many small terms behind a few large ones), and what rounding added
  // to the largest probabilities (bf16), as in the large kernel
  float m_run = kNegBig, l_run = 0.f, l_lo = 0.f, r_fix = 0.f;
  const float c = p.scale * kLog2e;

  const bool idle = __builtin_amdgcn_readfirstlane(tile * BM + strip * 32) >= m_all;
  if constexpr (F32) {
    // ---- fp32.  A product a b of floats is formed from their halves as  a_lo b_hi + a_hi b_lo + a_hi b_hi  on the 16-bit
    // matrix pipe, which is sixteen times as fast as the fp32 one.  A half holds 11 bits, and the rows are scaled by
    // powers of two so that the largest value of each piece is in [2^14, 2^15): q by row, K and V by the eight rows a
    // wavefront fetches, p by the piece of V it meets; what is left out, a_lo b_lo and the rounding of lo, is 2^-24 of
    // |a b| and 2^-40 of the largest one.  That is less than the rounding of a sum of fp32 products (relative error of
    // 128-term dot products 1.4e-7 against 2.0e-7), and sixteen products are added up before a sum is rounded.
    //
    // Tile t is converted in place, by the wavefront that fetched it, while tile t - 1 is worked on; tile t + 1 is on its way.
    //
    // Two kinds of keys are cleared, masked and added one by one at the end, from memory: those with an infinity, which has no
    // halves (inf - inf), and those more than 2^kSpread times as large as another of their piece, whose halves would
    // leave the other too few bits.  A row of Q with an infinity is done again key by key.  Tiles with the element-wise mask
    // and a NaN in V, which would come to the rows that do not see its key as 0 times that, are left to the end as a whole.
    constexpr int KS = D / 16, LOADS = 2 * PASSES;       // contraction steps, loads a fetch issues
    static_assert(C::OWN * (D / 8) == 64, "");
    const int run = (n_tiles + RUNS - 1) / RUNS;
    bool odd = false;
    auto mark_odd = [&](int t) __attribute__((always_inline)) {
      odd = true;
      if (lane == 0) s_odd[t / run] = 1;
    };
    f32x4 raw[2][2];
    float conv_s[2];
    int conv_adr[2];
#pragma unroll
    for (int kv = 0; kv < 2; ++kv) {
      const int r = C::OWN * wave + lane / (D / 8), pair = lane % (D / 8);
      conv_adr[kv] = kv * C::TILE_BYTES + r * C::RB + 32 * pair + 16 * C::pair_y(kv, r, pair);
    }
    auto conv_read = [&](int stage, int kv) __attribute__((always_inline)) {
      const unsigned char* st = smem + stage * C::STAGE_BYTES;
      raw[kv][0] = *reinterpret_cast<const f32x4*>(st + conv_adr[kv]);
      raw[kv][1] = *reinterpret_cast<const f32x4*>(st + (conv_adr[kv] ^ 16));
    };
    auto conv_scale = [&](int stage) __attribute__((always_inline)) {
      int mk = __builtin_bit_cast(int, abs_max8(raw[0][0], raw[0][1], 0.f)), mv = __builtin_bit_cast(int, abs_max8(raw[1][0], raw[1][1], 0.f));
      int ek, ev, lk, lv;
      row_exps<D / 8>(mk, ek, lk);
      row_exps<D / 8>(mv, ev, lv);
      const bool bad = max(ek, ev) == 128 || max(ek - lk, ev - lv) > kSpread;
      const int at = C::OWN == 4 ? 4 * (wave & 1) + (wave >> 1) : 4 * (lane & 1) + wave;
      if (__builtin_expect(bad, 0)) {
        int rows = 0;
        unsigned top_k = 0, top_v = 0;
#pragma unroll
        for (int r = 0; r < C::OWN; ++r) {
          const unsigned xk = __builtin_amdgcn_readlane(mk, D / 8 * r + D / 8 - 1), xv = __builtin_amdgcn_readlane(mv, D / 8 * r + D / 8 - 1);
          const int rk = static_cast<int>(xk >> 23) - 127, rv = static_cast<int>(xv >> 23) - 127;
          if (rk == 128 || rv == 128 || rk - lk > kSpread || rv - lv > kSpread) { rows |= 1 << r; continue; }
          top_k = max(top_k, xk);
          top_v = max(top_v, xv);
        }
        ek = max(static_cast<int>(top_k >> 23) - 127, kLeastExp);
        ev = max(static_cast<int>(top_v >> 23) - 127, kLeastExp);
        if (rows >> (lane / (D / 8)) & 1) {
#pragma unroll
          for (int kv = 0; kv < 2; ++kv) raw[kv][0] = raw[kv][1] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
        if (lane < 2) s_vt[stage][at] = pow2(ev);
        if (lane == 0) s_bad[stage][wave] = rows << (C::OWN * wave);
      }
      conv_s[0] = pow2(14 - ek);
      conv_s[1] = pow2(14 - ev);
      if (lane < 2) {                         // (four rows: one entry)
        s_kx[stage][at] = pow2(ek - 14);
        s_vx[stage][at] = bad ? __builtin_inff() : pow2(ev);
      }
    };
    auto conv_write = [&](int stage, int kv) __attribute__((always_inline)) {
      unsigned char* st = smem + stage * C::STAGE_BYTES;
      u32x4 hi, lo;
      split8(raw[kv][0], raw[kv][1], conv_s[kv], conv_s[kv], hi, lo);
      *reinterpret_cast<u32x4*>(st + conv_adr[kv]) = hi;
      *reinterpret_cast<u32x4*>(st + (conv_adr[kv] ^ 16)) = lo;
    };
    auto convert = [&](int stage) __attribute__((always_inline)) {
      conv_read(stage, 0);
      conv_read(stage, 1);
      conv_scale(stage);
      conv_write(stage, 0);
      conv_write(stage, 1);
    };
    if constexpr (!SERIAL) split_q();          // (here its loads have landed)
    // o holds the sums of P V times 2^(kProbExp + 14 - o_exp); o_exp follows the V of the tiles: up with every larger one, down
    // where one is 2^4 smaller, but not more than 2^64 below the largest so far (o may not overflow)
    int o_exp = kLeastExp, o_top = kLeastExp;
    // d = 64 has the registers for a second set of sums, which takes what 16 tiles have added to the first.  Relative error of
    // the output, no mask, 32 768 tokens: 5.9e-7 with one set, 5.3e-7 with two
    constexpr int FLUSH = 16, NSUM = D == 64 ? NDB : 0;
    f32x16 o_sum[NSUM > 0 ? NSUM : 1];
#pragma unroll
    for (int db = 0; db < NSUM; ++db) o_sum[db] = zero16();
    auto scale_sums = [&](float x) __attribute__((always_inline)) {
#pragma unroll
      for (int db = 0; db < NDB; ++db) o[db] *= x;
#pragma unroll
      for (int db = 0; db < NSUM; ++db) o_sum[db] *= x;
    };

    if (n_tiles > 0) {
      if (!linear) {
        locate(0);
        __syncthreads();
      }
      fetch(0, 0);
      if (n_tiles > 1) {
        fetch(1, 1);
        asm volatile("s_waitcnt vmcnt(%0)" :: "n"(LOADS) : "memory");
      } else {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      }
      convert(0);
    }
    int stage = 0;
    for (int t = 0; t < n_tiles; ++t, stage = stage == 2 ? 0 : stage + 1) {
      __syncthreads();               // tile t is converted; nobody reads tile t - 1 any more
      const int next = stage == 2 ? 0 : stage + 1;
      if (t + 2 < n_tiles) {
        fetch(t + 2, next == 2 ? 0 : next + 1);
        asm volatile("s_waitcnt vmcnt(%0)" :: "n"(LOADS) : "memory");     // what this wavefront converts of tile t + 1
      } else {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      }
      // three tiles before a chunk of keys begins: the half of the table it goes to has been left behind
      if (!linear && (t + 3) % (CHUNK / BT) == 0 && t + 3 < n_tiles) locate((t + 3) / (CHUNK / BT));
      const unsigned char* st = smem + stage * C::STAGE_BYTES;
      const f32x4 kx = *reinterpret_cast<const f32x4*>(&s_kx[stage][4 * h]);
      f32x4 vx = *reinterpret_cast<const f32x4*>(&s_vx[stage][4 * h]);
      auto top_exp = [&](const float* x) __attribute__((always_inline)) {
        const f32x4 a = *reinterpret_cast<const f32x4*>(x), b = *reinterpret_cast<const f32x4*>(x + 4);
        const float top = fmaxf(fmaxf(fmaxf(a[0], a[1]), fmaxf(a[2], a[3])), fmaxf(fmaxf(b[0], b[1]), fmaxf(b[2], b[3])));
        return (__builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, top)) >> 23) - 127;
      };
      int e_top = top_exp(&s_vx[stage][0]), bad = 0;
      if (__builtin_expect(e_top == 128, 0)) {
        e_top = kLeastExp;
        for (int w = 0; w < 8; ++w) {
          const float x = s_vx[stage][w] == __builtin_inff() ? s_vt[stage][w] : s_vx[stage][w];
          e_top = max(e_top, (__builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, x)) >> 23) - 127);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (vx[i] == __builtin_inff()) {
            vx[i] = s_vt[stage][4 * h + i];
            bad |= s_bad[stage][C::OWN == 4 ? 2 * i + h : i];
          }
        mark_odd(t);
      }
      const bool masked = is_masked(t, stage);   // by element
      bool leave = idle;
      if (masked && !idle) {                     // a NaN in V
        f16x2 z = {0, 0};
#pragma unroll 2
        for (int i = 0; i < D / 16; ++i) {
          const f16x8 x = *reinterpret_cast<const f16x8*>(st + C::TILE_BYTES + lq * C::RB + 32 * (i + h * (D / 16)) + 16 * C::pair_y(true, lq, i + h * (D / 16)));
#pragma unroll
          for (int e = 0; e < 4; ++e) z = f16x2{x[2 * e], x[2 * e + 1]} * f16x2{0, 0} + z;
        }
        if (__builtin_amdgcn_ballot_w64(!(z[0] == 0 && z[1] == 0)) != 0) {
          mark_odd(t);
          leave = true;
        }
      }
      if (leave) {
        convert(next);
        continue;
      }
      // ---- scores; the floats of tile t + 1 are read and their exponents found beside them
      f32x16 S = zero16();
      // (formed where they are used: held across the loop the fragment addresses are registers too many; the stage is a multiple
      // of what the swizzle moves)
      int ka = k_adr + stage * C::STAGE_BYTES, va = v_adr[0] + stage * C::STAGE_BYTES;
      asm volatile("" : "+v"(ka), "+v"(va));
      constexpr int PK = 2;
      u32x4 k_hi[PK], k_lo[PK];
      auto read_k = [&](auto jj) __attribute__((always_inline)) {
        constexpr int J = decltype(jj)::value;
        // pair 2 J + h: bit 3 of it (d = 128, J >= 4) stands as it is, 256 bytes on, and swaps the units of the pair
        constexpr int lo = 64 * (J % 4) ^ (D == 128 && J >= 4 ? 0 : 16), hi = lo ^ 16, on = J / 4 * 256;
        k_lo[J % PK] = *reinterpret_cast<const u32x4*>(smem + (ka ^ lo) + on);
        k_hi[J % PK] = *reinterpret_cast<const u32x4*>(smem + (ka ^ hi) + on);
      };
      static_for<PK>(read_k);
      __builtin_amdgcn_sched_barrier(0);
      static_for<KS>([&](auto jj) __attribute__((always_inline)) {
        constexpr int J = decltype(jj)::value;
        S = mfma_f16(k_lo[J % PK], qf[2 * J], S);
        if constexpr (J == 0) { conv_read(next, 0); conv_read(next, 1); }
        S = mfma_f16(k_hi[J % PK], qf[2 * J + 1], S);
        S = mfma_f16(k_hi[J % PK], qf[2 * J], S);
        if constexpr (J + PK < KS) read_k(std::integral_constant<int, J + PK>{});
        if constexpr (J == 1) conv_scale(next);
        if constexpr (J >= KS - 2) conv_write(next, J - (KS - 2));
        __builtin_amdgcn_sched_barrier(0);
      });
      // ---- V^T fragments: a block of O^T after the other, for each 16-key group
      constexpr int NV = 2 * NDB, PV = 2;
      u32x4 v_hi[PV], v_lo[PV];
      auto read_v = [&](auto ff) __attribute__((always_inline)) {
        constexpr int F = decltype(ff)::value;
        constexpr int db = F / 2, rows = F % 2 * 16 * C::RB;
        constexpr int xh = 128 * (db % 2) ^ (db >= 2 ? 16 : 0), xl = xh ^ 16, on = db / 2 * 256 + rows;
        v_hi[F % PV] = __builtin_bit_cast(u32x4, lds_tr8(smem + (va ^ xh) + on, smem + (va ^ xh) + on + 8 * C::RB));
        v_lo[F % PV] = __builtin_bit_cast(u32x4, lds_tr8(smem + (va ^ xl) + on, smem + (va ^ xl) + on + 8 * C::RB));
      };
      static_for<PV>(read_v);
      if (masked) mask_block(t, 0, S);
      if (__builtin_expect(__builtin_amdgcn_ballot_w64(bad != 0) != 0, 0)) {
        const int mine = bad >> 4 * h;
#pragma unroll
        for (int i = 0; i < 16; ++i)
          if (mine >> (8 * (i / 4) + i % 4) & 1) S[i] = -__builtin_inff();
      }
      float f[4], mx = -__builtin_inff();
#pragma unroll
      for (int i4 = 0; i4 < 4; ++i4) {
        f[i4] = __builtin_amdgcn_fmed3f(cq * kx[i4], 1.17549435e-38f, 3.402823466e38f);     // (0 and infinite times the mask's -inf and 0 are NaN)
        mx = fmaxf(mx, fmaxf(fmaxf(S[4 * i4], S[4 * i4 + 1]), fmaxf(S[4 * i4 + 2], S[4 * i4 + 3])) * f[i4]);
      }
      int new_exp = o_exp;
      o_top = max(o_top, e_top);
      if (e_top > o_exp) new_exp = e_top;
      else if (e_top < o_exp - 4 && e_top > kLeastExp) new_exp = max(e_top, o_top - 64);
      if (__builtin_amdgcn_ballot_w64(mx > m_run + kRescaleGapF32) != 0 || new_exp != o_exp) {
        const float m_new = fmaxf(m_run, fmaxf(mx, __shfl_xor(mx, 32)));         // both halves of a row agree
        float alpha = fast_exp2(m_run - m_new);
        m_run = m_new;
        l_run *= alpha; l_lo *= alpha;
        alpha *= pow2(max(o_exp - new_exp, -126));
        o_exp = new_exp;
        scale_sums(alpha);
      }
      // ---- probabilities, and their products with the pieces of V; pieces more than 2^6 below the largest, whose
      // probabilities would be left too few bits, in further passes
      float sum[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        S[i] = fast_exp2(__builtin_fmaf(S[i], f[i / 4], -m_run));
        sum[i & 3] += S[i];
      }
      float lim = pow2(max(o_exp - 6, -126)), above = __builtin_inff();
      bool more;
      do {
        more = __builtin_amdgcn_ballot_w64(fminf(fminf(vx[0], vx[1]), fminf(vx[2], vx[3])) < lim) != 0;
        const float p_scale = pow2(kProbExp - o_exp);
        float ps[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) ps[i] = vx[i] * p_scale;
        if (__builtin_expect(more || above < __builtin_inff(), 0)) {
#pragma unroll
          for (int i = 0; i < 4; ++i) ps[i] = vx[i] >= lim && vx[i] < above ? ps[i] : 0.f;
        }
        u32x4 p_hi[2], p_lo[2];
#pragma unroll
        for (int gg = 0; gg < 2; ++gg)
          split8(f32x4{S[8 * gg], S[8 * gg + 1], S[8 * gg + 2], S[8 * gg + 3]}, f32x4{S[8 * gg + 4], S[8 * gg + 5], S[8 * gg + 6], S[8 * gg + 7]},
                 ps[2 * gg], ps[2 * gg + 1], p_hi[gg], p_lo[gg]);
        __builtin_amdgcn_sched_barrier(0);
        // A tile's products are summed for themselves and then added to o, so that the error of the chain of additions grows
        // with the tiles, not with the products.
        f32x16 acc;
        static_for<NV>([&](auto ff) __attribute__((always_inline)) {
          constexpr int F = decltype(ff)::value, gg = F % 2, db = F / 2;
          acc = mfma_f16(v_lo[F % PV], p_hi[gg], gg == 0 ? zero16() : acc);
          acc = mfma_f16(v_hi[F % PV], p_lo[gg], acc);
          acc = mfma_f16(v_hi[F % PV], p_hi[gg], acc);
          if constexpr (F + PV < NV) read_v(std::integral_constant<int, F + PV>{});
          if constexpr (gg == 1) o[db] += acc;
          __builtin_amdgcn_sched_barrier(0);
        });
        if (__builtin_expect(more, 0)) {
          above = lim;
          float top = 0.f;
#pragma unroll
          for (int i = 0; i < 4; ++i) top = fmaxf(top, vx[i] < above ? vx[i] : 0.f);
          top = fmaxf(top, __shfl_xor(top, 32));
          const int e = (__builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, top)) >> 23) - 127;
          if (e <= kLeastExp) break;                       // what is left is zero
          new_exp = max(e, o_top - 64);
          const float up = pow2(min(o_exp - new_exp, 127));
          lim = new_exp > e ? 0.f : pow2(max(e - 6, -126));
          o_exp = new_exp;
          scale_sums(up);
          static_for<PV>(read_v);
        }
      } while (more);
      l_lo += (sum[0] + sum[1]) + (sum[2] + sum[3]);
      if ((t & 63) == 63) { l_run += l_lo; l_lo = 0.f; }
      if (NSUM > 0 && t % FLUSH == FLUSH - 1) {
#pragma unroll
        for (int db = 0; db < NSUM; ++db) { o_sum[db] += o[db]; o[db] = zero16(); }
      }
    }
#pragma unroll
    for (int db = 0; db < NSUM; ++db) o[db] += o_sum[db];
#pragma unroll
    for (int db = 0; db < NDB; ++db) o[db] *= pow2(o_exp - kProbExp - 14);
    // ---- what was left to the end, key by key.  As slow as it is rare: 16 heads of 128, 2 048 of 16 384 tokens, 583 us with
    // one infinite key (559 with none, in the same run), 3.1 ms with every 64th V row 2^20 times as large as the others.
    int late = lane;                 // (addresses formed anew, not kept across the loop)
    asm volatile("" : "+v"(late));
    const f32x4* const qr = reinterpret_cast<const f32x4*>(static_cast<const float*>(p.q) + bi * p.q_bstride + row_of(late & 31).idx * D) + (late >> 5);
    auto add_key = [&](int key, bool wanted) __attribute__((always_inline)) {
      const f32x4* const kk = reinterpret_cast<const f32x4*>(Kg + static_cast<unsigned long long>(key) * row_bytes) + h;
      float dot = 0.f;
#pragma unroll 4
      for (int j = 0; j < D / 8; ++j) {
        const f32x4 a = kk[2 * j], b = qr[2 * j];
#pragma unroll
        for (int e = 0; e < 4; ++e) dot = __builtin_fmaf(a[e], b[e], dot);
      }
      dot += __shfl_xor(dot, 32);
      if (key > q_pos || !wanted) return;
      const float m_new = fmaxf(m_run, dot * c), alpha = fast_exp2(m_run - m_new), pk = fast_exp2(__builtin_fmaf(dot, c, -m_new));
      m_run = m_new;
      l_run *= alpha;
      l_lo = l_lo * alpha + (h == 0 ? pk : 0.f);
      const float* vk = reinterpret_cast<const float*>(Vg + static_cast<unsigned long long>(key) * row_bytes);
#pragma unroll
      for (int i = 0; i < 16; ++i)
#pragma unroll
        for (int db = 0; db < NDB; ++db) o[db][i] = __builtin_fmaf(pk, vk[32 * db + 8 * (i / 4) + 4 * h + i % 4], o[db][i] * alpha);
    };
    const bool any_q_inf = !idle && __builtin_amdgcn_ballot_w64(q_inf) != 0;
    if (any_q_inf && q_inf) {                    // from the start again
      m_run = kNegBig;
      l_run = l_lo = 0.f;
#pragma unroll
      for (int db = 0; db < NDB; ++db) o[db] = zero16();
    }
    if (odd || any_q_inf) {
#pragma unroll 1
      for (int t = 0; t < n_tiles; ++t) {
        // rows of Q with an infinity are settled (NaN) with the first score that is infinite and positive
        const bool redo = any_q_inf && __builtin_amdgcn_ballot_w64(q_inf && l_run + l_lo == l_run + l_lo) != 0;
        const bool look = s_odd[t / run] != 0;
        if (!redo && !look) continue;
        const int v = t * BT + lq, tok = linear ? (v < n_keys ? goff + v : INT_MAX) : find(v);
        unsigned left = 0;
        if (look) {
          const unsigned long long at = static_cast<unsigned long long>(tok != INT_MAX ? tok : linear ? goff + n_keys - 1 : 0) * row_bytes;
          const float* const kr = reinterpret_cast<const float*>(Kg + at) + h * (D / 2);
          const float* const vr = reinterpret_cast<const float*>(Vg + at) + h * (D / 2);
          float mk = 0.f, mv = 0.f, z = 0.f;
#pragma unroll 1
          for (int e = 0; e < D / 2; ++e) {
            mk = abs_max3(mk, kr[e], kr[e]);
            mv = abs_max3(mv, vr[e], vr[e]);
            z = __builtin_fmaf(vr[e], 0.f, z);
          }
          // as in conv_scale: exponents of the row, and of the smallest of its piece
          auto far = [&](float m) __attribute__((always_inline)) {
            const unsigned x = __builtin_bit_cast(int, fmaxf(m, __shfl_xor(m, 32)));
            unsigned least = x - 1;
#pragma unroll
            for (int o = 1; o < C::OWN; o <<= 1) least = min(least, static_cast<unsigned>(__shfl_xor(static_cast<int>(least), o)));
            const int e = static_cast<int>(x >> 23) - 127;
            return e == 128 || e - max(min(static_cast<int>(least >> 23) - 127, 127), kLeastExp) > kSpread;
          };
          const bool far_k = far(mk), far_v = far(mv);
          const unsigned bad = static_cast<unsigned>(__builtin_amdgcn_ballot_w64(far_k || far_v));      // (both halves have the same)
          const unsigned long long nan = __builtin_amdgcn_ballot_w64(!(z == 0.f) && !(bad >> lq & 1));
          const bool masked = __builtin_amdgcn_ballot_w64(tok > q_first) != 0;
          left = masked && nan != 0 ? ~0u : bad;
        }
#pragma unroll 1
        for (int k = 0; k < BT; ++k) {
          const int key = __builtin_amdgcn_readlane(tok, k);
          if (key == INT_MAX) break;               // past the end, as all that follow
          const bool mine = left >> k & 1;
          if (mine || redo) add_key(key, q_inf || mine);
        }
      }
    }
  } else {
  if (n_tiles > 0) {
    if (!linear) {
      locate(0);
      __syncthreads();
    }
    fetch(0, 0);
  }
#pragma unroll
  for (int j = 0; j < NJ; ++j) asm volatile("" : "+v"(qf[j]));      // landed before the loop: its only wait on vector memory is the one on the tile
  for (int t = 0; t < n_tiles; ++t) {
    const int stage = t & 1;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();                 // tile t is complete; nobody reads the other stage any more
    if (t + 1 < n_tiles) fetch(t + 1, stage ^ 1);
    // two tiles before a chunk of keys begins: the half of the table it goes to has been left behind
    if (!linear && (t + 2) % (CHUNK / BT) == 0 && t + 2 < n_tiles) locate((t + 2) / (CHUNK / BT));
    if (idle) continue;
    const unsigned char* st = smem + stage * C::STAGE_BYTES;

    // The matrix instructions of both products take their A operands as streams of fragments read ahead, so
    // that a wavefront alone on its SIMD does not wait for LDS at each of them.
    f32x16 S[NKB];
    {
      constexpr int NF = NKB * NJ, PD = 6;
      bf16x8 ring[PD];
      auto read_k = [&](auto ff) __attribute__((always_inline)) {
        constexpr int F = decltype(ff)::value;
        ring[F % PD] = *reinterpret_cast<const bf16x8*>(st + F / NJ * 32 * C::RB + (k_adr ^ (32 * (F % NJ))));
      };
      static_for<PD>(read_k);
      __builtin_amdgcn_sched_barrier(0);
      static_for<NF>([&](auto ff) __attribute__((always_inline)) {
        constexpr int F = decltype(ff)::value, kb = F / NJ, j = F % NJ;
        if constexpr (j == 0) S[kb] = zero16();
        S[kb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ring[F % PD], __builtin_bit_cast(bf16x8, qf[j]), S[kb], 0, 0, 0);
        if constexpr (F + PD < NF) read_k(std::integral_constant<int, F + PD>{});
        __builtin_amdgcn_sched_barrier(0);
      });
    }
    constexpr int NV = 2 * NKB * NDB, PV = 4;       // bf16 V^T fragments: 16-key group f / NDB, block f % NDB of O^T
    bf16x8 vring[PV];
    auto read_v = [&](auto ff) __attribute__((always_inline)) {
      constexpr int F = decltype(ff)::value;
      const unsigned char* va = st + v_adr[F % NDB] + F / NDB * 16 * C::RB;
      vring[F % PV] = lds_tr8(va, va + 8 * C::RB);
    };
    static_for<PV>(read_v);               // on their way during the maxima
    if (is_masked(t, stage)) {       // by element
#pragma unroll
      for (int kb = 0; kb < NKB; ++kb) mask_block(t, kb, S[kb]);
    }
    float mx = S[0][0];
#pragma unroll
    for (int kb = 0; kb < NKB; ++kb)
#pragma unroll
      for (int i = 0; i < 16; ++i) mx = fmaxf(mx, S[kb][i]);
    if (__builtin_amdgcn_ballot_w64(mx * c > m_run + kRescaleGap) != 0) {
      const float m_new = fmaxf(m_run, fmaxf(mx, __shfl_xor(mx, 32)) * c);     // both halves of a row agree
      const float alpha = fast_exp2(m_run - m_new);
      m_run = m_new;
      l_run *= alpha; l_lo *= alpha; r_fix *= alpha;
#pragma unroll
      for (int db = 0; db < NDB; ++db)
#pragma unroll
        for (int i = 0; i < 16; ++i) o[db][i] *= alpha;
    }
    {
      const float p_top = fast_exp2(__builtin_fmaf(mx, c, -m_run));
      r_fix += static_cast<float>(static_cast<__bf16>(p_top)) - p_top;
    }
    float sum[4] = {0.f, 0.f, 0.f, 0.f};
    auto exps = [&](auto first, auto count) __attribute__((always_inline)) {      // of scores first .. first + count of the 16 NKB a lane holds
#pragma unroll
      for (int i = decltype(first)::value; i < decltype(first)::value + decltype(count)::value; ++i) {
        S[i / 16][i % 16] = fast_exp2(__builtin_fmaf(S[i / 16][i % 16], c, -m_run));
        sum[i & 3] += S[i / 16][i % 16];
      }
    };
    {
      // the exponentials of a 16-key group ride beside the matrix instructions of the group before
      constexpr int PER = 8 / NDB;
      exps(std::integral_constant<int, 0>{}, std::integral_constant<int, 8>{});
      bf16x8 pf;
      static_for<NV>([&](auto ff) __attribute__((always_inline)) {
        constexpr int F = decltype(ff)::value, gg = F / NDB, db = F % NDB;
        if constexpr (db == 0) {
#pragma unroll
          for (int e = 0; e < 8; ++e) pf[e] = static_cast<__bf16>(S[gg / 2][8 * (gg % 2) + e]);
        }
        o[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vring[F % PV], pf, o[db], 0, 0, 0);
        if constexpr (F + PV < NV) read_v(std::integral_constant<int, F + PV>{});
        if constexpr (gg + 1 < 2 * NKB) exps(std::integral_constant<int, 8 * (gg + 1) + PER * db>{}, std::integral_constant<int, PER>{});
        __builtin_amdgcn_sched_barrier(0);
      });
    }
    l_lo += (sum[0] + sum[1]) + (sum[2] + sum[3]);
    if ((t & 63) == 63) { l_run += l_lo; l_lo = 0.f; }
  }
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");     // no fetch may still be writing LDS when the workgroup ends

  // ---- epilogue: normalise and store, 4 consecutive columns a lane and turn
  const float l_mine = l_run + l_lo;
  const float l_tot = l_mine + __shfl_xor(l_mine, 32), r_tot = l_tot + (r_fix + __shfl_xor(r_fix, 32));
  const bool seen = l_tot > 0.f;
  float wb = seen && r_tot > 0.f ? 1.f / r_tot : 0.f;
  float lse_new = seen ? (m_run + __builtin_amdgcn_logf(l_tot)) * kLn2 : -__builtin_inff();
  int late = lane;                   // (the row's place formed anew, not kept across the loop)
  asm volatile("" : "+v"(late));
  const Row to = row_of(late & 31);
  const bool q_valid = to.valid;
  const int64_t ooff = bi * p.o_bstride + to.idx * D, loff = bi * p.lse_bstride + to.idx;
  // columns of register quad q of the lane: block q / 4 of O^T, 32 (q / 4) + 8 (q % 4) + 4 h
  auto quad = [&](auto qq, f32x4& x) __attribute__((always_inline)) {
    constexpr int Q = decltype(qq)::value;
#pragma unroll
    for (int e = 0; e < 4; ++e) x[e] = o[Q / 4][4 * (Q % 4) + e];
    return 32 * (Q / 4) + 8 * (Q % 4) + 4 * h;
  };
  if (SERIAL && ns > 1) {
    float r, w, mx_all = round > 0 ? s_all[0][thread] : -__builtin_inff(), den_all = round > 0 ? s_all[1][thread] : 0.f;
    fold(lse_new, mx_all, den_all, r, w);
    s_all[0][thread] = mx_all;
    s_all[1][thread] = den_all;
    const bool last = round == ns - 1;
    const float inv = den_all > 0.f ? 1.f / den_all : 0.f;
    float* od = static_cast<float*>(p.out_final) + ooff;
    if (q_valid) {
      static_for<D / 8>([&](auto qq) __attribute__((always_inline)) {
        f32x4 x, sum = {0.f, 0.f, 0.f, 0.f};
        const int col = quad(qq, x);
        if (round > 0) sum = *reinterpret_cast<const f32x4*>(od + col);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          x[e] *= wb;
          sum[e] = __builtin_fmaf(w, x[e], sum[e] * r);
          if (last) sum[e] *= inv;
        }
        *reinterpret_cast<f32x4*>(od + col) = sum;
      });
      if (last && h == 0) p.lse_dst[loff] = den_all > 0.f ? mx_all + __logf(den_all) : -__builtin_inff();
    }
  } else if (!q_valid) {
    // nothing
  } else if (p.merge == 0 && (ns > 1 || p.out_final == nullptr)) {
    // a share's pair, or the partial pair of a step
    const int64_t n_q = second ? t1.n_q : t0.n_q;
    const int64_t rh = ns > 1 ? (static_cast<int64_t>(share) * p.batch + bi) * n_q * p.Hq + to.idx - static_cast<int64_t>(q_row0) * p.Hq : 0;
    float* od = ns > 1 ? (second ? p.part_o[1] : p.part_o[0]) + rh * D : p.o_dst + ooff;
    float* ld = ns > 1 ? (second ? p.part_lse[1] : p.part_lse[0]) + rh : p.lse_dst + loff;
    static_for<D / 8>([&](auto qq) __attribute__((always_inline)) {
      f32x4 x;
      const int col = quad(qq, x);
#pragma unroll
      for (int e = 0; e < 4; ++e) x[e] *= wb;
      *reinterpret_cast<f32x4*>(od + col) = x;
    });
    if (h == 0) *ld = lse_new;
  } else if (p.merge == 0) {
    T* od = static_cast<T*>(p.out_final) + ooff;
    static_for<D / 8>([&](auto qq) __attribute__((always_inline)) {
      f32x4 x;
      const int col = quad(qq, x);
      if constexpr (F32) {
#pragma unroll
        for (int e = 0; e < 4; ++e) x[e] *= wb;
        *reinterpret_cast<f32x4*>(od + col) = x;
      } else {
        bf16x4 y;
#pragma unroll
        for (int e = 0; e < 4; ++e) y[e] = static_cast<__bf16>(x[e] * wb);
        *reinterpret_cast<bf16x4*>(od + col) = y;
      }
    });
    if (h == 0) p.lse_dst[loff] = lse_new;
  } else {
    // update_out_lse of Algorithm 3 folded into the store
    float wa = 0.f;
    const float lse_old = p.lse_dst[loff], mxl = fmaxf(lse_old, lse_new);
    if (mxl == -__builtin_inff()) {
      wb = 0.f;
    } else {
      const float ea = __expf(lse_old - mxl), eb = __expf(lse_new - mxl), rden = 1.f / (ea + eb);
      wa = ea * rden;
      wb *= eb * rden;
      lse_new = mxl + __logf(ea + eb);
    }
    float* od = p.o_dst + ooff;
    static_for<D / 8>([&](auto qq) __attribute__((always_inline)) {
      f32x4 x;
      const int col = quad(qq, x);
      const f32x4 old = *reinterpret_cast<const f32x4*>(od + col);
#pragma unroll
      for (int e = 0; e < 4; ++e) x[e] = __builtin_fmaf(wa, old[e], x[e] * wb);
      *reinterpret_cast<f32x4*>(od + col) = x;
    });
    if (h == 0) p.lse_dst[loff] = lse_new;      // (the lane of the other half has read the old one: same wavefront)
  }
  }  // next share (SERIAL)
}

template <typename T, int D, bool SERIAL = false>
hipError_t launch_tile_variant(const AttnLaunch& p, hipStream_t stream) {
  constexpr int BM = TCfg<T, D>::BM;
  if (SERIAL && !p.all_steps) return hipErrorInvalidValue;
  const int64_t G = p.Hq / p.Hkv;
  int64_t per_g = 0;
  for (int t = 0; t < p.n_tasks; ++t) {
    if (p.task[t].n_q * G > INT_MAX - BM || p.n_split[t] < 1) return hipErrorInvalidValue;
    per_g += (p.task[t].n_q * G + BM - 1) / BM * (SERIAL ? 1 : p.n_split[t]);
  }
  const int64_t units = static_cast<int64_t>(p.batch) * p.Hkv;
  if (per_g == 0 || units == 0) return hipSuccess;
  if (per_g * units > INT_MAX) return hipErrorInvalidValue;
  const int64_t blocks = xcd_balanced_blocks(units, per_g);
  if (blocks > INT_MAX) return hipErrorInvalidValue;
  return TASP_LAUNCH((attn_tile_kernel<T, D, SERIAL>), dim3(static_cast<unsigned>(blocks)), dim3(TCfg<T, D>::NTHREADS), stream, p);
}

// The pairs of a row's shares added up as in tasp_lse_merge_many, D / 4 lanes of 4 columns to a (row, head).
// bf16 with more than four shares (SPREAD): a wavefront per (row, head), the shares dealt to its 256 / D groups of
// lanes, eight of a lane's shares requested at once, so that a row costs one or two trips to memory (a share
// at a time, 16 shares of 1 024 rows took 7 us; now 4).  Otherwise a lane takes all shares of its columns; fp32 always,
// one after the other with sixteen requested at once, so that a workgroup that walks the shares itself gets the same sums.
// The rows of every task with shares, one task behind the other.
struct CombineTask {
  const float* o;          // [n, B, n_q, heads, D]
  const float* lse;
  int32_t n, n_q, row0;
  int64_t n_rh;            // B n_q heads
};
struct CombineTasks { CombineTask t[kMaxTasks]; };

template <typename T, int D, bool SPREAD>
__global__ __launch_bounds__(256) void combine_kernel(const CombineTasks tasks, T* __restrict__ out, float* __restrict__ lse_out, int heads, int L) {
  constexpr int PIECES = D / 4, GROUPS = SPREAD ? 64 / PIECES : 1, AT_ONCE = sizeof(T) == 4 ? 16 : SPREAD ? 8 : 4;
  const int lane = threadIdx.x & 63, c = lane % PIECES, grp = SPREAD ? lane / PIECES : 0;
  int64_t i = SPREAD ? static_cast<int64_t>(blockIdx.x) * 4 + (threadIdx.x >> 6)
                     : (static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x) / PIECES;
  const bool second = i >= tasks.t[0].n_rh;
  if (second) i -= tasks.t[0].n_rh;
  const int64_t n_rh = second ? tasks.t[1].n_rh : tasks.t[0].n_rh;
  if (i >= n_rh) return;
  const int n = second ? tasks.t[1].n : tasks.t[0].n, n_q = second ? tasks.t[1].n_q : tasks.t[0].n_q, row0 = second ? tasks.t[1].row0 : tasks.t[0].row0;
  const int64_t stride_lse = n_rh, stride_o = n_rh * D;
  const int64_t bi = i / (static_cast<int64_t>(n_q) * heads);
  const int64_t rh = i + (bi * (L - n_q) + row0) * heads;              // among the call's (row, head) pairs
  const float* op = (second ? tasks.t[1].o : tasks.t[0].o) + i * D + 4 * c;
  const float* lp = (second ? tasks.t[1].lse : tasks.t[0].lse) + i;
  float mx = -__builtin_inff(), den = 0.f;
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
  for (int s0 = grp; s0 < n; s0 += GROUPS * AT_ONCE) {
    float l[AT_ONCE];
    f32x4 x[AT_ONCE];
#pragma unroll
    for (int k = 0; k < AT_ONCE; ++k) {
      const int s = s0 + GROUPS * k;
      l[k] = -__builtin_inff();
      x[k] = f32x4{0.f, 0.f, 0.f, 0.f};
      if (s < n) {
        l[k] = lp[s * stride_lse];
        x[k] = *reinterpret_cast<const f32x4*>(op + s * stride_o);
      }
    }
    if constexpr (sizeof(T) == 4) {
#pragma unroll
      for (int k = 0; k < AT_ONCE; ++k) {
        if (s0 + k < n) {
          float r, w;
          fold(l[k], mx, den, r, w);
#pragma unroll
          for (int e = 0; e < 4; ++e) acc[e] = __builtin_fmaf(w, x[k][e], acc[e] * r);
        }
      }
    } else {
      float m = mx;
#pragma unroll
      for (int k = 0; k < AT_ONCE; ++k) m = fmaxf(m, l[k]);
      const float ref = m == -__builtin_inff() ? 0.f : m;
      const float r = __expf(mx - ref);
      den *= r;
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[e] *= r;
#pragma unroll
      for (int k = 0; k < AT_ONCE; ++k) {
        const float w = __expf(l[k] - ref);
        den += w;
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[e] = __builtin_fmaf(w, x[k][e], acc[e]);
      }
      mx = m;
    }
  }
  if constexpr (sizeof(T) == 4) {
    const float inv = den > 0.f ? 1.f / den : 0.f;
#pragma unroll
    for (int e = 0; e < 4; ++e) acc[e] *= inv;
    *reinterpret_cast<f32x4*>(out + rh * D + 4 * c) = acc;
    if (c == 0) lse_out[rh] = den > 0.f ? mx + __logf(den) : -__builtin_inff();
  } else {
    float m = mx;
#pragma unroll
    for (int o = PIECES; o < PIECES * GROUPS; o <<= 1) m = fmaxf(m, __shfl_xor(m, o));
    const float r = m > -__builtin_inff() ? __expf(mx - m) : 0.f;
    den *= r;
#pragma unroll
    for (int o = PIECES; o < PIECES * GROUPS; o <<= 1) den += __shfl_xor(den, o);
    const float w = den > 0.f ? r / den : 0.f;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      acc[e] *= w;
#pragma unroll
      for (int o = PIECES; o < PIECES * GROUPS; o <<= 1) acc[e] += __shfl_xor(acc[e], o);
    }
    if (grp != 0) return;
    bf16x4 y;
#pragma unroll
    for (int e = 0; e < 4; ++e) y[e] = static_cast<__bf16>(acc[e]);
    *reinterpret_cast<bf16x4*>(out + rh * D + 4 * c) = y;
    if (c == 0) lse_out[rh] = den > 0.f ? m + __logf(den) : -__builtin_inff();
  }
}

template <typename T, int D>
hipError_t launch_combine_variant(const AttnLaunch& p, hipStream_t stream) {
  CombineTasks tasks{};
  int k = 0, most = 0;
  int64_t n_rh = 0;
  for (int t = 0; t < p.n_tasks; ++t) {
    if (p.n_split[t] < 2) continue;
    CombineTask& c = tasks.t[k++];
    c = {p.part_o[t], p.part_lse[t], p.n_split[t], p.task[t].n_q, p.task[t].q_row0, static_cast<int64_t>(p.batch) * p.task[t].n_q * p.Hq};
    n_rh += c.n_rh;
    most = std::max(most, c.n);
  }
  if (n_rh == 0) return hipSuccess;
  const bool spread = sizeof(T) == 2 && most > 4;
  const int64_t L = p.lse_bstride / p.Hq, per_block = spread ? 4 : 1024 / D, blocks = (n_rh + per_block - 1) / per_block;
  if (blocks > INT_MAX) return hipErrorInvalidValue;
  const dim3 grid(static_cast<unsigned>(blocks));
  if constexpr (sizeof(T) == 2)
    if (spread) return TASP_LAUNCH((combine_kernel<T, D, true>), grid, dim3(256), stream, tasks, static_cast<T*>(p.out_final), p.lse_dst, p.Hq, static_cast<int>(L));
  return TASP_LAUNCH((combine_kernel<T, D, false>), grid, dim3(256), stream, tasks, static_cast<T*>(p.out_final), p.lse_dst, p.Hq, static_cast<int>(L));
}

}  // namespace

hipError_t launch_attn_tile(const AttnLaunch& p, int d, bool fp32, bool serial, hipStream_t stream) {
  if (serial && fp32 && d == 64) return launch_tile_variant<float, 64, true>(p, stream);
  if (serial && fp32 && d == 128) return launch_tile_variant<float, 128, true>(p, stream);
  if (serial) return hipErrorInvalidValue;
  if (d == 64) return fp32 ? launch_tile_variant<float, 64>(p, stream) : launch_tile_variant<__bf16, 64>(p, stream);
  if (d == 128) return fp32 ? launch_tile_variant<float, 128>(p, stream) : launch_tile_variant<__bf16, 128>(p, stream);
  return hipErrorInvalidValue;
}

hipError_t launch_combine(const AttnLaunch& p, int d, bool fp32, hipStream_t stream) {
  if (d == 64) return fp32 ? launch_combine_variant<float, 64>(p, stream) : launch_combine_variant<__bf16, 64>(p, stream);
  if (d == 128) return fp32 ? launch_combine_variant<float, 128>(p, stream) : launch_combine_variant<__bf16, 128>(p, stream);
  return hipErrorInvalidValue;
}

}  // namespace tasp
