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
// fp32 products are formed from three bf16 each (six products for one; see the loop): exact to the last bit or so whatever the
// range of the inputs, and six bf16 matrix instructions take 192 cycles where eight fp32 ones take 512.  The rows of K and V
// are split by the wavefront that fetched them, one tile ahead.  Eight wavefronts share a tile at d = 128: each splits
// an eighth of it.
//
// Joined steps take the keys by position (a tile is a run of neighbouring keys: nothing to look up, the addresses are
// scalar), a step by itself walks its segments.
//
// What bounds it: fp32 d = 128: the matrix pipe, 96 instructions or 3 072 of the 4 600 cycles a SIMD takes for 32 rows by 32 keys,
// beside some 400 vector instructions that two wavefronts in step do not always hide; bf16: the issue slots, 1 330 of the 1 450
// cycles a SIMD takes for 32 rows by 64 keys at d = 64; in the shortest calls the launch, the set-up and the latency of the
// first tiles.  Measured, whole calls:
//   fp32, 16 heads of 128, 2 048 of 16 384 tokens, causal: 0.67 ms (206 TFLOP/s of products of floats; the floor of six
//     products 0.44) against 1.13 ms with fp32 matrix instructions (0.90); two 16-bit floats to a value took 0.48 but hold a
//     narrow range only.  Error of the output against 64 bits: 2.9e-7 (fp32 instructions 5.2e-7, 16-bit floats 3.7e-7);
//     no mask, 4 heads of 64, 3 072 of 24 576 tokens: 4.1e-7 (5.7e-7, 4.9e-7);
//   fp32, 4 heads of 64, 256 of 1 024 tokens: 16 us;
//   bf16, 8 heads of 128, 512 of 4 096 tokens: 23 us against 117 with the large kernel on 16 CUs;
//   bf16, 128 sequences of 3 072 tokens, 20 heads of 64: 0.70 ms (0.72 with the sub-chunks in their order of arrival,
//     0.91 with the large kernel, which pads 192 rows to 256).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <climits>

#include "gfx950.hpp"
#include "internal.hpp"
#include "pipeline.hpp"

namespace tasp {
namespace {

constexpr float kLog2eLow = 1.92596298909e-8f;      // what kLog2e leaves of log2(e)
constexpr float kRescaleGapF32 = 2.0f;   // fp32: 2^2, see kHuge
constexpr int kHuge = (104 + 127) << 23; // fp32: bits of 2^104.  Rows with a value that large are left to the end, see the loop
constexpr float kVScale = 65536.f;       // fp32: V is taken times 2^16
constexpr float kLn2Low = -1.904654323e-9f;          // and kLn2 of ln(2)
constexpr int CHUNK = 512;               // keys located at a time
constexpr int RUNS = 512;                // fp32: entries of the table of tiles with something left to the end

template <typename T, int D>
struct TCfg {
  static constexpr bool F32 = sizeof(T) == 4;
  static constexpr int BM = tile_rows(F32, D);          // rows per workgroup, 32 to a wavefront
  static constexpr int NW = BM / 32, NTHREADS = 64 * NW;
  static constexpr int BT = F32 ? 32 : 64;              // keys per tile
  static constexpr int NKB = BT / 32;                   // 32-key blocks
  static constexpr int RB = D * static_cast<int>(sizeof(T));   // bytes of a row in memory
  static constexpr int LB = 2 * D;                      // bytes of a row in LDS (fp32: of one of its three pieces)
  static constexpr int UNITS = LB / 16;                 // 16-byte units of it
  static constexpr int RPP = NTHREADS / UNITS;          // bf16: rows filled per pass
  static constexpr int PASSES = BT / RPP;
  static constexpr int OWN = BT / NW;                   // fp32: rows of a tile that a wavefront fetches and converts, eight columns a lane
  static constexpr int PLANES = F32 ? 3 : 1;            // pieces of a value, each kind in a tile of its own
  static constexpr int PLANE_BYTES = BT * LB;
  static constexpr int TILE_BYTES = PLANES * PLANE_BYTES;
  static constexpr int STAGE_BYTES = 2 * TILE_BYTES;    // K tile, V tile
  static constexpr int STAGES = 2;
  static constexpr int RAW_BYTES = F32 ? 2 * BT * RB : 0;   // fp32: rows of K and V as fetched, behind the stages
  static constexpr int RPL = UNITS >= 16 ? 1 : 16 / UNITS;   // rows per 256-byte bank line
  static constexpr int NDB = D / 32;                    // 32-column blocks of O^T
  // Physical unit of logical unit u of row r.  K is read row-wise (32 lanes, one row each, the same
  // unit): neighbouring bank lines differ.  V through the transposing read (4 rows, 2 units).
  __device__ static int swz_k(int r, int u) { return u ^ ((r / RPL) % (UNITS < 16 ? UNITS : 16)); }
  __device__ static int swz_v(int r, int u) { return u ^ (4 * ((r / RPL) % (UNITS / 4))); }
};

// The lane's number, formed anew: for code off the ordinary way, so that no register holds it for that.
__device__ __forceinline__ int lane_id() {
  int l;
  asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(l));
  return l;
}
// Floats as three bf16 each, x = x1 + x2 + x3 exactly (8 bits each, rounded to nearest, so that the signs of the later ones
// vary): x2 is at most 2^-8 x and x3 2^-16 x.  The next piece of eight floats, which are left with the rest.
__device__ __forceinline__ u32x4 next_piece(f32x4& a, f32x4& b) {
  u32x4 r;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    float x = i < 2 ? a[2 * i] : b[2 * i - 4], y = i < 2 ? a[2 * i + 1] : b[2 * i - 3];
    const bf16x2 h = {static_cast<__bf16>(x), static_cast<__bf16>(y)};
    unsigned u = __builtin_bit_cast(unsigned, h);
    asm("" : "+v"(u));               // (or the compiler rounds x once more, by itself)
    x -= __builtin_bit_cast(float, u << 16);
    y -= __builtin_bit_cast(float, u & 0xffff0000u);
    if (i < 2) { a[2 * i] = x; a[2 * i + 1] = y; } else { b[2 * i - 4] = x; b[2 * i - 3] = y; }
    r[i] = u;
  }
  return r;
}
__device__ inline f32x16 mfma_bf16(const u32x4& a, const u32x4& b, const f32x16& c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
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
// The largest of the 32 integers that each half of a wavefront has (the same ones).
template <int CTRL>
__device__ __forceinline__ int dpp_max(int x) { return max(x, __builtin_amdgcn_update_dpp(0, x, CTRL, 15, 15, true)); }      // (a shift inside 16 lanes)
__device__ __forceinline__ int max32(int x) {
  x = dpp_max<0x118>(dpp_max<0x114>(dpp_max<0x112>(dpp_max<0x111>(x))));
  return max(__builtin_amdgcn_readlane(x, 15), __builtin_amdgcn_readlane(x, 31));
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
  constexpr int BT = C::BT, NKB = C::NKB, NDB = C::NDB, NJ = D / 16;       // NJ: contraction steps of the scores
  __shared__ __attribute__((aligned(16))) unsigned char smem[C::STAGES * C::STAGE_BYTES + C::RAW_BYTES];
  // fp32: the rows of a tile that a wavefront cleared; for runs of `run` tiles, whether they hold such rows (with a tile to a run:
  // which), and whether a tile that is left to the end as a whole.
  __shared__ __attribute__((aligned(16))) int s_bad[F32 ? C::STAGES : 1][NW];
  __shared__ int s_odd[F32 ? RUNS : 1], s_all_odd[F32 ? RUNS : 1];
  __shared__ __attribute__((aligned(16))) int s_qtop[NW];      // fp32: largest |Q| of a wavefront's rows
  __shared__ float s_scale[F32 && D == 128 && !SERIAL ? NTHREADS : 1];      // running maximum that the sums in memory refer to
  // One step's launch: global positions of the keys (INT_MAX: none), whether a wavefront fetched a key that some row of the
  // tile must not see, and the effective segments of the tile.
  __shared__ __attribute__((aligned(16))) int s_tok[2 * CHUNK];
  __shared__ __attribute__((aligned(16))) int s_msk[4][NW];
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

  // ---- Q fragments (B operand), columns 16 j + 8 h .. of the lane's row; fp32: as floats, two of `qf` each, later as three pieces
  u32x4 qf[(F32 ? 2 : 1) * NJ], qp[F32 ? 3 : 1][NJ];
  {
    const u32x4* src = reinterpret_cast<const u32x4*>(static_cast<const T*>(p.q) + bi * p.q_bstride + mine.idx * D) + (thread >> 5 & 1) * (F32 ? 2 : 1);
#pragma unroll
    for (int j = 0; j < (F32 ? 2 : 1) * NJ; ++j) qf[j] = src[F32 ? 4 * (j / 2) + j % 2 : 2 * j];
  }
  unsigned long long q_odd_rows = 0;    // fp32: lanes whose row holds an infinity or a value of 2^104 or more
  auto split_q = [&]() __attribute__((always_inline)) {
    if constexpr (F32) {
      float m = 0.f;
#pragma unroll
      for (int j = 0; j < NJ; ++j) m = abs_max8(__builtin_bit_cast(f32x4, qf[2 * j]), __builtin_bit_cast(f32x4, qf[2 * j + 1]), m);
      const int top = __builtin_bit_cast(int, fmaxf(m, __shfl_xor(m, 32)));
      q_odd_rows = __builtin_amdgcn_ballot_w64(top >= kHuge);
      const int all = max32(top >= kHuge ? 0 : top);
      if ((thread & 63) == 0) s_qtop[wave_u] = all;
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        f32x4 a = __builtin_bit_cast(f32x4, qf[2 * j]), b = __builtin_bit_cast(f32x4, qf[2 * j + 1]);
#pragma unroll
        for (int i = 0; i < 3; ++i) qp[i][j] = next_piece(a, b);
      }
    }
  };
  if constexpr (F32 && SERIAL) split_q();

  for (int round = 0; SERIAL ? round < ns : round == 0; ++round) {
  int tid = thread;
  if constexpr (SERIAL) {
    share = round;
    tid = 64 * wave_u + lane_id();       // (formed anew, and what follows from it, in every round, not kept across the epilogue of the one before)
    if (round > 0) __syncthreads();      // nobody reads the tiles of the share before any more
  }
  const int lane = tid & 63, wave = tid >> 6, h = lane >> 5, lq = lane & 31;
  if constexpr (F32)
    for (int i = tid; i < RUNS; i += NTHREADS) s_odd[i] = s_all_odd[i] = 0;
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
  // (with the segments of a step it comes from LDS: the compiler is told that all lanes have the same)
  const int n_tiles = F32 ? __builtin_amdgcn_readfirstlane((n_keys + BT - 1) / BT) : (n_keys + BT - 1) / BT;
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
  // wavefront fetches the rows that it will convert itself, OWN wave + RPW i, to a place of its own; of a row the even units of
  // four floats first, then the odd ones, so that a lane's eight columns are read without bank conflicts.
  constexpr int UPR = C::RB / 16, RPW = 64 / UPR, PASSES = F32 ? C::OWN / RPW : C::PASSES;
  const int fu = tid % UPR;
  auto fill_row = [&](int i, int ln) __attribute__((always_inline)) { return (F32 ? C::OWN * wave_u + RPW * i : RPW * wave_u + C::RPP * i) + ln / UPR; };
  auto column = [&](bool v, int r) __attribute__((always_inline)) {                              // what goes to physical unit fu of row r
    if constexpr (F32) return (2 * (fu % (UPR / 2)) + fu / (UPR / 2)) * 16;
    else return (v ? C::swz_v(r, fu) : C::swz_k(r, fu)) * 16;
  };
  const unsigned row_bytes = static_cast<unsigned>(p.Hkv) * C::RB;
  const int64_t head0 = (bi * p.kv_bstride + static_cast<int64_t>(g) * D) * static_cast<int64_t>(sizeof(T));
  const unsigned char* Kg = static_cast<const unsigned char*>(p.k) + head0;
  const unsigned char* Vg = static_cast<const unsigned char*>(p.v) + head0;
  const u32x4 k_buf = raw_buffer(Kg), v_buf = raw_buffer(Vg);
  const unsigned k_col = column(false, fill_row(0, lane)), v_col = column(true, fill_row(0, lane));
  static_assert(!F32 || (PASSES == 2 && C::OWN * C::UNITS == 64), "");
  static_assert(F32 || (C::RPP % 16 == 0), "the swizzle of a thread's rows does not depend on the pass");
  // Rows past the end are masked.  A step fetches the first key for them: every row sees that one, so nothing it holds
  // reaches a row that it should not (0 times infinity).  A run of positions fetches its last key, whose products the tile has anyway.
  auto fetch = [&](int t, int stage) __attribute__((always_inline)) {
    unsigned char* dst = smem + (F32 ? C::STAGES * C::STAGE_BYTES + wave_u * 2 * C::OWN * C::RB : stage * C::STAGE_BYTES + wave_u * 1024);
    constexpr int PASS_BYTES = F32 ? 1024 : NTHREADS * 16, V_AT = F32 ? C::OWN * C::RB : C::TILE_BYTES;
    unsigned ck = k_col, cv = v_col;
    int ln = lane;
    if constexpr (F32) asm volatile("" : "+v"(ck), "+v"(ln));        // (formed here, not held in registers across the loop)
    if constexpr (F32) cv = ck;
    if (linear) {
      // RPW neighbouring rows to a load: their common base is scalar
#pragma unroll
      for (int i = 0; i < PASSES; ++i) {
        const int first = t * BT + (F32 ? C::OWN * wave_u + RPW * i : RPW * wave_u + C::RPP * i);
        unsigned more = static_cast<unsigned>(ln / UPR) * row_bytes;
        int base = first;
        if ((t + 1) * BT > n_keys) {
          base = min(first, n_keys - 1);
          more = static_cast<unsigned>(min(first + ln / UPR, n_keys - 1) - base) * row_bytes;
        }
        base += goff;
        if constexpr (F32) {                                        // tensors may exceed what a 32-bit offset reaches
          const unsigned long long at = static_cast<unsigned long long>(static_cast<unsigned>(base)) * row_bytes;
          global_to_lds_16<true>(Kg + at, more + ck, dst + i * PASS_BYTES);
          global_to_lds_16<true>(Vg + at, more + cv, dst + V_AT + i * PASS_BYTES);
        } else {
          const unsigned at = static_cast<unsigned>(base) * row_bytes;
          buffer_to_lds_16<true>(k_buf, at, more + ck, dst + i * PASS_BYTES);
          buffer_to_lds_16<true>(v_buf, at, more + cv, dst + V_AT + i * PASS_BYTES);
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
        global_to_lds_16_far(Kg + (at + ck), dst + i * PASS_BYTES);
        global_to_lds_16_far(Vg + (at + cv), dst + V_AT + i * PASS_BYTES);
      } else {                                                      // both factors are below 2^24 (host check)
        const unsigned off = __umul24(key, row_bytes);
        buffer_to_lds_16<true>(k_buf, 0u, off + ck, dst + i * PASS_BYTES);
        buffer_to_lds_16<true>(v_buf, 0u, off + cv, dst + V_AT + i * PASS_BYTES);
      }
    }
    const bool any = __builtin_amdgcn_ballot_w64(last > q_first) != 0;
    if (lane == 0) s_msk[t & 3][wave] = any ? 1 : 0;
  };
  // whether tile t takes the element-wise mask; and the mask: keys 32 kb + 8 (i / 4) + 4 h + i % 4 of the tile
  auto is_masked = [&](int t) __attribute__((always_inline)) {
    if (linear) return (t + 1) * BT > n_keys || goff + (t + 1) * BT - 1 > q_first;
    int mk = 0;
#pragma unroll
    for (int i = 0; i < NW / 4; ++i) {
      const i32x4 m4 = *reinterpret_cast<const i32x4*>(&s_msk[t & 3][4 * i]);
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
  // K: unit 2 j + h sits at k_adr ^ 32 j; V: block db at v_adr[db], fp32 at v_adr[0] ^ 64 db
  const int k_adr = lq * C::LB + C::swz_k(lq, h) * 16;
  int v_adr[F32 ? 1 : NDB];
  {
    const int ga = lane >> 4, jj = lane & 15;
    const int vrow = 4 * (ga >> 1) + (jj >> 2);
#pragma unroll
    for (int db = 0; db < (F32 ? 1 : NDB); ++db)
      v_adr[db] = C::TILE_BYTES + vrow * C::LB + C::swz_v(vrow, 4 * db + 2 * (ga & 1) + ((jj & 3) >> 1)) * 16 + 8 * (jj & 1);
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
  // LEVELS: sums of many tiles are added up in memory, at the row's place in the call's output or in the pair of its share
  constexpr bool LEVELS = F32 && D == 128 && !SERIAL;
  const bool long_run = LEVELS && n_tiles > kSumTiles;
  int sum_next = kSumTiles;
  struct Place { float *o, *lse; bool valid; };
  auto place_of = [&](int id) __attribute__((always_inline)) {
    const Row to = row_of(id & 31);
    if (ns > 1) {
      const int64_t n_q = second ? t1.n_q : t0.n_q;
      const int64_t rh = (static_cast<int64_t>(share) * p.batch + bi) * n_q * p.Hq + to.idx - static_cast<int64_t>(q_row0) * p.Hq;
      return Place{(second ? p.part_o[1] : p.part_o[0]) + rh * D, (second ? p.part_lse[1] : p.part_lse[0]) + rh, to.valid};
    }
    float* const to_o = p.merge == 0 && p.out_final != nullptr ? static_cast<float*>(p.out_final) : p.o_dst;
    return Place{to_o + bi * p.o_bstride + to.idx * D, p.lse_dst + bi * p.lse_bstride + to.idx, to.valid};
  };
  if constexpr (F32) {
    // ---- fp32.  A float is the sum of three bf16 (next_piece), exactly, and a product a b of floats is formed on the bf16 matrix pipe
    // as  a3 b1 + a2 b2 + a1 b3 + a2 b1 + a1 b2 + a1 b1.  What is left out, a2 b3 + a3 b2 + a3 b3, is at most 2^-24 and
    // typically 2^-27 of a b: every product is as good as rounded to fp32, whatever stands beside it in its row, its column or
    // the tile, since bf16 has the exponents of fp32.  (Two 16-bit floats to a value, three products: 2^-40 of the largest
    // value of a row was lost, so that a column of V 2^30 times as large as the others left these two decimals.)
    // That holds down to 2^-109, below which the third piece begins to lose bits (the pipe keeps subnormals).  For V, whose
    // products go to the output as they are, that is the whole range of floats: it is split times 2^16, and a tile's sums
    // are multiplied by 2^-16.  For K and Q what is lost, 2^-134, is nothing beside a score unless the other factor is near 2^104.
    //
    // Tile t + 1 is split, by the wavefront that fetched it, while tile t is worked on; tile t + 2 is on its way.
    //
    // Keys with an infinity, which has no pieces (inf - inf), or a value of 2^104 or more (2^2 probabilities of it times 2^16 of 32
    // keys stay below 2^128) are masked and added at the end, from memory, and so are those whose K could let a sum of
    // products leave the floats (`huge_k`, by the largest |Q| of the workgroup): a score of minus infinity has no weight, but the
    // smaller products may leave them on the other side.  A row of Q with a value of 2^104 or more is done again.  Tiles with the
    // element-wise mask and a NaN in V, which would come to the rows that do not see its key as 0 times that, are left to the end
    // as a whole.
    const int run = (n_tiles + RUNS - 1) / RUNS;
    bool odd = false;
    auto mark_odd = [&](int* s, int t, int keys) __attribute__((always_inline)) {    // (the same from every wavefront, and each reads what it has written)
      odd = true;
      if (lane == 0) s[t / run] = keys;
    };
    const int conv_row = C::OWN * wave + lane / C::UNITS, conv_unit = lane % C::UNITS;
    const int raw_adr = C::STAGES * C::STAGE_BYTES + wave * 2 * C::OWN * C::RB + lane / C::UNITS * C::RB + conv_unit * 16;
    const int conv_adr[2] = {conv_row * C::LB + C::swz_k(conv_row, conv_unit) * 16, C::TILE_BYTES + conv_row * C::LB + C::swz_v(conv_row, conv_unit) * 16};
    // Rows of K (kv = 0) or V of the fetched tile to pieces.  The rows with a huge value count as if they were not there, their scores
    // are replaced; only what V would bring to 0 times infinity has to go.
    int huge_rows = 0, huge_k = kHuge;
    f32x4 raw[2];
    auto conv_read = [&](int kv) __attribute__((always_inline)) {
#pragma unroll
      for (int e = 0; e < 2; ++e) raw[e] = *reinterpret_cast<const f32x4*>(smem + raw_adr + kv * C::OWN * C::RB + e * (C::RB / 2));
    };
    // The matrix pipe cuts the sum of an instruction off downwards.  Over many tiles that would add up (131 072 keys: the mean of all errors 5e-7 of
    // the output, of an error of 8e-7); so V is taken with the other sign in every other tile, and the tile's sums are subtracted.
    auto v_scale = [](int stage) { return stage == 0 ? kVScale : -kVScale; };
    auto conv_write = [&](int stage, int kv) __attribute__((always_inline)) {
      const unsigned long long huge = __builtin_amdgcn_ballot_w64(__builtin_bit_cast(int, abs_max8(raw[0], raw[1], 0.f)) >= (kv == 0 ? huge_k : kHuge));
      if (kv == 0) huge_rows = 0;
      if (__builtin_expect(huge != 0, 0)) {
        unsigned lo = static_cast<unsigned>(huge), hi = static_cast<unsigned>(huge >> 32);
        asm("" : "+s"(lo), "+s"(hi));          // (as one 64-bit number the compiler compares it with constants from memory)
        int rows = 0;
#pragma unroll
        for (int r = 0; r < C::OWN; ++r) {
          const unsigned half = C::UNITS * r < 32 ? lo : hi;
          rows |= (half >> (C::UNITS * r % 32) & ((1u << C::UNITS) - 1)) != 0 ? 1 << r : 0;
        }
        if (kv == 1 && (rows >> (lane_id() / C::UNITS) & 1)) raw[0] = raw[1] = f32x4{0.f, 0.f, 0.f, 0.f};
        huge_rows |= rows;
      }
      if (kv == 1) {
        raw[0] *= v_scale(stage);
        raw[1] *= v_scale(stage);
        if (lane == 0) s_bad[stage][wave] = huge_rows << (C::OWN * wave);
      }
#pragma unroll
      for (int i = 0; i < 3; ++i) *reinterpret_cast<u32x4*>(smem + stage * C::STAGE_BYTES + conv_adr[kv] + i * C::PLANE_BYTES) = next_piece(raw[0], raw[1]);
    };
    // ... of tile t, all of it, and then the fetch of the next into the place that it leaves.  (What has been written was read.)
    auto convert = [&](int t) __attribute__((always_inline)) {
      conv_read(0);
      conv_write(t & 1, 0);
      conv_read(1);
      conv_write(t & 1, 1);
      if (t + 1 < n_tiles) fetch(t + 1, 0);
    };
    if constexpr (!SERIAL) split_q();          // (here its loads have landed)
    // d = 64 has the registers for a second set of sums, which takes what 16 tiles have added to the first.  With d = 128 the
    // sums of kSumTiles join those of the tiles before in memory, where the row's result goes in the end.  Error of the output, no
    // mask, 524 288 tokens, one launch: d = 64 6.3e-7, d = 128 4.9e-7 (2.3e-6 with one set for all tiles; fp32 matrix
    // instructions, two sets: 9.4e-7, 9.7e-7).
    constexpr int FLUSH = 16, NSUM = D == 64 ? NDB : 0;
    f32x16 o_sum[NSUM > 0 ? NSUM : 1];
#pragma unroll
    for (int db = 0; db < NSUM; ++db) o_sum[db] = zero16();
    // Sums in memory: those at the row's place, which refer to a maximum of their own, and o are added up there (`keep`; o starts
    // again) or in o, to which all else then refers.  A step that is folded into a running pair meets that pair there; its
    // weight is taken from its lse as it stands, and the new keys keep to their own maximum, so that nothing is rounded more.
    const bool from_pair = LEVELS && long_run && p.merge != 0 && !idle;
    auto pair_weight = [&](float lse, float ref) __attribute__((always_inline)) { return fast_exp2(__builtin_fmaf(lse, kLog2e, -ref) + lse * kLog2eLow); };
    auto sums_in_memory = [&](bool keep) __attribute__((always_inline)) {
      const int id = lane_id();
      const Place to = place_of(id);
      const bool first = sum_next == kSumTiles;            // nothing of this launch is there
      float ref = m_run, alpha = 0.f;
      const float lse_old = from_pair ? *to.lse : -__builtin_inff();
      const bool old = lse_old != -__builtin_inff();
      if (!first) {
        const float s = s_scale[64 * wave_u + id];
        ref = fmaxf(s, m_run);
        alpha = fast_exp2(s - ref);
      } else if (old) {
        ref = fmaxf(lse_old * kLog2e, m_run);
        alpha = pair_weight(lse_old, ref);
      }
      const float beta = fast_exp2(m_run - ref);
      if (to.valid && !(q_odd_rows >> id & 1)) {
        static_for<D / 8>([&](auto qq) __attribute__((always_inline)) {
          constexpr int Q = decltype(qq)::value;
          f32x4* const at = reinterpret_cast<f32x4*>(to.o + 32 * (Q / 4) + 8 * (Q % 4) + 4 * (id >> 5));
          f32x4 x = {0.f, 0.f, 0.f, 0.f};
          if (!first || from_pair) x = *at;
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            x[e] = __builtin_fmaf(x[e], alpha, o[Q / 4][4 * (Q % 4) + e] * beta);
            o[Q / 4][4 * (Q % 4) + e] = keep ? 0.f : x[e];
          }
          if (keep) *at = x;
        });
      }
      if (keep) {
        s_scale[64 * wave_u + id] = ref;
      } else {
        m_run = ref;
        l_run *= beta;
        l_lo = l_lo * beta + (old && id < 32 ? pair_weight(lse_old, ref) : 0.f);
      }
    };

    if (n_tiles > 0) {
      if (!linear) {
        locate(0);
        __syncthreads();
      }
      fetch(0, 0);
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      __syncthreads();
      int q_top = 0;
#pragma unroll
      for (int i = 0; i < NW / 4; ++i) {
        const i32x4 x = *reinterpret_cast<const i32x4*>(&s_qtop[4 * i]);
        q_top = max(q_top, max(max(x[0], x[1]), max(x[2], x[3])));
      }
      // |q| < 2^(e + 1), |k| < 2^(119 - e), 128 products: below 2^127
      huge_k = min(kHuge >> 23, 119 + 2 * 127 - (__builtin_amdgcn_readfirstlane(q_top) >> 23)) << 23;
      convert(0);
    }
    for (int t = 0; t < n_tiles; ++t) {
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");      // this wavefront's rows of tile t + 1
      __syncthreads();               // tile t is split; nobody reads tile t - 1 any more
      const int stage = t & 1, next = stage ^ 1;
      // three tiles before a chunk of keys begins: the half of the table it goes to has been left behind
      if (!linear && (t + 3) % (CHUNK / BT) == 0 && t + 3 < n_tiles) locate((t + 3) / (CHUNK / BT));
      const unsigned char* st = smem + stage * C::STAGE_BYTES;
      int bad = 0;
#pragma unroll
      for (int i = 0; i < NW / 4; ++i) {
        const i32x4 b = *reinterpret_cast<const i32x4*>(&s_bad[stage][4 * i]);
        bad |= b[0] | b[1] | b[2] | b[3];
      }
      bad = __builtin_amdgcn_readfirstlane(bad);
      if (__builtin_expect(bad != 0, 0)) mark_odd(s_odd, t, bad);
      const bool masked = is_masked(t);          // by element
      bool leave = idle;
      if (masked && !idle) {                     // a NaN in V
        unsigned top = 0;
#pragma unroll 2
        for (int i = 0; i < D / 16; ++i) {
          const u32x4 x = *reinterpret_cast<const u32x4*>(st + C::TILE_BYTES + lq * C::LB + (i + h * (D / 16)) * 16);
#pragma unroll
          for (int e = 0; e < 4; ++e) top = max(top, max(x[e] << 16 & 0x7fffffffu, x[e] & 0x7fffffffu));
        }
        if (__builtin_amdgcn_ballot_w64(top >= 0x7f810000u) != 0) {
          mark_odd(s_all_odd, t, 1);
          leave = true;
        }
      }
      if (leave) {
        convert(t + 1);
        continue;
      }
      if (LEVELS && __builtin_expect(t >= sum_next, 0)) {
        sums_in_memory(true);
        sum_next = t / kSumTiles * kSumTiles + kSumTiles;
      }
      // ---- scores; tile t + 1 is split beside them
      f32x16 S = zero16();
      // (formed where they are used: held across the loop the fragment addresses are registers too many; the stage is a multiple
      // of what the swizzle moves)
      int ka = k_adr + stage * C::STAGE_BYTES, va = v_adr[0] + stage * C::STAGE_BYTES;
      asm volatile("" : "+v"(ka), "+v"(va));
      // A fragment's place takes that of the next step as soon as its last product is under way.  The products of the first pieces
      // and the others, 2^-8 of them, are summed for themselves: fewer roundings of the large sum.
      u32x4 kf[3];
      auto read_k = [&](auto jj, auto ii) __attribute__((always_inline)) {
        constexpr int J = decltype(jj)::value, I = decltype(ii)::value;
        if constexpr (J < NJ) kf[I] = *reinterpret_cast<const u32x4*>(smem + (ka ^ (32 * J)) + I * C::PLANE_BYTES);
      };
      static_for<3>([&](auto i) __attribute__((always_inline)) { read_k(std::integral_constant<int, 0>{}, i); });
      __builtin_amdgcn_sched_barrier(0);
      f32x16 S_lo = zero16();
      __builtin_amdgcn_s_setprio(1);             // the matrix pipe before the other wavefront's vector work: 2 to 4 % (40 960 tokens, 8 heads of 128, 4.42 -> 4.25 ms)
      static_for<NJ>([&](auto jj) __attribute__((always_inline)) {
        constexpr int J = decltype(jj)::value;
        constexpr std::integral_constant<int, J + 1> on{};
        S_lo = mfma_bf16(kf[2], qp[0][J], S_lo);
        read_k(on, std::integral_constant<int, 2>{});
        S_lo = mfma_bf16(kf[0], qp[2][J], S_lo);
        S_lo = mfma_bf16(kf[0], qp[1][J], S_lo);
        S = mfma_bf16(kf[0], qp[0][J], S);
        read_k(on, std::integral_constant<int, 0>{});
        S_lo = mfma_bf16(kf[1], qp[1][J], S_lo);
        S_lo = mfma_bf16(kf[1], qp[0][J], S_lo);
        read_k(on, std::integral_constant<int, 1>{});
        if constexpr (J == 0) conv_read(0);
        if constexpr (J == 1) { conv_write(next, 0); conv_read(1); }
        if constexpr (J == 2) conv_write(next, 1);
        if constexpr (J == 3) { if (t + 2 < n_tiles) fetch(t + 2, 0); }
        __builtin_amdgcn_sched_barrier(0);
      });
      __builtin_amdgcn_s_setprio(0);
      S += S_lo;
      // ---- V^T fragments: a block of O^T after the other, for each 16-key group
      constexpr int NV = 2 * NDB;
      u32x4 vf[3];
      auto read_v = [&](auto ff, auto ii) __attribute__((always_inline)) {
        constexpr int F = decltype(ff)::value, I = decltype(ii)::value;
        if constexpr (F < NV) {
          const unsigned char* at = smem + (va ^ (64 * (F / 2))) + F % 2 * 16 * C::LB + I * C::PLANE_BYTES;
          vf[I] = __builtin_bit_cast(u32x4, lds_tr8(at, at + 8 * C::LB));
        }
      };
      static_for<3>([&](auto i) __attribute__((always_inline)) { read_v(std::integral_constant<int, 0>{}, i); });
      if (masked) mask_block(t, 0, S);
      if (__builtin_expect(bad != 0, 0)) {
        const int mine = bad >> 4 * h;
#pragma unroll
        for (int i = 0; i < 16; ++i)
          if (mine >> (8 * (i / 4) + i % 4) & 1) S[i] = -__builtin_inff();
      }
      float mx = S[0];
#pragma unroll
      for (int i = 1; i < 16; ++i) mx = fmaxf(mx, S[i]);
      if (__builtin_amdgcn_ballot_w64(mx * c > m_run + kRescaleGapF32) != 0) {
        const float m_new = fmaxf(m_run, fmaxf(mx, __shfl_xor(mx, 32)) * c);     // both halves of a row agree
        const float alpha = fast_exp2(m_run - m_new);
        m_run = m_new;
        l_run *= alpha; l_lo *= alpha;
#pragma unroll
        for (int db = 0; db < NDB; ++db) o[db] *= alpha;
#pragma unroll
        for (int db = 0; db < NSUM; ++db) o_sum[db] *= alpha;
      }
      // ---- probabilities, those of the second 16 keys beside the first products with V
      float sum[4] = {0.f, 0.f, 0.f, 0.f};
      u32x4 pf[2][3];
      auto probs = [&](auto g2) __attribute__((always_inline)) {
        constexpr int GG = decltype(g2)::value;
#pragma unroll
        for (int i = 8 * GG; i < 8 * GG + 8; ++i) {
          S[i] = fast_exp2(__builtin_fmaf(S[i], c, -m_run));
          sum[i & 3] += S[i];
        }
        f32x4 a = {S[8 * GG], S[8 * GG + 1], S[8 * GG + 2], S[8 * GG + 3]}, b = {S[8 * GG + 4], S[8 * GG + 5], S[8 * GG + 6], S[8 * GG + 7]};
#pragma unroll
        for (int i = 0; i < 3; ++i) pf[GG][i] = next_piece(a, b);
      };
      probs(std::integral_constant<int, 0>{});
      __builtin_amdgcn_sched_barrier(0);
      // A tile's products are summed for themselves and then added to o, so that the error of the chain of additions grows
      // with the tiles, not with the products.
      f32x16 acc;
      const float v_back = 1.f / kVScale * (stage == 0 ? 1.f : -1.f);
      __builtin_amdgcn_s_setprio(1);
      static_for<NV>([&](auto ff) __attribute__((always_inline)) {
        constexpr int F = decltype(ff)::value, gg = F % 2, db = F / 2;
        constexpr std::integral_constant<int, F + 1> on{};
        acc = mfma_bf16(vf[2], pf[gg][0], gg == 0 ? zero16() : acc);
        read_v(on, std::integral_constant<int, 2>{});
        acc = mfma_bf16(vf[0], pf[gg][2], acc);
        acc = mfma_bf16(vf[0], pf[gg][1], acc);
        acc = mfma_bf16(vf[0], pf[gg][0], acc);
        read_v(on, std::integral_constant<int, 0>{});
        acc = mfma_bf16(vf[1], pf[gg][1], acc);
        acc = mfma_bf16(vf[1], pf[gg][0], acc);
        read_v(on, std::integral_constant<int, 1>{});
        if constexpr (F == 0) probs(std::integral_constant<int, 1>{});
        if constexpr (gg == 1) {
#pragma unroll
          for (int i = 0; i < 16; ++i) o[db][i] = __builtin_fmaf(acc[i], v_back, o[db][i]);
        }
        __builtin_amdgcn_sched_barrier(0);
      });
      __builtin_amdgcn_s_setprio(0);
      l_lo += (sum[0] + sum[1]) + (sum[2] + sum[3]);
      if ((t & 63) == 63) { l_run += l_lo; l_lo = 0.f; }
      if (NSUM > 0 && t % FLUSH == FLUSH - 1) {
#pragma unroll
        for (int db = 0; db < NSUM; ++db) { o_sum[db] += o[db]; o[db] = zero16(); }
      }
    }
#pragma unroll
    for (int db = 0; db < NSUM; ++db) o[db] += o_sum[db];
    if (LEVELS && !idle && (sum_next > kSumTiles || from_pair)) sums_in_memory(false);
    // ---- what was left to the end, four keys at a time.  16 heads of 128, 2 048 of 16 384 tokens: 0.99 ms with
    // one V row in 64 infinite (0.78 without, in the same run; key by key 3.2), 14 ms with all V beyond 2^104.
    const int late = lane_id(), h = late >> 5, lq = late & 31;      // (addresses formed anew, not kept across the loop)
    const f32x4* const qr = reinterpret_cast<const f32x4*>(static_cast<const float*>(p.q) + bi * p.q_bstride + row_of(late & 31).idx * D) + (late >> 5);
    // Keys wait in a register, one to a lane, until there are four: then the rows that see them take them, those of `q_left` all of these,
    // the others those that are done again.
    int queue = 0, n_queue = 0;
    unsigned q_left = 0;
    auto add_keys = [&](bool again) __attribute__((always_inline)) {
      const unsigned char *kk[4], *vv[4];
      bool on[4];
      float dot[4] = {0.f, 0.f, 0.f, 0.f};
      const f32x4* qs = qr;
      asm volatile("" : "+v"(qs));               // (the row is read anew for every four keys, not held)
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int key = __builtin_amdgcn_readlane(queue, u < n_queue ? u : 0);          // (the first once more, for nobody)
        kk[u] = Kg + static_cast<unsigned long long>(key) * row_bytes;
        vv[u] = Vg + static_cast<unsigned long long>(key) * row_bytes;
        on[u] = u < n_queue && key <= q_pos && ((q_left >> u & 1) != 0 || again);
      }
      n_queue = 0;
      q_left = 0;
#pragma unroll 4
      for (int j = 0; j < D / 8; ++j) {
        const f32x4 b = qs[2 * j];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const f32x4 a = reinterpret_cast<const f32x4*>(kk[u])[2 * j + h];
#pragma unroll
          for (int e = 0; e < 4; ++e) dot[u] = __builtin_fmaf(a[e], b[e], dot[u]);
        }
      }
      float m_new = m_run, alpha, pk[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        dot[u] += __shfl_xor(dot[u], 32);
        if (on[u]) m_new = fmaxf(m_new, dot[u] * c);
      }
      alpha = fast_exp2(m_run - m_new);
      m_run = m_new;
      l_run *= alpha;
      l_lo *= alpha;
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        pk[u] = fast_exp2(__builtin_fmaf(dot[u], c, -m_new));
        if (on[u] && h == 0) l_lo += pk[u];
      }
#pragma unroll
      for (int db = 0; db < NDB; ++db) {
        o[db] *= alpha;
#pragma unroll
        for (int half = 0; half < 2; ++half) {           // (the call without a workspace has Q in registers here)
          f32x4 x[4][2];
#pragma unroll
          for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int i4 = 0; i4 < 2; ++i4) x[u][i4] = reinterpret_cast<const f32x4*>(vv[u])[8 * db + 4 * half + 2 * i4 + h];
#pragma unroll
          for (int u = 0; u < 4; ++u)
            if (on[u]) {
#pragma unroll
              for (int i = 0; i < 8; ++i) o[db][8 * half + i] = __builtin_fmaf(pk[u], x[u][i / 4][i % 4], o[db][8 * half + i]);
            }
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    };
    const bool any_q_odd = !idle && q_odd_rows != 0, q_odd = any_q_odd && (q_odd_rows >> late & 1) != 0;
    if (any_q_odd && q_odd) {                    // from the start again
      m_run = kNegBig;
      l_run = l_lo = 0.f;
#pragma unroll
      for (int db = 0; db < NDB; ++db) o[db] = zero16();
      if (from_pair) {                           // (sums_in_memory has left the row's pair alone)
        const Place to = place_of(late);
        const float lse_old = *to.lse;
        if (lse_old != -__builtin_inff()) {
          m_run = lse_old * kLog2e;
          l_lo = h == 0 ? 1.f : 0.f;
        }
        static_for<D / 8>([&](auto qq) __attribute__((always_inline)) {
          constexpr int Q = decltype(qq)::value;
          const f32x4 x = *reinterpret_cast<const f32x4*>(to.o + 32 * (Q / 4) + 8 * (Q % 4) + 4 * (late >> 5));
#pragma unroll
          for (int e = 0; e < 4; ++e) o[Q / 4][4 * (Q % 4) + e] = x[e];
        });
      }
    }
    if (odd || any_q_odd) {
      int t = 0, tok = 0;
      unsigned todo = 0, left = 0;               // keys of tile t - 1 that are still to be taken, and which of them by all rows
      for (;;) {
        // rows of Q with an infinity are settled (NaN) with the first score that is NaN or infinite and positive, those with a finite
        // value of 2^104 or more take every key
        const bool redo = any_q_odd && __builtin_amdgcn_ballot_w64(q_odd && h == 0 && l_run + l_lo == l_run + l_lo) != 0;
        if (!redo) todo &= left;
#pragma unroll 1
        while (n_queue < 4 && (todo != 0 || t < n_tiles)) {
          if (todo == 0) {
            left = s_all_odd[t / run] != 0 ? ~0u : static_cast<unsigned>(s_odd[t / run]);
            left = __builtin_amdgcn_readfirstlane(static_cast<int>(left));
            const int v = t++ * BT + lq;
            if (!redo && left == 0) continue;
            tok = linear ? (v < n_keys ? goff + v : INT_MAX) : find(v);
            if (left != 0 && run > 1) {
              const unsigned long long at = static_cast<unsigned long long>(tok != INT_MAX ? tok : linear ? goff + n_keys - 1 : 0) * row_bytes;
              const f32x4* const kr = reinterpret_cast<const f32x4*>(Kg + at) + h * (D / 8);
              const f32x4* const vr = reinterpret_cast<const f32x4*>(Vg + at) + h * (D / 8);
              float m = 0.f, mv = 0.f, z = 0.f;
#pragma unroll 4
              for (int e = 0; e < D / 8; ++e) {
                const f32x4 x = kr[e], y = vr[e];
                m = abs_max3(abs_max3(m, x[0], x[1]), x[2], x[3]);
                mv = abs_max3(abs_max3(mv, y[0], y[1]), y[2], y[3]);
#pragma unroll
                for (int i = 0; i < 4; ++i) z = __builtin_fmaf(y[i], 0.f, z);
              }
              const bool huge = __builtin_bit_cast(int, fmaxf(m, __shfl_xor(m, 32))) >= huge_k || __builtin_bit_cast(int, fmaxf(mv, __shfl_xor(mv, 32))) >= kHuge;   // as in conv_write
              left = static_cast<unsigned>(__builtin_amdgcn_ballot_w64(huge));                       // (both halves have the same)
              const unsigned long long nan = __builtin_amdgcn_ballot_w64(!(z == 0.f) && !(left >> lq & 1));
              if (nan != 0 && __builtin_amdgcn_ballot_w64(tok > q_first) != 0) left = ~0u;
            }
            todo = (redo ? ~0u : left) & static_cast<unsigned>(__builtin_amdgcn_ballot_w64(tok != INT_MAX));
            continue;
          }
          const int k = __builtin_ctz(todo), key = __builtin_amdgcn_readlane(tok, k);
          todo &= todo - 1;
          queue = late == n_queue ? key : queue;
          q_left |= (left >> k & 1) << n_queue++;
        }
        if (n_queue == 0) break;
        add_keys(q_odd);
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
    if (is_masked(t)) {              // by element
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
  float lse_new = -__builtin_inff();
  if (seen) {
    const float l2 = __builtin_amdgcn_logf(l_tot);
    // fp32: rounded once (running pairs that go through many steps would gather the rounding of the base-two number as well)
    if constexpr (F32) lse_new = __builtin_fmaf(m_run, kLn2, __builtin_fmaf(l2, kLn2, m_run * kLn2Low));
    else lse_new = (m_run + l2) * kLn2;
  }
  int late = lane;                   // (the row's place formed anew, not kept across the loop)
  asm volatile("" : "+v"(late));
  const Row to = row_of(late & 31);
  const bool q_valid = to.valid, folded = p.merge != 0 && !(LEVELS && long_run);      // (there the old pair is in the sums)
  const int64_t ooff = bi * p.o_bstride + to.idx * D, loff = bi * p.lse_bstride + to.idx;
  // columns of register quad q of the lane: block q / 4 of O^T, 32 (q / 4) + 8 (q % 4) + 4 h
  auto quad = [&](auto qq, f32x4& x) __attribute__((always_inline)) {
    constexpr int Q = decltype(qq)::value;
#pragma unroll
    for (int e = 0; e < 4; ++e) x[e] = o[Q / 4][4 * (Q % 4) + e];
    return 32 * (Q / 4) + 8 * (Q % 4) + 4 * h;
  };
  if (SERIAL && ns > 1) {
    float r, w, mx_all = round > 0 ? s_all[0][tid] : -__builtin_inff(), den_all = round > 0 ? s_all[1][tid] : 0.f;
    fold(lse_new, mx_all, den_all, r, w);
    s_all[0][tid] = mx_all;
    s_all[1][tid] = den_all;
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
  } else if (!folded && (ns > 1 || p.out_final == nullptr)) {
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
  } else if (!folded) {
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
  // bf16 with joined steps has a kernel of its own; this one has the single steps, and K and V that end within 256 rows of 2^32 bytes
  if (!fp32 && attn_run_takes(p, d)) return launch_attn_run(p, d, stream);
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
