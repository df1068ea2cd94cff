// Blockwise attention for fp32 inputs of any size and for short bf16 calls: 128 query rows per
// workgroup, the keys of a query tile dealt to as many workgroups as it takes to fill the chip.
//
// The large bf16 kernel (attn_bf16.hip) gives a workgroup 256 rows of one head and all its keys; a
// call with a few hundred local rows then runs on a few dozen of the 256 CUs and a workgroup's chain
// of key tiles is the length of the call.  Here the rows of a query tile are (local row, query head
// of the group) pairs, so that grouped heads fill tiles and share K/V, and n_split workgroups each
// take an equal run of the tile's visible keys; launch_combine adds the partial pairs up.
//
// Per wavefront 32 of the tile's rows, S^T = K Q^T and O^T = V^T P^T: one query per lane column, so
// the softmax is in-lane but for one exchange, and the score registers are the B operand of the second
// product as they stand.  bf16: v_mfma_f32_32x32x16_bf16, V through the transposing LDS read.  fp32:
// v_mfma_f32_32x32x2_f32 (full fp32 products and sums); the 16 bytes a lane reads of a K row feed
// four of them, and so do the 16 bytes (d = 64: two, from 8) it reads of a V row, because block c of
// O^T takes the columns 4 i + c (2 i + c) instead of 32 neighbouring ones.  K and V tiles come through
// direct global->LDS loads into two stages.
//
// What bounds it: fp32 the matrix pipe (a fp32 matrix instruction holds it for 64 cycles, which
// leaves room for everything else a SIMD has to issue); bf16 the issue slots (1 330 of the 1 450 cycles
// a SIMD takes for 32 rows by 64 keys at d = 64), and in the shortest calls the launch, the set-up and
// the latency of the first tiles.  Measured, whole calls:
//   fp32, 16 heads of 128, 2 048 of 16 384 tokens, causal: 1.12 ms (123 TFLOP/s of the 152 a large fp32
//     product reaches) against 20.1 ms with a wavefront per query row;
//   fp32, 4 heads of 64, 256 of 1 024 tokens: 16 us against 308;
//   bf16, 8 heads of 128, 512 of 4 096 tokens: 25 us against 117 with the large kernel on 16 CUs (a workgroup of
//     it: set-up 2.8 us, first tile 1.3, four tiles 8.4, epilogue 2.3);
//   bf16, 128 sequences of 3 072 tokens, 20 heads of 64: 0.71 ms against 0.91 with the large kernel,
//     which pads 192 rows to 256 and searches for the rows of 27-token sub-chunks in every tile.
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
constexpr float kNegBig = -1.0e30f;
constexpr int BM = kTileRows;            // rows per workgroup: four wavefronts of 32
constexpr int NTHREADS = 256;
constexpr int CHUNK = 512;               // keys located at a time

template <typename T, int D>
struct TCfg {
  static constexpr bool F32 = sizeof(T) == 4;
  static constexpr int BT = F32 ? 32 : 64;              // keys per tile
  static constexpr int NKB = BT / 32;                   // 32-key blocks
  static constexpr int RB = D * static_cast<int>(sizeof(T));   // bytes of a row
  static constexpr int UNITS = RB / 16;                 // 16-byte units per row
  static constexpr int RPP = NTHREADS / UNITS;          // rows filled per pass
  static constexpr int PASSES = BT / RPP;
  static constexpr int TILE_BYTES = BT * RB;
  static constexpr int STAGE_BYTES = 2 * TILE_BYTES;    // K tile, V tile
  static constexpr int RPL = UNITS >= 16 ? 1 : 16 / UNITS;   // rows per 256-byte bank line
  static constexpr int NDB = D / 32;                    // 32-column blocks of O^T
  // Physical unit of logical unit u of row r.  K is read row-wise (32 lanes, one row each, the same
  // unit): neighbouring bank lines differ.  V: fp32 rows are read whole; bf16 through the transposing
  // read (4 rows, 2 units).
  __device__ static int swz_k(int r, int u) { return u ^ ((r / RPL) % (UNITS < 16 ? UNITS : 16)); }
  __device__ static int swz_v(int r, int u) { return F32 ? u : u ^ (4 * ((r / RPL) % (UNITS / 4))); }
};

__device__ inline float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }
__device__ inline f32x16 zero16() {
  f32x16 z;
#pragma unroll
  for (int i = 0; i < 16; ++i) z[i] = 0.f;
  return z;
}
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
__global__ __launch_bounds__(NTHREADS, (D == 64 ? 3 : 2) - SERIAL) void attn_tile_kernel(const AttnLaunch p) {
  using C = TCfg<T, D>;
  constexpr bool F32 = C::F32;
  constexpr int BT = C::BT, NKB = C::NKB, NDB = C::NDB, NJ = C::UNITS / 2;
  __shared__ __attribute__((aligned(16))) unsigned char smem[2 * C::STAGE_BYTES];
  __shared__ __attribute__((aligned(16))) int s_tok[2 * CHUNK];   // global positions of the keys (INT_MAX: none)
  __shared__ __attribute__((aligned(16))) int s_msk[2][4];    // per wavefront: it fetched a key some row of the tile must not see
  // Effective segments of this workgroup's share of the keys.
  __shared__ int e_vbeg[kMaxSegAll + 1];   // start in the share
  __shared__ int e_goff[kMaxSegAll];       //   global position minus that
  __shared__ int e_n;

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, h = lane >> 5, lq = lane & 31;

  // What the set-up needs of the kernel arguments is asked for here, in one go and at fixed places: they
  // come from far (a first dependent read of them costs about as much as a tile).
  const AttnTask t0 = p.task[0], t1 = p.task[1];
  const int32_t* const seg_ext0 = p.seg_ext[0];
  const int32_t* const seg_ext1 = p.seg_ext[1];
  int* const s_pool = reinterpret_cast<int*>(smem);           // in the still unused tile stages
  static_assert(2 * kPoolSeg * 4 <= C::STAGE_BYTES, "");
  int pooled[2 * kPoolSeg / NTHREADS];
#pragma unroll
  for (int i = 0; i < 2 * kPoolSeg / NTHREADS; ++i) pooled[i] = p.pool[NTHREADS * i + tid];

  // ---- which (sequence, KV head, task, row tile, share of the keys)
  const int G = p.Hq / p.Hkv;
  const int m0 = t0.n_q * G, m1 = p.n_tasks > 1 ? t1.n_q * G : 0;
  const int tiles0 = (m0 + BM - 1) / BM, tiles1 = (m1 + BM - 1) / BM;
  const int items0 = tiles0 * (SERIAL ? 1 : p.n_split[0]), per_g = items0 + tiles1 * (SERIAL ? 1 : p.n_split[1]);
  const int w_all = xcd_balanced(blockIdx.x, p.batch * p.Hkv, per_g, xcd_window(D == 64 ? 96 : 64, per_g));
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
  const int n_seg = second ? t1.n_seg : t0.n_seg, seg0 = second ? t1.seg0 : t0.seg0;
  const int32_t* const seg_ext = second ? seg_ext1 : seg_ext0;
  const int m_all = second ? m1 : m0;
  // The strip of 32 rows a wavefront takes moves with the work item: wavefront i of a workgroup runs on
  // SIMD i, and tiles with few rows left leave strips without work.
  const int strip = (wave + w_all) & 3;
  const int m = tile * BM + strip * 32 + lq;                 // row of the tile: (local row, head of the group)
  const bool q_valid = m < m_all;
  const int mc = q_valid ? m : m_all - 1;
  const int row = mc / G, hq = g * G + mc - row * G;
  const int q_pos = p.causal ? q_pos0 + row : INT_MAX - 1;
  const int q_last = q_pos0 + (min(tile * BM + BM, m_all) - 1) / G;
  const int q_first = p.causal ? q_pos0 + tile * BM / G : INT_MAX - 1;   // a key at or before it is seen by every row

  // ---- Q fragments (B operand): 16-byte units 2 j + h of the lane's row
  const int64_t qoff = bi * p.q_bstride + (static_cast<int64_t>(q_row0 + row) * p.Hq + hq) * D;
  u32x4 qf[NJ];
  {
    const u32x4* src = reinterpret_cast<const u32x4*>(static_cast<const T*>(p.q) + qoff) + h;
#pragma unroll
    for (int j = 0; j < NJ; ++j) qf[j] = src[2 * j];
  }

  float mx_all = -__builtin_inff(), den_all = 0.f;       // SERIAL: of the shares so far
  for (int round = 0; SERIAL ? round < ns : round == 0; ++round) {
  if constexpr (SERIAL) {
    share = round;
    if (round > 0) {
#pragma unroll
      for (int i = 0; i < 2 * kPoolSeg / NTHREADS; ++i) pooled[i] = p.pool[NTHREADS * i + tid];
      __syncthreads();               // nobody reads the tiles and lists of the share before any more
    }
  }
  // ---- effective segments: what the mask leaves of every segment for this tile, then the share of it
  // that is this workgroup's.  The first wavefront works through the list, 64 segments per round.
  if (seg_ext == nullptr) {
#pragma unroll
    for (int i = 0; i < 2 * kPoolSeg / NTHREADS; ++i) s_pool[NTHREADS * i + tid] = pooled[i];
  }
  __syncthreads();
  if (wave == 0) {
    auto visible = [&](int s, int& a) __attribute__((always_inline)) {
      a = 0;
      if (s >= n_seg) return 0;
      int e;
      if (seg_ext != nullptr) { a = seg_ext[2 * s]; e = seg_ext[2 * s + 1]; }
      else { a = s_pool[2 * (seg0 + s)]; e = s_pool[2 * (seg0 + s) + 1]; }
      return max(0, (p.causal ? min(e, q_last + 1) : e) - a);
    };
    int lo = 0, hi = INT_MAX;                     // this workgroup's share of the tile's visible keys
    if (ns > 1) {                                 // only with joined steps: over them every key of the sequence comes once
      const int total = p.causal ? q_last + 1 : p.last_key + 1;
      const int chunk = ((total + ns - 1) / ns + BT - 1) / BT * BT;
      lo = share * chunk;
      hi = lo + chunk;
    }
    int n_base = 0, v_base = 0, o_base = 0;
    for (int s0 = 0; s0 < n_seg; s0 += 64) {
      int a;
      const int len = visible(s0 + lane, a);
      int sl = len;                               // inclusive scan of the lengths
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) { const int t = __shfl_up(sl, o); if (lane >= o) sl += t; }
      const int beg = v_base + sl - len;          // position in the tile's visible keys
      const int cb = max(beg, lo), ce = min(beg + len, hi), clen = max(0, ce - cb);
      const unsigned long long has = __builtin_amdgcn_ballot_w64(clen > 0);
      if (clen > 0) {
        const int idx = n_base + __builtin_popcountll(has & ((1ull << lane) - 1));
        e_vbeg[idx] = cb - lo;
        e_goff[idx] = a + (cb - beg) - (cb - lo);
        o_base = ce - lo;                         // (the last one of the round is taken below)
      }
      if (has != 0) o_base = __shfl(o_base, 63 - __builtin_clzll(has));
      n_base += __builtin_popcountll(has);
      v_base += __shfl(sl, 63);
    }
    if (lane == 0) { e_vbeg[n_base] = o_base; e_n = n_base; }
  }
  __syncthreads();
  const int n_eff = e_n, n_keys = e_vbeg[n_eff];
  const int n_tiles = (n_keys + BT - 1) / BT;

  // ---- positions of the keys, looked up for CHUNK of them at a time: chunk c in half c % 2 of s_tok.
  // With sub-chunks of a few dozen keys most tiles cross a segment boundary; a search per tile and
  // row cost more than the tile's exponentials.
  auto locate = [&](int chunk) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < CHUNK / NTHREADS; ++i) {
      const int v = chunk * CHUNK + i * NTHREADS + tid;
      int lo = 0, n = n_eff;                                        // the last segment that begins at or before v
      while (n > 1) {
        const int half = n >> 1;
        if (e_vbeg[lo + half] <= v) lo += half;
        n -= half;
      }
      s_tok[(chunk & 1) * CHUNK + i * NTHREADS + tid] = v < n_keys ? v + e_goff[lo] : INT_MAX;
    }
  };

  // ---- loader: this thread fills rows fr + RPP i, physical unit fu of the K and the V tile
  const int fr = tid / C::UNITS, fu = tid % C::UNITS;
  const unsigned row_bytes = static_cast<unsigned>(p.Hkv) * C::RB;
  const int64_t head0 = (bi * p.kv_bstride + static_cast<int64_t>(g) * D) * static_cast<int64_t>(sizeof(T));
  const unsigned char* Kg = static_cast<const unsigned char*>(p.k) + head0;
  const unsigned char* Vg = static_cast<const unsigned char*>(p.v) + head0;
  const u32x4 k_buf = raw_buffer(Kg), v_buf = raw_buffer(Vg);
  const int wave_u = __builtin_amdgcn_readfirstlane(wave);
  auto fetch = [&](int t, int stage) __attribute__((always_inline)) {
    unsigned char* dst = smem + stage * C::STAGE_BYTES + wave_u * 1024;
    int tok[C::PASSES], last = -1;
#pragma unroll
    for (int i = 0; i < C::PASSES; ++i) tok[i] = s_tok[(t * BT + fr + C::RPP * i) & (2 * CHUNK - 1)];     // one round trip for all passes
#pragma unroll
    for (int i = 0; i < C::PASSES; ++i) {
      const int r = fr + C::RPP * i;
      last = max(last, tok[i]);
      // rows past the end fetch the first key and are masked; every row sees that one, so nothing it holds reaches
      // a row that it should not (0 times infinity)
      const unsigned key = tok[i] == INT_MAX ? 0u : static_cast<unsigned>(tok[i]);
      if constexpr (F32) {                                          // tensors may exceed what a 32-bit offset reaches
        const unsigned long long off = static_cast<unsigned long long>(key) * row_bytes;
        global_to_lds_16_far(Kg + off + C::swz_k(r, fu) * 16, dst + i * NTHREADS * 16);
        global_to_lds_16_far(Vg + off + C::swz_v(r, fu) * 16, dst + C::TILE_BYTES + i * NTHREADS * 16);
      } else {                                                      // both factors are below 2^24 (host check)
        const unsigned off = __umul24(key, row_bytes);
        buffer_to_lds_16<true>(k_buf, 0u, off + C::swz_k(r, fu) * 16, dst + i * NTHREADS * 16);
        buffer_to_lds_16<true>(v_buf, 0u, off + C::swz_v(r, fu) * 16, dst + C::TILE_BYTES + i * NTHREADS * 16);
      }
    }
    const bool any = __builtin_amdgcn_ballot_w64(last > q_first) != 0;
    if (lane == 0) s_msk[stage][wave] = any ? 1 : 0;
  };

  // ---- LDS read addresses inside a stage
  const int k_row = lq * C::RB, k_sw = C::swz_k(lq, h) * 16;        // unit 2 j + h sits at k_sw ^ 32 j
  int v_adr[NDB];                                                   // bf16: as in the large kernel
  if constexpr (F32) {
    v_adr[0] = C::TILE_BYTES + 4 * h * C::RB + lq * (C::RB / 32);   // key 4 h (+ 8 (r / 4) + r % 4), 32 equal pieces of the row
  } else {
    const int ga = lane >> 4, jj = lane & 15;
    const int vrow = 4 * (ga >> 1) + (jj >> 2);
#pragma unroll
    for (int db = 0; db < NDB; ++db)
      v_adr[db] = C::TILE_BYTES + (vrow * C::UNITS + C::swz_v(vrow, 4 * db + 2 * (ga & 1) + ((jj & 3) >> 1))) * 16 + 8 * (jj & 1);
  }

  f32x16 o[NDB];
#pragma unroll
  for (int db = 0; db < NDB; ++db) o[db] = zero16();
  // fp32: what FLUSH tiles have added goes to a second set of sums, so that the error of the chain of additions does
  // not grow with the number of keys (2 048 of 16 384 tokens: error of the output 9.9e-7 with one set, 5.1e-7 so, for 1 % of the time)
  constexpr int FLUSH = 8;
  f32x16 o_sum[F32 ? NDB : 1];
#pragma unroll
  for (int db = 0; db < (F32 ? NDB : 1); ++db) o_sum[db] = zero16();
  // running max (exp2 domain), sum in two levels (the last 64 tiles, everything before: one fp32
  // accumulator would swallow the many small terms behind a few large ones), and what rounding added
  // to the largest probabilities (bf16), as in the large kernel
  float m_run = kNegBig, l_run = 0.f, l_lo = 0.f, r_fix = 0.f;
  const float c = p.scale * kLog2e;

  // fp32: an infinity or NaN in V of a key that a row does not see would come to it as 0 times that.  Only tiles with the
  // element-wise mask hold such pairs; those of them with such a V are left out and added key by key after the others.
  bool odd_tiles = false;
  const bool idle = __builtin_amdgcn_readfirstlane(tile * BM + strip * 32) >= m_all;
  if (n_tiles > 0) {
    locate(0);
    __syncthreads();
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
    if ((t + 2) % (CHUNK / BT) == 0 && t + 2 < n_tiles) locate((t + 2) / (CHUNK / BT));
    if (idle) continue;
    const unsigned char* st = smem + stage * C::STAGE_BYTES;

    bool masked = false;             // by element
    if constexpr (F32) {             // (asked here, where few registers are taken; bf16: under way with the V fragments)
      const i32x4 mk = *reinterpret_cast<const i32x4*>(&s_msk[stage][0]);
      masked = __builtin_amdgcn_readfirstlane(mk[0] | mk[1] | mk[2] | mk[3]) != 0;
      if (masked) {                              // see odd_tiles
        float z = 0.f;
#pragma unroll 4
        for (int r = 0; r < 16; ++r) z = add_zero_times<NDB>(st + v_adr[0] + (8 * (r / 4) + r % 4) * C::RB, z);
        if (__builtin_amdgcn_ballot_w64(!(z == 0.f)) != 0) { odd_tiles = true; continue; }
      }
    }
    // The matrix instructions of both products take their A operands as streams of fragments read ahead, so
    // that a wavefront alone on its SIMD does not wait for LDS at each of them (one fp32 K fragment feeds four
    // long instructions: the compiler's order does).
    f32x16 S[NKB];
    if constexpr (F32) {
      S[0] = zero16();
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        const f32x4 af = *reinterpret_cast<const f32x4*>(st + k_row + (k_sw ^ (32 * j))), bf = __builtin_bit_cast(f32x4, qf[j]);
#pragma unroll
        for (int e = 0; e < 4; ++e) S[0] = __builtin_amdgcn_mfma_f32_32x32x2f32(af[e], bf[e], S[0], 0, 0, 0);
      }
    } else {
      constexpr int NF = NKB * NJ, PD = 6;
      bf16x8 ring[PD];
      auto read_k = [&](auto ff) __attribute__((always_inline)) {
        constexpr int F = decltype(ff)::value;
        ring[F % PD] = *reinterpret_cast<const bf16x8*>(st + k_row + F / NJ * 32 * C::RB + (k_sw ^ (32 * (F % NJ))));
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
    constexpr int NV = F32 ? 1 : 2 * NKB * NDB, PV = 4;       // bf16 V^T fragments: 16-key group f / NDB, block f % NDB of O^T
    bf16x8 vring[PV];
    auto read_v = [&](auto ff) __attribute__((always_inline)) {
      constexpr int F = decltype(ff)::value;
      const unsigned char* va = st + v_adr[F % NDB] + F / NDB * 16 * C::RB;
      vring[F % PV] = lds_tr8(va, va + 8 * C::RB);
    };
    if constexpr (!F32) static_for<PV>(read_v);               // on their way during the maxima
    if constexpr (!F32) {
      const i32x4 mk = *reinterpret_cast<const i32x4*>(&s_msk[stage][0]);
      masked = __builtin_amdgcn_readfirstlane(mk[0] | mk[1] | mk[2] | mk[3]) != 0;
    }
    if (masked) {
#pragma unroll
      for (int kb = 0; kb < NKB; ++kb)
#pragma unroll
        for (int i4 = 0; i4 < 4; ++i4) {
          const i32x4 tk = *reinterpret_cast<const i32x4*>(&s_tok[((t * BT) & (2 * CHUNK - 1)) + 32 * kb + 8 * i4 + 4 * h]);
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (tk[e] > q_pos) S[kb][4 * i4 + e] = -__builtin_inff();
        }
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
        for (int i = 0; i < 16; ++i) {
          o[db][i] *= alpha;
          if constexpr (F32) o_sum[db][i] *= alpha;
        }
    }
    if constexpr (!F32) {
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
    if constexpr (F32) {
      exps(std::integral_constant<int, 0>{}, std::integral_constant<int, 16>{});
#pragma unroll
      for (int r = 0; r < 16; ++r) {             // keys 8 (r / 4) + r % 4 and four further on (the lane halves)
        const unsigned char* va = st + v_adr[0] + (8 * (r / 4) + r % 4) * C::RB;
        float vv[NDB];
        if constexpr (NDB == 4) {
          const f32x4 x = *reinterpret_cast<const f32x4*>(va);
#pragma unroll
          for (int e = 0; e < 4; ++e) vv[e] = x[e];
        } else {
          const f32x2 x = *reinterpret_cast<const f32x2*>(va);
          vv[0] = x[0]; vv[1] = x[1];
        }
#pragma unroll
        for (int db = 0; db < NDB; ++db) o[db] = __builtin_amdgcn_mfma_f32_32x32x2f32(vv[db], S[0][r], o[db], 0, 0, 0);
      }
    } else {
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
    if constexpr (F32) {
      if (t % FLUSH == FLUSH - 1) {
#pragma unroll
        for (int db = 0; db < NDB; ++db) { o_sum[db] += o[db]; o[db] = zero16(); }
      }
    }
  }
  if constexpr (F32) {
#pragma unroll
    for (int db = 0; db < NDB; ++db) o[db] += o_sum[db];
    if (odd_tiles) {
#pragma unroll 1
      for (int t = 0; t < n_tiles; ++t) {
        const int v = t * BT + lq;
        int lo = 0, n = n_eff;                     // as in locate
        while (n > 1) {
          const int half = n >> 1;
          if (e_vbeg[lo + half] <= v) lo += half;
          n -= half;
        }
        const int tok = v < n_keys ? v + e_goff[lo] : INT_MAX;
        if (__builtin_amdgcn_ballot_w64(tok > q_first) == 0) continue;
        const float* vr = reinterpret_cast<const float*>(Vg + static_cast<unsigned long long>(tok == INT_MAX ? 0 : tok) * row_bytes) + h * (D / 2);
        float z = 0.f;
        for (int e = 0; e < D / 2; ++e) z = __builtin_fmaf(vr[e], 0.f, z);
        if (__builtin_amdgcn_ballot_w64(!(z == 0.f)) == 0) continue;
#pragma unroll 1
        for (int k = 0; k < BT; ++k) {
          const int key = __builtin_amdgcn_readlane(tok, k);
          if (key == INT_MAX) break;               // past the end, as all that follow
          const u32x4* kr = reinterpret_cast<const u32x4*>(Kg + static_cast<unsigned long long>(key) * row_bytes) + h;
          float dot = 0.f;
#pragma unroll
          for (int j = 0; j < NJ; ++j) {
            const f32x4 a = __builtin_bit_cast(f32x4, kr[2 * j]), b = __builtin_bit_cast(f32x4, qf[j]);
#pragma unroll
            for (int e = 0; e < 4; ++e) dot = __builtin_fmaf(a[e], b[e], dot);
          }
          dot += __shfl_xor(dot, 32);
          if (key > q_pos) continue;
          const float m_new = fmaxf(m_run, dot * c), alpha = fast_exp2(m_run - m_new), pk = fast_exp2(__builtin_fmaf(dot, c, -m_new));
          m_run = m_new;
          l_run *= alpha;
          l_lo = l_lo * alpha + (h == 0 ? pk : 0.f);
          const float* vk = reinterpret_cast<const float*>(Vg + static_cast<unsigned long long>(key) * row_bytes);
#pragma unroll
          for (int i = 0; i < 16; ++i)
#pragma unroll
            for (int db = 0; db < NDB; ++db) o[db][i] = __builtin_fmaf(pk, vk[NDB * (8 * (i / 4) + 4 * h + i % 4) + db], o[db][i] * alpha);
        }
      }
    }
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");     // no fetch may still be writing LDS when the workgroup ends

  // ---- epilogue: normalise and store, 4 consecutive columns a lane and turn
  const float l_mine = l_run + l_lo;
  const float l_tot = l_mine + __shfl_xor(l_mine, 32), r_tot = l_tot + (r_fix + __shfl_xor(r_fix, 32));
  const bool seen = l_tot > 0.f;
  float wb = seen && r_tot > 0.f ? 1.f / r_tot : 0.f;
  float lse_new = seen ? (m_run + __builtin_amdgcn_logf(l_tot)) * kLn2 : -__builtin_inff();
  const int64_t ooff = bi * p.o_bstride + (static_cast<int64_t>(q_row0 + row) * p.Hq + hq) * D;
  const int64_t loff = bi * p.lse_bstride + static_cast<int64_t>(q_row0 + row) * p.Hq + hq;
  // columns of register quad q of the lane: bf16 block q / 4, 32 (q / 4) + 8 (q % 4) + 4 h; fp32 d = 128
  // row i of the blocks, 4 i; d = 64 rows i, i + 1, 2 i, where i = 8 (r / 4) + 4 h + r % 4
  auto quad = [&](auto qq, f32x4& x) __attribute__((always_inline)) {
    constexpr int Q = decltype(qq)::value;
    if constexpr (!F32) {
#pragma unroll
      for (int e = 0; e < 4; ++e) x[e] = o[Q / 4][4 * (Q % 4) + e];
      return 32 * (Q / 4) + 8 * (Q % 4) + 4 * h;
    } else if constexpr (NDB == 4) {
#pragma unroll
      for (int e = 0; e < 4; ++e) x[e] = o[e][Q];
      return 4 * (8 * (Q / 4) + 4 * h + Q % 4);
    } else {
      x = f32x4{o[0][2 * Q], o[1][2 * Q], o[0][2 * Q + 1], o[1][2 * Q + 1]};
      return 2 * (8 * (2 * Q / 4) + 4 * h + (2 * Q) % 4);
    }
  };
  if (SERIAL && ns > 1) {
    float r, w;
    fold(lse_new, mx_all, den_all, r, w);
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
    const int64_t rh = ns > 1 ? ((static_cast<int64_t>(share) * p.batch + bi) * n_q + row) * p.Hq + hq : 0;
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
  return TASP_LAUNCH((attn_tile_kernel<T, D, SERIAL>), dim3(static_cast<unsigned>(blocks)), dim3(NTHREADS), stream, p);
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
