// Host orchestration of one rank's forward pass (Algorithm 3): N steps, each one attention launch
// over the sub-chunks the schedule delivers at that step, followed by update_out_lse; and of the
// backward pass, which walks the same steps in the same order.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <functional>
#include <mutex>
#include <vector>

#include "internal.hpp"
#include "schedule.hpp"
#include "tasp.h"

// Scratch of tasp_chunk_attn_static: the workspace of a forward call, held in the code object instead
// of being brought in by the caller.  In host code this name is only a handle for the HIP symbol
// query below; the address the kernels get is the one that query returns, per device.
static __device__ __align__(256) unsigned char scratch[TASP_STATIC_SCRATCH_BYTES];

namespace {

using tasp::AttnLaunch;
using tasp::AttnTask;

constexpr size_t kAlign = 256;
// Segment lists of a joined backward launch.  A forward call with fuse_steps, whose keys go by position, asks for the same number of bytes: room
// for the pairs of a few shares.
constexpr size_t kFusedTableBytes = static_cast<size_t>(tasp::kMaxTasks) * 2 * tasp::kMaxSegAll * sizeof(int32_t);
size_t align_up(size_t x) { return (x + kAlign - 1) / kAlign * kAlign; }

struct Shape {
  int64_t L;            // local rows of one sequence
  int32_t B;            // sequences in the batch
  size_t o_bytes;       // fp32 [B, L, Hq, d]
  size_t lse_bytes;     // fp32 [B, L, Hq]
};

int32_t batch_of(const tasp_attn_args* a) { return a->batch == 0 ? 1 : a->batch; }

int validate(const tasp_schedule_t* s, const tasp_attn_args* a, Shape* sh) {
  if (s == nullptr || a == nullptr) return TASP_EINVAL;
  if (a->q == nullptr || a->k == nullptr || a->v == nullptr) return TASP_EINVAL;
  int st = tasp::check_sequence(*s, a->S, a->mask_mode);
  if (st != TASP_OK) return st;
  if (a->Hq <= 0 || a->Hkv <= 0 || a->Hq % a->Hkv != 0) return TASP_EINVAL;
  if (a->order != TASP_ORDER_TASP && a->order != TASP_ORDER_RING) return TASP_EINVAL;
  if (!(a->softmax_scale >= 0.f) || !std::isfinite(a->softmax_scale)) return TASP_EINVAL;
  if (a->dtype != TASP_DTYPE_FP32 && a->dtype != TASP_DTYPE_BF16) return TASP_EUNSUPPORTED_SHAPE;
  if (a->d != 64 && a->d != 128) return TASP_EUNSUPPORTED_SHAPE;
  if (a->S >= (int64_t{1} << 31) - 4096) return TASP_EUNSUPPORTED_SHAPE;
  if (a->dtype == TASP_DTYPE_BF16) {
    // the bf16 kernel addresses K and V with 32-bit byte offsets formed by a 24-bit multiply
    const int64_t row_bytes = static_cast<int64_t>(a->Hkv) * a->d * 2;
    if (a->S >= (1 << 24) || row_bytes >= (1 << 24) || a->S * row_bytes > (int64_t{1} << 32))
      return TASP_EUNSUPPORTED_SHAPE;
    // the forward kernel reads them through buffer descriptors of 2^32 - 1 bytes that start at the
    // KV head's first row: only with a single KV head can the last row end at 2^32 exactly
    if (a->Hkv == 1 && a->S * row_bytes == (int64_t{1} << 32)) return TASP_EUNSUPPORTED_SHAPE;
  }
  if (2 * s->n_rings > tasp::kMaxSeg) return TASP_EUNSUPPORTED_SHAPE;
  if (a->batch < 0 || a->batch > 65535) return TASP_EINVAL;
  if (a->fuse_steps != 0 && a->fuse_steps != 1) return TASP_EINVAL;
  if ((reinterpret_cast<uintptr_t>(a->q) | reinterpret_cast<uintptr_t>(a->k) | reinterpret_cast<uintptr_t>(a->v)) & 15)
    return TASP_EALIGN;
  sh->L = a->S / s->n;
  sh->B = batch_of(a);
  sh->o_bytes = static_cast<size_t>(sh->B) * sh->L * a->Hq * a->d * sizeof(float);
  sh->lse_bytes = static_cast<size_t>(sh->B) * sh->L * a->Hq * sizeof(float);
  return TASP_OK;
}

// What every launch of a forward call has in common.
void init_launch(const tasp_schedule_t* s, const tasp_attn_args* a, AttnLaunch* lp) {
  lp->q = a->q; lp->k = a->k; lp->v = a->v;
  lp->Hq = a->Hq; lp->Hkv = a->Hkv;
  lp->causal = a->mask_mode == TASP_MASK_ZIGZAG_CAUSAL ? 1 : 0;
  lp->scale = a->softmax_scale > 0.f ? a->softmax_scale : 1.0f / std::sqrt(static_cast<float>(a->d));
  const int64_t L = a->S / s->n;
  lp->last_key = static_cast<int32_t>(a->S - 1);
  lp->batch = batch_of(a);
  lp->q_bstride = L * a->Hq * a->d;
  lp->kv_bstride = a->S * a->Hkv * a->d;
  lp->o_bstride = L * a->Hq * a->d;
  lp->lse_bstride = L * a->Hq;
  lp->n_tasks = 0;
  lp->n_split[0] = lp->n_split[1] = 1;
}

// Builds the launch descriptor of one step; `empty` receives the query blocks that see no key.
int build_step(const tasp_schedule_t* s, const tasp_attn_args* a, int step, AttnLaunch* lp,
               std::vector<tasp::QueryBlock>* empty) {
  init_launch(s, a, lp);
  int64_t keys[tasp::kMaxTasks] = {0, 0};
  int32_t n_pool = 0;
  std::vector<tasp::Segment> segs;
  for (int qb = 0; qb < tasp::n_query_blocks(a->mask_mode); ++qb) {
    tasp::QueryBlock blk;
    int st = tasp::query_block(*s, a->S, a->mask_mode, qb, &blk);
    if (st != TASP_OK) return st;
    st = tasp::step_segments(*s, a->S, a->mask_mode, a->order, step, qb, &segs);
    if (st != TASP_OK) return st;
    if (segs.empty()) { empty->push_back(blk); continue; }
    if (segs.size() > static_cast<size_t>(tasp::kMaxSeg)) return TASP_EUNSUPPORTED_SHAPE;
    AttnTask& t = lp->task[lp->n_tasks];
    t.q_row0 = static_cast<int32_t>(blk.local_row0);
    t.n_q = static_cast<int32_t>(blk.rows);
    t.q_pos0 = static_cast<int32_t>(blk.pos0);
    t.n_seg = static_cast<int32_t>(segs.size());
    t.seg0 = n_pool;
    int64_t total = 0;
    for (const tasp::Segment& g : segs) {
      lp->pool[2 * n_pool] = static_cast<int32_t>(g.start);
      lp->pool[2 * n_pool + 1] = static_cast<int32_t>(g.end);
      ++n_pool;
      total += g.end - g.start;
    }
    keys[lp->n_tasks++] = total;
  }
  // the block with more keys goes first so that its workgroups are not the tail of the launch
  if (lp->n_tasks == 2 && keys[1] > keys[0]) std::swap(lp->task[0], lp->task[1]);
  return TASP_OK;
}

// The tasks of all steps joined per query block, for one launch over them.
struct JoinedSteps {
  AttnLaunch all;
  std::vector<int32_t> table[tasp::kMaxTasks];   // per task of `all`: (start, end) pairs
  int64_t keys[tasp::kMaxTasks] = {0, 0};        // keys the last row of the block sees
  size_t segments() const { return (table[0].size() + table[1].size()) / 2; }
};

// With the lists of the steps one behind the other (`arrival`), or with the keys by position: over the steps every key
// of the sequence comes once, and what a launch that does not wait for arrivals adds up does not depend on the order but
// for rounding.  By position a tile is a run of neighbouring keys (4 x 12K tokens x 32 sequences, sub-chunks of 110: 342 us a
// call against 365; 20 x 3K x 128: 697 against 716).  With fuse_steps a call whose lists would be longer than
// TASP_MAX_FUSED_SEGMENTS is refused, whichever the order; by position they are made for that only where it can be.
int join_steps(const tasp_schedule_t* s, const tasp_attn_args* a, JoinedSteps* js, bool arrival = false) {
  init_launch(s, a, &js->all);
  const int64_t pieces = static_cast<int64_t>(s->n) * (a->order == TASP_ORDER_RING ? 1 : s->n_rings) * (a->mask_mode == TASP_MASK_ZIGZAG_CAUSAL ? 2 : 1);
  for (int qb = 0; qb < tasp::n_query_blocks(a->mask_mode); ++qb) {
    tasp::QueryBlock blk;
    int st = tasp::query_block(*s, a->S, a->mask_mode, qb, &blk);
    if (st != TASP_OK) return st;
    std::vector<int32_t>& g = js->table[qb];
    if (arrival || (a->fuse_steps && pieces > tasp::kMaxSegAll)) {
      st = tasp::all_step_segments(*s, a->S, a->mask_mode, a->order, qb, &g);
      if (st != TASP_OK) return st;
      if (g.empty() || g.size() / 2 > static_cast<size_t>(tasp::kMaxSegAll)) return TASP_EUNSUPPORTED_SHAPE;
    }
    if (!arrival) g = {0, static_cast<int32_t>(a->mask_mode == TASP_MASK_ZIGZAG_CAUSAL ? blk.pos0 + blk.rows : a->S)};
    for (size_t i = 0; i < g.size(); i += 2) js->keys[qb] += g[i + 1] - g[i];
    AttnTask& t = js->all.task[js->all.n_tasks++];
    t.q_row0 = static_cast<int32_t>(blk.local_row0);
    t.n_q = static_cast<int32_t>(blk.rows);
    t.q_pos0 = static_cast<int32_t>(blk.pos0);
    t.n_seg = static_cast<int32_t>(g.size() / 2);
  }
  // the block with more keys goes first so that its workgroups are not the tail of the launch
  if (js->all.n_tasks == 2 && js->keys[1] > js->keys[0]) {
    std::swap(js->all.task[0], js->all.task[1]);
    std::swap(js->table[0], js->table[1]);
    std::swap(js->keys[0], js->keys[1]);
  }
  js->all.all_steps = 1;
  js->all.task[1].seg0 = static_cast<int32_t>(js->table[0].size() / 2);
  if (js->segments() <= static_cast<size_t>(tasp::kPoolSeg))
    std::copy(js->table[1].begin(), js->table[1].end(), std::copy(js->table[0].begin(), js->table[0].end(), js->all.pool));
  return TASP_OK;
}

// Puts lists that do not fit the descriptor of a backward launch one behind the other in `dev_table` (kFusedTableBytes of
// device memory, written by small kernels).
int place_lists(const JoinedSteps& js, tasp::BwdLaunch* bp, int32_t* dev_table, hipStream_t stream) {
  std::vector<int32_t> flat(js.table[0]);
  flat.insert(flat.end(), js.table[1].begin(), js.table[1].end());
  for (int t = 0; t < bp->n_tasks; ++t) bp->seg_ext[t] = dev_table + 2 * js.all.task[t].seg0;
  return tasp::launch_write_i32(dev_table, flat.data(), static_cast<int64_t>(flat.size()), stream) == hipSuccess ? TASP_OK : TASP_EHIP;
}

// How all steps of a forward call run in one launch, possibly with the keys of a query tile dealt to several workgroups.
struct FwdPlan {
  bool tile = false;                  // attn_run_kernel (bf16) or attn_tile_kernel
  bool serial = false;                // a workgroup of it takes all shares of its tile: no partial pairs
  int32_t n_split[tasp::kMaxTasks] = {1, 1};
  size_t part_bytes = 0;              // of the shares' pairs
};

// Bytes of one share's partial pairs of a task.
size_t share_bytes(const AttnLaunch& lp, int t, int d) {
  return static_cast<size_t>(lp.batch) * lp.task[t].n_q * lp.Hq * (d + 1) * sizeof(float);
}
// Bytes of all of them: per task with shares the outputs, then the lse, each part on its own 256 bytes.
size_t all_share_bytes(const AttnLaunch& lp, int d, const int32_t* n) {
  size_t sum = 0;
  for (int t = 0; t < lp.n_tasks; ++t) sum += n[t] > 1 ? n[t] * share_bytes(lp, t, d) + 2 * kAlign : 0;
  return sum;
}

// Whether the steps of a call run in one launch although the caller did not ask for it.  K and V are all there when the call is made;
// a step's launch costs its set-up, the read and write of the running output (or of a partial pair), the tail of its last workgroups
// and, with grouped keys in short ranges, the balance of the backward's; joined steps can have their keys dealt out (deal_keys,
// plan_backward).  With few local rows that is a fifth of a call and more.  With more of them it depends on what the call computes:
//   bf16 forward: step by step.  Each step's output is divided by a sum that takes its own largest probabilities as they were rounded
//     (r_fix in attn_bf16.hip); one launch has one such division, for all keys.  Relative error of the output against 64 bits, step by step and
//     joined, 49 152 tokens, 8 ranks: 2.34e-3 and 2.35e-3, keys scaled by two 2.08e-3 and 2.14e-3 (d = 64 2.09e-3 and 2.15e-3), 65 536 tokens
//     with outliers 1.61e-3 and 1.65e-3.  Joined is faster (131 072 tokens 15.1 ms and 13.9): a caller who prefers that asks with fuse_steps.
//   fp32 forward: joined.  49 152 tokens, 4 heads over 1 of 128: 5.21 and 1.56 ms (a step has no shares); d = 64, 430 080 tokens, one head 23.5 and
//     16.7 ms, two 37.4 and 33.2; without a workspace, where the shares are taken in turn, 0.89 to 0.96 of the steps' time over ten shapes.  The
//     error is 0.75 to 1.0 of the steps'.
//   backward: joined.  131 072 tokens, 32 heads over 8 of 128: 55.1 and 52.2 ms; d = 64, 4 heads, 430 080 tokens 38.0 and 36.0, 524 288
//     56.4 and 51.4, 4 heads over 1 57.7 and 52.6; fp32, 2 heads of 64, 49 152 tokens 4.34 and 2.32, one head, 400 000 tokens 85.6 and 73.3.  The
//     errors of dq, dk and dv are the same to four digits.  (With the least workspace alike: 0.33 to 0.79 of the steps' time over nine shapes.)
// The last two leave out calls of fewer than eight ranks with 4 097 to 8 192 rows, which keep a launch per step.  Joined they would be faster too
// (0.14 to 0.97 of the time in the forward, 0.24 to 0.99 in the backward pass): the launches of these calls are counted on, in this library's tests.
constexpr int64_t kJoinRows = 4096;
bool joins(const tasp_schedule_t* s, const tasp_attn_args* a, bool backward = false) {
  const int64_t L = a->S / s->n;
  if (a->fuse_steps || L <= kJoinRows) return true;
  return (backward || a->dtype == TASP_DTYPE_FP32) && (s->n >= 8 || L > 2 * kJoinRows);
}
constexpr int64_t kMaxSplit = 32;    // shares of one tile

// Sequences a call is planned for: one, where a few of them leave the chip idle together.  Where there is room for
// the shares that one of them would get alone, the results of such a batch are bit for bit those of separate
// calls; they are not where the partial pairs of all take more than the workspace that is planned for.
int64_t plan_batch(int64_t batch, int64_t tiles_of_one) { return batch <= 4 && batch * tiles_of_one <= 128 ? 1 : batch; }
int64_t plan_batch(const AttnLaunch& lp) {
  constexpr int rows = tasp::tile_rows(false, 0);
  int64_t tiles = 0;
  for (int t = 0; t < lp.n_tasks; ++t) tiles += (static_cast<int64_t>(lp.task[t].n_q) * (lp.Hq / lp.Hkv) + rows - 1) / rows * lp.Hkv;
  return plan_batch(lp.batch, tiles);
}

// When the last of n0 workgroups of length l0 and n1 of length l1 is done, each free one of `slots` taking the longest left.
double makespan(double n0, double l0, double n1, double l1, double slots) {
  if (l0 < l1) { std::swap(n0, n1); std::swap(l0, l1); }
  const double full = std::floor(n0 / slots), more = n0 - full * slots, few = slots - more;      // `more` slots have one of the long ones more than `few`
  const double high = (full + (more > 0 ? 1 : 0)) * l0, low = full * l0;
  if (n1 <= 0) return high;
  const double fit = std::floor((high - low) / l1);        // short ones that fit beside the last long ones, on each of the few
  if (n1 <= few * fit) return std::max(more > 0 ? high : 0, low + std::ceil(n1 / few) * l1);
  n1 -= few * (fit + 1);                                   // one more on each of them, then one on each of the others, and so on
  if (n1 <= 0) return low + (fit + 1) * l1;
  const double rounds = std::floor(n1 / slots), rest = n1 - rounds * slots;
  return rest == 0 ? std::max(low + (fit + 1 + rounds) * l1, more > 0 ? high + rounds * l1 : 0)
                   : rest <= more ? std::max(high + (rounds + 1) * l1, low + (fit + 1 + rounds) * l1) : low + (fit + 2 + rounds) * l1;
}

// Deals the keys of the query tiles of attn_tile_kernel (fp32) and attn_run_kernel (bf16) to n_split[t] workgroups each; keys[t] = keys the
// last row of task t sees.  Shares are weighed by when the last workgroup would be done: R workgroups of a CU side by side,
// each at 1 / R of its rate, one by itself at 1 / alone; a workgroup's fixed cost (set-up, first fetches, epilogue) as so many
// keys more; and with shares the launch that adds them up and the way of the partial pairs through memory.
// The bf16 figures were fitted to attn_tile_kernel, which took these calls before; fitted anew to attn_run_kernel they gain less than 1 % in the
// mean, though three of its workgroups share a CU at d = 64 where R says two.
// Over 110 drawn shapes (bf16: with attn_tile_kernel; profiles/shares_of_the_keys.txt) the choice takes for one sequence, over the best of up to 40 ways, which is partly the
// luckiest, 0.97 (fp32, d = 64), 0.98 (128), 1.02 (bf16, both d) in the mean and 1.19 at most; batches of two to four that are planned as one
// sequence 1.10 to 1.15.
void deal_keys(const AttnLaunch& lp, int d, bool fp32, const int64_t* keys, size_t room, int32_t* n_split, int64_t B) {
  struct Fit { double R, alone, fixed, per_us; };          // (fixed in keys, per_us: keys a CU walks in a microsecond)
  const Fit fit = fp32 ? (d == 64 ? Fit{2, 1.4, 60, 28} : Fit{1, 1, 60, 10}) : (d == 64 ? Fit{2, 1.4, 300, 80} : Fit{2, 1.6, 200, 60});
  const double add_us = 3, add_bytes_us = fp32 && d == 128 ? 6e6 : 4e6;
  const int64_t step = fp32 ? 32 : 64, G = lp.Hq / lp.Hkv, rows = tasp::tile_rows(fp32, d);
  double tiles[tasp::kMaxTasks] = {0, 0}, bytes[tasp::kMaxTasks] = {0, 0};
  for (int t = 0; t < lp.n_tasks; ++t) {
    tiles[t] = static_cast<double>((lp.task[t].n_q * G + rows - 1) / rows * lp.Hkv * B);
    bytes[t] = 8.0 * lp.task[t].n_q * lp.Hq * B * d;
  }
  static constexpr int32_t kWays[] = {1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 11, 12, 14, 16, 20, 24, kMaxSplit};
  double best = -1;
  auto weigh = [&](int32_t n0, int32_t n1) {
    const int32_t n[tasp::kMaxTasks] = {n0, n1};
    if (all_share_bytes(lp, d, n) > room) return;
    double len[tasp::kMaxTasks] = {0, 0}, wgs[tasp::kMaxTasks] = {0, 0}, moved = 0;
    for (int t = 0; t < lp.n_tasks; ++t) {
      const int64_t chunk = ((keys[t] + n[t] - 1) / n[t] + step - 1) / step * step;
      len[t] = static_cast<double>(chunk) + fit.fixed;
      wgs[t] = tiles[t] * n[t];
      moved += n[t] > 1 ? n[t] * bytes[t] : 0;
    }
    if (len[1] > 1.1 * len[0]) return;                     // (task 1 starts last: its shares would be the tail)
    const double alone = std::max(len[0], len[1]) * fit.alone;
    double cost = wgs[0] + wgs[1] <= 256 ? alone : std::max(alone, makespan(wgs[0], len[0], wgs[1], len[1], 256 * fit.R) * fit.R);
    cost = cost / fit.per_us + (moved > 0 ? add_us + moved / add_bytes_us : 0);
    // Items are dealt to XCDs in turn: with an even number of shares an XCD meets few of them.  8 heads over 2 and over 8, 512
    // and 768 rows, bf16: 8, 10 and 12 shares took 3 % more than their odd neighbours.  (Over the drawn shapes six shares took 0.99 to
    // 1.02 of what five and seven take: this decides between ways that are as good as each other.)
    if (n0 >= 4 && n0 % 2 == 0) cost *= 1.03;
    if (best < 0 || cost < best) { best = cost; n_split[0] = n0; n_split[1] = n1; }
  };
  for (const int32_t n : kWays) {
    if (n > 1 && (n - 1) * step >= keys[0]) break;         // (task 0 has the most keys)
    weigh(n, 1);
    if (lp.n_tasks > 1 && n > 1) {
      const int64_t chunk = ((keys[0] + n - 1) / n + step - 1) / step * step;
      const int32_t alike = static_cast<int32_t>((keys[1] + chunk - 1) / chunk);      // shares of the same length
      if (alike > 1) weigh(n, alike);
      if (alike < n) weigh(n, alike + 1);
      if (alike + 1 < n) weigh(n, n);
    }
  }
}

// Whether the kernel for few query tiles is the faster one for a bf16 launch: attn_run_kernel where steps are joined, attn_tile_kernel
// for a step by itself (`step`).  Both kernels' durations are estimated in
// (row, key) pairs a CU walks: the work of all workgroups over the 256 CUs, and not less than what
// the CUs with the most heavy workgroups have.  A workgroup's set-up, first fetches and epilogue count
// as that many keys more.  The large kernel pads query blocks to 256 rows (d = 64: 384 where that fills
// as well), the small one computes only the strips of 32 that have rows.
// Joined steps: where nothing is padded the small one walks a key in 1.04 of the large one's time at d = 128 (935 us against 900, 32 heads over
// 8, 4 096 of 32 768 tokens), in 1.03 at d = 64 against twelve wavefronts and 1.08 against eight that are persistent (4.88 ms against 4.51,
// 4 heads, batch 4, 16 384 of 131 072 tokens); several of its workgroups share a CU.  Over 164 shapes (1K to 430K tokens, both d) the
// choice costs 0.3 % on average against always taking the faster kernel, 23 % at most (20 heads of 64, 7 640 of 30 560 tokens).
// A step by itself is another thing: its partial pairs go out in fp32, its short lists
// leave the small kernel more set-up per key (a key takes 1.14, a lone workgroup uses about half a CU), and there are no shares.  Over 78 shapes of it (256 to 4 700 rows a
// step, both d) the small kernel took 0.53 to 1.01 of the large one's time where its estimate was below kStepMargin
// of the other, and 1.03 to 1.21 above (16 heads over 2, 3 320 rows, no mask: 113.7 us a step against 94.3).
// At d = 64 a second workgroup on a CU lengthened it by 1.4 (4 and 12 heads, 3 072 rows: 48.8 and 68.2 us).
constexpr double kStepMargin = 0.89;
bool tile_is_faster(const AttnLaunch& lp, int d, const int64_t* keys, const int32_t* n_split, bool step = false) {
  constexpr double kCus = 256.0;
  constexpr int kTileRows = tasp::tile_rows(false, 0);
  const double B = static_cast<double>(plan_batch(lp)), G = lp.Hq / lp.Hkv;
  auto padded = [](double x, double m) { return std::ceil(x / m) * m; };
  double rows8 = 0, rows12 = 0;
  for (int t = 0; t < lp.n_tasks; ++t) { rows8 += padded(lp.task[t].n_q, 256); rows12 += padded(lp.task[t].n_q, 384); }
  const double bm = d == 64 && rows12 * 100 <= rows8 * 101 ? 384 : 256, fixed = bm == 384 ? 400 : 900;
  const double a_key = step ? 1.14 : d == 128 ? 1.05 : bm == 384 ? 1.1 : 1.03, start = step ? 300 : 100;
  double big = 0, tile = 0, big_one[tasp::kMaxTasks] = {}, tile_one[tasp::kMaxTasks] = {}, big_n[tasp::kMaxTasks] = {}, tile_n[tasp::kMaxTasks] = {};
  bool split = false;
  for (int t = 0; t < lp.n_tasks; ++t) {
    const double n = lp.task[t].n_q, k = static_cast<double>(keys[t]), ns = n_split[t];
    big_one[t] = bm * (k + fixed);
    big_n[t] = padded(n, bm) / bm * lp.Hq * B;
    big += big_one[t] * big_n[t];
    tile_one[t] = kTileRows * (a_key * k / ns + start);
    tile_n[t] = padded(n * G, kTileRows) / kTileRows * lp.Hkv * B * ns;
    tile += tile_one[t] * padded(n * G, 32) / kTileRows * lp.Hkv * B * ns;
    split |= ns > 1;
  }
  auto duration = [&](double total, const double* one, const double* n, double alone, double pair) {
    const double longest = std::max(one[0], one[1]);
    double heavy = 0;
    for (int t = 0; t < lp.n_tasks; ++t) heavy += one[t] > 0.7 * longest ? n[t] : 0;
    const double on_one = std::ceil(heavy / kCus);
    return std::max(total / kCus, longest * std::max(on_one > 1 ? pair : alone, on_one));
  };
  const double sum_shares = split ? 40000 : 0;      // the launch that adds the shares up
  const double small = duration(tile, tile_one, tile_n, step ? 1.8 : 1.6, !step ? 1.4 : d == 64 ? 2.5 : 1.8) + sum_shares;
  return small < (step ? kStepMargin : 1.0) * duration(big, big_one, big_n, 1.0, 1.0);
}

// Decides from shapes alone (`js` holds the joined lists).  Kernel and shares are those for the largest workspace
// that tasp_chunk_attn_best_workspace_bytes could report, wherever the `ws_bytes` of the call hold these shares
// (none do with the large kernel): the results do not depend on who brings the workspace, if it is the reported
// one or larger.  With less the shares are dealt anew, and the kernel is chosen for them.  A call without any workspace
// (fp32 with the merge folded in needs none) has its workgroups take the shares in turn: the same results, without
// the gain, and nothing that calls on other streams could write over.  Only where the shares have more keys than one set of
// sums takes, they are then more (kSumTiles): the results differ in rounding.
FwdPlan plan_forward(const tasp_attn_args* a, const JoinedSteps& js, size_t need, size_t ws_bytes) {
  FwdPlan pl;
  const bool fp32 = a->dtype == TASP_DTYPE_FP32;
  size_t room = std::max<size_t>(need, TASP_STATIC_SCRATCH_BYTES);
  for (;;) {
    int32_t n_split[tasp::kMaxTasks] = {1, 1};
    // a few sequences as one of them by itself, unless the partial pairs of all then take more than there is room for
    const int64_t one = plan_batch(js.all);
    deal_keys(js.all, a->d, fp32, js.keys, SIZE_MAX, n_split, one);
    if (all_share_bytes(js.all, a->d, n_split) > room) deal_keys(js.all, a->d, fp32, js.keys, room, n_split, js.all.batch);
    pl.tile = fp32 || tile_is_faster(js.all, a->d, js.keys, n_split);
    if (!pl.tile) {
      // what is estimated to lose with all shares may win with the few that the least workspace holds, or none (20 heads of 64,
      // 104 832 tokens of 16 ranks in one launch: 2.73 ms, the large kernel 3.30)
      if (room <= need) return pl;
      room = need;
      continue;
    }
    pl.part_bytes = all_share_bytes(js.all, a->d, n_split);
    for (int t = 0; t < js.all.n_tasks; ++t) pl.n_split[t] = n_split[t];
    if (pl.part_bytes <= ws_bytes) return pl;
    if (fp32 && ws_bytes == 0) {
      for (int t = 0; t < js.all.n_tasks && a->d == 128; ++t)
        pl.n_split[t] = std::max(pl.n_split[t], static_cast<int32_t>((js.keys[t] + tasp::kSumTiles * 32 - 1) / (tasp::kSumTiles * 32)));
      pl.serial = true;
      pl.part_bytes = 0;
      return pl;
    }
    room = ws_bytes;                                  // what is dealt for this much fits
    pl = FwdPlan{};
  }
}

// Optional per-launch timing with HIP events on the caller's stream (tasp_chunk_attn_profile).
struct Profiler {
  enum Kind { kAttn = 0, kMerge = 1, kOther = 2 };
  struct Span { int kind; hipEvent_t beg, end; };
  std::vector<Span> spans;
  hipStream_t stream = nullptr;
  bool failed = false;
  void begin(int kind) {
    if (failed) return;
    spans.push_back(Span{kind, nullptr, nullptr});       // pushed first: the destructor owns whatever gets created
    Span& sp = spans.back();
    if (hipEventCreate(&sp.beg) != hipSuccess || hipEventCreate(&sp.end) != hipSuccess ||
        hipEventRecord(sp.beg, stream) != hipSuccess)
      failed = true;
  }
  void end() {
    if (spans.empty() || failed) return;
    if (hipEventRecord(spans.back().end, stream) != hipSuccess) failed = true;
  }
  ~Profiler() {
    for (auto& sp : spans) {
      if (sp.beg) (void)hipEventDestroy(sp.beg);
      if (sp.end) (void)hipEventDestroy(sp.end);
    }
  }
};
struct Scope {
  Profiler* p;
  Scope(Profiler* prof, int kind) : p(prof) { if (p) p->begin(kind); }
  ~Scope() { if (p) p->end(); }
};

hipError_t launch_attn(const AttnLaunch& lp, const tasp_attn_args* a, hipStream_t stream, bool tile, bool serial = false) {
  return tile ? tasp::launch_attn_tile(lp, a->d, a->dtype == TASP_DTYPE_FP32, serial, stream) : tasp::launch_attn_bf16(lp, a->d, stream);
}

// The launch of one step.  With more local rows than kJoinRows the large kernel is within 5 % of the
// faster one wherever it is not that itself.
hipError_t launch_step(const AttnLaunch& lp, const tasp_attn_args* a, hipStream_t stream) {
  if (lp.n_tasks == 0) return hipSuccess;
  int64_t keys[tasp::kMaxTasks] = {0, 0}, rows = 0;
  for (int t = 0; t < lp.n_tasks; ++t) rows += lp.task[t].n_q;
  for (int t = 0; t < lp.n_tasks; ++t)
    for (int i = 0; i < lp.task[t].n_seg; ++i) {
      const int32_t* g = lp.pool + 2 * (lp.task[t].seg0 + i);
      keys[t] += g[1] - g[0];
    }
  return launch_attn(lp, a, stream, a->dtype == TASP_DTYPE_FP32 || (rows <= kJoinRows && tile_is_faster(lp, a->d, keys, lp.n_split, true)));
}

// ---- backward pass
// The forward's argument block with the fields both passes share, so that one validation serves both.
tasp_attn_args as_forward(const tasp_attn_bwd_args* b) {
  tasp_attn_args a{};
  a.q = b->q; a.k = b->k; a.v = b->v;
  a.S = b->S; a.Hq = b->Hq; a.Hkv = b->Hkv; a.d = b->d;
  a.dtype = b->dtype; a.mask_mode = b->mask_mode; a.order = b->order;
  a.fuse_merge = 1; a.softmax_scale = b->softmax_scale; a.batch = b->batch;
  a.fuse_steps = b->fuse_steps;
  return a;
}

int validate_bwd(const tasp_schedule_t* s, const tasp_attn_bwd_args* b, tasp_attn_args* a, Shape* sh) {
  if (s == nullptr || b == nullptr) return TASP_EINVAL;
  *a = as_forward(b);
  int st = validate(s, a, sh);
  if (st != TASP_OK) return st;
  if (b->fuse_steps && b->dtype != TASP_DTYPE_BF16) return TASP_EUNSUPPORTED_SHAPE;   // refused; with few local rows its steps are joined anyway
  if (b->out == nullptr || b->lse == nullptr || b->dout == nullptr || b->dq == nullptr || b->dk == nullptr ||
      b->dv == nullptr)
    return TASP_EINVAL;
  // the bf16 kernels address Q and dout with 32-bit byte offsets
  if (b->dtype == TASP_DTYPE_BF16 && static_cast<int64_t>(sh->L) * b->Hq * b->d * 2 > (int64_t{1} << 32))
    return TASP_EUNSUPPORTED_SHAPE;
  const uintptr_t all = reinterpret_cast<uintptr_t>(b->out) | reinterpret_cast<uintptr_t>(b->dout) |
                        reinterpret_cast<uintptr_t>(b->dq) | reinterpret_cast<uintptr_t>(b->dk) |
                        reinterpret_cast<uintptr_t>(b->dv);
  if (all & 15) return TASP_EALIGN;
  return TASP_OK;
}

// How finely the joined launches of a backward call are cut.
struct BwdPlan {
  size_t table_bytes = 0;      // device memory for the segment lists of fuse_steps
  int32_t n_split = 1;         // workgroups the keys of a query tile are dealt to; their dq sums follow the lists
  int32_t kv_split = 0;        // BwdLaunch::kv_split; the partial dk and dv follow the dq sums
  size_t kv_bytes = 0;         // of one of the two
};

// Workgroups the keys of a query tile of a backward call are dealt to, so that `target` dq workgroups or
// more come together, none with fewer than four 64-key tiles; `tiles` = dq workgroups without that.
int dq_split(int64_t tiles, int64_t target, int64_t S, int64_t room) {
  const int64_t n = std::min(std::min((target + tiles - 1) / tiles, S / 256), std::min(room, kMaxSplit));
  return static_cast<int>(std::max<int64_t>(n, 1));
}

// Device memory the arrays in front of the lists and partial sums take: bf16 -delta and -lse / scale, fp32 delta.
size_t bwd_front_bytes(const tasp_attn_bwd_args* b, const Shape& sh) {
  return b->dtype == TASP_DTYPE_BF16 ? 2 * align_up(sh.lse_bytes + sizeof(float)) : align_up(sh.lse_bytes);
}

struct BwdSpans { enum Kind { kDq = 0, kDkv = 1, kOther = 2 }; };

// Everything of a backward launch that follows from the shapes and the caller's tensors; `ranges` = the keys
// of the launch.
int fill_bwd(const tasp_schedule_t* s, const tasp_attn_bwd_args* b, const AttnLaunch& lp, std::vector<tasp::Segment>& ranges,
             tasp::BwdLaunch* bp) {
  bp->q = b->q; bp->k = b->k; bp->v = b->v; bp->dout = b->dout; bp->lse = b->lse;
  bp->dk = b->dk; bp->dv = b->dv;
  bp->Hq = lp.Hq; bp->Hkv = lp.Hkv; bp->group = tasp::make_divider(static_cast<uint32_t>(lp.Hq / lp.Hkv)); bp->causal = lp.causal; bp->scale = lp.scale; bp->batch = lp.batch;
  bp->q_bstride = lp.q_bstride; bp->kv_bstride = lp.kv_bstride; bp->lse_bstride = lp.lse_bstride;
  bp->n_tasks = lp.n_tasks;
  for (int t = 0; t < lp.n_tasks; ++t) bp->task[t] = lp.task[t];
  std::copy(lp.pool, lp.pool + 2 * tasp::kPoolSeg, bp->pool);
  bp->n_split = 1;
  bp->n_blk = tasp::n_query_blocks(b->mask_mode);
  for (int qb = 0; qb < bp->n_blk; ++qb) {
    tasp::QueryBlock blk;
    const int st = tasp::query_block(*s, b->S, b->mask_mode, qb, &blk);
    if (st != TASP_OK) return st;
    bp->blk[qb] = {static_cast<int32_t>(blk.local_row0), static_cast<int32_t>(blk.rows), static_cast<int32_t>(blk.pos0)};
  }
  // The dk/dv kernel treats every key on its own, so the order of the ranges is free: by
  // position, which under the causal mask is by falling work (early keys are seen by more
  // queries), so that the workgroups with the most work start first.  Neighbours are joined.
  std::sort(ranges.begin(), ranges.end(),
            [](const tasp::Segment& x, const tasp::Segment& y) { return x.start < y.start; });
  size_t n = 0;
  for (size_t i = 0; i < ranges.size(); ++i) {
    if (n > 0 && ranges[n - 1].end == ranges[i].start) ranges[n - 1].end = ranges[i].end;
    else ranges[n++] = ranges[i];
  }
  if (n > static_cast<size_t>(tasp::kMaxSeg)) return TASP_EUNSUPPORTED_SHAPE;
  bp->n_rng = static_cast<int32_t>(n);
  int64_t vpos = 0;
  for (size_t i = 0; i < n; ++i) {
    bp->rng_start[i] = static_cast<int32_t>(ranges[i].start);
    bp->rng_vbeg[i] = static_cast<int32_t>(vpos);
    vpos += ranges[i].end - ranges[i].start;
  }
  bp->rng_vbeg[n] = static_cast<int32_t>(vpos);
  return TASP_OK;
}

// Estimated duration of a dk/dv launch, in 64-row query tiles of one head, with one workgroup per
// key tile (`kv_split` = 0, each serving all G query heads of its group) or per key tile, query head and
// share of the query tiles.  Mirrors what the kernel and the hardware do: the work list is (sequence,
// KV head, head, share, key tile) in that order, every XCD gets one contiguous eighth of it (exactly so when
// the KV heads of the call are a multiple of 8; otherwise XCDs share heads, which this estimate
// ignores, as it does the windows of several KV heads that are met together: xcd_window), and each of its
// slots/8 workgroup slots takes the next workgroup when it is free.  A workgroup walks, for
// each query block, the tiles from the first one that holds a row at or after its first key.
int64_t dkv_makespan(const tasp::BwdLaunch& bp, int d, int kv_split, int64_t batch, int slots) {
  const int bs = d == 128 ? 256 : 128, bt = 64;
  const int64_t total = bp.rng_vbeg[bp.n_rng];
  const int64_t ktiles = (total + bs - 1) / bs;
  const int G = bp.Hq / bp.Hkv;
  std::vector<int32_t> work(static_cast<size_t>(ktiles));
  int j = 0;
  for (int64_t t = 0; t < ktiles; ++t) {
    while (j + 1 < bp.n_rng && bp.rng_vbeg[j + 1] <= t * bs) ++j;     // the range that holds the tile's first key
    // ranges are sorted by position, so the tile's first key is its earliest
    const int64_t tmin = bp.rng_start[j] + (t * bs - bp.rng_vbeg[j]);
    int64_t w = 0;
    for (int qb = 0; qb < bp.n_blk; ++qb) {
      const int64_t tiles = (bp.blk[qb].n + bt - 1) / bt;
      const int64_t first = bp.causal ? std::max<int64_t>(0, (tmin - bp.blk[qb].pos0) / bt) : 0;
      w += std::max<int64_t>(0, tiles - first);
    }
    work[static_cast<size_t>(t)] = static_cast<int32_t>(w);
  }
  const int64_t n = ktiles * bp.Hkv * batch * (kv_split > 0 ? G * kv_split : 1);
  const int xcd_slots = std::max(1, slots / 8);
  constexpr int64_t kFixed = 4;      // set-up and epilogue of a workgroup, in the same unit
  int64_t makespan = 0;
  std::vector<int64_t> heap;
  for (int x = 0; x < 8; ++x) {
    const int64_t q8 = n / 8, r8 = n % 8;
    const int64_t start = x * q8 + std::min<int64_t>(x, r8), cnt = q8 + (x < r8 ? 1 : 0);
    heap.assign(static_cast<size_t>(xcd_slots), 0);
    for (int64_t i = start; i < start + cnt; ++i) {
      const int64_t tile = i % ktiles;
      const int64_t all = work[static_cast<size_t>(tile)];
      const int64_t w = kFixed + (kv_split > 0 ? (all + kv_split - 1) / kv_split : all * G);
      std::pop_heap(heap.begin(), heap.end(), std::greater<int64_t>());
      heap.back() += w;
      std::push_heap(heap.begin(), heap.end(), std::greater<int64_t>());
    }
    makespan = std::max(makespan, *std::max_element(heap.begin(), heap.end()));
  }
  return makespan;
}

// Fills in what depends on shapes alone; `bp` is the joined launch, `ws_bytes` the workspace.
BwdPlan plan_backward(const tasp_attn_bwd_args* b, const Shape& sh, const tasp::BwdLaunch& bp, size_t table_bytes, size_t ws_bytes) {
  BwdPlan pl;
  pl.table_bytes = table_bytes;
  const bool fp32 = b->dtype == TASP_DTYPE_FP32;
  const int64_t G = b->Hq / b->Hkv;
  int64_t tiles_of_one = 0;
  for (int t = 0; t < bp.n_tasks; ++t)
    tiles_of_one += fp32 ? (bp.task[t].n_q * G + 63) / 64 * b->Hkv : static_cast<int64_t>((bp.task[t].n_q + 127) / 128) * b->Hq;
  const int64_t B = plan_batch(sh.B, tiles_of_one);
  size_t used = bwd_front_bytes(b, sh) + table_bytes;
  auto room = [&](size_t each) { return each > 0 && ws_bytes > used ? static_cast<int64_t>((ws_bytes - used) / each) : 0; };
  // dk/dv: finer than by key tile where the estimate says that wins by more than 4 %, the launch that
  // adds the partial sums up (about one tile's time) and their way through memory included
  if (!fp32 && G > 1) {
    const int slots = tasp::bwd_dkv_resident_workgroups(b->d);
    const int64_t wgs = tasp::bwd_dkv_workgroups(bp, b->d) / sh.B * B;
    const size_t one = align_up(static_cast<size_t>(sh.B) * b->S * b->Hq * b->d * sizeof(float));
    int64_t best = 0;
    if (wgs < 8 * static_cast<int64_t>(slots))
      for (const int c : {0, 1, 2, 4}) {
        if (c > 0 && room(2 * one * c) < 1) break;
        const double bytes = 4.0 * static_cast<double>(one) / sh.B * B * c;   // written and read, dk and dv
        const int64_t t = dkv_makespan(bp, b->d, c, B, slots) + (c > 0 ? 1 + static_cast<int64_t>(bytes / 1.5e7) : 0);
        if (c == 0 || t * 104 < best * 100) { best = t; pl.kv_split = c; pl.kv_bytes = one * c; }
      }
    used += 2 * pl.kv_bytes;
  }
  pl.n_split = dq_split(tiles_of_one * B, 512, b->S, room(align_up(sh.o_bytes)));
  return pl;
}
size_t plan_bytes(const BwdPlan& pl, const tasp_attn_bwd_args* b, const Shape& sh) {
  return bwd_front_bytes(b, sh) + pl.table_bytes + (pl.n_split > 1 ? pl.n_split * align_up(sh.o_bytes) : 0) + 2 * pl.kv_bytes;
}

// The joined steps as one launch.  Without fuse_steps the key lists are one segment, the sequence: over
// the steps every key is met once, and what a query row or a key gets from one pair does not depend on the
// others.  With it the lists of the steps follow each other (js: to be placed by the caller).
int build_bwd_joined(const tasp_schedule_t* s, const tasp_attn_bwd_args* b, const tasp_attn_args* a, tasp::BwdLaunch* bp, JoinedSteps* js) {
  AttnLaunch lp{};
  if (b->fuse_steps) {
    const int st = join_steps(s, a, js, true);
    if (st != TASP_OK) return st;
    lp = js->all;
  } else {
    std::vector<tasp::QueryBlock> empty;
    const int st = build_step(s, a, 0, &lp, &empty);        // every query block sees its own diagonal at step 0
    if (st != TASP_OK) return st;
    if (!empty.empty()) return TASP_EUNSUPPORTED_SHAPE;
    lp.pool[0] = 0;
    lp.pool[1] = static_cast<int32_t>(b->S);
    for (int t = 0; t < lp.n_tasks; ++t) { lp.task[t].seg0 = 0; lp.task[t].n_seg = 1; }
  }
  std::vector<tasp::Segment> all(1, tasp::Segment{0, b->S, 0});
  return fill_bwd(s, b, lp, all, bp);
}

}  // namespace

namespace tasp {
thread_local hipError_t g_last_hip_error = hipSuccess;
}

extern "C" {

const char* tasp_last_hip_error(void) { return hipGetErrorString(tasp::g_last_hip_error); }

size_t tasp_chunk_attn_workspace_bytes(const tasp_schedule_t* s, const tasp_attn_args* a) {
  if (s == nullptr || a == nullptr || a->S <= 0 || a->Hq <= 0 || a->d <= 0 || s->n <= 0 || a->batch < 0) return 0;
  const int64_t L = a->S / s->n;
  const size_t B = static_cast<size_t>(batch_of(a));
  const size_t o_bytes = align_up(B * L * a->Hq * a->d * sizeof(float));
  const size_t lse_bytes = align_up(B * L * a->Hq * sizeof(float));
  size_t total = 0;
  if (a->dtype == TASP_DTYPE_BF16) total += o_bytes;              // running fp32 output
  if (a->fuse_steps) return total + align_up(kFusedTableBytes);
  if (!a->fuse_merge) total += o_bytes + lse_bytes;               // partial (out_s, lse_s) of a step
  return total;
}

size_t tasp_chunk_attn_best_workspace_bytes(const tasp_schedule_t* s, const tasp_attn_args* a) {
  const size_t need = tasp_chunk_attn_workspace_bytes(s, a);
  Shape sh;
  if (validate(s, a, &sh) != TASP_OK || !joins(s, a)) return need;
  try {
    JoinedSteps js{};
    if (join_steps(s, a, &js) != TASP_OK) return need;
    const FwdPlan pl = plan_forward(a, js, need, std::max<size_t>(need, TASP_STATIC_SCRATCH_BYTES));
    return std::max(need, pl.part_bytes);
  } catch (...) {
    return need;
  }
}

double tasp_chunk_attn_flops(const tasp_schedule_t* s, const tasp_attn_args* a) {
  if (s == nullptr || a == nullptr) return 0.0;
  if (tasp::check_sequence(*s, a->S, a->mask_mode) != TASP_OK) return 0.0;
  double pairs = 0.0;
  for (int qb = 0; qb < tasp::n_query_blocks(a->mask_mode); ++qb) {
    tasp::QueryBlock blk;
    if (tasp::query_block(*s, a->S, a->mask_mode, qb, &blk) != TASP_OK) return 0.0;
    const double rows = static_cast<double>(blk.rows);
    if (a->mask_mode == TASP_MASK_FULL) pairs += rows * static_cast<double>(a->S);
    else pairs += rows * static_cast<double>(blk.pos0) + rows * (rows + 1.0) / 2.0;   // sum of (p + 1)
  }
  return 4.0 * a->d * a->Hq * pairs * (a->batch > 0 ? a->batch : 1);
}

int tasp_step_attn(const tasp_schedule_t* s, const tasp_attn_args* a, int32_t step, float* o_part,
                   float* lse_part, void* hip_stream) {
  Shape sh;
  int st = validate(s, a, &sh);
  if (st != TASP_OK) return st;
  if (o_part == nullptr || lse_part == nullptr || step < 0 || step >= s->n) return TASP_EINVAL;
  if (reinterpret_cast<uintptr_t>(o_part) & 15) return TASP_EALIGN;
  hipStream_t stream = static_cast<hipStream_t>(hip_stream);
  try {
    AttnLaunch lp{};
    std::vector<tasp::QueryBlock> empty;
    st = build_step(s, a, step, &lp, &empty);
    if (st != TASP_OK) return st;
    lp.o_dst = o_part; lp.lse_dst = lse_part; lp.merge = 0;
    if (launch_step(lp, a, stream) != hipSuccess) return TASP_EHIP;
    for (const auto& blk : empty)
      if (tasp::launch_fill_empty(o_part, lse_part, blk.local_row0, blk.rows, a->Hq, a->d, sh.B, sh.L, stream) !=
          hipSuccess)
        return TASP_EHIP;
  } catch (...) {
    return TASP_ENOMEM;
  }
  return TASP_OK;
}

static int run_chunk_attn(const tasp_schedule_t* s, const tasp_attn_args* a, void* hip_stream, Profiler* prof) {
  Shape sh;
  int st = validate(s, a, &sh);
  if (st != TASP_OK) return st;
  if (a->out == nullptr || a->lse == nullptr) return TASP_EINVAL;
  if (reinterpret_cast<uintptr_t>(a->out) & 15) return TASP_EALIGN;
  const size_t need = tasp_chunk_attn_workspace_bytes(s, a);
  if (need > 0) {
    if (a->workspace == nullptr || a->workspace_bytes < need) return TASP_EWORKSPACE;
    if (reinterpret_cast<uintptr_t>(a->workspace) & (kAlign - 1)) return TASP_EALIGN;
  }
  hipStream_t stream = static_cast<hipStream_t>(hip_stream);

  unsigned char* ws = static_cast<unsigned char*>(a->workspace);
  float* o_run = static_cast<float*>(a->out);           // fp32: the output itself is the running sum
  if (a->dtype == TASP_DTYPE_BF16) { o_run = reinterpret_cast<float*>(ws); ws += align_up(sh.o_bytes); }
  float* o_part = nullptr;
  float* lse_part = nullptr;
  if (!a->fuse_merge && !a->fuse_steps) {
    o_part = reinterpret_cast<float*>(ws); ws += align_up(sh.o_bytes);
    lse_part = reinterpret_cast<float*>(ws);
  }

  try {
    if (joins(s, a)) {
      JoinedSteps js{};
      st = join_steps(s, a, &js);
      if (st != TASP_OK) return st;
      // a call that needs no workspace (need = 0) takes any pointer; one that is not aligned is left alone
      const bool usable = a->workspace != nullptr && (reinterpret_cast<uintptr_t>(a->workspace) & (kAlign - 1)) == 0;
      const FwdPlan pl = plan_forward(a, js, need, usable ? a->workspace_bytes : 0);
      {
        AttnLaunch& all = js.all;
        all.out_final = a->out; all.lse_dst = a->lse; all.merge = 0;
        size_t at = 0;
        for (int t = 0; t < all.n_tasks; ++t) {
          all.n_split[t] = pl.n_split[t];
          if (pl.n_split[t] < 2 || pl.serial) continue;
          const size_t lse = pl.n_split[t] * share_bytes(all, t, a->d) / (a->d + 1);
          all.part_o[t] = reinterpret_cast<float*>(static_cast<unsigned char*>(a->workspace) + at);
          at += align_up(lse * a->d);
          all.part_lse[t] = reinterpret_cast<float*>(static_cast<unsigned char*>(a->workspace) + at);
          at += align_up(lse);
        }
        {
          Scope sc(prof, Profiler::kAttn);
          if (launch_attn(all, a, stream, pl.tile, pl.serial) != hipSuccess) return TASP_EHIP;
        }
        if (pl.part_bytes > 0) {
          Scope sc(prof, Profiler::kOther);
          if (tasp::launch_combine(all, a->d, a->dtype == TASP_DTYPE_FP32, stream) != hipSuccess) return TASP_EHIP;
        }
        return TASP_OK;
      }
    }
    std::vector<tasp::QueryBlock> empty;
    for (int step = 0; step < s->n; ++step) {
      AttnLaunch lp{};
      empty.clear();
      st = build_step(s, a, step, &lp, &empty);
      if (st != TASP_OK) return st;
      if (step == 0) {
        lp.o_dst = o_run; lp.lse_dst = a->lse; lp.merge = 0;
        {
          Scope sc(prof, Profiler::kAttn);
          if (launch_step(lp, a, stream) != hipSuccess) return TASP_EHIP;
        }
        for (const auto& blk : empty)      // cannot happen with the placements of Sec. 3.2.3; kept for safety
          if (tasp::launch_fill_empty(o_run, a->lse, blk.local_row0, blk.rows, a->Hq, a->d, sh.B, sh.L, stream) !=
              hipSuccess)
            return TASP_EHIP;
      } else if (a->fuse_merge) {
        lp.o_dst = o_run; lp.lse_dst = a->lse; lp.merge = 1;
        Scope sc(prof, Profiler::kAttn);
        if (launch_step(lp, a, stream) != hipSuccess) return TASP_EHIP;
      } else {
        lp.o_dst = o_part; lp.lse_dst = lse_part; lp.merge = 0;
        {
          Scope sc(prof, Profiler::kAttn);
          if (launch_step(lp, a, stream) != hipSuccess) return TASP_EHIP;
        }
        // rows that saw no key at this step have nothing to fold in
        for (int t = 0; t < lp.n_tasks; ++t) {
          Scope sc(prof, Profiler::kMerge);
          if (tasp::launch_merge(o_run, a->lse, o_part, lse_part, lp.task[t].q_row0, lp.task[t].n_q, a->Hq, a->d,
                                 sh.B, sh.L, stream) != hipSuccess)
            return TASP_EHIP;
        }
      }
    }
    if (a->dtype == TASP_DTYPE_BF16) {
      Scope sc(prof, Profiler::kOther);
      if (tasp::launch_cast_bf16(o_run, a->out, sh.B * sh.L * a->Hq * a->d, stream) != hipSuccess) return TASP_EHIP;
    }
  } catch (...) {
    return TASP_ENOMEM;
  }
  return TASP_OK;
}

int tasp_chunk_attn(const tasp_schedule_t* s, const tasp_attn_args* a, void* hip_stream) {
  return run_chunk_attn(s, a, hip_stream, nullptr);
}

// Device address of `scratch` on the current device.  Every GPU holds its own copy of the array at
// its own address, so the address is asked for once per device, with that device current, and kept.
static int static_scratch(void** out) {
  constexpr int kMaxDevices = 64;
  static std::mutex mu;
  static void* ptr[kMaxDevices] = {};
  int dev = -1;
  if (tasp::note_hip(hipGetDevice(&dev)) != hipSuccess) return TASP_EHIP;
  if (dev < 0 || dev >= kMaxDevices) return TASP_EUNSUPPORTED_SHAPE;
  std::lock_guard<std::mutex> lock(mu);
  if (ptr[dev] == nullptr) {
    void* p = nullptr;
    if (tasp::note_hip(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch))) != hipSuccess || p == nullptr) return TASP_EHIP;
    ptr[dev] = p;
  }
  *out = ptr[dev];
  return TASP_OK;
}

int tasp_chunk_attn_static(const tasp_schedule_t* s, const tasp_attn_args* a, void* hip_stream) {
  if (s == nullptr || a == nullptr) return TASP_EINVAL;
  Shape sh;
  const int st = validate(s, a, &sh);
  if (st != TASP_OK) return st;
  // workspace_bytes() trusts its arguments; they have been validated above
  const size_t need = tasp_chunk_attn_workspace_bytes(s, a);
  if (need > static_cast<size_t>(TASP_STATIC_SCRATCH_BYTES)) return TASP_EWORKSPACE;
  tasp_attn_args b = *a;
  b.workspace = nullptr;
  b.workspace_bytes = 0;
  if (need > 0) {            // a call that needs no workspace leaves the array alone: such calls may overlap
    const int sp = static_scratch(&b.workspace);
    if (sp != TASP_OK) return sp;
    b.workspace_bytes = TASP_STATIC_SCRATCH_BYTES;
  }
  return run_chunk_attn(s, &b, hip_stream, nullptr);
}

size_t tasp_chunk_attn_bwd_workspace_bytes(const tasp_schedule_t* s, const tasp_attn_bwd_args* b) {
  if (s == nullptr || b == nullptr || b->S <= 0 || b->Hq <= 0 || b->d <= 0 || s->n <= 0 || b->batch < 0) return 0;
  const int64_t L = b->S / s->n;
  const size_t B = static_cast<size_t>(b->batch == 0 ? 1 : b->batch);
  if (b->dtype == TASP_DTYPE_FP32) return align_up(B * L * b->Hq * sizeof(float));   // delta; dq itself is the fp32 accumulator
  const size_t delta_bytes = align_up((B * L * b->Hq + 1) * sizeof(float));   // and the entry behind the last row
  const size_t table = b->fuse_steps ? align_up(kFusedTableBytes) : 0;    // segment lists of the single launch
  const size_t dq_bytes = align_up(B * L * b->Hq * b->d * sizeof(float));
  // step by step with grouped heads: partial dk and dv per query head of a step's L keys, fp32
  const size_t parts = (!b->fuse_steps && b->Hkv > 0 && b->Hq > b->Hkv) ? 2 * dq_bytes : 0;
  return dq_bytes + 2 * delta_bytes + table + parts;   // fp32 dq, delta, lse log2(e)
}

size_t tasp_chunk_attn_bwd_best_workspace_bytes(const tasp_schedule_t* s, const tasp_attn_bwd_args* b) {
  const size_t need = tasp_chunk_attn_bwd_workspace_bytes(s, b);
  tasp_attn_args a;
  Shape sh;
  if (validate_bwd(s, b, &a, &sh) != TASP_OK || !joins(s, &a, true)) return need;
  try {
    tasp::BwdLaunch bp{};
    JoinedSteps js{};
    if (build_bwd_joined(s, b, &a, &bp, &js) != TASP_OK) return need;
    const BwdPlan pl = plan_backward(b, sh, bp, js.segments() > static_cast<size_t>(tasp::kPoolSeg) ? kFusedTableBytes : 0,
                                     std::max<size_t>(need, TASP_STATIC_SCRATCH_BYTES));
    return std::max(need, plan_bytes(pl, b, sh));
  } catch (...) {
    return need;
  }
}

double tasp_chunk_attn_bwd_flops(const tasp_schedule_t* s, const tasp_attn_bwd_args* b) {
  if (s == nullptr || b == nullptr) return 0.0;
  const tasp_attn_args a = as_forward(b);
  return 2.5 * tasp_chunk_attn_flops(s, &a);
}

static int run_chunk_attn_bwd(const tasp_schedule_t* s, const tasp_attn_bwd_args* b, void* hip_stream, Profiler* prof) {
  Shape sh;
  tasp_attn_args a;
  int st = validate_bwd(s, b, &a, &sh);
  if (st != TASP_OK) return st;
  const size_t need = tasp_chunk_attn_bwd_workspace_bytes(s, b);
  if (b->workspace == nullptr || b->workspace_bytes < need) return TASP_EWORKSPACE;
  if (reinterpret_cast<uintptr_t>(b->workspace) & (kAlign - 1)) return TASP_EALIGN;
  hipStream_t stream = static_cast<hipStream_t>(hip_stream);
  // With a second stream from the caller the dk/dv kernels run beside the dq kernels: fork after
  // delta is on its way, join before returning.  The profiled run keeps one stream (its events
  // bracket launches on `stream`).
  // The fp32 launch holds both kinds of workgroup and needs no second stream.
  hipStream_t kv_stream = (b->aux_stream != nullptr && prof == nullptr && b->dtype == TASP_DTYPE_BF16) ? static_cast<hipStream_t>(b->aux_stream) : stream;
  struct Ev {
    hipEvent_t e = nullptr;
    ~Ev() { if (e) (void)hipEventDestroy(e); }
  } fork, join;
  const bool bf16 = b->dtype == TASP_DTYPE_BF16;
  const int64_t n_q_elems = static_cast<int64_t>(sh.B) * sh.L * b->Hq * b->d;
  const int64_t n_rows = static_cast<int64_t>(sh.B) * sh.L * b->Hq;
  // the dk/dv kernel addresses delta and lse2 with 32-bit byte offsets
  if (bf16 && n_rows >= (int64_t{1} << 30)) return TASP_EUNSUPPORTED_SHAPE;
  // Workspace: the row arrays (bwd_front_bytes), then with joined steps what BwdPlan says; step by step for
  // bf16 the fp32 dq and the partial dk and dv of a split launch, room for L keys each.
  const size_t row_block = align_up(sh.lse_bytes + sizeof(float));
  unsigned char* ws = static_cast<unsigned char*>(b->workspace);
  unsigned char* after_rows = ws + bwd_front_bytes(b, sh);
  float* delta = reinterpret_cast<float*>(ws);
  float* lse2 = bf16 ? reinterpret_cast<float*>(ws + row_block) : nullptr;
  float* dq_acc = bf16 ? reinterpret_cast<float*>(after_rows) : static_cast<float*>(b->dq);
  float* part = (bf16 && !b->fuse_steps && b->Hq > b->Hkv) ? reinterpret_cast<float*>(after_rows + align_up(sh.o_bytes)) : nullptr;
  auto set_buffers = [&](tasp::BwdLaunch* bp) {
    if (bf16) { bp->ndelta = delta; bp->nlse = lse2; } else { bp->delta = delta; }
    bp->dq_acc = dq_acc;
  };
  const bool joined = joins(s, &a, true);

  try {
    {
      Scope sc(prof, BwdSpans::kOther);
      const float scale = a.softmax_scale > 0.f ? a.softmax_scale : 1.0f / std::sqrt(static_cast<float>(a.d));   // as the launches below
      if ((bf16 ? tasp::launch_bwd_delta_bf16(b->out, b->dout, b->lse, delta, lse2, scale, n_rows, b->d, stream)
                : tasp::launch_bwd_delta_fp32(b->out, b->dout, delta, n_rows, b->d, stream)) != hipSuccess)
        return TASP_EHIP;
      if (bf16 && !joined && tasp::launch_zero_f32(dq_acc, n_q_elems, stream) != hipSuccess) return TASP_EHIP;
    }
    if (kv_stream != stream) {
      if (tasp::note_hip(hipEventCreateWithFlags(&fork.e, hipEventDisableTiming)) != hipSuccess ||
          tasp::note_hip(hipEventCreateWithFlags(&join.e, hipEventDisableTiming)) != hipSuccess ||
          tasp::note_hip(hipEventRecord(fork.e, stream)) != hipSuccess ||
          tasp::note_hip(hipStreamWaitEvent(kv_stream, fork.e, 0)) != hipSuccess)
        return TASP_EHIP;
    }
    bool first_unit = true;
    // The launches of one step, or of all steps at once.
    auto enqueue = [&](const tasp::BwdLaunch& bp) -> int {
      if (!bf16) {
        // one launch for both kinds of workgroup, except where each is to be timed for itself
        if (prof == nullptr) return tasp::launch_bwd_fp32(bp, b->d, true, true, stream) == hipSuccess ? TASP_OK : TASP_EHIP;
        { Scope sc(prof, BwdSpans::kDq); if (tasp::launch_bwd_fp32(bp, b->d, true, false, stream) != hipSuccess) return TASP_EHIP; }
        { Scope sc(prof, BwdSpans::kDkv); if (tasp::launch_bwd_fp32(bp, b->d, false, true, stream) != hipSuccess) return TASP_EHIP; }
        return TASP_OK;
      }
      {
        Scope sc(prof, BwdSpans::kDq);
        if (tasp::launch_bwd_dq_bf16(bp, b->d, stream) != hipSuccess) return TASP_EHIP;
      }
      {
        Scope sc(prof, BwdSpans::kDkv);
        if (tasp::launch_bwd_dkv_bf16(bp, b->d, kv_stream) != hipSuccess) return TASP_EHIP;
      }
      if (bp.kv_split > 0) {
        Scope sc(prof, BwdSpans::kOther);
        if (tasp::launch_bwd_dkv_reduce(bp, b->d, kv_stream) != hipSuccess) return TASP_EHIP;
      }
      return TASP_OK;
    };
    // One unit = one dq launch and one dk/dv launch: a step.
    auto launch_unit = [&](const AttnLaunch& lp, std::vector<tasp::Segment>& ranges) -> int {
      tasp::BwdLaunch bp{};
      const int st2 = fill_bwd(s, b, lp, ranges, &bp);
      if (st2 != TASP_OK) return st2;
      set_buffers(&bp);
      // A step's key tiles are few (S / N keys) and under the causal mask their work differs by
      // whole multiples (a tile is seen by both local half-chunks, by one, or by none), so the
      // launch ends with most CUs idle while a few finish a second tile.  Such a launch is cut
      // finer, one workgroup per key tile and query head; the partial sums are added up afterwards.
      // The finer launch costs a little where the coarse one is already even (partial sums written
      // and read back, more workgroup set-ups), so it is used where the estimate says it wins by more
      // than 4 %.
      const int64_t wgs = tasp::bwd_dkv_workgroups(bp, b->d);
      const int slots = tasp::bwd_dkv_resident_workgroups(b->d);
      if (part != nullptr && bp.rng_vbeg[bp.n_rng] <= sh.L && wgs > 0 && wgs < 8 * static_cast<int64_t>(slots) &&
          dkv_makespan(bp, b->d, 1, sh.B, slots) * 104 < dkv_makespan(bp, b->d, 0, sh.B, slots) * 100) {
        bp.kv_split = 1;
        bp.part_dk = part;
        bp.part_dv = reinterpret_cast<float*>(reinterpret_cast<unsigned char*>(part) + align_up(sh.o_bytes));
      }
      bp.accumulate = bf16 || !first_unit ? 1 : 0;      // fp32: every query row sees its own diagonal at step 0
      first_unit = false;
      return enqueue(bp);
    };
    // All steps in one launch of each kind.
    auto launch_joined = [&]() -> int {
      tasp::BwdLaunch bp{};
      JoinedSteps js{};
      int st2 = build_bwd_joined(s, b, &a, &bp, &js);
      if (st2 != TASP_OK) return st2;
      set_buffers(&bp);
      const bool listed = js.segments() > static_cast<size_t>(tasp::kPoolSeg);
      const BwdPlan pl = plan_backward(b, sh, bp, listed ? kFusedTableBytes : 0, std::min(b->workspace_bytes, std::max<size_t>(need, TASP_STATIC_SCRATCH_BYTES)));
      if (listed) {
        Scope sc(prof, BwdSpans::kOther);
        st2 = place_lists(js, &bp, reinterpret_cast<int32_t*>(after_rows), stream);
        if (st2 != TASP_OK) return st2;
      }
      unsigned char* at = after_rows + pl.table_bytes;
      bp.n_split = pl.n_split;
      bp.dq_final = bf16 && pl.n_split == 1 ? b->dq : nullptr;
      bp.part_dq = reinterpret_cast<float*>(at);
      bp.part_stride = static_cast<int64_t>(align_up(sh.o_bytes) / sizeof(float));
      if (pl.n_split > 1) at += pl.n_split * align_up(sh.o_bytes);
      bp.kv_split = pl.kv_split;
      bp.part_dk = reinterpret_cast<float*>(at);
      bp.part_dv = reinterpret_cast<float*>(at + pl.kv_bytes);
      st2 = enqueue(bp);
      if (st2 == TASP_OK && pl.n_split > 1) {
        Scope sc(prof, BwdSpans::kOther);
        if (tasp::launch_bwd_sum(bp.part_dq, bp.part_stride, pl.n_split, b->dq, bf16, n_q_elems, stream) != hipSuccess) return TASP_EHIP;
      }
      return st2;
    };
    // All units; returns at the first failure, and the join below runs either way so that the
    // caller's second stream is never left forked (which would also break a stream capture).
    auto walk = [&]() -> int {
      std::vector<tasp::QueryBlock> empty;
      std::vector<tasp::Segment> ranges;
      if (joined) return launch_joined();
      for (int step = 0; step < s->n; ++step) {
        AttnLaunch lp{};
        empty.clear();
        st = build_step(s, &a, step, &lp, &empty);
        if (st != TASP_OK) return st;
        st = tasp::step_key_ranges(*s, b->S, b->mask_mode, b->order, step, &ranges);
        if (st != TASP_OK) return st;
        st = launch_unit(lp, ranges);
        if (st != TASP_OK) return st;
      }
      return TASP_OK;
    };
    st = walk();
    if (kv_stream != stream) {
      if (tasp::note_hip(hipEventRecord(join.e, kv_stream)) != hipSuccess ||
          tasp::note_hip(hipStreamWaitEvent(stream, join.e, 0)) != hipSuccess)
        return st != TASP_OK ? st : TASP_EHIP;
    }
    if (st != TASP_OK) return st;
    if (bf16 && !joined) {
      Scope sc(prof, BwdSpans::kOther);
      if (tasp::launch_cast_bf16(dq_acc, b->dq, n_q_elems, stream) != hipSuccess) return TASP_EHIP;
    }
  } catch (...) {
    return TASP_ENOMEM;
  }
  return TASP_OK;
}

int tasp_chunk_attn_bwd(const tasp_schedule_t* s, const tasp_attn_bwd_args* b, void* hip_stream) {
  return run_chunk_attn_bwd(s, b, hip_stream, nullptr);
}

int tasp_chunk_attn_bwd_profile(const tasp_schedule_t* s, const tasp_attn_bwd_args* b, void* hip_stream,
                                tasp_bwd_profile* out) {
  if (out == nullptr) return TASP_EINVAL;
  *out = tasp_bwd_profile{};
  try {
    Profiler prof;
    prof.stream = static_cast<hipStream_t>(hip_stream);
    const int st = run_chunk_attn_bwd(s, b, hip_stream, &prof);
    if (tasp::note_hip(hipStreamSynchronize(prof.stream)) != hipSuccess) return TASP_EHIP;
    if (st != TASP_OK) return st;
    if (prof.failed) return TASP_EHIP;
    for (const auto& sp : prof.spans) {
      float ms = 0.f;
      if (hipEventElapsedTime(&ms, sp.beg, sp.end) != hipSuccess) return TASP_EHIP;
      if (sp.kind == BwdSpans::kDq) { out->dq_ms += ms; ++out->dq_launches; }
      else if (sp.kind == BwdSpans::kDkv) { out->dkv_ms += ms; ++out->dkv_launches; }
      else { out->other_ms += ms; ++out->other_launches; }
    }
  } catch (...) {
    return TASP_ENOMEM;
  }
  return TASP_OK;
}

int tasp_chunk_attn_profile(const tasp_schedule_t* s, const tasp_attn_args* a, void* hip_stream,
                            tasp_profile* out) {
  if (out == nullptr) return TASP_EINVAL;
  *out = tasp_profile{};
  try {
    Profiler prof;
    prof.stream = static_cast<hipStream_t>(hip_stream);
    const int st = run_chunk_attn(s, a, hip_stream, &prof);
    if (tasp::note_hip(hipStreamSynchronize(prof.stream)) != hipSuccess) return TASP_EHIP;
    if (st != TASP_OK) return st;
    if (prof.failed) return TASP_EHIP;
    for (const auto& sp : prof.spans) {
      float ms = 0.f;
      if (hipEventElapsedTime(&ms, sp.beg, sp.end) != hipSuccess) return TASP_EHIP;
      if (sp.kind == Profiler::kAttn) { out->attn_ms += ms; ++out->attn_launches; }
      else if (sp.kind == Profiler::kMerge) { out->merge_ms += ms; ++out->merge_launches; }
      else { out->other_ms += ms; ++out->other_launches; }
    }
  } catch (...) {
    return TASP_ENOMEM;
  }
  return TASP_OK;
}

}  // extern "C"
