// Launch descriptors shared by the host orchestration and the kernels of this library.
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

#include "divider.hpp"

namespace tasp {

constexpr int kMaxSeg = 64;      // KV segments one query block can see in one step (2(N-1) for zig-zag)
constexpr int kMaxTasks = 2;     // query blocks per step (the two half-chunks of the zig-zag layout)
// Rows (local row, head of the group) of a query tile of attn_tile_kernel and attn_run_kernel.
constexpr int tile_rows(bool fp32, int d) { return fp32 && d == 128 ? 256 : 128; }
// Tiles of 32 keys that attn_tile_kernel<float, 128> adds up in registers before their sums join those in memory.
constexpr int kSumTiles = 512;
constexpr int kMaxSegAll = 1024; // segments of one query block over ALL steps (steps joined in one launch)
// Segments a launch descriptor holds, all its query blocks together.  A launch of all steps of eight
// ranks fits (at most 112 + 56) and so do most of twelve; longer lists go through device memory, which
// costs a launch of their own.  The descriptor travels as kernel arguments: below 4 KiB.
constexpr int kPoolSeg = 384;
static_assert(kPoolSeg >= kMaxTasks * kMaxSeg, "one step always fits");

// One query block of one launch: rows [q_row0, q_row0 + n_q) of the local Q, contiguous in the
// sequence from q_pos0, attending to the concatenation of its n_seg segments: (start, end) pairs of
// the descriptor's pool from index seg0 on.
struct AttnTask {
  int32_t q_row0;
  int32_t n_q;
  int32_t q_pos0;
  int32_t n_seg;
  int32_t seg0;
};

struct AttnLaunch {
  const void* q;      // [L, Hq, d]
  const void* k;      // [S, Hkv, d]
  const void* v;      // [S, Hkv, d]
  float* o_dst;       // [L, Hq, d] fp32
  float* lse_dst;     // [L, Hq]    fp32
  int32_t Hq, Hkv;
  int32_t causal;     // key t visible to query p iff t <= p
  int32_t merge;      // 0: dst = partial of this step; 1: dst = update_out_lse(dst, partial)
  float scale;        // softmax scale (natural units)
  int32_t last_key;   // position of the last key of the sequence
  int32_t batch;      // independent sequences; element strides between them:
  int64_t q_bstride, kv_bstride, o_bstride, lse_bstride;
  int32_t n_tasks;
  AttnTask task[kMaxTasks];
  int32_t n_items;    // work items of the launch, for persistent workgroups; filled in by the launcher
  void* out_final;    // not null: the rows are final and go here in the inputs' type, not to o_dst (merge = 0)
  // attn_tile_kernel, attn_run_kernel: task t's keys are dealt to n_split[t] workgroups per query tile.  Where that is
  // more than one, share i leaves its normalised pair in part_o[t], part_lse[t] ([n_split, B, n_q, Hq(, d)],
  // the task's rows only) for launch_combine; tasks with one share write their rows themselves.
  int32_t n_split[kMaxTasks];
  float* part_o[kMaxTasks];
  float* part_lse[kMaxTasks];
  int32_t all_steps;  // the steps of the call are joined in this launch: every task has one segment, from key 0 on
  int32_t pool[2 * kPoolSeg];
};
static_assert(sizeof(AttnLaunch) <= 4096, "kernel arguments");

// One contiguous run of local query rows (a half-chunk of the zig-zag layout, or all rows).
struct BwdBlock {
  int32_t row0, n, pos0;   // first local row, rows, global position of the first row
};

// One step of the backward pass.  The dq kernel uses the forward's tasks (query block + the key
// segments it can see); the dk/dv kernel uses every key range that arrives at the step, laid end to
// end (rng_vbeg = start of each range in that concatenation), and the query blocks.
struct BwdLaunch {
  const void* q;        // [B, L, Hq, d] bf16 (fp32 for the fp32 kernel, as k, v, dout, dk, dv)
  const void* k;        // [B, S, Hkv, d]
  const void* v;
  const void* dout;     // [B, L, Hq, d]
  const float* lse;     // [B, L, Hq] final lse of the forward pass
  const float* delta;   // [B, L, Hq] sum_d dout * out (fp32 kernel)
  const float* ndelta;  // [B, L, Hq] -delta, then one 0 (bf16 kernels)
  const float* nlse;    // [B, L, Hq] -lse / scale, -inf where lse is -inf (the row saw no key), then one -inf (bf16 kernels)
  float* dq_acc;        // [B, L, Hq, d] fp32, accumulated into
  void* dk;             // [B, S, Hkv, d] bf16; the rows of this step's keys are written
  void* dv;
  int32_t Hq, Hkv;
  Divider group;        // by Hq / Hkv
  int32_t causal;
  float scale;
  int32_t batch;
  int64_t q_bstride, kv_bstride, lse_bstride;   // elements between sequences
  int32_t n_tasks;
  AttnTask task[kMaxTasks];
  // The lists of all steps may not fit the pool: they then live in device memory, task[t].n_seg (start, end) pairs at
  // seg_ext[t], and the pool is unused.
  const int32_t* seg_ext[kMaxTasks];
  int32_t pool[2 * kPoolSeg];
  int32_t n_blk;
  BwdBlock blk[kMaxTasks];
  int32_t n_rng;
  int32_t rng_start[kMaxSeg];
  int32_t rng_vbeg[kMaxSeg + 1];
  // dk/dv launch split finer than by key tile, for launches whose key tiles alone are too few and too
  // unequal to fill the chip: a workgroup per key tile, query head of the group and share of the query
  // tiles (kv_split > 0 shares: share i takes every kv_split-th tile).  The workgroups write fp32 partial sums
  // [B, Hq / Hkv, kv_split, keys of the launch, Hkv, d] (unscaled, keys in the order of the concatenated
  // ranges) and launch_bwd_dkv_reduce adds them up in a fixed order.  0: not split.
  int32_t kv_split;
  float* part_dk;
  float* part_dv;
  // The keys of a query tile are dealt to n_split workgroups; with more than one their dq sums go
  // to part_dq + i part_stride for launch_bwd_sum.  With one, dq_final (not null) takes the rows as bf16,
  // otherwise dq_acc is added to (accumulate) or written.
  int32_t n_split, accumulate;
  float* part_dq;
  int64_t part_stride;
  void* dq_final;
  // the work items of the launch and what else the bf16 kernels divide by; filled in by the launchers
  XcdMap map;
  Divider by_kv_heads, by_n_split, by_ktiles;
};
static_assert(sizeof(BwdLaunch) <= 4096, "kernel arguments");

// Last HIP error this thread saw inside the library (hipSuccess if none); see tasp_last_hip_error().
extern thread_local hipError_t g_last_hip_error;
inline hipError_t note_hip(hipError_t e) {
  if (e != hipSuccess) g_last_hip_error = e;
  return e;
}

// Launch with a clean error slot: an error left behind by an earlier, unrelated HIP call in this
// thread must not be mistaken for a failure of this launch.
#define TASP_LAUNCH(kernel, grid, block, stream, ...)                         \
  ({                                                                          \
    (void)hipGetLastError();                                                  \
    hipLaunchKernelGGL(kernel, grid, block, 0, stream, __VA_ARGS__);          \
    ::tasp::note_hip(hipGetLastError());                                      \
  })

// Implemented in attn_bf16.hip / attn_tile.hip / merge.hip.  Each returns a hipError_t from the launch.
hipError_t launch_attn_bf16(const AttnLaunch& p, int d, hipStream_t stream);
// `serial` (fp32, out_final): a workgroup takes all shares of its tile in turn, without part_o and part_lse.
hipError_t launch_attn_tile(const AttnLaunch& p, int d, bool fp32, bool serial, hipStream_t stream);
// bf16, joined steps, final rows: what launch_attn_tile passes on.  Implemented in attn_run.hip, whose fetches run up to three tiles past the
// last key with 32-bit offsets from the share's first key.
inline bool attn_run_takes(const AttnLaunch& p, int d) {
  return (d == 64 || d == 128) && p.all_steps != 0 && p.merge == 0 && p.out_final != nullptr &&
         (static_cast<int64_t>(p.last_key) + 1 + 256) * p.Hkv * d * 2 <= (int64_t{1} << 32);
}
hipError_t launch_attn_run(const AttnLaunch& p, int d, hipStream_t stream);
// After a launch_attn_tile with several shares: the rows of out_final and lse_dst from the pairs of the shares.
hipError_t launch_combine(const AttnLaunch& p, int d, bool fp32, hipStream_t stream);
// rows [row0, row0 + rows) of every one of `batch` sequences of L rows each
hipError_t launch_merge(float* o_acc, float* lse_acc, const float* o_part, const float* lse_part,
                        int64_t row0, int64_t rows, int32_t heads, int32_t d, int32_t batch, int64_t L,
                        hipStream_t stream);
hipError_t launch_fill_empty(float* o, float* lse, int64_t row0, int64_t rows, int32_t heads, int32_t d,
                             int32_t batch, int64_t L, hipStream_t stream);
hipError_t launch_cast_bf16(const float* src, void* dst, int64_t n, hipStream_t stream);
// Writes n host integers to device memory with small kernels that carry them as arguments (no copy
// from host memory is enqueued, so the call can be recorded into a graph).
hipError_t launch_write_i32(int32_t* dst, const int32_t* host_vals, int64_t n, hipStream_t stream);
// Implemented in attn_bwd_bf16.hip.
hipError_t launch_bwd_dq_bf16(const BwdLaunch& p, int d, hipStream_t stream);
hipError_t launch_bwd_dkv_bf16(const BwdLaunch& p, int d, hipStream_t stream);
// after a launch with kv_split: dk, dv = sum over the query heads of the partial sums, as bf16
hipError_t launch_bwd_dkv_reduce(const BwdLaunch& p, int d, hipStream_t stream);
// workgroups of the dk/dv launch without the split, and how many of them the chip holds at once
int64_t bwd_dkv_workgroups(const BwdLaunch& p, int d);
int bwd_dkv_resident_workgroups(int d);
// ndelta[r] = -sum_d dout out and nlse[r] = -lse[r] / scale (-inf for -inf) for the n_rows (row, head)
// pairs; both arrays hold n_rows + 1 floats, the last one being 0 and -inf.
hipError_t launch_bwd_delta_bf16(const void* out, const void* dout, const float* lse, float* ndelta, float* nlse,
                                 float scale, int64_t n_rows, int d, hipStream_t stream);
hipError_t launch_zero_f32(float* dst, int64_t n, hipStream_t stream);   // n a multiple of 4, dst 16-byte aligned
// Implemented in attn_bwd_fp32.hip (all tensors fp32; dq_acc is dq itself): the dq and the dk/dv
// workgroups of a launch, in one grid where both are asked for.
hipError_t launch_bwd_fp32(const BwdLaunch& p, int d, bool dq, bool dkv, hipStream_t stream);
// dst (fp32, or bf16) = sum over i < n of the n_elems floats at parts + i stride, in order
hipError_t launch_bwd_sum(const float* parts, int64_t stride, int n, void* dst, bool bf16, int64_t n_elems, hipStream_t stream);
hipError_t launch_bwd_delta_fp32(const void* out, const void* dout, float* delta, int64_t n_rows, int d,
                                 hipStream_t stream);

}  // namespace tasp
