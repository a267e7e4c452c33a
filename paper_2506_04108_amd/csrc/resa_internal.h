// Internal interface between the C-ABI layer (api.cpp) and the kernel launchers.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "resa.h"
#include "resa_device.h"

namespace resa {

// Eq. 5 (Sec. 2.1) in integer arithmetic; `keep_ppm` = round((1 - s) * 1e6).
// n = min(M, max(min_blocks, n_local, ceil(M * keep_ppm / 1e6))); 0 if M <= 0.
__host__ __device__ inline int32_t count_selected(int32_t M, int32_t keep_ppm,
                                                  int32_t min_blocks, int32_t n_local) {
  if (M <= 0) return 0;
  int64_t n = ((int64_t)M * keep_ppm + 999999) / 1000000;
  if (n < min_blocks) n = min_blocks;
  if (n < n_local) n = n_local;
  if (n > M) n = M;
  return (int32_t)n;
}

// Plain-value view of a resa_kv_cache_t for kernel arguments.
struct CacheArgs {
  const uint16_t* k;
  const uint16_t* v;
  uint16_t* kmin;
  uint16_t* kmax;
  int32_t batch, kv_heads, capacity, block_size, max_blocks;  // max_blocks = capacity / b
  int32_t log2_block;        // log2(block_size)
  const int32_t* table;      // paged layout: block table [batch, max_blocks], else nullptr
  int32_t num_pages;
};

// Row (of head_dim elements) of k / v that holds token t of group (bb, hk),
// or -1 when the block table sends its block outside the page pool.
__device__ __forceinline__ int64_t kv_row(const CacheArgs& c, int bb, int hk, int t) {
  if (c.table == nullptr) return ((int64_t)bb * c.kv_heads + hk) * c.capacity + t;
  const int m = t >> c.log2_block;
  const int page = c.table[(size_t)bb * c.max_blocks + m];
  if ((unsigned)page >= (unsigned)c.num_pages) return -1;
  return ((int64_t)page * c.kv_heads + hk) * c.block_size + (t - (m << c.log2_block));
}

// Eq. 3 over one wave: lane (r, c) has folded dims [8c, 8c + 8) of rows r,
// r + 4, ... of block m into mn / mx (fp32 bit patterns of bf16 values, so
// exact); the four row groups are combined across lanes and lanes 0 .. 15
// store the block's kmin / kmax row. Every lane must be active.
__device__ __forceinline__ void fold_minmax(const U4& x, float (&mn)[8], float (&mx)[8]) {
  const uint32_t w[4] = {x.x, x.y, x.z, x.w};
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    mn[2 * j] = fminf(mn[2 * j], bf_lo(w[j]));
    mn[2 * j + 1] = fminf(mn[2 * j + 1], bf_hi(w[j]));
    mx[2 * j] = fmaxf(mx[2 * j], bf_lo(w[j]));
    mx[2 * j + 1] = fmaxf(mx[2 * j + 1], bf_hi(w[j]));
  }
}
__device__ __forceinline__ void store_summary(const CacheArgs& c, size_t grp, int m, int r, int col,
                                              float (&mn)[8], float (&mx)[8]) {
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    mn[j] = fminf(mn[j], __shfl_xor(mn[j], 16));
    mx[j] = fmaxf(mx[j], __shfl_xor(mx[j], 16));
    mn[j] = fminf(mn[j], __shfl_xor(mn[j], 32));
    mx[j] = fmaxf(mx[j], __shfl_xor(mx[j], 32));
  }
  if (r == 0) {
    const size_t so = (grp * c.max_blocks + m) * kHeadDim + col;
    st16(c.kmin + so, U4{pack_exact(mn[0], mn[1]), pack_exact(mn[2], mn[3]),
                         pack_exact(mn[4], mn[5]), pack_exact(mn[6], mn[7])});
    st16(c.kmax + so, U4{pack_exact(mx[0], mx[1]), pack_exact(mx[2], mx[3]),
                         pack_exact(mx[4], mx[5]), pack_exact(mx[6], mx[7])});
  }
}

struct SelectArgs {
  CacheArgs c;
  const uint16_t* q;
  int32_t q_heads, group;      // group = q_heads / kv_heads
  const int32_t* seq_lens;
  int32_t max_blocks_seq;      // ceil(max_seq_len / b): row stride of the score array
  int32_t keep_ppm, min_blocks, n_local;
  uint32_t* keys;              // workspace [B, Hkv, score_stride]: order-preserving keys, 16-byte aligned rows
  int32_t score_stride;        // max_blocks_seq rounded up to a multiple of 4
  float* scores_out;           // optional [B, Hkv, max_blocks_seq]
  int32_t* block_idx;          // [B, Hkv, n_cap]
  int32_t* num_sel;            // [B, Hkv]
  int32_t n_cap;
  uint32_t* hist;              // [B, Hkv, workgroups, 256] per-workgroup key-digit counts
  uint32_t* counters;          // [B, Hkv], zero between calls
  int32_t blocks_per_wg;
  int32_t fused;               // top-n in the scoring kernel's last workgroup
  // Append fused in front of the selection (null k_new: plain selection).
  const uint16_t* k_new;       // [B, Hkv, D] key of the new token
  const uint16_t* v_new;       // [B, Hkv, D] value of the new token
  int32_t* lens_out;           // seq_lens, written once every group of the sequence is done
  uint32_t* seq_counters;      // [B], zero between calls
  uint32_t* window;            // [B, Hkv] digit-window hint kept across calls (any value is valid)
  uint32_t* stats;             // [B, Hkv] calls whose top-n finished on the in-window path (diagnostic)
  // Written by the scoring when the hint is set (fused top-n), for the
  // top-n's in-window path: per block, a bit for a key above the window,
  // and each range's in-window keys grouped by digit, descending.
  uint32_t* above_bits;        // [B, Hkv, bits_stride]
  int32_t bits_stride;         // words per group: ceil(max_blocks_seq / 32) rounded to 4
  uint64_t* win_keys;          // [B, Hkv, score_stride]: range r's list at its first block
};

struct DecodeArgs {
  CacheArgs c;
  const uint16_t* q;
  int32_t q_heads, group;
  const int32_t* seq_lens;
  const int32_t* block_idx;
  const int32_t* num_sel;
  int32_t n_cap, num_splits;
  float scale_log2;            // sm_scale * log2(e)
  float* out;                  // [B, Hq, D]
  float* lse;                  // [B, Hq] or null
  float* part_o;               // [B, Hkv, S, G, D]
  float* part_lse;             // [B, Hkv, S, G]
  uint32_t* counters;          // [B, Hkv] split tickets, zero between calls
  uint32_t* epochs;            // [B, Hkv] merged calls so far (kept from call to call)
  uint64_t* flags;             // [B, Hkv, S] split partial published: (epoch + 1) << 32 | S
};

struct RectifyArgs {
  CacheArgs c;
  const uint16_t* q_f;         // [B, Hq, f, D]
  const uint16_t* k_f;         // [B, Hkv, f, D]
  const uint16_t* v_f;
  int32_t q_heads, group, f;
  const int32_t* seq_lens;
  int32_t max_seq_len;
  int32_t chunk;               // keys per split
  int32_t num_splits;          // ceil(max_seq_len / chunk)
  int32_t ref_keys;            // keys a softmax reference serves, a multiple of 64
  int32_t num_qblocks;         // query blocks per group
  float scale_log2;
  float* out;                  // [B, Hq, f, D]
  float* lse;                  // [B, Hq, f] or null
  float* part_o;               // [B, Hkv, S, G*f, D]
  float* part_lse;             // [B, Hkv, S, G*f]
  int32_t refresh;
  const int32_t* seq_mask;     // [B]: sequences with 0 are left untouched (null: every sequence)
};

// Launchers: enqueue on `stream`; return the hipError_t of the launch.
hipError_t launch_summarize(const CacheArgs& c, const int32_t* seq_lens, int32_t blk_begin,
                            int32_t blk_end, hipStream_t stream);
hipError_t launch_append(const CacheArgs& c, const uint16_t* k_new, const uint16_t* v_new,
                         int32_t* seq_lens, hipStream_t stream);
hipError_t launch_select(const SelectArgs& a, hipStream_t stream);
hipError_t launch_decode(const DecodeArgs& a, hipStream_t stream);
hipError_t launch_rectify(const RectifyArgs& a, hipStream_t stream);
hipError_t launch_clear(void* p, size_t bytes, hipStream_t stream);
hipError_t launch_stream_read(const void* buf, size_t bytes, uint32_t* sink, uint32_t match,
                              int32_t workgroups, hipStream_t stream);

// Split-count and chunk heuristics (host).
int32_t select_fused_max_blocks();
int32_t select_blocks_per_wg(int32_t batch, int32_t kv_heads, int32_t max_blocks_seq);
int32_t select_hist_words(int32_t batch, int32_t kv_heads, int32_t max_blocks_seq);
int32_t decode_auto_splits(int32_t batch, int32_t kv_heads, int32_t n_cap, int32_t block_size);
int32_t rectify_num_qblocks(int32_t group, int32_t f);
int32_t rectify_chunk(int32_t batch, int32_t kv_heads, int32_t rows, int32_t max_seq_len, bool masked);
int32_t rectify_ref_keys(int32_t batch, int32_t kv_heads, int32_t rows, int32_t max_seq_len);
// An upper bound on the key splits of any call with lengths up to
// max_seq_len, non-decreasing in max_seq_len (workspace sizing).
int32_t rectify_max_splits(int32_t batch, int32_t kv_heads, int32_t rows, int32_t max_seq_len);

}  // namespace resa
