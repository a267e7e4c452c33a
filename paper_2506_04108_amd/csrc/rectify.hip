// Dense rectification (Sec. 2.2; Alg. 1 "DenseForward" every f steps) on
// gfx950 matrix cores.
//
// The f re-encoded query rows of a (sequence, kv head) group, times its g
// heads, are R = g * f rows (row rho = r * g + h sits at position L - f + r).
// Against the whole cache they form a dense contraction, so this is the one
// place the library uses MFMA.
//
// k_rectify_attn: workgroups of 4 waves (128 rows, 32-key tiles; windows of up
// to 128 rows, two workgroups per CU) or 8 waves (256 rows, 64-key tiles;
// longer windows such as prefill, one per CU), each wave owning 32 query
// rows. A workgroup walks its split of the key range tile by tile:
//   S^T = K . Q^T        (v_mfma_f32_32x32x16_bf16, keys x queries; lane l
//                          holds query l % 32 and keys 8 (i / 4) + 4 (l / 32)
//                          + i % 4, i = 0 .. 15, of each 32)
//   online softmax per query row in the log2 domain; weights P are rounded
//   to fp16 (11 significant bits)
//   O^T += V^T . P^T     (v_mfma_f32_32x32x16_f16, dims x queries; the
//                          contraction index is ordered so that P^T is
//                          already in the B-operand layout, and V^T comes
//                          from the row-major V tile through the LDS
//                          transpose read)
//
// The round of a tile is software-pipelined: its weights are formed while the
// matrix cores produce the next tile's scores (two MFMAs, then the VALU work
// of a few weights, kept in that order by scheduling barriers), then its P.V
// runs while the V of the tile after next is converted. Two things keep the
// VALU work per weight at fma, exp2, add and half a conversion: the row
// maximum is not taken per tile (see kMaxWeightSum), and every LDS read
// address is a per-lane constant plus an immediate (four K and four V stages,
// rounds unrolled by four). K rows go from HBM straight into LDS (buffer
// loads with the LDS destination), V rows through two registers per thread,
// converted to fp16 once per workgroup. One barrier per two tiles publishes
// both. What it measured (8 x 32/8 heads, 8K prompts / one 32K prompt, whole
// call): 5893 -> 4190 us and 10594 -> 7770 us against the earlier kernel
// (16x16x32 MFMAs, scores -> softmax -> P.V in series with a row maximum and
// a barrier per tile). The matrix cores are busy 53 % of the cycles and the
// VALU 51 %, at 1.9 GHz: the chip is at its power limit (the same launch on
// all-zero inputs runs the same cycles at 2.4 GHz, 6540 us), as are library
// matrix products (91 % busy at 1.7 GHz), so what is left is energy and
// cycles in equal parts. Measured and slower: 8-wave workgroups in two
// half-round phases (8050 against 7910 us), V staged raw in LDS three tiles
// ahead (8850 against 8540), one barrier per tile (7930 against 7770).
//
// V is used in fp16. Every bf16 value of magnitude 2^-14 .. 65280 is an fp16
// value (8 significant bits fit in 11), so in that range the conversion is
// exact; smaller values keep fp16's subnormal spacing of 2^-24 (an error of at
// most 2^-24 * P per key). A value above 65504 is noticed when it is
// converted; the workgroup then finishes the pass and takes its range again
// with V split by magnitude (see kBandExp), each part exact in fp16, so that
// every finite bf16 V gives a finite result and no row loses precision to a
// value it does not see. Such values do not occur in a model's caches: the
// second pass is a plain loop (64K rectification, batch 8: 1143 us with one
// large value in every group, 400 with none).
// Masking (causal cut, end of the split) is only evaluated on the tiles that
// reach it. A second kernel merges the splits by log-sum-exp (Alg. 2,
// "Combine"), spread over many workgroups.
#include <type_traits>

#include "resa_device.h"
#include "resa_internal.h"

namespace resa {
namespace {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef _Float16 f16x8_t __attribute__((ext_vector_type(8)));
typedef _Float16 f16x4_t __attribute__((ext_vector_type(4)));
typedef _Float16 f16x2_t __attribute__((ext_vector_type(2)));
typedef short i16x4_t __attribute__((ext_vector_type(4)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));
typedef int32_t i32x4_t __attribute__((ext_vector_type(4)));

constexpr int kRowsPerWave = 32;
__host__ __device__ constexpr int waves_for_rows(int rows) { return rows > 128 ? 8 : 4; }
constexpr int kMaxKeyTile = 64;
constexpr int kCus = 256;
// Whether a workgroup of a launch takes two query blocks (see k_rectify_attn):
// only where the pairs are more than one round of workgroups. Fewer run
// singly, longest first: where sequences differ in length, a CU that ends
// early takes another block (two sequences of 33001 and 23096 tokens, 448
// blocks of a 2033-row chunk: 1602 us singly, 1752 in pairs).
__host__ __device__ constexpr bool rectify_paired(int groups, int nq) { return (int64_t)groups * nq > 2 * kCus; }
// Workgroups per group and split.
__host__ __device__ constexpr int rectify_items(int groups, int nq) {
  return rectify_paired(groups, nq) ? (nq + 1) / 2 : nq;
}
constexpr int kRowBytes = kHeadDim * 2;           // one K or V row (16-bit values)
constexpr int kMaxRectSplits = 1024;              // splits per group (bounded by the host)
// The softmax reference m of a row is the maximum of its first tile; it moves
// (to the largest logit so far) only on a tile whose weights sum to more than
// this over a lane's keys. So no weight that is used exceeds 2^12, well
// inside fp16 and fp32 range, the accumulator rescale is rare, and no tile
// needs its row maximum beforehand; the normalisation by the sum uses the
// same reference.
constexpr float kMaxWeightSum = 4096.f;
// Every a.ref_keys keys the reference is taken again from the tile at hand,
// also downwards (by at most this many bits, so that sums stay in range: a
// split holds at most eight such ranges). The largest weight of that tile is
// then exactly 1, and it is among the heaviest of its range: the error against
// 64 bits falls with the number of references (32K, 7 heads a group: 2.07e-4
// with one over all keys, 2.05e-4 with 16, 1.99e-4 with 32).
constexpr float kRefDown = 8.f;

// V values above the fp16 range: band b > 0 holds magnitudes from
// 2^(16 + 30 (b - 1)) up to 2^(16 + 30 b) (b = 4: and infinities and NaN),
// which times 2^-30b are fp16 values of the normal range (2^-14 .. 2^16, the 8
// significant bits of a bf16 value fit); band 0 all below 2^16. The
// accumulators then carry 2^-40, so that sums of weights up to 2^32 times the
// largest float stay in range (what is lost lies below 2^-109 of a weight).
constexpr int kBandExp = 30, kLargeExp = -40;
__device__ __forceinline__ int band_of(uint32_t w) {  // of the bf16 value in the upper half of w
  const int e = (int)((w >> 23) & 0xff);
  return e < 143 ? 0 : min((e - 143) / kBandExp + 1, 4);
}
__device__ __forceinline__ constexpr float exp2_of(int e) { return __builtin_bit_cast(float, (uint32_t)(127 + e) << 23); }

// Tile rows are stored unpadded (256 B); 16-byte piece p of row r sits in
// slot p ^ swz(r). swz is a bijection on r % 16, so the K operand reads (16
// rows, one piece) hit 16 distinct slots; four neighbouring rows differ in
// its upper two bits, so the V transpose reads (4 aligned rows, four
// neighbouring pieces) hit 16 distinct slots too: no LDS bank conflicts
// (SQ_LDS_BANK_CONFLICT 0).
__host__ __device__ constexpr int swz(int r) { return ((r & 3) << 2) | ((r >> 2) & 3); }

// s_waitcnt immediates (vmcnt in bits 3:0 and 15:14, expcnt 6:4, lgkmcnt 11:8).
constexpr int wait_vm(int n) { return (n & 15) | ((n >> 4) << 14) | 0x0F70; }
constexpr int kWaitLgkm0 = 0xC07F;
// Buffer resource over `bytes` bytes at p (stride 0, 32-bit format), for
// values the caller knows are uniform across the wave: read from the first
// lane, so the resource sits in scalar registers. Offsets at or past
// `bytes` read as zero.
__device__ __forceinline__ i32x4_t rsrc_words(const void* p, int bytes) {
  const uint64_t u = reinterpret_cast<uint64_t>(p);
  return i32x4_t{(int32_t)__builtin_amdgcn_readfirstlane((uint32_t)u),
                 (int32_t)(__builtin_amdgcn_readfirstlane((uint32_t)(u >> 32)) & 0xffffu),
                 __builtin_amdgcn_readfirstlane(bytes), kBufWord3};
}
__device__ __forceinline__ __amdgpu_buffer_rsrc_t uniform_rsrc(const void* p, int bytes) {
  const uint64_t u = reinterpret_cast<uint64_t>(p);
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)u);
  const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(u >> 32));
  void* q = reinterpret_cast<void*>(((uint64_t)hi << 32) | lo);
  return __builtin_amdgcn_make_buffer_rsrc(q, (short)0, __builtin_amdgcn_readfirstlane(bytes), kBufWord3);
}
// LDS byte address of an LDS object.
__device__ __forceinline__ uint32_t lds_addr(const void* p) {
  return (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) void*)p;
}
// A wave's eight K rows of a tile straight into LDS (rows +0 .. 3 and
// +4 .. 7, two 1 KB buffer loads, no registers): lane i's 16 bytes at offset
// voff0 (voff1) land at LDS byte address lds + 16 i (lds + 1024 + 16 i); M0
// carries the LDS address. Written as assembly so that the compiler does not
// track them: it would otherwise make LDS reads wait for all of them. Their
// completion is ordered by hand (vmcnt waits, then a barrier). M0 is saved
// and restored, so whatever the compiler keeps in it survives; one wait state
// follows each write of M0 that a load reads.
template <bool kNt>
__device__ __forceinline__ void lds_load_rows8(uint32_t lds, uint32_t voff0, uint32_t voff1, i32x4_t rk) {
  uint32_t saved;
  if constexpr (kNt)
    __asm__ volatile(
        "s_mov_b32 %0, m0\n\t"
        "s_mov_b32 m0, %1\n\ts_nop 0\n\tbuffer_load_dwordx4 %2, %4, 0 offen nt lds\n\t"
        "s_add_i32 m0, %1, 1024\n\ts_nop 0\n\tbuffer_load_dwordx4 %3, %4, 0 offen nt lds\n\t"
        "s_mov_b32 m0, %0"
        : "=&s"(saved) : "s"(lds), "v"(voff0), "v"(voff1), "s"(rk) : "memory", "scc");
  else
    __asm__ volatile(
        "s_mov_b32 %0, m0\n\t"
        "s_mov_b32 m0, %1\n\ts_nop 0\n\tbuffer_load_dwordx4 %2, %4, 0 offen lds\n\t"
        "s_add_i32 m0, %1, 1024\n\ts_nop 0\n\tbuffer_load_dwordx4 %3, %4, 0 offen lds\n\t"
        "s_mov_b32 m0, %0"
        : "=&s"(saved) : "s"(lds), "v"(voff0), "v"(voff1), "s"(rk) : "memory", "scc");
}
// Keeps the compiler from moving memory accesses across this point; the
// hardware ordering comes from the explicit waits and barriers around it.
__device__ __forceinline__ void compiler_fence() { __asm__ volatile("" ::: "memory"); }
// Workgroup barrier without a wait for outstanding global loads.
__device__ __forceinline__ void bare_barrier() {
  compiler_fence();
  __builtin_amdgcn_s_barrier();
  compiler_fence();
}

__device__ __forceinline__ f32x16_t mfma32(bf16x8_t a, bf16x8_t b, f32x16_t c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ f32x16_t mfma32(f16x8_t a, f16x8_t b, f32x16_t c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b, c, 0, 0, 0);
}

// Writes the re-encoded rows k_f, v_f over cache rows [L - f, L) and, with
// `refresh`, re-summarises the blocks they touch (Eq. 3), one wave per block:
// lane (r, c) with r = lane / 16 and c = lane % 16 takes dims [8c, 8c + 8) of
// rows r, r + 4, ... of the block, from k_f where the row is rewritten and
// from the cache below the window. One launch in place of a copy and a
// summary pass over the same rows (64K, f = 32: 4.0 + 3.8 us of kernel time
// and a launch gap; 8K prompts, which it reads once instead of twice: 82 + 37
// us). Grid (ceil(blocks / 4), batch * kv_heads), blocks <= ceil(f / b) + 1.
template <int BS>
__global__ __launch_bounds__(256) void k_rectify_rows(RectifyArgs a) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int grp = blockIdx.y, bb = grp / a.c.kv_heads, hk = grp % a.c.kv_heads;
  if (a.seq_mask != nullptr && a.seq_mask[bb] == 0) return;
  const int L = a.seq_lens[bb];
  if (L < a.f) return;
  const int m = (L - a.f) / BS + blockIdx.x * 4 + wave;
  if (m >= min((L + BS - 1) / BS, a.c.max_blocks)) return;
  // A length past the capacity rewrites no row.
  const int first = L <= a.c.capacity ? L - a.f : L;
  const int64_t row0 = kv_row(a.c, bb, hk, m * BS);  // a block never straddles pages
  if (row0 < 0) return;
  const int r = lane >> 4, col = (lane & 15) * 8;
  uint16_t* kb = const_cast<uint16_t*>(a.c.k) + (size_t)row0 * kHeadDim + col;
  uint16_t* vb = const_cast<uint16_t*>(a.c.v) + (size_t)row0 * kHeadDim + col;
  const uint16_t* kf = a.k_f + (size_t)grp * a.f * kHeadDim + col;
  const uint16_t* vf = a.v_f + (size_t)grp * a.f * kHeadDim + col;
  // Every row is requested before the first is stored: the stores might alias
  // the later loads, so the compiler would not move them ahead (a round trip
  // per four rows otherwise; 64 groups, f = 32: 0.4 us a call). And without a
  // branch around any: a row outside the window takes its K from the cache
  // (the block lies in it whole) and an edge row's V, which is not used (blocks
  // of 64 tokens, 4K batch 1, f = 16: 26.7 -> 24.0 us a call).
  U4 rows[BS / 4], vrows[BS / 4];
#pragma unroll
  for (int i = 0; i < BS / 4; ++i) {
    const int t = m * BS + r + 4 * i;
    rows[i] = ld16(t >= first && t < L ? kf + (size_t)(t - first) * kHeadDim : kb + (size_t)(r + 4 * i) * kHeadDim);
    vrows[i] = ld16(vf + (size_t)min(max(t - first, 0), a.f - 1) * kHeadDim);
  }
#pragma unroll
  for (int i = 0; i < BS / 4; ++i) {
    const int t = m * BS + r + 4 * i;
    if (t < L && t >= first) {
      st16(kb + (size_t)(r + 4 * i) * kHeadDim, rows[i]);
      st16(vb + (size_t)(r + 4 * i) * kHeadDim, vrows[i]);
    }
  }
  if (a.refresh) {
    float mn[8], mx[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      mn[j] = __builtin_inff();
      mx[j] = -__builtin_inff();
    }
#pragma unroll
    for (int i = 0; i < BS / 4; ++i)
      if (m * BS + r + 4 * i < L) fold_minmax(rows[i], mn, mx);
    store_summary(a.c, (size_t)grp, m, r, col, mn, mx);
  }
}

// kNt: K and V are read once in the launch (one query block per group), so
// their loads are non-temporal (64K rectification 425 -> 414 us, 7B-class 32K
// 95.1 -> 92.4 us); with several query blocks a group's K and V are read
// again from L2, and non-temporal loads cost (8K prompts 4201 -> 4311 us).
//
// kStaged (full windows of 4 waves in several splits): the partial rows go out
// through LDS, instead of a lane pair's 32 bytes of each row at a time. 64
// groups of 128 rows over 1500 / 4096 tokens: 40.8 -> 38.5, 53.9 -> 51.9 us.
// Not with fewer rows (64 rows: 38.4 -> 39.0 us), nor with 8 waves, whose
// registers spill with it (7B-class 32K, f = 32: 91.9 -> 99.7 us).
template <int kWaves, bool kPaged, bool kNt, bool kStaged>
__global__ __launch_bounds__(64 * kWaves) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_rectify_attn(RectifyArgs a) {
  constexpr int kLoadRows = 8;                   // tile rows whose K and V each wave brings in
  constexpr int kKT = kLoadRows * kWaves;        // keys per tile
  constexpr int kKT32 = kKT / 32;
  constexpr int kRowsPerWg = kRowsPerWave * kWaves;
  constexpr int kTileBytes = kKT * kRowBytes;
  constexpr int kPolicy = kNt ? kPolicyNt : 0;
  constexpr bool kRenew = kWaves == 8;           // 4 waves: one reference a split (see rectify_ref_keys)
  // Tile t sits in K and V stage t % 4. All of the workgroup's LDS is one
  // object: with several, the compiler tags each access with the object it
  // touches and makes reads wait for loads into the others.
  struct Lds {
    uint8_t k[4][kTileBytes];
    uint8_t v[4][kTileBytes];   // fp16
    int large;                  // a V value above the fp16 range was met
    uint32_t bands[2];          // bands of V in the tile at hand (tiles in turn)
  };
  __shared__ __attribute__((aligned(1024))) Lds lds;
  // The wave index is uniform per wave (readfirstlane tells the compiler), so
  // the load addressing below stays in scalar registers.
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // Item i of a group and split is query block nq - 1 - i, and with `paired`
  // also block i after it: under the causal cut every pair of a prompt costs
  // the same, so the in-order dispatch leaves no CU waiting (CUs busy 76 ->
  // 97 % of the launch on 8K prompts). Workgroups go to the 8 XCDs in turn;
  // where every sequence has 8 (16, ...) kv heads,
  // each XCD works through whole groups, whose K and V its L2 then serves (8K
  // prompts 4540 -> 4476 us), and gets its share of every sequence. With
  // other head counts an XCD would get a share of the sequences instead: the
  // shorter ones would leave it idle (the chunk above: 1783 against 1752 us).
  const int nq = a.num_qblocks, S = a.num_splits;
  const bool paired = rectify_paired(a.c.batch * a.c.kv_heads, nq);
  const int np = rectify_items(a.c.batch * a.c.kv_heads, nq);
  int grp, rest;
  if (a.c.kv_heads % 8 == 0) {
    const int j = blockIdx.x >> 3;
    rest = j % (np * S);
    grp = 8 * (j / (np * S)) + (blockIdx.x & 7);
  } else {
    rest = blockIdx.x % (np * S);
    grp = blockIdx.x / (np * S);
  }
  const int split = rest % S, item = rest / S;
  const int bb = grp / a.c.kv_heads, hk = grp % a.c.kv_heads;
  // A sequence left out of this call: nothing is read or written (uniform
  // across the workgroup, before any barrier).
  if (a.seq_mask != nullptr && a.seq_mask[bb] == 0) return;
  const int G = a.group, f = a.f, R = G * f;
  const int L = a.seq_lens[bb];
  const bool seq_ok = L >= f && L <= a.c.capacity;
  const int k0 = split * a.chunk;
  const float ninf = -__builtin_inff();
  // Softmax scale: a negative one negates the queries, zero clears them (the
  // mask and the row maximum are taken of scores before a positive factor).
  const float c = a.scale_log2 == 0.f ? 1.f : fabsf(a.scale_log2);
  const uint32_t q_and = a.scale_log2 == 0.f ? 0u : ~0u, q_xor = a.scale_log2 < 0.f ? 0x80008000u : 0u;
  const int hi = lane >> 5, lq = lane & 31;

  // Wave w brings in tile rows 8 w .. + 8: lane i fills slot i % 16 of rows
  // 8 w + i / 16 and + 4, fetching the row's piece (i % 16) ^ swz(row).
  const int wrow = kLoadRows * wave;
  const int lrow = lane >> 4, lslot = lane & 15;
  auto piece_of = [&](int e) __attribute__((always_inline)) { return lslot ^ swz(wrow + 4 * e + lrow); };
  const uint32_t off0 = lrow * kRowBytes + 16 * piece_of(0), off1 = (4 + lrow) * kRowBytes + 16 * piece_of(1);

  // LDS read addresses of this lane; stage, 32-key part and k-step are
  // immediate offsets. K (A of S^T): row lq, piece 2 ks + hi. V^T (A of O^T,
  // transpose reads): each 16-lane group passes the addresses of four keys x
  // 16 dims (lane c: key c / 4, dims 4 (c % 4) ..) and lane i receives dim i
  // of the four keys; keys 4 hi .. and 8 + 4 hi .. of a 16-key step, dims 32 dt
  // + 16 (lane / 16 % 2) ...
  const uint32_t lds0 = lds_addr(&lds);
  const uint32_t lds_k = __builtin_amdgcn_readfirstlane(lds0) + (uint32_t)(wrow * kRowBytes);
  uint32_t kaddr[8], vaddr[4][2];
#pragma unroll
  for (int ks = 0; ks < 8; ++ks) kaddr[ks] = lds0 + lq * kRowBytes + 16 * ((2 * ks + hi) ^ swz(lq));
  {
    const int vr = 4 * hi + ((lane & 15) >> 2);
    const int vpiece = 2 * ((lane >> 4) & 1) + ((lane & 3) >> 1);
#pragma unroll
    for (int dt = 0; dt < 4; ++dt)
#pragma unroll
      for (int e = 0; e < 2; ++e)
        vaddr[dt][e] = lds0 + (uint32_t)offsetof(Lds, v) + (vr + 8 * e) * kRowBytes +
                       16 * ((4 * dt + vpiece) ^ swz(vr + 8 * e)) + 8 * (lane & 1);
  }
  typedef __attribute__((address_space(3))) const bf16x8_t lds_bf16x8;
  typedef __attribute__((address_space(3))) i16x4_t lds_i16x4;
  auto read_k = [&](auto stage, int ks, bf16x8_t (&ka)[kKT32]) __attribute__((always_inline)) {
    constexpr int st = decltype(stage)::value;
#pragma unroll
    for (int kt = 0; kt < kKT32; ++kt)
      ka[kt] = *(lds_bf16x8*)(uintptr_t)(kaddr[ks] + st * kTileBytes + kt * 32 * kRowBytes);
  };
  auto read_v32 = [&](int st, int ks, int dt) __attribute__((always_inline)) -> f16x8_t {
    f16x4_t x[2];
#pragma unroll
    for (int e = 0; e < 2; ++e)
      x[e] = __builtin_bit_cast(f16x4_t, __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                 (lds_i16x4*)(uintptr_t)(vaddr[dt][e] + st * kTileBytes + 16 * ks * kRowBytes)));
    return __builtin_shufflevector(x[0], x[1], 0, 1, 2, 3, 4, 5, 6, 7);
  };
  auto read_v = [&](auto stage, int ks, f16x8_t (&va)[4]) __attribute__((always_inline)) {
#pragma unroll
    for (int dt = 0; dt < 4; ++dt) va[dt] = read_v32(decltype(stage)::value, ks, dt);
  };

  for (int half = 0; half < 2; ++half) {
    const int qblk = half == 0 ? nq - 1 - item : item;
    if (half == 1 && (!paired || qblk == nq - 1 - item)) break;
    // Keys past the last causal limit of these rows are never needed (row rho
    // sits at L - f + rho / G).
    const int last_row = min(R - 1, (qblk + 1) * kRowsPerWg - 1);
    const int k1 = seq_ok ? min(min(k0 + a.chunk, L), L - f + last_row / G + 1) : k0;
    const int ntiles = k1 > k0 ? (k1 - k0 + kKT - 1) / kKT : 0;
    const int row_base = qblk * kRowsPerWg + wave * kRowsPerWave;
    // Keys at or past `cut` need the mask: the causal cut of the wave's first
    // row (the smallest limit) or the end of the range.
    const int cut = min(k1, L - f + row_base / G);
    const int rho = row_base + lq;

    // Q^T operand (B of S^T): lane holds query row lq, dims 16 s + 8 hi .. + 8
    // for k-step s; keys past lim are masked.
    bf16x8_t qb[8];
    int lim = -1;
    if (rho < R && seq_ok) {
      const int h = rho % G, r = rho / G;
      lim = min(L - f + r, k1 - 1);
      const uint16_t* qp = a.q_f + (((size_t)bb * a.q_heads + (size_t)hk * G + h) * f + r) * kHeadDim;
#pragma unroll
      for (int s = 0; s < 8; ++s) {
        const U4 x = ld16(qp + 16 * s + 8 * hi);
        qb[s] = __builtin_bit_cast(bf16x8_t, U4{(x.x & q_and) ^ q_xor, (x.y & q_and) ^ q_xor,
                                               (x.z & q_and) ^ q_xor, (x.w & q_and) ^ q_xor});
      }
    } else {
#pragma unroll
      for (int s = 0; s < 8; ++s) qb[s] = __builtin_bit_cast(bf16x8_t, U4{0, 0, 0, 0});
    }

    // Page of this wave's rows of tile ti (its rows lie in one block); tiles
    // past the table ask for its last entry, and read nothing. Requested as a
    // vector load, in front of a tile's V loads and waited for with them: a
    // scalar load in flight would make every LDS read wait for it.
    const __amdgpu_buffer_rsrc_t rt =
        uniform_rsrc(kPaged ? a.c.table + (size_t)bb * a.c.max_blocks : nullptr, kPaged ? a.c.max_blocks * 4 : 0);
    auto ask_page = [&](int ti) __attribute__((always_inline)) -> int {
      if constexpr (kPaged) {
        const int mb = min((k0 + ti * kKT + wrow) >> a.c.log2_block, a.c.max_blocks - 1);
        return (int)__builtin_amdgcn_raw_buffer_load_b32(rt, mb * 4, 0, 0);
      } else {
        return 0;
      }
    };
    auto page_of = [&](int asked) __attribute__((always_inline)) -> int {
      return kPaged ? __builtin_amdgcn_readfirstlane(asked) : 0;
    };
    // First row and byte count of this wave's rows of tile ti: rows at or past
    // k1 and rows of a page outside the pool fall outside and read as zero.
    auto tile_src = [&](int ti, int page, size_t& row) __attribute__((always_inline)) -> int {
      const int key = k0 + ti * kKT + wrow;
      int nrec = min(max(k1 - key, 0), kLoadRows) * kRowBytes;
      if constexpr (kPaged) {
        if ((unsigned)page >= (unsigned)a.c.num_pages) nrec = 0;
        row = ((size_t)page * a.c.kv_heads + hk) * a.c.block_size + (key & (a.c.block_size - 1));
      } else {
        row = ((size_t)bb * a.c.kv_heads + hk) * a.c.capacity + key;
      }
      return nrec;
    };
    auto issue_k = [&](int ti, int stage, int page) __attribute__((always_inline)) {
      size_t row;
      const int nrec = tile_src(ti, page, row);
      lds_load_rows8<kNt>(lds_k + (uint32_t)(stage * kTileBytes), off0, off1, rsrc_words(a.c.k + row * kHeadDim, nrec));
    };
    int p3 = 0, p4 = 0;  // pages asked for, of tiles ti + 3 and ti + 4
    U4 vv[2];
    auto load_v = [&](int ti, int page) __attribute__((always_inline)) {
      size_t row;
      const int nrec = tile_src(ti, page, row);
      const __amdgpu_buffer_rsrc_t rv = uniform_rsrc(a.c.v + row * kHeadDim, nrec);
      vv[0] = __builtin_bit_cast(U4, __builtin_amdgcn_raw_buffer_load_b128(rv, off0, 0, kPolicy));
      vv[1] = __builtin_bit_cast(U4, __builtin_amdgcn_raw_buffer_load_b128(rv, off1, 0, kPolicy));
    };
    // Piece e of vv to V stage st in fp16; vmax collects the largest magnitude.
    auto put_v = [&](int st, int e, float& vmax) __attribute__((always_inline)) {
      const uint32_t w[4] = {vv[e].x, vv[e].y, vv[e].z, vv[e].w};
      uint32_t h[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float x0 = bf_lo(w[i]), x1 = bf_hi(w[i]);
        vmax = fmaxf(vmax, fmaxf(fabsf(x0), fabsf(x1)));
        h[i] = __builtin_bit_cast(uint32_t, f16x2_t{(_Float16)x0, (_Float16)x1});
      }
      st16(lds.v[st] + (wrow + 4 * e) * kRowBytes + 16 * lane, U4{h[0], h[1], h[2], h[3]});
    };

    f32x16_t o[4];
#pragma unroll
    for (int dt = 0; dt < 4; ++dt)
#pragma unroll
      for (int i = 0; i < 16; ++i) o[dt][i] = 0.f;
    float m = ninf, l = 0.f;  // l: over this lane's keys; summed across the two halves at the end
    if (tid == 0) {
      lds.large = 0;
      lds.bands[0] = lds.bands[1] = 0u;
    }
    lds_sync();

    auto mask = [&](int t0, f32x16_t (&s)[kKT32]) __attribute__((always_inline)) {
      const int d = lim - t0 - 4 * hi;
#pragma unroll
      for (int kt = 0; kt < kKT32; ++kt)
#pragma unroll
        for (int i = 0; i < 16; ++i) s[kt][i] = 32 * kt + 8 * (i >> 2) + (i & 3) > d ? ninf : s[kt][i];
    };
    auto row_max = [&](const f32x16_t (&s)[kKT32]) __attribute__((always_inline)) {
      float x = ninf;
#pragma unroll
      for (int kt = 0; kt < kKT32; ++kt)
#pragma unroll
        for (int i = 0; i < 16; ++i) x = fmaxf(x, s[kt][i] * c);
      return max_xor32(x);
    };
    // Weight i of the tile: raw score times c is its log2-domain logit.
    auto weight = [&](const f32x16_t (&s)[kKT32], int i, float mref, f16x8_t (&ph)[2 * kKT32], float (&ps)[4]) __attribute__((always_inline)) {
      const float pe = fast_exp2(fmaf(s[i >> 4][i & 15], c, -mref));
      ps[i & 3] += pe;
      ph[i >> 3][i & 7] = (_Float16)pe;
    };
    // Weights of one tile (scores s) interleaved with the scores of the
    // next (K stage `stage`, into sn): per step two MFMAs, the next step's
    // operand reads and four weights; the scheduling barriers keep the
    // order. Returns the sum of the weights over this lane's keys.
    auto weights_scores = [&](auto stage, const f32x16_t (&s)[kKT32], f32x16_t (&sn)[kKT32], f16x8_t (&ph)[2 * kKT32]) __attribute__((always_inline)) {
      float ps[4] = {0.f, 0.f, 0.f, 0.f};
      bf16x8_t ka[2][kKT32];
      read_k(stage, 0, ka[0]);
#pragma unroll
      for (int kt = 0; kt < kKT32; ++kt)
#pragma unroll
        for (int i = 0; i < 16; ++i) sn[kt][i] = 0.f;
      __builtin_amdgcn_sched_barrier(0);
      // The SIMD's other wave, at another point of its round, fills the gaps
      // instead of delaying the MFMAs (8K prompts 4361 -> 4284 us).
      __builtin_amdgcn_s_setprio(1);
#pragma unroll
      for (int ks = 0; ks < 8; ++ks) {
        if (ks < 7) read_k(stage, ks + 1, ka[(ks + 1) & 1]);
#pragma unroll
        for (int kt = 0; kt < kKT32; ++kt) sn[kt] = mfma32(ka[ks & 1][kt], qb[ks], sn[kt]);
#pragma unroll
        for (int i = 2 * kKT32 * ks; i < 2 * kKT32 * (ks + 1); ++i) weight(s, i, m, ph, ps);
        __builtin_amdgcn_sched_barrier(0);
      }
      __builtin_amdgcn_s_setprio(0);
      return (ps[0] + ps[1]) + (ps[2] + ps[3]);
    };
    // One tile: its weights (scores s) with the next tile's scores (sn),
    // then its P.V, with the conversion of the V of the tile after next.
    //
    // Order between the waves, with a barrier before every even tile 2p
    // only. Rounds 2p and 2p + 1 read K(2p + 1), K(2p + 2), V(2p) and
    // V(2p + 1); they write V(2p + 2) and V(2p + 3), into the stages last
    // read in rounds 2p - 2 and 2p - 1, and at the end of round 2p request
    // K(2p + 3) and K(2p + 4), into the stages last read in the same two
    // rounds. All these were before the barrier, and what is written is
    // read after the next one, at which every wave has waited for its own
    // loads and stores: vmcnt counts in order, and only the two loads of
    // V(2p + 2), issued after the K loads that are needed, may be pending.
    // Tiles past the end are requested and converted too (empty
    // resources: zeros), so the counts never change.
    auto round = [&](int ti, auto stage, f32x16_t (&s)[kKT32], f32x16_t (&sn)[kKT32]) __attribute__((always_inline)) {
      constexpr int st = decltype(stage)::value;
      const int t0 = k0 + ti * kKT;
      if constexpr (st % 2 == 0) {
        __builtin_amdgcn_s_waitcnt(wait_vm(kPaged ? 3 : 2));
        __builtin_amdgcn_s_waitcnt(kWaitLgkm0);
        bare_barrier();
      }
      f16x8_t ph[2 * kKT32];
      __builtin_amdgcn_sched_barrier(0);
      float ps = weights_scores(std::integral_constant<int, (st + 1) & 3>{}, s, sn, ph);
      // Rare: move the reference and form the weights again. A row without
      // one so far (no tile with a finite score) has weights of inf or NaN
      // and takes this branch too, on every tile until one has.
      if (__builtin_expect(__any(!(ps <= kMaxWeightSum)), 0)) {
        const float mn = fmaxf(m, row_max(s));
        const float alpha = m == mn ? 1.f : fast_exp2(m - mn);
        m = mn;
        l *= alpha;
#pragma unroll
        for (int dt = 0; dt < 4; ++dt) o[dt] *= alpha;
        const float mref = m == ninf ? 0.f : m;
        float pt[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int i = 0; i < 16 * kKT32; ++i) weight(s, i, mref, ph, pt);
        ps = (pt[0] + pt[1]) + (pt[2] + pt[3]);
      }
      l += ps;
      if (__builtin_expect(t0 + 2 * kKT > cut, 0)) mask(t0 + kKT, sn);
      __builtin_amdgcn_sched_barrier(0);
      f16x8_t va[2][4];
      read_v(stage, 0, va[0]);
      __builtin_amdgcn_sched_barrier(0);
      constexpr int nv = (st + 2) & 3;
      float vmax = 0.f;
#pragma unroll
      for (int ks = 0; ks < 2 * kKT32; ++ks) {
        if (ks < 2 * kKT32 - 1) read_v(stage, ks + 1, va[(ks + 1) & 1]);
#pragma unroll
        for (int dt = 0; dt < 4; ++dt) o[dt] = mfma32(va[ks & 1][dt], ph[ks], o[dt]);
        if (ks >= 2 * kKT32 - 2) put_v(nv, ks - (2 * kKT32 - 2), vmax);
        __builtin_amdgcn_sched_barrier(0);
      }
      if (__builtin_expect(__any(!(vmax <= 65504.f)), 0)) lds.large = 1;
      // Here the pages of tiles ti + 3 and ti + 4 have arrived (with the V
      // pieces converted above, or earlier).
      const int g3 = page_of(p3), g4 = page_of(p4);
      if constexpr (st % 2 == 0) {
        issue_k(ti + 3, (st + 3) & 3, g3);
        issue_k(ti + 4, st, g4);
      }
      p3 = p4;
      p4 = ask_page(ti + 5);
      load_v(ti + 3, g3);
      __builtin_amdgcn_sched_barrier(0);
    };

    if (ntiles > 0) {
      f32x16_t sa[kKT32], sb[kKT32];
      // Pipeline start: everything is requested before anything is used.
      const int asked[3] = {ask_page(0), ask_page(1), ask_page(2)};
      p3 = ask_page(3);
      p4 = ask_page(4);
      const int pg[3] = {page_of(asked[0]), page_of(asked[1]), page_of(asked[2])};
      load_v(0, pg[0]);
      const U4 v0[2] = {vv[0], vv[1]};
      load_v(1, pg[1]);
      const U4 v1[2] = {vv[0], vv[1]};
#pragma unroll
      for (int t = 0; t < 3; ++t) issue_k(t, t, pg[t]);
      float vmax = 0.f;
#pragma unroll
      for (int e = 0; e < 2; ++e) vv[e] = v0[e];
      put_v(0, 0, vmax);
      put_v(0, 1, vmax);
#pragma unroll
      for (int e = 0; e < 2; ++e) vv[e] = v1[e];
      put_v(1, 0, vmax);
      put_v(1, 1, vmax);
      if (!(vmax <= 65504.f)) lds.large = 1;
      load_v(2, pg[2]);
      __builtin_amdgcn_s_waitcnt(wait_vm(2));
      __builtin_amdgcn_s_waitcnt(kWaitLgkm0);
      bare_barrier();
      {
        bf16x8_t ka[kKT32];
#pragma unroll
        for (int kt = 0; kt < kKT32; ++kt)
#pragma unroll
          for (int i = 0; i < 16; ++i) sa[kt][i] = 0.f;
#pragma unroll
        for (int ks = 0; ks < 8; ++ks) {
          read_k(std::integral_constant<int, 0>{}, ks, ka);
#pragma unroll
          for (int kt = 0; kt < kKT32; ++kt) sa[kt] = mfma32(ka[kt], qb[ks], sa[kt]);
        }
      }
      if (k0 + kKT > cut) mask(k0, sa);
      m = row_max(sa);
      // The reference taken again, before the weights of tile `renew` are
      // formed (between two rounds: within one it costs 6 % of a prefill).
      int renew = (a.ref_keys - k0 % a.ref_keys) / kKT;
      auto take_reference = [&](const f32x16_t (&s)[kKT32]) __attribute__((always_inline)) {
        renew += a.ref_keys / kKT;
        const float x = row_max(s);
        const float mn = x == ninf ? m : fmaxf(x, m - kRefDown);
        const float alpha = m == mn ? 1.f : fast_exp2(m - mn);
        m = mn;
        l *= alpha;
#pragma unroll
        for (int dt = 0; dt < 4; ++dt) o[dt] *= alpha;
      };
      for (int ti = 0; ti < ntiles; ti += 4) {
        if (kRenew && __builtin_expect(ti == renew, 0)) take_reference(sa);
        round(ti, std::integral_constant<int, 0>{}, sa, sb);
        if (ti + 1 >= ntiles) break;
        if (kRenew && __builtin_expect(ti + 1 == renew, 0)) take_reference(sb);
        round(ti + 1, std::integral_constant<int, 1>{}, sb, sa);
        if (ti + 2 >= ntiles) break;
        if (kRenew && __builtin_expect(ti + 2 == renew, 0)) take_reference(sa);
        round(ti + 2, std::integral_constant<int, 2>{}, sa, sb);
        if (ti + 3 >= ntiles) break;
        if (kRenew && __builtin_expect(ti + 3 == renew, 0)) take_reference(sb);
        round(ti + 3, std::integral_constant<int, 3>{}, sb, sa);
      }
      // No load may still be writing LDS when the stages are used again.
      __builtin_amdgcn_s_waitcnt(wait_vm(0));
      compiler_fence();
    }
    lds_sync();

    // If the pass met a V value above the fp16 range, its result is thrown
    // away and the range taken again, a tile at a time, with V split by
    // magnitude into bands (see kBandExp): a band's P.V is added in fp32 to
    // the accumulators, which then carry 2^kLargeExp. So every row keeps
    // the precision of the values it sees, whatever the others see.
    const bool banded = lds.large != 0;
    if (__builtin_expect(banded, 0)) {
#pragma unroll
      for (int dt = 0; dt < 4; ++dt)
#pragma unroll
        for (int i = 0; i < 16; ++i) o[dt][i] = 0.f;
      m = ninf;
      l = 0.f;
#pragma unroll 1
      for (int ti = 0; ti < ntiles; ++ti) {
        const int page = page_of(ask_page(ti));
        issue_k(ti, 0, page);
        load_v(ti, page);
        uint32_t has = 0;
#pragma unroll
        for (int e = 0; e < 2; ++e) {
          const uint32_t w[4] = {vv[e].x, vv[e].y, vv[e].z, vv[e].w};
#pragma unroll
          for (int i = 0; i < 4; ++i) has |= 1u << band_of(w[i] << 16) | 1u << band_of(w[i]);
        }
        if ((has & ~1u) != 0) atomicOr(&lds.bands[ti & 1], has);
        if (tid == 0) lds.bands[(ti + 1) & 1] = 0u;
        __builtin_amdgcn_s_waitcnt(wait_vm(0));
        lds_sync();
        const uint32_t bands = __builtin_amdgcn_readfirstlane(lds.bands[ti & 1]) | 1u;
        f32x16_t s[kKT32];
#pragma unroll
        for (int kt = 0; kt < kKT32; ++kt)
#pragma unroll
          for (int i = 0; i < 16; ++i) s[kt][i] = 0.f;
#pragma unroll
        for (int ks = 0; ks < 8; ++ks) {
          bf16x8_t ka[kKT32];
          read_k(std::integral_constant<int, 0>{}, ks, ka);
#pragma unroll
          for (int kt = 0; kt < kKT32; ++kt) s[kt] = mfma32(ka[kt], qb[ks], s[kt]);
        }
        if (k0 + (ti + 1) * kKT > cut) mask(k0 + ti * kKT, s);
        const float mn = fmaxf(m, row_max(s));
        const float alpha = m == mn ? 1.f : fast_exp2(m - mn);
        const float mref = mn == ninf ? 0.f : mn;
        m = mn;
        f16x8_t ph[2 * kKT32];
        float ps[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int i = 0; i < 16 * kKT32; ++i) weight(s, i, mref, ph, ps);
        l = fmaf(l, alpha, (ps[0] + ps[1]) + (ps[2] + ps[3]));
#pragma unroll
        for (int dt = 0; dt < 4; ++dt) o[dt] *= alpha;
#pragma unroll 1
        for (int band = 0; band <= 4; ++band) {
          if (((bands >> band) & 1u) == 0) continue;
          const float down = exp2_of(-kBandExp * band), back = exp2_of(kBandExp * band + kLargeExp);
#pragma unroll
          for (int e = 0; e < 2; ++e) {
            const uint32_t w[4] = {vv[e].x, vv[e].y, vv[e].z, vv[e].w};
            uint32_t h[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              const float x0 = band_of(w[i] << 16) == band ? bf_lo(w[i]) * down : 0.f;
              const float x1 = band_of(w[i]) == band ? bf_hi(w[i]) * down : 0.f;
              h[i] = __builtin_bit_cast(uint32_t, f16x2_t{(_Float16)x0, (_Float16)x1});
            }
            st16(lds.v[0] + (wrow + 4 * e) * kRowBytes + 16 * lane, U4{h[0], h[1], h[2], h[3]});
          }
          lds_sync();
#pragma unroll
          for (int dt = 0; dt < 4; ++dt) {
            f32x16_t y;
#pragma unroll
            for (int i = 0; i < 16; ++i) y[i] = 0.f;
#pragma unroll
            for (int ks = 0; ks < 2 * kKT32; ++ks) y = mfma32(read_v32(0, ks, dt), ph[ks], y);
            o[dt] += y * back;
          }
          lds_sync();  // read before the next band or tile is written
        }
      }
    }

    const float lt = sum_xor32(l);
    const float inv = lt > 0.f ? (banded ? exp2_of(-kLargeExp) : 1.f) / lt : 0.f;
    auto out4 = [&](int dt, int i4) __attribute__((always_inline)) {
      return f32x4_t{o[dt][4 * i4] * inv, o[dt][4 * i4 + 1] * inv, o[dt][4 * i4 + 2] * inv, o[dt][4 * i4 + 3] * inv};
    };
    if constexpr (kStaged) {
      // The wave's 32 rows through its share of the tile stages, two whole
      // 512-byte rows to a store; 16-byte piece p of row r sits in slot p ^ r.
      static_assert(sizeof(lds.k) + sizeof(lds.v) >= kRowsPerWg * kHeadDim * 4, "a wave's share of the stages");
      uint8_t* buf = &lds.k[0][0] + wave * (kRowsPerWave * kHeadDim * 4);
#pragma unroll
      for (int dt = 0; dt < 4; ++dt)
#pragma unroll
        for (int i4 = 0; i4 < 4; ++i4)
          *reinterpret_cast<f32x4_t*>(buf + lq * (kHeadDim * 4) + 16 * ((8 * dt + 2 * i4 + hi) ^ lq)) = out4(dt, i4);
      compiler_fence();  // a wave's LDS accesses run in order
      float* po = a.part_o + (((size_t)grp * S + split) * R + row_base) * kHeadDim + 4 * lq;
#pragma unroll 4
      for (int j = 0; j < kRowsPerWave / 2; ++j) {
        const int r = 2 * j + hi;
        const f32x4_t y = *reinterpret_cast<const f32x4_t*>(buf + r * (kHeadDim * 4) + 16 * (lq ^ r));
        if (row_base + r < R) *reinterpret_cast<f32x4_t*>(po + r * kHeadDim) = y;
      }
    }
    if (rho < R) {
      const float l2 = lt > 0.f ? m + fast_log2(lt) : ninf;
      const size_t oi = ((size_t)bb * a.q_heads + (size_t)hk * G + rho % G) * f + rho / G;
      if constexpr (!kStaged) {
        float* po = S == 1 ? a.out + oi * kHeadDim
                           : a.part_o + (((size_t)grp * S + split) * R + rho) * kHeadDim;
#pragma unroll
        for (int dt = 0; dt < 4; ++dt)
#pragma unroll
          for (int i4 = 0; i4 < 4; ++i4) *reinterpret_cast<f32x4_t*>(po + 32 * dt + 8 * i4 + 4 * hi) = out4(dt, i4);
      }
      if (hi == 0) {
        if (S > 1)
          a.part_lse[((size_t)grp * S + split) * R + rho] = l2;
        else if (a.lse)
          a.lse[oi] = lt > 0.f ? l2 * kLn2 : ninf;
      }
    }
    lds_sync();
  }
}

// Log-sum-exp merge of the splits (Alg. 2, "Combine"): kPerRow waves take one
// query row, each a share of its splits (wave w splits w, w + kPerRow, ...).
// Lane i holds dims 2i, 2i + 1 of the row, so a split's partial is one
// 512-byte load of the wave; a wave takes 64 splits at a time, whose lse sit
// one per lane: their weights are formed by all lanes at once and broadcast
// one by one, with the partial loads of 16 splits in flight. One wave per row
// where the splits are few (up to 16) and rows many; four otherwise. The
// weights carry a factor of 1 / (2 kMaxRectSplits), which the normalisation
// takes out again, so sums of rows near the largest float stay in range.
template <int kPerRow>
__global__ __launch_bounds__(256) void k_rectify_combine(RectifyArgs a) {
  constexpr int kRows = 4 / kPerRow;   // query rows per workgroup
  constexpr float kScale = 0.5f / kMaxRectSplits;
  __shared__ f2_t s_acc[4][64];
  __shared__ float s_m[4], s_l[4];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int grp = blockIdx.y, bb = grp / a.c.kv_heads, hk = grp % a.c.kv_heads;
  if (a.seq_mask != nullptr && a.seq_mask[bb] == 0) return;
  const int G = a.group, f = a.f, R = G * f, S = a.num_splits;
  const int rho = blockIdx.x * kRows + wave / kPerRow, part = wave % kPerRow;
  const float ninf = -__builtin_inff();
  const bool live = rho < R;
  const float* pl = a.part_lse + (size_t)grp * S * R + rho;
  const float* po = a.part_o + ((size_t)grp * S * R + rho) * kHeadDim + 2 * lane;
  const size_t stride = (size_t)R * kHeadDim;
  float m = ninf, l = 0.f;
  f2_t acc = {0.f, 0.f};
  const int n = live ? (S - part + kPerRow - 1) / kPerRow : 0;  // this wave's splits
  for (int b = 0; b < n; b += 64) {
    const int cnt = min(64, n - b);
    const float x = lane < cnt ? pl[(size_t)((b + lane) * kPerRow + part) * R] : ninf;
    const float mn = fmaxf(m, wave_max_f(x));
    const float e = x == ninf ? 0.f : fast_exp2(x - mn) * kScale;
    const float alpha = m == ninf ? 0.f : fast_exp2(m - mn);
    l = fmaf(l, alpha, wave_sum_f(e));
    acc *= alpha;
    m = mn;
    for (int q = 0; q < cnt; q += 16) {
      f2_t p[16];
#pragma unroll
      for (int u = 0; u < 16; ++u) {
        p[u] = f2_t{0.f, 0.f};
        if (q + u < cnt) p[u] = *reinterpret_cast<const f2_t*>(po + (size_t)((b + q + u) * kPerRow + part) * stride);
      }
#pragma unroll
      for (int u = 0; u < 16; ++u)
        acc += __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, e), (q + u) & 63)) * p[u];
    }
  }
  if constexpr (kPerRow > 1) {
    s_acc[wave][lane] = acc;
    if (lane == 0) {
      s_m[wave] = m;
      s_l[wave] = l;
    }
    lds_sync();
    if (part != 0) return;
    float mx = m;
#pragma unroll
    for (int w = 1; w < kPerRow; ++w) mx = fmaxf(mx, s_m[wave + w]);
    const float f0 = m == ninf ? 0.f : fast_exp2(m - mx);
    l *= f0;
    acc *= f0;
#pragma unroll
    for (int w = 1; w < kPerRow; ++w) {
      const float mw = s_m[wave + w], fw = mw == ninf ? 0.f : fast_exp2(mw - mx);
      l = fmaf(s_l[wave + w], fw, l);
      acc += fw * s_acc[wave + w][lane];
    }
    m = mx;
  }
  if (!live) return;
  const size_t oi = ((size_t)bb * a.q_heads + (size_t)hk * G + rho % G) * f + rho / G;
  *reinterpret_cast<f2_t*>(a.out + oi * kHeadDim + 2 * lane) = acc * (l > 0.f ? 1.f / l : 0.f);
  if (lane == 0 && a.lse) a.lse[oi] = l > 0.f ? (m + fast_log2(l * (1.f / kScale))) * kLn2 : ninf;
}

}  // namespace

int32_t rectify_num_qblocks(int32_t group, int32_t f) {
  const int rows = group * f;
  const int per = waves_for_rows(rows) * kRowsPerWave;
  return (rows + per - 1) / per;
}

// Short caches still fill the chip (4K, batch 1: 32 splits of 128 keys,
// 30.4 against 34.0 us per call with a 512-key minimum).
constexpr int kMinRectChunk = 128;

static int32_t chunk_for(int64_t target, int32_t max_seq_len) {
  int64_t chunk = (max_seq_len + target - 1) / target;
  chunk = (chunk + kMaxKeyTile - 1) / kMaxKeyTile * kMaxKeyTile;
  if (chunk < kMinRectChunk) chunk = kMinRectChunk;
  // At most kMaxRectSplits splits (the targets below stay below it).
  const int64_t least = ((int64_t)max_seq_len + kMaxRectSplits - 1) / kMaxRectSplits;
  if (chunk < least) chunk = (least + kMaxKeyTile - 1) / kMaxKeyTile * kMaxKeyTile;
  return (int32_t)chunk;
}

// Keys a softmax reference serves, at most: those of a split when the query
// blocks are dealt to about 512 workgroups (which windows of up to 128 rows
// are, so one reference a split there).
int32_t rectify_ref_keys(int32_t batch, int32_t kv_heads, int32_t rows, int32_t max_seq_len) {
  const int32_t per = waves_for_rows(rows) * kRowsPerWave;
  const int64_t wgs = (int64_t)batch * kv_heads * ((rows + per - 1) / per);
  return chunk_for((512 + wgs - 1) / wgs, max_seq_len);
}

// Key splits per group at most, whatever the length: about 512 workgroups in
// all for short windows (4 waves, two workgroups per CU; 64K batch 8: 527 us
// with 256, 414 with 512, 433 with 1024), up to two rounds of workgroups for
// long ones (8 waves, one per CU), one split where a round is full anyway.
static int64_t rectify_most_splits(int32_t batch, int32_t kv_heads, int32_t rows, int64_t* wgs) {
  const int64_t groups = (int64_t)batch * kv_heads;
  const int32_t per = waves_for_rows(rows) * kRowsPerWave;
  *wgs = groups * rectify_items((int)groups, (rows + per - 1) / per);  // workgroups per split
  if (waves_for_rows(rows) == 4) return (2 * kCus + groups - 1) / groups;
  return *wgs >= kCus ? 1 : (2 * kCus + *wgs - 1) / *wgs;
}

// Time of a split count for long windows, in nanoseconds, from what single
// query blocks measured: a first round 17 us and a later one 14 beside its
// 64-key tiles, a tile 1.4 us and more as more CUs run at once, and the partial
// rows and their merge 1 us and a share per workgroup. Fitted to 503 shapes (1
// to 4 query blocks a group, 4 and 7 heads, 4 to 248 workgroups per split, 260
// to 32768 keys, 1 to 64 splits).
static int64_t rectify_cost(int64_t wgs_per_split, int32_t chunk, int32_t max_seq_len) {
  const int64_t splits = (max_seq_len + chunk - 1) / chunk, wgs = wgs_per_split * splits;
  const int64_t rounds = (wgs + kCus - 1) / kCus;
  const int64_t cost = 17000 + 14000 * (rounds - 1) +
                       rounds * (chunk / kMaxKeyTile) * (1400 + 2 * (wgs < kCus ? wgs : kCus));
  return splits == 1 ? cost : cost + 1000 + 80 * (wgs < kCus / 2 ? wgs : kCus / 2) + 20 * wgs;
}

// Long windows: as many splits as fill the 256 CUs once (7B-class 32K, f = 32,
// 16 workgroups per split: 95.1 us with 16 splits, 115.3 with 32), or the count
// that rectify_cost puts at least a twentieth lower: one split where the cache
// is short, a fuller last round where it is long. Over the fitted shapes the
// count taken is 0.8 % off the best on average and 11 % at most (one full
// round whatever the length: 5.5 and 59 %; 64 workgroups over 400 keys 38.2 us,
// 29.2 in one split; 128 over 260 45.4 and 29.0). With a sequence mask, two rounds
// (the workgroups of sequences left out end at once; 2 sequences of 92K, one
// left out, R = 512: 146 us against 197 with one round) or one split, compared
// for half of the workgroups.
int32_t rectify_chunk(int32_t batch, int32_t kv_heads, int32_t rows, int32_t max_seq_len, bool masked) {
  int64_t W;
  const int64_t most = rectify_most_splits(batch, kv_heads, rows, &W);
  if (waves_for_rows(rows) == 4 || most == 1) return chunk_for(most, max_seq_len);
  // A split holds at most eight ranges of a softmax reference (see kRefDown).
  const int64_t longest = 8 * (int64_t)rectify_ref_keys(batch, kv_heads, rows, max_seq_len);
  int32_t best = chunk_for(masked ? most : kCus / W, max_seq_len), last = 0;
  if (masked) W = (W + 1) / 2;
  int64_t least = rectify_cost(W, best, max_seq_len) * 19 / 20;
  for (int64_t s = 1; s <= (masked ? 1 : most) && last != kMinRectChunk; s += 1 + s / 32) {
    const int32_t chunk = chunk_for(s, max_seq_len);
    if (chunk > longest || chunk == last) continue;
    last = chunk;
    const int64_t cost = rectify_cost(W, chunk, max_seq_len);
    if (cost < least) {
      best = chunk;
      least = cost;
    }
  }
  return best;
}

int32_t rectify_max_splits(int32_t batch, int32_t kv_heads, int32_t rows, int32_t max_seq_len) {
  // ceil(L / chunk) with chunk >= 128 and chunk >= ceil(L / most) (most <= 512
  // < kMaxRectSplits): at most min(ceil(L / 128), most), a bound that never
  // decreases as L grows, while the split count itself can (the chunk is
  // rounded up to whole 64-key tiles: 512 splits at L = 65536, 342 at 65537
  // for one group and one query block).
  int64_t W;
  const int64_t by_len = ((int64_t)max_seq_len + kMinRectChunk - 1) / kMinRectChunk;
  const int64_t most = rectify_most_splits(batch, kv_heads, rows, &W);
  const int64_t s = by_len < most ? by_len : most;
  return (int32_t)(s < 1 ? 1 : s);
}

hipError_t launch_rectify(const RectifyArgs& a, hipStream_t stream) {
  const int nblk = (a.f + a.c.block_size - 1) / a.c.block_size + 1;  // blocks rows [L - f, L) can touch
  const dim3 rows_grid((nblk + 3) / 4, a.c.batch * a.c.kv_heads);
  switch (a.c.block_size) {
    case 16: hipLaunchKernelGGL(k_rectify_rows<16>, rows_grid, dim3(256), 0, stream, a); break;
    case 32: hipLaunchKernelGGL(k_rectify_rows<32>, rows_grid, dim3(256), 0, stream, a); break;
    case 64: hipLaunchKernelGGL(k_rectify_rows<64>, rows_grid, dim3(256), 0, stream, a); break;
    default: return hipErrorInvalidValue;
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const int groups = a.c.batch * a.c.kv_heads;
  const dim3 grid(a.num_splits * rectify_items(groups, a.num_qblocks) * groups);
  const bool paged = a.c.table != nullptr;
  auto launch = [&](auto waves, auto nt, auto staged) {
    constexpr int W = decltype(waves)::value;
    constexpr bool N = decltype(nt)::value, P = decltype(staged)::value;
    if (paged)
      hipLaunchKernelGGL((k_rectify_attn<W, true, N, P>), grid, dim3(64 * W), 0, stream, a);
    else
      hipLaunchKernelGGL((k_rectify_attn<W, false, N, P>), grid, dim3(64 * W), 0, stream, a);
  };
  const int rows = a.group * a.f;
  if (waves_for_rows(rows) == 4 && rows > 3 * kRowsPerWave && a.num_splits > 1)
    launch(std::integral_constant<int, 4>{}, std::true_type{}, std::true_type{});
  else if (waves_for_rows(rows) == 4)
    launch(std::integral_constant<int, 4>{}, std::true_type{}, std::false_type{});
  else if (a.num_qblocks == 1)
    launch(std::integral_constant<int, 8>{}, std::true_type{}, std::false_type{});
  else
    launch(std::integral_constant<int, 8>{}, std::false_type{}, std::false_type{});
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  if (a.num_splits == 1) return hipSuccess;  // the attention kernel wrote out / lse
  if (a.num_splits <= 16)
    hipLaunchKernelGGL(k_rectify_combine<1>, dim3((rows + 3) / 4, groups), dim3(256), 0, stream, a);
  else
    hipLaunchKernelGGL(k_rectify_combine<4>, dim3(rows, groups), dim3(256), 0, stream, a);
  return hipGetLastError();
}

}  // namespace resa
