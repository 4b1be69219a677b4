// Shared host/device plumbing of libkvc: workspace layout, launch checks, a
// device-wide exclusive scan, and small wavefront helpers.  gfx950 only.
#pragma once

#include <hip/hip_runtime.h>
#include <atomic>
#include <stdint.h>
#include <stddef.h>

#include "kvc.h"

namespace kvc {

constexpr int kWave = 64;
constexpr int kScanThreads = 256;
constexpr int kScanItems = 8;                       // per thread
constexpr int kScanTile = kScanThreads * kScanItems; // 2048 elements per workgroup

// ---- workspace header: one int32 per field, zeroed by kvc_workspace_reset ----
enum HeaderWord {
  HW_STATUS = 0,      // sticky error word written by device-side guards
  HW_TOTAL_REQ = 1,   // blocks requested by the call in flight
  HW_TOTAL_FREE = 2,  // free blocks counted by the call in flight
  HW_TOTAL_ITEMS = 3, // decode work items
  HW_FREED = 4,       // blocks freed by the call in flight
  HW_SCRATCH0 = 5,
  HW_SCRATCH1 = 6,
  HW_ARRIVED = 7,     // workgroups of an append's first launch that are done (its last one sets it back to zero)
  HW_SHORT_ITEMS = 8,  // decode work items short enough for the one-wavefront launch
  HW_PLAN_BASE = 11,   // a kept work list's first record
  // decode work-list block: item counts per size class, per-class cursors, cursor of the
  // per-chunk partial results.  All zero between calls (the chunk kernel clears it).
  HW_DEC_BINS = 12,    // [16]
  HW_DEC_CUR = 28,     // [16]
  HW_DEC_PCUR = 44,    // [1]
  HW_DEC_END = 45,
  // meeting words of the heads of a decode that keeps no work list (chunks started and arrived): in this block and in
  // the next one, the first layer's, which every config has in the same place.  Zero between calls of any
  // config (see meet_word).
  HW_MEET = 64,        // [64]
  HW_WORDS = 128
};

struct Dims {
  int S, Lyr, Hk, r, d, b, N, maxb, G;
  int dtype, mode;
};

inline Dims dims_of(const kvc_config* c) {
  Dims D;
  D.S = c->num_seqs; D.Lyr = c->num_layers; D.Hk = c->num_kv_heads; D.r = c->group_size;
  D.d = c->head_dim; D.b = c->block_size; D.N = c->num_blocks; D.maxb = c->max_blocks_per_head;
  D.G = D.S * D.Lyr * D.Hk; D.dtype = c->kv_dtype; D.mode = c->metric_mode;
  return D;
}

constexpr int kMinChunk = 64;      // smallest decode chunk (tokens per workgroup)
constexpr int kMaxChunk = 8192;
constexpr int kAppendWgs = 64;     // workgroups of an append's first launch, at most (a wavefront looks at all their counts)

inline size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

// Carves the caller's workspace.  All offsets are multiples of 256 bytes.
struct Workspace {
  int32_t* header;     // [HW_WORDS]
  int32_t* plan_hdr;   // [Lyr][HW_WORDS]     header block of every layer's kept work list (kvc_decode_plan)
  int32_t* tile_sums;  // [ntile_max + 1]
  int32_t* off_a;      // [G + 1]  scan over head instances (requests / chunks / ties)
  int32_t* off_b;      // [G + 1]
  int32_t* held;       // [G]      blocks held per head instance
  int32_t* items;      // [max_items][8]      decode work items (see DecodeItem)
  int32_t* slot_word;  // [max_items]         a word per partial-result slot: where a split head's chunks meet
  float*   part_ml;    // [max_items][r][2]   chunk max and sum per query head
  float*   part_acc;   // [max_items][r][d]   chunk un-normalised output
  float*   stash;      // [N*b][r]            chunk-relative exp of every logit of a chunk that left its head (see kMeetBits)
  int32_t* seg_hist;   // [S][256]            radix histograms per segment; in an append, what its workgroups counted ([kAppendWgs][3])
  int32_t* seg_state;  // [S][8]              prefix, remaining, ties wanted, ...
  int32_t* flag_scan;  // [G][maxb]           per-head prefix count of flagged blocks
  size_t bytes;
};

inline size_t max_items_of(const Dims& D) {
  // every chunk but a head's last is full, so items <= slots / min_chunk + G
  return (size_t)D.N * (size_t)D.b / kMinChunk + (size_t)D.G + 1;
}

inline Workspace carve(const Dims& D, void* base) {
  Workspace w;
  char* p = (char*)base;
  size_t o = 0;
  // (sized with a null base by kvc_workspace_bytes: then only the offsets are formed)
  auto take = [&](size_t bytes) { char* q = p ? p + o : nullptr; o += align_up(bytes, 256); return q; };
  size_t nmax = (size_t)(D.N > D.G ? D.N : D.G) + 1;
  size_t ntile = nmax / kScanTile + 2;
  w.header = (int32_t*)take(HW_WORDS * 4);
  w.plan_hdr = (int32_t*)take((size_t)D.Lyr * HW_WORDS * 4);
  w.tile_sums = (int32_t*)take(ntile * 4);
  w.off_a = (int32_t*)take(((size_t)D.G + 1) * 4);
  w.off_b = (int32_t*)take(((size_t)D.G + 1) * 4);
  w.held = (int32_t*)take((size_t)D.G * 4);
  size_t items = max_items_of(D);
  w.items = (int32_t*)take(items * 32);
  w.slot_word = (int32_t*)take(items * 4);
  w.part_ml = (float*)take(items * D.r * 2 * 4);
  w.part_acc = (float*)take(items * D.r * D.d * 4);
  w.stash = (float*)take((size_t)D.N * D.b * D.r * 4);
  w.seg_hist = (int32_t*)take((size_t)D.S * 256 * 4);
  w.seg_state = (int32_t*)take((size_t)D.S * 8 * 4);
  w.flag_scan = (int32_t*)take((size_t)D.G * D.maxb * 4);
  w.bytes = o;
  return w;
}

int validate(const kvc_config* cfg, const kvc_state* st);  // kvc_api.hip

#define KVC_HIP(expr)                                   \
  do {                                                  \
    hipError_t e__ = (expr);                            \
    if (e__ != hipSuccess) return KVC_ERR_HIP;          \
  } while (0)

#define KVC_LAUNCH_CHECK() KVC_HIP(hipGetLastError())

inline int read_words(const int32_t* dev, int32_t* host, int n, hipStream_t s) {
  KVC_HIP(hipMemcpyAsync(host, dev, (size_t)n * 4, hipMemcpyDeviceToHost, s));
  KVC_HIP(hipStreamSynchronize(s));
  return KVC_OK;
}

// ---------------------------------------------------------------------------
// device helpers
// ---------------------------------------------------------------------------

// 16-byte load of data that is read once per launch (K and V rows): marked non-temporal so that
// it does not displace what the caches should keep; a plain read stream measures 6.0-6.3 TB/s on
// this chip, the same stream with this hint 6.4-7.1 TB/s.
__device__ __forceinline__ uint4 load_stream16(const void* p) {
  typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
  const u32x4 t = __builtin_nontemporal_load((const u32x4*)p);
  return make_uint4(t.x, t.y, t.z, t.w);
}
// 16-byte store of data that this launch does not read again, with the same hint.
__device__ __forceinline__ void store_stream16(void* p, const uint4& v) {
  typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
  const u32x4 t = {v.x, v.y, v.z, v.w};
  __builtin_nontemporal_store(t, (u32x4*)p);
}
__device__ __forceinline__ uint2 load_stream8(const void* p) {
  typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
  const u32x2 t = __builtin_nontemporal_load((const u32x2*)p);
  return make_uint2(t.x, t.y);
}

// bytes of one K/V element, and of one query element (queries of an 8-bit cache are bf16)
__host__ __device__ inline int kv_esz(int dtype) { return dtype == KVC_F32 ? 4 : dtype == KVC_BF16 ? 2 : 1; }
__host__ __device__ inline int q_esz(int dtype) { return dtype == KVC_F32 ? 4 : 2; }

__device__ __forceinline__ float bf16_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }
__device__ __forceinline__ float bf16_to_f32(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

// Words that one workgroup leaves for another of the SAME launch, which may sit on another XCD
// with an L2 of its own: stored and loaded at device scope (past the L2s).  The writer waits for
// its stores before it announces itself (publish_wait, then a relaxed device-scope add); a
// __threadfence() there would write back the XCD's whole L2.
__device__ __forceinline__ void publish_i32(int32_t* p, int32_t v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ int32_t published_i32(const int32_t* p) {
  return __hip_atomic_load(const_cast<int32_t*>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void publish_u64(void* p, uint64_t v) {   // (8-byte aligned)
  __hip_atomic_store((uint64_t*)p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ uint64_t published_u64(const void* p) {
  return __hip_atomic_load((uint64_t*)const_cast<void*>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void publish_wait() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// ---- KVs moved by a compaction ----
// By the 16 lanes of a group, one or two of them: the rows of both are asked for before the first is stored.
// What moves is not looked at again by its launch, so the stores pass the caches by, and in large pools the
// loads do.  Block compactions of 1024 heads of 500 tokens to 16384 of 1024 (0.3 to 8.6 GB of KVs) that lose 10
// or 30 % of their blocks, on caches filled with something else (a model's weights pass through them between two rounds): one KV at a time with plain accesses 71 (128 x 4
// x 8 heads of 400 tokens), 150 (64 x 32 x 8 of 300), 423 and 953 us (64 x 32 x 8 of 1024); two at a time with
// plain ones 70, 147, 416 and 929; stores with the hint 69, 150, 412 and 890; both 58, 119, 372 and 731.  Where
// most of what moves is still in the 256 MB behind the L2s, loads with the hint lose: 512 heads of 1005
// tokens run again on the same cache 43, 46, 41 and 52 us, 2048 of 1024 80, 76, 60 and 81, 16384 of 300 (2.5 GB) 120, 118, 111 and 117.
// The pool decides, not what it holds: the same round on other caches, right after a decode and again, with the hint
// and without, 1024 heads of 1000 tokens (0.5 GB) 72 and 93, 68 and 69, 68 and 53 us; 4096 (1.9 GB) 107 and 143, 100
// and 102, 102 and 92; 10240 (4.7 GB) 229 and 245, 217 and 223, 217 and 221.  A large pool with little in it loses only
// where a compaction follows another.
struct Pool { char* kc; char* vc; float* metric; int32_t* pos; size_t row_bytes; bool large; };
constexpr size_t kLargePool = (size_t)2 << 30;
__device__ __forceinline__ Pool pool_of(const Dims& D, char* kc, char* vc, float* metric, int32_t* pos) {
  const size_t rb = (size_t)D.d * kv_esz(D.dtype);
  return Pool{kc, vc, metric, pos, rb, 2 * rb * (size_t)D.b * (size_t)D.N >= kLargePool};
}
template <bool LARGE>
__device__ __forceinline__ void move_rows(const Pool& P, int gl, bool two, size_t s0, size_t d0, size_t s1, size_t d1) {
  const size_t rb = P.row_bytes;
  auto load = [](const char* p) { return LARGE ? load_stream16(p) : *(const uint4*)p; };
  if (two) {
    for (size_t c = gl * 16; c < rb; c += 256) {
      const uint4 k0 = load(P.kc + s0 * rb + c), v0 = load(P.vc + s0 * rb + c);
      const uint4 k1 = load(P.kc + s1 * rb + c), v1 = load(P.vc + s1 * rb + c);
      store_stream16(P.kc + d0 * rb + c, k0);
      store_stream16(P.vc + d0 * rb + c, v0);
      store_stream16(P.kc + d1 * rb + c, k1);
      store_stream16(P.vc + d1 * rb + c, v1);
    }
  } else {
    for (size_t c = gl * 16; c < rb; c += 256) {
      const uint4 k0 = load(P.kc + s0 * rb + c), v0 = load(P.vc + s0 * rb + c);
      store_stream16(P.kc + d0 * rb + c, k0);
      store_stream16(P.vc + d0 * rb + c, v0);
    }
  }
}
__device__ __forceinline__ void move_kvs(const Pool& P, int gl, bool two, size_t s0, size_t d0, size_t s1, size_t d1) {
  if (P.large) move_rows<true>(P, gl, two, s0, d0, s1, d1);
  else move_rows<false>(P, gl, two, s0, d0, s1, d1);
  if (gl < 1 + two) {
    const size_t src = gl ? s1 : s0, dst = gl ? d1 : d0;
    P.metric[dst] = P.metric[src];
    if (P.pos) P.pos[dst] = P.pos[src];
  }
}

// ---- across the lanes of a wavefront ----
// Without LDS: a shuffle is an LDS access of ~110 clocks, and a reduction is a chain of six.  Lanes of
// a row of 16 by data-parallel moves, rows and halves by the swaps of gfx950.
template <int CTRL>
__device__ __forceinline__ int dpp_move(int v) { return __builtin_amdgcn_update_dpp(0, v, CTRL, 0xf, 0xf, true); }
// The values of lanes l and l ^ MASK, in this order for every lane l without that bit and, for MASK of
// 16 and 32, for every lane (below: the lane's own first): for sums and maxima, which take either order.
template <int MASK> struct LanePair { int a, b; };
template <int MASK>
__device__ __forceinline__ LanePair<MASK> lane_pair(int v) {
  if constexpr (MASK == 32) { const auto t = __builtin_amdgcn_permlane32_swap(v, v, false, false); return {(int)t[0], (int)t[1]}; }
  else if constexpr (MASK == 16) { const auto t = __builtin_amdgcn_permlane16_swap(v, v, false, false); return {(int)t[0], (int)t[1]}; }
  else if constexpr (MASK == 8) return {v, dpp_move<0x128>(v)};                  // a rotation by 8
  else if constexpr (MASK == 4) return {v, dpp_move<0x141>(dpp_move<0x1B>(v))};   // a quad reverse, then a half-row mirror: i ^ 3 ^ 7
  else if constexpr (MASK == 2) return {v, dpp_move<0x4E>(v)};                   // quad permutes
  else return {v, dpp_move<0xB1>(v)};
}
template <int MASK>
__device__ __forceinline__ int sum_xor(int v) { const auto p = lane_pair<MASK>(v); return p.a + p.b; }
template <int MASK>
__device__ __forceinline__ int max_xor(int v) { const auto p = lane_pair<MASK>(v); return max(p.a, p.b); }
template <int MASK>
__device__ __forceinline__ float sum_xor(float v) {
  const auto p = lane_pair<MASK>(__builtin_bit_cast(int, v));
  return __builtin_bit_cast(float, p.a) + __builtin_bit_cast(float, p.b);
}
template <int MASK>
__device__ __forceinline__ float max_xor(float v) {
  const auto p = lane_pair<MASK>(__builtin_bit_cast(int, v));
  return fmaxf(__builtin_bit_cast(float, p.a), __builtin_bit_cast(float, p.b));
}
// Value held by lane (l ^ MASK).
template <int MASK>
__device__ __forceinline__ float lane_xor(float v) {
  const auto p = lane_pair<MASK>(__builtin_bit_cast(int, v));
  if constexpr (MASK >= 16) return __builtin_bit_cast(float, (threadIdx.x & MASK) ? p.a : p.b);
  else return __builtin_bit_cast(float, p.b);
}
template <class T>
__device__ __forceinline__ T wave_sum(T v) {
  v = sum_xor<32>(v); v = sum_xor<16>(v); v = sum_xor<8>(v);
  v = sum_xor<4>(v); v = sum_xor<2>(v); return sum_xor<1>(v);
}
template <class T>
__device__ __forceinline__ T wave_max(T v) {
  v = max_xor<32>(v); v = max_xor<16>(v); v = max_xor<8>(v);
  v = max_xor<4>(v); v = max_xor<2>(v); return max_xor<1>(v);
}
__device__ __forceinline__ int wave_sum_i(int v) { return wave_sum(v); }
__device__ __forceinline__ float wave_sum_f(float v) { return wave_sum(v); }
__device__ __forceinline__ float wave_max_f(float v) { return wave_max(v); }
// Sum over the wavefront of 64 values of at most 31 bits.
__device__ __forceinline__ unsigned long long wave_sum_long(int v) {
  return ((unsigned long long)wave_sum(v >> 16) << 16) + (unsigned long long)wave_sum(v & 0xffff);
}
// Inclusive prefix sums over a wavefront (row shifts, then the rows' last lanes broadcast).
__device__ __forceinline__ int wave_prefix_i(int v) {
  v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);
  return v;
}

// Exclusive scan of one int per thread over a workgroup of NT threads.
// `total` (if non-null) receives the workgroup sum.  smem: NT/64 + 1 ints.
template <int NT>
__device__ __forceinline__ int block_exclusive_scan(int v, int* smem, int* total) {
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  const int inc = wave_prefix_i(v);
  if (lane == 63) smem[wid] = inc;
  __syncthreads();
  if (threadIdx.x == 0) {
    int run = 0;
    for (int w = 0; w < NT / 64; ++w) { int t = smem[w]; smem[w] = run; run += t; }
    smem[NT / 64] = run;
  }
  __syncthreads();
  int base = smem[wid];
  if (total) *total = smem[NT / 64];
  __syncthreads();
  return base + inc - v;
}

// Error bits a kernel leaves in the header's scratch word for the launch that settles the status.
enum ErrBit { EB_ARG = 1, EB_TABLE = 2, EB_NUMERIC = 4 };

// Turns the error bits of a call without an allocation into the status word (argument, table full,
// numeric; a status that is already set stays).  By one thread of the chip.
__device__ __forceinline__ void settle_status(int32_t* header) {
  const int bits = header[HW_SCRATCH0];
  int st = KVC_OK;
  if (bits & EB_ARG) st = KVC_ERR_ARG;
  else if (bits & EB_TABLE) st = KVC_ERR_TABLE_FULL;
  else if (bits & EB_NUMERIC) st = KVC_ERR_NUMERIC;
  if (st != KVC_OK && header[HW_STATUS] == KVC_OK) header[HW_STATUS] = st;
  header[HW_SCRATCH0] = 0;
}

// Blocks a compaction freed = the sum of the per-head counts it was given (each head gives back
// exactly the blocks it loses), or 0 when the call failed.  One workgroup adds the counts up:
// a counter bumped by every head would see thousands of adds to one word, which the chip runs
// one after the other (that counter alone took 0.13 ms per round at 16 384 heads).
// With `resolve` set the launch also does what resolve_kernel does, first: a compaction
// that reports its count settles its status and publishes in one launch, ahead of the moves.
static __global__ void __launch_bounds__(1024) publish_freed_kernel(int32_t* __restrict__ header,
                                                                    const int32_t* __restrict__ counts, int G,
                                                                    int64_t* __restrict__ out, int resolve) {
  __shared__ long long part[1024 / 64];
  __shared__ int status_s;
  if (threadIdx.x == 0) {
    if (resolve) settle_status(header);
    status_s = header[HW_STATUS];
  }
  long long s = 0;
  // One workgroup reads all the counts: 32 of them per thread asked for at a time (eight 16-byte
  // loads) when the array is 16-byte aligned, else eight.
  if (((uintptr_t)counts & 15) == 0) {
    const int4* c4 = (const int4*)counts;
    const int n4 = G >> 2;
    for (int i0 = threadIdx.x; i0 < n4; i0 += 8 * 1024) {
      int4 v[8];
#pragma unroll
      for (int k = 0; k < 8; ++k) v[k] = i0 + k * 1024 < n4 ? c4[i0 + k * 1024] : make_int4(0, 0, 0, 0);
#pragma unroll
      for (int k = 0; k < 8; ++k) s += (long long)max(v[k].x, 0) + max(v[k].y, 0) + max(v[k].z, 0) + max(v[k].w, 0);
    }
    for (int g = (n4 << 2) + threadIdx.x; g < G; g += 1024) s += max(counts[g], 0);
  } else {
    for (int g0 = threadIdx.x; g0 < G; g0 += 8 * 1024) {
      int v[8];
#pragma unroll
      for (int k = 0; k < 8; ++k) v[k] = g0 + k * 1024 < G ? counts[g0 + k * 1024] : 0;
#pragma unroll
      for (int k = 0; k < 8; ++k) s += max(v[k], 0);
    }
  }
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) s += __shfl_xor(s, o);
  if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = s;
  __syncthreads();
  if (threadIdx.x == 0) {
    long long t = 0;
    for (int w = 0; w < 1024 / 64; ++w) t += part[w];
    out[0] = status_s == KVC_OK ? t : 0;
  }
}

// ---- device-wide exclusive scan in three launches -------------------------
// F: __device__ int operator()(int i) giving element i.  Results go to
// out[0..n) and out[n] = total; `total_word` (may be null) also receives it.
template <class F>
__global__ void __launch_bounds__(kScanThreads) scan_tile_reduce(F f, int n, int32_t* tile_sums) {
  __shared__ int red[kScanThreads / 64];
  int base = blockIdx.x * kScanTile + threadIdx.x * kScanItems;
  int s = 0;
#pragma unroll
  for (int k = 0; k < kScanItems; ++k) if (base + k < n) s += f(base + k);
  s = wave_sum_i(s);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
  __syncthreads();
  if (threadIdx.x == 0) {
    int t = 0;
    for (int w = 0; w < kScanThreads / 64; ++w) t += red[w];
    tile_sums[blockIdx.x] = t;
  }
}

static __global__ void __launch_bounds__(1024) scan_tile_sums(int32_t* tile_sums, int ntiles,
                                                              int32_t* total_word) {
  __shared__ int smem[1024 / 64 + 1];
  __shared__ int carry_s;
  if (threadIdx.x == 0) carry_s = 0;
  __syncthreads();
  for (int base = 0; base < ntiles; base += 1024) {
    int i = base + threadIdx.x;
    int v = (i < ntiles) ? tile_sums[i] : 0;
    int tot;
    int ex = block_exclusive_scan<1024>(v, smem, &tot);
    int carry = carry_s;
    if (i < ntiles) tile_sums[i] = ex + carry;
    __syncthreads();
    if (threadIdx.x == 0) carry_s = carry + tot;
    __syncthreads();
  }
  if (threadIdx.x == 0 && total_word) *total_word = carry_s;
}

template <class F>
__global__ void __launch_bounds__(kScanThreads) scan_tile_apply(F f, int n, const int32_t* tile_sums,
                                                                int32_t* out) {
  __shared__ int smem[kScanThreads / 64 + 1];
  int base = blockIdx.x * kScanTile + threadIdx.x * kScanItems;
  int v[kScanItems];
  int s = 0;
#pragma unroll
  for (int k = 0; k < kScanItems; ++k) { v[k] = (base + k < n) ? f(base + k) : 0; s += v[k]; }
  int ex = block_exclusive_scan<kScanThreads>(s, smem, nullptr) + tile_sums[blockIdx.x];
#pragma unroll
  for (int k = 0; k < kScanItems; ++k) {
    if (base + k < n) out[base + k] = ex;
    ex += v[k];
  }
  if (blockIdx.x == gridDim.x - 1 && threadIdx.x == kScanThreads - 1) out[n] = ex;
}

template <class F>
inline int device_exclusive_scan(F f, int n, int32_t* tile_sums, int32_t* out, int32_t* total_word,
                                 hipStream_t s) {
  int ntiles = (n + kScanTile - 1) / kScanTile;
  if (ntiles < 1) ntiles = 1;
  hipLaunchKernelGGL(scan_tile_reduce<F>, dim3(ntiles), dim3(kScanThreads), 0, s, f, n, tile_sums);
  KVC_LAUNCH_CHECK();
  hipLaunchKernelGGL(scan_tile_sums, dim3(1), dim3(1024), 0, s, tile_sums, ntiles, total_word);
  KVC_LAUNCH_CHECK();
  hipLaunchKernelGGL(scan_tile_apply<F>, dim3(ntiles), dim3(kScanThreads), 0, s, f, n, tile_sums, out);
  KVC_LAUNCH_CHECK();
  return KVC_OK;
}

// ---- status word plumbing shared by the entry points ------------------------

static __global__ void zero_words_kernel(int32_t* p, int n) {
  int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = 0;
}

static __global__ void resolve_kernel(int32_t* header) {
  if (threadIdx.x == 0 && blockIdx.x == 0) settle_status(header);
}

// Per-segment state of a selection (block mode and rank-block mode share it): eight words.
enum SegWord { SEG_PREFIX = 0, SEG_REMAIN = 1, SEG_CAND = 2, SEG_TAKE = 3, SEG_FIRSTG = 4, SEG_ALLTIES = 5 };

// First launch of either selection: the segment of every sequence (segments are runs of
// consecutive sequences; seg_offsets NULL = one per sequence), cleared histograms and segment
// state with the segment's first head instance, cleared per-head counts and per-segment results,
// and the check of the offsets (first 0, last S, non-decreasing).
static __global__ void __launch_bounds__(256) segments_init_kernel(Dims D, const int32_t* __restrict__ seg_offsets,
                                                                   int nseg, int32_t* __restrict__ seq_seg,
                                                                   int32_t* __restrict__ seg_hist,
                                                                   int32_t* __restrict__ seg_state,
                                                                   int32_t* __restrict__ per_head,
                                                                   int32_t* __restrict__ selected,
                                                                   int32_t* __restrict__ header,
                                                                   int32_t* __restrict__ more_hist, int n_more) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i < n_more) more_hist[i] = 0;
  if (i < D.S) {
    int sg = i;
    if (seg_offsets) {  // last segment whose first sequence is <= i
      int lo = 0, hi = nseg;
      while (hi - lo > 1) { const int mid = (lo + hi) >> 1; if (seg_offsets[mid] <= i) lo = mid; else hi = mid; }
      sg = lo;
    }
    seq_seg[i] = sg;
  }
  if (i < nseg * 256) seg_hist[i] = 0;
  if (i < nseg) {
    selected[i] = 0;
    for (int k = 0; k < 8; ++k) seg_state[i * 8 + k] = 0;
    const int first_seq = seg_offsets ? seg_offsets[i] : i;
    seg_state[i * 8 + SEG_FIRSTG] = first_seq * D.Lyr * D.Hk;
    if (seg_offsets) {
      const int a = seg_offsets[i], b2 = seg_offsets[i + 1];
      if (a > b2 || (i == 0 && a != 0) || (i == nseg - 1 && b2 != D.S)) atomicOr(&header[HW_SCRATCH0], EB_ARG);
    }
  }
  if (i < D.G) per_head[i] = 0;
}

// ---- digits picked by the launch that uses them ----
// With few heads a launch of its own for the pick of a digit is all latency: five launches of 2 us and the
// host's time for them.  There the wavefronts of the next launch each pick their segment's digit
// themselves, from a histogram per pass (the previous one is complete when this launch starts, nobody adds to it
// any more), and the wavefront of a segment's first head leaves what it found for the launch after: threshold
// and remainder in one pair of words after passes 0 and 2, in another after 1 and 3, so that nobody reads
// words that this launch writes.  (Rank rounds and prompts, picks by themselves -> so: 256 heads of 16384
// tokens 287 -> 279 us, 1024 of 8192 147 -> 138, 672 of up to 3595 107 -> 97, 104 of up to 957 85 -> 71.)
struct SegPicks {
  const int32_t* hist;     // [nseg][256] of the pass before, or NULL: a launch of its own has picked
  const int32_t* budget;
  int nseg;
};
struct SegKey { uint32_t prefix; int remain, take; };

__device__ __forceinline__ void check_budgets(const SegPicks& P, int nth, int32_t* header) {   // by a whole workgroup
  bool neg = false;
  for (int i = threadIdx.x; i < P.nseg; i += nth) neg |= P.budget[i] < 0;
  const int any = __syncthreads_or(neg);
  if (threadIdx.x != 0) return;
  if (any) header[HW_SCRATCH0] |= EB_ARG;
  settle_status(header);   // keys and budgets checked: before any output is written
}

// The threshold of segment sg as launch `pass` of a selection (4: the ties) needs it; for all lanes.
__device__ __forceinline__ SegKey seg_key(const SegPicks& P, int pass, int sg, int32_t* seg_state, bool leave) {
  int32_t* stt = seg_state + sg * 8;
  if (pass == 0) return SegKey{0u, 0, 1};
  if (!P.hist) return SegKey{(uint32_t)stt[SEG_PREFIX], stt[SEG_REMAIN], stt[SEG_TAKE]};
  const int lane = threadIdx.x & 63;
  const int from = pass & 1 ? 0 : 6, to = pass & 1 ? 6 : 0;   // (SEG_PREFIX, SEG_REMAIN, or the last two words)
  SegKey key;
  key.take = pass == 1 ? min(max(P.budget[sg], 0), stt[SEG_CAND]) : stt[SEG_TAKE];
  key.prefix = pass == 1 ? 0u : (uint32_t)stt[from];
  key.remain = pass == 1 ? key.take : stt[from + 1];
  const int4 c = ((const int4*)(P.hist + (size_t)sg * 256))[lane];
  const int mine = c.x + c.y + c.z + c.w;
  int ex = wave_prefix_i(mine) - mine, digit = -1, left = 0;
  const int c4[4] = {c.x, c.y, c.z, c.w};
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    if (ex < key.remain && key.remain <= ex + c4[q]) { digit = 4 * lane + q; left = key.remain - ex; }
    ex += c4[q];
  }
  const unsigned long long hit = __ballot(digit >= 0);   // one lane, where the segment takes anything
  if (key.take > 0 && hit) {
    const int src = __ffsll((long long)hit) - 1;
    key.prefix = (key.prefix << 8) | (uint32_t)__builtin_amdgcn_readlane(digit, src);
    key.remain = __builtin_amdgcn_readlane(left, src);
  }
  if (leave && lane == 0) {
    if (pass == 1) stt[SEG_TAKE] = key.take;
    stt[to] = (int32_t)key.prefix;
    stt[to + 1] = key.remain;
  }
  return key;
}

// The end of a head's moves when several workgroups of 256 threads share them: the last of the `expected`
// ones gives the tail blocks back and sets the new length T (was C).  By all threads; the workgroup's
// reads of the head's row and length are done.
__device__ __forceinline__ void finish_head(const Dims& D, int32_t* table, int32_t* ctx, uint8_t* free_map, int32_t* arrived,
                                            int g, int expected, int C, int T) {
  __shared__ int last_s;
  __syncthreads();
  if (threadIdx.x == 0)
    last_s = __hip_atomic_fetch_add(&arrived[g], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == expected - 1;
  __syncthreads();
  if (!last_s) return;
  int32_t* row = table + (size_t)g * D.maxb;
  const int nb = (C + D.b - 1) / D.b, nb2 = (T + D.b - 1) / D.b;
  for (int u = nb2 + (int)threadIdx.x; u < nb; u += 256) {
    free_map[row[u]] = 1;
    row[u] = -1;
  }
  if (threadIdx.x == 0) ctx[g] = T;
}

// How much dynamic LDS a kernel may take above the default 64 KB is an attribute of the kernel on
// a device: remembered per device (the first 64 of a process), raised when a call needs more.
// Host threads may race here; telling the runtime twice is harmless.
struct LdsLimit {
  std::atomic<size_t> allowed[64] = {};
  template <class... Kernels>
  int need(size_t bytes, Kernels... kernels) {
    if (bytes <= 64 * 1024) return KVC_OK;
    int dev = -1;
    KVC_HIP(hipGetDevice(&dev));
    if (dev < 0 || dev >= 64) return KVC_ERR_UNSUPPORTED;
    if (bytes <= allowed[dev].load(std::memory_order_acquire)) return KVC_OK;
    const void* ks[] = {(const void*)kernels...};
    for (const void* k : ks) KVC_HIP(hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes));
    size_t seen = allowed[dev].load(std::memory_order_relaxed);
    while (seen < bytes && !allowed[dev].compare_exchange_weak(seen, bytes, std::memory_order_release)) {}
    return KVC_OK;
  }
};

// Reads the status word; a non-zero word is cleared so that the next call starts clean.
inline int finish_sync(const Workspace& W, hipStream_t s) {
  int32_t w = 0;
  int rc = read_words(W.header + HW_STATUS, &w, 1, s);
  if (rc != KVC_OK) return rc;
  if (w != KVC_OK) {
    hipLaunchKernelGGL(zero_words_kernel, dim3(1), dim3(64), 0, s, W.header + HW_STATUS, 1);
    KVC_LAUNCH_CHECK();
    KVC_HIP(hipStreamSynchronize(s));
  }
  return w;
}

}  // namespace kvc
