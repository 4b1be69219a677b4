// On-device block manager: parallel counting and allocation over all
// (sequence, layer, head) instances against a flat length-N free map
// (KV-Compress, Method, "Block Layout and Parallel Allocation"), plus the
// append that stores a new token's key and value.
//
// Order rule (the paper leaves it open): requesters in ascending head-instance
// index; the k-th requested block is the k-th lowest-numbered free block.
// Every launch that writes cache state first reads the workspace status word
// and does nothing when an earlier step of the same call has failed.
#include "kvc_common.h"

namespace kvc {

// blocks held = non-negative prefix of the row; rows are prefix-filled and
// cover at least ceil(ctx_len / b) cells, so the search starts there.
__device__ __forceinline__ int held_blocks(const int32_t* row, int C, int b, int maxb) {
  int u = (C + b - 1) / b;
  while (u < maxb && row[u] >= 0) ++u;
  return u;
}

// Drop counts n[g] of kvc_block_free: blocks held per head instance, checked request.
__global__ void __launch_bounds__(256) count_drop_kernel(Dims D, const int32_t* __restrict__ table,
                                                         const int32_t* __restrict__ ctx,
                                                         const int32_t* __restrict__ n,
                                                         int32_t* __restrict__ held,
                                                         int32_t* __restrict__ req,
                                                         int32_t* __restrict__ header) {
  const int g = blockIdx.x * 256 + threadIdx.x;
  if (g >= D.G) return;
  const int h = held_blocks(table + (size_t)g * D.maxb, ctx[g], D.b, D.maxb);
  held[g] = h;
  int want = n[g];
  if (want < 0 || want > h) { atomicOr(&header[HW_SCRATCH0], EB_ARG); want = 0; }
  req[g] = want;
}

// What an allocation is asked for: the caller's counts n[g] (ALLOC_COUNTS); blocks up to
// ceil(n[s] / b) for every head of a sequence s with n[s] > 0 tokens (ALLOC_PREFILL).
enum AllocMode { ALLOC_COUNTS = 0, ALLOC_PREFILL = 1 };

// Launch 1 of an allocation: workgroups [0, gb) count requests per head instance, workgroups [gb, gb + ntiles) count the free blocks of one tile of the map.
__global__ void __launch_bounds__(256) count_and_free_tiles_kernel(Dims D, const int32_t* __restrict__ table,
                                                                   const int32_t* __restrict__ ctx,
                                                                   const int32_t* __restrict__ n, int mode, int gb,
                                                                   const uint8_t* __restrict__ free_map,
                                                                   int32_t* __restrict__ held,
                                                                   int32_t* __restrict__ req,
                                                                   int32_t* __restrict__ tile_sums,
                                                                   int32_t* __restrict__ header) {
  if ((int)blockIdx.x < gb) {
    const int g = blockIdx.x * 256 + threadIdx.x;
    if (g >= D.G) return;
    const int C = ctx[g];
    const int h = held_blocks(table + (size_t)g * D.maxb, C, D.b, D.maxb);
    held[g] = h;
    int want = 0, bits = 0;
    if (mode == ALLOC_COUNTS) {
      want = n[g];
    } else {
      const int t = n[g / (D.Lyr * D.Hk)];
      want = t > 0 ? max(0, (t + D.b - 1) / D.b - h) : t;
    }
    if (want < 0) { bits |= EB_ARG; want = 0; }
    else if (h + want > D.maxb) bits |= EB_TABLE;
    req[g] = want;
    if (bits) atomicOr(&header[HW_SCRATCH0], bits);
    return;
  }
  __shared__ int red[kScanThreads / 64];
  const int tile = blockIdx.x - gb;
  const int base = tile * kScanTile + threadIdx.x * kScanItems;
  int s = 0;
#pragma unroll
  for (int k = 0; k < kScanItems; ++k) if (base + k < D.N) s += free_map[base + k] != 0;
  s = wave_sum_i(s);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
  __syncthreads();
  if (threadIdx.x == 0) tile_sums[tile] = red[0] + red[1] + red[2] + red[3];
}

constexpr int kScanRun = 16;                   // elements per thread and tile in alloc_scan_kernel
constexpr int kScanWide = 1024 * kScanRun;     // elements per tile

// Exclusive scan of n ints over one workgroup of 1024 threads: every thread takes a run of 16
// consecutive elements (four 16-byte loads and, for the results, four 16-byte stores when the
// arrays are 16-byte aligned, which workspace arrays are: a thread's run is 64 bytes, so with
// 4-byte accesses every instruction of a wavefront touched 64 different lines), one workgroup
// scan joins the runs.  out[i] = exclusive prefix (out may be `in`).
__device__ __forceinline__ int wide_exclusive_scan(const int32_t* in, int n, int32_t* out, int* smem) {
  __shared__ int carry_s;
  if (threadIdx.x == 0) carry_s = 0;
  __syncthreads();
  const bool aligned = (((uintptr_t)in | (uintptr_t)out) & 15) == 0;
  for (int base = 0; base < n; base += kScanWide) {
    const int first = base + threadIdx.x * kScanRun;
    const bool whole = aligned && first + kScanRun <= n;
    int v[kScanRun], sum = 0;
    if (whole) {
#pragma unroll
      for (int k = 0; k < kScanRun; k += 4) {
        const int4 t = *(const int4*)(in + first + k);
        v[k] = t.x; v[k + 1] = t.y; v[k + 2] = t.z; v[k + 3] = t.w;
      }
    } else {
#pragma unroll
      for (int k = 0; k < kScanRun; ++k) v[k] = first + k < n ? in[first + k] : 0;
    }
#pragma unroll
    for (int k = 0; k < kScanRun; ++k) sum += v[k];
    int tot;
    int ex = block_exclusive_scan<1024>(sum, smem, &tot) + carry_s;
    int o[kScanRun];
#pragma unroll
    for (int k = 0; k < kScanRun; ++k) {
      o[k] = ex;
      ex += v[k];
    }
    if (whole) {
#pragma unroll
      for (int k = 0; k < kScanRun; k += 4) *(int4*)(out + first + k) = make_int4(o[k], o[k + 1], o[k + 2], o[k + 3]);
    } else {
#pragma unroll
      for (int k = 0; k < kScanRun; ++k) if (first + k < n) out[first + k] = o[k];
    }
    __syncthreads();
    if (threadIdx.x == 0) carry_s += tot;
    __syncthreads();
  }
  return carry_s;
}

// Launch 2, one workgroup: exclusive scan of the requests (off[g], off[G] = total), exclusive
// scan of the free-tile counts, and the status word.
__global__ void __launch_bounds__(1024) alloc_scan_kernel(Dims D, const int32_t* __restrict__ req,
                                                          int32_t* __restrict__ off,
                                                          int32_t* __restrict__ tile_sums, int ntiles,
                                                          int32_t* __restrict__ header) {
  __shared__ int smem[1024 / 64 + 1];
  const int total_req = wide_exclusive_scan(req, D.G, off, smem);
  const int total_free = wide_exclusive_scan(tile_sums, ntiles, tile_sums, smem);
  if (threadIdx.x == 0) {
    off[D.G] = total_req;
    header[HW_TOTAL_REQ] = total_req;
    header[HW_TOTAL_FREE] = total_free;
    const int bits = header[HW_SCRATCH0];
    int st = KVC_OK;
    if (bits & EB_ARG) st = KVC_ERR_ARG;
    else if (bits & EB_TABLE) st = KVC_ERR_TABLE_FULL;
    else if (total_req > total_free) st = KVC_ERR_OOM;
    if (st != KVC_OK && header[HW_STATUS] == KVC_OK) header[HW_STATUS] = st;
    header[HW_SCRATCH0] = 0;
  }
}

// Third phase of the scan over the free map, fused with the hand-out: the free block of
// rank k (ascending id) goes to the head instance g with off[g] <= k < off[g + 1], as its
// (k - off[g])-th new block.  A thread's free blocks are consecutive in rank: it searches for the
// head of its first one and looks at that head again before it searches for the next.  (The
// scan's single workgroup writing every request's head into a list instead was one thread's
// serial run per head: 595 us for a prompt of 1024 blocks a head, 8 us for the whole launch here.)
// seq_tokens (a prefill): the lengths of the heads follow in the same launch.
__global__ void __launch_bounds__(kScanThreads) pick_scatter_kernel(Dims D, int32_t* __restrict__ table,
                                                                    uint8_t* __restrict__ free_map,
                                                                    const int32_t* __restrict__ tile_sums,
                                                                    const int32_t* __restrict__ held,
                                                                    const int32_t* __restrict__ off,
                                                                    const int32_t* __restrict__ seq_tokens,
                                                                    int32_t* __restrict__ ctx,
                                                                    const int32_t* __restrict__ header) {
  __shared__ int smem[kScanThreads / 64 + 1];
  const int total_req = header[HW_TOTAL_REQ];
  if (header[HW_STATUS] != KVC_OK) return;
  if (seq_tokens)
    for (int g = blockIdx.x * kScanThreads + threadIdx.x; g < D.G; g += gridDim.x * kScanThreads) {
      const int t = seq_tokens[g / (D.Lyr * D.Hk)];
      if (t > 0) ctx[g] = t;
    }
  const int tile0 = tile_sums[blockIdx.x];
  if (tile0 >= total_req) return;  // uniform over the workgroup
  const int base = blockIdx.x * kScanTile + threadIdx.x * kScanItems;
  int v[kScanItems];
  int s = 0;
#pragma unroll
  for (int k = 0; k < kScanItems; ++k) { v[k] = (base + k < D.N) ? (free_map[base + k] != 0) : 0; s += v[k]; }
  int ex = block_exclusive_scan<kScanThreads>(s, smem, nullptr) + tile0;
  int g = -1, first = 0, end = 0;   // head instance in hand, its requests' ranks first .. end - 1
#pragma unroll
  for (int k = 0; k < kScanItems; ++k) {
    if (v[k]) {
      if (ex < total_req) {
        if (ex >= end) {   // the last head with off[g] <= ex: its own requests are not empty
          int lo = g < 0 ? 0 : g, hi = D.G;
          while (hi - lo > 1) { const int mid = (lo + hi) >> 1; if (off[mid] <= ex) lo = mid; else hi = mid; }
          g = lo;
          first = off[g];
          end = off[g + 1];
        }
        table[(size_t)g * D.maxb + held[g] + (ex - first)] = base + k;
        free_map[base + k] = 0;
      }
      ++ex;
    }
  }
}

__global__ void __launch_bounds__(256) drop_kernel(Dims D, int32_t* __restrict__ table,
                                                   int32_t* __restrict__ ctx,
                                                   uint8_t* __restrict__ free_map,
                                                   const int32_t* __restrict__ held,
                                                   const int32_t* __restrict__ req,
                                                   int32_t* __restrict__ header) {
  if (header[HW_STATUS] != KVC_OK) return;
  int g = blockIdx.x * 256 + threadIdx.x;
  int n = 0;
  if (g < D.G) {
    n = req[g];
    if (n > 0) {
      int h = held[g];
      int32_t* row = table + (size_t)g * D.maxb;
      for (int u = h - n; u < h; ++u) { free_map[row[u]] = 1; row[u] = -1; }
      int cap = (h - n) * D.b;
      if (ctx[g] > cap) ctx[g] = cap;
    }
  }
  int tot = wave_sum_i(n);
  if ((threadIdx.x & 63) == 0 && tot) atomicAdd(&header[HW_FREED], tot);
}

// What an append writes for one head, by a group of lanes (lane gl of lanes_per_head): the rows,
// metric 0, the logical index, the length.
struct AppendArgs {
  Dims D;
  int l0, nl, nsel;        // layers and head instances appended to
  int lanes_per_head;
  int lb;                  // log2 of the block size
  char* kc;
  char* vc;
  float* metric;
  int32_t* pos;
  int32_t* table;
  int32_t* ctx;
  uint8_t* free_map;
  const char* k_new;
  const char* v_new;
  const int32_t* new_pos;
  int32_t* header;
  int32_t* part;           // [workgroups][3] requests, free blocks, error bits
  int32_t* list;           // [nsel] requesters of workgroup w from its first head's place on
};

__device__ __forceinline__ int append_head(const AppendArgs& A, int idx) {
  const int s = idx / (A.nl * A.D.Hk);
  return (s * A.D.Lyr + A.l0 + (idx / A.D.Hk) % A.nl) * A.D.Hk + idx % A.D.Hk;
}

__device__ __forceinline__ void append_one(const AppendArgs& A, int idx, int gl) {
  const int g = append_head(A, idx);
  const int C = A.ctx[g];
  const int blk = A.table[(size_t)g * A.D.maxb + (C >> A.lb)];
  const size_t row_bytes = (size_t)A.D.d * kv_esz(A.D.dtype);
  const size_t slot = ((size_t)blk << A.lb) + (C & (A.D.b - 1));
  const int pieces = (int)(row_bytes / 16);
  for (int c = gl; c < 2 * pieces; c += A.lanes_per_head) {
    const bool is_v = c >= pieces;
    const int cc = is_v ? c - pieces : c;
    const uint4* src = (const uint4*)((is_v ? A.v_new : A.k_new) + (size_t)g * row_bytes) + cc;
    uint4* dst = (uint4*)((is_v ? A.vc : A.kc) + slot * row_bytes) + cc;
    *dst = *src;
  }
  // the lanes of a group belong to one wavefront (one instruction stream): all of them have read
  // ctx[g] by the time one of them writes it
  if (gl == 0) {
    A.metric[slot] = 0.0f;
    if (A.pos) A.pos[slot] = A.new_pos ? A.new_pos[g / (A.D.Lyr * A.D.Hk)] : C;
    A.ctx[g] = C + 1;
  }
}

// free bytes (non-zero) of a 32-bit word, as the top bits of its bytes
__device__ __forceinline__ uint32_t nonzero_bytes(uint32_t x) {
  return (((x & 0x7f7f7f7fu) + 0x7f7f7f7fu) | x) & 0x80808080u;
}
// 16 bytes of the free map from `at` on (bytes past `end` read as 0)
__device__ __forceinline__ uint4 free_bytes16(const uint8_t* map, size_t at, size_t end, bool wide) {
  if (wide && at + 16 <= end) return *(const uint4*)(map + at);
  uint32_t w[4] = {0, 0, 0, 0};
  for (int k = 0; k < 16; ++k)
    if (at + k < end) w[k >> 2] |= (uint32_t)map[at + k] << (8 * (k & 3));
  return make_uint4(w[0], w[1], w[2], w[3]);
}

// The whole reservation of an append in one launch: which heads need a block (their length fills
// the blocks they hold), the lowest free blocks for them in ascending head order, the error
// checks before anything is written; for few heads also the append itself.
//
// Workgroup w of n looks at its share of the heads and of the free map, leaves its counts and the
// list of its requesters, and announces itself; the last one to arrive reads all the counts (one
// wavefront: n <= 64), settles the status and hands the blocks out, walking only the shares of
// the map that hold the first blocks it needs.  In place of a launch each for counting, for a
// scan in one workgroup over all heads, and for a second walk over the whole map: a launch costs
// ~4.5 us in a busy stream whatever it does (with the rows: 16 384 heads, 1.35 M blocks 23.2 ->
// 12.8 us; one layer of one sequence 16.4 -> 6.6 us).
constexpr int kAppendThreads = 1024;
// Heads appended by the same launch.  One CU writing rows all over the pool pays for them one
// round of 32 heads after the other: 128 heads 12.3 us in one launch against 10.5 in two, 256 heads
// 19.6 against 10.0 (all rows of a round asked for at once), 8 heads 6.6 against 10.
constexpr int kAppendFused = 64;
__global__ void __launch_bounds__(kAppendThreads) append_reserve_kernel(AppendArgs A, int n_wg, int heads_per_wg,
                                                                        int map_per_wg, int fused) {
  __shared__ int smem[kAppendThreads / 64 + 1];
  __shared__ int req0[kAppendWgs + 1], free0[kAppendWgs + 1];
  __shared__ int bits_s, free_s, last_s, ok_s;
  const Dims& D = A.D;
  const int tid = threadIdx.x, w = blockIdx.x;
  const bool wide = ((uintptr_t)A.free_map & 15) == 0;   // (map_per_wg is a multiple of 16)
  if (tid == 0) { bits_s = 0; free_s = 0; }
  __syncthreads();
  // requesters of this share, listed in ascending order
  const int i0 = w * heads_per_wg, i1 = min(A.nsel, i0 + heads_per_wg);
  int n_req = 0;
  for (int base = i0; base < i1; base += kAppendThreads) {
    const int idx = base + tid;
    int g = 0, want = 0;
    if (idx < i1) {
      g = append_head(A, idx);
      const int C = A.ctx[g];
      if ((C & (D.b - 1)) == 0) {
        const int u = C >> A.lb;
        if (u >= D.maxb) { want = 1; atomicOr(&bits_s, EB_TABLE); }
        else want = A.table[(size_t)g * D.maxb + u] < 0;
      }
    }
    int tot;
    const int ex = block_exclusive_scan<kAppendThreads>(want, smem, &tot);
    if (want) publish_i32(&A.list[i0 + n_req + ex], g);
    n_req += tot;
  }
  // free blocks of this share of the map (a single workgroup counts them only when they are wanted)
  const size_t m0 = (size_t)w * map_per_wg, m1 = min((size_t)D.N, m0 + map_per_wg);
  if (n_wg > 1 || n_req) {
    int s = 0;
    for (size_t at = m0 + (size_t)tid * 16; at < m1; at += (size_t)kAppendThreads * 16) {
      const uint4 v = free_bytes16(A.free_map, at, m1, wide);
      s += __popc(nonzero_bytes(v.x)) + __popc(nonzero_bytes(v.y)) + __popc(nonzero_bytes(v.z)) + __popc(nonzero_bytes(v.w));
    }
    s = wave_sum_i(s);
    if ((tid & 63) == 0 && s) atomicAdd(&free_s, s);
  }
  publish_wait();      // this thread's part of the list is out
  __syncthreads();
  if (tid == 0) {
    bool last = true;
    if (n_wg > 1) {
      publish_i32(&A.part[3 * w], n_req);
      publish_i32(&A.part[3 * w + 1], free_s);
      publish_i32(&A.part[3 * w + 2], bits_s);
      publish_wait();
      last = __hip_atomic_fetch_add(&A.header[HW_ARRIVED], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == n_wg - 1;
    }
    last_s = last;
  }
  __syncthreads();
  if (!last_s) return;
  // ---- the last workgroup ----
  if (tid < 64) {
    int r = 0, f = 0, bits = 0;
    if (n_wg == 1) {
      if (tid == 0) { r = n_req; f = free_s; bits = bits_s; }
    } else if (tid < n_wg) {
      r = published_i32(&A.part[3 * tid]);
      f = published_i32(&A.part[3 * tid + 1]);
      bits = published_i32(&A.part[3 * tid + 2]);
    }
    int ri = r, fi = f;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int a = __shfl_up(ri, o), c = __shfl_up(fi, o);
      if (tid >= o) { ri += a; fi += c; }
    }
    req0[tid] = ri - r;
    free0[tid] = fi - f;
    const bool table_full = __any(bits & EB_TABLE);
    if (tid == 63) {
      req0[64] = ri;
      free0[64] = fi;
      if (n_wg > 1) A.header[HW_ARRIVED] = 0;
      int st = A.header[HW_STATUS];
      if (st == KVC_OK) {
        st = table_full ? KVC_ERR_TABLE_FULL : ri > fi ? KVC_ERR_OOM : KVC_OK;
        if (st != KVC_OK) A.header[HW_STATUS] = st;
      }
      ok_s = st == KVC_OK;
    }
  }
  __syncthreads();
  if (!ok_s) return;
  const int total = req0[64];
  for (int w2 = 0; w2 < n_wg && free0[w2] < total; ++w2) {
    if (free0[w2 + 1] == free0[w2]) continue;   // nothing free in this share (the same for every thread)
    const size_t a0 = (size_t)w2 * map_per_wg, a1 = min((size_t)D.N, a0 + map_per_wg);
    int rank0 = free0[w2];
    for (size_t base = a0; base < a1 && rank0 < total; base += (size_t)kAppendThreads * 16) {
      const size_t at = base + (size_t)tid * 16;
      uint4 v = make_uint4(0, 0, 0, 0);
      if (at < a1) v = free_bytes16(A.free_map, at, a1, wide);
      uint32_t m[4] = {nonzero_bytes(v.x), nonzero_bytes(v.y), nonzero_bytes(v.z), nonzero_bytes(v.w)};
      int tot;
      int k = rank0 + block_exclusive_scan<kAppendThreads>(__popc(m[0]) + __popc(m[1]) + __popc(m[2]) + __popc(m[3]), smem, &tot);
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        while (m[q] && k < total) {
          const int id = (int)at + 4 * q + (__builtin_ctz(m[q]) >> 3);
          m[q] &= m[q] - 1;
          int lo = 0, hi = 64;   // share that holds the k-th requester
          while (hi - lo > 1) { const int mid = (lo + hi) >> 1; if (req0[mid] <= k) lo = mid; else hi = mid; }
          const int g = published_i32(&A.list[lo * heads_per_wg + (k - req0[lo])]);
          A.table[(size_t)g * D.maxb + (A.ctx[g] >> A.lb)] = id;
          A.free_map[id] = 0;
          ++k;
        }
      }
      rank0 += tot;
    }
  }
  if (!fused) return;
  __syncthreads();   // the table cells written above are read below, by this workgroup
  const int groups = kAppendThreads / A.lanes_per_head;
  for (int idx = tid / A.lanes_per_head; idx < A.nsel; idx += groups) append_one(A, idx, tid % A.lanes_per_head);
}

// The append of many heads, as a launch of its own: as many lanes per head as the new key and
// value have 16-byte pieces (rounded up to a power of two, at most a wavefront; 32 for 256-byte
// rows).  A chain of three dependent loads per head, so heads in flight are what counts.
__global__ void __launch_bounds__(256) append_write_kernel(AppendArgs A) {
  if (A.header[HW_STATUS] != KVC_OK) return;
  const int idx = blockIdx.x * (256 / A.lanes_per_head) + threadIdx.x / A.lanes_per_head;
  if (idx < A.nsel) append_one(A, idx, threadIdx.x % A.lanes_per_head);
}

// Count, rank the free map, resolve errors, hand out (n: see AllocMode).
static int alloc_common(const Dims& D, const kvc_state* st, const Workspace& W, const int32_t* n,
                        int mode, hipStream_t s) {
  const int gb = (D.G + 255) / 256;
  const int ntiles = (D.N + kScanTile - 1) / kScanTile;
  hipLaunchKernelGGL(count_and_free_tiles_kernel, dim3(gb + ntiles), dim3(256), 0, s, D, st->block_table,
                     st->ctx_len, n, mode, gb, st->free_map, W.held, W.off_b, W.tile_sums, W.header);
  KVC_LAUNCH_CHECK();
  hipLaunchKernelGGL(alloc_scan_kernel, dim3(1), dim3(1024), 0, s, D, W.off_b, W.off_a, W.tile_sums,
                     ntiles, W.header);
  KVC_LAUNCH_CHECK();
  hipLaunchKernelGGL(pick_scatter_kernel, dim3(ntiles), dim3(kScanThreads), 0, s, D, st->block_table,
                     st->free_map, W.tile_sums, W.held, W.off_a, mode == ALLOC_PREFILL ? n : (const int32_t*)nullptr,
                     st->ctx_len, W.header);
  KVC_LAUNCH_CHECK();
  return KVC_OK;
}

// ---- scheduling helpers: counts per sequence, prefill allocation, preemption --------------

// needed[s] = blocks sequence s must get before its next decode step (head instances of the
// chosen layers whose blocks are all full); held[s] = blocks it holds over all layers.
__global__ void __launch_bounds__(256) count_blocks_kernel(Dims D, const int32_t* __restrict__ table,
                                                           const int32_t* __restrict__ ctx, int l0, int l1,
                                                           int32_t* __restrict__ needed,
                                                           int32_t* __restrict__ held_out) {
  const int g = blockIdx.x * 256 + threadIdx.x;
  const bool in = g < D.G;
  const int gg = in ? g : D.G - 1;
  const int s = gg / (D.Lyr * D.Hk), l = (gg / D.Hk) % D.Lyr;
  const int C = ctx[gg];
  const int h = held_blocks(table + (size_t)gg * D.maxb, C, D.b, D.maxb);
  int need = in && l >= l0 && l < l1 && C == h * D.b;
  int hh = in ? h : 0;
  // one atomic per wavefront when all its lanes belong to one sequence
  const int s0 = __builtin_amdgcn_readfirstlane(s);
  if (__all(s == s0)) {
    need = wave_sum_i(need);
    hh = wave_sum_i(hh);
    if ((threadIdx.x & 63) == 0) {
      if (needed && need) atomicAdd(&needed[s0], need);
      if (held_out && hh) atomicAdd(&held_out[s0], hh);
    }
  } else if (in) {
    if (needed && need) atomicAdd(&needed[s], need);
    if (held_out && hh) atomicAdd(&held_out[s], hh);
  }
}

// The batch of a compression round, one workgroup.  Rank of every running sequence in the order
// (time of last compression, never = first; then index) by counting, the order written out,
// a 64-bit running total of allocated KVs along it, and the cut at the first sequence that does
// not fit.  held[s] = blocks the sequence holds (from count_blocks_kernel); order: S ints.
__global__ void __launch_bounds__(1024) compression_batch_kernel(int S, int b, const int32_t* __restrict__ held,
                                                                 const int64_t* __restrict__ last,
                                                                 const uint8_t* __restrict__ running,
                                                                 long long limit, int32_t* __restrict__ order,
                                                                 uint8_t* __restrict__ in_batch,
                                                                 int64_t* __restrict__ batch_kvs) {
  __shared__ long long wave_tot[1024 / 64];
  __shared__ long long carry_s, total_s;
  __shared__ int cut_s, nrun_s;
  const int tid = threadIdx.x;
  if (tid == 0) { carry_s = 0; total_s = 0; cut_s = 0x7fffffff; nrun_s = 0; }
  __syncthreads();
  auto key = [&](int s) -> long long { const long long t = last[s]; return t < 0 ? -1 : t; };
  auto runs = [&](int s) -> bool { return running == nullptr || running[s] != 0; };
  for (int s = tid; s < S; s += 1024) {
    in_batch[s] = 0;
    if (!runs(s)) continue;
    const long long ks = key(s);
    int rank = 0;
    for (int t = 0; t < S; ++t) {
      if (!runs(t)) continue;
      const long long kt = key(t);
      rank += (kt < ks) || (kt == ks && t < s);
    }
    order[rank] = s;
    atomicAdd(&nrun_s, 1);
  }
  __syncthreads();   // the order is complete (global writes of this workgroup are visible to it)
  const int nrun = nrun_s;
  for (int base = 0; base < nrun; base += 1024) {
    const int p = base + tid;
    const int s = p < nrun ? order[p] : -1;
    const long long v = s >= 0 ? (long long)held[s] * b : 0;
    long long inc = v;   // inclusive scan over the wavefront
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const long long t = __shfl_up(inc, o);
      if ((tid & 63) >= o) inc += t;
    }
    if ((tid & 63) == 63) wave_tot[tid >> 6] = inc;
    __syncthreads();
    long long before = carry_s;
    for (int w = 0; w < (tid >> 6); ++w) before += wave_tot[w];
    const long long cum = before + inc;
    if (s >= 0 && cum > limit) atomicMin(&cut_s, p);
    __syncthreads();
    if (tid == 1023) carry_s = cum;
    __syncthreads();
    // positions before the cut of this or an earlier tile are in; a cut found in this tile is final
    const int cut = cut_s;
    if (s >= 0 && p < cut) in_batch[s] = 1;
    // the last position taken so far, if it lies in this tile, knows the batch's total
    const int last_in = min(min(cut, nrun), base + 1024) - 1;
    if (p == last_in && last_in >= base) total_s = cum;
    __syncthreads();
    if (cut != 0x7fffffff) break;
  }
  __syncthreads();
  if (tid == 0 && batch_kvs) *batch_kvs = total_s;
}

// One wavefront per head instance of a preempted sequence, kPreemptHeads of them per workgroup
// one after the other (the workgroup adds what it freed to the counter once: adds to one word run
// one after the other over the whole chip).  A row is a run of ids followed by -1s: 64 cells at a
// time until the run ends.  (One thread per head walked its row alone: 73 us for 256 heads of
// 128 blocks.)
constexpr int kPreemptHeads = 16;
__global__ void __launch_bounds__(256) preempt_kernel(Dims D, int32_t* __restrict__ table,
                                                      int32_t* __restrict__ ctx, uint8_t* __restrict__ free_map,
                                                      const uint8_t* __restrict__ seq_mask,
                                                      int32_t* __restrict__ header) {
  __shared__ int freed[4];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  int n = 0;   // blocks this wavefront freed: the same in every lane
  for (int i = wv; i < kPreemptHeads; i += 4) {
    const int g = blockIdx.x * kPreemptHeads + i;
    if (g >= D.G || !seq_mask[g / (D.Lyr * D.Hk)]) continue;
    int32_t* row = table + (size_t)g * D.maxb;
    for (int base = 0; base < D.maxb; base += 64) {
      const int u = base + lane;
      const int id = u < D.maxb ? row[u] : -1;
      if (id >= 0) { free_map[id] = 1; row[u] = -1; }
      const int run = __popcll(__ballot(id >= 0));
      n += run;
      if (run < 64) break;
    }
    if (lane == 0) ctx[g] = 0;
  }
  if (lane == 0) freed[wv] = n;
  __syncthreads();
  if (threadIdx.x == 0) {
    const int t = freed[0] + freed[1] + freed[2] + freed[3];
    if (t) atomicAdd(&header[HW_FREED], t);
  }
}

// State check.  One wavefront per head instance walks its table row: ids in [0, N) as a prefix,
// -1 after it, the length within what the prefix holds; every held block counted once in
// `owner` (zeroed before the launch) and not marked free.
__global__ void __launch_bounds__(256) check_state_kernel(Dims D, const int32_t* __restrict__ table,
                                                          const int32_t* __restrict__ ctx,
                                                          const uint8_t* __restrict__ free_map,
                                                          int32_t* __restrict__ owner,
                                                          int32_t* __restrict__ header) {
  const int g = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (g >= D.G) return;
  const int lane = threadIdx.x & 63;
  const int32_t* row = table + (size_t)g * D.maxb;
  bool bad = false;
  int held = 0;
  bool ended = false;   // a -1 has been seen (the same in every lane)
  for (int base = 0; base < D.maxb; base += 64) {
    const int u = base + lane;
    const int id = u < D.maxb ? row[u] : -1;
    const bool holds = id != -1;
    if (holds) {
      if (id < 0 || id >= D.N) bad = true;
      else {
        if (atomicAdd(&owner[id], 1) != 0) bad = true;   // held twice
        if (free_map[id] != 0) bad = true;               // held and marked free
      }
    }
    const unsigned long long m = __ballot(holds);
    const int run = m == ~0ull ? 64 : __ffsll((long long)~m) - 1;   // ids at the front of these 64 cells
    if (ended ? m != 0 : (run < 64 && (m >> run) != 0)) bad = true;   // an id behind a -1
    if (!ended) held += run;
    if (run < 64) ended = true;
  }
  const int C = ctx[g];
  if (C < 0 || (long long)C > (long long)held * D.b) bad = true;
  if (__any(bad) && lane == 0) atomicOr(&header[HW_SCRATCH0], EB_ARG);
}

}  // namespace kvc

using namespace kvc;

extern "C" {

int kvc_check_state(const kvc_config* cfg, const kvc_state* st, void* ws, void* stream, int flags) {
  int rc = validate(cfg, st);
  if (rc != KVC_OK) return rc;
  if (!ws || ((uintptr_t)ws & 255)) return KVC_ERR_ARG;
  Dims D = dims_of(cfg);
  Workspace W = carve(D, ws);
  hipStream_t s = (hipStream_t)stream;
  int32_t* owner = (int32_t*)W.stash;   // [N] fits where the decode keeps N * b * r floats
  hipLaunchKernelGGL(zero_words_kernel, dim3((D.N + 255) / 256), dim3(256), 0, s, owner, D.N);
  KVC_LAUNCH_CHECK();
  hipLaunchKernelGGL(check_state_kernel, dim3((D.G + 3) / 4), dim3(256), 0, s, D, st->block_table, st->ctx_len,
                     st->free_map, owner, W.header);
  KVC_LAUNCH_CHECK();
  hipLaunchKernelGGL(resolve_kernel, dim3(1), dim3(64), 0, s, W.header, 0);
  KVC_LAUNCH_CHECK();
  return (flags & KVC_ASYNC) ? KVC_OK : finish_sync(W, s);
}

int kvc_block_alloc(const kvc_config* cfg, const kvc_state* st, const int32_t* n_new, void* ws,
                    void* stream, int flags) {
  int rc = validate(cfg, st);
  if (rc != KVC_OK) return rc;
  if (!n_new || !ws || ((uintptr_t)ws & 255)) return KVC_ERR_ARG;
  Dims D = dims_of(cfg);
  Workspace W = carve(D, ws);
  hipStream_t s = (hipStream_t)stream;
  rc = alloc_common(D, st, W, n_new, ALLOC_COUNTS, s);
  if (rc != KVC_OK) return rc;
  return (flags & KVC_ASYNC) ? KVC_OK : finish_sync(W, s);
}

int kvc_block_free(const kvc_config* cfg, const kvc_state* st, const int32_t* n_drop,
                   int64_t* blocks_freed, void* ws, void* stream, int flags) {
  int rc = validate(cfg, st);
  if (rc != KVC_OK) return rc;
  if (!n_drop || !ws || ((uintptr_t)ws & 255)) return KVC_ERR_ARG;
  Dims D = dims_of(cfg);
  Workspace W = carve(D, ws);
  hipStream_t s = (hipStream_t)stream;
  const int gb = (D.G + 255) / 256;
  hipLaunchKernelGGL(zero_words_kernel, dim3(1), dim3(64), 0, s, W.header + HW_FREED, 1);
  KVC_LAUNCH_CHECK();
  hipLaunchKernelGGL(count_drop_kernel, dim3(gb), dim3(256), 0, s, D, st->block_table, st->ctx_len, n_drop,
                     W.held, W.off_b, W.header);
  KVC_LAUNCH_CHECK();
  hipLaunchKernelGGL(resolve_kernel, dim3(1), dim3(64), 0, s, W.header, 0);
  KVC_LAUNCH_CHECK();
  hipLaunchKernelGGL(drop_kernel, dim3(gb), dim3(256), 0, s, D, st->block_table, st->ctx_len,
                     st->free_map, W.held, W.off_b, W.header);
  KVC_LAUNCH_CHECK();
  if (flags & KVC_ASYNC) return KVC_OK;
  rc = finish_sync(W, s);
  if (rc != KVC_OK) return rc;
  if (blocks_freed) {
    int32_t f = 0;
    rc = read_words(W.header + HW_FREED, &f, 1, s);
    if (rc != KVC_OK) return rc;
    *blocks_freed = f;
  }
  return KVC_OK;
}

int kvc_append(const kvc_config* cfg, const kvc_state* st, const void* k_new, const void* v_new,
               const int32_t* new_pos, int layer_begin, int layer_end, void* ws, void* stream,
               int flags) {
  int rc = validate(cfg, st);
  if (rc != KVC_OK) return rc;
  if (!k_new || !v_new || !ws || ((uintptr_t)ws & 255)) return KVC_ERR_ARG;
  if (((uintptr_t)k_new | (uintptr_t)v_new) & 15) return KVC_ERR_ARG;
  Dims D = dims_of(cfg);
  if (layer_begin < 0 || layer_end > D.Lyr || layer_begin >= layer_end) return KVC_ERR_ARG;
  Workspace W = carve(D, ws);
  hipStream_t s = (hipStream_t)stream;
  AppendArgs A;
  A.D = D;
  A.l0 = layer_begin; A.nl = layer_end - layer_begin; A.nsel = D.S * A.nl * D.Hk;
  A.lanes_per_head = 8;   // 2 * pieces rounded up to a power of two, within [8, 64]
  while (A.lanes_per_head < 64 && A.lanes_per_head < 2 * (D.d * kv_esz(D.dtype) / 16)) A.lanes_per_head *= 2;
  A.lb = 0;
  while ((1 << A.lb) < D.b) ++A.lb;
  A.kc = (char*)st->k_cache; A.vc = (char*)st->v_cache; A.metric = st->metric; A.pos = st->pos;
  A.table = st->block_table; A.ctx = st->ctx_len; A.free_map = st->free_map;
  A.k_new = (const char*)k_new; A.v_new = (const char*)v_new; A.new_pos = new_pos;
  A.header = W.header; A.part = W.seg_hist; A.list = W.off_b;
  // a workgroup per 1024 heads or 16 KB of the map, whichever asks for more, at most kAppendWgs
  const int by_heads = (A.nsel + kAppendThreads - 1) / kAppendThreads;
  const int by_map = (int)(((size_t)D.N + 16 * kAppendThreads - 1) / (16 * kAppendThreads));
  int n_wg = by_heads > by_map ? by_heads : by_map;
  if (n_wg > kAppendWgs) n_wg = kAppendWgs;
  const int heads_per_wg = (A.nsel + n_wg - 1) / n_wg;
  const int map_per_wg = (int)(align_up(((size_t)D.N + n_wg - 1) / n_wg, 16));
  static_assert(kAppendWgs * 3 <= 256, "the counts fit one segment's histogram");
  const int fused = A.nsel <= kAppendFused;
  hipLaunchKernelGGL(append_reserve_kernel, dim3(n_wg), dim3(kAppendThreads), 0, s, A, n_wg, heads_per_wg, map_per_wg, fused);
  KVC_LAUNCH_CHECK();
  if (!fused) {
    const int heads_per_launch_wg = 256 / A.lanes_per_head;
    hipLaunchKernelGGL(append_write_kernel, dim3((A.nsel + heads_per_launch_wg - 1) / heads_per_launch_wg), dim3(256), 0, s, A);
    KVC_LAUNCH_CHECK();
  }
  return (flags & KVC_ASYNC) ? KVC_OK : finish_sync(W, s);
}

int kvc_count_blocks(const kvc_config* cfg, const kvc_state* st, int layer_begin, int layer_end,
                     int32_t* needed, int32_t* held, void* ws, void* stream) {
  int rc = validate(cfg, st);
  if (rc != KVC_OK) return rc;
  (void)ws;
  Dims D = dims_of(cfg);
  if (layer_begin < 0 || layer_end > D.Lyr || layer_begin >= layer_end) return KVC_ERR_ARG;
  if (!needed && !held) return KVC_ERR_ARG;
  hipStream_t s = (hipStream_t)stream;
  if (needed) { hipLaunchKernelGGL(zero_words_kernel, dim3((D.S + 63) / 64), dim3(64), 0, s, needed, D.S); KVC_LAUNCH_CHECK(); }
  if (held) { hipLaunchKernelGGL(zero_words_kernel, dim3((D.S + 63) / 64), dim3(64), 0, s, held, D.S); KVC_LAUNCH_CHECK(); }
  hipLaunchKernelGGL(count_blocks_kernel, dim3((D.G + 255) / 256), dim3(256), 0, s, D, st->block_table, st->ctx_len,
                     layer_begin, layer_end, needed, held);
  KVC_LAUNCH_CHECK();
  return KVC_OK;
}

int kvc_compression_batch(const kvc_config* cfg, const kvc_state* st, const int64_t* last_compressed,
                          const uint8_t* running, int64_t kv_limit, uint8_t* in_batch, int64_t* batch_kvs,
                          void* ws, void* stream) {
  int rc = validate(cfg, st);
  if (rc != KVC_OK) return rc;
  if (!last_compressed || !in_batch || !ws || ((uintptr_t)ws & 255) || kv_limit < 0) return KVC_ERR_ARG;
  if (((uintptr_t)last_compressed & 7) || (batch_kvs && ((uintptr_t)batch_kvs & 7))) return KVC_ERR_ARG;
  Dims D = dims_of(cfg);
  if (D.S > 8192) return KVC_ERR_UNSUPPORTED;   // ranks are found by counting, S^2 comparisons in one workgroup
  Workspace W = carve(D, ws);
  hipStream_t s = (hipStream_t)stream;
  int32_t* held = W.off_b;    // [S] fits in the [G + 1] array
  int32_t* order = W.off_a;
  hipLaunchKernelGGL(zero_words_kernel, dim3((D.S + 63) / 64), dim3(64), 0, s, held, D.S);
  KVC_LAUNCH_CHECK();
  hipLaunchKernelGGL(count_blocks_kernel, dim3((D.G + 255) / 256), dim3(256), 0, s, D, st->block_table, st->ctx_len,
                     0, D.Lyr, (int32_t*)nullptr, held);
  KVC_LAUNCH_CHECK();
  hipLaunchKernelGGL(compression_batch_kernel, dim3(1), dim3(1024), 0, s, D.S, D.b, held, last_compressed, running,
                     (long long)kv_limit, order, in_batch, batch_kvs);
  KVC_LAUNCH_CHECK();
  return KVC_OK;
}

int kvc_prefill_alloc(const kvc_config* cfg, const kvc_state* st, const int32_t* seq_tokens, void* ws,
                      void* stream, int flags) {
  int rc = validate(cfg, st);
  if (rc != KVC_OK) return rc;
  if (!seq_tokens || !ws || ((uintptr_t)ws & 255)) return KVC_ERR_ARG;
  Dims D = dims_of(cfg);
  Workspace W = carve(D, ws);
  hipStream_t s = (hipStream_t)stream;
  rc = alloc_common(D, st, W, seq_tokens, ALLOC_PREFILL, s);
  if (rc != KVC_OK) return rc;
  return (flags & KVC_ASYNC) ? KVC_OK : finish_sync(W, s);
}

int kvc_preempt(const kvc_config* cfg, const kvc_state* st, const uint8_t* seq_mask, int64_t* blocks_freed,
                void* ws, void* stream, int flags) {
  int rc = validate(cfg, st);
  if (rc != KVC_OK) return rc;
  if (!seq_mask || !ws || ((uintptr_t)ws & 255)) return KVC_ERR_ARG;
  Dims D = dims_of(cfg);
  Workspace W = carve(D, ws);
  hipStream_t s = (hipStream_t)stream;
  hipLaunchKernelGGL(zero_words_kernel, dim3(1), dim3(64), 0, s, W.header + HW_FREED, 1);
  KVC_LAUNCH_CHECK();
  hipLaunchKernelGGL(preempt_kernel, dim3((D.G + kPreemptHeads - 1) / kPreemptHeads), dim3(256), 0, s, D, st->block_table, st->ctx_len,
                     st->free_map, seq_mask, W.header);
  KVC_LAUNCH_CHECK();
  if ((flags & KVC_ASYNC) || !blocks_freed) return KVC_OK;
  int32_t f = 0;
  rc = read_words(W.header + HW_FREED, &f, 1, s);
  if (rc != KVC_OK) return rc;
  *blocks_freed = f;
  return KVC_OK;
}

}  // extern "C"
