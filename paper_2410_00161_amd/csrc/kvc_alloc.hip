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
// scan joins the runs.  out[i] = exclusive prefix (out may be `in`).  owner (or NULL): owner[out[i]] = i
// for every element that is not zero.
__device__ __forceinline__ int wide_exclusive_scan(const int32_t* in, int n, int32_t* out, int* smem,
                                                   int32_t* owner = nullptr, int owner_n = 0) {
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
    if (owner) {
#pragma unroll
      for (int k = 0; k < kScanRun; ++k)
        if (v[k] && (unsigned)o[k] < (unsigned)owner_n) owner[o[k]] = first + k;
    }
    __syncthreads();
    if (threadIdx.x == 0) carry_s += tot;
    __syncthreads();
  }
  return carry_s;
}

// Launch 2, one workgroup: exclusive scan of the requests (off[g], off[G] = total) with the owner of
// every head's first request (owner[off[g]] = g), exclusive scan of the free-tile counts, and the status
// word.
__global__ void __launch_bounds__(1024) alloc_scan_kernel(Dims D, const int32_t* __restrict__ req,
                                                          int32_t* __restrict__ off,
                                                          int32_t* __restrict__ owner,
                                                          int32_t* __restrict__ tile_sums, int ntiles,
                                                          int32_t* __restrict__ header) {
  __shared__ int smem[1024 / 64 + 1];
  const int total_req = wide_exclusive_scan(req, D.G, off, smem, owner, D.N);
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

// Last head instance of [lo, hi) with off[g] <= k (off[lo] <= k), by all lanes of a wavefront.
__device__ __forceinline__ int wave_find_head(const int32_t* off, int lo, int hi, int k, int lane) {
  while (hi - lo > 1) {
    const int step = (int)(((long long)hi - lo + 63) / 64);
    const long long at = (long long)lo + (long long)lane * step;
    const int below = __popcll(__ballot(at < hi && off[at < hi ? at : lo] <= k));   // the first lanes
    lo += (below - 1) * step;
    hi = hi - lo < step ? hi : lo + step;
  }
  return lo;
}

// Third phase of the scan over the free map, fused with the hand-out: the free block of
// rank k (ascending id) goes to the head instance g with off[g] <= k < off[g + 1], as its
// (k - off[g])-th new block.  A rank that starts a head finds it in the list (an entry counts when its
// head starts there, so nothing has to be cleared); every other rank goes where the one before it
// went, whichever thread has that, and the workgroup's first one is searched for.  (All owners in the
// list were one thread's serial run per head, without a list every thread searched for every head.
// Whole call, all owners listed, searched, and this way: 16 384 heads, 1000 of them asking for a block
// 23, 43 and 22 us, for one each 28, 35 and 28, for up to eight 52, 36 and 28; 2560 heads, five each 26, 30
// and 20; 64 prompts of 7000 tokens in 32 layers of 8 heads 3776, 57 and 64.)
// seq_tokens (a prefill): the lengths of the heads follow in the same launch.
__global__ void __launch_bounds__(kScanThreads) pick_scatter_kernel(Dims D, int32_t* __restrict__ table,
                                                                    uint8_t* __restrict__ free_map,
                                                                    const int32_t* __restrict__ tile_sums,
                                                                    const int32_t* __restrict__ held,
                                                                    const int32_t* __restrict__ off,
                                                                    const int32_t* __restrict__ owner,
                                                                    const int32_t* __restrict__ seq_tokens,
                                                                    int32_t* __restrict__ ctx,
                                                                    const int32_t* __restrict__ header) {
  __shared__ int smem[kScanThreads / 64 + 1];
  __shared__ int head_s[kScanThreads / 64 + 1];   // last head that starts in every wavefront's ranks; [4]: the first rank's
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
  if (((uintptr_t)free_map & 7) == 0 && base + kScanItems <= D.N) {   // (a load of eight bytes, not eight)
    const uint2 m = *(const uint2*)(free_map + base);
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) { v[k] = ((k < 4 ? m.x : m.y) >> (8 * (k & 3)) & 0xff) != 0; s += v[k]; }
  } else {
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) { v[k] = (base + k < D.N) ? (free_map[base + k] != 0) : 0; s += v[k]; }
  }
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  if (wv == 0) {
    const int ga = tile0 > 0 ? wave_find_head(off, 0, D.G, tile0, lane) : 0;   // (rank 0 starts a head: nothing goes by this one)
    if (lane == 0) head_s[kScanThreads / 64] = ga;
  }
  int ex = block_exclusive_scan<kScanThreads>(s, smem, nullptr) + tile0;
  int own[kScanItems], own_first[kScanItems], own_end[kScanItems], own_held[kScanItems];   // asked for together
  int e = ex;
#pragma unroll
  for (int k = 0; k < kScanItems; ++k) {
    own[k] = v[k] && e < total_req ? owner[e] : -1;
    if ((unsigned)own[k] >= (unsigned)D.G) own[k] = -1;
    e += v[k];
  }
#pragma unroll
  for (int k = 0; k < kScanItems; ++k) {
    own_first[k] = own[k] >= 0 ? off[own[k]] : -1;
    own_end[k] = own[k] >= 0 ? off[own[k] + 1] : 0;
    own_held[k] = own[k] >= 0 ? held[own[k]] : 0;
  }
  int last = -1;   // last head that starts in this thread's ranks
  e = ex;
#pragma unroll
  for (int k = 0; k < kScanItems; ++k) {
    if (own_first[k] != e || own_end[k] <= e) own[k] = -1;
    if (own[k] >= 0) last = own[k];
    e += v[k];
  }
  const unsigned long long starts = __ballot(last >= 0);
  const unsigned long long ahead = starts & ((1ull << lane) - 1);
  int g = __shfl(last, ahead ? 63 - __builtin_clzll(ahead) : 0);   // head in hand: of the rank before this thread's first
  if (!ahead) g = -1;
  const int wave_last = __shfl(last, starts ? 63 - __builtin_clzll(starts) : 0);
  if (lane == 0) head_s[wv] = starts ? wave_last : -1;
  __syncthreads();
  if (g < 0) {
    g = head_s[kScanThreads / 64];
    for (int w = 0; w < wv; ++w) if (head_s[w] >= 0) g = head_s[w];
  }
  int first = off[g], had = held[g];
#pragma unroll
  for (int k = 0; k < kScanItems; ++k) {
    if (v[k]) {
      if (ex < total_req) {
        if (own[k] >= 0) { g = own[k]; first = own_first[k]; had = own_held[k]; }
        table[(size_t)g * D.maxb + had + (ex - first)] = base + k;
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
  int n_wg, heads_per_wg, map_per_wg;   // workgroups of the reservation, and their shares (map_per_wg in whole tiles)
  int32_t* part;           // [workgroups][3] requests, free blocks, error bits; then [2][kAppendWgs] requests, free blocks ahead of each
  int32_t* rank;           // [nsel] rank of a head's request among its workgroup's, -1 = none (many heads)
  uint32_t* bits;          // [tiles][32] the free map as it was, a bit per block
  int32_t* tile_free;      // [tiles] free blocks per tile
};
constexpr int kAppendTile = 1024;   // blocks per tile of the map: what a wavefront reads at a time

__device__ __forceinline__ int append_head(const AppendArgs& A, int idx) {
  const int s = idx / (A.nl * A.D.Hk);
  return (s * A.D.Lyr + A.l0 + (idx / A.D.Hk) % A.nl) * A.D.Hk + idx % A.D.Hk;
}

// Block that is free block number k of the map (k below the number of them), by all lanes of a
// wavefront: the share, the tile, the word and the bit that hold it.  ahead: free blocks ahead of
// share `lane`.  FRESH: what this launch's other workgroups left (else an earlier launch's).
template <bool FRESH>
__device__ __forceinline__ int nth_free_block(const AppendArgs& A, int ahead, int k, int lane) {
  auto get = [&](const int32_t* p) { return FRESH ? published_i32(p) : *p; };
  const int share = __popcll(__ballot(ahead <= k)) - 1;   // the last one: shares without a free block have the next one's number
  int rest = k - __builtin_amdgcn_readlane(ahead, share);
  const int per = A.map_per_wg / kAppendTile, n_tiles = (int)(((size_t)A.D.N + kAppendTile - 1) / kAppendTile);
  const int t1 = min(n_tiles, (share + 1) * per);
  int tile = share * per;
  for (;; tile += 64) {
    if (tile >= t1) return -1;   // (fewer free blocks than were counted: cannot be)
    const int c = tile + lane < t1 ? get(&A.tile_free[tile + lane]) : 0;
    const int inc = wave_prefix_i(c);
    const unsigned long long past = __ballot(inc > rest);
    if (past) {
      const int l = __builtin_ctzll(past);
      rest -= __builtin_amdgcn_readlane(inc - c, l);
      tile += l;
      break;
    }
    rest -= __builtin_amdgcn_readlane(inc, 63);
  }
  const uint32_t word = lane < 32 ? (uint32_t)get((const int32_t*)A.bits + (size_t)tile * 32 + lane) : 0;
  const int c = __popc(word), inc = wave_prefix_i(c);
  const unsigned long long past = __ballot(inc > rest);
  if (!past) return -1;
  const int l = __builtin_ctzll(past);
  rest -= __builtin_amdgcn_readlane(inc - c, l);
  uint32_t w = (uint32_t)__builtin_amdgcn_readlane((int)word, l);
  for (; rest > 0; --rest) w &= w - 1;
  return tile * kAppendTile + l * 32 + __builtin_ctz(w);
}

// The new token of head instance g, which holds C tokens, into block blk.
__device__ __forceinline__ void append_one(const AppendArgs& A, int g, int C, int blk, int gl) {
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
  uint64_t lo = 0, hi = 0;
#pragma unroll 1
  for (int k = 0; k < 16 && at + k < end; ++k) {   // (rare, and in every place that reads the map: kept short)
    const uint64_t byte = (uint64_t)map[at + k] << (8 * (k & 7));
    if (k < 8) lo |= byte; else hi |= byte;
  }
  return make_uint4((uint32_t)lo, (uint32_t)(lo >> 32), (uint32_t)hi, (uint32_t)(hi >> 32));
}

// The reservation of an append in one launch: which heads need a block (their length fills the
// blocks they hold), the lowest free blocks for them in ascending head order, the error checks before
// anything is written; for few heads also the append itself.
//
// Workgroup w of n looks at its share of the heads and of the free map, leaves the counts, the ranks
// of its requesters and its share of the map as bits with a count per tile, and announces itself; the
// last one to arrive reads all the counts (one wavefront: n <= 64) and settles the status.  Every
// requester then finds its own block (nth_free_block), in the launch that writes the rows, or here for
// few heads: wherever the free blocks lie, nobody walks the map for them.  In place of a launch each for
// counting, for a scan in one workgroup over all heads, and for a second walk over the whole map: a
// launch costs ~4.5 us in a busy stream whatever it does.  Replayed from a graph, four launches against
// this: 16 384 heads, 1.35 M blocks of which a fifth or a thousandth is free 24.1 and 20.4 -> 12.1 and
// 12.2 us (23.5 and 265 when the last workgroup walked the map for all requests); a layer of one
// sequence 11.6 -> 3.8 without a request, 14.7 -> 6.1 with one from every head.
constexpr int kAppendThreads = 1024;
// Heads appended by the same launch, a wavefront's lanes of them at most.  One CU finds their blocks
// sixteen at a time and writes all their rows; a launch for the rows costs more wherever few ask.
// Together and apart: 8 heads without a request 3.8 and 6.8 us, with one from every head 6.1 and 7.4;
// 56 heads of 12 000 blocks 3.9 and 5.0, with four requests 5.9 and 6.5; 64 heads of 170 000 blocks with
// four requests 8.8 and 7.8, with 64 11.1 and 8.8 (from a graph; issued by the host, the launch saved
// is worth more: three layers of 38 heads 9 us).
constexpr int kAppendFused = 64;
constexpr int kWaitLoads = 0x0f70;   // s_waitcnt vmcnt(0)
template <bool FUSED>
__global__ void __launch_bounds__(kAppendThreads) append_reserve_kernel(AppendArgs A) {
  __shared__ __align__(16) int asks_s[kAppendThreads / 64];
  __shared__ int bits_s, free_s, req_s, last_s, ok_s;
  __shared__ int want_g[kAppendFused], ahead_s[kAppendWgs];
  const Dims& D = A.D;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, w = blockIdx.x;
  const int n_wg = A.n_wg;
  const bool wide = ((uintptr_t)A.free_map & 15) == 0;   // (map_per_wg is a multiple of 16)
  auto wants = [&](int g, bool* full) {
    const int C = A.ctx[g], u = C >> A.lb;
    if (C & (D.b - 1)) return false;
    *full = u >= D.maxb;
    return *full || A.table[(size_t)g * D.maxb + u] < 0;
  };
  // this share of the map, a tile per wavefront and round, kRounds asked for together
  const size_t m0 = (size_t)w * A.map_per_wg, m1 = min((size_t)D.N, m0 + A.map_per_wg);
  constexpr int kRounds = 2;
  size_t tile0 = m0 + (size_t)wv * kAppendTile;
  uint4 v[kRounds];
  auto ask = [&]() {
#pragma unroll
    for (int u = 0; u < kRounds; ++u) {
      const size_t at = tile0 + (size_t)u * 16 * kAppendThreads + (size_t)lane * 16;
      v[u] = at < m1 ? free_bytes16(A.free_map, at, m1, wide) : make_uint4(0, 0, 0, 0);
    }
  };
  const bool early = !FUSED && n_wg > 1;
  if (early) ask();   // (it hangs on nothing; few heads, and small pools, often need no look at the map)
  if (tid == 0) { bits_s = 0; free_s = 0; }
  __syncthreads();
  // requesters, in ascending order: of this share of the heads; of all of few heads, in every
  // workgroup, so that without any nobody looks at the map
  int n_req = 0;
  if (FUSED) {
    if (wv == 0) {
      bool full = false;
      const int g = lane < A.nsel ? append_head(A, lane) : 0;
      const unsigned long long asks = __ballot(lane < A.nsel && wants(g, &full));
      if (asks >> lane & 1) want_g[__popcll(asks & ((1ull << lane) - 1))] = g;
      const bool any_full = __any(full);
      if (lane == 0) { req_s = __popcll(asks); bits_s = any_full ? EB_TABLE : 0; }
    }
    __syncthreads();
    n_req = req_s;
  } else {
    const int i0 = w * A.heads_per_wg, i1 = min(A.nsel, i0 + A.heads_per_wg);
    for (int base = i0; base < i1; base += kAppendThreads) {
      const int idx = base + tid;
      bool full = false;
      const int want = idx < i1 && wants(append_head(A, idx), &full);
      if (full) atomicOr(&bits_s, EB_TABLE);
      const unsigned long long asks = __ballot(want);
      if (base > i0) __syncthreads();   // the counts of the round before have been read
      if (lane == 0) asks_s[wv] = __popcll(asks);
      __syncthreads();
      int ahead = __popcll(asks & ((1ull << lane) - 1)), tot = 0;
#pragma unroll
      for (int k = 0; k < kAppendThreads / 64; ++k) {
        const int c = asks_s[k];
        if (k < wv) ahead += c;
        tot += c;
      }
      if (idx < i1) A.rank[idx] = want ? n_req + ahead : -1;
      n_req += tot;
    }
  }
  // its free blocks (a single workgroup counts them only when they are wanted)
  const bool alone = n_wg == 1, counted = n_req > 0 || (!FUSED && !alone);
  if (counted && !early) ask();
  // The loads are done (or there are none), in words the compiler counts by: it would wait for them
  // further down, and with them for the stores below.
  __builtin_amdgcn_s_waitcnt(kWaitLoads);
  if (counted) {
    int s = 0;
    while (tile0 < m1) {
#pragma unroll
      for (int u = 0; u < kRounds; ++u) {
        const size_t first = tile0 + (size_t)u * 16 * kAppendThreads;   // the tile's first block
        if (first >= m1) break;
        // a bit per byte: the top bits of a word's four bytes, brought together by a product
        auto four = [](uint32_t x) { return ((nonzero_bytes(x) >> 7) * 0x10204080u) >> 28; };
        const uint32_t mine = four(v[u].x) | four(v[u].y) << 4 | four(v[u].z) << 8 | four(v[u].w) << 12;
        const uint32_t pair = mine | (uint32_t)__builtin_amdgcn_update_dpp(0, (int)mine, 0xb1, 0xf, 0xf, false) << 16;
        const int n = wave_prefix_i(__popc(mine));   // lane 63: of the tile
        int32_t* word = (int32_t*)A.bits + first / 32 + (lane >> 1);
        int32_t* count = &A.tile_free[first / kAppendTile];
        if (FUSED) {   // read by this launch's last workgroup, else by the next launch
          if (!(lane & 1)) publish_i32(word, (int)pair);
          if (lane == 63) publish_i32(count, n);
        } else {
          if (!(lane & 1)) *word = (int)pair;
          if (lane == 63) *count = n;
        }
        s += n;
      }
      tile0 += (size_t)kRounds * 16 * kAppendThreads;
      if (tile0 >= m1) break;
      ask();
      __builtin_amdgcn_s_waitcnt(kWaitLoads);
    }
    if (lane == 63 && s) atomicAdd(&free_s, s);
    if (FUSED) publish_wait();   // what this thread left is out
  }
  __syncthreads();
  if (tid == 0) {
    bool last = true;
    if (!alone) {   // (all of them, also without a request: nothing is written while one may still look)
      if (counted) {
        publish_i32(&A.part[3 * w], n_req);
        publish_i32(&A.part[3 * w + 1], free_s);
        publish_i32(&A.part[3 * w + 2], bits_s);
        publish_wait();
      }
      last = __hip_atomic_fetch_add(&A.header[HW_ARRIVED], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == n_wg - 1;
    }
    last_s = last;
  }
  __syncthreads();
  if (!last_s) return;
  // ---- the last workgroup ----
  if (tid < 64) {
    int r = 0, f = 0, bits = 0, st = A.header[HW_STATUS];
    if (alone || !counted) {
      if (tid == 0) { r = n_req; f = free_s; bits = bits_s; }
    } else if (tid < n_wg) {
      r = published_i32(&A.part[3 * tid]);
      f = published_i32(&A.part[3 * tid + 1]);
      bits = published_i32(&A.part[3 * tid + 2]);
    }
    const int ri = wave_prefix_i(r), fi = wave_prefix_i(f);
    if (FUSED) ahead_s[tid] = fi - f;
    else { A.part[tid] = ri - r; A.part[kAppendWgs + tid] = fi - f; }   // (the counts have been read, by this wavefront)
    const bool table_full = __any(bits & EB_TABLE);
    if (tid == 63) {
      if (!alone) A.header[HW_ARRIVED] = 0;
      if (st == KVC_OK) {
        st = table_full ? KVC_ERR_TABLE_FULL : (FUSED ? n_req : ri) > fi ? KVC_ERR_OOM : KVC_OK;
        if (st != KVC_OK) A.header[HW_STATUS] = st;
      }
      ok_s = st == KVC_OK;
    }
  }
  if (!FUSED) return;
  __syncthreads();
  if (!ok_s) return;
  // few heads: a wavefront per request, then the rows
  const int ahead = ahead_s[lane];
  for (int k = wv; k < n_req; k += kAppendThreads / 64) {
    const int g = want_g[k];
    const int id = nth_free_block<true>(A, ahead, k, lane);
    if (lane == 0 && id >= 0) {
      A.table[(size_t)g * D.maxb + (A.ctx[g] >> A.lb)] = id;
      A.free_map[id] = 0;
    }
  }
  __syncthreads();   // the table cells written above are read below, by this workgroup
  const int groups = kAppendThreads / A.lanes_per_head;
  for (int idx = tid / A.lanes_per_head; idx < A.nsel; idx += groups) {
    const int g = append_head(A, idx), C = A.ctx[g];
    const int blk = A.table[(size_t)g * D.maxb + (C >> A.lb)];
    if (blk >= 0) append_one(A, g, C, blk, tid % A.lanes_per_head);
  }
}

// The append of many heads, as a launch of its own: as many lanes per head as the new key and
// value have 16-byte pieces (rounded up to a power of two, at most a wavefront; 32 for 256-byte
// rows).  A chain of three dependent loads per head, so heads in flight are what counts.  The requests
// of a wavefront's heads find their blocks first, one after the other.
__global__ void __launch_bounds__(256) append_write_kernel(AppendArgs A) {
  const int idx = blockIdx.x * (256 / A.lanes_per_head) + threadIdx.x / A.lanes_per_head;
  const int lane = threadIdx.x & 63, gl = threadIdx.x % A.lanes_per_head;
  const bool real = idx < A.nsel;
  // (everything that hangs on nothing else is asked for together)
  const int g = real ? append_head(A, idx) : 0;
  const int rank = real ? A.rank[idx] : -1, C = A.ctx[g];
  const int before = A.part[lane], ahead = A.part[kAppendWgs + lane];
  if (A.header[HW_STATUS] != KVC_OK) return;
  int32_t* cell = &A.table[(size_t)g * A.D.maxb + (C >> A.lb)];
  int blk = real && rank < 0 ? *cell : -1;
  for (unsigned long long asks = __ballot(gl == 0 && rank >= 0); asks; asks &= asks - 1) {
    const int src = __builtin_ctzll(asks);
    const int share = __builtin_amdgcn_readlane(idx, src) / A.heads_per_wg;
    const int k = __builtin_amdgcn_readlane(before, share) + __builtin_amdgcn_readlane(rank, src);
    const int id = nth_free_block<false>(A, ahead, k, lane);
    if (lane / A.lanes_per_head == src / A.lanes_per_head) blk = id;
  }
  if (blk < 0) return;
  if (gl == 0 && rank >= 0) { *cell = blk; A.free_map[blk] = 0; }
  append_one(A, g, C, blk, gl);
}

// Count, rank the free map, resolve errors, hand out (n: see AllocMode).
static int alloc_common(const Dims& D, const kvc_state* st, const Workspace& W, const int32_t* n,
                        int mode, hipStream_t s) {
  const int gb = (D.G + 255) / 256;
  const int ntiles = (D.N + kScanTile - 1) / kScanTile;
  int32_t* owner = (int32_t*)W.stash;   // [N] fits where the decode keeps N * b * r floats
  hipLaunchKernelGGL(count_and_free_tiles_kernel, dim3(gb + ntiles), dim3(256), 0, s, D, st->block_table,
                     st->ctx_len, n, mode, gb, st->free_map, W.held, W.off_b, W.tile_sums, W.header);
  KVC_LAUNCH_CHECK();
  hipLaunchKernelGGL(alloc_scan_kernel, dim3(1), dim3(1024), 0, s, D, W.off_b, W.off_a, owner, W.tile_sums,
                     ntiles, W.header);
  KVC_LAUNCH_CHECK();
  hipLaunchKernelGGL(pick_scatter_kernel, dim3(ntiles), dim3(kScanThreads), 0, s, D, st->block_table,
                     st->free_map, W.tile_sums, W.held, W.off_a, owner, mode == ALLOC_PREFILL ? n : (const int32_t*)nullptr,
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
  hipLaunchKernelGGL(resolve_kernel, dim3(1), dim3(64), 0, s, W.header);
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
  hipLaunchKernelGGL(resolve_kernel, dim3(1), dim3(64), 0, s, W.header);
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
  A.header = W.header; A.part = W.seg_hist; A.rank = W.off_b;
  // a workgroup per 1024 heads or 16 KB of the map, whichever asks for more, at most kAppendWgs
  const int by_heads = (A.nsel + kAppendThreads - 1) / kAppendThreads;
  const int by_map = (int)(((size_t)D.N + 16 * kAppendThreads - 1) / (16 * kAppendThreads));
  int n_wg = by_heads > by_map ? by_heads : by_map;
  if (n_wg > kAppendWgs) n_wg = kAppendWgs;
  A.n_wg = n_wg;
  A.heads_per_wg = (A.nsel + n_wg - 1) / n_wg;
  A.map_per_wg = (int)align_up(((size_t)D.N + n_wg - 1) / n_wg, kAppendTile);
  // [tiles][32] bits and [tiles] counts, 132 bytes per 1024 blocks, fit where the decode keeps N * b * r floats
  A.bits = (uint32_t*)W.stash;
  A.tile_free = (int32_t*)W.stash + ((size_t)D.N + kAppendTile - 1) / kAppendTile * 32;
  static_assert(kAppendWgs * 3 <= 256, "the counts fit one segment's histogram");
  if (A.nsel <= kAppendFused) {
    hipLaunchKernelGGL(append_reserve_kernel<true>, dim3(n_wg), dim3(kAppendThreads), 0, s, A);
    KVC_LAUNCH_CHECK();
  } else {
    hipLaunchKernelGGL(append_reserve_kernel<false>, dim3(n_wg), dim3(kAppendThreads), 0, s, A);
    KVC_LAUNCH_CHECK();
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
