// Work list shared by the kernels that walk every head instance in chunks of T tokens (the
// decode and the observation-window metric): item records built on the device from the
// context lengths, ordered by size class, plus the cross-lane helpers those kernels use.
#pragma once

#include "kvc_common.h"

namespace kvc {

struct DecodeItem {   // 32 bytes
  int g;        // head instance
  int t0;       // first token of the chunk
  int n_tok;    // tokens in the chunk
  int nch;      // chunks of the head
  int pbase;    // first partial-result slot of the head (heads of more than one chunk)
  int pad[3];   // [0]: the head's length the list was made for (lists kept by kvc_decode_plan); [1]: tokens of the head's
                // chunks but the last; [2]: where a chunk of a head that meets is called
};

struct DecodeArgs {
  Dims D;
  const char* kc;
  const char* vc;
  float* metric;
  const int32_t* table;
  const int32_t* ctx;
  const char* q;
  float* out;
  int l0, nl, gsel;       // first layer, layer count, head instances selected
  int accumulate, T;      // metric on/off, chunk tokens (the most a chunk may hold when adapt_T is set)
  int adapt_T;            // the one-launch work list picks the chunk length from the lengths it sees (see there)
  int log2b;              // block size is a power of two on the tiled path
  int cap;                // item records and partial-result slots the workspace holds
  int all_partials;       // give every head a partial-result slot range, not only split heads (else the chunks of a split
                          // head are listed side by side, its last and shorter one too: they meet, see kMeetBits)
  int rotate_chunks;      // a head's full chunks take their places rotated by the head's index (see decode_items_kernel)
  int short_class, Ts;    // size classes from short_class up (at most Ts tokens) are "short" items; 16 = none
  DecodeItem* items;
  int32_t* slot_word;     // a word per partial-result slot: those of a head's first two are where its chunks meet
  float* part_ml;
  float* part_acc;
  float* stash;
  int32_t* header;
  // Work lists kept from one launch for every layer (kvc_decode_plan): layer l has its own header
  // block at header + l * HW_WORDS and its own stretch of the records of items / slot_word.
  int plan;               // the work-list kernel runs one workgroup per layer; a decode reads one layer's list
  int plan_stride;        // records of a layer's stretch; 0: it starts where its header block says
  int plan_cap;           // records of all layers the workspace holds
  int self_list;          // no work list: every workgroup finds its own item from the lengths (at most kSelfListHeads heads)
  int ctx_plus;           // the plan is made for heads ctx_plus tokens longer than they are now
  int32_t* status;        // the workspace's own header (status word), whatever `header` points at
  float scale_log2;       // log2(e) / sqrt(d)
  // (at the end: in front of the others they moved these to other lines, and a layer's call took 0.2 us more)
  int packed;             // rows of fewer than kMeetMost chunks: a head's counts of chunks are halves of one word
  int places;             // workgroups of four wavefronts that the chip runs at once (where a list's chunks are to fit them)
};

__device__ __forceinline__ int sel_to_g(const Dims& D, int l0, int nl, int gi) {
  const int s = gi / (nl * D.Hk);
  const int l = l0 + (gi / D.Hk) % nl;
  const int h = gi % D.Hk;
  return (s * D.Lyr + l) * D.Hk + h;
}

// Work items are ordered by size class, largest first, so that the short ones fill the end
// of the launch.  Class 0 = a full chunk of T tokens; class k >= 1 = (T / 2^k, T / 2^(k-1)).
__device__ __forceinline__ int size_class(int n, int T) {
  if (n >= T) return 0;
  int cls = 1, t = T >> 1;
  while (n <= t && cls < 15) { ++cls; t >>= 1; }
  return cls;
}

// Tokens of the chunks of a head of C, cut to at most T: as many chunks as full ones would make (or fewer), all
// of one length but the last.  The chunks of a head wait for one another, so one that is much shorter would
// hold its place on a CU for nothing (3256 heads of 395 tokens in 32-bit rows, cut at 384: 384 and 11 tokens
// 385 us, 208 and 187 313; 310 when chunks did not wait and a second launch combined them).
__device__ __forceinline__ int cut_tokens(int C, int T, int b) {
  if (C <= T) return T;
  const int nch = (C + T - 1) / T, g = max(16, b);   // (chunks start on blocks and on groups of 16 tokens; T is a multiple of 64)
  return ((C + nch - 1) / nch + g - 1) & ~(g - 1);
}

// Pass 1 of the work list: number of items per size class.
static __global__ void __launch_bounds__(256) decode_count_kernel(DecodeArgs A) {
  __shared__ int bins[16];
  if (threadIdx.x < 16) bins[threadIdx.x] = 0;
  __syncthreads();
  const int gi = blockIdx.x * 256 + threadIdx.x;
  if (gi < A.gsel) {
    const int C = A.ctx[sel_to_g(A.D, A.l0, A.nl, gi)];
    const int nfull = C / A.T, rem = C - nfull * A.T;
    const int nch = nfull + (rem ? 1 : 0);
    if (!A.all_partials && nch > 1) {
      const int Th = cut_tokens(C, A.T, A.D.b), n = (C + Th - 1) / Th;
      atomicAdd(&bins[0], n);
    } else {
      if (nfull) atomicAdd(&bins[0], nfull);
      if (rem) atomicAdd(&bins[size_class(rem, A.T)], 1);
    }
  }
  __syncthreads();
  if (threadIdx.x < 16 && bins[threadIdx.x]) atomicAdd(&A.header[HW_DEC_BINS + threadIdx.x], bins[threadIdx.x]);
}

// Pass 2: every head instance claims its places and writes its items; a head that holds no
// KV gets its zero output rows here.  Workgroup x of a launch runs on XCD x % 8, so with
// rotate_chunks a head's chunks are dealt to the XCDs starting from a different one for every
// head: where only the first few chunks of every head have work (a block of queries early in a
// prompt) and heads hold a multiple of eight chunks, that work would otherwise all land on the
// same few XCDs.  Places are claimed per workgroup (one global atomic
// per class) and handed out inside it through LDS, so the global counters see few updates.
static __global__ void __launch_bounds__(256) decode_items_kernel(DecodeArgs A) {
  __shared__ int base[16], want[17], got[17];
  const int tid = threadIdx.x;
  if (tid < 17) want[tid] = 0;
  if (tid == 0) {
    int run = 0;
    int shorts = 0;
    for (int k = 0; k < 16; ++k) {
      const int c = A.header[HW_DEC_BINS + k];
      base[k] = run;
      run += c;
      if (k >= A.short_class) shorts += c;
    }
    if (blockIdx.x == 0) {
      A.header[HW_TOTAL_ITEMS] = run;
      A.header[HW_SHORT_ITEMS] = shorts;
    }
  }
  __syncthreads();
  const int gi = blockIdx.x * 256 + tid;
  int T = A.T;   // (of the head's chunks, below)
  int g = 0, C = 0, nfull = 0, rem = 0, nch = 0, cls = 0;
  int my_full = 0, my_rem = 0, my_p = 0;  // offsets inside this workgroup's claims
  if (gi < A.gsel) {
    g = sel_to_g(A.D, A.l0, A.nl, gi);
    C = A.ctx[g];
    nfull = C / T;
    rem = C - nfull * T;
    nch = nfull + (rem ? 1 : 0);
    if (!A.all_partials && nch > 1) {   // side by side, in the class of full chunks
      T = cut_tokens(C, T, A.D.b);
      nfull = nch = (C + T - 1) / T;
      rem = 0;
    }
    cls = rem ? size_class(rem, T) : 0;
    if (nfull) my_full = atomicAdd(&want[0], nfull);
    if (rem) my_rem = atomicAdd(&want[cls], 1);       // class 0 never holds a remainder
    if (nch > 1 || (A.all_partials && nch > 0)) my_p = atomicAdd(&want[16], nch);
  }
  __syncthreads();
  if (tid < 17 && want[tid])
    got[tid] = atomicAdd(&A.header[tid < 16 ? HW_DEC_CUR + tid : HW_DEC_PCUR], want[tid]);
  __syncthreads();
  if (gi >= A.gsel) return;
  if (C == 0) {
    if (A.out) {
      float* o = A.out + (size_t)g * A.D.r * A.D.d;
      for (int i = 0; i < A.D.r * A.D.d; ++i) o[i] = 0.0f;
    }
    return;
  }
  const bool slotted = nch > 1 || A.all_partials;
  const int pbase = slotted ? got[16] + my_p : 0;
  // the counters start from zero, so these bounds hold by construction; a workspace that was
  // never reset is the one way to break them, and then nothing is written
  if (pbase < 0 || pbase + nch > A.cap) return;
  if (nfull) {
    const int at = base[0] + got[0] + my_full;
    if (at < 0 || at + nfull > A.cap) return;
    for (int c = 0; c < nfull; ++c) {
      DecodeItem it = {g, c * T, min(T, C - c * T), nch, pbase, {0, T, 0}};
      const int place = at + (A.rotate_chunks ? (c + g) % nfull : c);
      A.items[place] = it;
      if (slotted && c < 2) A.slot_word[pbase + c] = 0;
    }
  }
  if (rem) {
    const int at = base[cls] + got[cls] + my_rem;
    if (at < 0 || at >= A.cap) return;
    DecodeItem it = {g, nfull * T, rem, nch, pbase, {0, T, 0}};
    A.items[at] = it;
  }
}

// Chunk length of a call over few heads.  Such a call is over when its slowest item is.  One
// workgroup alone on its CU streams ~25 GB/s, two that share one ~12 each, the chip ~6 TB/s:
// the slowest item and the whole call end together when a chunk is 1/256 of all the tokens
// with up to 256 heads, 1/512 from 512 heads on; a quarter on top for heads of unequal length.
// Where that leaves every head whole there is nothing to combine and it stays (256 heads of 2048
// KVs: 54 us, 67 when cut in two); heads that are cut anyway are cut to 1/512, so that the two
// workgroups a CU has room for even out what the other leaves (256 ragged heads of up to 16384
// KVs, 2048 on average: 77 -> 71 us; 1/384, 1/768 and 1/1024: 77, 74 and 74).  Cutting costs: the
// chunks of a head meet, which takes longer the more there are, so they stay at 512 tokens as long as
// that is no more than 1/256 (8 heads of 8786 KVs, r = 8, 16-bit rows: 25 us in chunks of 192, 19 in
// 384; 12 of 5082 on average, the longest of far more, r = 1: 25 and 16; 64 of 3093, fp8: 24 in 512,
// 28 in 1024), and nothing is shorter than 128 (8 heads of 1000 KVs: 18.2 us at 256, 15.8 at 128 and
// at 64, with a second launch that combined them).
constexpr int kMeetingChunk = 512;
constexpr int kSmallCallChunk = 128;
__device__ __forceinline__ int small_call_chunk(int T_max, unsigned long long tokens, int live, int longest) {
  const unsigned long long want = tokens + tokens / 4;
  auto length = [&](int den) {
    // (a 64-bit division by a variable is ~150 instructions, in front of everything a small call does)
    const unsigned long long t = want >> 32 ? want / den : (unsigned long long)((unsigned)want / (unsigned)den);
    const int t64 = (int)((t < (unsigned long long)T_max ? t : (unsigned long long)T_max) + 63) & ~63;
    return min(T_max, max(kSmallCallChunk, t64));
  };
  const int T = length(min(512, max(256, live)));
  return longest <= T ? T : max(length(512), min(length(256), min(kMeetingChunk, T_max)));
}

// What the fraction cannot see is whether the chunks have places at once.  A few too many run by themselves in
// the end, each as long as what ran before (chunks longer than T / 2: shorter ones, whole heads all of them, fill gaps).
// Then T is the shortest that has places for all the longer ones at once, if the longest chunk has.  320 heads of
// 1650 to 8250 KVs, r = 4, d = 128, 512 places: chunks of 3328 tokens (545 long ones) 156 us, of 3648 (509) 139, of 6144
// (380) 163; 8-bit rows 103, 81 and 108.  Not two turns of as many chunks as there are places: 120 -> 108 us
// at the best of sizes, slower at others.
// long_chunks(T): chunks longer than T / 2 when heads are cut at T; no more, the longer T is.
template <class Count>
__device__ __forceinline__ int one_turn(int T, int T_max, int places, Count long_chunks) {
  if (T >= T_max || long_chunks(T) <= places || long_chunks(T_max) > places) return T;
  int lo = T / 64, hi = T_max / 64;   // too short; long enough
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (long_chunks(64 * mid) <= places) hi = mid; else lo = mid;
  }
  return 64 * hi;
}

// Both passes in one workgroup, for calls over at most kSmallWorklistHeads head instances (one
// layer of a model, one prompt): one launch instead of two.  Leaves the header words as the
// two-pass pair does.  (Measured with two heads per thread, 2048 heads: no faster than the pair.)
constexpr int kSmallWorklistHeads = 1024;
template <bool PLAN>
static __global__ void __launch_bounds__(1024) decode_worklist_small_kernel(DecodeArgs A) {
  __shared__ int bins[16], base[16], cur[17], tally[16];
  __shared__ unsigned long long tokens;
  __shared__ int live, longest;
  __shared__ unsigned long long before;
  const int tid = threadIdx.x;
  // a plan: workgroup l lists layer A.l0 + l into that layer's header block and stretch of records
  const int layer = PLAN ? (int)blockIdx.x : 0;
  int32_t* header = A.header + (size_t)layer * (PLAN ? HW_WORDS : 0);
  DecodeItem* items = A.items + (size_t)layer * A.plan_stride;
  int32_t* slot_word = A.slot_word + (size_t)layer * A.plan_stride;
  int cap = A.cap;
  if (tid == 0) { tokens = 0; live = 0; longest = 0; before = 0; }
  if (tid < 16) { bins[tid] = 0; tally[tid] = 0; }
  if (tid < 17) cur[tid] = 0;
  __syncthreads();
  int g = 0, C = 0, listed = 0, nfull = 0, rem = 0, nch = 0, cls = 0;
  if (tid < A.gsel) {
    g = sel_to_g(A.D, A.l0 + layer, A.nl, tid);
    C = A.ctx[g] + A.ctx_plus;
    // (A full head planned one token longer: its row ends in front of that token.  Its records, which a
    // decode looks up in the row before it compares the length, end there too.)
    listed = PLAN ? (int)min((long long)C, (long long)A.D.maxb * A.D.b) : C;
  }
  // Where stretches of equal length, for what full rows hold, do not fit: the layer's records start
  // behind the most that the layers before it can need from their lengths (a full chunk holds at least
  // kSmallCallChunk tokens, and a head has one shorter chunk).  That always fits: all layers together
  // need no more records than the workspace has for one call over them all.
  const bool placed = PLAN && A.plan_stride == 0;
  if (placed) {
    const int per = layer * A.D.Hk;
    unsigned long long t = 0;
    for (int i = tid; i < A.D.S * per; i += (int)blockDim.x) {
      const int s = i / per;
      t += (unsigned long long)max(A.ctx[(size_t)s * A.D.Lyr * A.D.Hk + (i - s * per)] + A.ctx_plus, 0);
    }
    for (int m = 32; m >= 1; m >>= 1) t += __shfl_xor(t, m);
    if ((tid & 63) == 0 && t) atomicAdd(&before, t);
    // (a plan picks its chunk length on the device: the barrier below serves)
  }
  int T = A.T;
  if (A.adapt_T) {
    const unsigned long long t = wave_sum_long(max(C, 0));
    const int lm = wave_max(C);
    const int lv = __popcll(__ballot(C > 0));
    if ((tid & 63) == 0 && t) { atomicAdd(&tokens, t); atomicAdd(&live, lv); atomicMax(&longest, lm); }
    __syncthreads();
    T = small_call_chunk(A.T, tokens, live, longest);
    if (longest > T && tokens + (unsigned long long)live * T > (unsigned long long)A.places * T) {   // (tokens / T and one per head at most)
      int step = 0;   // (nine at most: chunks are up to 8192 tokens)
      T = one_turn(T, A.T, A.places, [&](int t) {
        const int n = wave_sum_i(listed > t / 2 ? (listed + t - 1) / t : 0);
        if ((tid & 63) == 0 && n) atomicAdd(&tally[step], n);
        __syncthreads();
        return tally[step++];
      });
    }
  }
  if (placed) {
    const unsigned long long at = before / kSmallCallChunk + (unsigned long long)layer * A.gsel;
    const int start = (int)(at < (unsigned long long)A.plan_cap ? at : (unsigned long long)A.plan_cap);
    items += start;
    slot_word += start;
    cap = min(cap, A.plan_cap - start);
    if (tid == 0) header[HW_PLAN_BASE] = start;
  }
  if (tid < A.gsel) {
    nfull = listed / T;
    rem = listed - nfull * T;
    nch = nfull + (rem ? 1 : 0);
    if (!A.all_partials && nch > 1) {   // side by side, in the class of full chunks
      T = cut_tokens(listed, T, A.D.b);
      nfull = nch = (listed + T - 1) / T;
      rem = 0;
    }
    cls = rem ? size_class(rem, T) : 0;
    if (rem) atomicAdd(&bins[cls], 1);
  }
  // full chunks and partial-result slots are claimed per wavefront (a thousand adds to one LDS word are
  // run one after the other)
  const bool slotted = nch > 1 || (A.all_partials && nch > 0);
  const int lane = tid & 63, full_to = wave_prefix_i(nfull), slots_to = wave_prefix_i(slotted ? nch : 0);
  int full_at = 0, slots_at = 0;
  if (lane == 63) {
    if (full_to) { atomicAdd(&bins[0], full_to); full_at = atomicAdd(&cur[0], full_to); }
    if (slots_to) slots_at = atomicAdd(&cur[16], slots_to);
  }
  full_at = __builtin_amdgcn_readlane(full_at, 63) + full_to - nfull;
  const int pbase = slotted ? __builtin_amdgcn_readlane(slots_at, 63) + slots_to - nch : 0;
  __syncthreads();
  if (tid < 64) {
    const int n = tid < 16 ? bins[tid] : 0, to = wave_prefix_i(n);
    if (tid < 16) base[tid] = to - n;
    const int run = __builtin_amdgcn_readlane(to, 63), longs = A.short_class > 0 ? __builtin_amdgcn_readlane(to, A.short_class - 1) : 0;
    if (tid == 0) {
      // (a list that does not fit, which lengths the pool can hold never make, is one no decode takes)
      header[HW_TOTAL_ITEMS] = PLAN && run > cap ? 0x7fffffff : run;
      header[HW_SHORT_ITEMS] = run - longs;
    }
  }
  __syncthreads();
  if (tid >= A.gsel) return;
  if (C == 0) {
    if (A.out) {
      float* o = A.out + (size_t)g * A.D.r * A.D.d;
      for (int i = 0; i < A.D.r * A.D.d; ++i) o[i] = 0.0f;
    }
    return;
  }
  if (pbase < 0 || pbase + nch > cap) return;
  if (nfull) {
    const int at = base[0] + full_at;
    if (at < 0 || at + nfull > cap) return;
    for (int c = 0; c < nfull; ++c) {
      DecodeItem it = {g, c * T, min(T, listed - c * T), nch, pbase, {C, T, 0}};
      const int place = at + (A.rotate_chunks ? (c + g) % nfull : c);
      items[place] = it;
      if (slotted && c < 2) slot_word[pbase + c] = 0;
    }
  }
  if (rem) {
    const int at = base[cls] + atomicAdd(&cur[cls], 1);
    if (at < 0 || at >= cap) return;
    DecodeItem it = {g, nfull * T, rem, nch, pbase, {C, T, 0}};
    items[at] = it;
  }
}

// A call over at most kSelfListHeads head instances (a layer of one or a few sequences) keeps no
// work list: every wavefront (lane = head instance) reads the lengths, repeats the cut and picks
// its workgroup's item, one load and a few cross-lane scans in place of a launch (~7 us) and two
// dependent loads.  Item x: the chunks of the heads of more than one chunk, head by head, then the
// heads of one.  Returns false when there is no item x.  (Not for more heads, four a lane or one a thread: without the list's order by size long
// remainders meet on one CU, 256 ragged heads of 2048 KVs on average 62 -> 77 us; and at 512 heads
// the prologue of every workgroup, empty ones too, costs what the launch does.)
constexpr int kSelfListHeads = 64;
// Where the chunks of head x meet without a list: a word (from the workspace's first on) of the header block or of
// the first layer's behind it, whose other words serve kept lists.  Nothing but these calls writes it, whatever
// configs the calls on a workspace have, and every config's reset clears it; further blocks are another config's
// tables and records.  Atomics on one line are run one after the other, so heads are dealt out to the four lines of
// 128 bytes that the two blocks have free, then to the second halves of these.
static_assert(HW_DEC_END <= HW_MEET && HW_MEET + kSelfListHeads <= HW_WORDS && kSelfListHeads == 8 * 8, "room for the meeting words");
__device__ __forceinline__ int meet_word(int x) {
  return (x & 1) * HW_WORDS + HW_MEET + (x & 2) * 16 + (x & 4) * 4 + (x >> 3);
}
struct SelfList { DecodeItem it; int word; int C; int g; };   // item, its head's meeting word; this lane's head and length (g = -1: none)
__device__ __forceinline__ bool self_item(const DecodeArgs& A, int x, SelfList& out) {
  const int lane = threadIdx.x & 63;
  int g = -1, C = 0;
  if (lane < A.gsel) {
    g = sel_to_g(A.D, A.l0, A.nl, lane);
    C = max(A.ctx[g], 0);
  }
  int T = A.T;
  if (A.adapt_T) {
    T = small_call_chunk(A.T, wave_sum_long(C), __popcll(__ballot(C > 0)), wave_max(C));
  }
  T = cut_tokens(C, T, A.D.b);
  const int nch = (C + T - 1) / T;
  const int split = nch > 1 ? nch : 0;
  const int si = wave_prefix_i(split);   // inclusive
  const int P = __builtin_amdgcn_readlane(si, 63);
  const unsigned long long whole = __ballot(nch == 1);
  int t0 = -1;   // the item's first token, in the lane of its head
  if (x < P) {
    if (x >= si - split && x < si) t0 = (x - (si - split)) * T;
  } else if (nch == 1 && x - P == __popcll(whole & ((1ull << lane) - 1ull))) {
    t0 = 0;
  }
  out.C = C; out.g = g;
  const unsigned long long has = __ballot(t0 >= 0);
  if (has == 0) return false;
  const int src = __builtin_ctzll(has);
  const int Th = __builtin_amdgcn_readlane(T, src);
  out.word = src;
  out.it = DecodeItem{__builtin_amdgcn_readlane(g, src), __builtin_amdgcn_readlane(t0, src), 0,
                      __builtin_amdgcn_readlane(nch, src), __builtin_amdgcn_readlane(si - split, src), {0, Th, 0}};
  out.it.n_tok = min(Th, __builtin_amdgcn_readlane(C, src) - out.it.t0);
  return true;
}

template <int N, int MASK>
struct Butterfly {
  // Sums v[0..N) across the lanes that differ in the bits at and below MASK, halving the
  // number of live values at each step while more than one is left.
  static __device__ __forceinline__ void run(float* v, int lane) {
    if constexpr (MASK >= 1) {
      if constexpr (N > 1) {
        constexpr int H = N / 2;
        const bool up = (lane & MASK) != 0;
#pragma unroll
        for (int i = 0; i < H; ++i) {
          const float keep = up ? v[H + i] : v[i];
          const float send = up ? v[i] : v[H + i];
          v[i] = keep + lane_xor<MASK>(send);
        }
        Butterfly<H, MASK / 2>::run(v, lane);
      } else {
        v[0] += lane_xor<MASK>(v[0]);
        Butterfly<1, MASK / 2>::run(v, lane);
      }
    }
  }
};

}  // namespace kvc
