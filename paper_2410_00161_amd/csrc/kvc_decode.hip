// Paged decode attention with one block table and one context length per
// (sequence, layer, KV head), accumulating the per-KV eviction metric in the
// same pass (KV-Compress: Preliminaries "Multi-head Attention" and "Paged
// Attention"; Method "Query Group Compression", "Block Layout and Parallel
// Allocation", "Squared Attention Metric", "Continual Compression").
//
// Work decomposition.  The metric needs the NORMALISED probability of every KV,
// which is known only once a head's max and sum are.  A head instance is cut
// into chunks of T tokens; one workgroup owns one chunk, keeps the chunk's r x T
// logits in LDS between its pass over K and its pass over V, and therefore
// reads every key and value exactly once.  A head that fits one chunk is
// finished inside that workgroup (output and metric written directly).  The chunks of
// a longer head leave their (max, sum, un-normalised output) in the workspace, wait for one
// another and finish the head together (see kMeetBits).
//
// Data movement.  A KV row (d elements) is 256 bytes at d = 128 / bf16; a lane
// reads 16 bytes, so LPT = row_bytes / 16 lanes cover one token and a wavefront
// load covers 64 / LPT whole tokens: 1 KiB contiguous per load at b >= TPI.
// The r dot products of a token are finished with a halving butterfly over the
// LPT lanes, which leaves each lane with distinct (token, head) logits instead
// of every lane with all of them.
#include <algorithm>
#include <atomic>
#include <cmath>
#include <mutex>

#include "kvc_common.h"
#include "kvc_worklist.h"

namespace kvc {

// Host-side state of the process: the chunk-length knob (read once per call), what the runtime
// has been told about the chunk kernels' LDS, and the benchmark's event recording behind one lock.
static std::atomic<int> g_chunk_tokens{0};  // 0 = default; set by kvc_set_decode_chunk

// optional event pairs around the decode kernels (kvc_profile_begin / _collect)
struct ProfilePair { hipEvent_t a0, a1, s0, s1; };  // long-item, short-item launches
static std::mutex g_prof_lock;
static ProfilePair* g_prof = nullptr;
static int g_prof_cap = 0, g_prof_used = 0, g_prof_on = 1;
static std::atomic<bool> g_prof_any{false};   // recording asked for: only then a call takes the lock

static ProfilePair* claim_profile_pair() {
  if (!g_prof_any.load(std::memory_order_acquire)) return nullptr;
  std::lock_guard<std::mutex> hold(g_prof_lock);
  return (g_prof && g_prof_on && g_prof_used < g_prof_cap) ? &g_prof[g_prof_used++] : nullptr;
}

typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef short i16x4_t __attribute__((ext_vector_type(4)));

template <int ESZ> struct Row;
// P: the piece of a K or V row one lane loads (PB bytes, EPL elements); Q: the query elements
// that face it; QSZ: bytes of a query element.
template <> struct Row<2> {  // bf16: 8 elements in 16 bytes
  static constexpr int EPL = 8;
  static constexpr int QSZ = 2;
  static constexpr int PB = 16;
  typedef uint4 P;
  typedef uint4 Q;
  static __device__ __forceinline__ P load(const void* p) { return load_stream16(p); }
  static __device__ __forceinline__ P zero() { return make_uint4(0, 0, 0, 0); }
  static __device__ __forceinline__ Q load_q(const char* qrow, int seg) { return *(const uint4*)(qrow + (size_t)seg * 16); }
  static __device__ __forceinline__ float dot(const uint4& a, const uint4& b) {
    float s = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, a.x), __builtin_bit_cast(bf16x2_t, b.x), 0.0f, false);
    s = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, a.y), __builtin_bit_cast(bf16x2_t, b.y), s, false);
    s = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, a.z), __builtin_bit_cast(bf16x2_t, b.z), s, false);
    s = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, a.w), __builtin_bit_cast(bf16x2_t, b.w), s, false);
    return s;
  }
  static __device__ __forceinline__ uint4 as_bf16x8(const uint4& a) { return a; }
  static __device__ __forceinline__ void widen(const uint4& a, float* f) {
    f[0] = bf16_lo(a.x); f[1] = bf16_hi(a.x); f[2] = bf16_lo(a.y); f[3] = bf16_hi(a.y);
    f[4] = bf16_lo(a.z); f[5] = bf16_hi(a.z); f[6] = bf16_lo(a.w); f[7] = bf16_hi(a.w);
  }
};
template <> struct Row<4> {  // f32: 4 elements in 16 bytes
  static constexpr int EPL = 4;
  static constexpr int QSZ = 4;
  static constexpr int PB = 16;
  typedef uint4 P;
  typedef uint4 Q;
  static __device__ __forceinline__ P load(const void* p) { return load_stream16(p); }
  static __device__ __forceinline__ P zero() { return make_uint4(0, 0, 0, 0); }
  static __device__ __forceinline__ Q load_q(const char* qrow, int seg) { return *(const uint4*)(qrow + (size_t)seg * 16); }
  static __device__ __forceinline__ float dot(const uint4& a, const uint4& b) {
    float s = __uint_as_float(a.x) * __uint_as_float(b.x);
    s = fmaf(__uint_as_float(a.y), __uint_as_float(b.y), s);
    s = fmaf(__uint_as_float(a.z), __uint_as_float(b.z), s);
    s = fmaf(__uint_as_float(a.w), __uint_as_float(b.w), s);
    return s;
  }
  static __device__ __forceinline__ void widen(const uint4& a, float* f) {
    f[0] = __uint_as_float(a.x); f[1] = __uint_as_float(a.y);
    f[2] = __uint_as_float(a.z); f[3] = __uint_as_float(a.w);
  }
};

typedef float f32x2_t __attribute__((ext_vector_type(2)));
template <> struct Row<1> {  // OCP e4m3: 8 elements in 8 bytes, facing 8 bf16 query elements
  // Pieces of 8 bytes, not 16: a d = 128 row is then spread over 16 lanes as for bf16, and the
  // output accumulator of a lane (r x EPL floats) stays at the size the registers hold.
  static constexpr int EPL = 8;
  static constexpr int QSZ = 2;
  static constexpr int PB = 8;
  typedef uint2 P;
  typedef uint4 Q;
  static __device__ __forceinline__ P load(const void* p) { return load_stream8(p); }
  static __device__ __forceinline__ P zero() { return make_uint2(0, 0); }
  static __device__ __forceinline__ Q load_q(const char* qrow, int seg) { return *(const uint4*)(qrow + (size_t)seg * 16); }
  // four 8-bit floats -> two packed bf16 pairs (exact: 3 mantissa bits fit in 7; one instruction
  // per pair, scale 1), then the same packed dot product as for a bf16 cache
  static __device__ __forceinline__ float dot4(uint32_t k, uint32_t q01, uint32_t q23, float s) {
    const bf16x2_t p01 = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(k, 1.0f, false);
    const bf16x2_t p23 = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(k, 1.0f, true);
    s = __builtin_amdgcn_fdot2_f32_bf16(p01, __builtin_bit_cast(bf16x2_t, q01), s, false);
    return __builtin_amdgcn_fdot2_f32_bf16(p23, __builtin_bit_cast(bf16x2_t, q23), s, false);
  }
  static __device__ __forceinline__ uint4 as_bf16x8(const uint2& a) {
    return make_uint4(__builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(a.x, 1.0f, false)),
                      __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(a.x, 1.0f, true)),
                      __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(a.y, 1.0f, false)),
                      __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(a.y, 1.0f, true)));
  }
  static __device__ __forceinline__ float dot(const uint2& a, const Q& q) {
    return dot4(a.y, q.z, q.w, dot4(a.x, q.x, q.y, 0.0f));
  }
  static __device__ __forceinline__ void widen(const uint2& a, float* f) {
    const uint32_t w[2] = {a.x, a.y};
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const f32x2_t lo = __builtin_amdgcn_cvt_pk_f32_fp8((int)w[i], false);
      const f32x2_t hi = __builtin_amdgcn_cvt_pk_f32_fp8((int)w[i], true);
      f[4 * i] = lo.x; f[4 * i + 1] = lo.y; f[4 * i + 2] = hi.x; f[4 * i + 3] = hi.y;
    }
  }
};

// The exp of every logit against its group's running max, e in [0, 1], is kept in LDS as 16-bit fixed
// point: the error of e, and so of the probability it turns into (p = e * weight, weight <= 1), is at
// most 2^-17, which moves a metric increment (sum over r heads of p^2 or p) by at most r * 2^-16.
__device__ __forceinline__ uint32_t q16(float e) { return (uint32_t)(e * 65535.0f + 0.5f); }

// What a chunk that does not wait for the rest of its head (see kMeetBits) leaves of a KV: its exps
// against the chunk's max, as the chunk itself would go on with them, so that the metric has the same bits
// whoever adds it.
template <int R>
__device__ __forceinline__ void exps_publish(float* stash, size_t slot, const float (&e)[R]) {
  if constexpr (R == 1) publish_i32((int32_t*)stash + slot, __float_as_int(e[0]));
  else
#pragma unroll
    for (int i = 0; i < R; i += 2) publish_u64(stash + slot * R + i, (uint64_t)__float_as_uint(e[i]) | (uint64_t)__float_as_uint(e[i + 1]) << 32);
}
template <int R>
__device__ __forceinline__ void exps_published(const float* stash, size_t slot, float (&e)[R]) {
  if constexpr (R == 1) e[0] = __int_as_float(published_i32((const int32_t*)stash + slot));
  else
#pragma unroll
    for (int i = 0; i < R; i += 2) {
      const uint64_t t = published_u64(stash + slot * R + i);
      e[i] = __uint_as_float((uint32_t)t); e[i + 1] = __uint_as_float((uint32_t)(t >> 32));
    }
}

// The chunks of a head of more than one finish it themselves.  Each leaves its max, sum and
// un-normalised output and then needs the head's max and sum, for the metric of its own tokens (their exps are
// still in its LDS) and for its share of the head's output.  It counts itself as started when it begins and
// as arrived when its part is out, and waits for the others only if all of them have started by
// then: a chunk that has started runs, and arrives without waiting for anybody, so every wait ends.  A
// chunk that finds some not started leaves its exps and ends; those that waited (one at least, the one
// that started last) share out what is left of it.  The last one to arrive sets the counts back and
// calls the others, each at a word of its own: a hundred of them looking at the word that they add to keep
// the adds waiting, ~10 ns each (one layer of 8 ragged heads, up to 107 chunks: 22.4 us a layer so, 18.2 with
// words of their own, 19.1 as a launch for the chunks and one that combined them).
// Before, chunks left 2 r bytes of exps per KV and a second launch combined them: 4 x 131072 tokens at 8x, r = 8
// 4015 -> 3490 us (the exps were 16 of 528 bytes a KV; what is written costs this chip ten times what is
// read does), 16 sequences layer by layer 1174 -> 1080, a step of two sequences of 512 tokens 25 -> 21.7.
// Started and arrived are halves of one word per head: a header word in a call without a work list, else one
// where the list keeps the head's partial-result slots (the first two, in rows of so many chunks that a half could run over).
// The words are zero between calls.  Where they are not (a workspace never reset, or in use by two calls at
// once) too few or too many chunks seem to have come: a count beyond the head's chunks, an arrival ahead of its start,
// chunks that all left or a call that does not come say so in the status.
constexpr int kMeetBits = 16, kMeetMost = (1 << kMeetBits) - 1;   // of a half
constexpr int kMeetLooks = 1 << 19;   // for the call, ~0.5 us each
constexpr int kMeetStarts = 6;        // for the last chunk to start, ~1 us each: one that does soon is worth the wait

constexpr int kCus = 256;
constexpr int kDecodeThreads = 256;
constexpr int kDecodeWaves = kDecodeThreads / 64;

// A shape takes both products to the matrix cores where the plain ALUs are the bound: 16-bit or 8-bit
// rows (the latter widened to bf16 on their way into the operand tile) with eight query heads per
// KV head, 8-bit rows of d = 128 with four (half the bytes per logit: with the dot products on the plain
// ALUs that launch ran 8 % longer).  On the plain ALUs and here, decode steps over 32 layers x 8 KV heads
// at a quarter of 8192 tokens: d = 128 in blocks of 8 tokens, 16 sequences of bf16 with eight heads
// 1250 and 843 us, of fp8 with eight 1224 and 576, 24 of fp8 with four 766 and 705; d = 64, 32 sequences
// of bf16 with eight 1134 and 912, of fp8 with eight 1061 and 766, of fp8 with four 647 and 656 (left out).
__host__ __device__ constexpr bool decode_uses_mfma(int esz, int R, int HD) {
  return (HD == 128 || HD == 64) && ((R == 8 && esz <= 2) || (R == 4 && esz == 1 && HD == 128));
}

// Register buffers of K and V groups a wavefront rotates through (one less is in flight behind
// the group being worked on): three for rows of at most 16 bits when four wavefronts share a
// long chunk (up to four query heads, or the matrix-core shapes), else two.
__host__ __device__ constexpr int decode_depth(int esz, int R, int HD, int nw) {
  if (nw != 4 || esz > 2) return 2;
  return (R <= 4 || decode_uses_mfma(esz, R, HD)) ? 3 : 2;
}

__host__ __device__ inline size_t decode_lds_bytes(int T, int R, int HD, int b, int waves = kDecodeWaves,
                                                   bool mfma = false) {
  // per-wavefront un-normalised output; on the matrix-core path the same bytes serve, while
  // the main loop runs, as the wavefront's operand tile (16 tokens of d 16-bit elements)
  const size_t per_wave_out = mfma ? (size_t)16 * HD * 2 : (size_t)R * HD * 4;
  return (size_t)T * R * 2                       // exp of every logit against its group's running max, 16-bit
         + (size_t)(T / 16) * R * 4              // that running max, per 16-token group and head
         + (size_t)waves * per_wave_out
         + (size_t)waves * 16 * R * 4            // per-wavefront exp of the current group, f32
         + 2 * waves * R * 4                     // per-wavefront max and sum
         + ((size_t)T / b + 1) * 4;              // block ids of the chunk
}

// One workgroup = one chunk of up to T tokens of one head instance; one pass.
//
// Each wavefront walks its 16-token groups with the next group's K and V rows
// already in flight.  Per group: r dot products per token (butterfly over the
// lanes of a token), running max per query head (online softmax), exp of the
// group against the running max, rescale of the output accumulator when a max
// moved, then acc += p * v.  What the metric needs later, the exp of every
// logit, stays in LDS as 16-bit fixed point next to the running max it was
// taken against (one f32 per group and head): once the wavefronts have been
// merged, the normalised probability of every KV follows without touching K
// again.  The quantisation moves a probability by at most 2^-17.
//
// NW = 4 wavefronts share a chunk.  The short items at the end of the work list (at most
// A.Ts tokens) are latency-bound, a chain of dependent loads (item, block table, K and V) in
// front of a few groups of arithmetic: they get a launch of their own with NW = 1, small LDS
// and fewer registers, so that a CU holds many of those chains at once.
// Long chunks of 8-bit rows with four query heads in blocks shorter than 16 tokens: by itself the compiler takes
// 170 registers, two below which a third workgroup fits a CU (4096 heads of up to 120 tokens 70 us, 56 with
// it; of up to 1000 177 and 153).  With eight and blocks of 16 it takes 172, and a third workgroup is worth three
// registers spilt (see decode_groups).
constexpr int decode_waves(int esz, int HD, int R, bool b16, int nw) {
  return esz == 1 && HD == 128 && nw == 4 && (R == 4 ? !b16 : R == 8 && b16) ? 3 : 1;
}

// Workgroups of four wavefronts that should share a CU, where the registers let more than two: the default chunk
// is then the longest that leaves each its part of the LDS (what a chunk keeps grows with its tokens).  Over
// 32 x 8192, 4 x 65536 and 64 x 2048 tokens at 8x, 8 KV heads, two workgroups (3456 or 6144 tokens) and so, us:
// d = 64: 16-bit rows with eight query heads 984, 895, 497 and 849, 809, 466 (2368 tokens), with four 808, 773,
// 464 and 794, 765, 436 (5120); 8-bit rows with eight 1619, 1456, 795 and 1141, 1089, 621 (1664), with four
// 1180, 1215, 703 and 1037, 964, 571 (3840); d = 128, 8-bit rows with eight 1066, 971, 551 and 959, 929, 509 (1920).
// Not where nothing comes of it: 8-bit rows of d = 128 with four (3456 tokens 849, 812; 6144 849, 806), 16-bit ones
// with two (168 registers 751, 758, 392; 170 739, 740, 394).
constexpr int decode_groups(int esz, int HD, int R, bool b16) {
  return HD == 64 && R >= 4 ? (esz == 1 ? 4 : esz == 2 ? 3 : 2) : esz == 1 && HD == 128 && R == 8 && b16 ? 3 : 2;
}

template <int ESZ, int HD, int R, bool B16, int NW, bool MF = decode_uses_mfma(ESZ, R, HD)>
__global__ void __launch_bounds__(NW * 64, decode_waves(ESZ, HD, R, B16, NW)) decode_chunk_kernel(DecodeArgs A) {
  constexpr int NT = NW * 64;
  constexpr int DEPTH = decode_depth(ESZ, R, HD, NW);
  constexpr int EPL = Row<ESZ>::EPL;
  constexpr int PB = Row<ESZ>::PB;     // bytes a lane loads at once
  typedef typename Row<ESZ>::P Piece;
  constexpr int LPT = HD / EPL;        // lanes per token
  constexpr int TPI = 64 / LPT;        // tokens per wavefront load
  constexpr int U = 16 / TPI;          // loads per 16-token group
  constexpr int NV = R * U;            // partial logits per lane before the butterfly
  constexpr int PER = NV >= LPT ? NV / LPT : 1;  // logits per lane after it
  constexpr size_t ROWB = (size_t)HD * ESZ;
  constexpr size_t QROWB = (size_t)HD * Row<ESZ>::QSZ;
  static_assert(LPT >= 4 && LPT <= 32 && (16 % TPI) == 0, "row geometry");
  // Q K^T of a 16-token group on the matrix cores (rows = query heads, columns = tokens): d = 128 in blocks of 16
  // tokens or more by v_mfma_f32_16x16x32_bf16, four steps of 32 dimensions in one chain; the other shapes by
  // v_mfma_f32_16x16x16_bf16, products of 16 dimensions added up in pairs.  K still arrives by contiguous loads
  // (a load shaped like the operand is 12 % slower); a wavefront turns its tile into operand order through 32 d
  // bytes of LDS (16 tokens of d 16-bit elements), cells XOR-swizzled so that neither side has a bank conflict.
  // Head h sits in operand row 4 (h % 4) + h / 4, which leaves lane 16 a + t with the logits of token t against
  // head a, and with eight heads a + 4.
  constexpr int RW = MF ? 8 : R;      // output rows a wavefront's LDS region has room for
  constexpr int NVH = (R + 3) / 4;     // MF: logits per lane
  constexpr int OWN = MF ? NVH : PER;

  const int tid = threadIdx.x, lane = tid & 63, w = NW == 1 ? 0 : tid >> 6;
  extern __shared__ __align__(16) char smem_raw[];
  DecodeItem it;
  int word = 0;                          // meeting word of the head in a call without a list
  const int T = NW == 4 ? A.T : A.Ts;    // tokens this launch sizes its LDS arrays for
  int32_t* slot_words = A.slot_word;     // of this list
  int rec = 0;                           // record of this item
  if (NW == 4 && A.self_list) {
    SelfList sl;
    const bool found = self_item(A, blockIdx.x, sl);
    // heads without a KV (lane = head, the same in every wavefront): the first workgroup writes their zero rows
    if (blockIdx.x == 0)
      for (unsigned long long empty = __ballot(sl.g >= 0 && sl.C == 0); empty; empty &= empty - 1) {
        float* o = A.out + (size_t)__builtin_amdgcn_readlane(sl.g, __builtin_ctzll(empty)) * R * HD;
        for (int i = tid; i < R * HD; i += NT) o[i] = 0.0f;
      }
    if (!found) return;
    it = sl.it;
    word = sl.word;
    rec = blockIdx.x;   // (no list: the records' room serves the heads that meet)
  } else {
    const int total_items = A.header[HW_TOTAL_ITEMS];
    const int short_items = A.header[HW_SHORT_ITEMS];
    const bool placed = A.plan && A.plan_stride == 0;
    const int base = placed ? A.header[HW_PLAN_BASE] : 0;
    if (NW == 4 && blockIdx.x == 0 && tid < HW_DEC_END - HW_DEC_BINS) A.header[HW_DEC_BINS + tid] = 0;  // work-list block back to zero
    if (NW == 4 && A.plan && (int)blockIdx.x < A.gsel) {
      // a list kept from kvc_decode_plan was made without the output at hand: the zero rows of a
      // head that holds no KV are written here, by the workgroup with the head's index
      const int ge = sel_to_g(A.D, A.l0, A.nl, blockIdx.x);
      if (A.ctx[ge] == 0)
        for (int i = tid; i < R * HD; i += NT) A.out[(size_t)ge * R * HD + i] = 0.0f;
    }
    // (A long item's record is where the workgroup's index says: in a small call asked for together with the
    // header words.  In a large one the workgroups beyond the last item pay more for it than the others
    // gain, 64 x 8192 tokens at 8x 1451 us against 1445.)
    const bool early = NW == 4 && A.adapt_T && !placed;
    if (early && (int)blockIdx.x < A.cap) it = A.items[blockIdx.x];
    if (total_items > A.cap || short_items < 0 || short_items > total_items) return;
    const int n_long = total_items - short_items;
    if ((int)blockIdx.x >= (NW == 4 ? n_long : short_items)) return;
    if (placed && (base < 0 || base > A.plan_cap - total_items)) return;
    slot_words += base;
    rec = base + blockIdx.x;
    if (!early) it = A.items[base + (NW == 4 ? blockIdx.x : n_long + blockIdx.x)];   // the short items end the list
  }
  // (the same in every lane: in scalar registers)
  auto uniform = [](int v) { return __builtin_amdgcn_readfirstlane(v); };
  const int g = uniform(it.g), t0 = uniform(it.t0), n_tok = uniform(it.n_tok), nch = uniform(it.nch);
  it.pbase = uniform(it.pbase);
  it.pad[0] = uniform(it.pad[0]);
  const int Tc = uniform(it.pad[1]);     // tokens of the head's chunks but the last
  if ((unsigned)g >= (unsigned)A.D.G || n_tok <= 0 || n_tok > T || t0 < 0 || nch <= 0 || Tc < 16 || Tc > A.T ||
      (nch > 1 && (it.pbase < 0 || it.pbase + nch > A.cap)))
    return;  // not a record this call wrote
  const int C_now = A.plan ? A.ctx[g] : 0;   // (looked at below, behind the other loads)
  const int b = A.D.b, lb = A.log2b;

  uint4* s_kt = (uint4*)smem_raw;                      // MF: [waves][16 tokens][HD / 8 cells of 16 bytes]
  // [waves][RW][HD]; on the matrix-core path, where eight rows have room (RW * HD * 4 = 16 * HD * 2 bytes, also
  // with four heads), a wavefront's part of it is its operand tile until its main loop ends, so that no
  // wavefront touches another's tile
  float* s_acc = (float*)smem_raw;
  constexpr int PARTS = HD == 128 && B16 ? 2 : 3;   // MF: parts of 16 bits of a probability (see P V)
  constexpr int PROWS = R == 4 && PARTS == 3 ? 4 : 8;   // MF: operand rows between a head's parts
  constexpr int CELLS = HD / 8;        // MF: 16-byte cells of a token's row in the operand tile
  // position of cell c of token t's row: such that the 16 lanes that read one cell of 16 keys, and the 8
  // tokens x 32 bytes that half a wavefront reads of V, touch every bank once
  auto k_at = [](int t, int c) { return t * CELLS + (c ^ (CELLS == 16 ? t : t >> 1)); };
  auto v_swizzle = [](int t) { return CELLS == 16 ? 2 * (t & 7) : 2 * ((t >> 1) & 3); };
  static_assert(!MF || U == HD / 32, "a product of 32 dimensions per load");
  static_assert(!MF || (size_t)RW * HD * 4 == (size_t)16 * HD * 2, "output rows alias the operand tile wavefront by wavefront");
  float* s_e = s_acc + NW * RW * HD;         // [waves][16][R]
  float* s_red = s_e + NW * 16 * R;          // [2][waves][R]
  float* s_gm = s_red + 2 * NW * R;          // [T / 16][R]
  uint16_t* s_q = (uint16_t*)(s_gm + (T / 16) * R);    // [T][R]
  int* s_tab = (int*)(s_q + (size_t)T * R);            // [T / b + 1]

  const int sub = lane / LPT, seg = lane % LPT;

  {
    const int nblk = (n_tok + b - 1) >> lb;
    const int32_t* row = A.table + (size_t)g * A.D.maxb + (t0 >> lb);
    for (int i = tid; i < nblk; i += NT) s_tab[i] = row[i];
  }
  // VALU path: every head's q at this lane's dimensions.  MFMA path: A operand of step st: lane =
  // (row lane % 16, dimensions 32 st + 8 (lane / 16) .. + 8); rows without a head are zero.
  typename Row<ESZ>::Q qv[MF ? U : R];
  if constexpr (MF) {
    const int arow = lane & 15, ahead = (arow >> 2) + 4 * (arow & 3);
#pragma unroll
    for (int st = 0; st < U; ++st) {
      // (rows without a head read the last head and are zeroed: a select between values)
      const uint4 t = *(const uint4*)(A.q + ((size_t)g * R + min(ahead, R - 1)) * QROWB + (size_t)st * 64 + (size_t)(lane >> 4) * 16);
      qv[st] = ahead < R ? t : make_uint4(0, 0, 0, 0);
    }
  } else {
#pragma unroll
    for (int hh = 0; hh < R; ++hh) qv[hh] = Row<ESZ>::load_q(A.q + ((size_t)g * R + hh) * QROWB, seg);
  }
  // A head of a kept list must still be as long as the plan took it to be (the record carries that length).
  // A stale plan is an argument error, found here and left in the status word.
  auto argument_error = [&]() { if (A.status[HW_STATUS] == KVC_OK) A.status[HW_STATUS] = KVC_ERR_ARG; };
  if (A.plan && C_now != it.pad[0]) {
    if (tid == 0) argument_error();
    return;
  }
  const bool single = nch == 1;
  int32_t* const arrived = A.self_list ? A.status + meet_word(uniform(word)) : slot_words + it.pbase;
  int32_t* const started = arrived + (A.packed ? 0 : 1);
  const int one_started = A.packed ? 1 << kMeetBits : 1;
  int32_t* const call = &A.items[rec].pad[2];    // where this chunk is called, when all of its head have arrived
  if (!single && tid == 0) {
    publish_i32(call, 0);
    __hip_atomic_fetch_add(started, one_started, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  __syncthreads();

  // One 16-token group = U wavefront loads of 64 pieces each (1 KiB; 512 bytes for 8-bit
  // rows).  With b a multiple of 16 a group lies in one block, so one table lookup serves it
  // and the slots past the end of the head (still inside the block) are masked later, read or not.
  // Otherwise every load looks its block up and tokens past the end re-read the last token.
  const int last = n_tok - 1;
  auto load_group = [&](const char* __restrict__ basep, int grp, Piece (&buf)[U]) {
    if constexpr (B16) {
      const int tk = grp * 16;
      const size_t slot = ((size_t)s_tab[tk >> lb] << lb) + (tk & (b - 1));
      const char* p = basep + slot * ROWB + (size_t)lane * PB;
#pragma unroll
      for (int u = 0; u < U; ++u) {
        // A short item's last block is half empty on average, 7 % of what the item reads: the
        // one-wavefront launch leaves the slots past the head's end unread.  (In the long items'
        // loop the test costs more than the few rows it saves.)
        if (NW == 1 && tk + u * TPI + sub >= n_tok) buf[u] = Row<ESZ>::zero();
        else buf[u] = Row<ESZ>::load(p + (size_t)u * (64 * PB));
      }
    } else {
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int tok = min(grp * 16 + u * TPI + sub, last);
        const size_t slot = ((size_t)s_tab[tok >> lb] << lb) + (tok & (b - 1));
        buf[u] = Row<ESZ>::load(basep + slot * ROWB + (size_t)seg * PB);
      }
    }
  };
  const int ngroups = (n_tok + 15) >> 4;

  float acc[R][EPL];         // VALU path: un-normalised output, this lane's dimensions and tokens
#pragma unroll
  for (int hh = 0; hh < R; ++hh)
#pragma unroll
    for (int k = 0; k < EPL; ++k) acc[hh][k] = 0.0f;
  // MFMA path: P V as v_mfma_f32_16x16x16_bf16 per 16 dimensions (rows = heads, columns =
  // dimensions, k = the 16 tokens of a group).  A probability goes in as parts of 16 bits each, its
  // upper 16 bits, those of the remainder, and, where PARTS is 3, the rest: with two parts the product
  // carries 16 bits of p (one alone misses the output tolerance when one key dominates), with three
  // all 24.
  constexpr int NDT = HD / 16;
  static_assert(!MF || R == 8 || R == 4, "operand rows");
  f32x4_t pacc[MF ? NDT : 1];
#pragma unroll
  for (int i = 0; i < (MF ? NDT : 1); ++i) pacc[i] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
  float m_run[R];            // running max per query head, the same in every lane
  float m_own[OWN], l_own[OWN];  // this lane's head(s): running max and partial sum
#pragma unroll
  for (int hh = 0; hh < R; ++hh) m_run[hh] = -INFINITY;
#pragma unroll
  for (int i = 0; i < OWN; ++i) { m_own[i] = -INFINITY; l_own[i] = 0.0f; }
  const int idx0 = (seg * NV) / LPT;
  float* my_e = s_e + w * 16 * R;
  const bool gm_writer = (lane & 60) == 0;  // lanes 0..3 hold every head between them

  auto process = [&](Piece (&kcur)[U], Piece (&vcur)[U], int grp) {
      float m_new[R];
      bool moved = false;
      if constexpr (MF) {
        // this wavefront's K tile into operand order
        uint4* kt = s_kt + w * 16 * CELLS;
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const int t = u * TPI + sub;
          kt[k_at(t, seg)] = Row<ESZ>::as_bf16x8(kcur[u]);
        }
        const int tl = lane & 15, hrow = lane >> 4;
        float sacc[NVH];
        if constexpr (PARTS == 2) {
          f32x4_t acc4 = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
          for (int st = 0; st < U; ++st) {
            const uint4 kb = kt[k_at(tl, 4 * st + hrow)];
            acc4 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, qv[st]), __builtin_bit_cast(bf16x8_t, kb), acc4, 0, 0, 0);
          }
#pragma unroll
          for (int v = 0; v < NVH; ++v) sacc[v] = acc4[v];
        } else {
          // products of 16 dimensions each, added up in pairs: as near to 64 bits as the plain dot products
          f32x4_t dots[2 * U];
#pragma unroll
          for (int st = 0; st < U; ++st) {
            const uint4 kb = kt[k_at(tl, 4 * st + hrow)];
            const i16x4_t q2[2] = {__builtin_bit_cast(i16x4_t, make_uint2(qv[st].x, qv[st].y)), __builtin_bit_cast(i16x4_t, make_uint2(qv[st].z, qv[st].w))};
            const i16x4_t k2[2] = {__builtin_bit_cast(i16x4_t, make_uint2(kb.x, kb.y)), __builtin_bit_cast(i16x4_t, make_uint2(kb.z, kb.w))};
#pragma unroll
            for (int i = 0; i < 2; ++i)
              dots[2 * st + i] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(q2[i], k2[i], f32x4_t{0.0f, 0.0f, 0.0f, 0.0f}, 0, 0, 0);
          }
#pragma unroll
          for (int v = 0; v < NVH; ++v) {
#pragma unroll
            for (int half = U; half >= 1; half /= 2)
#pragma unroll
              for (int i = 0; i < half; ++i) dots[i][v] += dots[i + half][v];
            sacc[v] = dots[0][v];
          }
        }
        const bool live = grp * 16 + tl < n_tok;
        float x[NVH], gm[NVH], e[NVH];
#pragma unroll
        for (int v = 0; v < NVH; ++v) {
          x[v] = live ? sacc[v] * A.scale_log2 : -INFINITY;
          float m = x[v];   // max over the 16 tokens = over the 16 lanes of this row of lanes
          m = max_xor<1>(m);
          m = max_xor<2>(m);
          m = max_xor<4>(m);
          m = max_xor<8>(m);
          gm[v] = fmaxf(m, m_own[v]);
        }
#pragma unroll
        for (int v = 0; v < NVH; ++v) {
          e[v] = __builtin_amdgcn_exp2f(x[v] - gm[v]);
          l_own[v] = l_own[v] * __builtin_amdgcn_exp2f(m_own[v] - gm[v]) + e[v];
          m_own[v] = gm[v];
        }
#pragma unroll
        for (int v = 0; v < NVH; ++v) {
          const int hh = hrow + 4 * v;
          if (hh < R) {
            my_e[hh * 16 + tl] = e[v];      // [head][token] here: the P V operand reads four tokens of a head
            s_q[(grp * 16 + tl) * R + hh] = (uint16_t)q16(e[v]);
            if (tl == 0) s_gm[grp * R + hh] = gm[v];
          }
        }
#pragma unroll
        for (int hh = 0; hh < R; ++hh) {
          m_new[hh] = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, gm[hh / 4]), 16 * (hh % 4)));
          moved |= m_new[hh] > m_run[hh];
        }
      } else {
        // logits of the group
        float part[NV];
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
          for (int hh = 0; hh < R; ++hh) part[u * R + hh] = Row<ESZ>::dot(kcur[u], qv[hh]);
        Butterfly<NV, LPT / 2>::run(part, lane);
        float gm[PER];
#pragma unroll
        for (int i = 0; i < PER; ++i) {
          const int u = (idx0 + i) / R;
          const int tok = grp * 16 + u * TPI + sub;
          part[i] = tok < n_tok ? part[i] * A.scale_log2 : -INFINITY;
          // max over the group's tokens: the lanes that hold one head differ in lane bits 2..5
          float m = part[i];
          m = max_xor<4>(m);
          m = max_xor<8>(m);
          m = max_xor<16>(m);
          m = max_xor<32>(m);
          gm[i] = fmaxf(m, m_own[i]);
        }
        // exp of the group against the new running max; partial sums rescaled
#pragma unroll
        for (int i = 0; i < PER; ++i) {
          const int idx = idx0 + i;
          const int u = idx / R, hh = idx % R;
          const int tl = u * TPI + sub;
          const float e = __builtin_amdgcn_exp2f(part[i] - gm[i]);
          l_own[i] = l_own[i] * __builtin_amdgcn_exp2f(m_own[i] - gm[i]) + e;
          m_own[i] = gm[i];
          my_e[MF ? hh * 16 + tl : tl * R + hh] = e;   // [head][token] for the matrix-core P V
          s_q[(grp * 16 + tl) * R + hh] = (uint16_t)q16(e);
          if (gm_writer) s_gm[grp * R + hh] = gm[i];
        }
        // new running max of every head, read from the lane that owns it
#pragma unroll
        for (int hh = 0; hh < R; ++hh) {
          m_new[hh] = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, gm[hh % PER]), (hh * 4) / R));
          moved |= m_new[hh] > m_run[hh];
        }
      }
      const bool tail = B16 && grp * 16 + 16 > n_tok;
      if constexpr (MF) {
        if (moved) {
          // this lane's product rows 4 (lane / 16) + v belong to heads 4 ((lane / 16) % 2) + v (PROWS = 4: to heads v)
          const bool upper = (lane & 16) != 0;
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            const float a_lo = __builtin_amdgcn_exp2f(m_run[v] - m_new[v]);
            const float a_hi = R > 4 ? __builtin_amdgcn_exp2f(m_run[(4 + v) % R] - m_new[(4 + v) % R]) : a_lo;
            const float a = upper && R > 4 ? a_hi : a_lo;
#pragma unroll
            for (int dt = 0; dt < NDT; ++dt) pacc[dt][v] *= a;
          }
#pragma unroll
          for (int hh = 0; hh < R; ++hh) m_run[hh] = m_new[hh];
        }
        // The K tile has been consumed: its bytes take the V tile, row-major [token][d] in bf16.
        uint4* vt = s_kt + w * 16 * CELLS;
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const int t = u * TPI + sub;
          const bool dead = tail && grp * 16 + t >= n_tok;   // empty slot: may hold anything
          vt[t * CELLS + (seg ^ v_swizzle(t))] = Row<ESZ>::as_bf16x8(dead ? Row<ESZ>::zero() : vcur[u]);
        }
        // A operand: lane = (row lane % 16, tokens 4 (lane / 16) .. + 3), row = part * PROWS + head
        const int rho = lane & 15, kap = lane >> 4, part = rho / PROWS;
        float4 pe = *(const float4*)(my_e + (rho & (R - 1)) * 16 + 4 * kap);
        if (R < 8 && (rho % PROWS >= R || part >= PARTS)) pe = make_float4(0.0f, 0.0f, 0.0f, 0.0f);   // rows without a head or a part
        auto top16 = [](float p) { return __uint_as_float(__float_as_uint(p) & 0xffff0000u); };
        // With three parts of 16-bit rows, one that is zero (a probability of few bits) goes in as the least
        // normal number: zero times an infinite value would be NaN, where the plain product is infinite.
        // Next to the finite ones it adds 2^-126 of a value, nothing.
        auto live_part = [](float p) { return PARTS == 3 && ESZ == 2 ? fmaxf(p, 0x1p-126f) : p; };
        auto part_of = [&](float p) {   // a float whose upper 16 bits are this row's part of p
          const float mid = p - top16(p);   // exact
          if (PROWS == 4) return part == 0 ? p : part == 1 ? mid : mid - top16(mid);
          return live_part(part == 0 ? p : mid);
        };
        auto pack = [](float p0, float p1, float p2, float p3) {
          const uint2 u = make_uint2(__builtin_amdgcn_perm(__float_as_uint(p1), __float_as_uint(p0), 0x07060302u),
                                     __builtin_amdgcn_perm(__float_as_uint(p3), __float_as_uint(p2), 0x07060302u));
          return __builtin_bit_cast(i16x4_t, u);
        };
        const i16x4_t aop = pack(part_of(pe.x), part_of(pe.y), part_of(pe.z), part_of(pe.w));
        // the third part of eight heads does not fit: a second operand, the same rows
        i16x4_t aop3 = {0, 0, 0, 0};
        if constexpr (PARTS == 3 && R == 8) {
          auto last = [&](float p) { const float mid = p - top16(p); return live_part(part == 0 ? mid - top16(mid) : 0.0f); };
          aop3 = pack(last(pe.x), last(pe.y), last(pe.z), last(pe.w));
        }
        // B operand of dimension tile dt: lane = (column lane % 16, tokens 4 (lane / 16) .. + 3).
        // The transposing read delivers it when lane j of a group of 16 points at token
        // 4 (lane / 16) + j / 4, dimensions 16 dt + 4 (j % 4) .. + 3.
        const int tt = 4 * kap + (rho >> 2);
        const char* vrow = (const char*)vt + tt * (HD * 2) + 8 * (rho & 1);
        const int csw = v_swizzle(tt), chalf = (rho & 3) >> 1;
#pragma unroll
        for (int dt = 0; dt < NDT; ++dt) {
          const int c = (2 * dt + chalf) ^ csw;
          const i16x4_t bop = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
              (i16x4_t __attribute__((address_space(3)))*)(vrow + c * 16));
          pacc[dt] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(aop, bop, pacc[dt], 0, 0, 0);
          if constexpr (PARTS == 3 && R == 8) pacc[dt] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(aop3, bop, pacc[dt], 0, 0, 0);
        }
      } else {
        if (moved) {
#pragma unroll
          for (int hh = 0; hh < R; ++hh) {
            const float alpha = __builtin_amdgcn_exp2f(m_run[hh] - m_new[hh]);
#pragma unroll
            for (int k = 0; k < EPL; ++k) acc[hh][k] *= alpha;
            m_run[hh] = m_new[hh];
          }
        }
        // acc += p * v
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const int tl = u * TPI + sub;
          if (tail && grp * 16 + tl >= n_tok) vcur[u] = Row<ESZ>::zero();  // empty slot: may hold anything
          float vf[EPL];
          Row<ESZ>::widen(vcur[u], vf);
#pragma unroll
          for (int hh = 0; hh < R; ++hh) {
            const float p = my_e[tl * R + hh];
#pragma unroll
            for (int k = 0; k < EPL; ++k) acc[hh][k] = fmaf(p, vf[k], acc[hh][k]);
          }
        }
      }
  };
  {
    // DEPTH register buffers used in rotation (the loop is unrolled DEPTH times so that no
    // buffer is ever copied): DEPTH - 1 groups in flight behind the one being worked on
    Piece kb[DEPTH][U], vb[DEPTH][U];
#pragma unroll
    for (int st = 0; st < DEPTH - 1; ++st) {
      const int g2 = w + st * NW;
      if (g2 < ngroups) { load_group(A.kc, g2, kb[st]); load_group(A.vc, g2, vb[st]); }
    }
    for (int base = w; base < ngroups; base += DEPTH * NW) {
#pragma unroll
      for (int st = 0; st < DEPTH; ++st) {
        const int grp = base + st * NW;
        if (grp >= ngroups) break;
        const int gp = grp + (DEPTH - 1) * NW;
        if (gp < ngroups) {
          load_group(A.kc, gp, kb[(st + DEPTH - 1) % DEPTH]);
          load_group(A.vc, gp, vb[(st + DEPTH - 1) % DEPTH]);
        }
        process(kb[st], vb[st], grp);
      }
    }
  }
  // (the first look for chunks that have not started: on its way while the wavefronts merge)
  uint32_t seen = 0;
  if (!single && tid == 0) seen = (uint32_t)published_i32(started);
  // ---- merge: token groups of one wavefront, then the wavefronts ----
  if constexpr (MF) {
#pragma unroll
    for (int v = 0; v < NVH; ++v) {   // sums over the 16 token lanes of a row of lanes
      float l = l_own[v];
      l = sum_xor<1>(l);
      l = sum_xor<2>(l);
      l = sum_xor<4>(l);
      l_own[v] = sum_xor<8>(l);
    }
    if ((lane & 15) == 0) {
#pragma unroll
      for (int v = 0; v < NVH; ++v) {
        const int hh = (lane >> 4) + 4 * v;
        if (hh < R) {
          s_red[w * R + hh] = m_own[v];
          s_red[(NW + w) * R + hh] = l_own[v];
        }
      }
    }
  } else {
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      float l = l_own[i];
      l = sum_xor<4>(l);
      l = sum_xor<8>(l);
      l = sum_xor<16>(l);
      l_own[i] = sum_xor<32>(l);
    }
    if (lane < 4) {
#pragma unroll
      for (int i = 0; i < PER; ++i) {
        const int hh = (idx0 + i) % R;
        if ((hh * 4) / R == lane) {
          s_red[w * R + hh] = m_own[i];
          s_red[(NW + w) * R + hh] = l_own[i];
        }
      }
    }
  }
  if constexpr (MF) {
    // rows PROWS apart of the product are the parts of a head: rows h and h + 8 are 32 lanes apart
#pragma unroll
    for (int dt = 0; dt < NDT; ++dt)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        float a = sum_xor<32>(pacc[dt][v]);
        if (PROWS == 4) a = sum_xor<16>(a);
        if (lane < (R > 4 ? 32 : 16)) s_acc[(w * RW + 4 * (lane >> 4) + v) * HD + 16 * dt + (lane & 15)] = a;
      }
  } else {
#pragma unroll
    for (int hh = 0; hh < R; ++hh)   // the lanes that hold the same dimensions
#pragma unroll
      for (int k = 0; k < EPL; ++k) {
        if constexpr (LPT <= 4) acc[hh][k] = sum_xor<4>(acc[hh][k]);
        if constexpr (LPT <= 8) acc[hh][k] = sum_xor<8>(acc[hh][k]);
        if constexpr (LPT <= 16) acc[hh][k] = sum_xor<16>(acc[hh][k]);
        acc[hh][k] = sum_xor<32>(acc[hh][k]);
      }
    if (sub == 0) {
#pragma unroll
      for (int hh = 0; hh < R; ++hh)
#pragma unroll
        for (int k = 0; k < EPL; ++k) s_acc[(w * RW + hh) * HD + seg * EPL + k] = acc[hh][k];
    }
  }
  // (the first wavefront's exps have been used: its place serves for a word to all)
  int* s_say = (int*)s_e;
  __syncthreads();

  // chunk max and sum per head from the wavefronts' pairs
  float cm[R], cl[R], wsc[NW][R];
#pragma unroll
  for (int hh = 0; hh < R; ++hh) {
    float m = s_red[hh];
#pragma unroll
    for (int ww = 1; ww < NW; ++ww) m = fmaxf(m, s_red[ww * R + hh]);
    float l = 0.0f;
#pragma unroll
    for (int ww = 0; ww < NW; ++ww) {
      wsc[ww][hh] = __builtin_amdgcn_exp2f(s_red[ww * R + hh] - m);
      l += s_red[(NW + ww) * R + hh] * wsc[ww][hh];
    }
    cm[hh] = m;
    cl[hh] = l;
  }
  const int ci = t0 / Tc;                                // this chunk of the head,
  const size_t pslot = (size_t)it.pbase + (size_t)ci;    // and its partial-result slot
  // a wavefront per query head
#pragma unroll
  for (int hh = 0; hh < R; ++hh) {
    if (NW > 1 && hh % NW != w) continue;
    for (int k = 2 * lane; k < HD; k += 128) {
      float s0 = 0.0f, s1 = 0.0f;
#pragma unroll
      for (int ww = 0; ww < NW; ++ww) {
        const float2 v = *(const float2*)&s_acc[(ww * RW + hh) * HD + k];
        s0 += v.x * wsc[ww][hh];
        s1 += v.y * wsc[ww][hh];
      }
      if (single) {
        const f32x2_t o = {s0 / cl[hh], s1 / cl[hh]};
        __builtin_nontemporal_store(o, (f32x2_t*)&A.out[((size_t)g * R + hh) * HD + k]);
      } else {
        publish_u64(&A.part_acc[(pslot * R + hh) * HD + k], (uint64_t)__float_as_uint(s0) | (uint64_t)__float_as_uint(s1) << 32);
      }
    }
  }
  if (!single && tid == 0) {
    auto all = [&]() { return (A.packed ? seen >> kMeetBits : seen) == (uint32_t)nch; };
    for (int looks = 1; looks < kMeetStarts && !all(); ++looks) seen = (uint32_t)published_i32(started);
    s_say[0] = all();
#pragma unroll
    for (int hh = 0; hh < R; ++hh)   // (the sum's sign says that the chunk does not wait)
      publish_u64(&A.part_ml[(pslot * R + hh) * 2], (uint64_t)__float_as_uint(cm[hh]) |
                                                        (uint64_t)((__float_as_uint(cl[hh]) & 0x7fffffffu) | (all() ? 0u : 0x80000000u)) << 32);
  }
  if (single && !A.accumulate) return;
  // The stored 16-bit value of a KV times 2^(its group's running max - chunk max) is the exp of
  // its logit against the chunk max; for a head of one chunk, divided by the sum, its
  // probability.  That factor is the same for the 16 tokens of a group: formed once, in place.
  if (A.accumulate || !single) {
    for (int i = tid; i < ngroups * R; i += NT) {
      const int hh = i % R;
      float f = 0.0f;
#pragma unroll
      for (int h2 = 0; h2 < R; ++h2)
        if (h2 == hh) f = __builtin_amdgcn_exp2f(s_gm[i] - cm[h2]) * (single ? 1.0f / cl[h2] : 1.0f) * (1.0f / 65535.0f);
      s_gm[i] = f;
    }
    __syncthreads();
  }
  auto each_token = [&](auto use) {
    for (int tok = tid; tok < n_tok; tok += NT) {
      const size_t slot = ((size_t)s_tab[tok >> lb] << lb) + (tok & (b - 1));
      float e[R];
#pragma unroll
      for (int hh = 0; hh < R; ++hh) e[hh] = (float)s_q[tok * R + hh] * s_gm[(tok >> 4) * R + hh];
      use(slot, e);
    }
  };
  auto add = [&](size_t slot, float (&e)[R]) {
    float inc = 0.0f;
#pragma unroll
    for (int hh = 0; hh < R; ++hh) inc += A.D.mode == KVC_L2 ? e[hh] * e[hh] : e[hh];
    // one writer per slot in a launch, so the hardware add gives the same bits as load-add-store
    unsafeAtomicAdd(&A.metric[slot], inc);
  };
  if (single) {
    each_token(add);
    return;
  }
  if constexpr (NW == 4) {   // (a short item is a whole head)
    const bool waits = s_say[0];
    if (A.accumulate && !waits) each_token([&](size_t slot, float (&e)[R]) { exps_publish<R>(A.stash, slot, e); });
    publish_wait();
    __syncthreads();
    // (what the first wavefront finds on its way is looked at in the end, away from those that wait)
    uint32_t was = 0, begun = 1;
    bool came = true;
    if (w == 0) {
      if (lane == 0) was = (uint32_t)__hip_atomic_fetch_add(arrived, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      was = (uint32_t)__builtin_amdgcn_readfirstlane((int)was);
      begun = A.packed ? was >> kMeetBits : (uint32_t)nch;
      if (A.packed) was &= kMeetMost;
      bool go = waits;
      if (was == (uint32_t)nch - 1) {
        for (int c = lane; c < nch; c += 64)
          if (c != ci) publish_i32(call + (c - ci) * (int)(sizeof(DecodeItem) / 4), 1);
        if (lane == 0) {
          if (!A.packed) __hip_atomic_fetch_add(arrived, -nch, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          __hip_atomic_fetch_add(started, A.packed ? -nch * (one_started + 1) : -nch, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        if (!waits) {   // somebody has to
          bool one = false;
          for (int c = lane; c < nch; c += 64) one |= published_i32((const int32_t*)A.part_ml + ((size_t)it.pbase + c) * R * 2 + 1) >= 0;
          came = __any(one);
        }
      } else if (waits) {
        for (int looks = 0; !published_i32(call); ++looks)
          if (looks == kMeetLooks) { go = came = false; break; }
      }
      if (lane == 0) s_say[1] = go;
    }
    __syncthreads();
    auto look_back = [&]() {
      const uint32_t most = (uint32_t)nch;
      if (w == 0 && (was >= begun || begun > most || (A.packed ? seen >> kMeetBits : seen) > most || !came)) argument_error();
    };
    if (!s_say[1]) { look_back(); return; }   // (its part is out: the others see to it)
    // ---- every chunk of the head has arrived ----
    const float* ml = A.part_ml + (size_t)it.pbase * R * 2;
    const float* accs = A.part_acc + (size_t)it.pbase * R * HD;
    // A chunk's share of the head's output, in pairs of dimensions: a wavefront has at most 64 of them (the
    // head has two chunks at least), lanes on pairs, the chunks spread over the lanes that share one.
    // The first four of a lane are asked for ahead of the max and sum.
    constexpr int PAIRS = R * HD / 2, AHEAD = 4;
    static_assert((PAIRS + 1) / 2 <= 64 * NW, "a wavefront's share of the output");
    struct Share { int i, hh, ne, lnp; uint64_t v[AHEAD]; };
    auto share_ask = [&](int c, Share& o) {
      const int e0 = (int)((unsigned)(PAIRS * c) / (unsigned)nch), e1 = (int)((unsigned)(PAIRS * (c + 1)) / (unsigned)nch);
      const int per = (e1 - e0 + NW - 1) / NW, w0 = e0 + w * per;
      o.ne = max(0, min(per, e1 - w0));
      o.lnp = o.ne > 1 ? 32 - __builtin_clz(o.ne - 1) : 0;
      o.i = min(2 * (w0 + min(lane & ((1 << o.lnp) - 1), max(o.ne, 1) - 1)), 2 * PAIRS - 2);
      o.hh = o.i / HD;
#pragma unroll
      for (int k = 0; k < AHEAD; ++k) {
        const int cc = (lane >> o.lnp) + k * (64 >> o.lnp);
        o.v[k] = o.ne && cc < nch ? published_u64(accs + (size_t)cc * R * HD + o.i) : 0;
      }
    };
    Share own;
    share_ask(ci, own);
    // The chunks' pairs go into LDS (a word of a line that every chunk of the head reads costs each of them
    // ~5 ns: no wavefront asks for one that another has), and the head's max and sum come from there, a
    // wavefront per query head, lane = chunk.  The chunks that have left are shared out among those that
    // waited (one at least: the chunk that started last).
    constexpr int kPairs = NW * RW * HD / 2;   // pairs that the wavefronts' outputs leave room for
    uint64_t* s_ml = (uint64_t*)s_acc;
    float* s_m = s_red;                     // [R] max, [R] 1 / sum
    int* s_who = s_say + 2;                 // chunks that waited: in front of this one, and in all
    float m_all[(R + NW - 1) / NW], l_all[(R + NW - 1) / NW];
    int rank = 0, stay = 0;
    constexpr int kRoom = kPairs / R;       // chunks at a time
    for (int base = 0; base < nch; base += kRoom) {
      const int n = min(kRoom, nch - base);
      if (base) __syncthreads();
      for (int i = tid; i < n * R; i += NT) s_ml[i] = published_u64(ml + ((size_t)base * R + i) * 2);
      __syncthreads();
#pragma unroll
      for (int z = 0; z < (R + NW - 1) / NW; ++z) {
        const int hh = w + z * NW;
        if (hh >= R) break;
        float m = base ? m_all[z] : -INFINITY, l = base ? l_all[z] : 0.0f;
        for (int c0 = 0; c0 < n; c0 += 64) {
          const int cc = c0 + lane;
          const uint64_t v = cc < n ? s_ml[cc * R + hh] : (uint64_t)0xff800000u;
          const float vm = __uint_as_float((uint32_t)v), vl = __uint_as_float((uint32_t)(v >> 32) & 0x7fffffffu);
          const float nm = fmaxf(m, wave_max_f(vm));
          l = (base + c0 ? l * __builtin_amdgcn_exp2f(m - nm) : 0.0f) + wave_sum_f(cc < n ? vl * __builtin_amdgcn_exp2f(vm - nm) : 0.0f);
          m = nm;
          if (hh == 0) {
            const unsigned long long in = __ballot(cc < n && !(v >> 63));
            const int to = ci - base - c0;   // this chunk's lane
            stay += __popcll(in);
            rank += to >= 64 ? __popcll(in) : to > 0 ? __popcll(in & ((1ull << to) - 1ull)) : 0;
          }
        }
        m_all[z] = m;
        l_all[z] = l;
      }
    }
#pragma unroll
    for (int z = 0; z < (R + NW - 1) / NW; ++z)
      if (lane == 0 && w + z * NW < R) { s_m[w + z * NW] = m_all[z]; s_m[R + w + z * NW] = 1.0f / l_all[z]; }
    if (tid == 0) { s_who[0] = rank; s_who[1] = stay; }
    __syncthreads();
    rank = s_who[0];
    stay = s_who[1];
    const bool kept = nch <= kRoom;         // every pair is still in LDS
    auto max_of = [&](int c, int hh) {
      return kept ? __uint_as_float((uint32_t)s_ml[c * R + hh]) : __int_as_float(published_i32((const int32_t*)ml + ((size_t)c * R + hh) * 2));
    };
    auto share_put = [&](const Share& o) {
      if (!o.ne) return;
      const float top = s_m[o.hh], il = s_m[R + o.hh];
      float s0 = 0.0f, s1 = 0.0f;
      auto term = [&](int cc, uint64_t v) {
        const float wt = __builtin_amdgcn_exp2f(max_of(cc, o.hh) - top);
        s0 = fmaf(__uint_as_float((uint32_t)v), wt, s0);
        s1 = fmaf(__uint_as_float((uint32_t)(v >> 32)), wt, s1);
      };
#pragma unroll
      for (int k = 0; k < AHEAD; ++k) {
        const int cc = (lane >> o.lnp) + k * (64 >> o.lnp);
        if (cc < nch) term(cc, o.v[k]);
      }
      for (int cc = (lane >> o.lnp) + AHEAD * (64 >> o.lnp); cc < nch; cc += 64 >> o.lnp)
        term(cc, published_u64(accs + (size_t)cc * R * HD + o.i));
      for (int k = 1 << o.lnp; k < 64; k <<= 1) { s0 += __shfl_xor(s0, k); s1 += __shfl_xor(s1, k); }
      if (lane < o.ne) *(float2*)&A.out[(size_t)g * R * HD + o.i] = make_float2(s0 * il, s1 * il);
    };
    float wgt[R];
    auto weigh = [&](size_t slot, float (&e)[R]) {
#pragma unroll
      for (int hh = 0; hh < R; ++hh) e[hh] *= wgt[hh];
      add(slot, e);
    };
    if (A.accumulate) {
#pragma unroll
      for (int hh = 0; hh < R; ++hh) wgt[hh] = __builtin_amdgcn_exp2f(cm[hh] - s_m[hh]) * s_m[R + hh];
      each_token(weigh);
    }
    share_put(own);
    look_back();
    if (stay == nch) return;
    // chunks that did not wait: every stay-th of them from this one's rank on.  Their marks are looked at 64 at a time, lane
    // = chunk (one after the other from memory, 8-bit rows, d = 128, r = 8: one head of 4 million KVs 1059 us, 711 so, 16 of
    // 100417 140 and 122; 16-bit, two heads of 2 million 652 and 542).
    const int C = A.ctx[g];
    int next = rank, c0 = -64;   // of those to come, the one that is this chunk's; the chunks being looked at,
    unsigned long long gone = 0; // and those of them that left
    for (;;) {
      int here = __popcll(gone);
      while (next >= here) {
        next -= here;
        c0 += 64;
        if (c0 >= nch) return;
        const int cc = c0 + lane;
        bool left = false;
        if (cc < nch) left = kept ? (s_ml[cc * R] >> 63) != 0 : published_i32((const int32_t*)ml + (size_t)cc * R * 2 + 1) < 0;
        gone = __ballot(left);
        here = __popcll(gone);
      }
      for (; next; --next) gone &= gone - 1;
      const int c = c0 + __builtin_ctzll(gone);
      gone &= gone - 1;
      next = stay - 1;
      share_ask(c, own);
      share_put(own);
      if (!A.accumulate) continue;
      const int32_t* row = A.table + (size_t)g * A.D.maxb;
#pragma unroll
      for (int hh = 0; hh < R; ++hh) wgt[hh] = __builtin_amdgcn_exp2f(max_of(c, hh) - s_m[hh]) * s_m[R + hh];
      for (int j = c * Tc + tid; j < min(C, c * Tc + Tc); j += NT) {
        const size_t slot = ((size_t)row[j >> lb] << lb) + (j & (b - 1));
        float e[R];
        exps_published<R>(A.stash, slot, e);
        weigh(slot, e);
      }
    }
  }
}

// Fallback for shapes the tiled kernel does not cover (blocks of more than 64 tokens, any d that
// is a multiple of 16 bytes, any r <= 16): one workgroup per head instance, logits
// kept in the workspace.  Correct, not fast.
__global__ void __launch_bounds__(256) decode_generic_kernel(DecodeArgs A) {
  const int gi = blockIdx.x;
  const int g = sel_to_g(A.D, A.l0, A.nl, gi);
  const int R = A.D.r, HD = A.D.d, b = A.D.b;
  const int C = A.ctx[g];
  if (C == 0) {  // a head with no KV: zero output rows
    float* o = A.out + (size_t)g * R * HD;
    for (int i = threadIdx.x; i < R * HD; i += 256) o[i] = 0.0f;
    return;
  }
  extern __shared__ __align__(16) char smem_raw[];
  float* s_q = (float*)smem_raw;      // [R][HD]
  float* s_red = s_q + R * HD;        // [4][16]
  float* s_ml = s_red + 4 * 16;       // [2][16]
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int dt = A.D.dtype;
  const size_t rowb = (size_t)HD * kv_esz(dt), qrowb = (size_t)HD * q_esz(dt);
  auto elem = [&](const char* base, size_t row_off, int k) -> float {
    if (dt == KVC_BF16) return bf16_to_f32(((const uint16_t*)(base + row_off))[k]);
    if (dt == KVC_F32) return ((const float*)(base + row_off))[k];
    return __builtin_amdgcn_cvt_pk_f32_fp8((int)((const uint8_t*)(base + row_off))[k], false)[0];
  };
  for (int i = tid; i < R * HD; i += 256) {
    const char* qr = A.q + ((size_t)g * R + i / HD) * qrowb;
    s_q[i] = dt == KVC_F32 ? ((const float*)qr)[i % HD] : bf16_to_f32(((const uint16_t*)qr)[i % HD]);
  }
  __syncthreads();
  const int32_t* row = A.table + (size_t)g * A.D.maxb;
  float mx[16];
  for (int hh = 0; hh < R; ++hh) mx[hh] = -INFINITY;
  for (int j = tid; j < C; j += 256) {
    const size_t slot = (size_t)row[j / b] * b + (j % b);
    for (int hh = 0; hh < R; ++hh) {
      float s = 0.0f;
      for (int k = 0; k < HD; ++k) s = fmaf(s_q[hh * HD + k], elem(A.kc, slot * rowb, k), s);
      s *= A.scale_log2;
      A.stash[slot * R + hh] = s;
      mx[hh] = fmaxf(mx[hh], s);
    }
  }
  for (int hh = 0; hh < R; ++hh) {
    const float m = wave_max_f(mx[hh]);
    if (lane == 0) s_red[w * 16 + hh] = m;
  }
  __syncthreads();
  if (tid < R) s_ml[tid] = fmaxf(fmaxf(s_red[tid], s_red[16 + tid]), fmaxf(s_red[32 + tid], s_red[48 + tid]));
  __syncthreads();
  float sm[16];
  for (int hh = 0; hh < R; ++hh) sm[hh] = 0.0f;
  for (int j = tid; j < C; j += 256) {
    const size_t slot = (size_t)row[j / b] * b + (j % b);
    for (int hh = 0; hh < R; ++hh) {
      const float e = __builtin_amdgcn_exp2f(A.stash[slot * R + hh] - s_ml[hh]);
      A.stash[slot * R + hh] = e;
      sm[hh] += e;
    }
  }
  for (int hh = 0; hh < R; ++hh) {
    const float t = wave_sum_f(sm[hh]);
    if (lane == 0) s_red[w * 16 + hh] = t;
  }
  __syncthreads();
  if (tid < R) s_ml[16 + tid] = 1.0f / (s_red[tid] + s_red[16 + tid] + s_red[32 + tid] + s_red[48 + tid]);
  __syncthreads();  // also orders the stash writes above before the reads below
  for (int i = tid; i < R * HD; i += 256) {
    const int hh = i / HD, k = i % HD;
    float s = 0.0f;
    for (int j = 0; j < C; ++j) {
      const size_t slot = (size_t)row[j / b] * b + (j % b);
      s = fmaf(A.stash[slot * R + hh], elem(A.vc, slot * rowb, k), s);
    }
    A.out[(size_t)g * R * HD + i] = s * s_ml[16 + hh];
  }
  if (A.accumulate) {
    for (int j = tid; j < C; j += 256) {
      const size_t slot = (size_t)row[j / b] * b + (j % b);
      float inc = 0.0f;
      for (int hh = 0; hh < R; ++hh) {
        const float p = A.stash[slot * R + hh] * s_ml[16 + hh];
        inc += A.D.mode == KVC_L2 ? p * p : p;
      }
      A.metric[slot] += inc;
    }
  }
}

// What the runtime is told and says about the kernel of four wavefronts, by whether blocks are of 16 tokens or more.
template <int ESZ, int HD, int R>
struct TiledKernel {
  static inline LdsLimit limit[2];
  static inline std::atomic<uint64_t> shared[2];   // workgroups that share a CU (its last byte), and with how much LDS
  static auto of(bool b16) { return b16 ? decode_chunk_kernel<ESZ, HD, R, true, 4> : decode_chunk_kernel<ESZ, HD, R, false, 4>; }
  static int places(bool b16, size_t lds) {   // of the whole chip; no bound when the runtime does not say
    uint64_t v = shared[b16].load(std::memory_order_relaxed);
    if (v >> 8 != lds) {
      int n = 0;
      if (limit[b16].need(lds, of(b16)) != KVC_OK ||
          hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, of(b16), kDecodeThreads, lds) != hipSuccess || n <= 0) return 0x7fffffff;
      v = (uint64_t)lds << 8 | (uint64_t)(n < 255 ? n : 255);
      shared[b16].store(v, std::memory_order_relaxed);
    }
    return (int)(v & 255) * kCus;
  }
};

template <int ESZ, int HD>
static int tiled_places(const Dims& D, size_t lds) {
  const bool b16 = D.b % 16 == 0;
  switch (D.r) {
    case 1: return TiledKernel<ESZ, HD, 1>::places(b16, lds);
    case 2: return TiledKernel<ESZ, HD, 2>::places(b16, lds);
    case 4: return TiledKernel<ESZ, HD, 4>::places(b16, lds);
    case 8: return TiledKernel<ESZ, HD, 8>::places(b16, lds);
  }
  return 0x7fffffff;
}

template <int ESZ, int HD, int R>
static int launch_tiled(const DecodeArgs& A, int grid, size_t lds, int grid_short, hipStream_t s) {
  const auto kern = TiledKernel<ESZ, HD, R>::of(A.D.b % 16 == 0);
  auto kern_short = (A.D.b % 16 == 0) ? decode_chunk_kernel<ESZ, HD, R, true, 1> : decode_chunk_kernel<ESZ, HD, R, false, 1>;
  bool mf_short = decode_uses_mfma(ESZ, R, HD);
  if constexpr (ESZ == 1 && HD == 128 && R == 4)
    // short items in blocks of one token keep the plain ALUs, where a fourth wavefront fits a SIMD (152 registers
    // against 119; 16384 heads of up to 120 tokens 132 us and 117, of up to 300 243 and 229).  In blocks of two to
    // eight they are slower by a tenth up to 30 tokens only, and faster by 1 to 9 % from 300 on.
    if (A.D.b == 1) { kern_short = decode_chunk_kernel<ESZ, HD, R, false, 1, false>; mf_short = false; }
  ProfilePair* pp = claim_profile_pair();
  if (pp) KVC_HIP(hipEventRecord(pp->a0, s));
  {  // above the default cap the kernel must be told how much it may take (per instantiation and device)
    const int rc = TiledKernel<ESZ, HD, R>::limit[A.D.b % 16 == 0].need(lds, kern);
    if (rc != KVC_OK) return rc;
  }
  hipLaunchKernelGGL(kern, dim3(grid), dim3(kDecodeThreads), lds, s, A);
  KVC_LAUNCH_CHECK();
  if (pp) { KVC_HIP(hipEventRecord(pp->a1, s)); KVC_HIP(hipEventRecord(pp->s0, s)); }
  if (A.short_class < 16) {
    hipLaunchKernelGGL(kern_short, dim3(grid_short), dim3(64),
                       decode_lds_bytes(A.Ts, R, HD, A.D.b, 1, mf_short), s, A);
    KVC_LAUNCH_CHECK();
  }
  if (pp) KVC_HIP(hipEventRecord(pp->s1, s));
  return KVC_OK;
}

template <int ESZ, int HD>
static int launch_tiled_r(const DecodeArgs& A, int grid, size_t lds, int grid_short, hipStream_t s) {
  switch (A.D.r) {
    case 1: return launch_tiled<ESZ, HD, 1>(A, grid, lds, grid_short, s);
    case 2: return launch_tiled<ESZ, HD, 2>(A, grid, lds, grid_short, s);
    case 4: return launch_tiled<ESZ, HD, 4>(A, grid, lds, grid_short, s);
    case 8: return launch_tiled<ESZ, HD, 8>(A, grid, lds, grid_short, s);
  }
  return KVC_ERR_UNSUPPORTED;
}

constexpr size_t kLdsLimit = 160 * 1024;  // gfx950: 160 KiB of LDS per workgroup
constexpr size_t kLdsUnit = 1280, kLdsUnits = kLdsLimit / kLdsUnit;   // handed out in these

// Chunk length of large calls, before the LDS of a CU is shared out among more than two workgroups.
static int default_chunk(const Dims& D) { return D.r >= 8 ? 3456 : 6144; }

// Whether the tiled kernels cover this shape, and with which chunk length and LDS size.
static bool choose_chunk(const Dims& D, int gsel, int* T_out, size_t* lds_out, bool* small_call = nullptr,
                         bool* on_device = nullptr) {
  const int esz = kv_esz(D.dtype);
  const int lpt = D.d * esz / 16;
  const int tpi = (lpt >= 1 && lpt <= 64) ? 64 / lpt : 0;
  // (blocks shorter than the tokens one wavefront load covers are fine: off the 16-token-block
  // fast path every token of a load looks its own block up)
  bool tiled = (D.r == 1 || D.r == 2 || D.r == 4 || D.r == 8) && (D.d == 64 || D.d == 128) &&
               tpi >= 1 && 64 % D.b == 0;
  if (!tiled) return false;
  // default: a chunk that lets two workgroups share a CU (at r = 8, d = 128, 16-bit rows: 3456
  // tokens x 16 bytes of exps + the rest = 81 764 of the 81 920 bytes a half CU has), or as many as
  // decode_groups says
  const int knob = g_chunk_tokens.load(std::memory_order_relaxed);
  const bool mf = decode_uses_mfma(esz, D.r, D.d);   // a per-wavefront operand tile in LDS
  const int groups = decode_groups(esz, D.d, D.r, D.b % 16 == 0);
  int T = knob ? knob : default_chunk(D);
  const int T_two = T;
  int T_fits = T;
  if (!knob && groups > 2)
    while (T_fits > 1024 && decode_lds_bytes(T_fits, D.r, D.d, D.b, kDecodeWaves, mf) > kLdsUnits / groups * kLdsUnit) T_fits -= 64;
  // ... but not where rows then need two chunks that do not all have places, and whole ones do (512 heads of 3210 KVs,
  // r = 8, d = 128, fp8: 109 us in halves, whole 100; 512 of 3300, d = 64, bf16: 104 and 85)
  const long long row_tokens = (long long)D.maxb * D.b;
  if (row_tokens > T_fits && row_tokens <= T_two && gsel <= 2 * kCus && 2 * gsel > groups * kCus) T_fits = T_two;
  bool shrunk = false, device_side = false;
  if (!knob) {
    // a call over few head instances (one layer at a time) has too few long chunks to fill the
    // chip: shorten them until full rows would give a few thousand work items
    // (counted from the length that two workgroups leave each other, also where more share a CU: counted
    // from the shorter one, 960 heads of 1250 KVs and rows of 20000, r = 8, d = 128, fp8, took the two
    // launches of a large call, 121 us where one takes 80)
    const long long want_items = 6144;
    // (halved and rounded up to whole 64-token strips: a chunk starts on a block boundary)
    // (over a thousand heads fill the chip whole: their chunks only have to even out unequal lengths, and
    // shorter ones have to meet, so they stay at 768 or more (896 with eight query heads).  2990
    // heads of 609 KVs, r = 4, 16-bit rows: 317 us in chunks of 192, whole 173; 2048 of up to 600, r = 8, 174 in
    // chunks of 448, 129 whole, 8-bit 121 and 80; of 2000 and 4000 level)
    const int least = gsel > kSmallWorklistHeads ? 768 : 256;
    auto half = [&]() { return ((T / 2) + 63) & ~63; };
    while (half() >= least && (long long)gsel * (((long long)D.maxb * D.b + T - 1) / T) < want_items) T = half();
    shrunk = T < T_two;
    T = T < T_fits ? T : T_fits;
    // ... unless the one-launch work list serves the call: it sees the lengths themselves, not
    // just what the tables have room for, and picks the length (at most the default) on the device
    if (shrunk && gsel <= kSmallWorklistHeads) { T = T_fits; device_side = true; }
  }
  // the default is sized so that two workgroups share a CU's LDS with blocks of 16 tokens; shorter
  // blocks put more block ids next to the exps (eight heads, d = 128, blocks of 8: 82 628 bytes): a shorter
  // chunk keeps the second workgroup on the CU
  if (!g_chunk_tokens.load(std::memory_order_relaxed) && D.b < 16 &&
      decode_lds_bytes(T, D.r, D.d, 16, kDecodeWaves, mf) <= kLdsLimit / 2)
    while (T > 1024 && decode_lds_bytes(T, D.r, D.d, D.b, kDecodeWaves, mf) > kLdsLimit / 2) T -= 64;
  while (T > kMinChunk && decode_lds_bytes(T, D.r, D.d, D.b, kDecodeWaves, mf) > kLdsLimit) T -= 64;
  const size_t lds = decode_lds_bytes(T, D.r, D.d, D.b, kDecodeWaves, mf);
  if (lds > kLdsLimit || T % 64 != 0) return false;
  *T_out = T;
  *lds_out = lds;
  if (small_call) *small_call = shrunk;
  if (on_device) *on_device = device_side;
  return true;
}

// Items of at most 512 tokens go to the one-wavefront launch: the size classes from *cls up,
// whose items hold at most *max_tokens tokens; *lds_tokens is that bound in whole 64-token strips.
static void short_split(int T, int* cls, int* max_tokens, int* lds_tokens) {
  int k = 1;
  while (k < 15 && (T >> (k - 1)) > 512) ++k;
  *cls = k;
  *max_tokens = T >> (k - 1);
  *lds_tokens = (*max_tokens + 63) & ~63;
}

}  // namespace kvc

using namespace kvc;

extern "C" {

int kvc_profile_begin(int n) {
  if (n < 0 || n > 4096) return KVC_ERR_ARG;
  std::lock_guard<std::mutex> hold(g_prof_lock);
  g_prof_any.store(n > 0, std::memory_order_release);
  if (g_prof) {
    for (int i = 0; i < g_prof_cap; ++i) {
      hipEventDestroy(g_prof[i].a0); hipEventDestroy(g_prof[i].a1);
      hipEventDestroy(g_prof[i].s0); hipEventDestroy(g_prof[i].s1);
    }
    delete[] g_prof;
    g_prof = nullptr;
  }
  g_prof_cap = g_prof_used = 0;
  g_prof_on = 1;
  if (n == 0) return KVC_OK;
  g_prof = new ProfilePair[n];
  for (int i = 0; i < n; ++i) {
    KVC_HIP(hipEventCreate(&g_prof[i].a0)); KVC_HIP(hipEventCreate(&g_prof[i].a1));
    KVC_HIP(hipEventCreate(&g_prof[i].s0)); KVC_HIP(hipEventCreate(&g_prof[i].s1));
  }
  g_prof_cap = n;
  return KVC_OK;
}

int kvc_profile_enable(int on) {
  std::lock_guard<std::mutex> hold(g_prof_lock);
  g_prof_on = on != 0;
  return KVC_OK;
}

int kvc_profile_collect(float* chunk_ms, float* short_ms, float* combine_ms, int cap, int* count) {
  if (!count || cap < 0) return KVC_ERR_ARG;
  std::lock_guard<std::mutex> hold(g_prof_lock);
  *count = g_prof_used;
  for (int i = 0; i < g_prof_used && i < cap; ++i) {
    KVC_HIP(hipEventSynchronize(g_prof[i].s1));
    float ms = 0.0f;
    if (chunk_ms) { KVC_HIP(hipEventElapsedTime(&ms, g_prof[i].a0, g_prof[i].a1)); chunk_ms[i] = ms; }
    if (short_ms) { KVC_HIP(hipEventElapsedTime(&ms, g_prof[i].s0, g_prof[i].s1)); short_ms[i] = ms; }
    if (combine_ms) combine_ms[i] = 0.0f;   // (no launch combines: chunks finish their heads themselves)
  }
  return KVC_OK;
}

int kvc_get_decode_chunk(const kvc_config* cfg, int* tokens) {
  int rc = validate(cfg, nullptr);
  if (rc != KVC_OK) return rc;
  if (!tokens) return KVC_ERR_ARG;
  int T = 0;
  size_t lds = 0;
  const Dims D = dims_of(cfg);
  *tokens = choose_chunk(D, D.G, &T, &lds) ? T : 0;
  return KVC_OK;
}

int kvc_get_decode_short(const kvc_config* cfg, int* tokens) {
  int rc = validate(cfg, nullptr);
  if (rc != KVC_OK) return rc;
  if (!tokens) return KVC_ERR_ARG;
  int T = 0;
  size_t lds = 0;
  const Dims D = dims_of(cfg);
  *tokens = 0;
  if (choose_chunk(D, D.G, &T, &lds)) {
    int cls = 0, lds_tokens = 0;
    short_split(T, &cls, tokens, &lds_tokens);
  }
  return KVC_OK;
}

int kvc_set_decode_chunk(int tokens) {
  if (tokens != 0 && (tokens < kMinChunk || tokens > kMaxChunk || tokens % 64 != 0)) return KVC_ERR_ARG;
  g_chunk_tokens.store(tokens, std::memory_order_relaxed);
  return KVC_OK;
}

}  // extern "C"

// What both decode entry points check on the host before anything is launched.
static int decode_args_check(const kvc_config* cfg, const kvc_state* st, const void* q, const float* out,
                             int layer_begin, int layer_end) {
  const int rc = validate(cfg, st);
  if (rc != KVC_OK) return rc;
  if (!q || !out || ((uintptr_t)q & 15) || ((uintptr_t)out & 15)) return KVC_ERR_ARG;
  if (layer_begin < 0 || layer_end > cfg->num_layers || layer_begin >= layer_end) return KVC_ERR_ARG;
  return KVC_OK;
}

// plan_mode 0: an ordinary call (work list, chunks).  1: only the work lists, one per
// layer, kept in the workspace (q and out are not looked at).  2: layer `layer_begin` from its kept list.
enum { PLAN_NONE = 0, PLAN_BUILD = 1, PLAN_USE = 2 };
constexpr size_t kPlanRowChunk = 256;
static int paged_decode_impl(const kvc_config* cfg, const kvc_state* st, const void* q, float* out,
                             int layer_begin, int layer_end, int accumulate_metric, void* ws, void* stream,
                             int plan_mode = PLAN_NONE, int ctx_plus = 0) {
  int rc = plan_mode == PLAN_BUILD ? validate(cfg, st) : decode_args_check(cfg, st, q, out, layer_begin, layer_end);
  if (rc != KVC_OK) return rc;
  if (!ws || ((uintptr_t)ws & 255)) return KVC_ERR_ARG;
  Dims D = dims_of(cfg);
  if (plan_mode == PLAN_BUILD) { layer_begin = 0; layer_end = 1; }   // lists are per layer: sized as a one-layer call
  Workspace W = carve(D, ws);
  hipStream_t s = (hipStream_t)stream;

  DecodeArgs A;
  A.D = D;
  A.kc = (const char*)st->k_cache; A.vc = (const char*)st->v_cache;
  A.metric = st->metric; A.table = st->block_table; A.ctx = st->ctx_len;
  A.q = (const char*)q; A.out = out;
  A.l0 = layer_begin; A.nl = layer_end - layer_begin; A.gsel = D.S * A.nl * D.Hk;
  A.accumulate = accumulate_metric != 0;
  A.all_partials = 0;
  A.rotate_chunks = 0;
  A.cap = (int)(max_items_of(D) < 0x7fffffffull ? max_items_of(D) : 0x7fffffffull);
  A.items = (DecodeItem*)W.items; A.slot_word = W.slot_word; A.part_ml = W.part_ml; A.part_acc = W.part_acc; A.stash = W.stash;
  A.header = W.header;
  A.status = W.header;
  A.plan = 0; A.plan_stride = 0; A.plan_cap = 0; A.ctx_plus = 0; A.self_list = 0;
  A.packed = (size_t)D.maxb * D.b / kMinChunk < (size_t)kMeetMost;
  A.scale_log2 = (float)(1.4426950408889634 / sqrt((double)D.d));

  int T = 0;
  size_t lds = 0;
  bool small_call = false, on_device = false;
  bool tiled = choose_chunk(D, D.S * (layer_end - layer_begin) * D.Hk, &T, &lds, &small_call, &on_device);
  A.adapt_T = tiled && on_device;
  const int esz = kv_esz(D.dtype);
  A.T = tiled ? T : (1 << 30);  // generic path: one "chunk" per head
  A.short_class = 16;
  A.Ts = 0;
  // A small call (one layer of a model) is bound by the time of its slowest item, not by
  // throughput: there every item gets four wavefronts and the short-item launch is left out.
  if (tiled && !small_call) {
    int short_max = 0;
    short_split(T, &A.short_class, &short_max, &A.Ts);
  }
  A.log2b = 0;
  while ((1 << A.log2b) < D.b) ++A.log2b;

  // kept lists exist for what a model's layer-by-layer calls look like: the tiled kernels, few heads
  // per layer, the chunk length picked on the device
  if (plan_mode != PLAN_NONE && !(tiled && small_call && on_device && A.gsel <= kSmallWorklistHeads)) return KVC_ERR_UNSUPPORTED;
  if (!tiled) {
    const size_t gl = ((size_t)D.r * D.d + 4 * 16 + 2 * 16) * 4;
    hipLaunchKernelGGL(decode_generic_kernel, dim3(A.gsel), dim3(256), gl, s, A);
    KVC_LAUNCH_CHECK();
    return KVC_OK;
  }
  // items <= (slots in the pool) / T + heads, and <= heads * chunks a full row can hold.  A chunk
  // length picked on the device is T (then the first bound holds), or at least 1.25 / 512 of all
  // tokens, or the 128-token floor with under 128 * 512 / 1.25 tokens in all: at most 512 / 1.25
  // full chunks either way, and one shorter item per head.
  A.places = 0x7fffffff;
  if (A.adapt_T && A.gsel > kSelfListHeads) {   // (fewer heads make 410 chunks and one each, at most)
    if (esz == 1) A.places = D.d == 64 ? tiled_places<1, 64>(D, lds) : tiled_places<1, 128>(D, lds);
    else if (esz == 2) A.places = D.d == 64 ? tiled_places<2, 64>(D, lds) : tiled_places<2, 128>(D, lds);
    else A.places = D.d == 64 ? tiled_places<4, 64>(D, lds) : tiled_places<4, 128>(D, lds);
  }
  const size_t most_tokens = std::min((size_t)D.N * D.b, (size_t)A.gsel * D.maxb * D.b);   // pool, or the rows of the heads called for
  const size_t bound_pool = (A.adapt_T ? std::max(most_tokens / T, (size_t)410) : most_tokens / T) + (size_t)A.gsel;
  auto items_of_rows = [&](size_t chunk) { return std::min(bound_pool, (size_t)A.gsel * (((size_t)D.maxb * D.b + chunk - 1) / chunk)); };
  const size_t grid = items_of_rows(A.adapt_T ? (size_t)kSmallCallChunk : (size_t)T);
  if (grid > 0x7fffffffull) return KVC_ERR_UNSUPPORTED;   // before anything is launched: the work list stays clean
  const int list_threads = (A.gsel + 63) & ~63;   // of a one-launch list: a thread per head
  if (plan_mode != PLAN_NONE) {
    // Rows with far more room than the pool can fill have no lists: every layer's launch is as large as
    // full rows would need, and nearly all of it would be empty.  (Lists of chunks of kPlanRowChunk for
    // all layers' full rows have to fit the records that the workspace has.)
    // (counted in chunks of the length that two workgroups leave each other)
    const size_t bound_accept = std::max(most_tokens / default_chunk(D), (size_t)410) + (size_t)A.gsel;
    const size_t full_rows = (size_t)A.gsel * (((size_t)D.maxb * D.b + kPlanRowChunk - 1) / kPlanRowChunk);
    if (std::min(bound_accept, full_rows) * (size_t)D.Lyr > (size_t)A.cap) return KVC_ERR_UNSUPPORTED;
    A.plan = 1;
    A.plan_cap = A.cap;
    A.plan_stride = grid * (size_t)D.Lyr <= (size_t)A.cap ? (int)grid : 0;   // (a start of its own costs every launch a dependent load)
    A.cap = (int)std::min(grid, (size_t)A.cap);
    A.ctx_plus = ctx_plus;
    A.header = W.plan_hdr;
    if (plan_mode == PLAN_BUILD) {
      A.out = nullptr;    // (the zero rows of heads without a KV are written when the layer is decoded)
      hipLaunchKernelGGL(decode_worklist_small_kernel<true>, dim3(D.Lyr), dim3(list_threads), 0, s, A);
      KVC_LAUNCH_CHECK();
      return KVC_OK;
    }
    A.header += (size_t)layer_begin * HW_WORDS;
    A.items += (size_t)layer_begin * A.plan_stride;
    A.slot_word += (size_t)layer_begin * A.plan_stride;
  } else if (small_call && A.gsel <= kSelfListHeads && A.packed) {
    A.self_list = 1;
  } else if (A.gsel <= kSmallWorklistHeads) {
    hipLaunchKernelGGL(decode_worklist_small_kernel<false>, dim3(1), dim3(list_threads), 0, s, A);
    KVC_LAUNCH_CHECK();
  } else {
    hipLaunchKernelGGL(decode_count_kernel, dim3((A.gsel + 255) / 256), dim3(256), 0, s, A);
    KVC_LAUNCH_CHECK();
    hipLaunchKernelGGL(decode_items_kernel, dim3((A.gsel + 255) / 256), dim3(256), 0, s, A);
    KVC_LAUNCH_CHECK();
  }
  const int gs = A.gsel;   // a head ends in at most one item shorter than a chunk
  if (esz == 1) return D.d == 64 ? launch_tiled_r<1, 64>(A, (int)grid, lds, gs, s) : launch_tiled_r<1, 128>(A, (int)grid, lds, gs, s);
  if (esz == 2) return D.d == 64 ? launch_tiled_r<2, 64>(A, (int)grid, lds, gs, s) : launch_tiled_r<2, 128>(A, (int)grid, lds, gs, s);
  return D.d == 64 ? launch_tiled_r<4, 64>(A, (int)grid, lds, gs, s) : launch_tiled_r<4, 128>(A, (int)grid, lds, gs, s);
}

// ---- the decode for callers that cannot allocate --------------------------------------------
// The temporaries of kvc_paged_decode (work items, per-chunk partial results, the exps of chunks
// that left their head) in a fixed array of this library's own instead of a caller's workspace.  Every
// GPU holds its own copy of the array at its own address; host code never uses the array's name
// as an address, only what hipGetSymbolAddress returned for the device that is current.
static __device__ __align__(256) unsigned char scratch[KVC_STATIC_SCRATCH_BYTES];

static constexpr int kMaxDevices = 64;
static std::mutex g_scratch_lock;
static void* g_scratch_ptr[kMaxDevices] = {};   // per device, filled on the first call there

static int scratch_of_current_device(void** out) {
  int dev = -1;
  KVC_HIP(hipGetDevice(&dev));
  if (dev < 0 || dev >= kMaxDevices) return KVC_ERR_UNSUPPORTED;
  std::lock_guard<std::mutex> hold(g_scratch_lock);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    KVC_HIP(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
    if (!p || ((uintptr_t)p & 255)) return KVC_ERR_HIP;
    g_scratch_ptr[dev] = p;
  }
  *out = g_scratch_ptr[dev];
  return KVC_OK;
}

extern "C" {

int kvc_paged_decode(const kvc_config* cfg, const kvc_state* st, const void* q, float* out,
                     int layer_begin, int layer_end, int accumulate_metric, void* ws, void* stream) {
  return paged_decode_impl(cfg, st, q, out, layer_begin, layer_end, accumulate_metric, ws, stream);
}

int kvc_decode_plan(const kvc_config* cfg, const kvc_state* st, int ctx_plus, void* ws, void* stream) {
  if (ctx_plus < 0 || ctx_plus > 1) return KVC_ERR_ARG;
  return paged_decode_impl(cfg, st, nullptr, nullptr, 0, 1, 0, ws, stream, PLAN_BUILD, ctx_plus);
}

int kvc_paged_decode_planned(const kvc_config* cfg, const kvc_state* st, const void* q, float* out, int layer,
                             int accumulate_metric, void* ws, void* stream) {
  return paged_decode_impl(cfg, st, q, out, layer, layer + 1, accumulate_metric, ws, stream, PLAN_USE, 0);
}

int kvc_paged_decode_static(const kvc_config* cfg, const kvc_state* st, const void* q, float* out,
                            int layer_begin, int layer_end, int accumulate_metric, void* stream) {
  int rc = decode_args_check(cfg, st, q, out, layer_begin, layer_end);
  if (rc != KVC_OK) return rc;
  if (carve(dims_of(cfg), nullptr).bytes > (size_t)KVC_STATIC_SCRATCH_BYTES) return KVC_ERR_UNSUPPORTED;
  void* ws = nullptr;
  rc = scratch_of_current_device(&ws);
  if (rc != KVC_OK) return rc;
  // The array keeps what the last call left, possibly a call that was cut short: the header words (item counts,
  // work-list cursors) and the meeting words start from zero again.  A fill kernel, not a memset, so that
  // the call may be recorded into a HIP graph.
  const int words = 2 * HW_WORDS;   // (chunks meet in the first layer's block too, see meet_word)
  hipLaunchKernelGGL(zero_words_kernel, dim3((words + 63) / 64), dim3(64), 0, (hipStream_t)stream, (int32_t*)ws, words);
  KVC_LAUNCH_CHECK();
  return paged_decode_impl(cfg, st, q, out, layer_begin, layer_end, accumulate_metric, ws, stream);
}

}  // extern "C"
