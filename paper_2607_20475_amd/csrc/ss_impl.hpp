// ss_impl.hpp -- device implementation shared by the kernel translation units.
//
// Two launches per call (plus the materialising pass of ss_process_logits); the
// grids depend only on the shapes, nothing synchronises with the host, so every
// call can be captured in a HIP graph.
//
// Streaming kernel.  Every wavefront owns one "unit": 2048 consecutive logits
// of one row (16-byte loads, 32 elements per lane, read exactly once).  It
// turns them into order-preserving keys (grammar allow bits applied, NaN ->
// invalid), finds a unit threshold t -- the largest 16-bit key prefix such
// that at least q group maxima of the unit reach it, q being the unit's share
// of the row's top-k plus a statistical margin -- and writes every group of
// consecutive elements whose maximum reaches t to the unit's candidate region
// (when ties at t overflow the region, the lowest-index tie groups, and the
// unit's threshold becomes the composite (t, last kept index)).  This is the
// paper's bounded candidate set of the two-stage scheme (Section 3.2), chosen
// per unit by ballots instead of a per-tile sort.  The region holds elements,
// not groups (4 bytes each for bf16, 8 for fp32): the merge reads a quarter of
// the bytes and looks at a quarter of the slots.  The unit stream does not
// depend on the request's penalty history or logit bias: those touch at most
// a few hundred ids per row, and extra workgroups at the front of the same
// launch build each row's patch table: the listed ids' counts and ordered
// bias sums in an LDS hash, their raw logits gathered and put through the
// Appendix C.1 prologue (repetition, frequency, presence penalty, bias; Alg. 8
// order).
//
// Merge kernel, one workgroup per row: ss_row.hpp.
#pragma once
#include <hip/hip_runtime.h>
#include <limits.h>
#include <stddef.h>
#include <stdint.h>

#include "ss.h"
#include "ss_device.hpp"

namespace ss {

constexpr int kPBLog = 17;                  // patched-id bitmap: 2^17 bits
constexpr int kPB = 1 << kPBLog;
constexpr int kUE = 2048;                    // elements per unit (one wavefront)
constexpr int kMaxU = SS_MAX_V / kUE;        // units per row at most (512)
constexpr int kH = 2048;                     // patch hash slots (LDS)
constexpr int kProbe = 64;                   // longest probe sequence before giving up
constexpr int kGH = 16384;                   // per-row patch table in global memory (LDS table overflow)
constexpr int kGProbe = 1024;
constexpr uint32_t kLinear = 0xFFFFFFFFu;    // patched-list count meaning "look the lists up"
constexpr uint32_t kTable = 0xFFFFFFFEu;     // patched-list count meaning "the row's patch table"
constexpr int kStage = 128;                  // emission groups a wavefront stages in LDS at a time
constexpr int kQScan = 256;                  // sparse draft lists up to this length are scanned, longer ones sorted
constexpr uint32_t kNoEmit = 0xFFFFFFFFu;    // threshold of a unit that emits nothing
constexpr uint32_t kOvf = 0xFFFFFFFFu;       // element count of a unit whose candidates overflow its region
constexpr double kFix = 1125899906842624.0;  // 2^50: fixed-point scale of probability mass

enum { OP_TOPK = SS_OP_TOPK, OP_SAMPLE = SS_OP_SAMPLE, OP_VERIFY = SS_OP_VERIFY, OP_PROCESS = SS_OP_PROCESS,
       OP_LOGPROBS = SS_OP_LOGPROBS,
       OP_SAMPLE_X = 5 };  // merge only: sampling with full-row truncation or the Gumbel-max draw
// the merge instantiations that sample (the plain one carries neither extension)
constexpr bool sampling_op(int op) { return op == OP_SAMPLE || op == OP_SAMPLE_X; }
enum { KIND_EMPTY = 0, KIND_GREEDY = 1, KIND_DIST = 2 };

struct RowSummary {
  uint64_t thr;  // composite key of the last kept element
  double Z;      // sum of kept weights
  float M;       // row maximum (processed logit)
  float tau;
  int32_t argmax;
  int32_t kind;
};
struct RowResult {
  uint64_t word;     // (token << 32) | (flags << 1) | accept
  uint32_t arrived;  // of a request's first row: merged rows of the request
  uint32_t pad;
};

struct KArgs {
  const void* x;
  int64_t ld;
  int op, B, rows, V, U, L, k_cap, cap, pcap, k_out;  // cap: candidate region of a unit in 16-byte words
  uint32_t feat;
  int have;  // kHave* bits; a NULL parameter array points at the workspace instead, so it can be read (and ignored)
  const uint32_t* mode;
  const float* temperature;
  const int32_t* top_k;
  const float* top_p;
  const float* min_p;
  const float* rep;
  const float* freq;
  const float* pres;
  const int32_t* hist_off;
  const int32_t* hist_ids;
  const int32_t* bias_off;
  const int32_t* bias_ids;
  const float* bias_vals;
  const uint32_t* bitmask;
  int64_t mask_ld;
  const uint64_t* seed;
  const int64_t* position;
  const float* draft_probs;  // dense q [B, L, ld_q] (NULL when sparse)
  int64_t ld_q;
  const int32_t* dq_idx;     // sparse q: ids [B, L, kq]
  const float* dq_val;       //           probabilities [B, L, kq]
  int kq;                    // entries per draft position (0: dense q)
  const float* gum;          // sampling with the Gumbel-max draw: g = ln z per token [B, ld_g] (else NULL)
  int64_t ld_g;
  const int32_t* rmap;       // verification of a tree path: path position -> target row [B, L+1] (else NULL)
  int Lt;                    // target rows per request (L+1 without a map)
  int full;                  // sampling: full-row top-p / min-p for requests without a top-k cut
  const int32_t* draft_tokens;
  int32_t* out_token;
  float* out_logprob;
  int32_t* out_idx;
  float* out_prob;
  int32_t* flags;
  float* out_val;
  int32_t* out_tokens;
  int32_t* out_nacc;
  float* out_logits;
  float* out_probs;
  uint4* rec;
  uint4* cand;
  RowResult* res;
  RowSummary* summ;
  uint2* patched;      // process: per row kGH (id, final key) pairs (lists beyond the patch table)
  uint64_t* gtag;      // per row kGH slots: (generation << 32) | (id + 1)
  uint32_t* gcnt;      // occurrence count | has-bias bit 31
  uint32_t* gfin;      // final key
  uint32_t* npatched;  // process: per row count
  int32_t* pstat;      // per row: 0 no lists, 1 patch table in ptab, 2 more ids than the table holds
  uint32_t* ptab;      // per row 2 kH words: slot ids (-1 empty), then final keys
  int patch_wgs;       // patch-table workgroups at the front of the streaming grid (0: the call has no lists)
  int unit_wgs;        // workgroups of the streaming grid behind them
  int tpu, tpu_inv;    // merge: threads per unit of the candidate loads, and ceil(2^20 / tpu)
  int nq;              // merge: 16-byte candidate loads a thread issues before anything is known
  double* usum;        // log-probabilities: per unit, sum of exp((x - unit max) / tau) over its valid logits
};

constexpr uint32_t kListBits = SS_REP | SS_FREQ | SS_PRES | SS_BIAS;  // requests with history or bias lists
enum { kHaveTopK = 1, kHaveSeed = 2, kHavePos = 4 };

// Brings the kernel arguments into the scalar cache in one round trip: each
// 64-byte line costs about 540 cycles on first touch, and the compiler reads
// them where they are used, one wait after another (2.0 us of a merge row's
// first barrier, 0.9 us with the lines fetched together).  Returns zero, which
// the caller adds to its block number so that nothing is read before; the asm
// is not volatile, so later loads of uniform data stay scalar.
__device__ __forceinline__ int warm_args() {
  const auto* p = (const uint32_t __attribute__((address_space(4)))*)__builtin_amdgcn_kernarg_segment_ptr();
  static_assert(sizeof(KArgs) > 7 * 64 && sizeof(KArgs) <= 8 * 64, "one word of each line");
  int zero;
  asm("s_mov_b32 %0, 0"
      : "=s"(zero)
      : "s"(p[0]), "s"(p[16]), "s"(p[32]), "s"(p[48]), "s"(p[64]), "s"(p[80]), "s"(p[96]), "s"(p[112]));
  return zero;
}
// The kernel arguments through a pointer the compiler cannot connect with
// earlier reads: arguments used late are read late (from the scalar cache)
// instead of being held, and spilled, across the whole kernel.
__device__ __forceinline__ const KArgs& late_args() {
  uint64_t p = (uint64_t)__builtin_amdgcn_kernarg_segment_ptr();
  asm("" : "+s"(p));
  return *(const KArgs*)(const KArgs __attribute__((address_space(4)))*)p;
}

// ---------------------------------------------------------------------------
// Element layout: lane l, slot s (0..31) holds element (s / VW * 64 + l) * VW
// + s % VW of its unit; a chunk of VW consecutive elements is one 16-byte load.
// Emission groups are GE consecutive elements (two key dwords).
// ---------------------------------------------------------------------------
template <int DT>
struct DTT;
template <>
struct DTT<SS_F32> {
  static constexpr int VW = 4, NLD = 8, ES = 4, GE = 2;
};
template <>
struct DTT<SS_BF16> {
  static constexpr int VW = 8, NLD = 4, ES = 2, GE = 4;
};

__host__ __device__ inline int groups_per_unit(int dt) { return dt == SS_BF16 ? 512 : 1024; }

// key without the positive-NaN fold; callers fold when the maximum exceeds +inf
__device__ __forceinline__ uint32_t key_raw(uint32_t u) {
  const uint32_t s = (uint32_t)((int32_t)u >> 31);
  return (u ^ s) + (s ? 1u : 0x80000000u);
}
__device__ __forceinline__ uint32_t fold_nan(uint32_t k) { return k > kKeyPosInf ? 0u : k; }

typedef unsigned short us2 __attribute__((ext_vector_type(2)));
typedef short ss2 __attribute__((ext_vector_type(2)));
// two packed bfloat16 -> two packed 16-bit keys (the upper halves of their
// float32 keys: bf16 keys have zero low halves)
__device__ __forceinline__ uint32_t key2_bf16(uint32_t d) {
  const ss2 v = __builtin_bit_cast(ss2, d);
  const uint32_t s = __builtin_bit_cast(uint32_t, (ss2)(v >> (ss2){15, 15}));
  const uint32_t c = (s & 0x80018001u) ^ 0x80008000u;
  const us2 r = __builtin_bit_cast(us2, d ^ s) + __builtin_bit_cast(us2, c);
  return __builtin_bit_cast(uint32_t, r);
}
__device__ __forceinline__ uint32_t pkmax16(uint32_t a, uint32_t b) {
  return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(us2, a), __builtin_bit_cast(us2, b)));
}
__device__ __forceinline__ uint32_t hmax16(uint32_t d) { return max(d & 0xFFFFu, d >> 16); }
// positive bf16 NaN keys (above +inf = 0xFF80) -> 0 in both halves
__device__ __forceinline__ uint32_t fold_nan2(uint32_t d) {
  uint32_t lo = d & 0xFFFFu, hi = d >> 16;
  lo = lo > 0xFF80u ? 0u : lo;
  hi = hi > 0xFF80u ? 0u : hi;
  return lo | (hi << 16);
}

// 16 bytes at any alignment (one load: global accesses need none on this target)
__device__ __forceinline__ uint4 load16(const unsigned char* p) {
  uint4 v;
  __builtin_memcpy(&v, p, 16);
  return v;
}

// float32 bit pattern of element i of a row (scalar access, any alignment)
template <int DT>
__device__ __forceinline__ uint32_t load_elem_bits(const unsigned char* xrow, int64_t i) {
  if constexpr (DT == SS_F32) {
    return reinterpret_cast<const uint32_t*>(xrow)[i];
  } else {
    return ((uint32_t)reinterpret_cast<const uint16_t*>(xrow)[i]) << 16;
  }
}

// ---------------------------------------------------------------------------
// Per-row context
// ---------------------------------------------------------------------------
struct Ctx {
  int row;
  uint32_t mode;
  const unsigned char* xrow;
  const int32_t* hist;
  int nhist;
  const int32_t* extra;
  int nextra;
  const int32_t* bias_ids;
  const float* bias_vals;
  int nbias;
  const uint32_t* mask;
  float rep, freq, pres;
  bool pexact;              // the patched-id bitmap is exact (V <= kPB)
};

// Allow bits of a target row that a tree path maps outside the tree: none
// (zero-initialised device memory, never written).
static __device__ uint32_t g_none_allowed[SS_MAX_V / 32];

// Logits row read for verification row `row` (request b, path position
// row mod (L+1)): through the path's row map when there is one; -1 when the
// map points outside the request's Lt target rows.
__device__ __forceinline__ int64_t source_row(const KArgs& a, int row) {
  if (!a.rmap) return row;
  const int b = row / (a.L + 1);
  const int t = a.rmap[row];
  return (t >= 0 && t < a.Lt) ? (int64_t)b * a.Lt + t : -1;
}

template <int DT>
__device__ __forceinline__ Ctx make_ctx(const KArgs& a, int row) {
  Ctx c;
  c.row = row;
  int b = row, ell = 0;
  if (a.op == OP_VERIFY) {
    b = row / (a.L + 1);
    ell = row % (a.L + 1);
  }
  const uint32_t m = (a.op == OP_TOPK ? SS_TOPK : a.mode[b]) & a.feat;
  c.mode = m;
  // read together, used if their bits are set
  const int h0 = a.hist_off[b], h1 = a.hist_off[b + 1], e0 = a.bias_off[b], e1 = a.bias_off[b + 1];
  const float rep = a.rep[b], freq = a.freq[b], pres = a.pres[b];
  const int64_t srow = a.op == OP_VERIFY ? source_row(a, row) : row;
  c.xrow = reinterpret_cast<const unsigned char*>(a.x) + (size_t)(srow < 0 ? 0 : srow) * (size_t)a.ld * DTT<DT>::ES;
  c.hist = nullptr;
  c.nhist = 0;
  c.extra = nullptr;
  c.nextra = 0;
  if (m & (SS_REP | SS_FREQ | SS_PRES)) {
    c.hist = a.hist_ids + h0;
    c.nhist = h1 - h0;
    if (a.op == OP_VERIFY && a.draft_tokens) {
      c.extra = a.draft_tokens + (size_t)b * a.L;
      c.nextra = ell;
    }
  }
  c.bias_ids = nullptr;
  c.bias_vals = nullptr;
  c.nbias = 0;
  if (m & SS_BIAS) {
    c.bias_ids = a.bias_ids + e0;
    c.bias_vals = a.bias_vals + e0;
    c.nbias = e1 - e0;
  }
  c.mask = (m & SS_GRAMMAR) ? a.bitmask + (size_t)row * (size_t)a.mask_ld : nullptr;
  if (srow < 0) c.mask = g_none_allowed;  // every token masked
  c.rep = (m & SS_REP) ? rep : 1.0f;
  c.freq = (m & SS_FREQ) ? freq : 0.0f;
  c.pres = (m & SS_PRES) ? pres : 0.0f;
  c.pexact = a.V <= kPB;
  return c;
}

// Candidate quota of one unit when a full unit's share of the row's top-k is kt: the
// unit keeps at least its q largest elements, q well above that share (five
// standard deviations plus six), so that the largest unit threshold lies below
// the row's k-th value except with negligible probability.
__host__ __device__ inline int quota(int k, int kt) {
  int s = 0;
  while (s * s < kt) ++s;
  const int q = kt + 5 * s + 6;
  return q < k ? q : k;
}
// The quota of a unit of a row of V elements in U units.  The share of few units goes
// by elements: a short last one leaves the others more (k = 4096 at V = 5000 took the
// slow path in every row, 115 us at B = 64).  Beyond 12 units that is at most a
// standard deviation of the margin's five, and quotas stay what their loads hold.
__host__ __device__ inline int unit_quota(int k, int U, int V) {
  if (U <= 1 || k <= 1) return k;
  const uint32_t num = (uint32_t)(U <= 12 ? k * kUE : k), den = (uint32_t)(U <= 12 ? V : U);
  return quota(k, (int)((num + den - 1u) / den));
}
// A row of one unit emits its top k, and twice as many when penalties can push some of
// those down (rows of V = 1000 with 528 listed ids: 43 us with the slow path).
__host__ __device__ inline int emit_k(int k, int V, uint32_t mode) {
  const uint32_t m = mode & (V <= kUE ? kListBits : 0u);
  static_assert(kListBits == 30u, "the sum below reaches 32 with any of the bits");
  return k << ((m + 30u) >> 5);  // (scalar; a condition goes through a vector register)
}

// Threshold groups per lane for quota q (32 / G elements each).  Groups of
// several elements need four times as many groups as the quota, so that two of the
// largest elements seldom share one; single elements (G = 32) give the exact
// threshold of any quota, at 32 comparisons per search step.  0, and the unit emits all
// it has, when the quota is half of it: that adds less than the search takes and leaves
// the row nothing to miss.  (Quotas beyond 128 groups in bf16 used to emit
// everything, which overflowed the merge: k <= 4096 at V = 102438, B = 138 took 783 us,
// 45 us with the thresholds.)
__host__ __device__ inline int thr_groups(int q) {
  for (int G = 1; G <= 16; G <<= 1)
    if (64 * G >= 4 * q) return G;
  return q < kUE / 2 ? 32 : 0;
}

// capacity (groups, 16 bytes each) of one unit's candidate region
__host__ __device__ inline int unit_cap(int k_cap, int U, int dt) {
  const int gpu = groups_per_unit(dt);
  const int q = unit_quota(k_cap, U, U * kUE);
  if (thr_groups(q) == 0) return gpu;
  // room for twice the quota, and, when less than a whole unit, for k_cap
  // elements of one unit: a row tied at its maximum then finds its top-k
  // among the lowest-index tie groups of its first unit (the tie cut keeps
  // them)
  const int ge = dt == SS_BF16 ? 4 : 2;
  const int kg = (k_cap + ge - 1) / ge;
  int c = 2 * q + 64;
  if (kg < gpu && c < kg) c = kg;
  if ((c & 63) == 0) c += 4;  // regions not a multiple of 1 KB apart: their heads spread over the memory channels
  return c < gpu ? c : gpu;
}

// ---------------------------------------------------------------------------
// Prologue of one patched element in Appendix C.1 order, each step one
// float32 op: repetition penalty, frequency and presence penalties (count >
// 0), then the logit bias.  Grammar masking is applied by the caller.
// ---------------------------------------------------------------------------
__device__ __forceinline__ uint32_t penalised_key(uint32_t bits, uint32_t mode, float rep, float freq, float pres,
                                                  int count, bool has_bias, float bsum) {
  float v = canon(__uint_as_float(bits));
  if (count > 0) {
    if (mode & SS_REP) v = (v > 0.0f) ? v / rep : v * rep;
    if (mode & SS_FREQ) {
      const float t = freq * (float)count;
      v = v - t;
    }
    if (mode & SS_PRES) v = v - pres;
  }
  if (has_bias) v = v + bsum;
  return key_of_float(v);
}

// ===========================================================================
// Streaming phase: one unit per wavefront
// ===========================================================================
template <int NW>
__device__ __forceinline__ uint32_t thr_search(const uint32_t (&gm)[NW], uint32_t q, int shift) {
  // largest 16-bit prefix p with at least q of the wavefront's values >= p << shift
  // (or, once exactly q values lie at or above it, that shorter prefix).  The
  // caller guarantees q <= 64 NW, so p lies between the wavefront's smallest
  // and largest prefix: the search starts at their highest differing bit.
  uint32_t lmin = gm[0], lmax = gm[0];
#pragma unroll
  for (int i = 1; i < NW; ++i) {
    lmin = min(lmin, gm[i]);
    lmax = max(lmax, gm[i]);
  }
  const uint32_t vmin = wave_min(lmin) >> shift, vmax = wave_max_u32(lmax) >> shift;
  const uint32_t diff = vmin ^ vmax;
  if (diff == 0u) return vmin << shift;
  const int hb = 31 - __clz(diff);
  uint32_t prefix = vmax & ~((2u << hb) - 1u);
#pragma unroll 1
  for (int b = hb; b >= 0; --b) {
    const uint32_t cand = (prefix | (1u << b)) << shift;
    uint32_t cnt = 0u;
#pragma unroll
    for (int i = 0; i < NW; ++i) cnt += (uint32_t)__popcll(__ballot(gm[i] >= cand));
    if (cnt >= q) {
      prefix |= 1u << b;
      // exactly q values at or above the prefix: the lower bits cannot drop
      // any of them, and a lower threshold is still a valid one
      if (cnt == q) break;
    }
  }
  return prefix << shift;
}

// threshold over G groups per lane of the 32 keys held as bf16 pairs
template <int G>
__device__ __forceinline__ uint32_t thr_bf16(const uint32_t (&kd)[16], uint32_t q) {
  constexpr int D = 16 / G;
  uint32_t gm[G];
#pragma unroll
  for (int g = 0; g < G; ++g) {
    uint32_t m = kd[g * D];
#pragma unroll
    for (int j = 1; j < D; ++j) m = pkmax16(m, kd[g * D + j]);
    gm[g] = hmax16(m);
  }
  return thr_search<G>(gm, q, 0);
}
// the same over pairs (H = 1) or single elements (H = 2), the group maxima
// formed at each step instead of held; vmax is the unit's largest key
template <int H>
__device__ __forceinline__ uint32_t thr_bf16_wide(const uint32_t (&kd)[16], uint32_t q, uint32_t vmax) {
  uint32_t prefix = 0u;
#pragma unroll 1
  for (int b = 31 - __clz(vmax | 1u); b >= 0; --b) {
    const uint32_t cand = prefix | (1u << b);
    uint32_t cnt = 0u;
#pragma unroll
    for (int j = 0; j < 16; ++j) {
      if constexpr (H == 1) {
        cnt += (uint32_t)__popcll(__ballot(hmax16(kd[j]) >= cand));
      } else {
        cnt += (uint32_t)__popcll(__ballot((kd[j] & 0xFFFFu) >= cand)) + (uint32_t)__popcll(__ballot((kd[j] >> 16) >= cand));
      }
    }
    if (cnt >= q) {
      prefix = cand;
      if (cnt == q) break;
    }
  }
  return prefix;
}
template <int G>
__device__ __forceinline__ uint32_t thr_f32(const uint32_t (&kk)[32], uint32_t q) {
  constexpr int D = 32 / G;
  uint32_t gm[G];
#pragma unroll
  for (int g = 0; g < G; ++g) {
    uint32_t m = kk[g * D];
#pragma unroll
    for (int j = 1; j < D; ++j) m = max(m, kk[g * D + j]);
    gm[g] = m;
  }
  return thr_search<G>(gm, q, 16);
}

// Ties at a unit threshold t can put more groups at or above t than the
// unit's candidate region holds.  Then every group whose maximum exceeds t is
// kept (when those alone fit) together with the lowest-index groups whose
// maximum equals t, up to the capacity: the unit still holds every element
// whose composite (key, lower index first) is at or above (t, cut), where
// cut is the last element index of the last kept tie group.  gm[g] is group
// g's maximum key; group g of a lane starts at element (g / 2 * 64 + lane) VW
// + (g % 2) GE of the unit, so index order is (g / 2, lane, g % 2).  Returns
// false (a true overflow) when the groups above t alone exceed the capacity.
template <int NG, int VW, int GE>
__device__ __forceinline__ bool tie_trim(const uint32_t (&gm)[NG], uint32_t t, uint32_t cap, uint32_t& gmask,
                                         uint32_t& cut_rel) {
  const int ln = lane();
  uint32_t gtm = 0u, eqm = 0u;
#pragma unroll
  for (int g = 0; g < NG; ++g) {
    gtm |= (gm[g] > t ? 1u : 0u) << g;
    eqm |= (gm[g] == t ? 1u : 0u) << g;
  }
  uint32_t ngt;
  (void)wave_excl_small((uint32_t)__popc(gtm), ngt);
  if (ngt > cap) return false;
  const uint32_t rem = cap - ngt;
  uint32_t keep = 0u, base = 0u, last = 0u;
#pragma unroll
  for (int c = 0; c < NG / 2; ++c) {
    const uint32_t e2 = (eqm >> (2 * c)) & 3u;
    uint32_t tc;
    uint32_t r = base + wave_excl_small((uint32_t)__popc(e2), tc);
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      if ((e2 >> h) & 1u) {
        if (r < rem) {
          keep |= 1u << (2 * c + h);
          last = max(last, (uint32_t)((c * 64 + ln) * VW + h * GE + GE - 1));
        }
        ++r;
      }
    }
    base += tc;
  }
  gmask = gtm | keep;
  cut_rel = wave_max_u32(last);
  return true;
}

// Temperature of a row's log-probabilities: its own when the temperature bit
// is on, tau > 0 and the row is not greedy, else 1.
__device__ __forceinline__ float lp_tau(const KArgs& a, uint32_t mode, int b) {
  if ((mode & SS_TEMP) && !(mode & SS_GREEDY) && a.temperature[b] > 0.0f) return a.temperature[b];
  return 1.0f;
}
// One term of a unit's normaliser sum, exp((v - mu) / tau) as 2^((v - mu) c)
// in float32 with c = log2(e) / tau rounded once: one rounding of the constant,
// one of the product and the hardware's 2^x (1 ulp), the same number of
// roundings as expf of (v - mu) (1 / tau) at a fifth of its instructions.  The
// merge recomputes a term bit for bit for the raw copies of patched ids.
// Terms below 2^-126 of the unit's largest count as zero; so do NaNs.
// (The constant stays finite at subnormal temperatures: the maximum's term is 1.)
__device__ __forceinline__ float lp_scale(float tau) {
  return fminf((float)(1.4426950408889634 / (double)tau), 3.402823466e38f);
}
__device__ __forceinline__ float lp_term(float v, float mu, float c) {
  return fmaxf(__builtin_amdgcn_exp2f((v - mu) * c), 0.0f);
}
// Rows whose units add their share of the full-row normaliser: requests with
// the log-probability bit, or, in full-row sampling, stochastic requests
// without a top-k cut.
__device__ __forceinline__ bool usum_row(const KArgs& a, uint32_t mode, int b) {
  if (a.op == OP_LOGPROBS) return (mode & SS_LOGPROBS) != 0u;
  if (!a.full) return false;
  const bool greedy = (mode & SS_GREEDY) || ((mode & SS_TEMP) && a.temperature[b] <= 0.0f);
  return !greedy && !((mode & SS_TOPK) && a.top_k[b] >= 1);
}

// Per-wavefront staging strip of the emission: the keys of up to kStage
// emission groups (GE consecutive elements, two dwords) and their group
// numbers within the unit.
struct WStage {
  uint2 k[kStage];
  uint16_t g[kStage];
};

// Writes the elements at or above t of the groups in gmask (NG groups per
// lane, `off` the lane's first rank, `total` the wavefront's count) densely
// to the unit's region and returns their number.  Groups are compacted into
// LDS (about one in forty is emitted), then 64 elements at a time are tested
// and compacted by ballot: one store per element instead of a 16-byte record
// per group.  An element is stored so that one unsigned comparison ranks it
// (key, lower index first): bf16 as (key16 << 16) | (0xFFFF - index within the
// unit), fp32 as its 64-bit composite.  Group g of a lane starts at element ((g / 2) 64 + lane)
// VW + (g % 2) GE of the unit, i.e. is group ((g / 2) 64 + lane) 2 + g % 2.
template <int DT, int NG>
__device__ __forceinline__ uint32_t emit_elems(const uint2 (&gk)[NG], uint32_t gmask, uint32_t off, uint32_t total,
                                               uint32_t t, uint32_t lo, uint4* region, WStage& W) {
  constexpr int GE = DTT<DT>::GE;
  const int ln = lane();
  uint32_t out = 0u;
  for (uint32_t c0 = 0u; c0 < total; c0 += (uint32_t)kStage) {
#pragma unroll
    for (int g = 0; g < NG; ++g) {
      if ((gmask >> g) & 1u) {
        const uint32_t p = off + (uint32_t)__popc(gmask & ((1u << g) - 1u)) - c0;
        if (p < (uint32_t)kStage) {
          W.k[p] = gk[g];
          W.g[p] = (uint16_t)(((g >> 1) * 64 + ln) * 2 + (g & 1));
        }
      }
    }
    wave_lds_fence();
    const uint32_t n = min(total - c0, (uint32_t)kStage) * GE;
    for (uint32_t i0 = 0u; i0 < n; i0 += 64u) {
      const uint32_t i = i0 + (uint32_t)ln;
      uint32_t key;
      if constexpr (DT == SS_BF16) key = reinterpret_cast<const uint16_t*>(W.k)[i];
      else key = reinterpret_cast<const uint32_t*>(W.k)[i];
      const uint32_t e = (uint32_t)W.g[i / GE] * GE + (i & (GE - 1));
      const bool hit = i < n && key >= t;
      const uint64_t m = __ballot(hit);
      const uint32_t pos = out + __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
      if (hit) {
        if constexpr (DT == SS_BF16) reinterpret_cast<uint32_t*>(region)[pos] = (key << 16) | (0xFFFFu - e);
        else reinterpret_cast<uint2*>(region)[pos] = make_uint2(~(lo + e), key);
      }
      out += (uint32_t)__popcll(m);
    }
    wave_lds_fence();
  }
  return out;
}

// Streams unit `gu` (wave-uniform) and writes its record and candidates.
// The record is (threshold key, elements written or kOvf when the candidate
// groups overflow the region, unit maximum key, last index of the tie cut or
// ~0u when every group at or above the threshold was written).
template <int DT, bool LP>
__device__ __forceinline__ void scan_unit(const KArgs& a, int gu, WStage& W) {
  constexpr int VW = DTT<DT>::VW, NLD = DTT<DT>::NLD, ES = DTT<DT>::ES;
  const int ln = lane();
  const int row = gu / a.U;
  const int u = gu - row * a.U;
  const int lo = u * kUE;
  const int64_t srow = a.op == OP_VERIFY ? source_row(a, row) : row;
  const int n = srow < 0 ? 0 : min(kUE, a.V - lo);  // a row outside the tree reads nothing
  const int b = a.op == OP_VERIFY ? row / (a.L + 1) : row;
  const unsigned char* xrow =
      reinterpret_cast<const unsigned char*>(a.x) + (size_t)(srow < 0 ? 0 : srow) * (size_t)a.ld * ES;

  // 1. loads: the unit's chunks (16 bytes at any element alignment: rows of odd
  // length need no path of their own), then the request's parameters, read
  // together before they are known to be needed, then the grammar words
  uint4 r[NLD];
  if (n == kUE) {
    const unsigned char* src = xrow + (size_t)lo * ES;
#pragma unroll
    for (int i = 0; i < NLD; ++i) r[i] = load16(src + (size_t)(i * 64 + ln) * 16);
  } else {
#pragma unroll
    for (int i = 0; i < NLD; ++i) {
      const int l0 = (i * 64 + ln) * VW;
      r[i] = make_uint4(0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu);  // negative NaN: invalid
      if (l0 + VW <= n) {
        r[i] = load16(xrow + (size_t)(lo + l0) * ES);
      } else if (l0 < n) {  // the row's last chunk
        uint32_t w[4] = {0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu};
#pragma unroll
        for (int e = 0; e < VW; ++e) {
          if (l0 + e < n) {
            if constexpr (DT == SS_F32) {
              w[e] = reinterpret_cast<const uint32_t*>(xrow)[lo + l0 + e];
            } else {
              const uint32_t h = reinterpret_cast<const uint16_t*>(xrow)[lo + l0 + e];
              const int q = e >> 1;
              w[q] = (e & 1) ? ((w[q] & 0x0000FFFFu) | (h << 16)) : ((w[q] & 0xFFFF0000u) | h);
            }
          }
        }
        r[i] = make_uint4(w[0], w[1], w[2], w[3]);
      }
    }
  }
  const uint32_t mode_v = a.mode[b];
  const float temp = a.temperature[b];
  const int topk = a.top_k[b];
  const uint32_t mode = (a.op == OP_TOPK ? SS_TOPK : mode_v) & a.feat;
  const uint32_t* mask = (mode & SS_GRAMMAR) ? a.bitmask + (size_t)row * (size_t)a.mask_ld : nullptr;
  uint32_t mw[NLD];
  if (mask) {
    const int W = (a.V + 31) >> 5;
#pragma unroll
    for (int i = 0; i < NLD; ++i) {
      const int wi = (lo + (i * 64 + ln) * VW) >> 5;
      mw[i] = wi < W ? mask[wi] : 0u;
    }
  }

  // 2. row parameters (scalar), read while the chunks are in flight
  int k_eff;
  if (a.op == OP_TOPK) {
    const int k = (a.have & kHaveTopK) ? topk : a.k_cap;
    k_eff = k < 0 ? 0 : min(k, a.k_cap);
  } else if (a.op == OP_LOGPROBS) {
    k_eff = (mode & SS_LOGPROBS) ? emit_k(a.k_cap, a.V, mode) : 0;
  } else {
    const bool greedy = (mode & SS_GREEDY) || ((mode & SS_TEMP) && temp <= 0.0f);
    const int k = ((mode & SS_TOPK) && topk >= 1) ? min(topk, a.k_cap) : a.k_cap;
    k_eff = greedy ? 1 : emit_k(k, a.V, mode);
  }

  // 3. keys, unit maximum, threshold, emission
  uint4* region = a.cand + (size_t)gu * (size_t)a.cap;
  const uint32_t cap = (uint32_t)a.cap;
  uint32_t t, wm, total, count, cut = 0xFFFFFFFFu;
  if constexpr (DT == SS_BF16) {
    uint32_t rd[16], kd[16];
#pragma unroll
    for (int i = 0; i < NLD; ++i) {
      rd[4 * i + 0] = r[i].x;
      rd[4 * i + 1] = r[i].y;
      rd[4 * i + 2] = r[i].z;
      rd[4 * i + 3] = r[i].w;
    }
    if (mask) {  // masked elements become -inf
#pragma unroll
      for (int i = 0; i < NLD; ++i) {
        const uint32_t bits = mw[i] >> (((i * 64 + ln) * 8) & 31);
#pragma unroll
        for (int w = 0; w < 4; ++w) {
          const uint32_t m = ((uint32_t)((int32_t)(bits << (31 - 2 * w)) >> 31) & 0x0000FFFFu) |
                             ((uint32_t)((int32_t)(bits << (30 - 2 * w)) >> 31) & 0xFFFF0000u);
          rd[4 * i + w] = (rd[4 * i + w] & m) | (~m & 0xFF80FF80u);
        }
      }
    }
#pragma unroll
    for (int j = 0; j < 16; ++j) kd[j] = key2_bf16(rd[j]);
    uint32_t lm = kd[0];
#pragma unroll
    for (int j = 1; j < 16; ++j) lm = pkmax16(lm, kd[j]);
    uint32_t wm16 = wave_max_u32(hmax16(lm));
    if (wm16 > 0xFF80u) {  // a positive NaN in this unit: fold it to invalid
#pragma unroll
      for (int j = 0; j < 16; ++j) kd[j] = fold_nan2(kd[j]);
      lm = kd[0];
#pragma unroll
      for (int j = 1; j < 16; ++j) lm = pkmax16(lm, kd[j]);
      wm16 = wave_max_u32(hmax16(lm));
    }
    if constexpr (LP) {  // the unit's share of the full-row normaliser
      if (usum_row(a, mode, b)) {
        double sl = 0.0;
        if (wm16 >= 0x0081u) {
          const float mu = float_of_key(wm16 << 16), c = lp_scale(lp_tau(a, mode, b));
          double s1 = 0.0;  // two chains of additions
#pragma unroll
          for (int j = 0; j < 16; ++j) {  // -inf terms are zero
            sl += (double)lp_term(__uint_as_float(rd[j] << 16), mu, c);
            s1 += (double)lp_term(__uint_as_float(rd[j] & 0xFFFF0000u), mu, c);
          }
          sl += s1;
        }
        sl = wave_sum(sl);
        if (ln == 0) a.usum[gu] = sl;
      }
    }
    uint32_t t16;
    if (k_eff <= 0) {
      t16 = 0x10000u;  // above every key: nothing emitted
    } else if (wm16 < 0x0081u) {
      t16 = 0x0081u;  // nothing valid
    } else {
      const uint32_t q = (uint32_t)unit_quota(k_eff, a.U, a.V);
      const int G = thr_groups((int)q);
      if (q <= 1) t16 = wm16;
      else if (G == 1) t16 = thr_bf16<1>(kd, q);
      else if (G == 2) t16 = thr_bf16<2>(kd, q);
      else if (G == 4) t16 = thr_bf16<4>(kd, q);
      else if (G == 8) t16 = thr_bf16<8>(kd, q);
      else if (G == 16) t16 = thr_bf16_wide<1>(kd, q, wm16);
      else if (G == 32) t16 = thr_bf16_wide<2>(kd, q, wm16);
      else t16 = 0x0081u;
      t16 = max(t16, 0x0081u);
    }
    uint32_t gmask = 0u, gm[8];
#pragma unroll
    for (int g = 0; g < 8; ++g) {
      gm[g] = hmax16(pkmax16(kd[2 * g], kd[2 * g + 1]));
      gmask |= (gm[g] >= t16) ? (1u << g) : 0u;
    }
    uint32_t off = wave_excl_small((uint32_t)__popc(gmask), total);
    if (total > cap && t16 < 0x10000u) {
      uint32_t cr;
      if (tie_trim<8, 8, 4>(gm, t16, cap, gmask, cr)) {
        cut = (uint32_t)lo + cr;
        off = wave_excl_small((uint32_t)__popc(gmask), total);
      }
    }
    if (total > cap) {
      count = t16 < 0x10000u ? kOvf : 0u;
    } else {
      uint2 gk[8];
#pragma unroll
      for (int g = 0; g < 8; ++g) gk[g] = make_uint2(kd[2 * g], kd[2 * g + 1]);
      count = emit_elems<DT>(gk, gmask, off, total, t16, (uint32_t)lo, region, W);
    }
    // a unit that emitted all it has states the lowest valid key: patched finals are
    // float32 and may lie below every finite bf16 value (a bias of -FLT_MAX)
    const bool whole = t16 == 0x0081u && cut == 0xFFFFFFFFu;
    t = t16 >= 0x10000u ? kNoEmit : (whole ? kKeyFloor : t16 << 16);
    wm = wm16 << 16;
  } else {
    uint32_t kk[32];
#pragma unroll
    for (int i = 0; i < NLD; ++i) {
      kk[4 * i + 0] = key_raw(r[i].x);
      kk[4 * i + 1] = key_raw(r[i].y);
      kk[4 * i + 2] = key_raw(r[i].z);
      kk[4 * i + 3] = key_raw(r[i].w);
    }
    if (mask) {
#pragma unroll
      for (int i = 0; i < NLD; ++i) {
        const uint32_t bits = mw[i] >> (((i * 64 + ln) * 4) & 31);
#pragma unroll
        for (int w = 0; w < 4; ++w) kk[4 * i + w] = ((bits >> w) & 1u) ? kk[4 * i + w] : 0u;
      }
    }
    uint32_t lm = kk[0];
#pragma unroll
    for (int j = 1; j < 32; ++j) lm = max(lm, kk[j]);
    wm = wave_max_u32(lm);
    if (wm > kKeyPosInf) {
#pragma unroll
      for (int j = 0; j < 32; ++j) kk[j] = fold_nan(kk[j]);
      lm = kk[0];
#pragma unroll
      for (int j = 1; j < 32; ++j) lm = max(lm, kk[j]);
      wm = wave_max_u32(lm);
    }
    if constexpr (LP) {  // the unit's share of the full-row normaliser
      if (usum_row(a, mode, b)) {
        double sl = 0.0;
        if (wm >= kKeyFloor) {
          const float mu = float_of_key(wm), c = lp_scale(lp_tau(a, mode, b));
          double s1 = 0.0;  // two chains of additions
#pragma unroll
          for (int j = 0; j < 32; j += 2) {  // invalid keys are those of -inf and below
            sl += (double)lp_term(kk[j] >= kKeyFloor ? float_of_key(kk[j]) : -__builtin_inff(), mu, c);
            s1 += (double)lp_term(kk[j + 1] >= kKeyFloor ? float_of_key(kk[j + 1]) : -__builtin_inff(), mu, c);
          }
          sl += s1;
        }
        sl = wave_sum(sl);
        if (ln == 0) a.usum[gu] = sl;
      }
    }
    if (k_eff <= 0) {
      t = kNoEmit;
    } else if (wm < kKeyFloor) {
      t = kKeyFloor;
    } else {
      const uint32_t q = (uint32_t)unit_quota(k_eff, a.U, a.V);
      const int G = thr_groups((int)q);
      if (q <= 1) t = wm;
      else if (G == 1) t = thr_f32<1>(kk, q);
      else if (G == 2) t = thr_f32<2>(kk, q);
      else if (G == 4) t = thr_f32<4>(kk, q);
      else if (G == 8) t = thr_f32<8>(kk, q);
      else if (G == 16) t = thr_f32<16>(kk, q);
      else if (G == 32) t = thr_f32<32>(kk, q);
      else t = kKeyFloor;
      t = max(t, kKeyFloor);
    }
    uint32_t gmask = 0u, gm[16];
#pragma unroll
    for (int g = 0; g < 16; ++g) {
      gm[g] = max(kk[2 * g], kk[2 * g + 1]);
      gmask |= (t != kNoEmit && gm[g] >= t) ? (1u << g) : 0u;
    }
    uint32_t off = wave_excl_small((uint32_t)__popc(gmask), total);
    if (total > cap && t != kNoEmit) {
      uint32_t cr;
      if (tie_trim<16, 4, 2>(gm, t, cap, gmask, cr)) {
        cut = (uint32_t)lo + cr;
        off = wave_excl_small((uint32_t)__popc(gmask), total);
      }
    }
    if (total > cap) {
      count = kOvf;  // nothing is in gmask when the unit emits nothing
    } else {
      uint2 gk[16];
#pragma unroll
      for (int g = 0; g < 16; ++g) gk[g] = make_uint2(kk[2 * g], kk[2 * g + 1]);
      count = emit_elems<DT>(gk, gmask, off, total, t, (uint32_t)lo, region, W);
    }
  }
  if (ln == 0) {
    a.rec[gu] = make_uint4(t, count, wm, cut);
    if (a.op == OP_VERIFY && u == 0 && row == b * (a.L + 1)) a.res[row].arrived = 0u;
  }
}

// ===========================================================================
// Lists of a row (history, drafts, bias)
// ===========================================================================
__device__ __forceinline__ uint32_t hslot(int id) { return ((uint32_t)id * 2654435761u) >> 21; }  // 11 bits
static_assert(kH == 2048, "hslot assumes 2048 slots");

// linear lookups in the row's lists (last resort, any list length)
__device__ __forceinline__ bool lin_info(const Ctx& c, int id, int* count, bool* hb, float* bsum) {
  int n = 0;
  for (int h = 0; h < c.nhist; ++h) n += c.hist[h] == id;
  for (int h = 0; h < c.nextra; ++h) n += c.extra[h] == id;
  float bs = 0.0f;
  bool has = false;
  for (int e = 0; e < c.nbias; ++e)
    if (c.bias_ids[e] == id) {
      bs = bs + c.bias_vals[e];
      has = true;
    }
  *count = n;
  *hb = has;
  *bsum = bs;
  return n > 0 || has;
}
// entry e of the concatenated list (history, drafts, bias ids)
__device__ __forceinline__ int lin_entry(const Ctx& c, int e) {
  if (e < c.nhist) return c.hist[e];
  e -= c.nhist;
  if (e < c.nextra) return c.extra[e];
  return c.bias_ids[e - c.nextra];
}

// final key of a patched id found by a linear lookup in the row's lists
template <int DT>
__device__ __forceinline__ uint32_t lin_final(const KArgs& a, const Ctx& c, int id) {
  int cn;
  bool hb;
  float bs;
  lin_info(c, id, &cn, &hb, &bs);
  const int Wm = (a.V + 31) >> 5;
  const bool allowed = !c.mask || ((((id >> 5) < Wm ? c.mask[id >> 5] : 0u) >> (id & 31)) & 1u);
  if (!allowed) return 0u;
  return fold_nan(penalised_key(load_elem_bits<DT>(c.xrow, id), c.mode, c.rep, c.freq, c.pres, cn, hb, bs));
}


// ===========================================================================
// Patch tables (workgroups of the streaming launch)
// ===========================================================================
struct PSmem {
  int32_t hk[kH];   // listed id (or -1)
  uint32_t hc[kH];  // occurrence count | has-bias bit 31 | duplicate-bias bit 30
  uint32_t hf[kH];  // bias value, then the final key
  uint32_t flagsw;  // nonzero: more distinct ids than kH slots
  uint32_t pad[3];
};

// Builds a row's patch table: the history, draft and bias ids are counted and
// summed in an LDS hash table (bias entries of one id summed in list order),
// each listed id's raw logit is gathered and its final key computed by the
// Appendix C.1 prologue (Alg. 8 order; grammar-masked ids get the invalid
// key).  The table goes to the workspace slot for slot, with the row's
// status: 0 no lists, 1 table written, 2 more distinct ids than the table
// holds (the merge then builds a table in global memory itself).  It needs
// the logits and the lists only, so it runs beside the row stream.
template <int DT>
__device__ __forceinline__ void patch_row(const KArgs& a, int row, PSmem& P) {
  const int tid = threadIdx.x;
  const Ctx c = make_ctx<DT>(a, row);
  const int ne = c.nhist + c.nextra + c.nbias;
  if (ne == 0) {
    if (tid == 0) a.pstat[row] = 0;
    return;
  }
  int hid0[4];
#pragma unroll
  for (int m = 0; m < 4; ++m) {
    const int h = tid + m * kSBlock;
    hid0[m] = h < c.nhist ? c.hist[h] : -1;
  }
  const int bid0 = tid < c.nbias ? c.bias_ids[tid] : -1;
  const float bval0 = tid < c.nbias ? c.bias_vals[tid] : 0.0f;
  for (int sl = tid; sl < kH / 4; sl += kSBlock) {
    reinterpret_cast<int4*>(P.hk)[sl] = make_int4(-1, -1, -1, -1);
    reinterpret_cast<uint4*>(P.hc)[sl] = make_uint4(0u, 0u, 0u, 0u);
  }
  if (tid == 0) P.flagsw = 0u;
  lds_barrier();
  // a second bias entry for one id sets the "duplicate" bit; the finals then
  // sum that id's entries in list order
  auto ins = [&](int id, uint32_t addc, bool bias, float bval) {
    if (id < 0 || id >= a.V) return;
    uint32_t sl = hslot(id);
#pragma unroll 1
    for (int p = 0; p < kProbe; ++p) {
      const int old = atomicCAS(&P.hk[sl], -1, id);
      if (old == -1 || old == id) {
        if (addc) atomicAdd(&P.hc[sl], addc);
        if (bias) {
          const uint32_t prev = atomicOr(&P.hc[sl], 0x80000000u);
          if (prev & 0x80000000u) atomicOr(&P.hc[sl], 0x40000000u);
          else P.hf[sl] = __float_as_uint(bval);
        }
        return;
      }
      sl = (sl + 1) & (kH - 1);
    }
    P.flagsw = 1u;
  };
#pragma unroll
  for (int m = 0; m < 4; ++m) ins(hid0[m], 1u, false, 0.0f);
  for (int h = tid + 4 * kSBlock; h < c.nhist; h += kSBlock) ins(c.hist[h], 1u, false, 0.0f);  // long histories
  for (int h = tid; h < c.nextra; h += kSBlock) ins(c.extra[h], 1u, false, 0.0f);
  ins(bid0, 0u, true, bval0);
  for (int e = tid + kSBlock; e < c.nbias; e += kSBlock) ins(c.bias_ids[e], 0u, true, c.bias_vals[e]);
  lds_barrier();
  if (P.flagsw != 0u) {
    if (tid == 0) a.pstat[row] = 2;
    return;
  }
  // final keys: every slot's raw logit (and grammar word) is loaded before
  // any is used
  constexpr int kSl = kH / kSBlock;
  const int Wm = (a.V + 31) >> 5;
  int id[kSl];
  uint32_t bits[kSl], mw[kSl];
#pragma unroll
  for (int m = 0; m < kSl; ++m) {
    id[m] = P.hk[tid + m * kSBlock];
    const int ld = id[m] >= 0 ? id[m] : 0;  // element 0 stands in for an empty slot
    bits[m] = load_elem_bits<DT>(c.xrow, ld);
    mw[m] = c.mask ? ((ld >> 5) < Wm ? c.mask[ld >> 5] : 0u) : 0xFFFFFFFFu;
  }
  uint32_t* dst = a.ptab + (size_t)row * 2 * kH;
  if (a.usum) {  // raw keys, for the row's normaliser (the global table's space: unused beside this table)
    uint32_t* raw = a.gfin + (size_t)row * kGH;
#pragma unroll
    for (int m = 0; m < kSl; ++m)
      raw[tid + m * kSBlock] = (id[m] >= 0 && ((mw[m] >> (id[m] & 31)) & 1u)) ? fold_nan(key_raw(bits[m])) : 0u;
  }
#pragma unroll
  for (int m = 0; m < kSl; ++m) {
    const int sl = tid + m * kSBlock;
    uint32_t k = 0u;
    if (id[m] >= 0) {
      const uint32_t hcv = P.hc[sl];
      const bool hb = (hcv >> 31) != 0u;
      float bsum = 0.0f;
      if (hb) {
        if (hcv & 0x40000000u) {  // duplicate bias ids: list order
          for (int e = 0; e < c.nbias; ++e)
            if (c.bias_ids[e] == id[m]) bsum = bsum + c.bias_vals[e];
        } else {
          bsum = 0.0f + __uint_as_float(P.hf[sl]);
        }
      }
      if ((mw[m] >> (id[m] & 31)) & 1u)
        k = fold_nan(penalised_key(bits[m], c.mode, c.rep, c.freq, c.pres, (int)(hcv & 0x3FFFFFFFu), hb, bsum));
    }
    dst[sl] = (uint32_t)id[m];
    dst[kH + sl] = k;
  }
  if (tid == 0) a.pstat[row] = 1;
}

// ===========================================================================
// Kernels
// ===========================================================================
// Streaming kernel: one unit per wavefront, an LDS strip each, no barrier.  Workgroups
// are remapped so that consecutive units (one row) share an XCD and its L2.
// For the operations that apply penalties and bias, the first workgroups of
// the grid build the rows' patch tables (dynamic LDS) beside the stream.
template <int DT, bool LP>
__global__ __launch_bounds__(kSBlock) void ss_stream_kernel(KArgs a) {
  extern __shared__ __align__(16) unsigned char psmem[];
  int bid = blockIdx.x + warm_args();
  if (bid < a.patch_wgs) {  // patch-table workgroups (a multiple of 8) come first
    // on the XCD that streams the row (below), so the gathers of its listed
    // ids and its units' loads share that XCD's L2
    int row = bid;
    if ((a.rows & 7) == 0 && ((a.rows * a.U) & 31) == 0) row = (bid & 7) * (a.rows >> 3) + (bid >> 3);
    if (row < a.rows) patch_row<DT>(a, row, *reinterpret_cast<PSmem*>(psmem));
    return;
  }
  bid -= a.patch_wgs;
  const int nb = a.unit_wgs;
  if (bid < (nb & ~7)) bid = (bid & 7) * (nb >> 3) + (bid >> 3);
  const int gu = __builtin_amdgcn_readfirstlane(bid * kSWaves + wave());
  if (gu < a.rows * a.U) scan_unit<DT, LP>(a, gu, reinterpret_cast<WStage*>(psmem)[wave()]);
}

// ---------------------------------------------------------------------------
// Materialising pass of ss_process_logits: processed logits and final
// probabilities for every element, from the per-row summary; patched ids take
// their final values from the row's patch table (or the merge's list).
// Bound by memory (bf16: 2 bytes read and 8 written per element), so a thread
// takes four consecutive elements: one load, one 16-byte store per output at any
// row alignment.  The tile's patched ids are found by a bit each.  Element by
// element it took 17.5 us at B=32 V=2^17 bf16.
// ---------------------------------------------------------------------------
template <int DT>
__global__ __launch_bounds__(kBlock) void ss_materialize_kernel(KArgs a) {
  constexpr int TILE = 4096, VE = 4, IT = TILE / (VE * kBlock);
  const int tid = threadIdx.x;
  const int T = (a.V + TILE - 1) / TILE;
  const int bid = blockIdx.x + warm_args();
  const int row = bid / T;
  const int tile = bid - row * T;
  const int lo = tile * TILE;
  const int hi = min(a.V, lo + TILE);
  const unsigned char* xrow = reinterpret_cast<const unsigned char*>(a.x) + (size_t)row * (size_t)a.ld * DTT<DT>::ES;
  // raw bits of this thread's elements
  uint32_t x[IT][VE];
#pragma unroll
  for (int t = 0; t < IT; ++t) {
    const int i0 = lo + (t * kBlock + tid) * VE;
    if (i0 + VE <= hi) {
      if constexpr (DT == SS_F32) {
        const uint4 v = load16(xrow + (size_t)i0 * 4);
        x[t][0] = v.x, x[t][1] = v.y, x[t][2] = v.z, x[t][3] = v.w;
      } else {
        uint2 v;
        __builtin_memcpy(&v, xrow + (size_t)i0 * 2, 8);
        x[t][0] = v.x << 16, x[t][1] = v.x & 0xFFFF0000u, x[t][2] = v.y << 16, x[t][3] = v.y & 0xFFFF0000u;
      }
    } else {
#pragma unroll
      for (int e = 0; e < VE; ++e) x[t][e] = i0 + e < hi ? load_elem_bits<DT>(xrow, i0 + e) : 0u;
    }
  }
  const uint32_t mode = a.mode[row] & a.feat;
  const RowSummary s = a.summ[row];
  const uint32_t np = a.npatched[row];
  const uint32_t* mask = (mode & SS_GRAMMAR) ? a.bitmask + (size_t)row * (size_t)a.mask_ld : nullptr;
  const double sitau = 1.0 / (double)s.tau;
  const int Wm = (a.V + 31) >> 5;
  // final keys of this tile's patched ids, and a bit for each
  __shared__ uint32_t pv[TILE];
  __shared__ uint32_t pbit[TILE / 32];
  if (tid < TILE / 32) pbit[tid] = 0u;
  __syncthreads();
  auto put = [&](uint32_t id, uint32_t key) {
    pv[id - lo] = key;
    atomicOr(&pbit[(id - lo) >> 5], 1u << (id & 31));
  };
  if (np == kTable) {
    const uint4* pt = reinterpret_cast<const uint4*>(a.ptab + (size_t)row * 2 * kH);
    for (int w = tid; w < kH / 4; w += kBlock) {
      const uint4 q = pt[w];
      const int ids[4] = {(int)q.x, (int)q.y, (int)q.z, (int)q.w};  // -1: empty slot
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (ids[e] >= lo && ids[e] < hi) put((uint32_t)ids[e], reinterpret_cast<const uint32_t*>(pt)[kH + 4 * w + e]);
    }
  } else if (np != kLinear) {
    const uint2* pl = a.patched + (size_t)row * kGH;
    for (uint32_t j = tid; j < np; j += kBlock) {
      const uint2 e = pl[j];
      if ((int)e.x >= lo && (int)e.x < hi) put(e.x, e.y);
    }
  }
  __syncthreads();
#pragma unroll
  for (int t = 0; t < IT; ++t) {
    const int l = (t * kBlock + tid) * VE;
    const int i0 = lo + l;
    if (i0 >= hi) break;
    const uint32_t mw = mask ? mask[min(i0 >> 5, Wm - 1)] >> (i0 & 31) : 0xFu;
    const uint32_t pb = pbit[l >> 5] >> (l & 31);
    float yo[VE], po[VE];
#pragma unroll
    for (int e = 0; e < VE; ++e) {
      const uint32_t i = (uint32_t)(i0 + e);
      uint32_t k = fold_nan(key_raw(x[t][e]));
      if (!((mw >> e) & 1u)) k = 0u;
      if ((pb >> e) & 1u) k = pv[l + e];
      if (np == kLinear && (int)i < hi) {  // very long lists: look every id up
        const Ctx c = make_ctx<DT>(a, row);
        int cn;
        bool hb;
        float bs;
        if (lin_info(c, (int)i, &cn, &hb, &bs) && k != 0u) k = lin_final<DT>(a, c, (int)i);
      }
      yo[e] = k >= kKeyFloor ? float_of_key(k) : -__builtin_inff();
      float p = 0.0f;
      if (s.kind == KIND_GREEDY) {
        p = (int)i == s.argmax ? 1.0f : 0.0f;
      } else if (s.kind == KIND_DIST && k >= kKeyFloor && comp_of(k, i) >= s.thr) {
        p = (float)(weight_fast((double)float_of_key(k), (double)s.M, sitau) / s.Z);
      }
      po[e] = p;
    }
    const size_t o = (size_t)row * (size_t)a.V + i0;
    if (i0 + VE <= hi) {
      if (a.out_logits) __builtin_memcpy(a.out_logits + o, yo, 16);
      if (a.out_probs) __builtin_memcpy(a.out_probs + o, po, 16);
    } else {
#pragma unroll
      for (int e = 0; e < VE; ++e) {
        if (i0 + e < hi) {
          if (a.out_logits) a.out_logits[o + e] = yo[e];
          if (a.out_probs) a.out_probs[o + e] = po[e];
        }
      }
    }
  }
}

}  // namespace ss
