// ss_row.hpp -- the merge kernel: one workgroup finishes one row.
//
//   1. One round trip loads everything: the request's parameters, the unit
//      records, the first candidates of every unit (a fixed share of threads
//      per unit, issued before the counts are known) and the row's patch table.
//   2. Every emitted element whose composite (key, lower index first) reaches
//      tc, the largest unit threshold, and every patched final value at or above
//      it takes part; raw copies of patched ids drop out by a bitmap.  No unit
//      having overflowed, these are all of the row's elements at or above tc: if
//      at least k of them are, they hold its exact top-k.  Otherwise (skewed or
//      tied rows, patched top tokens) an exact slow path re-reads the units that
//      could hide a top-k element.
//   3. Greedy rows take the maximum.  Other rows are sorted in one pass: a
//      histogram over kNB equal key ranges between tc and the row maximum, a
//      scan, a scatter into bin order, and each element's rank inside its bin by
//      comparing it with the bin's few others.  Bins past the k-th element are
//      left out.  Crowded bins (ties) are split again by their own extent.
//      (Radix selection, two radix searches for the cuts and a bitonic sort for
//      lists took 26.8 us at B=64 V=2^17 bf16 with a 64-entry list, 87 us for
//      top-k at B=256 V=2^18 fp32 k<=4096; this takes 7.4 and 16.9 us.)
//   4. On the sorted list the Alg. 11 epilogue is one prefix sum of 2^-50
//      fixed-point weights: top-p, min-p and the draw are each the first rank
//      whose running mass crosses a target, found by the one thread that holds it.
//
// What bounds it is latency: a row is one workgroup's chain of one global round
// trip, eleven barriers (LDS only, so loads stay in flight across them) and some
// 1500 instructions a wavefront at four cycles each, hence straight-line code for
// the usual numbers of loads and list entries.  B=64 V=2^17 bf16 sampling: 19.6 us
// with the pool, radix and key-bin stages this replaced, 10.9 us now.
#pragma once
#include <type_traits>

#include "ss_impl.hpp"

namespace ss {

constexpr int kNBLog = 11;
constexpr int kNB = 1 << kNBLog;  // key bins of the one-pass sort
constexpr int kCrowd = 256;       // bins up to this occupancy are ranked by comparison
constexpr uint32_t kNone = 0xFFFFFFFFu;

// Threads of a merge workgroup.  A wavefront issues a dependent instruction
// every four cycles and a SIMD keeps two wavefronts at that rate, so 512 threads
// run the fixed part of a row (reductions, scans) as fast as one wavefront
// would; 1024 made every row of up to 1024 entries slower (this merge in an earlier
// form, now 10.8 and 7.4 us: B=64 V=2^17 bf16 sampling 12.4 -> 13.9 us, its 64-entry
// lists 8.9 -> 11.5 us).  Top-k alone lists up to 4096 entries and has little else to do:
// 1024.
template <int OP>
constexpr int merge_threads() {
  return OP == OP_TOPK ? 1024 : kBlock;
}
constexpr int kMaxWaves = 16;

struct MSmem {
  uint64_t x64[3][kMaxWaves];  // scratch of the workgroup reductions
  double rd[kMaxWaves];
  uint32_t x32[4][kMaxWaves];
  uint64_t bc64[4];
  uint32_t bc[12];
  uint64_t best;               // greedy rows: the maximum
  uint4 wred[kMaxWaves];       // per wave: largest threshold key, its lowest cut, row maximum, longest list
  uint32_t rmask[kMaxU / 32];  // units re-read by the slow path
  alignas(16) uint32_t pbits[kPB / 32];  // bit pbit(id) set for every patched id
  int32_t hk[kH];                        // patched id (or -1)
  uint32_t hf[kH];                       // final key
  alignas(16) uint32_t bins[kNB];        // counts, then starts, then ends; the slow path's digit counts
};
constexpr int kSmemFixed = (int)((sizeof(MSmem) + 15) & ~(size_t)15);
// The sorted list (rank loops read up to three entries past a bin), and the staging
// area of its sort before it: room for the k_cap leading elements and the rest of the
// bin that holds the last of them.  Bins of tied fp32 values are as long as their ties,
// so it holds 2 k_cap + 128 (at least 1024) elements, but at most 2560 more than the
// list (sort_ranges keeps a thread's share in registers) and up to k_cap = 2048 only
// what lets two workgroups share a CU's 160 KB, at least 864 more than the list.
// (512 more beyond 1088: sampling of 4096 at B=32 V=2^17 fp32 with values in steps of a
// quarter took the slow path, 145 us.)
__host__ __device__ constexpr int sorted_cap(int k_cap) { return k_cap + 8; }
__host__ __device__ constexpr int stage_cap(int k_cap) {
  const int most = (k_cap < 2432 ? 2 * k_cap + 128 : k_cap + 2560) + 255;
  const int t = most > 1024 ? most & ~255 : 1024;
  const int two = ((80 * 1024 - kSmemFixed) / 8 - sorted_cap(k_cap)) & ~31;
  return k_cap <= 2048 && two < t ? two : t;
}
constexpr int merge_smem(int k_cap) { return kSmemFixed + 8 * (stage_cap(k_cap) + sorted_cap(k_cap)); }
static_assert(merge_smem(SS_MAX_K) <= 160 * 1024, "merge LDS beyond a CU's 160 KiB");
// The verification epilogue keeps a sparse draft list (one 64-bit entry per
// listed id) over the patch bitmap and table, which are dead by then.
static_assert(offsetof(MSmem, hk) == offsetof(MSmem, pbits) + sizeof(uint32_t) * (kPB / 32) &&
                  offsetof(MSmem, hf) == offsetof(MSmem, hk) + sizeof(int32_t) * kH &&
                  offsetof(MSmem, pbits) % 8 == 0 &&
                  sizeof(uint32_t) * (kPB / 32 + 2 * kH) >= sizeof(uint64_t) * SS_MAX_K,
              "sparse draft list view");
__device__ __forceinline__ uint64_t* qlist_view(MSmem& S) { return reinterpret_cast<uint64_t*>(S.pbits); }

// A value read from LDS that every thread knows to be the same.
__device__ __forceinline__ uint32_t uniform(uint32_t v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ uint64_t uniform(uint64_t v) {
  return ((uint64_t)uniform((uint32_t)(v >> 32)) << 32) | uniform((uint32_t)v);
}

// Workgroup reductions (scratch reusable on return).
template <int BS, typename T, typename Op>
__device__ __forceinline__ T wg_reduce(T v, T* scratch, Op op) {
  v = wave_reduce(v, op);
  if (lane() == 0) scratch[wave()] = v;
  lds_barrier();
  T r = scratch[0];
#pragma unroll
  for (int w = 1; w < BS / 64; ++w) r = op(r, scratch[w]);
  lds_barrier();
  return r;
}
template <int BS, typename T>
__device__ __forceinline__ T wg_sum(T v, T* scratch) {
  return wg_reduce<BS>(v, scratch, [](T x, T y) { return x + y; });
}
template <int BS, typename T>
__device__ __forceinline__ T wg_max(T v, T* scratch) {
  return wg_reduce<BS>(v, scratch, [](T x, T y) { return x > y ? x : y; });
}

// Patched-id bitmap position: the id itself when V <= kPB (the bitmap is then
// exact), else a 17-bit hash (a set bit then needs a table lookup).
__device__ __forceinline__ uint32_t pbit(int id, bool exact) {
  return exact ? (uint32_t)id : (((uint32_t)id * 0x9E3779B1u) >> (32 - kPBLog));
}
// false only when id is certainly not patched (one LDS read)
__device__ __forceinline__ bool maybe_patched(const MSmem& S, int id, bool exact) {
  const uint32_t h = pbit(id, exact);
  return (S.pbits[h >> 5] >> (h & 31)) & 1u;
}
__device__ __forceinline__ int hfind(const MSmem& S, int id) {
  uint32_t s = hslot(id);
#pragma unroll 1
  for (int p = 0; p < kProbe; ++p) {
    const int k = S.hk[s];
    if (k == id) return (int)s;
    if (k < 0) return -1;
    s = (s + 1) & (kH - 1);
  }
  return -1;
}
__device__ __forceinline__ bool lds_patched(const MSmem& S, int id, bool exact) {
  return maybe_patched(S, id, exact) && (exact || hfind(S, id) >= 0);
}


// ---------------------------------------------------------------------------
// Patch table of a row in global memory, used when the row's history and
// bias lists hold more distinct ids than the LDS table: open addressing over
// kGH slots.  The row's merge clears the tags before it inserts (a tag of
// generation `gen` marks a slot of this call), so nothing depends on what the
// workspace held before the call.
// ---------------------------------------------------------------------------
struct PatchG {
  uint64_t* tag;
  uint32_t* cnt;
  uint32_t* fin;
  uint32_t gen;
};
__device__ __forceinline__ uint32_t ghslot(int id) { return ((uint32_t)id * 2654435761u) >> 18; }  // 14 bits
static_assert(kGH == 16384, "ghslot assumes 16384 slots");

__device__ __forceinline__ int gfind(const PatchG& g, int id) {
  const uint64_t want = ((uint64_t)g.gen << 32) | (uint32_t)(id + 1);
  uint32_t s = ghslot(id);
  for (int p = 0; p < kGProbe; ++p) {
    const uint64_t t = __hip_atomic_load(&g.tag[s], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (t == want) return (int)s;
    if ((uint32_t)(t >> 32) != g.gen) return -1;
    s = (s + 1) & (kGH - 1);
  }
  return -1;
}
// claims a slot for id (the claiming thread zeroes its count); -1 when full
__device__ __forceinline__ int gclaim(const PatchG& g, int id) {
  const uint64_t want = ((uint64_t)g.gen << 32) | (uint32_t)(id + 1);
  uint32_t s = ghslot(id);
  for (int p = 0; p < kGProbe; ++p) {
    uint64_t t = __hip_atomic_load(&g.tag[s], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    for (;;) {
      if (t == want) return (int)s;
      if ((uint32_t)(t >> 32) == g.gen) break;  // another id of this call
      const uint64_t old = atomicCAS((unsigned long long*)&g.tag[s], (unsigned long long)t, (unsigned long long)want);
      if (old == t) {
        g.cnt[s] = 0u;
        return (int)s;
      }
      t = old;
    }
    s = (s + 1) & (kGH - 1);
  }
  return -1;
}

// patch modes: 0 none, 1 LDS table, 2 global table, 3 linear lookups
template <int DT>
__device__ __forceinline__ bool is_patched(const Ctx& c, const MSmem& S, int pmode, const PatchG& g, int id) {
  if (pmode == 0) return false;
  if (pmode == 1) return lds_patched(S, id, c.pexact);
  if (pmode == 2) return gfind(g, id) >= 0;
  int cn;
  bool hb;
  float bs;
  return lin_info(c, id, &cn, &hb, &bs);
}

// Builds the row's patch table in global memory when its lists hold more
// distinct ids than the LDS table (status 2); returns the patch mode: 2, or 3
// (linear lookups) when that table overflows too.
template <int DT, int BS>
__device__ __forceinline__ int global_table(const KArgs& a, const Ctx& c, MSmem& S, int row, PatchG& pg) {
  const int tid = threadIdx.x;
  const int Wm = (a.V + 31) >> 5;
  pg.tag = a.gtag + (size_t)row * kGH;
  pg.cnt = a.gcnt + (size_t)row * kGH;
  pg.fin = a.gfin + (size_t)row * kGH;
  // cleared first (its contents before the call are unspecified)
  for (int sl = tid; sl < kGH / 2; sl += BS) reinterpret_cast<uint4*>(pg.tag)[sl] = make_uint4(0u, 0u, 0u, 0u);
  pg.gen = 1u;
  if (tid == 0) S.bc[9] = 0u;
  __threadfence();
  __syncthreads();
  const int ne = c.nhist + c.nextra + c.nbias;
  bool full = false;
  for (int e = tid; e < ne; e += BS) {
    const int id = lin_entry(c, e);
    if (id >= 0 && id < a.V && gclaim(pg, id) < 0) full = true;
  }
  if (full) S.bc[9] = 1u;
  __threadfence();
  __syncthreads();
  if (S.bc[9] != 0u) return 3;
  for (int e = tid; e < ne; e += BS) {
    const int id = lin_entry(c, e);
    if (id < 0 || id >= a.V) continue;
    const int sl = gfind(pg, id);
    if (e < c.nhist + c.nextra) atomicAdd(&pg.cnt[sl], 1u);
    else atomicOr(&pg.cnt[sl], 0x80000000u);
  }
  __threadfence();
  __syncthreads();
  for (int sl = tid; sl < kGH; sl += BS) {
    const uint64_t t = pg.tag[sl];
    if ((uint32_t)(t >> 32) != pg.gen) continue;
    const int id = (int)((uint32_t)t - 1u);
    const uint32_t hcv = pg.cnt[sl];
    const bool hb = (hcv >> 31) != 0u;
    float bsum = 0.0f;
    if (hb) {
      for (int e = 0; e < c.nbias; ++e)
        if (c.bias_ids[e] == id) bsum = bsum + c.bias_vals[e];
    }
    const bool allowed = !c.mask || ((((id >> 5) < Wm ? c.mask[id >> 5] : 0u) >> (id & 31)) & 1u);
    pg.fin[sl] = allowed ? fold_nan(penalised_key(load_elem_bits<DT>(c.xrow, id), c.mode, c.rep, c.freq,
                                                  c.pres, (int)(hcv & 0x7FFFFFFFu), hb, bsum))
                         : 0u;
  }
  __threadfence();
  __syncthreads();
  return 2;
}

// ---------------------------------------------------------------------------
// Exact slow path: writes to pool elements that include the row's `want`
// largest composites (raw copies of patched ids left out, patched finals
// among them) and returns their number.  v0, at or just below the want-th
// largest element among the emitted ones, bounds the k-th of the row from below,
// so only units whose threshold lies above v0 (or that overflowed) can hide a
// top-k element: they are re-read whole, and everything at or above v0 is collected
// (if that is more than the pool holds, after a second selection).  want == 1 needs
// the maximum only.  One visiting loop serves every pass: its operation is `op`.
// Passes are what it costs, and in them adds of many threads to one digit's count:
// hence a bound found to the digit that suffices, and runs added at once (top-k of
// 1024 at B=32 V=5000 bf16, 700 of the largest in one unit: 92.7 -> 35.3 us; of 4096
// in a tied row at V=2^17: 536 -> 205 us).
// ---------------------------------------------------------------------------
template <int DT, int BS>
__device__ __forceinline__ int slow_select(const KArgs& a, const Ctx& c, MSmem& S, uint64_t* pool, int pmode,
                                           const PatchG& pg, uint32_t want) {
  enum { V_KEY, V_IDX, V_COLLECT, V_MAX };
  constexpr int VW = DTT<DT>::VW, EPW = DT == SS_BF16 ? 1 : 2;  // words of a candidate
  const int tid = threadIdx.x;
  const int U = a.U;
  const int W = (a.V + 31) >> 5;
  int op = want == 1u ? V_MAX : V_KEY;
  bool second = false;            // the marked units are re-read
  uint64_t thr = 0ull;            // composites at or above it are the wanted ones (so far)
  // goal: elements to select; need: those of them below the digits found so far
  uint32_t goal = want, need = want, prefix = 0u, ip = 0u;
  int sh = 24, ib = 10;
  for (;;) {
    for (int i = tid; i < 1024; i += BS) S.bins[i] = 0u;
    if (tid == 0) S.bc[8] = 0u;
    lds_barrier();
    uint64_t best = 0ull;
    // digit counts, a thread's run of one digit added at once: tied and close keys
    // share their digits, and adds to one address wait for each other
    uint32_t digit = 0u, run = 0u;
    auto count_digit = [&](uint32_t d) {
      if (d != digit) {
        if (run != 0u) atomicAdd(&S.bins[digit], run);
        digit = d;
        run = 0u;
      }
      ++run;
    };
    auto apply = [&](uint32_t k, uint32_t i) {
      if (k < kKeyFloor || is_patched<DT>(c, S, pmode, pg, (int)i)) return;
      const uint64_t cm = comp_of(k, i);
      if (cm < thr) return;
      if (op == V_MAX) {
        best = max(best, cm);
      } else if (op == V_KEY) {
        if (sh == 24 || (k >> (sh + 8)) == prefix) count_digit((k >> sh) & 255u);
      } else if (op == V_IDX) {
        if (k == prefix && (ib == 10 || (i >> 10) == ip)) count_digit((i >> ib) & 1023u);
      } else {
        const uint32_t p = atomicAdd(&S.bc[8], 1u);
        if (p < (uint32_t)a.pcap) pool[p] = cm;
      }
    };
    // 1. candidates of the units that are not marked
    {
      const int tpu = a.tpu;
      const int u = (tid * a.tpu_inv) >> 20, sub = tid - u * tpu;
      const bool act = u < U && !((S.rmask[u >> 5] >> (u & 31)) & 1u);
      const size_t g = (size_t)c.row * U + (u < U ? u : 0);
      const uint32_t cn = act ? a.rec[g].y : 0u;
      const uint32_t* src = reinterpret_cast<const uint32_t*>(a.cand + g * a.cap);
      // four loads in flight (one at a time: a tied row's top 4096 with penalties at
      // B=32 V=2^17 bf16 took 940 us, now 775)
      constexpr int ND = 4;
#pragma unroll 1
      for (uint32_t i = (uint32_t)sub; i < cn; i += (uint32_t)(ND * tpu)) {
        uint32_t lo[ND], hi[ND];
#pragma unroll
        for (int j = 0; j < ND; ++j) {
          const uint32_t at = min(i + (uint32_t)(j * tpu), cn - 1u) * EPW;
          lo[j] = src[at];
          if constexpr (DT == SS_F32) hi[j] = src[at + 1];
        }
#pragma unroll 1
        for (uint32_t at = i; at < min(i + (uint32_t)(ND * tpu), cn); at += (uint32_t)tpu) {
          if constexpr (DT == SS_BF16) apply(lo[0] & 0xFFFF0000u, (uint32_t)(u * kUE) + 0xFFFFu - (lo[0] & 0xFFFFu));
          else apply(hi[0], ~lo[0]);
#pragma unroll
          for (int j = 1; j < ND; ++j) {
            lo[j - 1] = lo[j];
            if constexpr (DT == SS_F32) hi[j - 1] = hi[j];
          }
        }
      }
    }
    // 2. every element of the marked units (grammar mask applied, NaN
    // invalid): eight of them at a time, a share of the threads each
    if (second) {
      constexpr int SH = BS / 8;  // threads per unit
      int nth = tid / SH;         // this share's unit: the nth marked one
      int seen = 0;
      for (int w = 0; w < (U + 31) >> 5; ++w) {
        uint32_t mk = S.rmask[w];
        while (mk) {
          const int u = w * 32 + __builtin_ctz(mk);
          mk &= mk - 1u;
          if (seen++ != nth) continue;
          nth += 8;
          const int lo = u * kUE;
#pragma unroll 1
          for (int l0 = (tid & (SH - 1)) * VW; l0 < kUE; l0 += SH * VW) {
            uint32_t w4[4] = {0u, 0u, 0u, 0u};
            if (lo + l0 + VW <= a.V) {
              const uint4 r = load16(c.xrow + (size_t)(lo + l0) * DTT<DT>::ES);
              w4[0] = r.x;
              w4[1] = r.y;
              w4[2] = r.z;
              w4[3] = r.w;
            } else {
#pragma unroll
              for (int e = 0; e < VW; ++e) {
                if (lo + l0 + e < a.V) {
                  const uint32_t bits = load_elem_bits<DT>(c.xrow, lo + l0 + e);
                  if constexpr (DT == SS_F32) w4[e] = bits;
                  else w4[e >> 1] |= (bits >> 16) << (16 * (e & 1));
                }
              }
            }
            uint32_t mw = 0xFFFFFFFFu;
            if (c.mask) {
              const int wi = (lo + l0) >> 5;
              mw = wi < W ? (c.mask[wi] >> ((lo + l0) & 31)) : 0u;
            }
#pragma unroll 1
            for (int e = 0; e < VW; ++e) {
              const int i = lo + l0 + e;
              if (i >= a.V) break;
              uint32_t bits;
              if constexpr (DT == SS_F32) {
                bits = w4[0];
                w4[0] = w4[1];
                w4[1] = w4[2];
                w4[2] = w4[3];
              } else {
                bits = w4[0] << 16;
                w4[0] = (w4[0] >> 16) | (w4[1] << 16);
                w4[1] = (w4[1] >> 16) | (w4[2] << 16);
                w4[2] = (w4[2] >> 16) | (w4[3] << 16);
                w4[3] >>= 16;
              }
              uint32_t k = fold_nan(key_raw(bits));
              if (!((mw >> e) & 1u)) k = 0u;
              apply(k, (uint32_t)i);
            }
          }
        }
      }
    }
    // 3. patched final values
    auto final_value = [&](uint32_t k, uint32_t id) {
      const uint64_t cm = comp_of(k, id);
      if (k < kKeyFloor || cm < thr) return;
      if (op == V_MAX) {
        best = max(best, cm);
      } else if (op == V_KEY) {
        if (sh == 24 || (k >> (sh + 8)) == prefix) count_digit((k >> sh) & 255u);
      } else if (op == V_IDX) {
        if (k == prefix && (ib == 10 || (id >> 10) == ip)) count_digit((id >> ib) & 1023u);
      } else {
        const uint32_t p = atomicAdd(&S.bc[8], 1u);
        if (p < (uint32_t)a.pcap) pool[p] = cm;
      }
    };
    const int nf = pmode == 1 ? kH : (pmode == 2 ? kGH : (pmode == 3 ? c.nhist + c.nextra + c.nbias : 0));
#pragma unroll 1
    for (int sl = tid; sl < nf; sl += BS) {
      int id = -1;
      uint32_t k = 0u;
      if (pmode == 1) {
        id = S.hk[sl];
        k = S.hf[sl];
      } else if (pmode == 2) {
        const uint64_t t = pg.tag[sl];
        if ((uint32_t)(t >> 32) == pg.gen) {
          id = (int)((uint32_t)t - 1u);
          k = pg.fin[sl];
        }
      } else {
        id = lin_entry(c, sl);
        for (int e2 = 0; e2 < sl && id >= 0; ++e2)
          if (lin_entry(c, e2) == id) id = -1;  // listed before
        if (id >= 0 && id < a.V) k = lin_final<DT>(a, c, id);
        else id = -1;
      }
      if (id >= 0) final_value(k, (uint32_t)id);
    }
    if (run != 0u) atomicAdd(&S.bins[digit], run);
    lds_barrier();

    // what the pass found
    bool have_thr = false;
    if (op == V_MAX) {
      best = uniform(wg_max<BS>(best, S.x64[0]));
      if (second) {
        if (tid == 0) pool[0] = best;
        lds_barrier();
        return best != 0ull ? 1 : 0;
      }
      thr = best;
      have_thr = true;
    } else if (op == V_COLLECT) {
      const uint32_t n = uniform(S.bc[8]);
      if (n <= (uint32_t)a.pcap) {
        lds_barrier();
        return (int)n;
      }
      goal = need = min(want, n);
      sh = 24;
      prefix = 0u;
      op = V_KEY;
    } else {
      // the digit holding the need-th element: keys descending, indices ascending
      const bool key = op == V_KEY;
      const int nb = key ? 256 : 1024;
      constexpr int PER = 1024 / BS;
      uint32_t h[PER], s = 0u;
#pragma unroll
      for (int q = 0; q < PER; ++q) {
        const int r = tid * PER + q;
        h[q] = r < nb ? S.bins[key ? nb - 1 - r : r] : 0u;
        s += h[q];
      }
      const uint32_t inc = wave_incl_scan(s);
      if (lane() == 63) S.x32[0][wave()] = inc;
      lds_barrier();
      uint32_t run = inc - s, total = 0u;
      for (int w = 0; w < BS / 64; ++w) {
        const uint32_t x = S.x32[0][w];
        if (w < wave()) run += x;
        total += x;
      }
      total = uniform(total);
#pragma unroll
      for (int q = 0; q < PER; ++q) {
        const int r = tid * PER + q;
        if (run < need && run + h[q] >= need) {
          S.bc[4] = (uint32_t)(key ? nb - 1 - r : r);
          S.bc[5] = run;
          S.bc[6] = h[q];
        }
        run += h[q];
      }
      lds_barrier();
      const uint32_t d = uniform(S.bc[4]), before = uniform(S.bc[5]), hd = uniform(S.bc[6]);
      // a bound with an eighth more elements above it will do: it saves the last digits'
      // passes, and few more units than the exact one has them re-read (a bound that fills
      // half of the pool re-read every unit of rows with one dense one); once the units are
      // read, whatever the pool holds
      const uint32_t slack = (uint32_t)a.pcap - goal;
      const uint32_t room = goal + (second ? slack : min(goal / 8u + 16u, slack / 2u));
      if (total < need) {  // too few emitted: everything valid takes part
        thr = comp_of(kKeyFloor, kNone);
        have_thr = true;
      } else {
        need -= before;
        const bool fits = goal - need + hd <= room;
        if (key) {
          prefix = (prefix << 8) | d;
          if (fits) {
            thr = comp_of(max(prefix << sh, kKeyFloor), kNone);
            have_thr = true;
          } else if (sh == 0 || (DT == SS_BF16 && pmode == 0 && sh == 16)) {  // (raw bf16 keys end here)
            prefix <<= sh;
            op = V_IDX;
            ib = 10;
          } else {
            sh -= 8;
          }
        } else if (ib == 10 && !fits) {
          ip = d;
          ib = 0;
        } else {
          const uint32_t last = ib == 10 ? (d << 10) | 1023u : (ip << 10) | d;
          thr = comp_of(prefix, last);
          have_thr = true;
        }
      }
    }
    if (have_thr) {
      if (!second) {
        // units whose threshold (ties cut by index) lies above the bound
        for (int u = tid; u < U; u += BS) {
          const uint4 r4 = a.rec[(size_t)c.row * U + u];
          if (r4.x != kNoEmit && comp_of(r4.x, r4.w) > thr) atomicOr(&S.rmask[u >> 5], 1u << (u & 31));
        }
        second = true;
      }
      if (op != V_MAX) op = V_COLLECT;
    }
    lds_barrier();
  }
}

// The slow path of rows that want one element (a greedy row whose largest raw
// logits are all patched: a penalised top token).  The best unpatched candidate
// or final value bounds every unit whose threshold is no higher; the few others
// are re-read whole, one per wavefront, all their loads in flight together.  The
// general slow path took three passes, each element by element: 5 us more for a
// call with one such row.
template <int DT, int BS>
__device__ __forceinline__ int greedy_refill(const KArgs& a, const Ctx& c, MSmem& S, uint64_t* pool, bool patch) {
  constexpr int VW = DTT<DT>::VW, NLD = DTT<DT>::NLD, EPW = DT == SS_BF16 ? 1 : 2;
  const int tid = threadIdx.x, ln = lane();
  const int tpu = a.tpu;
  const int u = (tid * a.tpu_inv) >> 20, sub = tid - u * tpu;
  const bool act = u < a.U;
  const size_t g = (size_t)c.row * a.U + (act ? u : 0);
  const uint4 r4 = a.rec[g];
  const uint32_t* src = reinterpret_cast<const uint32_t*>(a.cand + g * a.cap);
  if (tid == 0) S.bc[8] = 0u;
  uint64_t best = 0ull;
  for (uint32_t i = (uint32_t)sub; act && i < r4.y; i += (uint32_t)tpu) {
    const uint32_t w = src[i * EPW];
    uint64_t cm;
    if constexpr (DT == SS_BF16) cm = comp_of(w & 0xFFFF0000u, (uint32_t)(u * kUE) + 0xFFFFu - (w & 0xFFFFu));
    else cm = ((uint64_t)src[i * EPW + 1] << 32) | w;
    if (cm > best && !(patch && lds_patched(S, (int)comp_idx(cm), c.pexact))) best = cm;
  }
  if (patch) {
    for (int sl = tid; sl < kH; sl += BS)
      if (S.hk[sl] >= 0 && S.hf[sl] >= kKeyFloor) best = max(best, comp_of(S.hf[sl], (uint32_t)S.hk[sl]));
  }
  best = uniform(wg_max<BS>(best, S.x64[0]));
  if (act && sub == 0 && r4.x != kNoEmit && comp_of(r4.x, r4.w) > best) S.bins[atomicAdd(&S.bc[8], 1u)] = (uint32_t)u;
  lds_barrier();
  const int nre = (int)uniform(S.bc[8]);
#pragma unroll 1
  for (int j = __builtin_amdgcn_readfirstlane(wave()); j < nre; j += BS / 64) {
    const int lo = (int)uniform(S.bins[j]) * kUE;
    uint4 r[NLD];
    uint32_t mw[NLD];
#pragma unroll
    for (int i = 0; i < NLD; ++i) {
      const int l0 = lo + (i * 64 + ln) * VW;
      r[i] = make_uint4(kNone, kNone, kNone, kNone);  // negative NaN: invalid
      mw[i] = kNone;
      if (l0 + VW <= a.V) r[i] = load16(c.xrow + (size_t)l0 * DTT<DT>::ES);
      if (c.mask && l0 < a.V) mw[i] = c.mask[l0 >> 5] >> (l0 & 31);
    }
#pragma unroll
    for (int i = 0; i < NLD; ++i) {
      const int l0 = lo + (i * 64 + ln) * VW;
      const uint32_t w4[4] = {r[i].x, r[i].y, r[i].z, r[i].w};
      const bool part = l0 < a.V && l0 + VW > a.V;  // the row's last chunk
#pragma unroll
      for (int e = 0; e < VW; ++e) {
        uint32_t bits;
        if constexpr (DT == SS_F32) bits = w4[e];
        else bits = (e & 1) ? w4[e >> 1] & 0xFFFF0000u : w4[e >> 1] << 16;
        if (part && l0 + e < a.V) bits = load_elem_bits<DT>(c.xrow, l0 + e);
        const uint32_t k = ((mw[i] >> e) & 1u) ? fold_nan(key_raw(bits)) : 0u;
        const uint64_t cm = comp_of(k, (uint32_t)(l0 + e));
        if (k >= kKeyFloor && cm > best && !(patch && lds_patched(S, l0 + e, c.pexact))) best = cm;
      }
    }
  }
  best = wg_max<BS>(best, S.x64[1]);
  if (tid == 0) pool[0] = best;
  lds_barrier();
  return best != 0ull ? 1 : 0;
}

// This thread's share of the full-row normaliser sum_j exp((y_j - M) / tau)
// over the row's valid processed logits, for rows whose lists exceed the LDS
// table: every element's processed value.
template <int DT, int BS>
__device__ __forceinline__ double row_norm_all(const KArgs& a, const Ctx& c, const MSmem& S, int pmode, const PatchG& pg,
                                               double M, double tau) {
  const int Wm = (a.V + 31) >> 5;
  double z = 0.0;
#pragma unroll 1
  for (int i = threadIdx.x; i < a.V; i += BS) {
    uint32_t k = fold_nan(key_raw(load_elem_bits<DT>(c.xrow, i)));
    if (c.mask && !((((i >> 5) < Wm ? c.mask[i >> 5] : 0u) >> (i & 31)) & 1u)) k = 0u;
    if (is_patched<DT>(c, S, pmode, pg, i)) k = pmode == 2 ? pg.fin[gfind(pg, i)] : lin_final<DT>(a, c, i);
    if (k >= kKeyFloor) z += exp(((double)float_of_key(k) - M) / tau);
  }
  return z;
}

// This thread's share of the normaliser terms, relative to M, of the n units listed in
// `units`, ids in the LDS patch table left out.  The workgroup reads a unit at a time,
// a few consecutive logits per thread, the next unit's loads ahead of this one's terms.
template <int DT, int BS>
__device__ __forceinline__ double units_norm(const KArgs& a, const MSmem& S, int row, uint32_t mode,
                                             const uint32_t* units, int n, float M, float c) {
  constexpr int VE = kUE / BS, ES = DTT<DT>::ES;
  static_assert(32 % VE == 0, "a thread's logits share a word of the mask");
  const unsigned char* xrow = reinterpret_cast<const unsigned char*>(a.x) + (size_t)row * (size_t)a.ld * ES;
  const uint32_t* mask = (mode & SS_GRAMMAR) ? a.bitmask + (size_t)row * (size_t)a.mask_ld : nullptr;
  const bool pexact = a.V <= kPB;
  uint32_t x[VE], mw = 0u, nx[VE], nmw = 0u;  // raw bits and allow bits, of this unit and the next
  auto load = [&](int j, uint32_t (&r)[VE], uint32_t& m) {
    const int i0 = (int)uniform(units[j]) * kUE + (int)threadIdx.x * VE;
    m = i0 < a.V ? (mask ? mask[i0 >> 5] >> (i0 & 31) : kNone) : 0u;
#pragma unroll
    for (int e = 0; e < VE; ++e) r[e] = load_elem_bits<DT>(xrow, min(i0 + e, a.V - 1));
#pragma unroll
    for (int e = 0; e < VE; ++e) m &= i0 + e < a.V ? ~0u : ~(1u << e);
  };
  double z = 0.0;
  load(0, x, mw);
#pragma unroll 1
  for (int j = 0; j < n; ++j) {
    if (j + 1 < n) load(j + 1, nx, nmw);
    const int i0 = (int)uniform(units[j]) * kUE + (int)threadIdx.x * VE;
#pragma unroll
    for (int e = 0; e < VE; ++e) {
      const bool in = ((mw >> e) & 1u) && !lds_patched(S, i0 + e, pexact);
      z += in ? (double)lp_term(__uint_as_float(x[e]), M, c) : 0.0;  // -inf and NaN give zero
      x[e] = nx[e];
    }
    mw = nmw;
  }
  return z;
}

// Sums of the NW wave totals in scratch: of those before this wave, and of all
// (one read and a few DPP steps per lane instead of a loop over the waves).
template <int NW, typename T>
__device__ __forceinline__ void wave_prefix(const T* scratch, int wv, T& before, T& total) {
  const int w = lane() & (NW - 1);
  T x = scratch[w];
  T y = w < wv ? x : T(0);
  auto step = [&](auto c) {
    constexpr int C = decltype(c)::value;
    x += dppT<T, C>(x, x);
    y += dppT<T, C>(y, y);
  };
  step(std::integral_constant<int, 0xB1>{});   // quad_perm [1,0,3,2]
  step(std::integral_constant<int, 0x4E>{});   // quad_perm [2,3,0,1]
  step(std::integral_constant<int, 0x141>{});  // row_half_mirror
  static_assert(NW == 8 || NW == 16, "wave totals fill half a row or a row");
  if constexpr (NW == 16) step(std::integral_constant<int, 0x140>{});  // row_mirror
  before = y;
  total = x;
}

// Rank of e among the staged entries [bs, be) of its bin, from the list's start.
__device__ __forceinline__ uint32_t rank_in_bin(const uint64_t* stage, uint64_t e, uint32_t bs, uint32_t be) {
  uint32_t r = bs;
  for (uint32_t j = bs; j < be; j += 4u) {
    const uint64_t s0 = stage[j], s1 = stage[j + 1u], s2 = stage[j + 2u], s3 = stage[j + 3u];
    r += (s0 > e ? 1u : 0u) + ((j + 1u < be && s1 > e) ? 1u : 0u) + ((j + 2u < be && s2 > e) ? 1u : 0u) +
         ((j + 3u < be && s3 > e) ? 1u : 0u);
  }
  return r;
}

// Lists with crowded bins (ties, or a few outliers that stretch the key range) and those
// of the slow path.  Ranges of `stage` still to be sorted, start << 16 | end, are kept in
// the wavefronts' record words, their number in bc[5].
static_assert(stage_cap(SS_MAX_K) / kCrowd <= 4 * kMaxWaves && stage_cap(SS_MAX_K) < 65536,
              "ranges are disjoint and longer than kCrowd");
__device__ __forceinline__ uint32_t* ranges(MSmem& S) { return reinterpret_cast<uint32_t*>(S.wred); }

// Entries [s0, s1) of `stage`, in the bins of `bin` (S.bins holds their ends): those of
// small bins to their place in `sorted`, crowded bins to the ranges, or, when a bin is
// one composite (`last`), as they stand.
template <int BS, typename Bin>
__device__ __forceinline__ void place_or_defer(MSmem& S, const uint64_t* stage, uint64_t* sorted, uint32_t s0,
                                               uint32_t s1, uint32_t want, int tid, bool last, Bin&& bin) {
#pragma unroll 1
  for (uint32_t p = s0 + (uint32_t)tid; p < s1; p += (uint32_t)BS) {
    const uint64_t e = stage[p];
    const uint32_t bn = bin(e);
    const uint32_t bs = bn != 0u ? S.bins[bn - 1u] : s0, be = S.bins[bn];
    if (be - bs > (uint32_t)kCrowd) {
      if (last) {
        if (p < want) sorted[p] = e;
      } else if (p == bs && bs < want) ranges(S)[atomicAdd(&S.bc[5], 1u)] = (bs << 16) | be;
    } else {
      const uint32_t r = rank_in_bin(stage, e, bs, be);
      if (r < want) sorted[r] = e;
    }
  }
}

// Sorts the ranges: one is split into kNB equal ranges of its composites (keys, and
// among tied keys indices) by its own extent, small ones ranked by comparison and
// crowded ones split again.  Each split takes eleven bits off a range, so this ends, also
// where calls that overlap on one workspace leave composites that do not differ.
// (A bitonic network, 66 steps of a barrier and two LDS round trips at 2048 entries:
// top-k of 50 at B=32 V=2^17 fp32 with 1310 maxima tied took 35.2 us, now 22.4.)
template <int BS>
__device__ __forceinline__ void sort_ranges(MSmem& S, uint64_t* stage, uint64_t* sorted, uint32_t want) {
  constexpr int NW = BS / 64, EL = (stage_cap(SS_MAX_K) + BS - 1) / BS, BPT = kNB / BS;
  // (values of its own: masks and addresses shared with the usual path would be kept
  // in registers, and others spilled, across the whole kernel: 14.3 instead of 14.0 us
  // for B=64 V=2^17 bf16 with a 64-entry list)
  int tid = threadIdx.x;
  asm("" : "+v"(tid));
  const int ln = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
#pragma unroll 1
  for (;;) {
    const uint32_t left = uniform(S.bc[5]);
    if (left == 0u) return;
    uint32_t s1 = ranges(S)[left - 1u], s0 = s1 >> 16;
    s1 &= 0xFFFFu;
    auto keep_in_vgpr = [](uint32_t& x) { asm("" : "+v"(x)); };
    keep_in_vgpr(s0);
    keep_in_vgpr(s1);
    const int n = (int)uniform(s1 - s0);
    uint64_t el[EL], hi = 0ull, lo = ~0ull;
#pragma unroll
    for (int j = 0; j < EL; ++j) {
      if (j * BS >= n) break;
      const uint32_t p = s0 + (uint32_t)(tid + j * BS);
      el[j] = p < s1 ? stage[p] : 0ull;
      if (p < s1) {
        hi = max(hi, el[j]);
        lo = min(lo, el[j]);
      }
    }
    for (int i = tid; i < kNB / 4; i += BS) reinterpret_cast<uint4*>(S.bins)[i] = make_uint4(0u, 0u, 0u, 0u);
    hi = wave_reduce(hi, [](uint64_t x, uint64_t y) { return x > y ? x : y; });
    lo = wave_reduce(lo, [](uint64_t x, uint64_t y) { return x < y ? x : y; });
    if (ln == 0) {
      S.x64[0][wv] = hi;
      S.x64[1][wv] = lo;
    }
    lds_barrier();
    if (tid == 0) S.bc[5] = left - 1u;
#pragma unroll 1
    for (int w = 0; w < NW; ++w) {
      hi = max(hi, S.x64[0][w]);
      lo = min(lo, S.x64[1][w]);
    }
    const int sh = max(0, 64 - __clzll((long long)((hi - lo) | 1ull)) - kNBLog);
    keep_in_vgpr(s1);
    auto bin = [&](uint64_t e) { return (uint32_t)((hi - e) >> sh); };
#pragma unroll
    for (int j = 0; j < EL; ++j) {
      if (j * BS < n && s0 + (uint32_t)(tid + j * BS) < s1) atomicAdd(&S.bins[bin(el[j])], 1u);
    }
    keep_in_vgpr(s1);
    lds_barrier();
    uint32_t h[BPT], sum = 0u, run, total;
#pragma unroll
    for (int q = 0; q < BPT; ++q) {
      h[q] = S.bins[tid * BPT + q];
      sum += h[q];
    }
    const uint32_t inc = wave_incl_scan(sum);
    if (ln == 63) S.x32[0][wv] = inc;
    lds_barrier();
    wave_prefix<NW>(S.x32[0], wv, run, total);
    run += s0 + inc - sum;
#pragma unroll
    for (int q = 0; q < BPT; ++q) {
      S.bins[tid * BPT + q] = run;
      run += h[q];
    }
    lds_barrier();
#pragma unroll
    for (int j = 0; j < EL; ++j) {
      if (j * BS < n && s0 + (uint32_t)(tid + j * BS) < s1) stage[atomicAdd(&S.bins[bin(el[j])], 1u)] = el[j];
    }
    lds_barrier();
    place_or_defer<BS>(S, stage, sorted, s0, s1, want, tid, sh == 0, bin);
    lds_barrier();
  }
}

// Maximum over the NW lanes of every half row (row): lane l holds wave l mod
// NW's value; uniform.
template <int NW>
__device__ __forceinline__ uint32_t waves_max(uint32_t x) {
  x = max(x, dpp_mov<0xB1>(x));
  x = max(x, dpp_mov<0x4E>(x));
  x = max(x, dpp_mov<0x141>(x));
  if constexpr (NW == 16) x = max(x, dpp_mov<0x140>(x));
  return __builtin_amdgcn_readfirstlane(x);
}

// Merge of one row by the whole workgroup.
template <int DT, int OP, int BS>
__device__ __forceinline__ void merge_row(const KArgs& early, int row, MSmem& S, uint64_t* stage) {
  const KArgs& a = early;
  constexpr int NW = BS / 64;
  constexpr int EPQ = DT == SS_BF16 ? 4 : 2;   // candidates per 16-byte load
  constexpr int NQM = DT == SS_BF16 ? 3 : 6;   // candidate loads a thread holds at most
  constexpr int EM = SS_MAX_K / BS;            // list entries per thread at most
  static_assert(OP == OP_TOPK || BS <= kH / 4, "every thread loads words of the patch table");
  const int tid = threadIdx.x;
  const int ln = lane(), wv = __builtin_amdgcn_readfirstlane(wave());
  const int U = a.U;
  int b = row, ell = 0;
  if constexpr (OP == OP_VERIFY) {
    b = row / (a.L + 1);
    ell = row - b * (a.L + 1);
  }

  // 1. every load of the row, none depending on another
  const int tpu = a.tpu;
  int u = (tid * a.tpu_inv) >> 20;
  const int sub = tid - u * tpu;
  const bool act = u < U;
  if (!act) u = 0;
  const size_t gu = (size_t)row * U + u;
  const uint4* region = a.cand + gu * (size_t)a.cap;
  const uint4 r4 = a.rec[gu];
  // the candidates as stored: bf16 words, fp32 composites
  std::conditional_t<DT == SS_BF16, uint32_t, uint64_t> cw[NQM * EPQ];
  // whose candidates this thread looks at: its share of its unit's
  const uint4* sreg = region;
  int stpu = tpu, ssub = sub;
  auto load_one = [&](int j, int at) {
    const uint4 q = sreg[min(at, a.cap - 1)];
    if constexpr (DT == SS_BF16) {
      cw[4 * j] = q.x;
      cw[4 * j + 1] = q.y;
      cw[4 * j + 2] = q.z;
      cw[4 * j + 3] = q.w;
    } else {
      cw[2 * j] = ((uint64_t)q.y << 32) | q.x;
      cw[2 * j + 1] = ((uint64_t)q.w << 32) | q.z;
    }
  };
  auto load_batch = [&](int batch) {
#pragma unroll
    for (int j = 0; j < NQM; ++j) load_one(j, (batch * NQM + j) * stpu + ssub);
  };
#pragma unroll
  for (int j = 0; j < NQM; ++j)
    if (j < a.nq) load_one(j, j * tpu + sub);
  const bool tables = OP != OP_TOPK && a.patch_wgs > 0;
  constexpr int KT = (kH / 4 + BS - 1) / BS;  // 16-byte words per thread and table half
  uint4 tid4[KT], tfin4[KT];
  int pst = 0;
  if (tables) {
    const uint4* tsrc = reinterpret_cast<const uint4*>(a.ptab + (size_t)row * 2 * kH);
#pragma unroll
    for (int m = 0; m < KT; ++m) {
      const int w = min(tid + m * BS, kH / 4 - 1);
      tid4[m] = tsrc[w];
      tfin4[m] = tsrc[kH / 4 + w];
    }
    pst = a.pstat[row];
  }
  // the units' normaliser sums and the listed ids' raw keys (log-probabilities, full-row truncation)
  constexpr bool NORM = OP == OP_LOGPROBS || OP == OP_SAMPLE_X;
  double us = 0.0;
  uint4 traw4[KT];
  if constexpr (NORM) {
    if (a.usum) us = a.usum[gu];
    if (tables) {
#pragma unroll
      for (int m = 0; m < KT; ++m)
        traw4[m] = reinterpret_cast<const uint4*>(a.gfin + (size_t)row * kGH)[min(tid + m * BS, kH / 4 - 1)];
    }
  }
  uint32_t mode = SS_TOPK;
  float temp = 1.0f, topp_v = 1.0f, minp_v = 0.0f;
  int kreq_v = 0, dtok = -1;
  uint64_t seed = 0ull;
  int64_t pos = ell;
  if constexpr (OP == OP_TOPK) {
    kreq_v = a.top_k[b];
    if (!(a.have & kHaveTopK)) kreq_v = a.k_cap;
  } else {
    mode = a.mode[b];
    temp = a.temperature[b];
    kreq_v = a.top_k[b];
    topp_v = a.top_p[b];
    minp_v = a.min_p[b];
    const uint64_t sd = a.seed[b];
    const int64_t ps = a.position[b];
    mode &= a.feat;
    seed = (a.have & kHaveSeed) ? sd : 0ull;
    pos += (a.have & kHavePos) ? ps : 0;
    if constexpr (OP == OP_VERIFY) {
      if (ell < a.L) dtok = a.draft_tokens[(size_t)b * a.L + ell];
    }
  }
  // the tables in LDS are cleared while the loads are in flight
  for (int i = tid; i < kNB / 4; i += BS) reinterpret_cast<uint4*>(S.bins)[i] = make_uint4(0u, 0u, 0u, 0u);
  const bool pexact = a.V <= kPB;
  if (tables) {
    const int pwords = pexact ? (a.V + 31) >> 5 : kPB / 32;
    for (int s = tid; s < (pwords + 3) >> 2; s += BS) reinterpret_cast<uint4*>(S.pbits)[s] = make_uint4(0u, 0u, 0u, 0u);
  }
  if (tid < kMaxU / 32) S.rmask[tid] = 0u;
  if (tid == 0) {
    S.bc[0] = 0u;     // entries of the bins that hold the list
    S.bc[1] = 0u;     // set when one of them is crowded
    S.bc[2] = kNone;  // top-p: last rank kept
    S.bc[3] = kNone;  // min-p: first rank dropped
    S.bc[5] = 0u;     // crowded ranges of the list
    S.bc[7] = kNone;  // top-p against the whole row: last rank kept
    S.bc[10] = 0u;    // normaliser: units to sum again
    S.bc64[3] = 0ull;
    S.best = 0ull;
  }
  lds_barrier();

  // the request, and what its epilogue needs (while the loads are in flight)
  bool greedy = false, kcap = false, full_row = false;
  int want;
  double tau = 1.0, itau = 1.0, lt = 0.0, u0 = 0.0;
  bool minp = false, topp = false;
  if constexpr (OP == OP_TOPK) {
    want = kreq_v < 0 ? 0 : min(kreq_v, a.k_cap);
  } else if constexpr (OP == OP_LOGPROBS) {
    want = (mode & SS_LOGPROBS) ? a.k_cap : 0;
  } else {
    const float tm = (mode & SS_TEMP) ? temp : 1.0f;
    greedy = (mode & SS_GREEDY) || ((mode & SS_TEMP) && tm <= 0.0f);
    const bool cutk = (mode & SS_TOPK) && kreq_v >= 1;
    const int kreq = cutk ? kreq_v : INT_MAX;
    kcap = !greedy && kreq > a.k_cap;
    full_row = a.full && !greedy && !cutk;
    want = greedy ? 1 : min(kreq, a.k_cap);
    if (!greedy) {
      tau = (double)tm;
      itau = 1.0 / tau;
      minp = (mode & SS_MINP) && minp_v > 0.0f;
      topp = (mode & SS_TOPP) && topp_v < 1.0f;
      if (minp) lt = log((double)minp_v);
      if (OP != OP_PROCESS) u0 = uniform01(seed, (uint32_t)b, pos, 0);
    }
  }

  // 2. largest threshold, row maximum, longest candidate list; the patch table
  uint32_t cnt = (act && r4.y != kOvf) ? r4.y : 0u;
  if (act && r4.y == kOvf) atomicOr(&S.rmask[u >> 5], 1u << (u & 31));
  uint32_t hfmax = 0u;
  if (pst == 1) {
#pragma unroll
    for (int m = 0; m < KT; ++m) {
      if (tid + m * BS >= kH / 4) {
        tid4[m] = make_uint4(kNone, kNone, kNone, kNone);
        continue;
      }
      reinterpret_cast<uint4*>(S.hk)[tid + m * BS] = tid4[m];
      reinterpret_cast<uint4*>(S.hf)[tid + m * BS] = tfin4[m];
      const int ids[4] = {(int)tid4[m].x, (int)tid4[m].y, (int)tid4[m].z, (int)tid4[m].w};
      const uint32_t fk[4] = {tfin4[m].x, tfin4[m].y, tfin4[m].z, tfin4[m].w};
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        if (ids[q] < 0) continue;
        const uint32_t hb = pbit(ids[q], pexact);
        atomicOr(&S.pbits[hb >> 5], 1u << (hb & 31));
        hfmax = max(hfmax, fk[q]);
      }
    }
  }
  // (the largest threshold composite: its key first, then the lowest cut of
  // that key; shared LDS words would serialise the units, one after another)
  {
    const uint32_t key = (act && r4.x != kNoEmit) ? r4.x : 0u;
    const uint32_t kw = wave_max_u32(key);
    const uint32_t cw = ~wave_max_u32(key == kw ? ~r4.w : 0u);
    const uint32_t hw = wave_max_u32(act ? r4.z : 0u);
    const uint32_t lw = wave_max_u32(act ? r4.y : 0u);  // kOvf when a unit overflowed
    hfmax = wave_max_u32(hfmax);
    if (ln == 0) {
      S.wred[wv] = make_uint4(kw, cw, hw, lw);
      S.x32[1][wv] = hfmax;
    }
  }
  lds_barrier();
  const uint4 wr = S.wred[ln & (NW - 1)];
  hfmax = waves_max<NW>(S.x32[1][ln & (NW - 1)]);
  const uint32_t hi = waves_max<NW>(wr.z), cmax = waves_max<NW>(wr.w);
  const uint32_t tkw = waves_max<NW>(wr.x);
  const uint64_t tc = tkw == 0u ? 0ull : comp_of(tkw, ~waves_max<NW>(wr.x == tkw ? ~wr.y : 0u));
  const uint32_t tck = comp_key(tc), tcut = comp_idx(tc);

  int flags = kcap ? SS_FLAG_KCAP : 0;
  const bool empty = hi < kKeyFloor;
  bool slow = cmax == kOvf || pst == 2;

  // 3. the elements that take part.  The code below is written for a fixed
  // number of candidate loads (with_nq), so that a row runs straight through it;
  // units with more candidates than those loads cover (`many`: k in the thousands,
  // heavy ties) are walked in batches of NQM loads instead.
  const bool go = !empty && want > 0 && !slow;
  const bool single = want == 1;
  const bool many = cmax > (uint32_t)(a.nq * tpu * EPQ);
  const int nbatch = many ? (int)((cmax + (uint32_t)(NQM * tpu * EPQ) - 1u) / (uint32_t)(NQM * tpu * EPQ)) : 1;
  constexpr int NE = NQM * EPQ;
  auto with_nq = [&](auto&& f) {
    if (a.nq == 1) f(std::integral_constant<int, 1>{});
    else if (a.nq == 2) f(std::integral_constant<int, 2>{});
    else if (NQM == 3 || a.nq == 3) f(std::integral_constant<int, 3>{});
    else if (a.nq == 4) f(std::integral_constant<int, 4>{});
    else f(std::integral_constant<int, NQM>{});
  };
  // composite of candidate x = EPQ j + e
  uint32_t ubase = ~(uint32_t)(u * kUE) - 0xFFFFu;
  auto elem = [&](int x) -> uint64_t {
    if constexpr (DT == SS_BF16) return ((uint64_t)(cw[x] & 0xFFFF0000u) << 32) | (ubase + (cw[x] & 0xFFFFu));
    else return cw[x];
  };
  // bf16: tc as a stored word of this thread's unit
  auto word_threshold = [&](int v) -> uint32_t {
    const uint32_t lo = (uint32_t)(v * kUE);
    const uint32_t in = tcut - lo < (uint32_t)kUE ? tck | (0xFFFFu - (tcut - lo)) : tck;
    return tcut < lo ? tck + 0x10000u : in;
  };
  uint32_t wthr = word_threshold(u);
  uint32_t scnt = cnt;
  // the candidates of a batch that are at or above tc and no raw copy of a
  // patched id (every LDS read is issued before any is used)
  auto select = [&](auto nq, int batch) -> uint32_t {
    constexpr int NQ = decltype(nq)::value, N = NQ * EPQ;
    uint32_t sel = 0u;
#pragma unroll
    for (int j = 0; j < NQ; ++j) {
      const int rem = (int)scnt - ((batch * NQ + j) * stpu + ssub) * EPQ;
#pragma unroll
      for (int e = 0; e < EPQ; ++e) {
        bool at;
        if constexpr (DT == SS_BF16) at = cw[j * EPQ + e] >= wthr;
        else at = elem(j * EPQ + e) >= tc;
        sel |= (at && e < rem) ? 1u << (j * EPQ + e) : 0u;
      }
    }
    if (pst == 1) {
      uint32_t pw[N];
#pragma unroll
      for (int x = 0; x < N; ++x) pw[x] = S.pbits[(pbit((int)comp_idx(elem(x)), pexact) >> 5) & (kPB / 32 - 1)];
      uint32_t hit = 0u;
#pragma unroll
      for (int x = 0; x < N; ++x)
        hit |= ((pw[x] >> (pbit((int)comp_idx(elem(x)), pexact) & 31u)) & 1u) << x;
      hit &= sel;
      if (__builtin_expect(pexact, 1)) {
        sel &= ~hit;
      } else {  // hashed bitmap: confirmed in the table
        while (hit != 0u) {
          const uint32_t low = hit & (0u - hit);
          int id = 0;
#pragma unroll
          for (int x = 0; x < N; ++x) id = low == (1u << x) ? (int)comp_idx(elem(x)) : id;
          if (hfind(S, id) >= 0) sel &= ~low;
          hit ^= low;
        }
      }
    }
    return sel;
  };
  // Bins in canonical order: 2^sh steps of an order value below the largest
  // possible key.  bf16 keys lie on a grid of 2^16, so the order value of a grid
  // element carries its index in the low half (a key that a hundred ids share
  // spreads over bins of a few); an off-grid final value goes behind every index
  // of the grid key above it.  Finals above the raw maximum (biases) share the first bin
  // where bins stretched to reach them would be four times as wide or more (sampling of
  // 1024 from uniform values with biases up to 5 at B=32 V=2^17: 27.4 us, now 19.5;
  // fp32 rows that span fewer than 2048 keys have their ties in one bin either way).
  auto shift = [&](uint32_t top) -> int {
    return max(0, 32 - __clz((top - tck) | (DT == SS_BF16 ? 0xFFFFu : 0u)) - kNBLog);
  };
  const int ish = max(0, 16 - __clz(max(a.V - 1, 1)));
  uint32_t kmax = hi;
  int sh = shift(hi);
  if (hfmax > hi) {
    const uint32_t kall = DT == SS_BF16 ? (hfmax + 0xFFFFu) & 0xFFFF0000u : hfmax;
    if (sh == 0 || shift(kall) < sh + 2) {
      kmax = kall;
      sh = shift(kall);
    }
  }
  auto bin_of = [&](uint64_t cm) -> uint32_t {
    const uint32_t key = comp_key(cm);
    if (key > kmax) return 0u;
    uint32_t o = kmax - key;
    if constexpr (DT == SS_BF16) o |= (key & 0xFFFFu) ? 0xFFFFu : comp_idx(cm) >> ish;
    return o >> sh;
  };
  auto grid_bin = [&](int x) -> uint32_t {  // of a candidate: a raw value, on the grid
    const uint64_t cm = elem(x);
    uint32_t o = kmax - comp_key(cm);
    if constexpr (DT == SS_BF16) o |= comp_idx(cm) >> ish;
    return (o >> sh) & (kNB - 1);
  };
  uint64_t* sorted = stage + a.pcap;
  const uint64_t* T = sorted;  // the row's list in canonical order
  int nT = 0;
  bool crowded = false;  // ranges of stage hold (a superset of) the list, unsorted
  uint32_t nB = 0u;      // entries of stage
  if (go) {
    uint32_t sel = 0u, bp[NE];
    // first pass: the maximum (single) or the bins' counts
    auto count = [&](auto nq, int batch) {
      constexpr int N = decltype(nq)::value * EPQ;
      sel = select(nq, batch);
      if (single) {
        uint64_t mc = 0ull;
#pragma unroll
        for (int x = 0; x < N; ++x) mc = ((sel >> x) & 1u) ? max(mc, elem(x)) : mc;
        if (mc != 0ull) atomicMax((unsigned long long*)&S.best, (unsigned long long)mc);
      } else {
#pragma unroll
        for (int x = 0; x < N; ++x) bp[x] = grid_bin(x);
#pragma unroll
        for (int x = 0; x < N; ++x)
          if ((sel >> x) & 1u) atomicAdd(&S.bins[bp[x]], 1u);
      }
    };
    // second pass: every element to its bin's next place (all asked for before any is used)
    auto place = [&](auto nq) {
      constexpr int N = decltype(nq)::value * EPQ;
#pragma unroll
      for (int x = 0; x < N; ++x)
        if ((sel >> x) & 1u) bp[x] = atomicAdd(&S.bins[bp[x]], 1u);
#pragma unroll
      for (int x = 0; x < N; ++x)
        if (((sel >> x) & 1u) && bp[x] < nB) stage[bp[x]] = elem(x);
    };
    constexpr auto all = std::integral_constant<int, NQM>{};
    // f(batch) for every batch of candidates when there are many: each thread
    // walks its share of its unit, or, when lists are far longer than that (rows
    // tied at their threshold: a few units hold everything), each wavefront whole
    // units.  Shares keep all threads busy (B=32 V=2^17 bf16, 1024 of uniform values:
    // 19.6 us, 43.3 by units); units bring all loads to the few useful ones (1024 of a
    // tied row: 28.6 us, 48.0 by shares); four batches a thread lie between the two.
    // A unit whose first possible element lies below tc has nothing to give (of a
    // tied row, every unit but the first ones: 74.4 us if they are read).
    auto walk = [&](auto&& f) {
      if (nbatch <= 4) {
        if (comp_of(r4.z, (uint32_t)(u * kUE)) < tc) scnt = 0u;
#pragma unroll 1
        for (int batch = 0; batch < nbatch; ++batch) {
          if (__ballot(scnt > (uint32_t)(batch * NQM * tpu * EPQ)) == 0ull) break;
          load_batch(batch);
          f(batch);
        }
        return;
      }
      stpu = 64;
      ssub = ln;
#pragma unroll 1
      for (int v = wv; v < U; v += NW) {
        const uint4 q4 = a.rec[(size_t)row * U + v];
        if (q4.x == kNoEmit || comp_of(q4.z, (uint32_t)(v * kUE)) < tc) continue;
        scnt = q4.y;
        sreg = a.cand + ((size_t)row * U + v) * (size_t)a.cap;
        ubase = ~(uint32_t)(v * kUE) - 0xFFFFu;
        wthr = word_threshold(v);
#pragma unroll 1
        for (int batch = 0; batch * NQM * 64 * EPQ < (int)scnt; ++batch) {
          load_batch(batch);
          f(batch);
        }
      }
    };
    if (__builtin_expect(!many, 1)) {
      with_nq([&](auto nq) { count(nq, 0); });
    } else {
      walk([&](int batch) { count(all, batch); });
    }
    // patched final values at or above tc
    uint32_t fsel = 0u;
    uint64_t fc[4 * KT];
    const bool finals = pst == 1 && hfmax >= tck;
    if (finals) {
#pragma unroll
      for (int m = 0; m < KT; ++m) {
        const uint32_t ids[4] = {tid4[m].x, tid4[m].y, tid4[m].z, tid4[m].w};
        const uint32_t fk[4] = {tfin4[m].x, tfin4[m].y, tfin4[m].z, tfin4[m].w};
#pragma unroll
        for (int q = 0; q < 4; ++q) {  // (empty slots have key 0, below every tc)
          fc[4 * m + q] = comp_of(fk[q], ids[q]);
          if (fc[4 * m + q] >= tc) {
            fsel |= 1u << (4 * m + q);
            if (single) atomicMax((unsigned long long*)&S.best, (unsigned long long)fc[4 * m + q]);
            else atomicAdd(&S.bins[bin_of(fc[4 * m + q])], 1u);
          }
        }
      }
    }
    lds_barrier();
    if (single) {
      const uint64_t mc = uniform(S.best);
      slow = mc == 0ull;
      nT = slow ? 0 : 1;
      if (tid == 0) sorted[0] = mc;
      lds_barrier();
    } else {
      // counts to starts; the bins that hold the list end at nB
      constexpr int BPT = kNB / BS;  // bins per thread
      uint32_t h[BPT], s = 0u;
#pragma unroll
      for (int q = 0; q < BPT; ++q) {
        h[q] = S.bins[tid * BPT + q];
        s += h[q];
      }
      const uint32_t inc = wave_incl_scan(s);
      if (ln == 63) S.x32[3][wv] = inc;
      lds_barrier();
      uint32_t run, total;
      wave_prefix<NW>(S.x32[3], wv, run, total);
      run += inc - s;
      total = uniform(total);
      if (total < (uint32_t)want) {
        // at the lowest threshold there is the list is the whole row (few
        // tokens allowed by a grammar); otherwise elements may be missing
        if (tc <= comp_of(kKeyFloor, kNone)) want = (int)total;
        else slow = true;
      }
#pragma unroll
      for (int q = 0; q < BPT; ++q) {
        S.bins[tid * BPT + q] = run;
        if (run < (uint32_t)want) {
          if (h[q] > (uint32_t)kCrowd) S.bc[1] = 1u;
          if (run + h[q] >= (uint32_t)want) S.bc[0] = run + h[q];
        }
        run += h[q];
      }
      lds_barrier();
      nB = uniform(S.bc[0]);
      if (nB > (uint32_t)a.pcap) slow = true;  // ties beyond the staging area
      if (!slow) {
        if (__builtin_expect(!many, 1)) {
          with_nq([&](auto nq) { place(nq); });
        } else {
          walk([&](int batch) {
            sel = select(all, batch);
#pragma unroll
            for (int x = 0; x < NE; ++x) bp[x] = grid_bin(x);
            place(all);
          });
        }
        if (fsel != 0u) {
#pragma unroll
          for (int x = 0; x < 4 * KT; ++x) {
            if ((fsel >> x) & 1u) {
              const uint32_t p = atomicAdd(&S.bins[bin_of(fc[x])], 1u);
              if (p < nB) stage[p] = fc[x];
            }
          }
        }
        lds_barrier();
        crowded = uniform(S.bc[1]) != 0u;
        nT = want;
        if (__builtin_expect(!crowded, 1)) {
          for (uint32_t p = (uint32_t)tid; p < nB; p += (uint32_t)BS) {
            const uint64_t e = stage[p];
            const uint32_t bn = bin_of(e);
            const uint32_t bs = bn != 0u ? S.bins[bn - 1u] : 0u, be = S.bins[bn];
            const uint32_t r = rank_in_bin(stage, e, bs, be);
            if (r < (uint32_t)want) sorted[r] = e;
          }
        } else {
          place_or_defer<BS>(S, stage, sorted, 0u, nB, (uint32_t)want, tid, false, bin_of);
        }
        lds_barrier();
      }
    }
  }

  // 4. the exact slow path, and lists beyond the patch table
  int pmode = pst == 1 ? 1 : 0;
  PatchG pg = {};
  Ctx c = {};
  if (__builtin_expect(!empty && want > 0 && slow, 0)) {
    const KArgs& a = late_args();
    flags |= SS_FLAG_FALLBACK;
    c = make_ctx<DT>(a, row);
    if (pst == 2) pmode = global_table<DT, BS>(a, c, S, row, pg);
    if (want == 1 && pmode <= 1 && cmax != kOvf)
      nB = (uint32_t)greedy_refill<DT, BS>(a, c, S, stage, pmode == 1);
    else
      nB = (uint32_t)slow_select<DT, BS>(a, c, S, stage, pmode, pg, (uint32_t)want);
    nT = min(want, (int)nB);
    crowded = nB > 1u;
    if (!crowded) T = stage;
    if (tid == 0) {
      ranges(S)[0] = nB;
      S.bc[5] = 1u;
    }
    lds_barrier();
  }
  if (__builtin_expect(crowded, 0)) sort_ranges<BS>(S, stage, sorted, (uint32_t)nT);
  const bool none = empty || nT == 0;
  if (none) flags = empty ? SS_FLAG_EMPTY : flags | SS_FLAG_EMPTY;
  const uint64_t Mcomp = none ? 0ull : uniform(T[0]);
  const int argmax = none ? -1 : (int)comp_idx(Mcomp);

  // The row's normaliser relative to M: the units' sums (taken relative to each
  // unit's raw maximum) rescaled, each patched id's raw term replaced by its
  // final value's.  The units' factors go through the bins' memory.
  // A unit whose raw maximum lies above M by more than ln kLead owes it to patched
  // ids: their terms would be taken from a sum that holds little else (a lead of 36
  // leaves nothing of the rest, one of 710 overflows), so it is summed again from
  // the logits, relative to M and without them.  Below that, what the subtraction
  // leaves is off by at most kLead 2^-46 of Z, and the terms' exponents by ln kLead
  // float32 roundings more than those of other units.  One such unit in every row costs
  // 1 us: log-probabilities at B=32 V=2^17 17.6 -> 18.3 us, full-row sampling 22.6 -> 23.6.
  auto row_norm = [&](double M, float tauf) -> double {
    const double tau2 = (double)tauf;
    double z = 0.0;
    if (__builtin_expect(pmode <= 1, 1)) {
      constexpr double kLead = 16.0;
      const float c2 = lp_scale(tauf);
      double* uf = reinterpret_cast<double*>(S.bins);
      float* um = reinterpret_cast<float*>(S.bins + 2 * kMaxU);
      uint32_t* again = S.bins + 3 * kMaxU;  // units to sum again
      static_assert(4 * kMaxU <= kNB, "unit factors, maxima and the list of units over the bins");
      if (act && sub == 0) {
        const float mu = float_of_key(r4.z);
        const bool some = r4.z >= kKeyFloor;
        double f = some ? exp(((double)mu - M) / tau2) : 0.0;
        if (pmode == 1 && f > kLead) {
          again[atomicAdd(&S.bc[10], 1u)] = (uint32_t)u;
          f = 0.0;
        } else if (some) {
          z = f * us;
        }
        uf[u] = f;
        um[u] = mu;
      }
      lds_barrier();
      if (pmode == 1) {
#pragma unroll
        for (int m = 0; m < KT; ++m) {
          const int ids[4] = {(int)tid4[m].x, (int)tid4[m].y, (int)tid4[m].z, (int)tid4[m].w};
          const uint32_t fk[4] = {tfin4[m].x, tfin4[m].y, tfin4[m].z, tfin4[m].w};
          const uint32_t rk[4] = {traw4[m].x, traw4[m].y, traw4[m].z, traw4[m].w};
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            if (ids[q] < 0) continue;
            if (rk[q] >= kKeyFloor)
              z -= uf[ids[q] / kUE] * (double)lp_term(float_of_key(rk[q]), um[ids[q] / kUE], c2);
            if (fk[q] >= kKeyFloor) z += exp(((double)float_of_key(fk[q]) - M) / tau2);
          }
        }
        const int n = (int)uniform(S.bc[10]);
        if (__builtin_expect(n > 0, 0)) z += units_norm<DT, BS>(late_args(), S, row, mode, again, n, (float)M, c2);
      }
    } else {
      z = row_norm_all<DT, BS>(a, c, S, pmode, pg, M, tau2);
    }
    return wg_sum<BS>(z, S.rd);
  };

  // 5. outputs
  {
  const KArgs& a = late_args();
  if constexpr (OP == OP_TOPK) {
    for (int r = tid; r < a.k_cap; r += BS) {
      const size_t o = (size_t)b * a.k_cap + r;
      const uint64_t cm = r < nT ? T[r] : 0ull;
      a.out_val[o] = r < nT ? float_of_key(comp_key(cm)) : -__builtin_inff();
      a.out_idx[o] = r < nT ? (int32_t)comp_idx(cm) : -1;
    }
    if (a.flags && tid == 0) a.flags[b] = flags & SS_FLAG_FALLBACK;
    return;
  } else if constexpr (OP == OP_LOGPROBS) {
    const float tauf = lp_tau(a, mode, b);
    const double tau = (double)tauf;
    const double M = none ? 0.0 : (double)float_of_key(comp_key(Mcomp));
    const double lz = none ? 0.0 : log(row_norm(M, tauf));
    for (int r = tid; r < a.k_cap; r += BS) {
      const size_t o = (size_t)b * a.k_cap + r;
      const uint64_t cm = r < nT ? T[r] : 0ull;
      a.out_idx[o] = r < nT ? (int32_t)comp_idx(cm) : -1;
      a.out_val[o] = r < nT ? (float)(((double)float_of_key(comp_key(cm)) - M) / tau - lz) : -__builtin_inff();
    }
    if (a.flags && tid == 0) a.flags[b] = (mode & SS_LOGPROBS) ? flags & (SS_FLAG_FALLBACK | SS_FLAG_EMPTY) : 0;
    return;
  } else {
    if constexpr (OP == OP_PROCESS) {  // patched ids for the materialising pass
      if (empty || pmode <= 1) {
        if (tid == 0) a.npatched[row] = (pst == 1 && !empty) ? kTable : 0u;
      } else if (pmode == 3) {
        if (tid == 0) a.npatched[row] = kLinear;
      } else {
        if (tid == 0) S.bc[8] = 0u;
        lds_barrier();
        for (int s = tid; s < kGH; s += BS) {
          const uint64_t t = pg.tag[s];
          if ((uint32_t)(t >> 32) == pg.gen)
            a.patched[(size_t)row * kGH + atomicAdd(&S.bc[8], 1u)] = make_uint2((uint32_t)t - 1u, pg.fin[s]);
        }
        lds_barrier();
        if (tid == 0) a.npatched[row] = S.bc[8];
      }
    }
    const bool has_draft = OP == OP_VERIFY && ell < a.L && dtok >= 0 && dtok < a.V;
    if (none || greedy) {
      if constexpr (OP == OP_PROCESS) {
        if (tid == 0) {
          RowSummary s;
          s.thr = Mcomp;
          s.Z = 1.0;
          s.M = none ? 0.0f : float_of_key(comp_key(Mcomp));
          s.tau = 1.0f;
          s.argmax = argmax;
          s.kind = none ? KIND_EMPTY : KIND_GREEDY;
          a.summ[row] = s;
          if (a.flags) a.flags[b] = flags;
        }
      } else if constexpr (sampling_op(OP)) {
        if (tid == 0) {
          a.out_token[b] = argmax;
          if (a.out_logprob) a.out_logprob[b] = 0.0f;
          if (a.flags) a.flags[b] = flags;
        }
        if (a.out_idx) {
          for (int r = tid; r < a.k_out; r += BS) {
            a.out_idx[(size_t)b * a.k_out + r] = r == 0 ? argmax : -1;
            a.out_prob[(size_t)b * a.k_out + r] = (r == 0 && !none) ? 1.0f : 0.0f;
          }
        }
      } else {
        if (tid == 0) {
          S.bc[9] = (has_draft && !none && dtok == argmax) ? 1u : 0u;
          S.bc[10] = (uint32_t)argmax;
          S.bc[11] = (uint32_t)flags;
        }
      }
      return;
    }

    // ---- truncation and selection (Alg. 11 order) on T[0, nT): entry r =
    // 64 (E wave + j) + lane is held by one thread, E entries per thread
    const double M = (double)float_of_key(comp_key(Mcomp));
    auto epilogue = [&](auto ec) {
    constexpr int E = decltype(ec)::value;
    const int r0 = 64 * E * wv + ln;
    auto yval = [&](uint64_t cm) { return (double)float_of_key(comp_key(cm)); };
    auto weight = [&](uint64_t cm) { return weight_fast(yval(cm), M, itau); };
    auto dropped = [&](uint64_t cm) {  // by min-p; never the first
      const double y = yval(cm);
      double l = y == M ? 0.0 : (y - M) * itau;
      if (fabs(l - lt) < 1e-9 * fabs(lt)) l = (y - M) / tau;  // the product may round to the other side
      return cm != Mcomp && !(l >= lt);
    };
    // exclusive prefix sums of wt over the list; returns the total
    uint64_t el[E], wt[E], ex[E];
    auto scan_list = [&](uint64_t* scratch) -> uint64_t {
      uint64_t run = 0ull;
#pragma unroll
      for (int j = 0; j < E; ++j) {
        {
          const uint64_t inc = wave_incl_scan(wt[j]);
          ex[j] = run + inc - wt[j];
          run += readlane_T(inc, 63);
        }
      }
      if (ln == 0) scratch[wv] = run;
      lds_barrier();
      uint64_t before, total;
      wave_prefix<NW>(scratch, wv, before, total);
#pragma unroll
      for (int j = 0; j < E; ++j)
        ex[j] += before;
      return total;
    };
#pragma unroll
    for (int j = 0; j < E; ++j) {
      {
        const int r = r0 + 64 * j;
        el[j] = r < nT ? T[r] : 0ull;
        wt[j] = r < nT ? (uint64_t)__double2ll_rn(weight(el[j]) * kFix) : 0ull;
      }
    }
    const uint64_t Zk = uniform(scan_list(S.x64[1]));
    // Full-row truncation takes its boundary against the whole row's mass;
    // its result stands when fewer than k_max tokens are kept, else the bounded
    // one (mass of the list) is taken with KCAP.
    double zrow = 0.0;
    if (OP == OP_SAMPLE_X && full_row) zrow = kFix * row_norm(M, (float)tau);
    const double Xp = (double)topp_v * (double)Zk, Xr = (double)topp_v * zrow;
#pragma unroll
    for (int j = 0; j < E; ++j) {
      {
        const int r = r0 + 64 * j;
        if (r < nT) {
          const double in = (double)(ex[j] + wt[j]), be = (double)ex[j];
          // the first entry whose inclusive mass reaches the boundary is kept, the next are not
          if (topp && in >= Xp && (r == 0 || be < Xp)) {
            S.bc[2] = (uint32_t)r;
            S.bc64[0] = ex[j] + wt[j];
          }
          if (OP == OP_SAMPLE_X && full_row && topp && in >= Xr && (r == 0 || be < Xr)) {
            S.bc[7] = (uint32_t)r;
            S.bc64[2] = ex[j] + wt[j];
          }
        }
        if (minp) {  // the kept ones are a prefix: the first dropped one follows a kept one
          const bool dr = r < nT && dropped(el[j]);
          const uint64_t dm = __ballot(dr);
          if (dm != 0ull && ln == (int)__builtin_ctzll(dm) && (ln > 0 || !dropped(T[r - 1]))) {
            S.bc[3] = (uint32_t)r;
            S.bc64[1] = ex[j];
          }
        }
      }
    }
    lds_barrier();
    const uint32_t np = uniform(S.bc[2]), nm = uniform(S.bc[3]);
    const uint64_t zp = uniform(S.bc64[0]), zm = uniform(S.bc64[1]);
    uint32_t n_s = (uint32_t)nT;
    uint64_t Zs = Zk;
    auto cut_at = [&](uint32_t last, uint64_t z) {  // the shorter of the top-p and min-p prefixes
      n_s = (uint32_t)nT;
      Zs = Zk;
      if (last != kNone) {
        n_s = last + 1u;
        Zs = z;
      }
      if (nm < n_s) {
        n_s = nm;
        Zs = zm;
      }
    };
    cut_at(np, zp);
    if (OP == OP_SAMPLE_X && full_row) {
      cut_at(uniform(S.bc[7]), uniform(S.bc64[2]));
      if (n_s < (uint32_t)a.k_cap) {
        flags &= ~SS_FLAG_KCAP;
      } else {
        flags |= SS_FLAG_KCAP;
        cut_at(np, zp);
      }
    }
    const double Zsd = (double)Zs / kFix;
    // calls f(composite) in the thread that holds the drawn entry: the first
    // kept one whose inclusive mass exceeds u0 * total (else the last one)
    auto draw = [&](double total, auto&& f) {
      const double X = u0 * total;
#pragma unroll
      for (int j = 0; j < E; ++j) {
        {
          const int r = r0 + 64 * j;
          if (r < (int)n_s && ((double)(ex[j] + wt[j]) > X || r == (int)n_s - 1) && (r == 0 || (double)ex[j] <= X))
            f(el[j]);
        }
      }
    };
    if constexpr (OP == OP_PROCESS) {
      if (tid == 0) {
        RowSummary s;
        s.thr = T[n_s - 1u];
        s.Z = Zsd;
        s.M = (float)M;
        s.tau = (float)tau;
        s.argmax = argmax;
        s.kind = KIND_DIST;
        a.summ[row] = s;
        if (a.flags) a.flags[b] = flags;
      }
    } else if constexpr (sampling_op(OP)) {
      if (a.out_idx && (int)n_s > a.k_out) flags |= SS_FLAG_OUT_TRUNC;
      auto emit = [&](uint64_t cm) {
        a.out_token[b] = (int32_t)comp_idx(cm);
        if (a.out_logprob) a.out_logprob[b] = (float)log(weight(cm) / Zsd);
        if (a.flags) a.flags[b] = flags;
      };
      if (OP == OP_SAMPLE_X && a.gum) {
        // Gumbel-max over the kept set (Appendix C.3): the largest
        // (y - M)/tau - g[id] in double, the lower id on equal scores
        const float* grow = a.gum + (size_t)b * (size_t)a.ld_g;
        double bs = -__builtin_inf();
        uint64_t bk = 0ull;  // (~id << 32) | key of this thread's best
#pragma unroll
        for (int j = 0; j < E; ++j) {
          {
            const int r = r0 + 64 * j;
            if (r < (int)n_s) {
              const uint64_t cm = el[j];
              const double y = yval(cm);
              const double sc = (y == M ? 0.0 : (y - M) / tau) - (double)grow[comp_idx(cm)];
              const uint64_t k2 = ((uint64_t)(~comp_idx(cm)) << 32) | comp_key(cm);
              if (sc > bs || (sc == bs && k2 > bk)) {
                bs = sc;
                bk = k2;
              }
            }
          }
        }
        const double top = wg_max<BS>(bs, S.rd);
        const uint64_t win = wg_max<BS>(bs == top ? bk : (uint64_t)0, S.x64[2]);
        if (tid == 0) emit(comp_of((uint32_t)win, ~(uint32_t)(win >> 32)));
      } else {
        draw((double)Zs, emit);
      }
      if (a.out_idx) {
        for (int r = tid; r < a.k_out; r += BS) {
          const bool in = r < (int)n_s;
          const uint64_t cm = in ? T[r] : 0ull;
          a.out_idx[(size_t)b * a.k_out + r] = in ? (int32_t)comp_idx(cm) : -1;
          a.out_prob[(size_t)b * a.k_out + r] = in ? (float)(weight(cm) / Zsd) : 0.0f;
        }
      }
    } else {
      // verification: this row's decision; assemble_request combines a request's rows
      auto publish = [&](int accept, int token) {
        S.bc[9] = (uint32_t)accept;
        S.bc[10] = (uint32_t)token;
        S.bc[11] = (uint32_t)flags;
      };
      if (!has_draft) {
        draw((double)Zs, [&](uint64_t cm) { publish(0, (int)comp_idx(cm)); });
        return;
      }
      // P(d): zero (bc64[3]) unless the draft token is kept
#pragma unroll
      for (int j = 0; j < E; ++j) {
        {
          const int r = r0 + 64 * j;
          if (r < (int)n_s && (int)comp_idx(el[j]) == dtok) S.bc64[3] = __builtin_bit_cast(uint64_t, weight(el[j]) / Zsd);
        }
      }
      const float* qrow = a.draft_probs ? a.draft_probs + ((size_t)b * a.L + ell) * (size_t)a.ld_q : nullptr;
      // sparse q: the entries naming an id summed, an unlisted id at 0
      const bool sparse = a.kq > 0;
      const size_t qo = ((size_t)b * a.L + ell) * (size_t)a.kq;
      uint64_t* ql = qlist_view(S);
      int NQ = 0;
      double qd;
      if (sparse) {
        // the list into LDS as (id << 32 | q bits), ids outside [0, V)
        // as 0xFFFFFFFF, padded to a power of two when it will be sorted
        NQ = a.kq <= kQScan ? a.kq : next_pow2(a.kq);
        double qs = 0.0;
        for (int i = tid; i < NQ; i += BS) {
          uint64_t e = ~0ull;
          if (i < a.kq) {
            const int id = a.dq_idx[qo + i];
            const float v = a.dq_val[qo + i];
            if (id == dtok) qs += (double)v;
            if (id >= 0 && id < a.V) e = ((uint64_t)(uint32_t)id << 32) | __float_as_uint(v);
          }
          ql[i] = e;
        }
        qd = wg_sum<BS>(qs, S.rd);  // its barriers publish the list and P(d)
      } else {
        qd = (double)qrow[dtok];
        lds_barrier();
      }
      const double Pd = __builtin_bit_cast(double, S.bc64[3]);
      const double u1 = uniform01(seed, (uint32_t)b, pos, 1);
      if (Pd > 0.0 && u1 * qd <= Pd) {
        if (tid == 0) publish(1, -1);
        return;
      }
      // a long list is sorted (ids descending, padding first) for binary
      // search; a short one is scanned in list order, every lane reading
      // the same entry
      const bool qsorted = sparse && a.kq > kQScan;
      if (qsorted) lds_sort_desc<BS>(ql, NQ);
      auto q_of = [&](uint32_t id) -> double {
        if (!sparse) return (double)qrow[id];
        double s = 0.0;
        if (!qsorted) {
#pragma unroll 8
          for (int j = 0; j < NQ; ++j) {
            const uint64_t e = ql[j];
            if ((uint32_t)(e >> 32) == id) s += (double)__uint_as_float((uint32_t)e);
          }
          return s;
        }
        int lo = 0, hi2 = NQ;  // first entry whose id is at most `id`
        while (lo < hi2) {
          const int mid = (lo + hi2) >> 1;
          if ((uint32_t)(ql[mid] >> 32) > id) lo = mid + 1;
          else hi2 = mid;
        }
        for (; lo < NQ && (uint32_t)(ql[lo] >> 32) == id; ++lo) s += (double)__uint_as_float((uint32_t)ql[lo]);
        return s;
      };
      // residual max(0, P - q) over the kept set, canonical order; the kept
      // weights again when it is empty
      uint64_t rs[E];
#pragma unroll 1
      for (int j = 0; j < E; ++j) {
        const int r = r0 + 64 * j;
        uint64_t v64 = 0ull;
        if (r < (int)n_s) {
          const uint64_t cm = T[r];
          const double v = weight(cm) / Zsd - q_of(comp_idx(cm));
          v64 = v > 0.0 ? (uint64_t)__double2ll_rn(v * kFix) : 0ull;
        }
#pragma unroll
        for (int jj = 0; jj < E; ++jj)
          if (jj == j) rs[jj] = v64;
      }
      uint64_t any = 0ull;
#pragma unroll
      for (int j = 0; j < E; ++j)
        any |= rs[j];
      any = wg_max<BS>(any, S.x64[2]);
      double total = (double)Zs;
      if (any != 0ull) {
#pragma unroll
        for (int j = 0; j < E; ++j)
          wt[j] = rs[j];
        total = (double)scan_list(S.x64[0]);
      }
      draw(total, [&](uint64_t cm) { publish(0, (int)comp_idx(cm)); });
    }
    };
    // straight-line code for the usual list lengths
    if (nT <= BS) epilogue(std::integral_constant<int, 1>{});
    else if (nT <= 2 * BS) epilogue(std::integral_constant<int, 2>{});
    else epilogue(std::integral_constant<int, EM>{});
  }
  }
}

// Verification: publishes the row's decision (bc[9..11]: accept, token, flags)
// and, in the workgroup that is the last of its request, writes the request's
// outputs: the accepted drafts, then the first row's correction (or the bonus
// token), then -1.  The streaming launch cleared the request's arrival count
// (the first row's `arrived`).  A decision is one 64-bit word, written and read by
// agent-scope atomics, which go past the XCD's L2 by themselves: the arrival
// follows once the word's store has completed, so no fence has to write back and
// invalidate the L2 (that took 1.5 us).  A launch of its own for this cost 4.1 us.
__device__ __forceinline__ void assemble_request(const KArgs& a, int row, const MSmem& S) {
  if (wave() != 0) return;
  const int ln = lane(), L = a.L;
  const int b = row / (L + 1);
  RowResult* res = a.res + (size_t)b * (L + 1);
  int last = 0;
  if (ln == 0) {
    const uint64_t word = ((uint64_t)S.bc[10] << 32) | (S.bc[11] << 1) | S.bc[9];
    __hip_atomic_store(&a.res[row].word, word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the store has completed
    last = __hip_atomic_fetch_add(&res->arrived, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == (uint32_t)L;
  }
  if (__builtin_amdgcn_readfirstlane(last) == 0) return;
  asm volatile("" ::: "memory");  // the words are read after the last arrival
  static_assert(SS_MAX_L < 64, "one lane per position");
  int accept = 0, emit = -1, fl = 0, draft = -1;
  if (ln <= L) {
    const uint64_t word = __hip_atomic_load(&res[ln].word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    accept = (int)(word & 1u);
    fl = (int)((uint32_t)word >> 1);
    emit = (int)(uint32_t)(word >> 32);
    if (ln < L) draft = a.draft_tokens[(size_t)b * L + ln];
  }
  // the first position that does not accept (the bonus position never does)
  const int stop = (int)__builtin_ctzll(__ballot(ln == L || (ln < L && accept == 0)));
  int all = 0;
#pragma unroll
  for (int f = 0; f < 4; ++f) all |= __ballot(ln <= stop && ((fl >> f) & 1)) != 0ull ? 1 << f : 0;
  static_assert((SS_FLAG_EMPTY | SS_FLAG_FALLBACK | SS_FLAG_OUT_TRUNC | SS_FLAG_KCAP) == 15, "four flag bits");
  if (ln <= L) a.out_tokens[(size_t)b * (L + 1) + ln] = ln < stop ? draft : (ln == stop ? emit : -1);
  if (ln == 0) {
    a.out_nacc[b] = stop;
    if (a.flags) a.flags[b] = all;
  }
}

// Merge kernel: one workgroup per row (the launch boundary orders the
// streaming kernel's records and candidates before it).
// (At most 128 registers, so that two workgroups share a CU when there are more
// rows than CUs; the extended sampling merge needs a few more.)
template <int DT, int OP, int BS>
__global__ __launch_bounds__(BS, OP == OP_SAMPLE_X ? 3 : 4) void ss_merge_kernel(KArgs a) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  MSmem& S = *reinterpret_cast<MSmem*>(smem_raw);
  uint64_t* stage = reinterpret_cast<uint64_t*>(smem_raw + kSmemFixed);
  // The streaming kernel placed row r's units on XCD floor(8 r / rows) when
  // its grid splits evenly over the 8 XCDs; the same remap here runs the
  // row's merge on that XCD as well.
  int row = blockIdx.x + warm_args();
  const int nunits = a.rows * a.U;
  if ((a.rows & 7) == 0 && (nunits & 31) == 0) row = (row & 7) * (a.rows >> 3) + (row >> 3);
  merge_row<DT, OP, BS>(a, row, S, stage);
  if constexpr (OP == OP_VERIFY) {
    lds_barrier();
    assemble_request(late_args(), row, S);
  }
}

}  // namespace ss
