// Rows whose survivors are not a short prefix that the single-pass kernel's candidate list can hold:
// a nucleus over the whole vocabulary that is wider than the list (top-p over all of V, section 2.1
// Eq. (2)), no truncation at all (every column survives), a min-p cut below the list's reach, or
// top-k alone with k above what the list certifies.
//
// The single-pass kernel queues such rows with their threshold g.  Their remaining work is two more
// reads of the row, which one workgroup per row would do at the latency of a single compute unit;
// here every queued row is cut into slices of 4096 columns that spread over the whole chip:
//
//   bins      per slice, the penalised, tempered logits below g are binned (bins linear in the
//             tempered logit, 1/64 of a factor two in probability wide) with their masses relative
//             to the mass at g (integers, LDS atomics); the mass at or above g goes to one more
//             slot.  The bins are exact sums, so they also give the mass of the whole row, and they
//             point at the bin that holds the cut.
//   classify  that bin follows from the cumulated masses.  Tempered value, bin and the comparison
//             with g are monotone in the logit, so the class of a column (surely inside, in the
//             cut's bin, outside) is decided by two thresholds on the logit itself, found once per
//             row by a search over floats.  Per tile, the exact (integer) masses of the columns
//             surely inside are summed by class (tail / hot) and the columns of the cut's bin are
//             collected.
//   finish    one workgroup per row checks that the cut does lie in the collected bin (else the
//             general kernel takes the row), finds it exactly among those columns by buckets of equal
//             width over (value, id), weighted by mass, spread again inside the bucket that holds it
//             while many share that (total order: value descending, id ascending), applies the SHVS acceptance test (section 5.3), walks
//             the per-tile masses of the drawn class in ascending id and reads one tile a last time
//             to locate the drawn id (inverse CDF, step (3) of section 2.1).
//
// The first two kernels are software pipelines over a workgroup's slices: the loads of the next
// slice (logits, hot-set bits, history mask) are requested before the current one is processed, and
// a slice's own dependent loads (history counts, logits of its history columns) are requested
// before its main line runs, so that no trip through memory is waited for in full.  Loads return in
// order: what is needed first is requested first.
//
// Rows without truncation have no cut and are read once, by the first kernel: per slice and wave it leaves
// the columns' mass, from which the third kernel draws.  Where a column stands too far above g for the fixed
// point, the second kernel weighs the row again, in double precision and each slice relative to its largest
// column (one column may hold almost the whole mass; only a slice more than FAR_LIMIT above all others sends the
// row to the general kernel).  Rows with a min-p cut use the first
// kernel for the row maximum only (the cut is a value).  Rows with top-k alone run the same three
// kernels by count instead of mass: a bin counts its columns, the cut's bin is the one in which
// the count from the top reaches k, and the buckets inside it weigh every column as one.
//
// Penalties (section 2.2) are applied on the fly: the single-pass kernel leaves the row's history
// tables (presence mask, rank directory, counts by rank) in the row's workspace slot, and a slice
// loads its part of them into LDS.  All masses are integers (far untruncated rows: per slice, scaled and added
// in a fixed order), so no result depends on the order of the additions.  A row for which a table overflows
// or the passes disagree is handed to the general kernel.
#include <type_traits>

#include "simple_rowdev.hpp"

namespace simple {
namespace fast {


constexpr int WT = 256;      // threads per workgroup
constexpr int WNW = WT / 64;
constexpr uint32_t LDS_PER_CU = 163840u;
constexpr int WGS = 4;       // workgroups of the bins and the classifying kernel on a compute unit, by registers and LDS ...
template <typename DT, bool RUNS> constexpr int bins_wgs() { return sizeof(DT) == 2 && !RUNS ? 5 : WGS; }  // ... more where they fit
constexpr int SLC = 4096;    // columns per slice
constexpr int ICAP = 512;    // places for boundary columns that a slice finds free in the stage (more go to the row's list one by one)
constexpr int MAX_SLICES = FAST_MAX_V / SLC;
static_assert(WS_HT == WIDE_SLOT_FIXED, "workspace slot size");
static_assert(sizeof(WideRec) == 64, "queue record size");

// Per-row constants of a queued row, identical in every thread.
struct WideRow {
  int row;
  StreamCtx C;
  float tau, top_p, min_p, ln_min_p;
  uint32_t mode, flags;
  bool h_active;
  float rep, freq, pres;
  double inv_rep;
  uint32_t distinct;
  int top_k;
  bool f64, far;
  MassRef M;  // (f64)
  unsigned char* ws;
};

// The record is the same in every lane; saying so keeps the row's constants in scalar registers.
__device__ __forceinline__ uint32_t uni(uint32_t v) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)v); }
__device__ __forceinline__ int uni(int v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ float uni(float v) { return __uint_as_float(uni(__float_as_uint(v))); }
__device__ __forceinline__ double uni(double v) {
  const unsigned long long b = (unsigned long long)__double_as_longlong(v);
  return __longlong_as_double((long long)(((unsigned long long)uni((uint32_t)(b >> 32)) << 32) | (unsigned long long)uni((uint32_t)b)));
}

__device__ __forceinline__ WideRow load_row(const SampleArgs& a, unsigned slot) {
  WideRow W;
  slot = uni(slot);
  const WideRec rec = reinterpret_cast<const WideRec*>(a.wq + WQ_HEAD)[slot];
  W.row = uni((int)rec.row); W.mode = uni(rec.mode & WIDE_MODE); W.far = (uni(rec.mode) & WIDE_FAR) != 0u; W.f64 = (uni(rec.mode) & WIDE_F64) != 0u; W.flags = uni(rec.flags);
  W.tau = uni(rec.tau); W.top_p = uni(rec.top_p); W.min_p = uni(rec.min_p); W.ln_min_p = uni(rec.ln_min_p);
  W.C.g = uni(rec.g); W.C.y_g = uni(rec.g / rec.tau); W.C.inv_tau = uni(1.0 / (double)rec.tau); W.C.need_sum = true;
  W.C.l2e_tau = 0.0f;
  const bool by_max = (uni(rec.mode) & WIDE_MAX) != 0u;
  const float y_max = uni(rec.y_max);  // (requested with the rest of the record, not once the mode is known)
  W.M = {by_max ? y_max : W.C.y_g, uni(by_max ? y_max : W.C.y_g + F64_REACH), by_max ? F64_MAX_BITS : F64_BITS};
  W.rep = uni(rec.rep); W.freq = uni(rec.freq); W.pres = uni(rec.pres);
  W.inv_rep = uni(1.0 / (double)rec.rep);
  W.h_active = uni(rec.h_active) != 0;
  W.distinct = uni(rec.distinct);
  W.top_k = uni(rec.top_k);
  W.ws = a.wws + (size_t)slot * a.ws_stride;
  return W;
}

// threadIdx.x as a value the compiler cannot trace: what is derived from it below (table indices, LDS
// addresses) is then formed where it is used instead of being kept across the kernels' item loops,
// where a register too many is spilled and its reload waits behind every load in flight.
__device__ __forceinline__ int fresh_tid() {
  int t = threadIdx.x;
  asm volatile("" : "+v"(t));
  return t;
}

// A slice's part of the row's history tables, in LDS: the mask words of its columns, the
// rank at the start of each of its word pairs (and of the next slice), and the counts of its
// columns, indexed by rank minus the slice's first rank.
constexpr int HCAP = 512;  // history columns of a slice that are spread over all threads; more stay with their mask word's thread
struct SliceTabs {
  uint32_t bm[SLC / 32];
  uint32_t dir[SLC / 64 + 2];
  uint16_t cnt[HCAP];   // counts of the first HCAP of them; the others' are read where they are needed
  float hz[HCAP];       // logit of the history column of rank j in the slice, as read
  uint16_t hcol[HCAP];  // its column, counted from the slice's first
};
static_assert(SLC / 32 + SLC / 64 + 1 <= WT, "one mask word or directory entry per thread");
// The tables of the slice that starts at column c0 come in two steps, so that their loads overlap
// with the other loads of an item.  First this thread's mask word or directory entry (the addresses
// follow from the slot alone):
__device__ __forceinline__ uint32_t slice_fetch(const unsigned char* ws, const SampleArgs& a, int c0) {
  const int tid = fresh_tid();
  const unsigned char* ht = ws + WS_HT;
  const int n_pairs = (((a.V + 31) >> 5) + 1) >> 1;  // the mask is stored in whole pairs of words
  const int w0 = c0 >> 5, p0 = c0 >> 6;
  uint32_t v = 0u;
  if (tid < SLC / 32) { if (w0 + tid < 2 * n_pairs) v = as_global(reinterpret_cast<const uint32_t*>(ht))[w0 + tid]; }
  else if (tid < SLC / 32 + SLC / 64 + 1) {
    const int j = tid - SLC / 32;
    if (p0 + j < n_pairs) v = (uint32_t)as_global(reinterpret_cast<const uint16_t*>(ht + a.F.dir))[p0 + j];
  }
  return v;
}
// ... stored to LDS (past the directory's end stands the number of distinct columns); a barrier must follow.
__device__ __forceinline__ void slice_store(SliceTabs& T, uint32_t v, const SampleArgs& a, int c0, uint32_t distinct) {
  const int tid = fresh_tid();
  const int n_pairs = (((a.V + 31) >> 5) + 1) >> 1;
  if (tid < SLC / 32) T.bm[tid] = v;
  else if (tid < SLC / 32 + SLC / 64 + 1) {
    const int j = tid - SLC / 32;
    T.dir[j] = ((c0 >> 6) + j < n_pairs) ? v : distinct;
  }
}
// Then, once the directory is in LDS, the counts of the slice's columns; a barrier must follow.
template <int NTHR>
__device__ __forceinline__ void slice_counts(SliceTabs& T, const unsigned char* ws, const SampleArgs& a) {
  const uint16_t* gcnt = reinterpret_cast<const uint16_t*>(ws + WS_HT + a.F.cnt);
  const unsigned r0 = T.dir[0];
  const unsigned nc = min(T.dir[SLC / 64] - r0, (unsigned)HCAP);
  for (unsigned t = threadIdx.x; t < nc; t += NTHR) T.cnt[t] = as_global(gcnt)[r0 + t];
}
// The count of the slice's column of rank r in it.
__device__ __forceinline__ uint32_t slice_count(const SliceTabs& T, const unsigned char* ws, const SampleArgs& a, unsigned r) {
  if (r < (unsigned)HCAP) return (uint32_t)T.cnt[r];
  return (uint32_t)as_global(reinterpret_cast<const uint16_t*>(ws + WS_HT + a.F.cnt))[T.dir[0] + min(r, (unsigned)SLC - 1u)];
}
// Z' of column c0 + o, whose mask bit is set.
__device__ __forceinline__ float slice_value(float z, int o, const SliceTabs& T, const WideRow& W, const SampleArgs& a) {
  const int wl = o >> 5;
  const uint32_t word = T.bm[wl];
  unsigned r = T.dir[wl >> 1] - T.dir[0];
  if (wl & 1) r += (unsigned)__popc(T.bm[wl - 1]);
  r += (unsigned)__popc(word & ((1u << (o & 31)) - 1u));
  return apply_penalties(z, slice_count(T, W.ws, a, r), W.rep, W.inv_rep, W.freq, W.pres);
}
__device__ __forceinline__ bool slice_bit(int o, const SliceTabs& T) { return (T.bm[o >> 5] >> (o & 31)) & 1u; }
// The history columns of a slice, one mask word per thread.  Their logits and the slice's counts are
// requested first (hist_fetch, right after the mask and directory reached LDS) and used later
// (hist_columns), so that their way through memory overlaps with the slice's main line, which skips
// these columns and carries no table lookups.
constexpr int HPRE = 4;  // history columns per mask word whose logits are requested ahead; more are read in place
template <typename DT>
struct HistPre { typename Io<DT>::Elem z[HPRE]; uint32_t cnt; };
template <typename DT>
__device__ __forceinline__ void hist_fetch(HistPre<DT>& P, const SliceTabs& T, const unsigned char* ws, const SampleArgs& a,
                                           const DT* rowp, int c0, int V) {
  const int tid = fresh_tid();
  const uint16_t* gcnt = reinterpret_cast<const uint16_t*>(ws + WS_HT + a.F.cnt);
  const unsigned r0 = T.dir[0];
  const unsigned nc = min(T.dir[SLC / 64] - r0, (unsigned)SLC);
  P.cnt = 0u;
  if ((unsigned)tid < nc) P.cnt = (uint32_t)as_global(gcnt)[r0 + tid];
#pragma unroll
  for (int k = 0; k < HPRE; ++k) P.z[k] = typename Io<DT>::Elem();
  if (tid < SLC / 32) {
    uint32_t word = T.bm[tid];
#pragma unroll
    for (int k = 0; k < HPRE; ++k) {
      if (word) {
        const int idx = c0 + 32 * tid + (__ffs((int)word) - 1);
        word &= word - 1u;
        if (idx < V) P.z[k] = Io<DT>::raw(rowp + idx);
      }
    }
  }
}
// The counts of the first HCAP columns go to LDS (WT of them from the registers, the rest from memory), and so do the
// logits and columns of the first HCAP history columns, by rank; a barrier must follow.
template <typename DT>
__device__ __forceinline__ void hist_stage(SliceTabs& T, const HistPre<DT>& P, const unsigned char* ws, const SampleArgs& a,
                                           const DT* rowp, int c0, int V) {
  const int tid = fresh_tid();
  const uint16_t* gcnt = reinterpret_cast<const uint16_t*>(ws + WS_HT + a.F.cnt);
  const unsigned r0 = T.dir[0];
  const unsigned nc = min(T.dir[SLC / 64] - r0, (unsigned)SLC);
  if ((unsigned)tid < nc) T.cnt[tid] = (uint16_t)P.cnt;
  for (unsigned t = tid + WT; t < min(nc, (unsigned)HCAP); t += WT) T.cnt[t] = as_global(gcnt)[r0 + t];
  if (tid < SLC / 32) {
    uint32_t word = T.bm[tid];
    unsigned r = T.dir[tid >> 1] - r0 + ((tid & 1) ? (unsigned)__popc(T.bm[tid - 1]) : 0u);
    auto put = [&](float z_raw) {
      T.hz[r] = z_raw;
      T.hcol[r] = (uint16_t)(32 * tid + (__ffs((int)word) - 1));
      word &= word - 1u;
      ++r;
    };
#pragma unroll
    for (int k = 0; k < HPRE; ++k) if (word && r < (unsigned)HCAP) put(Io<DT>::cvt(P.z[k]));
    while (word && r < (unsigned)HCAP) {
      const int idx = c0 + 32 * tid + (__ffs((int)word) - 1);
      put(idx < V ? Io<DT>::one(rowp + idx) : 0.0f);
    }
  }
}
// f(z', idx) for each history column of the slice, with its penalised value: the staged ones one per
// thread, the rest (a slice with more than HCAP of them) by their mask word's thread.
template <typename DT, typename F>
__device__ __forceinline__ void hist_columns(const SliceTabs& T, const WideRow& W, const SampleArgs& a, const DT* rowp, int c0, int V, F&& f) {
  const int tid = fresh_tid();
  const unsigned nc = min(T.dir[SLC / 64] - T.dir[0], (unsigned)SLC);
  for (unsigned j = tid; j < min(nc, (unsigned)HCAP); j += WT) {
    const int idx = c0 + (int)T.hcol[j];
    if (idx < V) f(apply_penalties(T.hz[j], (uint32_t)T.cnt[j], W.rep, W.inv_rep, W.freq, W.pres), idx);
  }
  if (nc > (unsigned)HCAP && tid < SLC / 32) {
    uint32_t word = T.bm[tid];
    unsigned r = T.dir[tid >> 1] - T.dir[0] + ((tid & 1) ? (unsigned)__popc(T.bm[tid - 1]) : 0u);
    while (word) {
      const int idx = c0 + 32 * tid + (__ffs((int)word) - 1);
      word &= word - 1u;
      if (r >= (unsigned)HCAP && idx < V)
        f(apply_penalties(Io<DT>::one(rowp + idx), slice_count(T, W.ws, a, r), W.rep, W.inv_rep, W.freq, W.pres), idx);
      ++r;
    }
  }
}

// f(z', idx) for every column of the slice that starts at c0, one at a time and from the cache (barriers inside if
// the row has a history): rows that are weighed in double precision.  (The slice was requested in 16-byte
// groups already: the groups' unrolled form with double weights, or the next slice's groups in flight
// beside this loop, took more registers than there are.)
template <typename DT, typename F>
__device__ __forceinline__ void weighed_columns(SliceTabs& T, const HistPre<DT>& HP, const WideRow& W, const SampleArgs& a, const DT* rowp,
                                                int c0, int V, F&& f) {
  const int tid = fresh_tid();
  const int n = min(V - c0, SLC);
  const DT* p = rowp + c0;
  const Exp2Poly P = exp2_poly_from_memory();
  typename Io<DT>::Elem z = tid < n ? Io<DT>::raw(p + tid) : typename Io<DT>::Elem();
#pragma unroll 1
  for (int i = tid; i < n; i += WT) {
    const typename Io<DT>::Elem next = Io<DT>::raw(p + min(i + WT, n - 1));
    if (!(W.h_active && slice_bit(i, T))) f(Io<DT>::cvt(z), c0 + i, P);
    z = next;
  }
  if (W.h_active) {
    hist_stage<DT>(T, HP, W.ws, a, rowp, c0, V);
    __syncthreads();
    hist_columns<DT>(T, W, a, rowp, c0, V, [&](float z1, int idx) { f(z1, idx, P); });
  }
}

// The bin that holds the cut, from the masses of the first pass: cumulative mass from the top
// reaches top_p * total.  bstar < 0 if none.  Ends with a barrier.
__device__ inline int find_cut(FS& S, const WideRow& W, u64& s_tot) {
  const int tid = threadIdx.x;
  constexpr int BPT = NBW / WT;
  const u64* gh = reinterpret_cast<const u64*>(W.ws + WS_HIST);
  const u64 m_top = as_global(reinterpret_cast<const u64*>(W.ws + WS_SCAL))[0];
  u64 hm[BPT]; u64 loc = 0ull;
#pragma unroll
  for (int j = 0; j < BPT; ++j) { hm[j] = as_global(gh)[tid * BPT + j]; loc += hm[j]; }
  if (tid == 0) S.bk = -1;
  unsigned ce, ct; u64 me, mt;
  blk_excl_scan2<WNW>(S, 0u, loc, ce, me, ct, mt);
  s_tot = m_top + mt;  // the bins are exact sums: this is the mass of the whole row
  const u64 target = (u64)__double2ull_ru((double)W.top_p * (double)s_tot);
  u64 run = m_top + me;
#pragma unroll
  for (int j = 0; j < BPT; ++j) {
    if (run < target && run + hm[j] >= target) S.bk = tid * BPT + j;
    run += hm[j];
  }
  __syncthreads();
  const int bstar = S.bk;
  __syncthreads();
  return bstar;
}
// The same by count, for top-k alone: the bin in which the number of columns from the top reaches
// top_k.  bstar < 0 if none (already top_k columns at or above g, or fewer than top_k in all).
__device__ inline int find_cut_k(FS& S, const WideRow& W) {
  const int tid = threadIdx.x;
  constexpr int BPT = NBW / WT;
  const u64* gh = reinterpret_cast<const u64*>(W.ws + WS_HIST);
  const unsigned n_top = as_global(reinterpret_cast<const uint32_t*>(W.ws + WS_SCAL))[7];
  unsigned hc[BPT], loc = 0u;
#pragma unroll
  for (int j = 0; j < BPT; ++j) { hc[j] = (unsigned)as_global(gh)[tid * BPT + j]; loc += hc[j]; }
  if (tid == 0) S.bk = -1;
  unsigned ce, ct; u64 me, mt;
  blk_excl_scan2<WNW>(S, loc, 0ull, ce, me, ct, mt);
  const unsigned target = (unsigned)W.top_k;
  unsigned run = n_top + ce;
#pragma unroll
  for (int j = 0; j < BPT; ++j) {
    if (run < target && run + hc[j] >= target) S.bk = tid * BPT + j;
    run += hc[j];
  }
  __syncthreads();
  const int bstar = S.bk;
  __syncthreads();
  return bstar;
}

// How a column is classified, per route: it surely survives iff its tempered value reaches thr_y and it
// lies at or above g or in a bin before bstar; columns of bin bstar are resolved one by one.
struct RowCut { int bstar; float thr_y; bool valid; u64 s_tot; /* top-p route: exact mass of the row */ };
__device__ inline RowCut row_cut(FS& S, const WideRow& W) {  // every thread calls; barriers inside on one route
  RowCut c;
  c.thr_y = -INFINITY; c.valid = true; c.s_tot = 0ull;
  if (W.mode == WIDE_TOP_P) { c.bstar = find_cut(S, W, c.s_tot); c.valid = c.bstar >= 0; }
  else if (W.mode == WIDE_TOP_K) { c.bstar = find_cut_k(S, W); c.valid = c.bstar >= 0; }
  else c.bstar = NBW;  // no bin holds a cut
  if (W.min_p > 0.0f) {  // min-p, alone or on top of top-p: the shorter prefix wins
    const uint32_t kmax = as_global(reinterpret_cast<const uint32_t*>(W.ws + WS_SCAL))[6];
    c.valid = c.valid && kmax > KEY_NEG_INF;
    c.thr_y = keyf(kmax) + W.ln_min_p;  // fl(y_max + fl(ln min_p)), as in the list's epilogue
  }
  return c;
}

// Smallest float, in the order of the keys, at which a predicate that is monotone in its argument
// (false, then true) holds; +inf if it holds nowhere.  One wave, 64 candidates per round, no LDS
// and no barrier; the result is the same in every lane.
template <typename P>
__device__ __forceinline__ float wave_lower_bound(P&& pred) {
  const unsigned lane = threadIdx.x & 63u;
  uint32_t lo = KEY_NEG_INF, hi = KEY_POS_INF;
  if (__ballot(pred(keyf(hi))) == 0ull) return INFINITY;
  while (lo < hi) {  // the answer lies in [lo, hi] and the predicate holds at hi
    const u64 step = ((u64)hi - (u64)lo + 63ull) / 64ull;
    const u64 c = (u64)lo + step * (u64)lane;
    const uint32_t cand = (c < (u64)hi) ? (uint32_t)c : hi;
    const u64 m = __ballot(pred(keyf(cand)));
    if (m == 0ull) { lo = (uint32_t)((u64)lo + 63ull * step) + 1u; continue; }  // lane 63 stood below hi
    const unsigned f = (unsigned)__ffsll((long long)m) - 1u;
    const u64 cf = (u64)lo + step * (u64)f;
    const uint32_t top = (cf < (u64)hi) ? (uint32_t)cf : hi;
    lo = f ? (uint32_t)((u64)lo + step * (u64)(f - 1u)) + 1u : top;
    hi = top;
  }
  return keyf(uni(lo));
}
// The same, trying first the 64 floats around a guess: one round when the answer lies among them.
template <typename P>
__device__ __forceinline__ float wave_lower_bound_near(float guess, P&& pred) {
  const unsigned lane = threadIdx.x & 63u;
  const uint32_t kg = fkey(uni(guess));
  if (guess == guess && kg >= KEY_NEG_INF + 32u && kg <= KEY_POS_INF - 32u) {
    const u64 m = __ballot(pred(keyf(kg - 32u + lane)));
    if (!(m & 1ull) && (m >> 63)) return keyf(uni(kg - 32u + (uint32_t)__ffsll((long long)m) - 1u));
  }
  return wave_lower_bound(pred);
}
// The classification of a column by its logit alone.  Tempered value, bin and the comparison with
// g are all monotone in z, so each test holds from one float upwards, and so do their
// combinations: a column surely survives iff z >= z_sure, and is a boundary column iff
// z_edge <= z < z_sure.  Every wave computes the same two numbers.
struct ZCut { float z_sure, z_edge; };
__device__ __forceinline__ ZCut z_cut(const WideRow& W, int bstar, float thr_y) {
  // smallest z whose tempered value reaches the min-p threshold
  float z_thr = -INFINITY;
  if (thr_y > -INFINITY) z_thr = wave_lower_bound_near(thr_y * W.tau, [&](float z) { return tempered(z, W.C) >= thr_y; });
  // smallest z whose bin lies before `limit` (bins count downwards from y_g, 1 / BINS_PER_LOG2 of a log2 each)
  auto before_bin = [&](int limit) -> float {
    if (limit >= NBW) return -INFINITY;
    if (limit <= 0) return INFINITY;
    const float y_guess = W.C.y_g - (float)limit * (0.6931471805599453f / BINS_PER_LOG2);
    return wave_lower_bound_near(y_guess * W.tau, [&](float z) { int b; (void)mass_term(z, W.C, b); return b < limit; });
  };
  const float z_a = before_bin(bstar), z_b = before_bin(bstar + 1);
  ZCut c;  // sure: y >= thr and (z >= g or bin < bstar); sure or boundary: the same with bin <= bstar
  c.z_sure = fmaxf(z_thr, fminf(W.C.g, z_a));
  c.z_edge = fmaxf(z_thr, fminf(W.C.g, z_b));
  return c;
}

// Work split: items are (queued row, slice) pairs in row-major order; a workgroup takes a
// contiguous range, so that it meets few distinct rows.
struct Items { unsigned i0, i1, n_sl, chunk; };
__device__ __forceinline__ Items my_items(const SampleArgs& a) {
  Items I;
  const unsigned n_wide = min(as_global(a.wq)[0], (unsigned)a.wide_slots);
  I.n_sl = (unsigned)((a.V + SLC - 1) / SLC);
  const unsigned items = n_wide * I.n_sl;
  I.chunk = (items + gridDim.x - 1u) / gridDim.x;
  I.i0 = min(items, blockIdx.x * I.chunk);
  I.i1 = min(items, I.i0 + I.chunk);
  return I;
}

// What an item needs from memory before its columns can be processed; requested one item ahead.
template <typename DT>
struct ItemLoads {
  static constexpr int G = SLC / (WT * Io<DT>::EPL);  // 16-byte groups per thread and slice
  typename Io<DT>::Raw A[G];
  uint32_t hq[G];  // hot-set bits of each group's columns
  uint32_t pre;    // this thread's mask word or directory entry
};
// classify: rows without truncation never come here; else (the bins kernel) only they need the hot bits
template <typename DT, bool use_hot, bool classify>
__device__ __forceinline__ void item_fetch(ItemLoads<DT>& L, const SampleArgs& a, const WideRow& W, int c0) {
  constexpr int EPL = Io<DT>::EPL;
  const int tid = threadIdx.x;
  const DT* rowp = reinterpret_cast<const DT*>(a.logits) + (size_t)W.row * (size_t)a.stride;
  L.pre = W.h_active ? slice_fetch(W.ws, a, c0) : 0u;
#pragma unroll
  for (int j = 0; j < ItemLoads<DT>::G; ++j) {
    const int idx0 = c0 + (j * WT + tid) * EPL;
    L.hq[j] = 0u;
    L.A[j] = typename Io<DT>::Raw();
    if (idx0 + EPL <= a.V) L.A[j] = Io<DT>::load(rowp + idx0);
    if (use_hot && (classify || W.mode == WIDE_ALL) && idx0 < a.V) L.hq[j] = (as_global(a.hot_bits)[idx0 >> 5] >> ((unsigned)idx0 & 31u)) & ((1u << EPL) - 1u);
  }
}

// ---------------------------------------------------------------- runs of slices -------------
// bfloat16 rows with a nucleus take a workgroup's slices of one row in a run.  Under one temperature a column's bin, mass and
// class are functions of its 16 bits, so the bins kernel counts columns per pattern and the classifying kernel looks them up, one
// LDS access a column, with no barrier and no table of the history from slice to slice; what the run's history columns change is settled
// once behind it: their weight as read is taken off, the penalised one added (integers: the sums are those of the column by column form).
// What bounded it: 39 and 54 vector instructions a column, and per slice of 4096 columns four barriers, its tables and its
// history columns, 2 to 3 us of a slice's 5 to 9.  338 rows of 256,000 columns with 8192 ids each: bins kernel 101 us, 83 so (the slices
// take 25 to 30, the 173 MB at the HBM rate; the history columns 18); classifying kernel 185, 112 (slices 55).  float32 rows the
// same way, each column weighed: no gain (90 of 128,256 columns, 21 and 26 us either way).
// A run's table and the settling of its history columns cost the workgroups of one resident round the same whether they take few
// slices or many, and the history columns of a run cost more than a slice's: so from so many slices a workgroup, the more history columns
// a slice has, up to so many of these.  By slices over by runs, the whole call, V = 20,000 / 40,000 / 128,256 / 256,000 columns:
//   64 ids a row       2 to 9 history columns a slice:   4 slices a workgroup 1.00 1.01 1.04 0.98, 6: 1.01 1.04 1.04 1.01, 8: 1.06 1.11 1.19 1.10, 16: 1.08 1.15 1.36 1.21
//   2048 ids           152, 81, 27, 15 of them:          6: 0.93 0.97 1.02 1.01, 9: 0.95 1.05 1.11 1.20, 16: 0.94 1.02 1.28 1.20
//   8192 ids           431, 238, 85, 45 of them:         7: 0.79 0.84 0.96 1.06, 9: 0.79 0.89 1.02 1.09, 16: 0.79 0.85 1.06 1.11
// (80,000 columns, 129 history columns a slice: 0.98 with 16 slices, 0.99 with 24.)  Pieces of a row with one or two slices are taken by
// slices: with 6 slices a workgroup 1.04 against 1.02 (128,256 columns, 64 ids), a longer limit 0.99.
// The two kernels divide the slices alike (one grid), so that the same slices are counted and looked up.
constexpr int RUN_MIN = 6, RUN_IDS = 24, RUN_MAX_IDS = 96, RUN_PIECE = 3;
// A lane's group with a value that has no entry goes column by column, at a cost that only few groups may have: rows whose threshold
// lies where there is none (a sample's quantile, it stands for the large values), or from which -256 has mass, are taken by
// slices.  (512 rows of 256,000 columns, every logit raised by 300, by runs and by slices: 14.2 and 3.9 ms a call.)
__device__ __forceinline__ bool values_in_table(const StreamCtx& C) {
  int b;
  const float w = mass_term(-256.0f, C, b), m = fabsf(C.g);
  return m >= 0x1p-6f && m < 256.0f && b == NBW - 1 && mass_integer(w) == 0.0f;
}
__device__ __forceinline__ bool takes_run(const WideRow& W, const Items& I, int sl0, int sl1) {
  const unsigned per_slice = W.distinct / I.n_sl;
  return W.mode == WIDE_TOP_P && !W.f64 && sl1 - sl0 >= RUN_PIECE && per_slice <= (unsigned)RUN_MAX_IDS && I.chunk >= RUN_MIN + per_slice / RUN_IDS && values_in_table(W.C);
}
// One 4-byte entry a pattern: magnitude index 0 is zero itself, 1 .. QMAX - 1 one pattern each, QMAX, among the negative
// ones, -256 and all below it (-inf among them), which has no mass.  None: other magnitudes below 2^-14, 256 and more, NaN.
constexpr uint32_t PT_NEG = 0x4000u;  // byte offset of the negative patterns' entries: the sign bit, moved down one
constexpr uint32_t PT_BYTES = PT_NEG + (uint32_t)NMAG * 4u;
// Byte offsets of the two patterns of a word, low pattern in the low half.
__device__ __forceinline__ uint32_t pattern_offsets2(uint32_t x) {
  u16x2 q = __builtin_elementwise_sub_sat(__builtin_bit_cast(u16x2, x & 0x7FFF7FFFu), (u16x2)((unsigned short)(PLO - 1)));
  q = __builtin_elementwise_min(q, (u16x2)((unsigned short)QMAX)) << (unsigned short)2;
  uint32_t off = ((x >> 1) & (PT_NEG | PT_NEG << 16)) | __builtin_bit_cast(uint32_t, q);
  asm("" : "+v"(off));  // (formed once: the compiler forms it anew for either half)
  return off;
}
__device__ __forceinline__ uint32_t pattern_offset(float z) { return pattern_offsets2(__float_as_uint(z) >> 16) & 0xFFFFu; }
// Value and byte offset of table index i (< 2 NMAG).
__device__ __forceinline__ float pattern_value(int i, uint32_t& off) {
  const int neg = i >= NMAG ? 1 : 0, q = i - neg * NMAG;
  off = (uint32_t)neg * PT_NEG + (uint32_t)q * 4u;
  return __uint_as_float(((uint32_t)neg << 31) | ((q ? (uint32_t)(q + PLO - 1) : 0u) << 16));
}
// Whether all patterns of some groups have an entry.
struct PatternRange {
  s16x2 smax = {0, 0};            // the largest positive pattern
  u16x2 umax = {0, 0};            // the negative one of the largest magnitude
  u16x2 pmin = {0xFFFF, 0xFFFF};  // the smallest magnitude less one: zero itself is out of the way
  __device__ __forceinline__ void take(uint32_t x) {
    smax = __builtin_elementwise_max(smax, __builtin_bit_cast(s16x2, x));
    umax = __builtin_elementwise_max(umax, __builtin_bit_cast(u16x2, x));
    pmin = __builtin_elementwise_min(pmin, (u16x2)(__builtin_bit_cast(u16x2, x & 0x7FFF7FFFu) - (u16x2)((unsigned short)1)));
  }
  __device__ __forceinline__ bool ok() const {
    return max((int)smax.x, (int)smax.y) < PHI && max((uint32_t)umax.x, (uint32_t)umax.y) <= 0xFF80u && min((uint32_t)pmin.x, (uint32_t)pmin.y) >= (uint32_t)(PLO - 1);
  }
};

// f(idx, z, z', hot) for every history column of the slices [sl0, sl1) of a row: the logit as read and the penalised one.
// The mask's columns first go to a list in LDS, a column's place its rank less the run's first, so that all threads then have
// the same number of them, four on their way at a time.  (Taken from a thread's own mask words they came one or two at a
// time, a trip to memory each: 35 us of a row's 21 slices with 1300 such columns, 18 so.)  Barriers inside.
constexpr int HLIST = 1024;
template <typename DT, bool use_hot, typename F>
__device__ __forceinline__ void hist_run(const WideRow& W, const SampleArgs& a, const DT* rowp, int sl0, int sl1, uint32_t* list, F&& f) {
  const int n_pairs = (((a.V + 31) >> 5) + 1) >> 1, p0 = sl0 * (SLC / 64), p1 = min(sl1 * (SLC / 64), n_pairs);
  const unsigned char* ht = W.ws + WS_HT;
  const u64* mask = reinterpret_cast<const u64*>(ht);
  const uint16_t* dir = reinterpret_cast<const uint16_t*>(ht + a.F.dir);
  const uint16_t* cnt = reinterpret_cast<const uint16_t*>(ht + a.F.cnt);
  const unsigned r0 = uni((uint32_t)as_global(dir)[p0]), n = (p1 < n_pairs ? uni((uint32_t)as_global(dir)[p1]) : W.distinct) - r0;
  constexpr int AT = 4;
#pragma unroll 1
  for (unsigned first = 0; first < n; first += HLIST) {
    __syncthreads();  // (the list's last use)
#pragma unroll 1
    for (int q = p0 + fresh_tid(); q < p1; q += AT * WT) {
      u64 m[AT]; unsigned r[AT];
#pragma unroll
      for (int k = 0; k < AT; ++k) {
        const int p = min(q + k * WT, p1 - 1);
        m[k] = as_global(mask)[p]; r[k] = (unsigned)as_global(dir)[p];
      }
#pragma unroll
      for (int k = 0; k < AT; ++k) {
        if (q + k * WT >= p1) continue;
        unsigned at = r[k] - r0 - first;
#pragma unroll 1
        for (u64 x = m[k]; x; x &= x - 1ull, ++at) if (at < (unsigned)HLIST) list[at] = (uint32_t)(64 * (q + k * WT) + __ffsll((long long)x) - 1);
      }
    }
    __syncthreads();
    const unsigned nl = min(n - first, (unsigned)HLIST);
#pragma unroll 1
    for (unsigned t = (unsigned)fresh_tid(); t < nl; t += AT * WT) {
      int idx[AT]; typename Io<DT>::Elem z[AT]; uint32_t c[AT], h[AT];
#pragma unroll
      for (int k = 0; k < AT; ++k) {
        const unsigned u = min(t + (unsigned)(k * WT), nl - 1u);
        idx[k] = (int)list[u];
        c[k] = (uint32_t)as_global(cnt)[r0 + first + u];
      }
#pragma unroll
      for (int k = 0; k < AT; ++k) {
        z[k] = Io<DT>::raw(rowp + min(idx[k], a.V - 1));
        h[k] = use_hot ? as_global(a.hot_bits)[min(idx[k], a.V - 1) >> 5] : 0u;
      }
#pragma unroll
      for (int k = 0; k < AT; ++k) {
        if (t + (unsigned)(k * WT) >= nl || idx[k] >= a.V) continue;
        const float zr = Io<DT>::cvt(z[k]);
        f(idx[k], zr, apply_penalties(zr, c[k], W.rep, W.inv_rep, W.freq, W.pres), ((h[k] >> (idx[k] & 31)) & 1u) != 0u);
      }
    }
  }
}
__device__ __forceinline__ bool hist_bit(const WideRow& W, int idx) {  // (from memory)
  return W.h_active && ((as_global(reinterpret_cast<const uint32_t*>(W.ws + WS_HT))[idx >> 5] >> (idx & 31)) & 1u) != 0u;
}
// The 16-byte groups of a slice, and the hot-set words of their columns.  (No load under a branch: at a join the compiler waits
// for all that is in flight.  A group that the row's end cuts reads other columns, and is not used.)
template <typename DT> struct RunLoads { typename Io<DT>::Raw A[ItemLoads<DT>::G]; uint32_t hq[ItemLoads<DT>::G]; };
template <typename DT, bool use_hot>
__device__ __forceinline__ void run_fetch(RunLoads<DT>& L, const SampleArgs& a, const DT* rowp, int sl, bool none) {
  constexpr int EPL = Io<DT>::EPL;
  const int tid = threadIdx.x;
#pragma unroll
  for (int j = 0; j < ItemLoads<DT>::G; ++j) {
    const int idx0 = sl * SLC + (j * WT + tid) * EPL;
    L.A[j] = Io<DT>::load(rowp + (none ? 0 : min(idx0, a.V - EPL)));
    L.hq[j] = 0u;
    if (use_hot) L.hq[j] = as_global(a.hot_bits)[none || idx0 >= a.V ? 0 : idx0 >> 5];
  }
}
template <typename DT>
__device__ __forceinline__ void run_settle(RunLoads<DT>& L) {  // waits for them
#pragma unroll
  for (int j = 0; j < ItemLoads<DT>::G; ++j) asm volatile("" : "+v"(L.A[j]), "+v"(L.hq[j]));
}
// The i-th of four words (by selects: an indexed array goes to scratch memory).
__device__ __forceinline__ uint32_t select4(uint32_t x0, uint32_t x1, uint32_t x2, uint32_t x3, int i) {
  asm("" : "+v"(x0), "+v"(x1), "+v"(x2), "+v"(x3));
  const uint32_t lo = (i & 1) ? x1 : x0, hi = (i & 1) ? x3 : x2;
  return (i & 2) ? hi : lo;
}
// Sum over each row of sixteen lanes of values below 2^54, in two halves (one instruction per step: the move is part of the addition).
__device__ __forceinline__ u64 row16_sum_u64(u64 v) {
  auto sum = [](uint32_t x) {
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, DPP_XOR1, 0xF, 0xF, true);
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, DPP_XOR2, 0xF, 0xF, true);
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, DPP_HALF_MIRROR, 0xF, 0xF, true);
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, DPP_MIRROR, 0xF, 0xF, true);
    return x;
  };
  constexpr uint32_t LOW = (1u << 27) - 1u;
  return (u64)sum((uint32_t)v & LOW) + ((u64)sum((uint32_t)(v >> 27)) << 27);
}
static_assert(SLC / WT * 2 <= 32, "a lane's columns of a slice, below 2^49 each, sum below 2^54");
// Whether all eight patterns of a group have an entry.
__device__ __forceinline__ bool group_ok(const u32x4& w) {
  PatternRange R;
  R.take(w.x); R.take(w.y); R.take(w.z); R.take(w.w);
  return R.ok();
}

// ---------------------------------------------------------------- no truncation ---------------
// exp(y - m) for y <= m (float32, split log2(e)); a NaN stays one
__device__ __forceinline__ float mass_rel(float y, float m) {
  const float d = y - m;
  return __builtin_amdgcn_exp2f(fmaf(d, L2E_HI, d * L2E_LO));
}
// q where bit e of hq is set, else 0
__device__ __forceinline__ float hot_only(float q, uint32_t hq, int e) {
  int m = __builtin_amdgcn_sbfe((int)hq, (unsigned)e, 1u);
  asm("" : "+v"(m));  // (kept a mask: else a test and two selects of the sum's term)
  return __uint_as_float(__float_as_uint(q) & (uint32_t)m);
}
// One slice of a row without truncation: every wave leaves the mass of its columns.  The row is read once;
// bound: HBM, with about 25 vector instructions a column beside it.  (128,256 float32 columns x 256 rows:
// classified in the second kernel, a column 2^21 above g sending the row to the general kernel, the call
// took 120 us, 229 with three such rows; 64 so.)
template <typename DT, bool use_hot>
__device__ __forceinline__ void all_slice(const ItemLoads<DT>& L, const HistPre<DT>& HP, SliceTabs& Tb, const WideRow& W, const SampleArgs& a,
                                          const DT* rowp, int c0, int sl, int slot) {
  constexpr int EPL = Io<DT>::EPL, G = ItemLoads<DT>::G;
  const int tid = fresh_tid(), V = a.V;
  float y[G][EPL];
  float m = LOWEST;
  bool far = false;  // a mass the fixed point cannot carry, or a NaN
  u64 s = 0ull, h = 0ull;
  auto weigh = [&](float yv) {  // exp(y - y_g), as in mass_term
    const float w = mass_rel(yv, W.C.y_g);
    far = far || !(w <= W_LIMIT);
    return w;
  };
#pragma unroll
  for (int j = 0; j < G; ++j) {
    const int o = (j * WT + tid) * EPL;
    Io<DT>::unpack(L.A[j], y[j]);
    if (c0 + o + EPL > V) {  // the ragged end of the row
#pragma unroll
      for (int e = 0; e < EPL; ++e) y[j][e] = c0 + o + e < V ? Io<DT>::one(rowp + c0 + o + e) : -INFINITY;
    }
    const uint32_t nib = W.h_active ? Tb.bm[o >> 5] >> ((unsigned)o & 31u) : 0u;  // history columns: below
    double gs = SUM_BASE, gh = SUM_BASE;  // <= 8 terms of <= 2^49
#pragma unroll
    for (int e = 0; e < EPL; ++e) {
      y[j][e] = ((nib >> e) & 1u) ? -INFINITY : tempered(y[j][e], W.C);
      m = fmaxf(m, y[j][e]);
      const float q = mass_integer(weigh(y[j][e]));
      gs += (double)q;
      if (use_hot) gh += (double)hot_only(q, L.hq[j], e);
    }
    s += sum_to_u64(gs);
    if (use_hot) h += sum_to_u64(gh);
  }
  if (W.h_active) {
    hist_stage<DT>(Tb, HP, W.ws, a, rowp, c0, V);
    __syncthreads();
    hist_columns<DT>(Tb, W, a, rowp, c0, V, [&](float z, int idx) {
      const float yv = tempered(z, W.C);
      m = fmaxf(m, yv);
      const u64 f = mass_fix(weigh(yv));
      s += f;
      if (use_hot && hot_bit(a.hot_bits, (uint32_t)idx)) h += f;
    });
  }
  const float M = wave_max(m);
  s = wave_sum(s);
  if (use_hot) h = wave_sum(h);
  if (W.h_active) __syncthreads();  // the tables are rewritten by the next item
  const bool any_far = __ballot(far) != 0ull;
  if ((tid & 63) == 0) {
    AllPart* part = reinterpret_cast<AllPart*>(W.ws + WS_HIST) + sl * WNW + (tid >> 6);
    part->s = s; part->h = h; part->m = M;
    if (any_far || (W.f64 && sl == 0)) mark_far(a.wq, (unsigned)slot);  // the second kernel weighs the row again
  }
}

// ---------------------------------------------------------------- bins ------------------------
template <typename DT, bool use_hot, bool RUNS>  // RUNS: the call may bring runs of slices (bfloat16)
__global__ __launch_bounds__(WT, (bins_wgs<DT, RUNS>())) void wide_bins_kernel(const SampleArgs a) {
  constexpr int EPL = Io<DT>::EPL;
  constexpr int G = ItemLoads<DT>::G;
  __shared__ SliceTabs Tb;
  constexpr uint32_t ACC_BYTES = RUNS ? PT_BYTES : (uint32_t)(NBW + 1) * 8u;
  static_assert(ACC_BYTES >= (uint32_t)(NBW + 1) * 8u, "the bins fit");
  __shared__ __align__(16) u64 lh[(ACC_BYTES + 15u) / 16u * 2u];  // the bins, and the mass at or above g; runs: columns per pattern
  __shared__ uint32_t odd[4];  // runs: slices with groups that went column by column
  __shared__ uint32_t hlist[HLIST];
  __shared__ FS S;
  static_assert((sizeof(Tb) + sizeof(lh) + (RUNS ? sizeof(odd) + sizeof(hlist) : 0u) + sizeof(S)) * bins_wgs<DT, RUNS>() <= LDS_PER_CU, "a resident round by LDS");
  const int tid = threadIdx.x;
  const int V = a.V;
  // mask word and bit of this thread's first column in each of its groups (a group step is whole words)
  const int wbase = (tid * EPL) >> 5;
  const unsigned wsh = (unsigned)(tid * EPL) & 31u;
  static_assert((WT * EPL) % 32 == 0, "group stride in mask words");
  const Items I = my_items(a);
  for (unsigned i0 = I.i0, i1; i0 < I.i1; i0 = i1) {  // the slices [sl0, sl1) of one row
  const unsigned slot = i0 / I.n_sl;
  i1 = min(I.i1, (slot + 1u) * I.n_sl);
  const int sl0 = (int)(i0 - slot * I.n_sl), sl1 = sl0 + (int)(i1 - i0);
  const WideRow W = load_row(a, slot);
  const DT* rowp = reinterpret_cast<const DT*>(a.logits) + (size_t)W.row * (size_t)a.stride;
  if (i0 != I.i0) __syncthreads();  // (what the row before left in LDS has been read)
  zero16(lh, (int)ACC_BYTES, tid, WT);
  u64 mtop = 0ull;
  unsigned ntop = 0u;      // top-k route: columns at or above g seen by this thread
  float ymax = -INFINITY;  // rows with a min-p cut: largest tempered value seen by this thread
  const bool run = RUNS && takes_run(W, I, sl0, sl1);
  auto flush = [&]() {
    __syncthreads();
    if (W.mode == WIDE_TOP_P || W.mode == WIDE_TOP_K) {
      u64* gh = reinterpret_cast<u64*>(W.ws + WS_HIST);
      if (run) {
#pragma unroll 1
        for (int i = tid; i < 2 * NMAG - 1; i += WT) {  // (the last entry has no mass)
          uint32_t off;
          const float z = pattern_value(i, off);
          const uint32_t c = reinterpret_cast<const uint32_t*>(lh)[off / 4u];
          if (c == 0u) continue;
          int b; float y;
          const float w = mass_term(z, W.C, b, y);
          ymax = fmaxf(ymax, y);
          const u64 m = (u64)c * sum_to_u64(SUM_BASE + (double)mass_integer(fminf(w, W_LIMIT)));
          if (!(z < W.C.g)) mtop += m;
          else if (m) atomicAdd(&gh[b], m);
        }
        if (tid < 4 && odd[tid]) atomicOr(reinterpret_cast<uint32_t*>(W.ws + WS_ODD) + tid, odd[tid]);
      } else {
        for (int b = tid; b < NBW; b += WT) { const u64 v = lh[b]; if (v) atomicAdd(&gh[b], v); }
      }
      const u64 t = blk_sum_u64<WNW>(S, mtop) + (run ? 0ull : lh[NBW]);
      if (tid == 0 && t) atomicAdd(reinterpret_cast<u64*>(W.ws + WS_SCAL), t);
      if (W.mode == WIDE_TOP_K) {
        const unsigned nt = wave_sum(ntop);
        if ((tid & 63) == 0 && nt) atomicAdd(reinterpret_cast<uint32_t*>(W.ws + WS_SCAL) + 7, nt);
      }
    }
    if (W.min_p > 0.0f || run) {  // (counted rows: the classifying kernel does not form it again)
      const float m = wave_max(ymax);
      if ((tid & 63) == 0 && m > -INFINITY) atomicMax(reinterpret_cast<uint32_t*>(W.ws + WS_SCAL) + 6, fkey(m));
    }
  };
  if constexpr (RUNS) if (run) {
    if (tid < 4) odd[tid] = 0u;
    RunLoads<DT> N;
    run_fetch<DT, false>(N, a, rowp, sl0, false);
    __syncthreads();  // the zeroed bins are visible
    // a column that is not counted by its pattern: straight to the row's bins
    auto add_column = [&](float z) {
      int b; float y;
      const float w = mass_term(z, W.C, b, y);
      const u64 m = sum_to_u64(SUM_BASE + (double)mass_integer(fminf(w, W_LIMIT)));
      ymax = fmaxf(ymax, y);
      if (!(z < W.C.g)) mtop += m;
      else if (m) atomicAdd(&reinterpret_cast<u64*>(W.ws + WS_HIST)[b], m);
    };
    auto count = [&](uint32_t off, uint32_t n) {
      __hip_atomic_fetch_add(reinterpret_cast<uint32_t*>(lh) + off / 4u, n, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    };
#pragma unroll 1
    for (int sl = sl0; sl < sl1; ++sl) {
      RunLoads<DT> L = N;
      run_settle(L);
      run_fetch<DT, false>(N, a, rowp, sl + 1, sl + 1 == sl1);
#pragma unroll
      for (int j = 0; j < G; ++j) {
        const int idx0 = sl * SLC + (j * WT + tid) * EPL;
        if (idx0 + EPL > V) {  // the ragged end of the row
          for (int idx = idx0; idx < V; ++idx) if (!hist_bit(W, idx)) add_column(Io<DT>::one(rowp + idx));
        } else {
          const u32x4 w = L.A[j];
          if (group_ok(w)) {
            const uint32_t w4[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
            for (int k = 0; k < 4; ++k) { const uint32_t off = pattern_offsets2(w4[k]); count(off & 0xFFFFu, 1u); count(off >> 16, 1u); }
          } else {
            atomicOr(&odd[sl >> 5], 1u << (sl & 31));
#pragma unroll 1
            for (int e = 0; e < EPL; ++e) if (!hist_bit(W, idx0 + e)) add_column(Io<DT>::one(rowp + idx0 + e));
          }
        }
        __builtin_amdgcn_sched_barrier(0);  // one group at a time: interleaving them costs registers
      }
    }
    if (W.h_active) {
      const int whole = V & ~(EPL - 1);  // (not those behind the last whole group)
      hist_run<DT, false>(W, a, rowp, sl0, sl1, hlist, [&](int idx, float z, float zp, bool) {
        const bool slice_odd = ((odd[idx / SLC >> 5] >> (idx / SLC & 31)) & 1u) != 0u;
        if (idx < whole && (!slice_odd || group_ok(Io<DT>::load(rowp + (idx & ~(EPL - 1)))))) count(pattern_offset(z), 0xFFFFFFFFu);
        add_column(zp);
      });
    }
    flush();
    continue;
  }
  ItemLoads<DT> N;  // the next item's loads
  item_fetch<DT, use_hot, false>(N, a, W, sl0 * SLC);
  for (int sl = sl0; sl < sl1; ++sl) {
    const int c0 = sl * SLC;
    const ItemLoads<DT> L = N;
    const bool more = sl + 1 < sl1;
    HistPre<DT> HP;
    if (W.h_active) {
      slice_store(Tb, L.pre, a, c0, W.distinct);
      __syncthreads();
      hist_fetch<DT>(HP, Tb, W.ws, a, rowp, c0, V);  // this item's own loads go first: loads return in order
    } else __syncthreads();  // the zeroed bins are visible
    if (W.f64 && W.mode == WIDE_TOP_P) {
      weighed_columns<DT>(Tb, HP, W, a, rowp, c0, V, [&](float z, int, const Exp2Poly& P) {
        int b; float y;
        (void)mass_term(z, W.C, b, y);
        ymax = fmaxf(ymax, y);
        const u64 m = mass_fix64(y, W.M, P);
        if (z < W.C.g) atomicAdd(&lh[b], m); else mtop += m;
      });
      if (W.h_active) __syncthreads();  // the tables are rewritten by the next item
      if (more) item_fetch<DT, use_hot, false>(N, a, W, c0 + SLC);
      continue;
    }
    if (more) item_fetch<DT, use_hot, false>(N, a, W, c0 + SLC);
    if (W.mode == WIDE_ALL) {  // every column survives: this wave's masses
      all_slice<DT, use_hot>(L, HP, Tb, W, a, rowp, c0, sl, (int)slot);
      continue;
    }
    auto one = [&](float z, int) {
      if (W.mode == WIDE_MIN_P) { ymax = fmaxf(ymax, tempered(z, W.C)); return; }
      int b; float y;
      const float w = mass_term(z, W.C, b, y);
      ymax = fmaxf(ymax, y);
      // top-k route: a bin counts its columns
      if (z < W.C.g) atomicAdd(&lh[b], W.mode == WIDE_TOP_K ? 1ull : mass_fix_below(w));
      else { mtop += mass_fix(fminf(w, W_LIMIT)); ++ntop; }
    };
    if (W.mode == WIDE_MIN_P) {  // the row maximum is all a value cut needs
#pragma unroll
      for (int j = 0; j < G; ++j) {
        const int idx0 = c0 + (j * WT + tid) * EPL;
        if (idx0 + EPL <= V) {
          float z[EPL];
          Io<DT>::unpack(L.A[j], z);
          const uint32_t nib = W.h_active ? (Tb.bm[wbase + j * (WT * EPL / 32)] >> wsh) & ((1u << EPL) - 1u) : 0u;
          float zm = -INFINITY;  // the tempered value is monotone in z: one division per group
#pragma unroll
          for (int e = 0; e < EPL; ++e) zm = ((nib >> e) & 1u) ? zm : fmaxf(zm, z[e]);
          ymax = fmaxf(ymax, tempered(zm, W.C));
        } else {
          for (int idx = idx0; idx < V; ++idx)
            if (!(W.h_active && slice_bit(idx - c0, Tb))) one(Io<DT>::one(rowp + idx), idx);
        }
      }
    } else {
      auto sweep = [&](auto unit_tau_c, auto top_k_c) {
        constexpr bool UT = decltype(unit_tau_c)::value, TOPK = decltype(top_k_c)::value;
#pragma unroll
        for (int j = 0; j < G; ++j) {
          const int idx0 = c0 + (j * WT + tid) * EPL;
          if (idx0 + EPL <= V) {
            float z[EPL];
            Io<DT>::unpack(L.A[j], z);
            uint32_t nib = 0u;
            if (W.h_active) {  // history columns are handled below: here they count as -inf (no mass)
              nib = (Tb.bm[wbase + j * (WT * EPL / 32)] >> wsh) & ((1u << EPL) - 1u);
#pragma unroll
              for (int e = 0; e < EPL; ++e) z[e] = ((nib >> e) & 1u) ? -INFINITY : z[e];
            }
#pragma unroll
            for (int e = 0; e < EPL; ++e) {  // straight-line: the columns at or above g share one more slot
              int b;
              const float w = mass_term<UT>(z[e], W.C, b);
              const bool below = z[e] < W.C.g;
              u64 v = sum_to_u64(SUM_BASE + (double)mass_integer(fminf(w, W_LIMIT)));
              if (TOPK) {  // the bin counts the column instead (not the history columns, handled below)
                v = (below && !((nib >> e) & 1u)) ? 1ull : 0ull;
                ntop += below ? 0u : 1u;
              }
              atomicAdd(&lh[below ? b : NBW], v);
            }
            if (W.min_p > 0.0f) {  // the tempered value is monotone in z: one division per group
              float zm = z[0];
#pragma unroll
              for (int e = 1; e < EPL; ++e) zm = fmaxf(zm, z[e]);
              ymax = fmaxf(ymax, tempered(zm, W.C));
            }
          } else {
            for (int idx = idx0; idx < V; ++idx)
              if (!(W.h_active && slice_bit(idx - c0, Tb))) one(Io<DT>::one(rowp + idx), idx);
          }
          __builtin_amdgcn_sched_barrier(0);  // one group at a time: interleaving them costs registers
        }
      };
      const std::true_type yes{};
      const std::false_type no{};
      if (W.mode == WIDE_TOP_K) { if (W.tau == 1.0f) sweep(yes, yes); else sweep(no, yes); }
      else { if (W.tau == 1.0f) sweep(yes, no); else sweep(no, no); }
    }
    if (W.h_active) {  // the history columns, whose logits and counts were requested before the main line
      hist_stage<DT>(Tb, HP, W.ws, a, rowp, c0, V);
      __syncthreads();
      hist_columns<DT>(Tb, W, a, rowp, c0, V, one);
      __syncthreads();  // the tables are rewritten by the next item
    }
  }
  flush();
  }
}

// ---------------------------------------------------------------- classify --------------------
// The far rows: the masses of their slices again, in double precision and relative to the slice's largest column.
// The slices of all of them are dealt out over the workgroups (with each row's to the few that hold it, as the
// other rows' are, one such row among 256 untruncated ones took 26 us).
template <typename DT, bool use_hot>
__device__ __forceinline__ void far_rows(SliceTabs& Tb, FS& S, const SampleArgs& a) {
  const int tid = threadIdx.x, V = a.V;
  const unsigned n_sl = (unsigned)((V + SLC - 1) / SLC), n = min(as_global(a.wq)[1], (unsigned)a.wide_slots) * n_sl;
  for (unsigned it = blockIdx.x; it < n; it += gridDim.x) {
    const int sl = (int)(it % n_sl), c0 = sl * SLC;
    const WideRow W = load_row(a, uni(reinterpret_cast<const WideRec*>(a.wq + WQ_HEAD)[it / n_sl].far_slot));
    const DT* rowp = reinterpret_cast<const DT*>(a.logits) + (size_t)W.row * (size_t)a.stride;
    AllPart* part = reinterpret_cast<AllPart*>(W.ws + WS_HIST) + sl * WNW;
    float M = LOWEST;
#pragma unroll
    for (int k = 0; k < WNW; ++k) M = fmaxf(M, part[k].m);
    HistPre<DT> HP;
    if (W.h_active) {
      slice_store(Tb, slice_fetch(W.ws, a, c0), a, c0, W.distinct);
      __syncthreads();
      hist_fetch<DT>(HP, Tb, W.ws, a, rowp, c0, V);
    }
    u64 s = 0ull, h = 0ull, mx = 0ull;
    unsigned bad = 0u, none = 0u;
    weighed_columns<DT>(Tb, HP, W, a, rowp, c0, V, [&](float z, int idx, const Exp2Poly& P) {
      const float y = tempered(z, W.C);
      bad |= y != y ? 1u : 0u;
      const u64 m = exp_fix<44>(y, M, P);
      s += m;
      if (use_hot && hot_bit(a.hot_bits, (uint32_t)idx)) h += m;
    });
    blk_reduce<WNW>(S, bad, none, mx, s);  // barriers inside: the parts' maxima and the tables have been read
    if (use_hot) h = blk_sum_u64<WNW>(S, h);
    if (tid < WNW) {
      part[tid].s = tid == 0 ? s : 0ull; part[tid].h = tid == 0 ? h : 0ull;
      part[tid].m = bad ? INFINITY : M;  // (a NaN: the finishing kernel hands the row on)
    }
  }
}
template <typename DT, bool use_hot, bool RUNS>  // use_hot: a hot set is installed (section 5.3): masses are split by class
__global__ __launch_bounds__(WT, WGS) void wide_classify_kernel(const SampleArgs a) {
  constexpr int EPL = Io<DT>::EPL;
  constexpr int G = ItemLoads<DT>::G;  // a slice is one tile of the draw's walk
  constexpr unsigned EMASK = (1u << EPL) - 1u;
  constexpr int LCAP = RUNS ? 768 : 2048;  // size of the stage, which is written out once fewer than ICAP places are free
  // runs: an entry per pattern of the current row; else the tables of a slice
  __shared__ __align__(16) uint32_t ptab[((RUNS ? PT_BYTES : (uint32_t)sizeof(SliceTabs)) + 15u) / 16u * 4u];
  static_assert(sizeof(SliceTabs) <= PT_BYTES, "either");
  SliceTabs& Tb = *reinterpret_cast<SliceTabs*>(ptab);
  __shared__ u64 lrl[LCAP];  // boundary columns of the current row found by this workgroup, not yet written out
  __shared__ u64 ltile[2];
  __shared__ u64 lt[2][MAX_SLICES];  // runs: the slices' masses by class
  __shared__ uint32_t odd[4];        // runs: slices with groups that go column by column
  __shared__ uint32_t hlist[HLIST];
  __shared__ unsigned l_n, l_over;
  __shared__ FS S;
  static_assert((sizeof(ptab) + sizeof(lrl) + sizeof(ltile) + (RUNS ? sizeof(lt) + sizeof(odd) + sizeof(hlist) : 0u) + 8u + sizeof(S)) * WGS <= LDS_PER_CU, "a resident round by LDS");
  const int tid = threadIdx.x, lane = tid & 63;
  const int V = a.V;
  // mask word and bit of this thread's first column in each of its groups (a group step is whole words)
  const int wbase = (tid * EPL) >> 5;
  const unsigned wsh = (unsigned)(tid * EPL) & 31u;
  static_assert((WT * EPL) % 32 == 0, "group stride in mask words");
  const uint32_t* hot_bits = a.hot_bits;
  far_rows<DT, use_hot>(Tb, S, a);
  const Items I = my_items(a);
  if (tid == 0) l_n = 0u;
  for (unsigned i0 = I.i0, i1; i0 < I.i1; i0 = i1) {  // the slices [sl0, sl1) of one row
  const unsigned slot = i0 / I.n_sl;
  i1 = min(I.i1, (slot + 1u) * I.n_sl);
  const int sl0 = (int)(i0 - slot * I.n_sl), sl1 = sl0 + (int)(i1 - i0);
  if ((uni(as_global(reinterpret_cast<const uint32_t*>(reinterpret_cast<const WideRec*>(a.wq + WQ_HEAD) + slot))[2]) & WIDE_MODE) == (uint32_t)WIDE_ALL) continue;  // (done by the bins kernel, or above)
  const WideRow W = load_row(a, slot);
  const DT* rowp = reinterpret_cast<const DT*>(a.logits) + (size_t)W.row * (size_t)a.stride;
  const RowCut rc = row_cut(S, W);  // barriers inside
  if (!rc.valid) continue;  // the finishing kernel hands the row on
  const int bstar = rc.bstar;
  const float thr_y = rc.thr_y;
  if (tid == 0) l_over = 0u;  // (a barrier follows before any column is classified)
  if (sl0 == 0 && tid == 0) {  // for the finishing kernel
    reinterpret_cast<uint32_t*>(W.ws + WS_SCAL)[8] = (uint32_t)bstar + 1u;
    reinterpret_cast<u64*>(W.ws + WS_SCAL)[5] = rc.s_tot;
  }
  const ZCut zc = z_cut(W, bstar, thr_y);
  // What a thread gathers over this workgroup's slices of one row, reduced when the row ends:
  unsigned n_sure = 0u;    // sure columns (those of the main line: counted per wave, in the lane with its first column)
  u64 acc_all = 0ull;      // exact mass of every column (routes without bins)
  float ymax = -INFINITY;  // largest tempered value
  bool bad = false;        // a mass the fixed point cannot carry, or a NaN
  // Boundary columns go to the stage, in a run by their ids (those that are boundary columns as read), else with their logits
  // (the others and what finds the stage full: straight to the row's list).
  bool ids_only = false;
  uint32_t* lid = reinterpret_cast<uint32_t*>(lrl);
  // Once the row's list is full the finishing kernel hands the row on, whatever else is counted: nothing more is collected.  (512 rows
  // of 256,000 columns around 250, steps of 1 apart: 365 us with every boundary column counted in the row's word, 136 so.)
  auto place = [&](unsigned at, u64 c) {
    if (at < (unsigned)RCAP) reinterpret_cast<u64*>(W.ws + WS_RL)[at] = c; else l_over = 1u;
  };
  auto put = [&](float z, int idx) {
    if (!l_over) place(atomicAdd(&reinterpret_cast<uint32_t*>(W.ws + WS_SCAL)[3], 1u), ((u64)__float_as_uint(z) << 32) | (u64)(uint32_t)idx);
  };
  auto stage = [&](unsigned s, u64 c) { if (s < (unsigned)LCAP) lrl[s] = c; else put(__uint_as_float((uint32_t)(c >> 32)), (int)(uint32_t)c); };
  // Writes the staged boundary columns to the row's list.  All threads call, after a barrier that
  // follows the last append; ends with a barrier.
  auto list_out = [&]() {
    const unsigned nb = min(l_n, ids_only ? 2u * (unsigned)LCAP : (unsigned)LCAP);
    if (nb == 0u) return;
    uint32_t* sc = reinterpret_cast<uint32_t*>(W.ws + WS_SCAL);
    for (unsigned t0 = 0; t0 < nb; t0 += WT) {
      const unsigned t = min(t0 + (unsigned)tid, nb - 1u);
      u64 c = 0ull;
      bool in = t0 + (unsigned)tid < nb;
      if (ids_only) {
        const uint32_t id = lid[t];
        c = ((u64)__float_as_uint(Io<DT>::one(rowp + id)) << 32) | (u64)id;
        in = in && !hist_bit(W, (int)id);  // (settled with the history's columns)
      } else c = lrl[t];
      const u64 m = __ballot(in);
      unsigned base = 0u;
      if (lane == 0 && m) base = atomicAdd(&sc[3], (unsigned)__popcll(m));
      base = uni(base) + lanes_before(m);
      if (in) place(base, c);
    }
    __syncthreads();
    if (tid == 0) l_n = 0u;
    __syncthreads();
  };
  auto leave_row = [&]() {  // barriers inside
    __syncthreads();
    list_out();
    uint32_t* sc = reinterpret_cast<uint32_t*>(W.ws + WS_SCAL);
    const float m = wave_max(ymax);
    if (lane == 0 && m > -INFINITY) atomicMax(&sc[6], fkey(m));
    if (__ballot(bad) && lane == 0) atomicAdd(&sc[3], (unsigned)RCAP + 1u);  // the finishing kernel hands the row on
    unsigned ns = n_sure, dz = 0u; u64 mx = 0ull, dsum = acc_all;
    blk_reduce<WNW>(S, ns, dz, mx, dsum);
    if (tid == 0) {
      if (ns) atomicAdd(&sc[2], ns);
      if (dsum) atomicAdd(reinterpret_cast<u64*>(W.ws + WS_SCAL + 16), dsum);
    }
  };
  u64 acc_s = 0ull, acc1 = 0ull;  // a slice's mass of the sure columns, and of the hot ones among them
  // one column the slow way: history columns and the ragged end of the row
  auto one_of = [&](float z, int idx, bool hot) {
    int b; float y;
    const float w = mass_term(z, W.C, b, y);
    const bool below = z < W.C.g;
    if (!below && !(w <= W_LIMIT)) { bad = true; return; }
    const u64 m = below ? mass_fix_below(w) : mass_fix(w);
    acc_all += m;
    ymax = fmaxf(ymax, y);
    if (!(y >= thr_y)) return;
    if (!below || b < bstar) {
      acc_s += m;
      if (use_hot && hot) acc1 += m;
      ++n_sure;
    } else if (b == bstar) { if (ids_only) put(z, idx); else stage(atomicAdd(&l_n, 1u), ((u64)__float_as_uint(z) << 32) | (u64)(uint32_t)idx); }
  };
  auto one = [&](float z, int idx) { one_of(z, idx, use_hot && hot_bit(hot_bits, (uint32_t)idx)); };
  if constexpr (RUNS) if (takes_run(W, I, sl0, sl1)) {
    // An entry is the mass of one of the pattern's columns if they surely survive and it is below 2^30 (four times the mass
    // at g), and MARKED for columns that are looked at one by one: boundary columns, and those with more mass.
    constexpr uint32_t MARKED = 0x80000000u;
    // (over: more than the fixed point carries, which the row's later kernels cannot take unless the column is the history's)
    auto clamped = [&](float z, bool& over) -> u64 {
      int b;
      const float w = mass_term(z, W.C, b);
      over = !(w <= W_LIMIT);
      return sum_to_u64(SUM_BASE + (double)mass_integer(fminf(w, W_LIMIT)));
    };
    ids_only = true;
    uint32_t odd_words = 0u;  // (lanes 0 to 3) slices with groups that go column by column
    RunLoads<DT> N;
    run_fetch<DT, use_hot>(N, a, rowp, sl0, false);
    for (int i = tid; i < 2 * MAX_SLICES; i += WT) lt[i / MAX_SLICES][i % MAX_SLICES] = 0ull;
    odd_words = as_global(reinterpret_cast<const uint32_t*>(W.ws + WS_ODD))[lane & 3];
    if (tid < 4) odd[tid] = odd_words;
#pragma unroll 1
    for (int i = tid; i < 2 * NMAG; i += WT) {
      uint32_t off;
      const float z = pattern_value(i, off);
      uint32_t e = z >= zc.z_edge ? MARKED : 0u;
      if (z >= zc.z_sure) { bool over; const u64 m = clamped(z, over); e = m >> 30 ? MARKED : (uint32_t)m; }
      ptab[off / 4u] = i == 2 * NMAG - 1 ? 0u : e;
    }
    __syncthreads();
    const bool want_n = a.diag != nullptr;  // (the number of survivors is a diagnostic here)
    // the columns of a lane's group that are looked at one by one: bit e of em, few
    auto stage_lane = [&](uint32_t em, int idx0, uint32_t hq, auto&& bits) {
#pragma unroll 1
      for (; em; em &= em - 1u) {
        const int e = __ffs((int)em) - 1;
        const uint32_t zb = bits(e);
        const float z = __uint_as_float(zb);
        if (z >= zc.z_sure) {
          bool over;
          const u64 m = clamped(z, over);
          acc_s += m;
          if (use_hot && ((hq >> e) & 1u)) acc1 += m;
          if (over && !hist_bit(W, idx0 + e)) bad = true;
        } else {
          const unsigned at = atomicAdd(&l_n, 1u);
          if (at < 2u * (unsigned)LCAP) lid[at] = (uint32_t)(idx0 + e);
          else if (!hist_bit(W, idx0 + e)) put(z, idx0 + e);
        }
      }
    };
#pragma unroll 1
    for (int sl = sl0; sl < sl1; ++sl) {
      RunLoads<DT> L = N;
      run_settle(L);
      run_fetch<DT, use_hot>(N, a, rowp, sl + 1, sl + 1 == sl1);
      acc_s = 0ull; acc1 = 0ull;
#pragma unroll
      for (int j = 0; j < G; ++j) {
        const int idx0 = sl * SLC + (j * WT + tid) * EPL;
        const uint32_t hq = use_hot ? L.hq[j] >> wsh : 0u;
        if (idx0 + EPL > V) {  // the ragged end of the row
          for (int idx = idx0; idx < V; ++idx) if (!hist_bit(W, idx)) one(Io<DT>::one(rowp + idx), idx);
        } else {
          const u32x4 w = L.A[j];
          if (!((read_lane(odd_words, sl >> 5) >> (sl & 31)) & 1u) || group_ok(w)) {
            const uint32_t w4[4] = {w.x, w.y, w.z, w.w};
            uint32_t ev[EPL], any = 0u, sum[2] = {0u, 0u}, sum_h[2] = {0u, 0u};  // (of four columns: below 2^32, and a mark is 2^31)
#pragma unroll
            for (int k = 0; k < 4; ++k) {
              const uint32_t off = pattern_offsets2(w4[k]);
              ev[2 * k] = ptab[(off & 0xFFFFu) / 4u];
              ev[2 * k + 1] = ptab[(off >> 16) / 4u];
            }
#pragma unroll
            for (int e = 0; e < EPL; ++e) {
              sum[e / 4] += ev[e];
              any |= ev[e];
              if (use_hot) sum_h[e / 4] += ev[e] & (uint32_t)__builtin_amdgcn_sbfe((int)hq, (unsigned)e, 1u);
            }
            if (want_n) {
              float z[EPL];
              Io<DT>::unpack(w, z);
#pragma unroll
              for (int e = 0; e < EPL; ++e) n_sure += z[e] >= zc.z_sure ? 1u : 0u;
            }
            if ((any & MARKED) && !l_over) {
              uint32_t em = 0u;
#pragma unroll
              for (int e = 0; e < EPL; ++e) em |= (ev[e] >> (31 - e)) & (1u << e);
#pragma unroll
              for (int k = 0; k < 2; ++k) {
                sum[k] -= (uint32_t)__popc(em & (15u << 4 * k)) << 31;
                if (use_hot) sum_h[k] -= (uint32_t)__popc(em & hq & (15u << 4 * k)) << 31;
              }
              stage_lane(em, idx0, hq, [&](int e) {
                const uint32_t x = select4(w.x, w.y, w.z, w.w, e >> 1);
                return (e & 1) ? x & 0xFFFF0000u : x << 16;
              });
            }
            acc_s += (u64)sum[0] + (u64)sum[1];
            if (use_hot) acc1 += (u64)sum_h[0] + (u64)sum_h[1];
          } else {
#pragma unroll 1
            for (int e = 0; e < EPL; ++e) if (!hist_bit(W, idx0 + e)) one(Io<DT>::one(rowp + idx0 + e), idx0 + e);
          }
        }
        __builtin_amdgcn_sched_barrier(0);  // one group at a time: interleaving them costs registers
      }
      // (four lanes add to the slice's words: less work than the rest of a reduction)
      const u64 s0 = row16_sum_u64(acc_s - acc1), s1 = use_hot ? row16_sum_u64(acc1) : 0ull;
      if ((lane & 15) == 0) {
        atomicAdd(&lt[0][sl], s0);
        if (use_hot) atomicAdd(&lt[1][sl], s1);
      }
    }
    if (W.h_active) {
      const int whole = V & ~(EPL - 1);  // (not those behind the last whole group)
      hist_run<DT, use_hot>(W, a, rowp, sl0, sl1, hlist, [&](int idx, float z, float zp, bool hot) {
        const int sl = idx / SLC;
        u64 was = 0ull;  // what it was taken for
        if (idx < whole && (!((odd[sl >> 5] >> (sl & 31)) & 1u) || group_ok(Io<DT>::load(rowp + (idx & ~(EPL - 1)))))) {
          was = (u64)ptab[pattern_offset(z) / 4u];
          if (was & (u64)MARKED) { bool over; was = z >= zc.z_sure ? clamped(z, over) : 0ull; }
          if (z >= zc.z_sure) --n_sure;
        }
        acc_s = 0ull; acc1 = 0ull;
        one_of(zp, idx, hot);
        if (acc_s != was) atomicAdd(&lt[use_hot && hot ? 1 : 0][sl], acc_s - was);
      });
    }
    __syncthreads();  // the slices' masses are complete
    for (int i = tid; i < 2 * (sl1 - sl0); i += WT) {
      const int cls = i & 1, sl = sl0 + (i >> 1);
      const u64 m = lt[cls][sl];
      reinterpret_cast<u64*>(W.ws + WS_TILES)[cls * 256 + sl] = m;
      if (m >> 55) bad = true;  // 128 tiles of two classes below 2^55 sum below 2^63; more mass in one is not carried
    }
    leave_row();
    continue;
  }
  ItemLoads<DT> N;  // the next item's loads
  item_fetch<DT, use_hot, true>(N, a, W, sl0 * SLC);
  for (int sl = sl0; sl < sl1; ++sl) {
    const int c0 = sl * SLC;
    const ItemLoads<DT> L = N;
    const bool more = sl + 1 < sl1;
    if (tid < 2) ltile[tid] = 0ull;
    if (W.h_active) slice_store(Tb, L.pre, a, c0, W.distinct);
    __syncthreads();
    HistPre<DT> HP;
    if (W.h_active) hist_fetch<DT>(HP, Tb, W.ws, a, rowp, c0, V);  // this item's own loads go first: loads return in order
    if (more && !W.f64) item_fetch<DT, use_hot, true>(N, a, W, c0 + SLC);
    acc_s = 0ull; acc1 = 0ull;
    if (W.f64) {
      weighed_columns<DT>(Tb, HP, W, a, rowp, c0, V, [&](float z, int idx, const Exp2Poly& P) {
        int b; float y;
        (void)mass_term(z, W.C, b, y);
        bad = bad || !(y <= W.M.top);  // a mass the fixed point cannot carry, or a NaN
        const u64 m = mass_fix64(y, W.M, P);
        acc_all += m;
        ymax = fmaxf(ymax, y);
        if (!(y >= thr_y)) return;
        if (!(z < W.C.g) || b < bstar) {
          acc_s += m;
          if (use_hot && hot_bit(hot_bits, (uint32_t)idx)) acc1 += m;
          ++n_sure;
        } else if (b == bstar) {
          stage(atomicAdd(&l_n, 1u), ((u64)__float_as_uint(z) << 32) | (u64)(uint32_t)idx);
        }
      });
      if (more) item_fetch<DT, use_hot, true>(N, a, W, c0 + SLC);
    } else {
    // The main line: every column's mass, and its class by the logit alone; boundary columns follow
    // under a wave-wide test.
    auto sweep = [&](auto unit_tau_c, auto want_all_c) {
      // UT: tau == 1; WANT_ALL: the row's mass is summed here (no bins)
      constexpr bool UT = decltype(unit_tau_c)::value, WANT_ALL = decltype(want_all_c)::value;
#pragma unroll
      for (int j = 0; j < G; ++j) {
        const int idx0 = c0 + (j * WT + tid) * EPL;
        if (idx0 + EPL <= V) {
          float z[EPL];
          Io<DT>::unpack(L.A[j], z);
          u64 edge[EPL], any_edge = 0ull;  // the wave's boundary columns
          unsigned ns = 0u;
          uint32_t live = ~0u;
          if (W.h_active) {  // history columns are handled below: here they carry no mass
            live = ~((Tb.bm[wbase + j * (WT * EPL / 32)] >> wsh) & EMASK);
#pragma unroll
            for (int e = 0; e < EPL; ++e) z[e] = ((live >> e) & 1u) ? z[e] : -INFINITY;
            // ... but -inf counts as sure when every value does
            if (zc.z_sure == -INFINITY) n_sure -= (unsigned)__popc(~live & EMASK);
          }
          double gs = SUM_BASE, gh = SUM_BASE, ga = SUM_BASE;  // the group's masses: <= 8 terms of <= 2^49
#pragma unroll
          for (int e = 0; e < EPL; ++e) {
            int b; float y;
            const float w = mass_term<UT>(z[e], W.C, b, y);
            bad = bad || !(w <= W_LIMIT);  // a mass the fixed point cannot carry, or a NaN
            const float q = mass_integer(w);
            ymax = fmaxf(ymax, y);
            const bool sure = z[e] >= zc.z_sure;
            const u64 ms = __ballot(sure);
            const float qs = sure ? q : 0.0f;
            gs += (double)qs;
            if (use_hot) gh += (double)hot_only(qs, L.hq[j], e);
            if (WANT_ALL) ga += (double)q;
            ns += (unsigned)__popcll(ms);  // (scalar, as the tests below are: the vector unit is what is short)
            edge[e] = __ballot(z[e] >= zc.z_edge) & ~ms;
            any_edge |= edge[e];
          }
          if (lane == 0) n_sure += ns;
          acc_s += sum_to_u64(gs);
          if (use_hot) acc1 += sum_to_u64(gh);
          if (WANT_ALL) acc_all += sum_to_u64(ga);
          // boundary columns: few per wave, an element at a time, one reservation for the wave.  (Tested and reserved
          // lane by lane: 1024 float32 rows of 128,256 columns 195.0 us a call, 192.3 so with the counts of the sure columns.)
          if (any_edge && !l_over) {
#pragma unroll
            for (int e = 0; e < EPL; ++e) {
              if (edge[e] == 0ull) continue;
              const u64 m = edge[e] & __ballot((live >> e) & 1u);
              unsigned base = 0u;
              if (lane == 0) base = atomicAdd(&l_n, (unsigned)__popcll(m));
              const unsigned s = uni(base) + lanes_before(m);
              if ((m >> lane) & 1ull) stage(s, ((u64)__float_as_uint(z[e]) << 32) | (u64)(uint32_t)(idx0 + e));
            }
          }
        } else {
          for (int idx = idx0; idx < V; ++idx)
            if (!(W.h_active && slice_bit(idx - c0, Tb))) one(Io<DT>::one(rowp + idx), idx);
        }
        __builtin_amdgcn_sched_barrier(0);  // one group at a time: interleaving them costs registers
      }
    };
    // the top-p route has the row's mass from its bins; the other routes sum it here
    const std::true_type yes{};
    const std::false_type no{};
    if (W.tau == 1.0f) {
      if (W.mode == WIDE_TOP_P || W.mode == WIDE_TOP_K) sweep(yes, no); else sweep(yes, yes);
    } else {
      if (W.mode == WIDE_TOP_P || W.mode == WIDE_TOP_K) sweep(no, no); else sweep(no, yes);
    }
    if (W.h_active) {  // the history columns, whose logits and counts were requested before the main line
      hist_stage<DT>(Tb, HP, W.ws, a, rowp, c0, V);
      __syncthreads();
      hist_columns<DT>(Tb, W, a, rowp, c0, V, one);
    }
    }
    {
      const u64 s0 = wave_sum(acc_s - acc1);
      if (lane == 0 && s0) atomicAdd(&ltile[0], s0);
      if (use_hot) { const u64 s1 = wave_sum(acc1); if (lane == 0 && s1) atomicAdd(&ltile[1], s1); }
    }
    __syncthreads();  // the tile sums and this slice's appends are complete
    if (tid < 2 && sl < 256) {
      reinterpret_cast<u64*>(W.ws + WS_TILES)[tid * 256 + sl] = ltile[tid];
      if (ltile[tid] >> 55) bad = true;  // 128 tiles of two classes below 2^55 sum below 2^63; more mass in one is not carried
    }
    if (l_n > (unsigned)(LCAP - ICAP)) list_out();
  }
  leave_row();
  }
}

// ---------------------------------------------------------------- finish ----------------------
__device__ inline void hand_on(const SampleArgs& a, int row) {
  const unsigned slot = atomicAdd(&a.pend[0], 1u);
  a.pend[2 + slot] = (uint32_t)row;
  a.out[row] = PENDING;
}

// The slice that starts at c0 in LDS: column o at slice_place(o), so that the columns a thread takes, side by side, lie in
// other banks than its neighbours'; -inf behind the row's end and, with by_class, for columns that are hot or not other than
// `cls`.  A row's history tables of the slice are left in Tb, and this thread's own columns are penalised.
// (Column by column in registers, 256 threads with every weight's code unrolled sixteen times, finding the drawn column
// took 7 us of a row's 16, much of it the code's own way from memory; 4 us so.)
constexpr int FT = 512, FNW = FT / 64;  // threads of the finishing kernel's workgroups: two waves per SIMD hide each other's latency
constexpr int EPT = SLC / FT;
__device__ __forceinline__ int slice_place(int o) { return o + o / EPT; }
static_assert(EPT == 8, "a thread's columns are a byte of a mask word, and not less than a 16-byte group's");
constexpr int SLICE_FLOATS = SLC + FT;
template <typename DT>
__device__ __forceinline__ void stage_slice(float* zt, SliceTabs& Tb, const WideRow& W, const SampleArgs& a, const DT* rowp, int c0, bool by_class, unsigned cls) {
  constexpr int EPL = Io<DT>::EPL, G = SLC / (FT * EPL);
  const int tid = fresh_tid(), V = a.V;
  const uint32_t tab = W.h_active ? slice_fetch(W.ws, a, c0) : 0u;
  typename Io<DT>::Raw r[G];
  uint32_t hq[G];
#pragma unroll
  for (int j = 0; j < G; ++j) {
    const int idx0 = c0 + (j * FT + tid) * EPL;
    r[j] = typename Io<DT>::Raw();
    hq[j] = 0u;
    if (idx0 + EPL <= V) r[j] = Io<DT>::load(rowp + idx0);
    if (by_class && idx0 < V) hq[j] = as_global(a.hot_bits)[idx0 >> 5] >> ((unsigned)idx0 & 31u);
  }
  if (W.h_active) slice_store(Tb, tab, a, c0, W.distinct);
#pragma unroll
  for (int j = 0; j < G; ++j) {
    const int o = (j * FT + tid) * EPL;
    float z[EPL];
    Io<DT>::unpack(r[j], z);
    if (c0 + o + EPL > V) {
#pragma unroll
      for (int e = 0; e < EPL; ++e) z[e] = c0 + o + e < V ? Io<DT>::one(rowp + c0 + o + e) : -INFINITY;
    }
#pragma unroll
    for (int e = 0; e < EPL; ++e) zt[slice_place(o) + e] = (by_class && ((hq[j] >> e) & 1u) != cls) ? -INFINITY : z[e];
  }
  __syncthreads();
  if (!W.h_active) return;
  slice_counts<FT>(Tb, W.ws, a);
  __syncthreads();
  for (uint32_t m = (Tb.bm[tid >> 2] >> ((tid & 3) * EPT)) & 0xFFu; m; m &= m - 1u) {
    const int o = tid * EPT + __ffs((int)m) - 1;
    zt[slice_place(o)] = slice_value(zt[slice_place(o)], o, Tb, W, a);
  }
}
// The sum of f(z, column) over this thread's columns; and, where the running sum over all threads' columns exceeds
// `at` among them, the column and its term.
template <int UNROLL_, typename F>
__device__ __forceinline__ u64 sum_columns(const float* zt, int c0, F&& f) {
  const int o0 = fresh_tid() * EPT;
  const float* p = zt + slice_place(o0);
  u64 s = 0ull;
#pragma unroll UNROLL_
  for (int e = 0; e < EPT; ++e) s += f(p[e], c0 + o0 + e);
  return s;
}
template <typename F>
__device__ __forceinline__ void find_column(FS& S, const float* zt, int c0, u64 run, u64 sum, u64 at, F&& f) {
  if (!(run <= at && at < run + sum)) return;
  const int o0 = fresh_tid() * EPT;
  const float* p = zt + slice_place(o0);
#pragma unroll 1
  for (int e = 0; e < EPT; ++e) {
    const u64 m = f(p[e], c0 + o0 + e);
    if (m > 0ull && run <= at && at < run + m) { S.out_id = c0 + o0 + e; S.out_w = m; }
    run += m;
  }
}

constexpr int NBK_BITS = 10, NBK = 1 << NBK_BITS;  // buckets of the cut bin's columns
template <typename DT>
__device__ inline bool finish_row(const SampleArgs& a, const WideRow& W, FS& S, SliceTabs& Tb, u64* rcmp, uint32_t* rl,
                                  u64* dmass, u64* tiles, simple_row_diag& dg) {
  constexpr int T = SLC;            // a tile of the draw's walk is a slice
  const int tid = threadIdx.x;
  const int V = a.V;
  const StreamCtx& C = W.C;
  const uint32_t* hot_bits = a.hot_bits;
  const bool use_hot = hot_bits != nullptr;
  const DT* rowp = reinterpret_cast<const DT*>(a.logits) + (size_t)W.row * (size_t)a.stride;
  double u3[3];
  row_uniforms(a.seed, a.row_offset + (uint64_t)W.row, a.step, u3);
  // every value of the slot this workgroup needs is requested before the first barrier
  const uint32_t* sc = reinterpret_cast<const uint32_t*>(W.ws + WS_SCAL);
  const unsigned n_sure = as_global(sc)[2], n_r = as_global(sc)[3];
  const u64 S_sum = as_global(reinterpret_cast<const u64*>(W.ws + WS_SCAL))[2];  // mass of the row, summed by the classifying pass
  static_assert(FT == 512, "a tile of one of the two classes per thread");
  const u64 tv = as_global(reinterpret_cast<const u64*>(W.ws + WS_TILES))[tid];
  const uint32_t kmax = as_global(sc)[6];
  // the cut as the classifying kernel found it
  const int bstar = (int)as_global(sc)[8] - 1;
  const u64 s_bins = as_global(reinterpret_cast<const u64*>(W.ws + WS_SCAL))[5];
  if (bstar < 0) { return false; }
  const float thr_y = W.min_p > 0.0f ? keyf(kmax) + W.ln_min_p : -INFINITY;
  const bool top_p_route = W.mode == WIDE_TOP_P, top_k_route = W.mode == WIDE_TOP_K;
  const bool cut_route = top_p_route || top_k_route;  // a cut inside a bin: by mass, or by count
  const u64 S_tot = top_p_route ? s_bins : S_sum;  // exact mass of the row (from the bins where there are bins)
  // a count past the limit is also how the classifying pass reports a row it could not handle; no
  // collected column on the top-p route means that a min-p cut ended the survivors above the bin
  const bool minp_too = top_p_route && W.min_p > 0.0f;
  if (n_r > (unsigned)RCAP || (!cut_route && n_r != 0u) || (cut_route && n_r == 0u && !minp_too)) { return false; }
  if (tid == 0) { S.bd = -1; S.cut_k = 0ull; S.cut_p = ~0ull; S.e_tfix = 0ull; S.out_id = -1; S.out_w = 0ull; }
  tiles[tid] = tv;
  u64 cut_found = 0ull;  // every collected column at or after it in the order survives; 0: no collected columns
  unsigned r_in = 0;
  if (cut_route && n_r == 0u) cut_found = ~0ull;  // nothing of the bin survives
  if (cut_route && n_r != 0u) {
  // exact masses (top-k: counts) from here: the columns surely inside must stay below the target, the
  // collected bin must reach it
  const u64 m_sure = blk_sum_u64<FNW>(S, tv);  // barriers inside
  Exp2Poly P{};  // (from memory where they are needed: as literals they took registers from end to end)
  if (W.f64) P = exp2_poly_from_memory();
  auto mass_at = [&](unsigned t) -> u64 { return W.f64 ? mass_fix64(keyf((uint32_t)(rcmp[t] >> 32)), W.M, P) : (u64)rl[t]; };
  const u64 m_above = top_k_route ? (u64)n_sure : m_sure;
  const u64 target = top_k_route ? (u64)W.top_k : (u64)__double2ull_ru((double)W.top_p * (double)S_tot);
  if (m_above >= target) { return false; }
  // -- the boundary bin, exactly: shortest prefix in the total order whose mass reaches the target --
  {
    u64 cmax_t = 0ull, cmin_t = ~0ull;
    const u64* grl = reinterpret_cast<const u64*>(W.ws + WS_RL);
    for (unsigned t0 = 0; t0 < n_r; t0 += 4u * FT) {  // four independent loads per thread and round
      u64 e[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) { const unsigned t = t0 + (unsigned)(k * FT + tid); e[k] = (t < n_r) ? as_global(grl)[t] : 0ull; }
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const unsigned t = t0 + (unsigned)(k * FT + tid);
        if (t >= n_r) continue;
        const float z = __uint_as_float((uint32_t)(e[k] >> 32));
        int b; float y;
        const float w = mass_term(z, C, b, y);
        const u64 c = composite(fkey(y), (uint32_t)e[k]);
        rcmp[t] = c;
        rl[t] = (uint32_t)mass_fix_below(w);
        cmax_t = (c > cmax_t) ? c : cmax_t; cmin_t = (c < cmin_t) ? c : cmin_t;
      }
    }
    cmax_t = wave_all(cmax_t, [](u64 x, u64 y) { return x > y ? x : y; });
    cmin_t = wave_all(cmin_t, [](u64 x, u64 y) { return x < y ? x : y; });
    if ((tid & 63) == 0) { atomicMax(&S.cut_k, cmax_t); atomicMin(&S.cut_p, cmin_t); }
  }
  __syncthreads();
  // The columns between the largest and the smallest (key, ~id) go to 1024 buckets of equal width; the
  // bucket whose mass carries the running total over the target holds the cut.  With at most a thread per
  // member it is resolved at once, else (many ties) its members are spread again.  (A radix descent by eight bits
  // took five levels of six barriers for the same; a kernel of 90 such rows 22.7 us, 17.1 so.)
  {
    u64 hi = S.cut_k, lo = S.cut_p, prefix = 0ull, acc = m_above;
    bool ok = true;
    for (;;) {
      const int sh = max(0, 64 - NBK_BITS - (int)__clzll((long long)(hi - lo)));
      for (int i = tid; i < NBK; i += FT) dmass[i] = 0ull;
      if (tid == 0) { S.bp = -1; S.memb = 0u; }
      __syncthreads();
      if (tid == 0) { S.cut_k = 0ull; S.cut_p = ~0ull; }  // (every thread has read them)
      for (unsigned t = tid; t < n_r; t += FT) {
        const u64 c = rcmp[t];
        if (c >= lo && c <= hi) atomicAdd(&dmass[(unsigned)((hi - c) >> sh)], top_k_route ? 1ull : mass_at(t));
      }
      __syncthreads();
      {
        constexpr int PT4 = NBK / FT;
        u64 mb[PT4], m = 0ull;
#pragma unroll
        for (int k = 0; k < PT4; ++k) { mb[k] = dmass[tid * PT4 + k]; m += mb[k]; }
        unsigned ce2, ct2; u64 me2, mt2;
        blk_excl_scan2<FNW>(S, 0u, m, ce2, me2, ct2, mt2);
        u64 run = acc + me2;
#pragma unroll
        for (int k = 0; k < PT4; ++k) {
          if (run < target && run + mb[k] >= target) { S.bp = tid * PT4 + k; S.mab_p = run; }
          run += mb[k];
        }
      }
      __syncthreads();
      const int d = S.bp;
      if (d < 0) { ok = false; break; }  // the collected columns do not reach the target: the passes disagree
      acc = S.mab_p;
      const u64 width = 1ull << sh;
      hi -= (u64)(unsigned)d << sh;
      if (hi - lo >= width) lo = hi - (width - 1ull);
      if (sh == 0) { prefix = hi; break; }
      u64* mc = dmass;        // its members, and their masses
      u64* mw = dmass + FT;
      u64 vmax = 0ull, vmin = ~0ull;
      for (unsigned t = tid; t < n_r; t += FT) {
        const u64 c = rcmp[t];
        if (c >= lo && c <= hi) {
          vmax = c > vmax ? c : vmax; vmin = c < vmin ? c : vmin;
          const unsigned slot = atomicAdd(&S.memb, 1u);
          if (slot < (unsigned)FT) { mc[slot] = c; mw[slot] = top_k_route ? 1ull : mass_at(t); }
        }
      }
      __syncthreads();
      const unsigned nm = S.memb;
      if (nm <= (unsigned)FT) {
        if ((unsigned)tid < nm) {
          const u64 c = mc[tid], w = mw[tid];
          unsigned above;
          const u64 G = acc + sum_where<true>(mc, mw, nm, c, above);
          if (G >= target && G - w < target) S.e_tfix = c;
        }
        __syncthreads();
        prefix = S.e_tfix;
        break;
      }
      // Ties, most often: the next buckets divide the range that the members do take (ids of one value), not all of this
      // one's.  (Dividing the whole of it took up to four rounds, 26 us of a bfloat16 row whose cut's bin held 3000 ties.)
      vmax = wave_all(vmax, [](u64 x, u64 y) { return x > y ? x : y; });
      vmin = wave_all(vmin, [](u64 x, u64 y) { return x < y ? x : y; });
      if ((tid & 63) == 0) { atomicMax(&S.cut_k, vmax); atomicMin(&S.cut_p, vmin); }
      __syncthreads();
      hi = S.cut_k; lo = S.cut_p;
    }
    // the collected columns do not reach the target: with a min-p cut those below it were never
    // collected, and the min-p prefix is the shorter one (all collected columns survive)
    if (!ok && !minp_too) { return false; }
    cut_found = ok ? prefix : 1ull;
  }
  if (cut_found == 0ull) { return false; }
  for (unsigned t = tid; t < n_r; t += FT) {
    if (rcmp[t] >= cut_found) {
      const uint32_t id = 0xFFFFFFFFu - (uint32_t)rcmp[t];
      const unsigned hot = use_hot ? hot_bit(hot_bits, id) : 0u;
      atomicAdd(&tiles[hot * 256u + id / (unsigned)T], mass_at(t));
      ++r_in;
    }
  }
  }  // a cut inside a bin
  const u64 cut_c = cut_found;
  __syncthreads();  // the tile masses are complete
  // -- masses of the classes, acceptance (section 5.3), the tile that holds the draw --
  u64 S0, S1, t0 = tid < 256 ? tiles[tid] : 0ull, t1 = tid < 256 ? tiles[256 + tid] : 0ull, e0, e1;  // a tile of each class per thread
  unsigned ns = r_in + (tid == 0 ? n_sure : 0u);
  {
    const u64 i0 = wave_incl_scan(t0), i1 = use_hot ? wave_incl_scan(t1) : 0ull;
    ns = wave_sum(ns);
    if (lane_id() == 63) { const int w = wave_id(); S.r64a[w] = i0; S.r64b[w] = i1; S.r32a[w] = ns; }
    __syncthreads();
    S0 = 0ull; S1 = 0ull; e0 = i0 - t0; e1 = i1 - t1; ns = 0u;
#pragma unroll
    for (int w = 0; w < FNW; ++w) {
      const u64 x = S.r64a[w], y = S.r64b[w];
      if (w < wave_id()) { e0 += x; e1 += y; }
      S0 += x; S1 += y; ns += S.r32a[w];
    }
  }
  if (top_k_route && ns != (unsigned)W.top_k) { return false; }  // the passes disagree
  const u64 S_K = S0 + S1;
  bool pick_hot = false;
  if (use_hot) {
    pick_hot = (S1 > 0ull) && (u3[1] * (double)S_K <= (double)S1);
    dg.alpha = (double)S1 / (double)S_K;
    dg.flags |= SIMPLE_DIAG_SHVS | (pick_hot ? SIMPLE_DIAG_ACCEPTED : 0u);
  }
  const unsigned cls = pick_hot ? 1u : 0u;
  const u64 S_cls = use_hot ? (pick_hot ? S1 : S0) : S_K;
  const double u = use_hot ? (pick_hot ? u3[0] : u3[2]) : u3[0];
  dg.n_survivors = (int)ns;
  if (a.diag) dg.s_k = (double)(top_k_route ? S_K : S_tot) / (W.f64 ? (double)(1ull << W.M.bits) : (double)MSCALE) * exp((double)(W.f64 ? W.M.y : C.y_g) - (double)keyf(kmax));
  if (S_cls == 0ull) { return false; }
  u64 tfix = (u64)__double2ull_rd(u * (double)S_cls);
  if (tfix >= S_cls) tfix = S_cls - 1ull;
  {
    const u64 m2 = pick_hot ? t1 : t0, me2 = pick_hot ? e1 : e0;
    if (m2 > 0ull && me2 <= tfix && me2 + m2 > tfix) { S.bd = tid; S.mab_d = me2; }
  }
  __syncthreads();
  const int tstar = S.bd;
  if (tstar < 0) { return false; }
  // -- the drawn id inside one tile --
  const int c0 = tstar * T;
  float* zt = reinterpret_cast<float*>(rcmp);  // (the collected columns are done with)
  stage_slice<DT>(zt, Tb, W, a, rowp, c0, use_hot, cls);
  // (straight-line, a few columns at a time: a branch per column waits for each one's arithmetic)
  auto mass = [&](float z, int idx) -> u64 {
    int b; float y;
    const float w = mass_term(z, C, b, y);
    const bool below = z < C.g;
    const bool in = (!below || b < bstar || (b == bstar && composite(fkey(y), (uint32_t)idx) >= cut_c)) && y >= thr_y;
    const u64 m = mass_fix(fminf(w, W_LIMIT));  // (the same integer as mass_fix_below for what lies below)
    return in ? m : 0ull;
  };
  Exp2Poly P{};
  if (W.f64) P = exp2_poly_from_memory();
  auto mass64 = [&](float z, int idx) -> u64 {
    int b; float y;
    (void)mass_term(z, C, b, y);
    const bool in = (!(z < C.g) || b < bstar || (b == bstar && composite(fkey(y), (uint32_t)idx) >= cut_c)) && y >= thr_y;
    return in ? mass_fix64(y, W.M, P) : 0ull;
  };
  const u64 lsum = W.f64 ? sum_columns<1>(zt, c0, mass64) : sum_columns<2>(zt, c0, mass);
  unsigned ce3, ct3; u64 me3, tot3;
  blk_excl_scan2<FNW>(S, 0u, lsum, ce3, me3, ct3, tot3);
  if (W.f64) find_column(S, zt, c0, S.mab_d + me3, lsum, tfix, mass64);
  else find_column(S, zt, c0, S.mab_d + me3, lsum, tfix, mass);
  __syncthreads();
  dg.p_chosen = (float)((double)S.out_w / (double)S_K);
  return S.out_id >= 0;
}

// A slice that stands this far above all others holds the row's whole mass; such rows are left to the general kernel.
constexpr float FAR_LIMIT = 88.0f;
// A row without truncation, from its waves' parts: acceptance (section 5.3), the slice that holds the draw, and
// that slice's columns once more.  Where the bins kernel's integers hold, the slices' masses are their sums;
// else (WIDE_FAR) they are scaled to the row maximum, and the draw's place inside its slice is a fraction of
// the slice's mass.
template <typename DT>
__device__ inline bool finish_all_row(const SampleArgs& a, const WideRow& W, FS& S, SliceTabs& Tb, float* zt, simple_row_diag& dg) {
  const int tid = threadIdx.x, V = a.V;
  const int n_sl = (V + SLC - 1) / SLC;
  static_assert(FAST_MAX_V / SLC <= FT, "a slice per thread");
  const uint32_t* hot_bits = a.hot_bits;
  const bool use_hot = hot_bits != nullptr;
  const DT* rowp = reinterpret_cast<const DT*>(a.logits) + (size_t)W.row * (size_t)a.stride;
  const AllPart* parts = reinterpret_cast<const AllPart*>(W.ws + WS_HIST);
  u64 ps[WNW], ph[WNW];
  float pm[WNW], m = LOWEST;
#pragma unroll
  for (int k = 0; k < WNW; ++k) {
    ps[k] = 0ull; ph[k] = 0ull; pm[k] = LOWEST;
    if (tid < n_sl) {
      const AllPart* q = parts + tid * WNW + k;
      ps[k] = as_global(q)->s; ph[k] = as_global(q)->h; pm[k] = as_global(q)->m;
    }
  }
  double u3[3];
  row_uniforms(a.seed, a.row_offset + (uint64_t)W.row, a.step, u3);
  if (tid == 0) { S.bd = -1; S.out_id = -1; S.out_w = 0ull; S.flags = 0u; }
#pragma unroll
  for (int k = 0; k < WNW; ++k) m = fmaxf(m, pm[k]);
  {
    const float wm = wave_max(m);
    if ((tid & 63) == 0) S.wmax[tid >> 6] = wm;
  }
  __syncthreads();
  float y_max = S.wmax[0];
  const bool rel = W.far;
#pragma unroll
  for (int w = 1; w < FNW; ++w) y_max = fmaxf(y_max, S.wmax[w]);
  if (!(y_max > LOWEST) || y_max == INFINITY) return false;
  u64 m_all = 0ull, m_hot = 0ull;
  bool lost = false;
  if (!rel) {
#pragma unroll
    for (int k = 0; k < WNW; ++k) { m_all += ps[k]; m_hot += ph[k]; }
    lost = (m_all >> 56) != 0ull;  // 128 slices below 2^56 sum below 2^63
  } else {
    const double f = tid < n_sl ? exp((double)m - (double)y_max) : 0.0;
    m_all = (u64)__double2ull_rn((double)ps[0] * f); m_hot = min(m_all, (u64)__double2ull_rn((double)ph[0] * f));
  }
  if (lost) atomicOr(&S.flags, 1u);
  unsigned near = (tid < n_sl && m >= y_max - FAR_LIMIT) ? 1u : 0u, finite = (tid < n_sl && m > LOWEST) ? 1u : 0u;
  u64 S_K = m_all, mx = 0ull;
  blk_reduce<FNW>(S, near, finite, mx, S_K);  // barriers inside
  const u64 S_H = use_hot ? blk_sum_u64<FNW>(S, m_hot) : 0ull;
  if (S.flags || (rel && near == 1u && finite > 1u)) return false;
  bool pick_hot = false;
  if (use_hot) {
    pick_hot = (S_H > 0ull) && (u3[1] * (double)S_K <= (double)S_H);
    dg.alpha = (double)S_H / (double)S_K;
    dg.flags |= SIMPLE_DIAG_SHVS | (pick_hot ? SIMPLE_DIAG_ACCEPTED : 0u);
  }
  const u64 S_cls = use_hot ? (pick_hot ? S_H : S_K - S_H) : S_K;
  const double u = use_hot ? (pick_hot ? u3[0] : u3[2]) : u3[0];
  if (S_cls == 0ull) return false;
  u64 tfix = (u64)__double2ull_rd(u * (double)S_cls);
  if (tfix >= S_cls) tfix = S_cls - 1ull;
  {
    const u64 mc = use_hot ? (pick_hot ? m_hot : m_all - m_hot) : m_all;
    unsigned ce, ct; u64 me, mt;
    blk_excl_scan2<FNW>(S, 0u, mc, ce, me, ct, mt);
    if (mc > 0ull && me <= tfix && tfix < me + mc) { S.bd = tid; S.mab_d = tfix - me; S.mab_k = mc; S.wmax[15] = m; }
  }
  __syncthreads();
  const int t = S.bd;
  if (t < 0) return false;
  // the columns' masses in the slice, in ascending id
  const int c0 = t * SLC;
  const float y_ref = rel ? S.wmax[15] : W.C.y_g;
  u64 rq = S.mab_d;
  const double place = (double)S.mab_d / (double)S.mab_k;
  stage_slice<DT>(zt, Tb, W, a, rowp, c0, use_hot, pick_hot ? 1u : 0u);
  auto mass = [&](float z, int) -> u64 { return float_to_u64(mass_rel(tempered(z, W.C), y_ref) * MSCALE); };
  Exp2Poly P{};
  if (rel) P = exp2_poly_from_memory();
  auto mass64 = [&](float z, int) -> u64 { return exp_fix<44>(tempered(z, W.C), y_ref, P); };
  const u64 lsum = rel ? sum_columns<1>(zt, c0, mass64) : sum_columns<2>(zt, c0, mass);
  unsigned ce, ct; u64 me, Q;
  blk_excl_scan2<FNW>(S, 0u, lsum, ce, me, ct, Q);
  if (rel) {
    rq = (u64)__double2ull_rd(place * (double)Q);
    if (Q > 0ull && rq >= Q) rq = Q - 1ull;
  }
  if (rel) find_column(S, zt, c0, me, lsum, rq, mass64);
  else find_column(S, zt, c0, me, lsum, rq, mass);
  __syncthreads();
  dg.n_survivors = V;
  if (a.diag) dg.s_k = rel ? (double)S_K / WSCALE : (double)S_K / (double)MSCALE * exp((double)W.C.y_g - (double)y_max);
  dg.p_chosen = (float)((double)S.out_w * (rel ? exp((double)y_ref - (double)y_max) : 1.0) / (double)S_K);
  return S.out_id >= 0;
}

template <typename DT>
__global__ __launch_bounds__(FT, 4) void wide_finish_kernel(const SampleArgs a) {
  __shared__ SliceTabs Tb;
  __shared__ u64 rcmp[RCAP];
  static_assert(SLICE_FLOATS * 4 <= RCAP * 8, "a slice takes the collected columns' place");
  __shared__ uint32_t rl[RCAP];
  __shared__ u64 dmass[NBK];
  __shared__ u64 tiles[512];
  __shared__ FS S;
  const int tid = threadIdx.x;
  const unsigned n_wide = min(as_global(a.wq)[0], (unsigned)a.wide_slots);
  for (unsigned slot = blockIdx.x; slot < n_wide; slot += gridDim.x) {
    __syncthreads();
    const WideRow W = load_row(a, slot);
    simple_row_diag dg;
    dg.alpha = __longlong_as_double(0x7FF8000000000000ll);
    dg.s_k = 0.0; dg.p_chosen = 0.0f; dg.n_survivors = 0; dg.reserved = 0u;
    dg.flags = SIMPLE_DIAG_WIDE | W.flags;
    if (a.hot_bits && a.hot_flags && *a.hot_flags) dg.flags |= SIMPLE_DIAG_BAD_HOT_SET;
    const bool ok = W.mode == WIDE_ALL ? finish_all_row<DT>(a, W, S, Tb, reinterpret_cast<float*>(rcmp), dg) : finish_row<DT>(a, W, S, Tb, rcmp, rl, dmass, tiles, dg);
    if (tid == 0) {
      if (!ok) hand_on(a, W.row);
      else {
        a.out[W.row] = S.out_id;
        if (a.diag) a.diag[W.row] = dg;
        if (a.stats) stats_add(a.stats, dg.flags, dg.alpha);
        write_decision(a, W.row, S.out_id, dg.p_chosen, false);
      }
    }
  }
}

}  // namespace fast


// One resident round of workgroups each, as many per compute unit as fit by registers and LDS; a workgroup then takes a contiguous
// range of slices, mostly of one row.
template <typename DT, bool use_hot, bool RUNS>
static void launch_slices(const SampleArgs& a, hipStream_t st) {
  const dim3 blk(fast::WT);
  hipLaunchKernelGGL((fast::wide_bins_kernel<DT, use_hot, RUNS>), dim3((unsigned)(a.n_cu * fast::bins_wgs<DT, RUNS>())), blk, 0, st, a);
  hipLaunchKernelGGL((fast::wide_classify_kernel<DT, use_hot, RUNS>), dim3((unsigned)(a.n_cu * fast::WGS)), blk, 0, st, a);
}
hipError_t launch_wide(const SampleArgs& a, int dtype, hipStream_t st) {
  // The finishing kernel, two workgroups per compute unit by its LDS, takes a row at a time.
  const dim3 fin((unsigned)(a.B < 2 * a.n_cu ? a.B : 2 * a.n_cu)), fblk(fast::FT);
  if (dtype == SIMPLE_F32) {
    if (a.hot_bits) launch_slices<float, true, false>(a, st); else launch_slices<float, false, false>(a, st);
    hipLaunchKernelGGL((fast::wide_finish_kernel<float>), fin, fblk, 0, st, a);
  } else {
    // whether a workgroup can come by enough slices of a row for a run, were every row queued
    const int64_t n_sl = (a.V + fast::SLC - 1) / fast::SLC, wgs = (int64_t)a.n_cu * fast::WGS;
    const bool runs = !a.f64 && (a.B * n_sl + wgs - 1) / wgs >= fast::RUN_MIN;
    if (a.hot_bits) { if (runs) launch_slices<uint16_t, true, true>(a, st); else launch_slices<uint16_t, true, false>(a, st); }
    else { if (runs) launch_slices<uint16_t, false, true>(a, st); else launch_slices<uint16_t, false, false>(a, st); }
    hipLaunchKernelGGL((fast::wide_finish_kernel<uint16_t>), fin, fblk, 0, st, a);
  }
  return hipGetLastError();
}

}  // namespace simple
