// Single-pass row kernel for gfx950: one workgroup per logits row, every logit read from HBM once.
//
// A row needs little LDS (one region is shared in time between the history tables and the
// candidate list), so four row workgroups fit a compute unit and their latency-bound phases
// overlap with the streaming of the others.
//
//   history   the row's token history becomes, in LDS, a presence bit per column, a 16-bit count
//             of set bits before each pair of mask words and 16-bit generated-token counts indexed
//             by the rank of the id among the set bits.  The V-wide histograms of section 2.2 are
//             never materialised; a column's penalty is looked up only where its bit is set, so
//             unpenalised columns are never touched (column-wise penalties, section 5.2).
//   sample    every wave's first tiles (history columns masked) give, by counts in equal steps or, where the row's
//             masses are relative to it, by wave-ballot bisection, a value g that is expected to admit a small
//             multiple of the requested prefix length, wherever in the row its large logits lie.
//   stream    one coalesced pass of 16-byte loads per lane over the raw logits.  Columns with
//             z >= g go to an LDS candidate list that now occupies the history's region (penalties
//             that only lower a logit keep z >= z', so nothing with z' >= g is missed); rows whose
//             nucleus is taken over the whole vocabulary also accumulate exp((z - g) / tau) below g.
//   epilogue  the list moves to registers and the listed columns are penalised, by a hash table of the
//             list that the history looks up, or (rows that need the mass below g) by the history tables,
//             rebuilt in the region; the mass below g is corrected, exactly, for the
//             history columns.  The list then certifies itself: every column whose tempered value
//             exceeds fl(g / tau) is in it, so any prefix of the total order (value descending, id
//             ascending) that ends above that value is known exactly (truncation first, section
//             5.2).  Top-k, top-p and min-p cuts, the survivors' mass and the inverse-CDF draw
//             (Eq. (2), step (3)) use integer (fixed-point) masses, so no result depends on the
//             order in which waves appended candidates.  SHVS (section 5.3): acceptance test on the
//             hot mass, then the draw walks the hot or the tail survivors only.
// A row whose nucleus over the whole vocabulary is wider than the list is queued, with its threshold
// and its history tables, for the sliced kernels that run next on the stream.  Rows the kernel
// cannot certify (threshold missed, list overflow, ties wider than a table, penalties that raise
// logits, parameter errors) are queued for the general kernel, which runs last.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "simple_rowdev.hpp"

namespace simple {
namespace fast {



// A key t with need <= #{keys >= t} among the 64 x N keys held by a wave (N per lane), found by
// bisection between lo and hi with wave ballots; no LDS, no barrier.  Stops as soon as the count is
// within need + slack, else converges to the need-th largest key.  Requires #{keys >= lo} >= need
// and hi >= every key; returns lo unchanged if the interval is empty.
template <int N>
__device__ __forceinline__ uint32_t wave_threshold(const uint32_t (&k)[N], unsigned need, unsigned slack, uint32_t lo, uint32_t hi) {
#pragma unroll 1
  for (int it = 0; it < 34 && lo < hi; ++it) {
    const uint32_t mid = lo + ((hi - lo + 1u) >> 1);
    unsigned c = 0;
#pragma unroll
    for (int j = 0; j < N; ++j) c += (unsigned)__popcll(__ballot(k[j] >= mid));
    if (c >= need) { lo = mid; if (c <= need + slack) break; } else hi = mid - 1u;
  }
  return lo;
}

// Fixed-point weight exp(y - y_max) * 2^44 (stable softmax numerator, section 2.1 Eq. (2)); the sums are
// exact integers.  In double precision, as the general kernel weighs a row: with a float32 exponential
// p~ was up to 4e-7 off, here it is the float32 nearest to the exact one.
__device__ __forceinline__ u64 wfix(uint32_t key, float y_max) { return exp_fix<44>(keyf(key), y_max); }

// Unpacks one 16-byte group of a sample tile; columns that are in the history are masked out, so
// the threshold comes from unpenalised columns only (history columns can only add to the prefix).
template <typename DT>
__device__ __forceinline__ void sample_group(const typename Io<DT>::Raw& A, int idx0, const Hist& H, float (&z)[Io<DT>::EPL]) {
  constexpr int EPL = Io<DT>::EPL;
  Io<DT>::unpack(A, z);
  if (H.active) {
    const uint32_t nib = H.bm[idx0 >> 5] >> ((unsigned)idx0 & 31u);
#pragma unroll
    for (int e = 0; e < EPL; ++e) {  // (a column's bit, spread over a word, selects -inf: two instructions)
      const uint32_t m = (uint32_t)__builtin_amdgcn_sbfe((int)nib, (unsigned)e, 1u);
      z[e] = __uint_as_float((m & 0xFF800000u) | (~m & __float_as_uint(z[e])));
    }
  }
}

// ---- the threshold of a row whose result does not depend on it (greedy rows, top-k rows) ----
// From counts of the largest value of every lane in each of its wave's two tiles, whichever of two ranks is reached first:
//   the k-th of them all: what lies there is certified, so the list holds k columns wherever in the row they stand;
//   a rank that a sample of independent columns would give, counted over groups of lanes, of which each counts once: columns of
//   one place (ids in order of frequency, a run of allowed ids) cannot fill it, however many they are.
// (With the second rank alone, over the three largest values of every lane in one tile, the first tile of a vocabulary in
// order of frequency filled it, the list held fewer than k columns and the general kernel took the row: 256 float32 rows
// of 128,256 columns, top-k 50, 161.7 us a call, 41.9 so; 53.8 with the search by ballots.  Both ranks and both tiles cost
// 0.8 us where every compute unit has a row, 256 bfloat16 rows of 151,936 columns 40.3 -> 41.1.)
// Equal steps between the largest and the smallest value; a step that holds too many is divided again, in the order of the
// keys, as is a range too wide for equal steps of the value (columns masked with the lowest finite value: divided by value, its
// upper step held every real logit, and 191 to 270 of 270 such rows went to the general kernel).
// (A bisection by ballots in every wave and one over all that they kept, 16 waves on one scalar unit: 8 us
// of a row of 151,936 bfloat16 columns.)
struct SampleRanks {
  unsigned lanes, groups;  // the two ranks
  int shift;               // lanes of a group, as a power of two; -1: a lane's two tiles are two groups
  bool ok;                 // groups enough for the second one
};
// r: the rank of a sample of independent columns (see below), n_waves waves of it.  A wave's groups are about as many as
// the keys it would hand over to a search by ballots, r / n_waves and three deviations, but not half of r, and in all
// not fewer than 3/2 r.  r columns then lie in G (1 - exp(-x)) of the G groups, x = r / G, with a deviation of
// sqrt(G exp(-x) (1 - (1 + x) exp(-x))); with one of them more a list that holds fewer than k columns is as unlikely as
// with r itself (5 10^-6 and less by the exact sums; without it up to 7 10^-5).
__device__ __forceinline__ SampleRanks sample_ranks(unsigned k, unsigned r, int n_waves) {
  const float r_w = (float)r / (float)n_waves, q = r_w + 3.0f * __builtin_amdgcn_sqrtf(r_w) + 2.0f;
  int c = 4, bits = 2;
#pragma unroll
  for (int i = 0; i < 5; ++i) {
    const bool more = ((float)c * 1.1f <= q && 4u * (unsigned)c <= r) || 2u * (unsigned)(c * n_waves) < 3u * r;
    c += more ? c : 0; bits += more ? 1 : 0;
  }
  const float G = (float)(c * n_waves);
  SampleRanks R;  // (of the row, not of a lane)
  R.ok = 2u * (unsigned)(c * n_waves) >= 3u * r;
  R.lanes = (unsigned)__builtin_amdgcn_readfirstlane((int)k);
  const float x = (float)r * __builtin_amdgcn_rcpf(G), ex = __expf(-x);
  const float n = G * (1.0f - ex) + __builtin_amdgcn_sqrtf(G * ex * (1.0f - (1.0f + x) * ex));
  R.groups = (unsigned)__builtin_amdgcn_readfirstlane((int)ceilf(n));
  R.shift = __builtin_amdgcn_readfirstlane(6 - bits);
  return R;
}
constexpr int QUICK_BITS = 9, QUICK_NB = 1 << QUICK_BITS;
static_assert(QUICK_NB == (int)SAMPLE_COUNTS, "the counters' room");
constexpr float QUICK_SPAN = 64.0f;  // steps of at most an eighth; key steps end a search after four rounds whatever the values
constexpr int QUICK_FINE = 14;       // key steps of this many bits are a 512th of their value: wider ones are divided again
// mA, mB: the lane's largest unpenalised value in each tile (-inf: none); fin: its wave's finite columns among those that
// begin a 16-byte load.  `counts` (LDS) holds QUICK_NB zeros, the list `cap` columns.  Sets complete where the list may take
// every finite column.  The result is the same in every lane; barriers inside.
template <int NTHR, int EPL>
__device__ __forceinline__ float quick_threshold(FS& S, float mA, float mB, unsigned fin, SampleRanks R, int V, unsigned cap, uint32_t* counts, bool& complete) {
  constexpr int NWV = NTHR / 64, PER_LANE = EPL * UNR;
  constexpr float SAMPLE = (float)(NTHR * PER_LANE * 2);
  const int lane = lane_id(), wave = wave_id();
  const int gs = R.shift;
  const bool apart = gs < 0;
  float mG = fmaxf(mA, mB);  // the largest of the lane's group
  if (gs > 0) mG = fmaxf(mG, dpp_move<DPP_XOR1, 0xF>(mG, mG));
  if (gs > 1) mG = fmaxf(mG, dpp_move<DPP_XOR2, 0xF>(mG, mG));
  if (gs > 2) mG = fmaxf(mG, dpp_move<DPP_HALF_MIRROR, 0xF>(mG, mG));
  if (gs > 3) mG = fmaxf(mG, dpp_move<DPP_MIRROR, 0xF>(mG, mG));
  bool inA = mA > -INFINITY, inB = mB > -INFINITY;
  bool inG = !apart && mG > -INFINITY && (lane & ((1 << max(gs, 0)) - 1)) == 0;  // (counted by its first lane)
  {
    const unsigned every = (unsigned)(__popcll(__ballot(inA)) + __popcll(__ballot(inB)));
    const unsigned groups = apart ? every : (unsigned)__popcll(__ballot(inG));
    const float top = wave_max(fmaxf(mA, mB)), low = -wave_max(-fminf(inA ? mA : INFINITY, inB ? mB : INFINITY));
    if (lane == 0) { S.wmax[wave] = top; S.r32a[wave] = __float_as_uint(low); S.r32b[wave] = fin; S.wcnt[wave] = every | groups << 16; }
  }
  __syncthreads();
  float hi = -INFINITY, lo = INFINITY;
  unsigned total = 0u;
#pragma unroll
  for (int w = 0; w < NWV; ++w) { hi = fmaxf(hi, S.wmax[w]); lo = fminf(lo, __uint_as_float(S.r32a[w])); total += S.wcnt[w]; }
  hi = __uint_as_float((uint32_t)__builtin_amdgcn_readfirstlane((int)__float_as_uint(hi)));
  lo = __uint_as_float((uint32_t)__builtin_amdgcn_readfirstlane((int)__float_as_uint(lo)));
  total = (unsigned)__builtin_amdgcn_readfirstlane((int)total);
  unsigned need = R.lanes;
  const unsigned need_g = R.groups;
  auto reached = [&](unsigned n) { return (n & 0xFFFFu) >= need || (n >> 16) >= need_g; };
  if (!reached(total)) {
    // Few finite columns in the sample.  The list takes all there are, if they fit by the sample's share of them or,
    // should they be neighbours, a run of them that fits touches no more waves' tiles; else a share of them that
    // leaves between k and `cap` whether they number what was seen or what that stands for.
    unsigned finite = 0u, waves = 0u;
    {
      const unsigned f = lane < NWV ? S.r32b[lane] : 0u;
      finite = wave_sum(f); waves = (unsigned)__popcll(__ballot(f != 0u));
    }
    const float k = (float)need, seen = (float)finite * (float)EPL, ratio = (float)V / SAMPLE;
    const float share = 1.8f * k / seen;
    const bool between = 1.8f * k * ratio <= (float)cap && share * (float)PER_LANE <= 4.5f;  // (what a lane's largest value resolves)
    complete = ((float)finite + 3.0f * sqrtf((float)finite) + 4.0f) * (float)EPL * ratio <= (float)cap ||
               (!between && ((float)waves - 1.0f) * (float)V <= ((float)cap + 2.0f * (float)(64 * PER_LANE)) * (float)NWV);
    complete = __builtin_amdgcn_readfirstlane(complete ? 1 : 0) != 0;
    if (complete) return LOWEST;
    const float x = (float)PER_LANE * (between ? share : 2.0f * k / (seen * ratio));
    need = max(1u, (unsigned)ceilf((float)(total & 0xFFFFu) * (1.0f - __expf(-x))));
    need = (unsigned)__builtin_amdgcn_readfirstlane((int)need);
  }
  unsigned acc = 0u;  // values above those that are still in question; groups from bit 16
  bool by_key = !(hi - lo <= QUICK_SPAN);
  uint32_t khi = fkey(hi), klo = fkey(lo);
#pragma unroll 1
  for (;;) {
    const float scale = (float)QUICK_NB / fmaxf(hi - lo, 1e-30f);
    const int sh = max(0, 32 - QUICK_BITS - (int)__clz((int)(khi - klo)));
    auto step_of = [&](float v) -> int {  // (monotone in the value; what rounding puts beyond an end belongs to its step)
      return by_key ? (int)((khi - min(max(fkey(v), klo), khi)) >> sh) : (int)fminf((hi - v) * scale, (float)(QUICK_NB - 1));
    };
    const int sA = step_of(mA), sB = step_of(mB), sG = step_of(mG);
    const unsigned one = apart ? 0x10001u : 1u;
    if (inA) atomicAdd(&counts[sA], one);
    if (inB) atomicAdd(&counts[sB], one);
    if (inG) atomicAdd(&counts[sG], 0x10000u);
    __syncthreads();
    if (wave == 0) {
      constexpr int PL = QUICK_NB / 64;
      unsigned c[PL], loc = 0u;
#pragma unroll
      for (int j = 0; j < PL; ++j) { c[j] = counts[lane * PL + j]; counts[lane * PL + j] = 0u; loc += c[j]; }
      unsigned run = acc + wave_incl_scan(loc) - loc;
#pragma unroll
      for (int j = 0; j < PL; ++j) {
        if (!reached(run) && reached(run + c[j])) { S.q_step = lane * PL + j; S.q_before = run; S.q_through = run + c[j]; }
        run += c[j];
      }
    }
    __syncthreads();
    const int b = __builtin_amdgcn_readfirstlane(S.q_step);
    const unsigned through = (unsigned)__builtin_amdgcn_readfirstlane((int)S.q_through);
    auto close = [](unsigned n, unsigned want) { return n >= want && n <= want + want / 4u + 4u; };
    const bool fine = close(through & 0xFFFFu, need) || close(through >> 16, need_g);
    // a little lower than the step's end, so that values there are certified
    if (!by_key) {
      const float step = (hi - lo) * (1.0f / (float)QUICK_NB);
      float low = b == QUICK_NB - 1 ? lo : hi - (float)(b + 1) * step;
      low = low - 0.05f * step - fabsf(low) * 1e-6f - 1e-30f;
      if (fine) return fmaxf(low, LOWEST);
      klo = fkey(low);
      khi = max(fkey(hi - (float)b * step), klo);
      by_key = true;
    } else {
      khi -= (uint32_t)b << sh;
      if (khi - klo >= (1u << sh)) klo = khi - ((1u << sh) - 1u);
      const float low = keyf(klo);
      if ((fine && sh <= QUICK_FINE) || sh == 0) return fmaxf(low - fabsf(low) * 1e-6f - 1e-30f, LOWEST);
    }
    acc = (unsigned)__builtin_amdgcn_readfirstlane((int)S.q_before);
    inA = inA && sA == b; inB = inB && sB == b; inG = inG && sG == b;
  }
}

// Appends the flagged elements of one 16-byte group per lane with a single list reservation.
// m[e]: the wave's ballot of "element e is at or above g".
template <int EPL>
__device__ __forceinline__ void append_group(FS& S, uint32_t* lz, uint32_t* li, unsigned cap, const float (&z)[EPL], float g,
                                             const u64 (&m)[EPL], int idx0) {
  const int lane = lane_id();
  unsigned pre[EPL], tot = 0;
#pragma unroll
  for (int e = 0; e < EPL; ++e) { pre[e] = tot; tot += (unsigned)__popcll(m[e]); }
  unsigned base = 0;
  if (lane == 0) base = atomicAdd(&S.cand_count, tot);
  base = __builtin_amdgcn_readfirstlane(base);
#pragma unroll
  for (int e = 0; e < EPL; ++e) {
    if (!(z[e] < g)) {  // the lanes of m[e]
      const unsigned slot = base + pre[e] + lanes_before(m[e]);
      if (slot < cap) { lz[slot] = __float_as_uint(z[e]); li[slot] = (uint32_t)(idx0 + e); }
    }
  }
}

// One tile of the stream: raw logits against g; rows that need it also sum the mass below g (per lane).
template <typename DT>
__device__ __forceinline__ void stream_tile(const typename Io<DT>::Raw (&A)[UNR], int tb, const StreamCtx& C,
                                            FS& S, uint32_t* lz, uint32_t* li, unsigned cap, u64& below_mass) {
  constexpr int EPL = Io<DT>::EPL;
  const int lane = lane_id();
#pragma unroll
  for (int u = 0; u < UNR; ++u) {
    float z[EPL];
    Io<DT>::unpack(A[u], z);
    const int idx0 = tb + u * 64 * EPL + lane * EPL;
    if (C.need_sum) {
      uint32_t grp = 0u;  // straight-line: a column at or above g adds 2^28 (taken off after the stream); <= 8 terms
#pragma unroll
      for (int e = 0; e < EPL; ++e) grp += below_term_clamped(z[e], C);
      below_mass += (u64)grp;
    }
    u64 m[EPL], any = 0ull;  // one compare per element, straight into the wave's mask; the rest is scalar
#pragma unroll
    for (int e = 0; e < EPL; ++e) { m[e] = __ballot(!(z[e] < C.g)); any |= m[e]; }
    if (any) append_group<EPL>(S, lz, li, cap, z, C.g, m, idx0);
  }
}

// ---------------------------------------------------------------- epilogue --------------------
constexpr unsigned SHORT_WAVE = 1u << 16;  // mark beside a wave's sample count: fewer finite columns than asked for
enum { FIN_DONE = 0, FIN_PENDING = 1, FIN_WIDE = 2 };

// Mass of the top-k prefix when top-k is off: the whole row (list, uncertified entries, below g).
__device__ __forceinline__ u64 whole_row_mass(u64 total_m, unsigned n_unc, uint32_t key_g, float y_max, float g, float tau,
                                              double S_below) {
  (void)g; (void)tau;
  const double f0 = exp((double)keyf(key_g) - (double)y_max);  // S_below is relative to the mass at y_g
  return total_m + (u64)n_unc * wfix(key_g, y_max) + (u64)__double2ull_rn(S_below * f0 * WSCALE);
}

// ---- the certified entries in the total order ----
// What follows needs them sorted (value descending, id ascending), and only as many as the survivors can be: with
// top-k the first k.  Short lists are ranked by counting, longer ones go to buckets linear in the tempered value and are
// ranked among their bucket's members.  No place depends on the order in which the waves appended, but for entries so far below
// the maximum that they have no mass: those share the last bucket as they come, behind all others, where they add to no sum and
// are never drawn.  A sorted entry is its weight and its id in one word.  Bound: the latency of LDS and barriers, so their number is what was cut down: with the
// longer lists in bucket tables of masses and counts and the others' decisions on eight entries per lane, 4 float32 rows of
// 1024 columns (top-k 50, top-p) took 22.8 us a call, 17.3 so; 4096 bfloat16 rows of 256,000 1011 and 973.
constexpr int COUNT_MAX = 128;   // entries ranked by counting (several threads share an entry's comparisons)
constexpr int SORT_BITS = 10, SORT_NB = 1 << SORT_BITS;  // buckets
constexpr int SORT_MAX = 2048;   // entries that are sorted
constexpr int SORT_CROWD = 512;  // members of a bucket that are ranked by counting; a list with more (ties) is left to finalize_long
constexpr float MASS_SPAN = 44.0f;  // this far below the maximum an entry has no mass (exp_fix): its place does not matter
constexpr uint32_t SORT_OUT = SORT_MAX * 8, SORT_BASE = 2 * SORT_MAX * 8, SORT_END = SORT_BASE + SORT_NB * 4;  // offsets in the shared region
static_assert(SORT_END <= FAST_REGION_MIN, "the epilogue's arrays fit the smallest region");
static_assert(COUNT_MAX <= SORT_MAX && NBF * 16 + MEMB2 * 12 <= SORT_MAX * 8, "and so do those that take the unsorted entries' place");
constexpr int ID_BITS = 19;
static_assert(FAST_MAX_V <= (1 << ID_BITS) && 44 + 1 + ID_BITS <= 64, "a weight of up to 2^44 and an id in one word");
__device__ __forceinline__ u64 pack_entry(u64 c, float y_max) {  // from the composite of a key and an id
  return (wfix((uint32_t)(c >> 32), y_max) << ID_BITS) | (u64)(0xFFFFFFFFu - (uint32_t)c);
}
__device__ __forceinline__ u64 entry_mass(u64 e) { return e >> ID_BITS; }
__device__ __forceinline__ uint32_t entry_id(u64 e) { return (uint32_t)e & ((1u << ID_BITS) - 1u); }

// n composites at the start of the region to sorted entries at SORT_OUT: an entry's place is the number of entries before
// it, counted by 16, 4 or 2 neighbouring lanes.  S.memb, zero on entry, receives the number of those at or above key_thr.
template <int NTHR>
__device__ __forceinline__ void sort_by_counting(FS& S, unsigned n, float y_max, uint32_t key_thr, unsigned char* region) {
  static_assert(2 * COUNT_MAX <= NTHR, "two threads per entry at least");
  const u64* mc = reinterpret_cast<const u64*>(region);
  const unsigned tid = threadIdx.x;
  const unsigned sh = n * 16u <= (unsigned)NTHR ? 4u : n * 4u <= (unsigned)NTHR ? 2u : 1u, P = 1u << sh;
  if ((tid & ~63u) >> sh >= n) return;  // (whole waves)
  const unsigned e = tid >> sh;
  const u64 c = e < n ? mc[e] : 0ull;
  unsigned r = 0u;
#pragma unroll 4
  for (unsigned q = tid & (P - 1u); q < n; q += P) r += mc[q] > c ? 1u : 0u;
  r += dpp_move<DPP_XOR1, 0xF>(0u, r);
  if (sh > 1u) r += dpp_move<DPP_XOR2, 0xF>(0u, r);
  if (sh > 2u) { r += dpp_move<DPP_HALF_MIRROR, 0xF>(0u, r); r += dpp_move<DPP_MIRROR, 0xF>(0u, r); }
  const bool first = e < n && (tid & (P - 1u)) == 0u;
  const u64 m = __ballot(first && (uint32_t)(c >> 32) >= key_thr);
  if (lane_id() == 0 && m) atomicAdd(&S.memb, (unsigned)__popcll(m));
  if (first) reinterpret_cast<u64*>(region + SORT_OUT)[r] = pack_entry(c, y_max);
}

// The same from this thread's entries (key 0: none), n_all in all threads; with top-k only the buckets down to the one that
// holds the k-th.  S.memb, zero on entry, receives the number of sorted entries at or above key_thr.  Returns the number of
// sorted entries, or 0 if they are too many or too crowded.  The counters at SORT_BASE are zero.  Barriers inside.
template <int NTHR, int PER>
__device__ __forceinline__ unsigned sort_by_buckets(FS& S, const RowCfg& R, const uint32_t (&key)[PER], const uint32_t (&eid)[PER], unsigned n_all,
                                                    float y_max, uint32_t key_lo, uint32_t key_thr, unsigned char* region) {
  constexpr int NWV = NTHR / 64, BPT = SORT_NB / NTHR;
  const int tid = threadIdx.x;
  u64* sc = reinterpret_cast<u64*>(region);
  uint32_t* base = reinterpret_cast<uint32_t*>(region + SORT_BASE);
  const float span = y_max - keyf(key_lo);
  const bool zero_tail = span > MASS_SPAN;  // the last bucket holds all entries without mass
  const float scale = (float)(zero_tail ? SORT_NB - 1 : SORT_NB) / fmaxf(zero_tail ? MASS_SPAN : span, 1e-30f);
  auto bucket_of = [&](uint32_t k) { return (int)fminf((y_max - keyf(k)) * scale, (float)(SORT_NB - 1)); };
#pragma unroll
  for (int j = 0; j < PER; ++j) {
    if (key[j]) atomicAdd(&base[bucket_of(key[j])], 1u);
    __builtin_amdgcn_sched_barrier(0);
  }
  __syncthreads();
  unsigned c[BPT], loc = 0u;
#pragma unroll
  for (int j = 0; j < BPT; ++j) { c[j] = base[tid * BPT + j]; loc += c[j]; }
  const unsigned incl = wave_incl_scan(loc);
  if (lane_id() == 63) S.r32a[wave_id()] = incl;
  __syncthreads();
  unsigned run = incl - loc;
#pragma unroll
  for (int w = 0; w < NWV; ++w) { const unsigned x = S.r32a[w]; if (w < wave_id()) run += x; }
  const unsigned want = R.k_on ? (unsigned)R.top_k : n_all;
#pragma unroll
  for (int j = 0; j < BPT; ++j) {
    const int b = tid * BPT + j;
    base[b] = run;
    if (run < want && c[j] > (unsigned)SORT_CROWD && !(zero_tail && b == SORT_NB - 1)) S.bp = 0;
    if (run < want && want <= run + c[j]) { S.e_n = run + c[j]; S.bk = b; }
    run += c[j];
  }
  __syncthreads();
  const unsigned n_sort = S.e_n;
  const int last = S.bk;
  if (S.bp == 0 || n_sort > (unsigned)SORT_MAX) return 0u;
#pragma unroll
  for (int j = 0; j < PER; ++j) {
    if (key[j]) {
      const int b = bucket_of(key[j]);
      if (b <= last) sc[atomicAdd(&base[b], 1u)] = composite(key[j], eid[j]);
    }
    __builtin_amdgcn_sched_barrier(0);
  }
  __syncthreads();  // base[b] is the end of bucket b now
  unsigned above = 0u;
#pragma unroll 1
  for (unsigned i = tid; i < n_sort; i += NTHR) {
    const u64 e = sc[i];
    const int b = bucket_of((uint32_t)(e >> 32));
    unsigned r = i;
    if (!(zero_tail && b == SORT_NB - 1)) {
      const unsigned from = b ? base[b - 1] : 0u, to = base[b];
      r = from;
      for (unsigned q = from; q < to; ++q) r += sc[q] > e ? 1u : 0u;
    }
    above += (uint32_t)(e >> 32) >= key_thr ? 1u : 0u;
    reinterpret_cast<u64*>(region + SORT_OUT)[r] = pack_entry(e, y_max);
  }
  above = wave_sum(above);
  if (lane_id() == 0 && above) atomicAdd(&S.memb, above);
  return n_sort;
}

// Where the sorted prefix ends (section 2.1): what both deciding functions below share.  total_m: the mass of the list,
// with top-k of its first k entries.
struct Cuts { u64 S_k_fix, target; bool p_found, known; };
__device__ __forceinline__ Cuts list_cuts(const RowCfg& R, u64 total_m, unsigned n_unc, uint32_t key_g, float y_max, float g, double S_below, bool m_cert) {
  Cuts c;
  c.S_k_fix = R.k_on ? total_m : whole_row_mass(total_m, n_unc, key_g, y_max, g, R.tau, S_below);
  c.target = 0ull;
  c.p_found = R.p_le0;
  if (!R.p_le0 && R.p_on) {
    c.target = (u64)__double2ull_ru((double)R.top_p * (double)c.S_k_fix);
    if (c.target == 0ull) c.target = 1ull;
    c.p_found = total_m >= c.target;
  }
  c.known = R.k_on || c.p_found || m_cert || R.all;
  return c;
}
// A cut below the list's reach: the sliced kernels find it, or the general kernel.
__device__ __forceinline__ int beyond_list(const RowCfg& R) {
  return (R.need_sum || (!R.k_on && !R.p_on && R.minp_on)) ? FIN_WIDE : FIN_PENDING;
}
// What the sorted entries are decided from: their number and that of the listed columns that are not certified, the
// row maximum, the threshold, the mass below it, and with a min-p bound above the threshold (m_cert) the entries at or above it.
struct Listed { unsigned n, n_unc; float y_max; uint32_t key_g; float g; double S_below; bool m_cert; unsigned n_minp; };

// Survivors, masses and the draw (Eq. (2), step (3)) from n <= 64 sorted entries: one per lane of one wave, no
// barrier and no LDS on the way.  The other waves wait.
__device__ __forceinline__ void decide_wave(FS& S, const RowCfg& R, const Listed& L, const u64* entries, const uint32_t* __restrict__ hot_bits) {
  const unsigned lane = lane_id(), n = L.n;
  const bool in = lane < n;
  const u64 e = in ? entries[lane] : 0ull;
  const uint32_t id = entry_id(e);
  const bool use_hot = hot_bits != nullptr;
  const bool hot = use_hot && in && hot_bit(hot_bits, id);
  const u64 w = entry_mass(e);
  const u64 cum = wave_incl_scan(w);
  const Cuts cut = list_cuts(R, read_lane(cum, 63), L.n_unc, L.key_g, L.y_max, L.g, L.S_below, L.m_cert);
  int rc = cut.known ? FIN_DONE : beyond_list(R);
  bool o = in;  // (every cut ends a prefix of the order; the first entry always survives)
  if (R.p_le0) o = lane == 0u;
  else if (R.p_on && cut.p_found) o = o && (cum - w < cut.target);
  if (L.m_cert) o = o && lane < L.n_minp;
  o = o || lane == 0u;
  const unsigned ns = (unsigned)__popcll(__ballot(o));
  const u64 S_K = read_lane(cum, (int)ns - 1);
  const u64 S_H = use_hot ? wave_sum(o && hot ? w : 0ull) : 0ull;
  bool pick_hot = false;
  if (use_hot) pick_hot = (S_H > 0ull) && (S.u[1] * (double)S_K <= (double)S_H);
  const u64 S_cls = use_hot ? (pick_hot ? S_H : S_K - S_H) : S_K;
  const double u = S.u[use_hot && !pick_hot ? 2 : 0];
  if (rc == FIN_DONE && S_cls == 0ull) rc = FIN_PENDING;  // the chosen class holds no mass here: general kernel
  u64 tfix = (u64)__double2ull_rd(u * (double)S_cls);
  if (S_cls > 0ull && tfix >= S_cls) tfix = S_cls - 1ull;
  // inverse CDF in ascending token id over the survivors of the chosen class: the lanes in the order of their ids
  const u64 m = (o && (!use_hot || hot == pick_hot)) ? w : 0ull;
  // (Eight lanes' ids a round and no branch, the lanes behind the list above every id.  With a test and a branch for
  // every lane read, 50 survivors took 3.4 us of their row, 1.6 so; 256 bfloat16 rows of 151,936 columns, top-k 20, 40.6 us a
  // call, 40.2 so.)
  const uint32_t place = in ? id : 0xFFFFFFFFu;
  unsigned before = 0u;
#pragma unroll 1
  for (unsigned q = 0u; q < n; q += 8u) {
    uint32_t other[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) other[j] = read_lane(place, (int)q + j);
#pragma unroll
    for (int j = 0; j < 8; ++j) before += other[j] < place ? 1u : 0u;
  }
  const int to = (int)((in ? before : lane) * 4u);
  const u64 m2 = ((u64)(uint32_t)__builtin_amdgcn_ds_permute(to, (int)(uint32_t)(m >> 32)) << 32) | (u64)(uint32_t)__builtin_amdgcn_ds_permute(to, (int)(uint32_t)m);
  const uint32_t id2 = (uint32_t)__builtin_amdgcn_ds_permute(to, (int)id);
  const u64 run = wave_incl_scan(m2);
  if (lane == 0u) { S.e_rc = rc; S.e_n = ns; S.e_SK = S_K; S.e_SH = S_H; S.e_skfix = cut.S_k_fix; S.e_acc = pick_hot ? 1 : 0; }
  if (rc == FIN_DONE && run > tfix && run - m2 <= tfix) { S.out_id = (int)id2; S.out_w = m2; }
}

// The same for up to SORT_MAX entries, a thread's lie side by side.  Barriers inside.
template <int NTHR>
__device__ __forceinline__ void decide_block(FS& S, const RowCfg& R, const Listed& L, unsigned char* region, const uint32_t* __restrict__ hot_bits) {
  constexpr int NWV = NTHR / 64;
  const int tid = threadIdx.x;
  const u64* entries = reinterpret_cast<const u64*>(region + SORT_OUT);
  u64* fmass = reinterpret_cast<u64*>(region);  // masses of the survivors by ranges of ids, all and the hot ones
  u64* hmass = fmass + NBF;
  u64* mw = hmass + NBF;  // members of the range that holds the draw
  uint32_t* mid = reinterpret_cast<uint32_t*>(mw + MEMB2);
  const bool use_hot = hot_bits != nullptr;
  const unsigned per = (L.n + NTHR - 1u) / NTHR, p0 = min((unsigned)tid * per, L.n), p1 = min(p0 + per, L.n);
  for (int i = tid; i < NBF; i += NTHR) { fmass[i] = 0ull; hmass[i] = 0ull; }
  if (tid == 0) { S.bp = -1; S.bd = -1; }
  u64 loc = 0ull;
  for (unsigned r = p0; r < p1; ++r) loc += entry_mass(entries[r]);
  unsigned z0, z1; u64 me, total_m;
  blk_excl_scan2<NWV>(S, 0u, loc, z0, me, z1, total_m);
  const Cuts cut = list_cuts(R, total_m, L.n_unc, L.key_g, L.y_max, L.g, L.S_below, L.m_cert);
  const bool by_p = R.p_on && cut.p_found && !R.p_le0;
  if (tid == 0) S.memb = 0u;
  if (by_p) {
    u64 run = me;
    for (unsigned r = p0; r < p1; ++r) {
      const u64 w = entry_mass(entries[r]);
      if (run < cut.target && run + w >= cut.target) S.bp = (int)r + 1;
      run += w;
    }
    __syncthreads();
  }
  unsigned ns = R.p_le0 ? 1u : by_p ? (unsigned)S.bp : L.n;
  if (L.m_cert) ns = min(ns, L.n_minp);
  ns = max(ns, 1u);
  const int ishift = max(0, 32 - (int)__clz((unsigned)(R.V - 1) | 1u) - NBF_BITS);
  for (unsigned r = p0; r < min(p1, ns); ++r) {
    const u64 e = entries[r];
    atomicAdd(&fmass[entry_id(e) >> ishift], entry_mass(e));
    if (use_hot && hot_bit(hot_bits, entry_id(e))) atomicAdd(&hmass[entry_id(e) >> ishift], entry_mass(e));
  }
  __syncthreads();
  const u64 fm = (tid < NBF) ? fmass[tid] : 0ull, hm = (use_hot && tid < NBF) ? hmass[tid] : 0ull;
  u64 ea, eh = 0ull, S_K, S_H = 0ull;
  blk_excl_scan2<NWV>(S, 0u, fm, z0, ea, z1, S_K);
  if (use_hot) blk_excl_scan2<NWV>(S, 0u, hm, z0, eh, z1, S_H);
  bool pick_hot = false;
  if (use_hot) pick_hot = (S_H > 0ull) && (S.u[1] * (double)S_K <= (double)S_H);
  const u64 S_cls = use_hot ? (pick_hot ? S_H : S_K - S_H) : S_K;
  const double u = S.u[use_hot && !pick_hot ? 2 : 0];
  int rc = cut.known ? FIN_DONE : beyond_list(R);
  if (rc == FIN_DONE && S_cls == 0ull) rc = FIN_PENDING;  // the chosen class holds no mass here: general kernel
  u64 tfix = (u64)__double2ull_rd(u * (double)S_cls);
  if (S_cls > 0ull && tfix >= S_cls) tfix = S_cls - 1ull;
  {
    const u64 m2 = pick_hot ? hm : fm - hm, me2 = pick_hot ? eh : ea - eh;
    if (m2 > 0ull && me2 <= tfix && me2 + m2 > tfix) { S.bd = tid; S.mab_d = me2; }
  }
  __syncthreads();
  const int bd = S.bd;
  // this thread's entries of the drawn class with a mass in range `to` of ids, ranges of 1 << width ids
  auto each = [&](int width, int to, auto&& f) {
    for (unsigned r = p0; r < min(p1, ns); ++r) {
      const u64 e = entries[r];
      if ((int)(entry_id(e) >> width) != to || entry_mass(e) == 0ull) continue;
      if (use_hot && (hot_bit(hot_bits, entry_id(e)) != 0u) != pick_hot) continue;
      f(e);
    }
  };
  auto gather = [&](int width, int to) {
    each(width, to, [&](u64 e) {
      const unsigned slot = atomicAdd(&S.memb, 1u);
      if (slot < (unsigned)MEMB2) { mid[slot] = entry_id(e); mw[slot] = entry_mass(e); }
    });
    __syncthreads();
  };
  gather(ishift, bd);
  if (S.memb > (unsigned)MEMB2) {  // neighbouring ids (a run of allowed ones, say): the range is divided into as many again
    // (Left to the general kernel: 14 bfloat16 rows of 151,936 columns, 500 neighbouring ones allowed, top-k 1024, 238 us a
    // call; 37.5 so.)
    static_assert(FAST_MAX_V <= NBF * NBF * MEMB2, "a divided range holds no more ids than there is room for");
    const int fshift = max(0, ishift - NBF_BITS), f0 = bd << (ishift - fshift);
    for (int i = tid; i < NBF; i += NTHR) fmass[i] = 0ull;
    __syncthreads();
    each(ishift, bd, [&](u64 e) { atomicAdd(&fmass[(int)(entry_id(e) >> fshift) - f0], entry_mass(e)); });
    if (tid == 0) S.memb = 0u;
    __syncthreads();
    const u64 m = (tid < NBF) ? fmass[tid] : 0ull, before = S.mab_d;
    u64 ex, all;
    blk_excl_scan2<NWV>(S, 0u, m, z0, ex, z1, all);
    if (m > 0ull && before + ex <= tfix && before + ex + m > tfix) { S.bd = f0 + tid; S.mab_d = before + ex; }
    __syncthreads();
    gather(fshift, S.bd);
  }
  const unsigned nm = S.memb;
  if ((unsigned)tid < nm && rc == FIN_DONE) {
    unsigned dummy;
    const u64 G = S.mab_d + sum_where<false>(mid, mw, nm, mid[tid], dummy);
    if (G > tfix && G - mw[tid] <= tfix) { S.out_id = (int)mid[tid]; S.out_w = mw[tid]; }
  }
  if (tid == 0) { S.e_rc = rc; S.e_n = ns; S.e_SK = S_K; S.e_SH = S_H; S.e_skfix = cut.S_k_fix; S.e_acc = pick_hot ? 1 : 0; }
}

constexpr float MAX_SPAN = 64.0f;  // a complete list may reach further down: what lies there has no mass and shares the last bucket

// Lists that are not sorted (more than SORT_MAX entries that may survive, or crowded by ties; in LDS as keys lk[] /
// ids li[]): bucket tables over the key range locate each cut; only the bucket that holds a cut is resolved entry by entry.
// Same decisions as above.  SPREAD (rows listed whole): a bucket with more members than are resolved
// at once is spread again; a sampled list leaves its row to the kernels that follow.
template <int NTHR, bool SPREAD>
__device__ __forceinline__ int finalize_long(FS& S, const RowCfg& R, unsigned n, unsigned n_unc, uint32_t kmax,
                                             uint32_t key_g, uint32_t key_lo, bool sliced, float g, double S_below, const uint32_t* lk, const uint32_t* li,
                                             unsigned char* tables, const uint32_t* __restrict__ hot_bits, simple_row_diag& dg) {
  constexpr int NWV = NTHR / 64;
  const int tid = threadIdx.x;
  uint32_t* fcnt = reinterpret_cast<uint32_t*>(tables);             // NBF * 4
  u64* fmass = reinterpret_cast<u64*>(tables + NBF * 4);             // NBF * 8
  u64* mc = reinterpret_cast<u64*>(tables + NBF * 12);               // MEMB2 * 8
  u64* mw = reinterpret_cast<u64*>(tables + NBF * 12 + MEMB2 * 8);   // MEMB2 * 8
  const float y_max = keyf(kmax);
  // buckets are linear in the tempered value (key space is logarithmic around zero), down to the list's
  // lower end; monotone in the key.  A sampled list (key_lo is its threshold) ends a little below the cut, however
  // far that is from the maximum: at a low temperature a long top-k reaches hundreds down.
  const float span = y_max - keyf(key_lo);
  const float bscale = (float)NBF / fmaxf(key_lo == key_g ? span : fminf(span, MAX_SPAN), 1e-30f);
  auto bucket_of = [&](uint32_t k) { return (unsigned)min((int)((y_max - keyf(k)) * bscale), NBF - 1); };
  u64 cl = 0ull;
  for (unsigned i = tid; i < n; i += NTHR) { const u64 c = composite(lk[i], li[i]); cl = (c > cl) ? c : cl; }
  unsigned da = 0, db = 0; u64 cmax = cl, dd = 0ull;
  blk_reduce<NWV>(S, da, db, cmax, dd);
  constexpr u64 MANY = ~0ull;
  // Among the entries that `in` selects, in descending order of their (distinct) values: the one at which the
  // running mass (or count), `acc` before the first, reaches the target (its value; 0 if none does).  Up to MEMB2 of
  // them are resolved at once; more (ties, most often) are spread over the buckets of their range of values
  // until the bucket that holds the place has no more (without SPREAD: MANY).  If they were not spread
  // (direct), e_SK is the mass of the entries down to the one returned.
  bool direct = true;
  auto mass_of = [&](unsigned i) { return wfix(lk[i], y_max); };
  auto resolve = [&](auto&& in, auto&& value, const bool by_count, u64 acc, u64 target) -> u64 {
    direct = true;
    u64 lo = 0ull, hi = ~0ull;
    for (;;) {
      if (tid == 0) { S.memb = 0u; S.e_tfix = 0ull; }
      __syncthreads();
      for (unsigned i = tid; i < n; i += NTHR) {
        if (!in(i)) continue;
        const u64 v = value(i);
        if (v < lo || v > hi) continue;
        const unsigned slot = atomicAdd(&S.memb, 1u);
        if (slot < (unsigned)MEMB2) { mc[slot] = v; mw[slot] = mass_of(i); }
      }
      __syncthreads();
      const unsigned nm = S.memb;
      if (nm <= (unsigned)MEMB2) {
        for (unsigned mi = tid; mi < nm; mi += NTHR) {
          unsigned r;
          const u64 mass = sum_where<true>(mc, mw, nm, mc[mi], r);
          const u64 G = acc + (by_count ? (u64)r + 1ull : mass), w = by_count ? 1ull : mw[mi];
          if (G >= target && G - w < target) { S.e_tfix = mc[mi]; S.e_SK = mass; }
        }
        __syncthreads();
        return S.e_tfix;
      }
      if constexpr (!SPREAD) return MANY;
      direct = false;
      if (hi == ~0ull) {  // the range of their values
        u64 vmax = 0ull, nmin = 0ull, none = 0ull;
        unsigned z0 = 0u, z1 = 0u;
        for (unsigned i = tid; i < n; i += NTHR) {
          if (!in(i)) continue;
          const u64 v = value(i);
          vmax = v > vmax ? v : vmax; nmin = ~v > nmin ? ~v : nmin;
        }
        blk_reduce<NWV>(S, z0, z1, vmax, none);
        blk_reduce<NWV>(S, z0, z1, nmin, none);
        hi = vmax; lo = ~nmin;
      }
      const int sh = max(0, 64 - NBF_BITS - (int)__clzll((long long)(hi - lo)));
      for (int i = tid; i < NBF; i += NTHR) fmass[i] = 0ull;
      if (tid == 0) S.bk = -1;
      __syncthreads();
      for (unsigned i = tid; i < n; i += NTHR) {
        if (!in(i)) continue;
        const u64 v = value(i);
        if (v >= lo && v <= hi) atomicAdd(&fmass[(unsigned)((hi - v) >> sh)], by_count ? 1ull : mass_of(i));
      }
      __syncthreads();
      const u64 m = (tid < NBF) ? fmass[tid] : 0ull;
      unsigned c0, c1; u64 me, mt;
      blk_excl_scan2<NWV>(S, 0u, m, c0, me, c1, mt);
      if (acc + me < target && acc + me + m >= target) { S.bk = tid; S.mab_p = acc + me; }
      __syncthreads();
      const int d = S.bk;
      if (d < 0) return 0ull;
      acc = S.mab_p;
      const u64 width = 1ull << sh;
      hi -= (u64)(unsigned)d << sh;
      if (hi - lo >= width) lo = hi - (width - 1ull);
      if (sh == 0) return hi;
    }
  };
  auto comp_of = [&](unsigned i) { return composite(lk[i], li[i]); };
  for (int i = tid; i < NBF; i += NTHR) { fcnt[i] = 0u; fmass[i] = 0ull; }
  __syncthreads();
  for (unsigned i = tid; i < n; i += NTHR) {
    const uint32_t k = lk[i];
    const unsigned b = bucket_of(k);
    atomicAdd(&fcnt[b], 1u);
    atomicAdd(&fmass[b], wfix(k, y_max));
  }
  __syncthreads();
  const unsigned c = (tid < NBF) ? fcnt[tid] : 0u;
  const u64 m = (tid < NBF) ? fmass[tid] : 0ull;
  unsigned ce, total_c; u64 me, total_m;
  blk_excl_scan2<NWV>(S, c, m, ce, me, total_c, total_m);
  const unsigned n_k = R.k_on ? (unsigned)R.top_k : (unsigned)R.V;
  // ---- top-k cut: the bucket that holds the n_k-th entry, then its members exactly ----
  const bool kcut = R.k_on && n > n_k;
  if (kcut && tid < NBF && c > 0u && ce < n_k && n_k <= ce + c) { S.bk = tid; S.cab_k = ce; S.mab_k = me; }
  __syncthreads();
  u64 cut_k = 0ull, S_klist = total_m;
  int bk = -1;
  if (kcut) {
    bk = S.bk;
    const u64 above = S.mab_k;
    cut_k = resolve([&](unsigned i) { return (int)bucket_of(lk[i]) == bk; }, comp_of, true, (u64)S.cab_k, (u64)n_k);
    if (cut_k == 0ull || cut_k == MANY) return FIN_PENDING;
    S_klist = above + S.e_SK;
    if (!direct) {
      u64 part = 0ull;
      for (unsigned i = tid; i < n; i += NTHR) if ((int)bucket_of(lk[i]) == bk && comp_of(i) >= cut_k) part += mass_of(i);
      S_klist = above + blk_sum_u64<NWV>(S, part);
    }
    __syncthreads();
  }
  // ---- mass of the top-k prefix (all of V when top-k is off) ----
  const u64 S_k_fix = R.k_on ? S_klist : whole_row_mass(total_m, n_unc, key_g, y_max, g, R.tau, S_below);
  // ---- nucleus cut: shortest prefix whose mass reaches top_p * S_k ----
  u64 cut_p = 0ull;
  bool p_found = false;
  if (R.p_le0) { cut_p = cmax; p_found = true; }
  else if (R.p_on) {
    u64 target = (u64)__double2ull_ru((double)R.top_p * (double)S_k_fix);
    if (target == 0ull) target = 1ull;
    if (tid < NBF && c > 0u && (bk < 0 || tid <= bk)) {
      const u64 incl = (tid == bk) ? S_klist : me + m;
      if (me < target && incl >= target) { S.bp = tid; S.mab_p = me; }
    }
    __syncthreads();
    const int bp = S.bp;
    if (bp >= 0) {
      cut_p = resolve([&](unsigned i) { return (int)bucket_of(lk[i]) == bp && comp_of(i) >= cut_k; }, comp_of, false, S.mab_p, target);
      if (cut_p == MANY) {  // the sliced kernels resolve them, from the bucket's upper end down
        if (!sliced) return FIN_PENDING;
        if (tid == 0) S.wmax[0] = y_max - (float)bp / bscale;
        return FIN_WIDE;
      }
      if (cut_p == 0ull) return FIN_PENDING;  // cannot happen: the bucket's mass reaches the target
      p_found = true;
    }
  }
  // ---- min-p cut: y >= fl32(y_max + fl32(ln min_p)) ----
  u64 cut_m = 0ull;
  bool m_cert = false;
  if (R.minp_on) {
    const float thr = y_max + (float)log((double)R.min_p);
    const uint32_t key_thr = fkey(thr);
    if (key_thr > key_g) { cut_m = (u64)key_thr << 32; m_cert = true; }
  }
  const bool known = R.k_on || p_found || m_cert || R.all;
  if (!known) return (R.need_sum || (!R.k_on && !R.p_on && R.minp_on)) ? FIN_WIDE : FIN_PENDING;
  if (R.k_on && R.p_on && !p_found) { return FIN_PENDING; }  // cannot happen: the top-k prefix holds its own mass
  u64 cut = cut_k;
  if (p_found && cut_p > cut) cut = cut_p;
  if (m_cert && cut_m > cut) cut = cut_m;
  if (cut > cmax) cut = cmax;  // never empty
  // ---- survivors K_b by ranges of ids, all and the hot ones: their masses (Eq. (7)) and where the draw lies ----
  // (one weighing of the list for both)
  const bool use_hot = hot_bits != nullptr;
  const int ishift = max(0, 32 - (int)__clz((unsigned)(R.V - 1) | 1u) - 8);
  u64* hmass = mc;  // the member table is free here
  for (int i = tid; i < NBF; i += NTHR) { fmass[i] = 0ull; if (use_hot) hmass[i] = 0ull; }
  __syncthreads();
  unsigned ns = 0;
  for (unsigned i = tid; i < n; i += NTHR) {
    const uint32_t k = lk[i], id = li[i];
    if (composite(k, id) >= cut) {
      const u64 w = wfix(k, y_max);
      ++ns;
      atomicAdd(&fmass[id >> ishift], w);
      if (use_hot && hot_bit(hot_bits, id)) atomicAdd(&hmass[id >> ishift], w);
    }
  }
  __syncthreads();
  unsigned n_before, n_surv; u64 ea, eh = 0ull, S_K, S_H = 0ull;
  blk_excl_scan2<NWV>(S, ns, (tid < NBF) ? fmass[tid] : 0ull, n_before, ea, n_surv, S_K);
  if (use_hot) { unsigned c2, ct2; blk_excl_scan2<NWV>(S, 0u, (tid < NBF) ? hmass[tid] : 0ull, c2, eh, ct2, S_H); }
  bool pick_hot = false;
  if (use_hot) {
    pick_hot = (S_H > 0ull) && (S.u[1] * (double)S_K <= (double)S_H);
    dg.alpha = (double)S_H / (double)S_K;
    dg.flags |= SIMPLE_DIAG_SHVS | (pick_hot ? SIMPLE_DIAG_ACCEPTED : 0u);
  }
  const u64 S_cls = use_hot ? (pick_hot ? S_H : S_K - S_H) : S_K;
  const double u = S.u[use_hot && !pick_hot ? 2 : 0];
  dg.n_survivors = (int)n_surv;
  dg.s_k = (double)S_k_fix / WSCALE;
  if (S_cls == 0ull) { return FIN_PENDING; }  // the chosen class holds no mass here: general kernel
  // ---- inverse CDF in ascending token id: first id whose running mass exceeds u * S ----
  u64 tfix = (u64)__double2ull_rd(u * (double)S_cls);
  if (tfix >= S_cls) tfix = S_cls - 1ull;
  auto in_class = [&](uint32_t k, uint32_t id) {
    if (composite(k, id) < cut) return false;
    if (!use_hot) return true;
    return (hot_bit(hot_bits, id) != 0u) == pick_hot;
  };
  if (tid < NBF) {
    const u64 mh = use_hot ? hmass[tid] : 0ull;
    const u64 m2 = pick_hot ? mh : fmass[tid] - mh, me2 = pick_hot ? eh : ea - eh;
    if (m2 > 0ull && me2 <= tfix && me2 + m2 > tfix) { S.bd = tid; S.mab_d = me2; }
  }
  __syncthreads();
  const int bd = S.bd;
  if (bd < 0) { return FIN_PENDING; }  // cannot happen: tfix < S_cls
  {
    const u64 v = resolve([&](unsigned i) { return in_class(lk[i], li[i]) && (int)(li[i] >> ishift) == bd; },
                          [&](unsigned i) { return (u64)(0xFFFFFFFFu - li[i]); }, false, S.mab_d, tfix + 1ull);
    if (v == MANY) return FIN_PENDING;
    const uint32_t id = 0xFFFFFFFFu - (uint32_t)v;  // (distinct ids below 2^31: no value is zero)
    for (unsigned i = tid; i < n; i += NTHR) if (v != 0ull && li[i] == id) { S.out_id = (int)id; S.out_w = mass_of(i); }
  }
  __syncthreads();
  dg.p_chosen = (float)((double)S.out_w / (double)S_K);
  return (S.out_id >= 0) ? FIN_DONE : FIN_PENDING;
}

// History entry i (fewer than 2^16 of them: an offset of 32 bits, one register an entry instead of two).
__device__ __forceinline__ int hist_at(const int32_t* h, int i) {
  return *as_global(reinterpret_cast<const int32_t*>(reinterpret_cast<const char*>(h) + (uint32_t)(i * 4)));
}

// The penalties of a row's listed columns, without its tables: the listed columns go to a hash table (a row listed
// whole has a counter per column), the history's ids look themselves up in it and count, then each column takes what was
// counted for it.  Work goes with the list and the history; the tables go with the vocabulary too (mask cleared, scanned into a
// directory, looked up through it): 8 bfloat16 rows of 151,936 columns with 2048 ids each 37.9 us a call, 35.9 so.  For rows with a
// compute unit to themselves: where several share one, the tables' lookups, all in flight at once, are hidden better than
// the table's chains (4096 rows of 256,000 columns with 8192 ids, 512 threads: 947 us with the tables, 964 with this).
// Entry j of this thread is list entry tid + j * NTHR; ids[j] is history entry tid + j * NTHR.  Barriers inside; one must follow.
constexpr unsigned HASH_LIST_MAX = 192;  // listed columns
// Fewer of them leave shorter chains for the ids that are not listed, most of a history.  Measured on 14 bfloat16 rows of
// 151,936 columns, 200 float32 rows of 128,256 and 64 of 50,000, with tables less with the hash, us a call: 50 listed columns
// 2.4 to 9.4 at 512 to 32,000 ids, 150 0.6 to 3.6 up to 12,000, 200 -0.1 to 3.2 up to 8192; 256 -1.2 to 0.1 at 8192, 350 -3.9 to
// -2.8, 500 -15 to -9.  (A second, higher line for short histories, worth 2 us between 192 and 320 columns, had the compiler
// write out the loops over the history twice and cost every such call 0.8.)
static_assert(MAX_WHOLE * 4 <= FAST_REGION_MIN, "the counters fit the region");
template <int NTHR, int PER, int NID, bool WHOLE>
__device__ __forceinline__ void penalise_listed(FS& S, const Hist& H, float (&ez)[PER], const uint32_t (&eid)[PER], unsigned n, const int (&ids)[NID],
                                                const int32_t* __restrict__ hist, int nnz, int n_prompt, int V, unsigned char* region) {
  constexpr int ROUNDS = WHOLE ? PER : 1;
  static_assert(HASH_LIST_MAX <= 1024, "a hashed list takes one round of the workgroups that hash it");
  const int tid = threadIdx.x;
  constexpr unsigned bits = 10u, slots = 1u << bits;
  uint32_t* count = reinterpret_cast<uint32_t*>(region);  // occurrences in the high half, generated ones in the low half
  uint32_t* owner = count + slots;                        // column + 1; 0: free
  auto first = [&](uint32_t id) { return (id * 0x9E3779B1u) >> (32u - bits); };
  zero16(region, WHOLE ? V * 4 : (int)slots * 8, tid, NTHR);
  __syncthreads();
  if constexpr (!WHOLE) {
#pragma unroll
    for (int j = 0; j < ROUNDS; ++j) {
      if ((unsigned)(j * NTHR) >= n) break;
      if ((unsigned)(tid + j * NTHR) < n) {  // (a column is listed once)
        uint32_t h = first(eid[j]);
        while (atomicCAS(&owner[h], 0u, eid[j] + 1u) != 0u) h = (h + 1u) & (slots - 1u);
      }
    }
    __syncthreads();
  }
  n_prompt = min(max(n_prompt, 0), nnz);
  bool bad = false;
  // (four ids' first places are read before any is used)
  auto occur4 = [&](const int (&id)[4], int i0) {
    uint32_t o[4];
    if constexpr (!WHOLE) {
#pragma unroll
      for (int k = 0; k < 4; ++k) o[k] = owner[first((uint32_t)id[k])];
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int i = i0 + k * NTHR;
      if (i >= nnz) continue;
      if ((unsigned)id[k] >= (unsigned)V) { bad = true; continue; }
      const uint32_t one = 0x10000u + (i >= n_prompt ? 1u : 0u);
      if constexpr (WHOLE) atomicAdd(&count[id[k]], one);
      else {
        uint32_t h = first((uint32_t)id[k]);
        while (o[k] != 0u && o[k] != (uint32_t)id[k] + 1u) { h = (h + 1u) & (slots - 1u); o[k] = owner[h]; }
        if (o[k]) atomicAdd(&count[h], one);
      }
    }
  };
  static_assert(NID % 4 == 0, "whole groups");
#pragma unroll
  for (int j = 0; j < NID; j += 4) {
    if (j * NTHR >= nnz) break;
    const int id4[4] = {ids[j], ids[j + 1], ids[j + 2], ids[j + 3]};
    occur4(id4, tid + j * NTHR);
  }
  for (int i0 = tid + NID * NTHR; i0 < nnz; i0 += 4 * NTHR) {
    int id4[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) id4[k] = i0 + k * NTHR < nnz ? hist[i0 + k * NTHR] : 0;
    occur4(id4, i0);
  }
  if (bad) atomicOr(&S.flags, SIMPLE_DIAG_BAD_HISTORY_ID);
  __syncthreads();
#pragma unroll
  for (int j = 0; j < ROUNDS; ++j) {
    if ((unsigned)(j * NTHR) >= n) break;
    if ((unsigned)(tid + j * NTHR) >= n) continue;
    uint32_t h = eid[j];
    if constexpr (!WHOLE) {
      h = first(eid[j]);
      while (owner[h] != eid[j] + 1u) h = (h + 1u) & (slots - 1u);
    }
    const uint32_t c = count[h];
    if (c) ez[j] = H.apply(ez[j], c & 0xFFFFu);
  }
}

__device__ inline void queue_pending(const SampleArgs& a, int row) {
  const unsigned slot = atomicAdd(&a.pend[0], 1u);
  a.pend[2 + slot] = (uint32_t)row;
  a.out[row] = PENDING;
}

// ---------------------------------------------------------------- the rows' order -------------
// Which row a workgroup takes, in a launch with more rows than compute units: rows with long epilogues first.  Workgroups are
// handed to the compute units in turn, so that a compute unit holds workgroups b, b + (number of compute units), ...: with
// the long rows at the front every compute unit gets its share of them instead of some holding four (measured on the
// heterogeneous batch: a compute unit with four such rows finishes 20 us after one with two), and a launch of several rounds starts
// its longest rows first.  In a bfloat16 call the kernel ahead of this one writes that order for the whole launch; in a float32 call
// there is none, and a workgroup finds its row among those of 64 neighbouring compute units (16 rounds of them at most), long
// ones first, each kind in row order.  (A kernel of one workgroup that wrote the order for all: 5 us of the call and its gap.  1024
// rows of 128,256 columns 197.2 us a call, 195.5 so; 512 with a state 134.8 and 133.9.)  The same in every thread; a barrier inside.
template <int NTHR>
__device__ __forceinline__ int pick_row(const SampleArgs& a, FS& S) {
  constexpr int NWV = NTHR / 64, CUS = 64, ROUNDS = 16;
  static_assert(CUS * ROUNDS / 64 <= 16, "a word of the workgroup's state per 64 rows");
  const int lane = lane_id(), n_cu = a.n_cu, b = (int)blockIdx.x;
  const int q = b / n_cu, j = b - q * n_cu, c0 = j / CUS * CUS, wd = min(CUS, n_cu - c0), q0 = q / ROUNDS * ROUNDS;
  const int base = q0 * n_cu + c0;
  const int words = (min(ROUNDS, (a.B - base + n_cu - 1) / n_cu) * wd + 63) / 64;
  auto member = [&](int m) { const int r = m / wd; return base + r * n_cu + (m - r * wd); };  // the group's m-th row
#pragma unroll 1
  for (int k = wave_id(); k < words; k += NWV) {
    const int m = k * 64 + lane, r = member(m);
    const bool in = m < wd * ROUNDS && r < a.B;
    const bool is_long = in && long_epilogue(a.params[in ? r : 0], a.V);
    const u64 ml = __ballot(is_long), ms = __ballot(in && !is_long);
    if (lane == 0) { S.r64a[k] = ml; S.r64b[k] = ms; }
  }
  __syncthreads();
  const u64 ml = lane < words ? S.r64a[lane] : 0ull, ms = lane < words ? S.r64b[lane] : 0ull;
  unsigned at = (unsigned)((q - q0) * wd + (j - c0));  // this workgroup's place
  const unsigned n_long = wave_sum((unsigned)__popcll(ml));
  const u64 mask = at < n_long ? ml : ms;
  at -= at < n_long ? 0u : n_long;
  const unsigned c = (unsigned)__popcll(mask), incl = wave_incl_scan(c);
  const int k = __builtin_amdgcn_readfirstlane(__ffsll((long long)__ballot(at >= incl - c && at < incl)) - 1);
  const u64 word = read_lane(mask, k);
  at -= read_lane(incl, k) - (unsigned)__popcll(word);
  const u64 hit = __ballot(((word >> lane) & 1ull) != 0ull && lanes_before(word) == at);
  return __builtin_amdgcn_readfirstlane(member(k * 64 + __ffsll((long long)hit) - 1));
}

// ---------------------------------------------------------------- the kernel ------------------
// (The second launch bound is HIP's: waves per SIMD, not workgroups per compute unit.  Four waves per
// SIMD, 128 registers each, are sixteen waves per compute unit at every workgroup size: four
// workgroups of 256 threads, two of 512, one of 1024.)
// STATEFUL: the rows' histories come from an incremental penalty state (its own instantiation, so
// that the stateless kernel carries none of that code).
// WHOLE: the list holds every column of a row (a.F.whole; its own instantiation, since with the test at run
// time the sampled rows' prologue was 1 us slower: 8 bfloat16 rows of 151,936 columns 44.4 against 45.9 us).
template <typename DT, int NTHR, bool STATEFUL, bool WHOLE>
__global__ __launch_bounds__(NTHR, 4) void fast_rows_kernel(const SampleArgs a) {
  constexpr int NWV = NTHR / 64;
  constexpr int EPL = Io<DT>::EPL;
  constexpr int T = 64 * EPL * UNR;
  constexpr int PER = capf_per_thread(NTHR, WHOLE);
  constexpr int IDR = idr(NTHR);
  typedef typename Io<DT>::Raw Raw;
  extern __shared__ __align__(16) unsigned char lds[];
  __shared__ FS S;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  int row = (int)blockIdx.x;
  if constexpr (!WHOLE) {
    if (sizeof(DT) == 2 && a.order) row = a.order[blockIdx.x];
    else if (sizeof(DT) == 4 && a.pick) row = pick_row<NTHR>(a, S);
  }
  const int V = a.V;
  const DT* rowp = reinterpret_cast<const DT*>(a.logits) + (size_t)row * (size_t)a.stride;
  // the pattern-count kernel, when it ran before this one, has left NOT_TAKEN on every row that is still to do
  if (a.pattern_on && a.out[row] != NOT_TAKEN) return;
  // this wave's first two tiles (its threshold sample): issued before anything else
  // (a row that fits the list whole has at most one tile per wave and no sample)
  const int nfull = V / T;  // else the host guarantees nfull >= 2 * NWV
  const int t0 = (int)(((long long)wave * nfull) / NWV);
  const int t_end = (int)(((long long)(wave + 1) * nfull) / NWV);
  constexpr bool whole = WHOLE;
  Raw A[UNR], Bf[UNR];
  if (!whole || t0 < t_end) {
#pragma unroll
    for (int u = 0; u < UNR; ++u) A[u] = Io<DT>::load(rowp + (size_t)t0 * T + u * 64 * EPL + lane * EPL);
  }
  if (!whole) {
#pragma unroll
    for (int u = 0; u < UNR; ++u) Bf[u] = Io<DT>::load(rowp + (size_t)(t0 + 1) * T + u * 64 * EPL + lane * EPL);
  }
  const simple_row_params par = a.params[row];
  uint32_t* samp = reinterpret_cast<uint32_t*>(lds + a.F.samp);

  // ---- row configuration (identical in every thread) ----
  const bool bad_par = !(par.temperature >= 0.0f) || !(par.rep_penalty > 0.0f);
  RowCfg R;
  R.greedy = par.temperature == 0.0f;
  R.k_on = par.top_k >= 1 && par.top_k < V;
  R.top_k = par.top_k; R.V = V;
  R.tau = R.greedy ? 1.0f : par.temperature;
  R.top_p = par.top_p; R.min_p = par.min_p;
  R.p_on = par.top_p < 1.0f;
  R.p_le0 = par.top_p <= 0.0f;
  R.minp_on = par.min_p > 0.0f;
  R.need_sum = !R.greedy && !R.k_on && R.p_on && !R.p_le0;
  // the call's CSR arrays, or the row's slot of an incremental state
  const RowHist rh = STATEFUL ? row_history_state(a, row, par.n_prompt) : row_history_csr(a, row, par.n_prompt);
  const int nnz = rh.nnz;
  constexpr bool stateful = STATEFUL;
  const bool too_long = nnz > a.max_nnz;
  const bool pen_on = par.rep_penalty != 1.0f || par.freq_penalty != 0.0f || par.pres_penalty != 0.0f;
  const bool lowering = par.rep_penalty >= 1.0f && par.freq_penalty >= 0.0f && par.pres_penalty >= 0.0f;
  const bool h_active = (nnz > 0) && pen_on;
  const bool no_trunc = !R.greedy && !R.k_on && !R.p_on && !R.minp_on;
  // Rows that keep no candidate list and only pass through here on their way to the kernels of the
  // whole-vocabulary routes, which apply any penalties column by column: rows without any
  // truncation, and rows without top-k whose penalties raise logits (the list's threshold test on
  // raw logits would miss columns).
  // ... and rows with top-k alone beyond the list's reach (any penalties).
  const bool big_k = !R.greedy && R.k_on && par.top_k > KMAXF && !R.p_on && !R.minp_on;
  // (a list that holds the whole row needs no threshold and decides all of these itself)
  const bool straight = !whole && (no_trunc || big_k || (!R.greedy && !R.k_on && !R.p_le0 && h_active && !lowering));
  R.all = whole && no_trunc;
  const uint32_t straight_mode = no_trunc ? (uint32_t)WIDE_ALL : big_k ? (uint32_t)WIDE_TOP_K
                                          : (R.p_on ? (uint32_t)WIDE_TOP_P : (uint32_t)WIDE_MIN_P);
  const bool eligible = (straight || whole) ? (!bad_par && !too_long)
                                            : (!bad_par && !too_long && (!h_active || lowering) &&
                                               (R.greedy || !R.k_on || par.top_k <= KMAXF));
  if (!eligible) {  // the general kernel takes the row (it also reports parameter errors)
    if (tid == 0) queue_pending(a, row);
    return;
  }
  // (top-k beyond the list: the threshold is only the reference of the masses and must leave fewer
  // than top_k columns above it, so it aims at a quarter of them)
  const int k_sel = R.greedy ? 1 : (R.k_on ? (big_k ? par.top_k / 4 : par.top_k) : (R.p_le0 ? 1 : KMAXF));
  if (tid == 0) {
    S.cand_count = 0u; S.flags = 0u; S.kmax = 0u; S.memb = 0u; S.bk = -1; S.bp = -1; S.bd = -1;
    S.cut_k = 0ull; S.cut_p = 0ull; S.out_id = -1; S.out_w = 0ull; S.kmin = 0xFFFFFFFFu;
    S.n2 = 0u; S.nunc = 0u; S.e_rc = FIN_PENDING; S.e_n = 0u; S.tile_ctr = 0u;
  }
  if (!whole && NWV > 4) for (int i = tid; i < QUICK_NB; i += NTHR) samp[i] = 0u;  // (the sample's counts: see quick_threshold)
  // ---- loads first: history ids, then this wave's two sample tiles ----
  const int32_t* hist = rh.ids;
  // (by a 64-bit place where the row is listed whole: 4 rows of 1024 columns 14.7 us a call, 15.0 to 15.2 with the other)
  auto hist_entry = [&](int i) -> int { return WHOLE ? hist[i] : hist_at(hist, i); };
  // With a state the tables come ready-made from the row's slot (section 5.2: carried from step to
  // step, not rebuilt): `whole` = mask, rank directory and counts, else the mask alone.  Ends with a barrier.
  auto load_tables = [&](bool whole) {
    const unsigned n_pairs = (unsigned)((((V + 31) >> 5) + 1) >> 1);
    const unsigned units = whole ? (a.F.cnt + (unsigned)((nnz + 3) / 2) * 4u + 15u) / 16u : (n_pairs * 8u + 15u) / 16u;
    const u32x4* src = reinterpret_cast<const u32x4*>(a.st_tables + (size_t)rh.slot * a.st_stride);
    u32x4* dst = reinterpret_cast<u32x4*>(lds);
    for (unsigned i = tid; i < units; i += NTHR) dst[i] = as_global(src)[i];
    if (tid == 0) { S.distinct = (unsigned)a.st_rec[rh.slot].distinct; if (rh.flags) atomicOr(&S.flags, rh.flags); }
    __syncthreads();
  };
  Hist H;
  H.bm = reinterpret_cast<uint32_t*>(lds + a.F.bitmap);
  H.dir = reinterpret_cast<uint16_t*>(lds + a.F.dir);
  H.cnt32 = reinterpret_cast<uint32_t*>(lds + a.F.cnt);
  H.n_words = (V + 31) >> 5;
  H.rep = par.rep_penalty; H.freq = par.freq_penalty; H.pres = par.pres_penalty;
  H.inv_rep = 1.0 / (double)par.rep_penalty;
  H.active = h_active;
  {
    int ids[IDR];
#pragma unroll
    for (int j = 0; j < IDR; ++j) { const int i = tid + j * NTHR; ids[j] = (!whole && h_active && !stateful && i < nnz) ? hist_entry(i) : -1; }
    if (wave == NWV - 1) {  // (one wave of the row, for all)
      double u[3];
      row_uniforms(a.seed, a.row_offset + (uint64_t)row, a.step, u);
      if (lane < 3) S.u[lane] = lane == 0 ? u[0] : lane == 1 ? u[1] : u[2];
    }
    __syncthreads();
    // ---- presence mask of the history (in the shared region); all tables for a row that leaves early ----
    // (a row that is listed whole has no sample to keep the history out of)
    if (!whole && H.active) {
      if (stateful) load_tables(straight);
      else if (straight) { unsigned own; build_history<NTHR>(S, H, ids, hist, nnz, rh.n_prompt, V, own); }
      else build_bitmap<NTHR>(S, H, ids, hist, nnz, V);
    }
  }
  const uint32_t* hot_bits = R.greedy ? nullptr : a.hot_bits;
  StreamCtx C;
  C.g = 0.0f;
  // Hands the row to the kernels of the whole-vocabulary routes: a queue record, a cleared workspace
  // slot and the row's history tables (rebuilt first if the region no longer holds them).  False if
  // no slot is free.  All threads call.
  auto queue_wide = [&](uint32_t mode, bool tables_live, float g_ref, float y_max) -> bool {
    __syncthreads();
    if (H.active && !tables_live) {
      if (stateful) load_tables(true);
      else {
        int ids2[IDR];
#pragma unroll
        for (int j = 0; j < IDR; ++j) { const int i = tid + j * NTHR; ids2[j] = (i < nnz) ? hist_entry(i) : -1; }
        unsigned own;
        build_history<NTHR>(S, H, ids2, hist, nnz, rh.n_prompt, V, own);
      }
    }
    if (tid == 0) S.e_n = atomicAdd(&a.wq[0], 1u);
    __syncthreads();
    const unsigned slot = S.e_n;
    const unsigned hb = H.active ? (a.F.cnt + (unsigned)((nnz + 3) / 2) * 4u + 15u) / 16u : 0u;  // 16-byte units of history tables
    if (slot >= (unsigned)a.wide_slots || WS_HT + hb * 16u > a.ws_stride) return false;
    u32x4* ws = reinterpret_cast<u32x4*>(a.wws + (size_t)slot * a.ws_stride);
    const u32x4 zero = {0u, 0u, 0u, 0u};
    for (unsigned i = tid; i < WS_RL / 16u; i += NTHR) ws[i] = zero;
    if (H.active) {
      const u32x4* src = reinterpret_cast<const u32x4*>(lds);
      for (unsigned i = tid; i < hb; i += NTHR) ws[WS_HT / 16u + i] = src[i];
    }
    if (tid == 0) {
      WideRec rec;
      rec.row = (uint32_t)row; rec.g = g_ref; rec.mode = mode | ((a.f64 || g_ref > C.g) ? WIDE_F64 : 0u) | (y_max > -INFINITY ? WIDE_MAX : 0u); rec.flags = S.flags & 0x3FFFFFFFu;
      rec.tau = R.tau; rec.top_p = R.top_p; rec.rep = par.rep_penalty; rec.freq = par.freq_penalty;
      rec.pres = par.pres_penalty; rec.ln_min_p = R.minp_on ? (float)log((double)R.min_p) : 0.0f; rec.y_max = y_max; rec.h_active = h_active ? 1 : 0;
      rec.min_p = R.min_p; rec.top_k = par.top_k; rec.distinct = H.active ? S.distinct : 0u;
      rec.far_slot = 0u;
      reinterpret_cast<WideRec*>(a.wq + WQ_HEAD)[slot] = rec;
      a.out[row] = PENDING;
    }
    return true;
  };

  bool complete = whole;  // the list takes every finite column
  if (!whole) {
  // ---- threshold from the sample (its unpenalised values) ----
  // rank in the sample whose value leaves, with high probability, >= k_sel columns above it in the row
  const float m_exp = (float)k_sel * (float)(NWV * 2 * T) / (float)V;
  const unsigned r_samp = (unsigned)ceilf(1.15f * m_exp + 3.2f * sqrtf(m_exp) + 3.5f);
  const SampleRanks ranks = sample_ranks((unsigned)k_sel, r_samp, NWV);
  // Rows that the list alone decides: any value that admits enough columns serves, and with eight waves and more it
  // comes from counts.  (With four waves the search by ballots is the shorter one: 1024 float32 rows of 128,256
  // columns 201.1 against 202.6 us a call.  The other rows' masses are rounded relative to the threshold, so theirs is
  // kept as it always was, to the bit: sums of the same columns do not depend on the build.)
  const bool quick = NWV > 4 && (R.greedy || (R.k_on && !big_k) || R.p_le0) && ranks.ok;
  // (either branch takes copies of the tiles: the compiler unpacks them ahead of both otherwise, into registers that then spill)
  if (quick) {
    float m[2] = {-INFINITY, -INFINITY};
    unsigned fin = 0u;
    auto take_group = [&](const Raw& X, int idx0, float& mx) {
      float z[EPL];
      Raw Y = X;
      asm volatile("" : "+v"(Y));
      sample_group<DT>(Y, idx0, H, z);
      fin += (unsigned)__popcll(__ballot(z[0] > -INFINITY));
#pragma unroll
      for (int e = 0; e < EPL; ++e) mx = fmaxf(mx, z[e]);  // (a NaN is ignored)
    };
#pragma unroll
    for (int u = 0; u < UNR; ++u) take_group(A[u], t0 * T + u * 64 * EPL + lane * EPL, m[0]);
#pragma unroll
    for (int u = 0; u < UNR; ++u) take_group(Bf[u], (t0 + 1) * T + u * 64 * EPL + lane * EPL, m[1]);
    C.g = quick_threshold<NTHR, EPL>(S, m[0], m[1], fin, ranks, V, (unsigned)a.F.list_cap, samp, complete);
    C.y_g = R.greedy ? C.g : C.g / R.tau;
  } else {
  float a1 = -INFINITY, a2 = -INFINITY, a3 = -INFINITY;  // three largest values per lane
  auto take_group = [&](const Raw& X, int idx0) {
    float z[EPL];
    Raw Y = X;
    asm volatile("" : "+v"(Y));
    sample_group<DT>(Y, idx0, H, z);
#pragma unroll
    for (int e = 0; e < EPL; ++e) {  // sorted insertion: the median of two neighbours and the new value is the lower one's successor
      a3 = __builtin_amdgcn_fmed3f(a2, a3, z[e]);
      a2 = __builtin_amdgcn_fmed3f(a1, a2, z[e]);
      a1 = fmaxf(a1, z[e]);
    }
  };
#pragma unroll
  for (int u = 0; u < UNR; ++u) take_group(A[u], t0 * T + u * 64 * EPL + lane * EPL);
#pragma unroll
  for (int u = 0; u < UNR; ++u) take_group(Bf[u], (t0 + 1) * T + u * 64 * EPL + lane * EPL);
  {
    const float r_w = (float)r_samp / (float)NWV;
    const unsigned q = min((unsigned)(SPW * 3 / 4), (unsigned)ceilf(r_w + 3.0f * sqrtf(r_w) + 2.0f));
    const uint32_t k3[3] = {fkey(a1), fkey(a2), fkey(a3)};
    // every lane's largest is >= the smallest of the lanes' largest: at least 64 >= q keys qualify
    // (-inf is never kept: a wave short of q finite columns hands all of them on)
    const uint32_t Kw = max(KEY_NEG_INF + 1u, wave_threshold<3>(k3, q, q / 4u + 1u, wave_min_u32(k3[0]), wave_max_u32(k3[0])));
    if (lane < SPW) samp[wave * SPW + lane] = 0u;
    unsigned have = 0;
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      const u64 m = __ballot(k3[j] >= Kw);
      const unsigned p = have + lanes_before(m);
      if (((m >> lane) & 1ull) && p < (unsigned)SPW) samp[wave * SPW + p] = k3[j];
      have = min(have + (unsigned)__popcll(m), (unsigned)SPW);
    }
    const float wp = wave_max(a1);
    if (lane == 0) { S.wmax[wave] = wp; S.wcnt[wave] = have | (have < q ? SHORT_WAVE : 0u); }
  }
  __syncthreads();
  if (wave == 0) {  // (one wave for all: a search by ballots keeps the scalar unit busy, which the row's waves share)
    constexpr int NS = (NWV * SPW) / 64;
    uint32_t ks[NS];
    unsigned total = 0;
    float Mp = S.wmax[0];
#pragma unroll
    for (int w = 0; w < NWV; ++w) { const unsigned c = S.wcnt[w]; total += c & (SHORT_WAVE - 1u); complete = complete || (c & SHORT_WAVE) != 0u; Mp = fmaxf(Mp, S.wmax[w]); }
    uint32_t kmn = 0xFFFFFFFFu, kmx = 0u;
#pragma unroll
    for (int j = 0; j < NS; ++j) { ks[j] = samp[j * 64 + lane]; kmx = max(kmx, ks[j]); if (ks[j]) kmn = min(kmn, ks[j]); }
    kmn = wave_min_u32(kmn); kmx = wave_max_u32(kmx);
    // Few finite columns in the sample (an allow-list masked the rest): the list takes all there are
    // instead of a prefix of them.  Before, such rows admitted the masked columns too, overflowed the list
    // and went to the general kernel (32 float32 rows of 128,256 columns, 8 of them with 2000 columns
    // left: the call 451 to 536 us, 106 so).
    complete = complete && total < r_samp;
    const unsigned need = max(1u, min(r_samp, total));
    // (all that was handed over: the smallest, where the search would end)
    float g = keyf(need == total ? min(kmn, kmx) : wave_threshold<NS>(ks, need, need / 8u + 1u, min(kmn, kmx), kmx));
    // A rank beyond what the waves hand over (a long top-k on a short row): the value there, from the slope between
    // the sample's largest value and the last one handed over, with a margin.  (Without, such rows were streamed
    // with a threshold that admits too few, and went to the general kernel after all.)
    if (R.k_on && !complete && r_samp > total && total >= 8u) {
      const float l2 = __builtin_amdgcn_logf((float)total);
      g -= 1.35f * (Mp - g) * (__builtin_amdgcn_logf((float)r_samp) - l2) / l2;
    }
    if (!R.greedy && !R.k_on && R.minp_on) {
      // min-p survivors lie within ln(min_p) of the row maximum, which is at least the sample's
      const float thr_lb = Mp / R.tau + (float)log((double)R.min_p);
      float gm = thr_lb * R.tau;
      gm = gm - fabsf(gm) * 1e-6f - 1e-30f;
      // (a row with few finite columns: the bound, and what lies below it need not be listed)
      if (complete && gm > LOWEST) { complete = false; g = gm; }
      else g = fmaxf(g, gm);
    }
    if (lane == 0) { S.g = g; S.q_step = complete ? 1 : 0; }
  }
  __syncthreads();
  // (the same in every lane: said so, the stream's tests on them stay scalar)
  complete = __builtin_amdgcn_readfirstlane(S.q_step) != 0;
  C.g = __uint_as_float((uint32_t)__builtin_amdgcn_readfirstlane((int)__float_as_uint(S.g)));
  C.y_g = R.greedy ? C.g : C.g / R.tau;
  }
  }
  {
    if (complete) { C.g = LOWEST; C.y_g = -INFINITY; }  // every finite column is listed, and certified
    C.inv_tau = 1.0 / (double)R.tau;
    C.need_sum = R.need_sum && !complete;  // (nothing lies below the list)
    C.l2e_tau = (float)(1.4426950408889634 / (double)R.tau);
  }
  // A threshold within the double-precision masses' reach of the row's maximum, as far as the sample knows it.
  // (Only where such a row is queued: taken with the threshold, it cost every row of a call 1 us.)
  auto below_sample_top = [&]() -> float {
    float g = C.g;
#pragma unroll 1
    for (int w = 0; w < NWV; ++w) g = fmaxf(g, S.wmax[w] - F64_MARGIN * R.tau);
    return g;
  };
  if (straight) {  // (without truncation the threshold is only the reference of the masses)
    if (!queue_wide(straight_mode, true, a.f64 ? below_sample_top() : C.g, -INFINITY) && tid == 0) queue_pending(a, row);
    return;
  }
  const bool minp_only = !R.greedy && !R.k_on && !R.p_on && R.minp_on;
  // the history mask is dead from here (every wave passed the barrier above after its last lookup):
  // the region becomes the candidate list
  uint32_t* lz = reinterpret_cast<uint32_t*>(lds);
  const unsigned cap = (unsigned)a.F.list_cap;
  uint32_t* li = lz + cap;
  u64 below_mass = 0ull;  // this thread's share of the mass below g (integer: the total is order-free)
  // ---- the stream (raw logits) ----
  // Every wave starts with its two sample tiles (in registers).  With four waves per row each then
  // takes the rest of its contiguous share of the row; with more, the other tiles are handed out one
  // at a time from a counter, so that the waves finish together whatever each of them met (measured:
  // 1 % slower at four waves, 1.5 to 3 % faster at eight).  No result depends on which wave took
  // which tile (the list is ranked by value and id, the masses are integers).
  constexpr bool HAND_OUT = NWV > 4;
  const unsigned n_dyn = (unsigned)max(nfull - 2 * NWV, 0);
  int t_own = t0 + 2;  // contiguous shares: this wave's next tile
  auto grab = [&]() -> int {  // the next tile for this wave, -1 if none; the same in every lane
    if constexpr (!HAND_OUT) {
      const int t = t_own++;
      return t < t_end ? t : -1;
    } else {
      unsigned c = 0u;
      if (lane == 0) c = atomicAdd(&S.tile_ctr, 1u);
      c = (unsigned)__builtin_amdgcn_readfirstlane((int)c);
      if (c >= n_dyn) return -1;
      int t = (int)c;  // the c-th tile that is no wave's sample tile
#pragma unroll
      for (int w = 0; w < NWV; ++w) { const int s0 = (int)(((long long)w * nfull) / NWV); if (s0 <= t) t += 2; }
      return t;
    }
  };
  auto fill = [&](Raw (&X)[UNR], int t) {
#pragma unroll
    for (int u = 0; u < UNR; ++u) X[u] = Io<DT>::load(rowp + (size_t)t * T + u * 64 * EPL + lane * EPL);
  };
  {
    int tA = (!whole || t0 < t_end) ? t0 : -1, tB = whole ? -1 : t0 + 1;
    int nx = grab();
    if constexpr (sizeof(DT) == 2) {
      // two buffers in turn, each refilled as soon as it has been consumed, so no registers are
      // copied (bf16: 7 % faster on C5 than the rotation below, which in turn is 1.5 % faster for
      // float32 on C3)
      while (tA >= 0) {
        stream_tile<DT>(A, tA * T, C, S, lz, li, cap, below_mass);
        tA = nx;
        if (tA >= 0) { fill(A, tA); nx = grab(); }
        if (tB < 0) continue;
        stream_tile<DT>(Bf, tB * T, C, S, lz, li, cap, below_mass);
        tB = nx;
        if (tB >= 0) { fill(Bf, tB); nx = grab(); }
      }
    } else {
      if (!whole || tA >= 0) stream_tile<DT>(A, tA * T, C, S, lz, li, cap, below_mass);
      while (tB >= 0) {
#pragma unroll
        for (int u = 0; u < UNR; ++u) A[u] = Bf[u];
        tA = tB;
        tB = nx;
        if (tB >= 0) { fill(Bf, tB); nx = grab(); }
        stream_tile<DT>(A, tA * T, C, S, lz, li, cap, below_mass);
      }
    }
  }
  // the epilogue rebuilds the history tables: fetch the ids while the other waves finish
  int ids[IDR], tid_again = tid;  // (formed again: the entries' places, kept from the first fetch, spilled others)
  if constexpr (!WHOLE) asm volatile("" : "+v"(tid_again));
#pragma unroll
  for (int j = 0; j < IDR; ++j) { const int i = tid_again + j * NTHR; ids[j] = (h_active && (!stateful || R.need_sum) && i < nnz) ? hist_entry(i) : -1; }
  // ragged tail, element by element
  for (int idx = nfull * T + tid; idx < V; idx += NTHR) {
    const float zz = Io<DT>::one(rowp + idx);
    if (C.need_sum) below_mass += (u64)below_term_clamped(zz, C);
    if (!(zz < C.g)) {
      const unsigned slot = atomicAdd(&S.cand_count, 1u);
      if (slot < cap) { lz[slot] = __float_as_uint(zz); li[slot] = (uint32_t)idx; }
    }
  }
  __syncthreads();

  // ---- epilogue ----
  simple_row_diag dg;
  dg.alpha = __longlong_as_double(0x7FF8000000000000ll);
  dg.s_k = 0.0; dg.p_chosen = 0.0f; dg.n_survivors = 0; dg.flags = 0u; dg.reserved = 0u;
  if (a.hot_bits && a.hot_flags && *a.hot_flags) dg.flags |= SIMPLE_DIAG_BAD_HOT_SET;
  int rc = FIN_PENDING;
  const unsigned n = S.cand_count;
  // the stream added 2^28 for every column at or above g: all of them were counted for the list
  if (C.need_sum && tid == 0) below_mass -= (u64)n << 28;
  float g_ref = C.g;         // threshold for the sliced kernels
  float y_rel = -INFINITY;   // what masses are relative to there, if not to the threshold
  bool tables_live = false;  // the region holds the history tables
  // more columns at or above g than the list holds, and a cut that the whole-vocabulary routes find
  // without the list
  if (n > cap && !complete && (R.need_sum || minp_only)) {
    rc = FIN_WIDE;
    if (a.f64) g_ref = below_sample_top();
  }
  if (n <= cap) {
    // the list moves to registers; the region takes the history tables again
    float ez[PER]; uint32_t eid[PER];
#pragma unroll
    for (int j = 0; j < PER; ++j) {
      const unsigned i = (unsigned)tid + (unsigned)j * NTHR;
      ez[j] = (i < n) ? __uint_as_float(lz[i]) : -INFINITY;
      eid[j] = (i < n) ? li[i] : 0u;
    }
    __syncthreads();
    if ((whole || NTHR == 1024) && H.active && !stateful && !C.need_sum && (whole || n <= HASH_LIST_MAX)) {
      penalise_listed<NTHR, PER, IDR, WHOLE>(S, H, ez, eid, n, ids, hist, nnz, rh.n_prompt, V, lds);
      __syncthreads();
    } else if (H.active) {
      unsigned own = 0u;
      if (stateful) load_tables(true);
      else build_history<NTHR>(S, H, ids, hist, nnz, rh.n_prompt, V, own);
#pragma unroll
      for (int j = 0; j < PER; ++j) {
        const unsigned i = (unsigned)tid + (unsigned)j * NTHR;
        if (i < n) ez[j] = H.penalised_at(ez[j], (int)eid[j]);
      }
      if (C.need_sum) {
        // exact correction of the mass below g for the history columns (the stream summed their raw
        // values), once per distinct column: by the thread that first marked it when all ids sit in
        // registers, else by the thread that first claims the column's rank
        const bool by_claim = stateful || nnz > IDR * NTHR;  // (ready-made tables come without first-marker flags)
        uint32_t* claim = reinterpret_cast<uint32_t*>(lds + a.F.claim);
        if (by_claim) {
          zero16(claim, ((nnz + 31) / 32) * 4, tid, NTHR);
          __syncthreads();
        }
        auto claims = [&](int id) -> bool {  // true for exactly one of the entries that name this column
          if ((unsigned)id >= (unsigned)V) return false;
          const unsigned r = H.rank(id, H.bm[id >> 5]);
          const uint32_t bit = 1u << (r & 31u);
          return !(atomicOr(&claim[r >> 5], bit) & bit);
        };
        auto correct = [&](float z_raw, int id) {  // columns at or above g are in the list: their terms are settled there
          if (z_raw < C.g) {
            below_mass -= (u64)below_term(z_raw, C);
            below_mass += (u64)below_term(H.penalised_at(z_raw, id), C);
          }
        };
        if (by_claim) {
          own = 0u;
#pragma unroll
          for (int j = 0; j < IDR; ++j) if (tid + j * NTHR < nnz && claims(ids[j])) own |= 1u << j;
        }
        typename Io<DT>::Elem zr[IDR];  // (as loaded, all of them in flight: converted in its branch, each was waited for)
#pragma unroll
        for (int j = 0; j < IDR; ++j) zr[j] = Io<DT>::raw(rowp + (((own >> j) & 1u) ? ids[j] : 0));
#pragma unroll
        for (int j = 0; j < IDR; ++j) if ((own >> j) & 1u) correct(Io<DT>::cvt(zr[j]), ids[j]);
        // entries beyond the registers, four at a time (their trips to memory overlap)
        for (int i0 = tid + IDR * NTHR; i0 < nnz; i0 += 4 * NTHR) {
          int id4[4]; bool mine[4]; typename Io<DT>::Elem z4[4];
#pragma unroll
          for (int k = 0; k < 4; ++k) id4[k] = (i0 + k * NTHR < nnz) ? hist[i0 + k * NTHR] : -1;
#pragma unroll
          for (int k = 0; k < 4; ++k) mine[k] = claims(id4[k]);
#pragma unroll
          for (int k = 0; k < 4; ++k) z4[k] = Io<DT>::raw(rowp + (mine[k] ? id4[k] : 0));
#pragma unroll
          for (int k = 0; k < 4; ++k) if (mine[k]) correct(Io<DT>::cvt(z4[k]), id4[k]);
        }
      }
      __syncthreads();
    }
    // keys of the tempered values; listed columns that fell below g return to the mass below g
    uint32_t key[PER];
    bool err = false, peaked = false;
    uint32_t kloc = 0u;
    u64 mlist = 0ull, mcert = 0ull;  // mass (relative to the one at y_g) of the listed / certified columns
    const uint32_t key_g = fkey(C.y_g);
#pragma unroll
    for (int j = 0; j < PER; ++j) {
      const unsigned i = (unsigned)tid + (unsigned)j * NTHR;
      key[j] = 0u;
      if (i < n) {
        const float z = ez[j];
        if (z != z || z == INFINITY) err = true;
        else if (!(z < C.g)) {
          const float y = R.greedy ? z : tempered(z, C);  // the IEEE quotient z / tau
          if (y == INFINITY) err = true;
          else {
            key[j] = fkey(y);
            if (C.need_sum) {
              int b;
              const float w = mass_term(z, C, b);
              if (w > 2097152.0f) peaked = true;  // 2^21: far too peaked for a wide nucleus
              mlist += mass_fix(w);
              if (key[j] > key_g) mcert += mass_fix(w);
            }
          }
        } else if (C.need_sum) below_mass += (u64)below_term(z, C);
      }
      kloc = max(kloc, key[j]);
    }
    // What the branches below derive from an entry is formed there: carried across them all, it cost the instances
    // for rows listed whole 40 to 150 spilled registers (4 rows of 1024 columns 27.7 us, 22.4 so).
#pragma unroll
    for (int j = 0; j < PER; ++j) asm volatile("" : "+v"(key[j]), "+v"(eid[j]));
    kloc = wave_max_u32(kloc);  // (one atomic per wave)
    if (kloc && lane == 0) atomicMax(&S.kmax, kloc);
    if (complete) {
      uint32_t kmin = 0xFFFFFFFFu;
#pragma unroll
      for (int j = 0; j < PER; ++j) if (key[j] > key_g) kmin = min(kmin, key[j]);
      kmin = wave_min_u32(kmin);
      if (kmin != 0xFFFFFFFFu && lane == 0) atomicMin(&S.kmin, kmin);
    }
    if (err) atomicOr(&S.flags, SIMPLE_DIAG_ERROR | SIMPLE_DIAG_BAD_LOGIT);
    if (peaked) atomicOr(&S.flags, 1u << 30);
    __syncthreads();
    // mass below g (integer, exact) and the decision between the list and the kernels that follow
    u64 S_below_int = 0ull, M_list = 0ull, M_cert = 0ull;
    bool wide = false, ties_at_g = false;
    if (C.need_sum) {
      blk_sum3<NWV>(S, below_mass, mlist, mcert, S_below_int, M_list, M_cert);
      const u64 target = (u64)__double2ull_ru((double)R.top_p * (double)(M_list + S_below_int));
      // (a column more than 2^21 above g: these sums say nothing, the sorted list does)
      wide = !R.minp_on && M_cert < target && !((S.flags >> 30) & 1u);
      ties_at_g = wide && M_list >= target - (target >> 18);  // (the margin: this sum's error against the bins' one)
    }
    const double S_below = (double)S_below_int / (double)MSCALE;
    const uint32_t kmax = S.kmax;
    // Lower end of what the sliced kernels may take as above their threshold, below which they look for the cut: where the cut lies
    // among columns equal to g, just above these (WIDE_MAX).  (They gave such a row up and it went to the general kernel: one of 41,000
    // bfloat16 rows of 256,000 columns with penalties, every tenth call of 4096 rows; such a call 1765 us, 1027 so, 865 without such a row.)
    if (tid == 0) S.wmax[0] = ties_at_g ? C.y_g + (0.01f + 1e-6f * fabsf(C.y_g)) : -INFINITY;
    if (S.flags & SIMPLE_DIAG_ERROR) rc = FIN_DONE;
    else if (kmax <= key_g || kmax <= KEY_NEG_INF) rc = FIN_PENDING;
    else if (wide) {
      rc = FIN_WIDE;
      tables_live = true;
    } else {
      // certified entries: tempered value strictly above fl(g / tau).  One reservation per wave and round (a wave's
      // 64 additions to one word take their turns).  A short list goes to LDS here.
      u64* mc = reinterpret_cast<u64*>(lds);
      {
        uint32_t* base = reinterpret_cast<uint32_t*>(lds + SORT_BASE);
        for (int i = tid; i < SORT_NB; i += NTHR) base[i] = 0u;
      }
      unsigned nul = 0;
#pragma unroll
      for (int j = 0; j < PER; ++j) {
        if ((unsigned)(j * NTHR) >= n) break;
        const bool cert = key[j] > key_g;
        const u64 m = __ballot(cert);
        nul += (unsigned)__popcll(__ballot(key[j] != 0u)) - (unsigned)__popcll(m);
        if (m == 0ull) { key[j] = 0u; continue; }
        unsigned slot = 0u;
        if (lane == 0) slot = atomicAdd(&S.n2, (unsigned)__popcll(m));
        slot = (unsigned)__builtin_amdgcn_readfirstlane((int)slot) + lanes_before(m);
        if (cert && slot < (unsigned)COUNT_MAX) mc[slot] = composite(key[j], eid[j]);
        if (!cert) key[j] = 0u;
      }
      if (nul && lane == 0) atomicAdd(&S.nunc, nul);
      __syncthreads();
      const unsigned n_cert = S.n2, n_unc = S.nunc;
      const int k_asked = R.top_k;  // a complete list shorter than k: the rest of the prefix has no mass
      if (complete && R.k_on) R.top_k = min(R.top_k, (int)n_cert);
      if (R.k_on && !R.greedy && n_cert < (unsigned)R.top_k) rc = FIN_PENDING;  // the sampled threshold admitted too few
      else if (R.greedy) {  // the first of the total order
        u64 cmax = 0ull, zero = 0ull;
        unsigned z0 = 0u, z1 = 0u;
#pragma unroll
        for (int j = 0; j < PER; ++j) { const u64 c = key[j] ? composite(key[j], eid[j]) : 0ull; cmax = c > cmax ? c : cmax; }
        blk_reduce<NWV>(S, z0, z1, cmax, zero);
        if (tid == 0) S.out_id = (int)(0xFFFFFFFFu - (uint32_t)cmax);
        dg.n_survivors = 1; dg.p_chosen = 1.0f;
        rc = FIN_DONE;
      } else {
        const float y_max = keyf(kmax);
        Listed L = {n_cert, n_unc, y_max, key_g, C.g, S_below, false, 0u};
        uint32_t key_thr = 0u;
        if (R.minp_on) {
          key_thr = fkey(y_max + (float)log((double)R.min_p));
          L.m_cert = key_thr > key_g;
        }
        if (n_cert <= (unsigned)COUNT_MAX) sort_by_counting<NTHR>(S, n_cert, y_max, key_thr, lds);
        else if (!R.k_on && n_cert > (unsigned)SORT_MAX) L.n = 0u;
        else L.n = sort_by_buckets<NTHR, PER>(S, R, key, eid, n_cert, y_max, complete ? S.kmin : key_g, key_thr, lds);
        __syncthreads();
        if (L.n) {
          if (R.k_on) L.n = min(L.n, (unsigned)R.top_k);
          L.n_minp = S.memb;
          if (L.n <= 64u) {
            if (wave == 0) decide_wave(S, R, L, reinterpret_cast<const u64*>(lds + SORT_OUT), hot_bits);
          } else decide_block<NTHR>(S, R, L, lds, hot_bits);
          __syncthreads();
          rc = S.e_rc;
          if (rc == FIN_DONE) {
            dg.n_survivors = (int)S.e_n;
            dg.s_k = (double)S.e_skfix / WSCALE;
            if (hot_bits != nullptr) {
              dg.alpha = (double)S.e_SH / (double)S.e_SK;
              dg.flags |= SIMPLE_DIAG_SHVS | (S.e_acc ? SIMPLE_DIAG_ACCEPTED : 0u);
            }
            dg.p_chosen = (float)((double)S.out_w / (double)S.e_SK);
            if (S.out_id < 0) rc = FIN_PENDING;
          }
        } else if (n_cert <= (unsigned)a.F.long_cap) {
          // too many, or crowded by ties: keys and ids go back to the region, the bucket tables behind them
          const unsigned lcap = (unsigned)a.F.long_cap;
          uint32_t* lk = reinterpret_cast<uint32_t*>(lds);
          uint32_t* lid = lk + lcap;
          __syncthreads();
          if (tid == 0) { S.n2 = 0u; S.memb = 0u; S.bk = -1; S.bp = -1; }
          __syncthreads();
#pragma unroll
          for (int j = 0; j < PER; ++j) {
            if (key[j]) { const unsigned slot = atomicAdd(&S.n2, 1u); lk[slot] = key[j]; lid[slot] = eid[j]; }
          }
          __syncthreads();
          rc = finalize_long<NTHR, WHOLE>(S, R, n_cert, n_unc, kmax, key_g, complete ? S.kmin : key_g, C.need_sum, C.g, S_below, lk, lid, lds + (size_t)lcap * 8u, hot_bits, dg);
        }
      }
      // -inf columns without mass among the survivors of a count alone, or where nothing is truncated
      if (complete && !R.greedy && !R.p_on && !R.minp_on) dg.n_survivors = R.k_on ? k_asked : V;
      if (R.all && V > KMAXF) dg.flags |= SIMPLE_DIAG_WIDE;  // (K_b is all of V)
    }

    // ---- a cut below the list's reach: the row goes to the kernels that follow ----
    // (masses there are relative to the threshold and reach 2^21 above it: where the row maximum stands
    // higher, the threshold is moved up to e^10 below it, and above a bucket of ties that holds the cut; above ties
    // at g alone, masses are relative to the maximum)
    if (rc == FIN_WIDE) {
      __syncthreads();
      const float y_m = keyf(kmax);
      const float y_ref = (a.f64 || y_m - C.y_g > 13.5f || (S.wmax[0] > -INFINITY && !ties_at_g)) ? y_m - F64_MARGIN : -INFINITY;
      if (ties_at_g && !(y_ref > C.y_g)) y_rel = y_m;
      g_ref = fmaxf(g_ref, fmaxf(y_ref, S.wmax[0]) * R.tau);
    }
  }
  if (rc == FIN_WIDE) {
    if (!whole && queue_wide(R.need_sum ? WIDE_TOP_P : WIDE_MIN_P, tables_live, g_ref, y_rel)) return;  // (no such kernel runs behind rows listed whole)
    rc = FIN_PENDING;  // no free slot: the general kernel takes the row
  }
  if (tid == 0) {
    if (rc != FIN_DONE) {
      queue_pending(a, row);
    } else {
      const unsigned f = S.flags & 0x3FFFFFFFu;
      const bool err = (f & SIMPLE_DIAG_ERROR) != 0u;
      a.out[row] = err ? -1 : S.out_id;
      dg.flags |= f | (R.greedy ? SIMPLE_DIAG_GREEDY : 0u);
      if (err) dg.p_chosen = 0.0f;
      if (a.diag) a.diag[row] = dg;
      if (a.stats) stats_add(a.stats, dg.flags, dg.alpha);
      write_decision(a, row, err ? -1 : S.out_id, dg.p_chosen, R.greedy);
    }
  }
}

}  // namespace fast

}  // namespace simple
namespace simple {

template <typename DT, bool STATEFUL, bool WHOLE>
static hipError_t launch_fast_instance(const SampleArgs& a, hipStream_t st) {
  const dim3 grid((unsigned)a.B);
  if (a.F.threads == 256) hipLaunchKernelGGL((fast::fast_rows_kernel<DT, 256, STATEFUL, WHOLE>), grid, dim3(256), a.F.total, st, a);
  else if (a.F.threads == 512) hipLaunchKernelGGL((fast::fast_rows_kernel<DT, 512, STATEFUL, WHOLE>), grid, dim3(512), a.F.total, st, a);
  else hipLaunchKernelGGL((fast::fast_rows_kernel<DT, 1024, STATEFUL, WHOLE>), grid, dim3(1024), a.F.total, st, a);
  return hipGetLastError();
}
template <typename DT>
static hipError_t launch_fast_dtype(const SampleArgs& a, hipStream_t st) {
  if (a.F.whole) return a.st_rec ? launch_fast_instance<DT, true, true>(a, st) : launch_fast_instance<DT, false, true>(a, st);
  return a.st_rec ? launch_fast_instance<DT, true, false>(a, st) : launch_fast_instance<DT, false, false>(a, st);
}
hipError_t launch_fast(const SampleArgs& a, int dtype, hipStream_t st) {
  return dtype == SIMPLE_F32 ? launch_fast_dtype<float>(a, st) : launch_fast_dtype<uint16_t>(a, st);
}

template <typename DT, int NTHR>
static hipError_t set_max_lds_instances(unsigned bytes) {
  const void* fns[4] = {
    reinterpret_cast<const void*>(fast::fast_rows_kernel<DT, NTHR, false, false>), reinterpret_cast<const void*>(fast::fast_rows_kernel<DT, NTHR, true, false>),
    reinterpret_cast<const void*>(fast::fast_rows_kernel<DT, NTHR, false, true>), reinterpret_cast<const void*>(fast::fast_rows_kernel<DT, NTHR, true, true>)};
  for (const void* f : fns) {
    const hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}
hipError_t set_max_lds_fast(unsigned bytes) {
  hipError_t (*const set[6])(unsigned) = {set_max_lds_instances<float, 256>, set_max_lds_instances<float, 512>, set_max_lds_instances<float, 1024>,
                                          set_max_lds_instances<uint16_t, 256>, set_max_lds_instances<uint16_t, 512>, set_max_lds_instances<uint16_t, 1024>};
  for (auto f : set) {
    const hipError_t e = f(bytes);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace simple
