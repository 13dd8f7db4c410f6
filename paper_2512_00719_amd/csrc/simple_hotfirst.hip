// Speculative hot-vocab sampling that reads only the hot columns on acceptance (paper section 5.3).
//
// The paper's samplers draw on a small hot set and fall back to the tail only on rejection, with the
// weights w = exp(z' - max) "pre-computed on GPUs when writing logits".  On a GPU the row mass is the
// obstacle: alpha_b = S_H / (S_H + S_T) needs the tail's mass S_T, and summing the tail means
// reading it.  This kernel takes S_T from the producer of the logits instead: the vocabulary is laid
// out hot-first (the hot set is the columns [0, H)), and every row comes with the maximum of its
// tail logits and the sum of exp((z - tail_max) / tau) over the tail.  A row whose draw is accepted
// then costs H columns; only a rejected row streams its V - H tail columns (the cost model of
// section 5.4: c H + c0 on acceptance, the rest of the vocabulary on rejection).
//
// Rows the kernel takes itself: temperature > 0 and no truncation (no top-k, top-p, min-p) — with a
// survivor set that is all of V, Eq. (7) needs nothing of the tail but its mass.  (A truncated
// row's survivor set may reach into the tail, and which tail columns survive cannot be told from a
// maximum and a sum.)  Every other row is served with the hot set [0, H) as a membership mask: in
// a bfloat16 call the pattern-count kernel, which runs ahead of this one, completes the truncated
// rows without penalties; the rest is queued for the general kernel.  So each row of the call gets
// the ids of the speculative sampler as the definition over the whole row gives them.
//
// One workgroup per row for the hot columns and the acceptance; a rejected row is queued, and its tail is cut
// into tiles that spread over the whole chip (a kernel for the tile sums, one for the draw).  Masses are relative to the row maximum (the stable softmax numerator of Eq.
// (2)); a 16-byte group of columns is summed in double precision in column order and rounded once to a
// 2^44 fixed-point integer, and everything above a group adds integers, so no sum depends on the order
// of the additions.  The inverse CDF runs in ascending token id: per tile of 2048 groups a sum, the
// tile that holds the target, the group in it, the column in the group.
//
// What bounds it: an accepted row is one trip through memory for its hot columns and a chain of
// barriers.  A rejected row's tail, 12 vector instructions a column, took one compute unit 45 us, and the
// launch ended with those rows while most of the chip was idle: 1024 rows of 201,088 bfloat16 columns with
// H = 8192, 82 of them rejected, 68.6 us a call; 41 with the tails' tiles spread out (984 workgroups).
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "simple_rowdev.hpp"

namespace simple {
namespace hotfirst {

using fast::FS;
using fast::Io;
using fast::u32x4;
using fast::u64;

// Threads of a workgroup.  A row's hot columns: 256, so that six rows share a compute unit and hide each
// other's barriers (3548 bfloat16 rows, H = 8192: 108 us a call with 512, 63 so).  A tail's tile: 512.
constexpr int ROW_T = 256, TAIL_T = 512;
constexpr int HU = 4;              // 16-byte groups per thread and tile
constexpr int STEP = 256;          // the hot set is a whole number of steps of 256 groups
constexpr int MAX_STEPS = 1024;    // steps of hot set or tail (V below 2^20 with float32, 2^21 with bfloat16)
constexpr int max_tiles(int threads) { return MAX_STEPS * STEP / (threads * HU); }  // of whole steps
constexpr int MAX_TAIL_TILES = max_tiles(TAIL_T) + 1;                              // (a tail may end in part of one)
static_assert(max_tiles(ROW_T) <= ROW_T && MAX_TAIL_TILES <= TAIL_T, "one tile per thread in the scan over tiles");
// A tail of up to 128 KB is streamed by its row's own workgroup, and so is any tail of a batch of up to three rows:
// there the two launches for the tails' tiles cost more than the 10 us they save now and then.
constexpr int OWN_TAIL_BYTES = 128 << 10, OWN_TAIL_ROWS = 3;
constexpr int64_t OWN_TAIL_MAX = (int64_t)(max_tiles(ROW_T) - 1) * ROW_T * HU * 16;  // tiles that a row's workgroup can index
static_assert(OWN_TAIL_BYTES < OWN_TAIL_MAX, "a short tail fits the tile sums");

// Tempered value (the IEEE quotient z / tau) and mass exp(y - y_max) of a column: float32 exponential
// with a split log2(e).
template <typename DT> using Raw = typename Io<DT>::Raw;
__device__ __forceinline__ float mass_of(float z, double inv_tau, float y_max) {
  const float d = (float)((double)z * inv_tau) - y_max;
  return __builtin_amdgcn_exp2f(fmaf(d, fast::L2E_HI, d * fast::L2E_LO));
}
__device__ __forceinline__ u64 to_fix(double m) { return (u64)__double2ull_rn(m * fast::WSCALE); }

// The columns [c0, c1) of a row as 16-byte groups (c0 is a whole number of them); the columns behind the
// last whole group make one more, filled up with -inf (no mass).
template <typename DT, int HT>
struct Span {
  static constexpr int EPL = Io<DT>::EPL;
  static constexpr uint32_t NONE = sizeof(DT) == 4 ? 0xFF800000u : 0xFF80FF80u;  // -inf
  const DT* p;
  int c0, whole, n_tiles;
  Raw<DT> last;
  __device__ __forceinline__ Span(const DT* rowp, int c0_, int c1) {
    c0 = c0_; p = rowp + c0;
    whole = (c1 - c0) / EPL;
    n_tiles = ((c1 - c0 + EPL - 1) / EPL + HT * HU - 1) / (HT * HU);
    uint32_t w[4] = {NONE, NONE, NONE, NONE};
#pragma unroll 1
    for (int i = c1 - c0 - 1; i >= whole * EPL; --i) {  // they move in from the low end
      if constexpr (sizeof(DT) == 4) { w[3] = w[2]; w[2] = w[1]; w[1] = w[0]; w[0] = __float_as_uint(p[i]); }
      else {
        w[3] = (w[3] << 16) | (w[2] >> 16); w[2] = (w[2] << 16) | (w[1] >> 16); w[1] = (w[1] << 16) | (w[0] >> 16);
        w[0] = (w[0] << 16) | (uint32_t)p[i];
      }
    }
    last = __builtin_bit_cast(Raw<DT>, u32x4{w[0], w[1], w[2], w[3]});
  }
};
// A thread's groups of one tile: group tile * HT * HU + u * HT + tid.
template <typename DT>
struct Tile { Raw<DT> r[HU]; };
template <typename DT, int HT>
__device__ __forceinline__ void tile_load(Tile<DT>& T, const Span<DT, HT>& C, int tile) {
  const int g0 = tile * HU * HT + (int)threadIdx.x;
  const Raw<DT>* q = reinterpret_cast<const Raw<DT>*>(C.p);
  if ((tile + 1) * HU * HT <= C.whole) {
#pragma unroll
    for (int u = 0; u < HU; ++u) T.r[u] = fast::as_global(q)[g0 + u * HT];
  } else {
    const Raw<DT> none = __builtin_bit_cast(Raw<DT>, u32x4{Span<DT, HT>::NONE, Span<DT, HT>::NONE, Span<DT, HT>::NONE, Span<DT, HT>::NONE});
#pragma unroll
    for (int u = 0; u < HU; ++u) {
      const int g = g0 + u * HT;
      T.r[u] = g == C.whole ? C.last : none;
      if (g < C.whole) T.r[u] = fast::as_global(q)[g];
    }
  }
}
// Mass of one group, as summed everywhere; a NaN or +inf among its columns makes `sum` one.
template <typename DT>
__device__ __forceinline__ u64 group_mass(const Raw<DT>& r, double inv_tau, float y_max, double& sum) {
  float z[Io<DT>::EPL];
  Io<DT>::unpack(r, z);
  sum = 0.0;
#pragma unroll
  for (int e = 0; e < Io<DT>::EPL; ++e) sum += (double)mass_of(z[e], inv_tau, y_max);
  return to_fix(sum);
}
// Sums of the masses of columns [c0, c1) by tile into tsum[]; returns (all threads) their total.  bad is
// raised for a NaN or +inf tempered value.  `first`: the first tile, already loaded; the next tile is
// in flight while one is summed.
template <typename DT, int HT>
__device__ __forceinline__ u64 tile_masses(const Tile<DT>& first, const Span<DT, HT>& C, double inv_tau, float y_max, u64* tsum, FS& S, bool& bad) {
  const int tid = threadIdx.x, lane = tid & 63;
  const int n_tiles = C.n_tiles;
  for (int i = tid; i < n_tiles; i += HT) tsum[i] = 0ull;
  __syncthreads();
  u64 total = 0ull;
  double check = 0.0;
  Tile<DT> T = first;
  for (int i = 0; i < n_tiles; ++i) {
    Tile<DT> N = T;
    if (i + 1 < n_tiles) tile_load<DT, HT>(N, C, i + 1);
    u64 m = 0ull;
#pragma unroll
    for (int u = 0; u < HU; ++u) {
      double s;
      m += group_mass<DT>(T.r[u], inv_tau, y_max, s);
      check += s;
      __builtin_amdgcn_sched_barrier(0);  // one group at a time: eight columns are enough to fill the pipe, four groups spill
    }
    const u64 w = wave_sum(m);
    if (lane == 0 && w) atomicAdd(&tsum[i], w);
    total += m;
    T = N;
  }
  bad = bad || !(check < (double)INFINITY);
  return fast::blk_sum_u64<HT / 64>(S, total);  // barriers inside: the tile sums are complete after it
}

// The column of [c0, c1) at which the running mass (ascending id) first exceeds tfix; its mass in w_out.
template <typename DT, int HT>
__device__ __forceinline__ int locate(const Span<DT, HT>& C, double inv_tau, float y_max, const u64* tsum, u64 tfix, FS& S, u64 (&part)[HU][HT / 64], u64& w_out) {
  constexpr int HWV = HT / 64;
  constexpr int EPL = Io<DT>::EPL;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int n_tiles = C.n_tiles;
  if (tid == 0) { S.bd = -1; S.out_id = -1; S.out_w = 0ull; }
  __syncthreads();
  {
    const u64 m = tid < n_tiles ? tsum[tid] : 0ull;
    unsigned ce, ct; u64 me, mt;
    fast::blk_excl_scan2<HWV>(S, 0u, m, ce, me, ct, mt);
    if (m > 0ull && me <= tfix && me + m > tfix) { S.bd = tid; S.mab_d = me; }
  }
  __syncthreads();
  const int tile = S.bd;
  if (tile < 0) return -1;
  Tile<DT> T;
  tile_load<DT, HT>(T, C, tile);
  u64 g[HU], incl[HU];
#pragma unroll
  for (int u = 0; u < HU; ++u) {
    double s;
    g[u] = group_mass<DT>(T.r[u], inv_tau, y_max, s);
    incl[u] = wave_incl_scan(g[u]);
    if (lane == 63) part[u][wave] = incl[u];
    __builtin_amdgcn_sched_barrier(0);
  }
  __syncthreads();
  u64 base = S.mab_d, start = 0ull;
  Raw<DT> r = T.r[0];
  int hit = -1;  // the group that holds the target, if it is one of this thread's
#pragma unroll
  for (int u = 0; u < HU; ++u) {
    u64 before = base;
#pragma unroll
    for (int w = 0; w < HWV; ++w) { const u64 x = part[u][w]; if (w < wave) before += x; base += x; }
    const u64 lo = before + incl[u] - g[u];
    if (g[u] > 0ull && lo <= tfix && lo + g[u] > tfix) { hit = u; start = lo; r = T.r[u]; }
  }
  if (hit >= 0) {
    float z[EPL];
    Io<DT>::unpack(r, z);
    double sum = 0.0;
    u64 lo = 0ull;
#pragma unroll
    for (int e = 0; e < EPL; ++e) {
      const double m = (double)mass_of(z[e], inv_tau, y_max);
      sum += m;
      const u64 hi = to_fix(sum);  // the last one is the group's mass
      if (start + lo <= tfix && start + hi > tfix) { S.out_id = C.c0 + ((tile * HU + hit) * HT + tid) * EPL + e; S.out_w = to_fix(m); }
      lo = hi;
    }
  }
  __syncthreads();
  w_out = S.out_w;
  return S.out_id;
}

// What the kernels behind this one need of a rejected row (a queue record), and its workspace slot.
struct Rejected { uint32_t row, flags; float y_max; uint32_t unused; u64 s_h; double alpha; u64 pad[4]; };
static_assert(sizeof(Rejected) == 64, "queue record size");
struct TailSums { u64 tsum[MAX_TAIL_TILES]; uint32_t bad[MAX_TAIL_TILES]; };  // per tile of the tail; bad: a NaN or +inf among its columns
static_assert(sizeof(TailSums) <= WIDE_SLOT_FIXED, "workspace slot size");
__device__ __forceinline__ Rejected* rejected(const SampleArgs& a) { return reinterpret_cast<Rejected*>(a.wq + fast::WQ_HEAD); }
__device__ __forceinline__ TailSums* tail_sums(const SampleArgs& a, unsigned slot) { return reinterpret_cast<TailSums*>(a.wws + (size_t)slot * a.ws_stride); }

// The results of a row decided here.
__device__ __forceinline__ void write_row(const SampleArgs& a, int row, int id, uint32_t flags, double alpha, u64 w_id, u64 S_K) {
  const bool err = (flags & SIMPLE_DIAG_ERROR) != 0u;
  simple_row_diag dg;
  dg.alpha = alpha; dg.s_k = 0.0; dg.n_survivors = err ? 0 : a.V; dg.reserved = 0u;
  dg.flags = flags;
  if (a.hot_flags && *a.hot_flags) dg.flags |= SIMPLE_DIAG_BAD_HOT_SET;
  dg.p_chosen = err ? 0.0f : (float)((double)w_id / (double)S_K);
  a.out[row] = err ? -1 : id;
  if (a.diag) a.diag[row] = dg;
  if (a.stats) stats_add(a.stats, dg.flags, dg.alpha);
  write_decision(a, row, err ? -1 : id, dg.p_chosen, false);
}
__device__ __forceinline__ void leave_pending(const SampleArgs& a, int row) {
  const unsigned slot = atomicAdd(&a.pend[0], 1u);
  a.pend[2 + slot] = (uint32_t)row;
  a.out[row] = PENDING;
}

template <typename DT>
__global__ __launch_bounds__(ROW_T, 6) void hot_first_rows_kernel(const SampleArgs a, int H, const simple_tail_stats* __restrict__ tail, bool own_tail) {
  constexpr int EPL = Io<DT>::EPL, HT = ROW_T, HWV = HT / 64;
  __shared__ FS S;
  __shared__ u64 tsum[max_tiles(ROW_T)];
  __shared__ u64 part[HU][HWV];
  const int tid = threadIdx.x;
  const int row = blockIdx.x;
  const int V = a.V;
  const DT* rowp = reinterpret_cast<const DT*>(a.logits) + (size_t)row * (size_t)a.stride;
  const simple_row_params par = a.params[row];
  const simple_tail_stats ts = tail[row];
  // the pattern-count kernel, when it ran before this one, has left NOT_TAKEN on every row that is still to do
  if (a.pattern_on && a.out[row] != NOT_TAKEN) return;
  const bool plain = hot_first_plain(par, V);
  if (!plain) {  // truncated, penalised, greedy or invalid rows: the general kernel, with [0, H) as the hot set
    if (tid == 0) leave_pending(a, row);
    return;
  }
  Tile<DT> T0;  // the first tile of the hot columns (all of them up to 8192 or 16,384): read once, used for the maximum and the masses
  const Span<DT, HT> hot(rowp, 0, H);
  tile_load<DT, HT>(T0, hot, 0);
  const double inv_tau = 1.0 / (double)par.temperature;
  double u[3];
  row_uniforms(a.seed, a.row_offset + (uint64_t)row, a.step, u);
  // ---- maximum of the hot columns, then of the row ----
  uint32_t kmax = KEY_NEG_INF;
  bool bad = false;
  auto take_max = [&](const Tile<DT>& T) {
#pragma unroll
    for (int q = 0; q < HU; ++q) {
      float z[EPL];
      Io<DT>::unpack(T.r[q], z);
#pragma unroll
      for (int e = 0; e < EPL; ++e) { bad = bad || (z[e] != z[e]); kmax = max(kmax, fkey(z[e])); }
    }
  };
  take_max(T0);
  for (int i = 1; i < hot.n_tiles; ++i) { Tile<DT> T; tile_load<DT, HT>(T, hot, i); take_max(T); }
  kmax = fast::wave_max_u32(kmax);
  if (tid == 0) { S.kmax = KEY_NEG_INF; S.flags = 0u; }
  __syncthreads();
  if ((tid & 63) == 0) atomicMax(&S.kmax, kmax);
  __syncthreads();
  const bool has_tail = H < V;
  const float z_hot = keyf(S.kmax);
  const float z_top = has_tail ? fmaxf(z_hot, ts.tail_max) : z_hot;      // tempering is monotone: the maximum is taken on z
  const float y_max = (float)((double)z_top * inv_tau);
  const float y_tmax = (float)((double)ts.tail_max * inv_tau);
  if (has_tail && (ts.tail_max != ts.tail_max || ts.tail_max == INFINITY || !(ts.tail_sum >= 0.0) || ts.tail_sum == (double)INFINITY)) bad = true;
  if (y_max == INFINITY || z_top == -INFINITY) bad = true;               // overflow of z / tau, or nothing to draw
  // ---- hot mass by tile, tail mass from the caller's statistics (Eq. (7)) ----
  const u64 S_H = tile_masses<DT, HT>(T0, hot, inv_tau, y_max, tsum, S, bad);
  if (bad) atomicOr(&S.flags, SIMPLE_DIAG_ERROR | SIMPLE_DIAG_BAD_LOGIT);
  __syncthreads();
  uint32_t flags = SIMPLE_DIAG_SHVS;
  double alpha = __longlong_as_double(0x7FF8000000000000ll);
  int id = -1;
  u64 w_id = 0ull, S_K = 0ull;
  if (!(S.flags & SIMPLE_DIAG_ERROR)) {
    u64 S_T = 0ull;
    if (has_tail && ts.tail_sum > 0.0) S_T = (u64)__double2ull_rn(ts.tail_sum * exp((double)y_tmax - (double)y_max) * fast::WSCALE);
    S_K = S_H + S_T;
    const bool pick_hot = (S_H > 0ull) && (u[1] * (double)S_K <= (double)S_H);   // accept iff u <= alpha_b (Eq. (8))
    alpha = S_K ? (double)S_H / (double)S_K : 0.0;
    if (pick_hot) {
      flags |= SIMPLE_DIAG_ACCEPTED;
      u64 tfix = (u64)__double2ull_rd(u[0] * (double)S_H);
      if (tfix >= S_H) tfix = S_H - 1ull;
      id = locate<DT, HT>(hot, inv_tau, y_max, tsum, tfix, S, part, w_id);
    } else if (own_tail) {  // rejected: the tail proposal r of Eq. (8), over the columns not read yet
      bool bad_t = false;
      const Span<DT, HT> rest(rowp, H, V);
      tile_load<DT, HT>(T0, rest, 0);
      const u64 S_T_exact = tile_masses<DT, HT>(T0, rest, inv_tau, y_max, tsum, S, bad_t);
      if (bad_t) atomicOr(&S.flags, SIMPLE_DIAG_ERROR | SIMPLE_DIAG_BAD_LOGIT);
      __syncthreads();
      if (!(S.flags & SIMPLE_DIAG_ERROR) && S_T_exact > 0ull) {
        u64 tfix = (u64)__double2ull_rd(u[2] * (double)S_T_exact);
        if (tfix >= S_T_exact) tfix = S_T_exact - 1ull;
        id = locate<DT, HT>(rest, inv_tau, y_max, tsum, tfix, S, part, w_id);
        S_K = S_H + S_T_exact;  // p~ of the drawn id over the masses as summed here
      }
    } else if (has_tail) {
      if (tid == 0) {
        const unsigned slot = atomicAdd(&a.wq[0], 1u);  // a launch has a slot for every row
        Rejected* r = rejected(a) + slot;
        r->row = (uint32_t)row; r->flags = flags | S.flags; r->y_max = y_max; r->s_h = S_H; r->alpha = alpha;
        a.out[row] = PENDING;
      }
      return;
    }
  }
  if (tid != 0) return;
  flags |= S.flags;
  if (!(flags & SIMPLE_DIAG_ERROR) && id < 0) leave_pending(a, row);  // nothing could be located (a class without mass): the general kernel decides
  else write_row(a, row, id, flags, alpha, w_id, S_K);
}

// The tile sums of the rejected rows' tails: items are (queued row, tile) pairs, taken in turn.
template <typename DT>
__global__ __launch_bounds__(TAIL_T, 4) void hot_tail_sums_kernel(const SampleArgs a, int H) {
  constexpr int HT = TAIL_T, HWV = HT / 64;
  __shared__ FS S;
  const int V = a.V;
  const unsigned n = min(fast::as_global(a.wq)[0], (unsigned)a.wide_slots);
  const int n_tiles = ((V - H + Io<DT>::EPL - 1) / Io<DT>::EPL + HT * HU - 1) / (HT * HU);
  for (unsigned it = blockIdx.x; it < n * (unsigned)n_tiles; it += gridDim.x) {
    const unsigned slot = it / (unsigned)n_tiles;
    const int tile = (int)(it % (unsigned)n_tiles);
    const Rejected* r = rejected(a) + slot;
    const int row = (int)r->row;
    const float y_max = r->y_max;
    const Span<DT, HT> rest(reinterpret_cast<const DT*>(a.logits) + (size_t)row * (size_t)a.stride, H, V);
    Tile<DT> T;
    tile_load<DT, HT>(T, rest, tile);
    const double inv_tau = 1.0 / (double)a.params[row].temperature;
    u64 m = 0ull, mx = 0ull;
    double check = 0.0;
#pragma unroll
    for (int u = 0; u < HU; ++u) {
      double s;
      m += group_mass<DT>(T.r[u], inv_tau, y_max, s);
      check += s;
      __builtin_amdgcn_sched_barrier(0);  // one group at a time
    }
    unsigned bad = !(check < (double)INFINITY) ? 1u : 0u, none = 0u;
    fast::blk_reduce<HWV>(S, bad, none, mx, m);  // barriers inside
    if (threadIdx.x == 0) { TailSums* t = tail_sums(a, slot); t->tsum[tile] = m; t->bad[tile] = bad; }
  }
}

// The draw from a rejected row's tail, one workgroup per row.
template <typename DT>
__global__ __launch_bounds__(TAIL_T, 4) void hot_tail_draw_kernel(const SampleArgs a, int H) {
  constexpr int HT = TAIL_T, HWV = HT / 64;
  __shared__ FS S;
  __shared__ u64 tsum[MAX_TAIL_TILES];
  __shared__ u64 part[HU][HWV];
  const int tid = threadIdx.x;
  const int V = a.V;
  const unsigned n = min(fast::as_global(a.wq)[0], (unsigned)a.wide_slots);
  for (unsigned slot = blockIdx.x; slot < n; slot += gridDim.x) {
    __syncthreads();
    const Rejected r = rejected(a)[slot];
    const int row = (int)r.row;
    const Span<DT, HT> rest(reinterpret_cast<const DT*>(a.logits) + (size_t)row * (size_t)a.stride, H, V);
    const TailSums* t = tail_sums(a, slot);
    u64 S_T = 0ull, mx = 0ull;
    unsigned bad = 0u, none = 0u;
    if (tid < rest.n_tiles) { S_T = t->tsum[tid]; bad = t->bad[tid]; tsum[tid] = S_T; }
    double u[3];
    row_uniforms(a.seed, a.row_offset + (uint64_t)row, a.step, u);
    fast::blk_reduce<HWV>(S, bad, none, mx, S_T);  // barriers inside: the tile sums are in place after it
    int id = -1;
    u64 w_id = 0ull;
    uint32_t flags = r.flags | (bad ? SIMPLE_DIAG_ERROR | SIMPLE_DIAG_BAD_LOGIT : 0u);
    if (!bad && S_T > 0ull) {
      u64 tfix = (u64)__double2ull_rd(u[2] * (double)S_T);
      if (tfix >= S_T) tfix = S_T - 1ull;
      id = locate<DT, HT>(rest, 1.0 / (double)a.params[row].temperature, r.y_max, tsum, tfix, S, part, w_id);
    }
    if (tid == 0) {
      if (!bad && id < 0) leave_pending(a, row);  // a class without mass: the general kernel decides
      else write_row(a, row, id, flags, r.alpha, w_id, r.s_h + S_T);  // p~ of the drawn id over the masses as summed here
    }
  }
}

// The membership mask of the hot set [0, H): V bits.
__global__ void hot_range_kernel(uint32_t* bits, int n_words, int H, uint32_t* flags) {
  const int w = blockIdx.x * blockDim.x + threadIdx.x;
  if (w < n_words) {
    const int lo = w << 5;
    bits[w] = lo + 32 <= H ? 0xFFFFFFFFu : (lo >= H ? 0u : ((1u << (H - lo)) - 1u));
  }
  if (w == 0) *flags = 0u;
}

}  // namespace hotfirst

hipError_t launch_hot_range(uint32_t* bits, uint32_t* flags, int V, int H, hipStream_t st) {
  const int n_words = (V + 31) >> 5;
  hipLaunchKernelGGL(hotfirst::hot_range_kernel, dim3((n_words + 255) / 256), dim3(256), 0, st, bits, n_words, H, flags);
  return hipGetLastError();
}

template <typename DT>
static void launch_hot_first_dtype(const SampleArgs& a, int H, const simple_tail_stats* tail, hipStream_t st) {
  // Two workgroups of 512 threads a compute unit fit: one resident round for the tails' tiles and draws.
  const unsigned round = 2u * (unsigned)a.n_cu, rows = (unsigned)a.B;
  const int64_t tail_bytes = (int64_t)(a.V - H) * (int64_t)sizeof(DT);
  const bool own_tail = tail_bytes <= hotfirst::OWN_TAIL_BYTES || (rows <= (unsigned)hotfirst::OWN_TAIL_ROWS && tail_bytes < hotfirst::OWN_TAIL_MAX);
  hipLaunchKernelGGL((hotfirst::hot_first_rows_kernel<DT>), dim3(rows), dim3(hotfirst::ROW_T), 0, st, a, H, tail, own_tail);
  if (own_tail) return;
  hipLaunchKernelGGL((hotfirst::hot_tail_sums_kernel<DT>), dim3(round), dim3(hotfirst::TAIL_T), 0, st, a, H);
  hipLaunchKernelGGL((hotfirst::hot_tail_draw_kernel<DT>), dim3(rows < round ? rows : round), dim3(hotfirst::TAIL_T), 0, st, a, H);
}

hipError_t launch_hot_first(const SampleArgs& a, int dtype, int H, const simple_tail_stats* tail, hipStream_t st) {
  if (dtype == SIMPLE_F32) launch_hot_first_dtype<float>(a, H, tail, st);
  else launch_hot_first_dtype<uint16_t>(a, H, tail, st);
  return hipGetLastError();
}

int hot_first_tile(int dtype) { return hotfirst::STEP * (dtype == SIMPLE_F32 ? 4 : 8); }
int hot_first_max_tiles() { return hotfirst::MAX_STEPS; }

}  // namespace simple
