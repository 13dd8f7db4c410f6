// Logit bias and allow-lists (paper section 5.2 lists allow-lists among the constraints that compose
// on the survivor set; its implementation section mentions optional biases).  They are applied by a
// pass of their own, ahead of the sampling call: out[b, v] = allowed(b, v) ? fl32(z[b, v] + bias(b, v))
// : -inf, written as float32 to a matrix the caller owns and then samples (dtype float32).  The
// sampling kernels are untouched by it: a call that uses no constraint pays nothing, one that does
// pays one more read and one write of its logits.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "simple_sample.h"

namespace simple {
namespace constraints {

constexpr int CT = 256;        // threads per workgroup
constexpr int CSL = 8192;      // columns per slice of a row, one workgroup each
constexpr int CG = CSL / 4 / CT;  // 4-column groups per thread and slice, all of them in flight at once
constexpr int AG = 4;          // allow-list ids in flight per thread
constexpr int BCAP = 2048;     // bias ids of a row that are staged in LDS; a longer list is read from memory
constexpr int64_t MAX_ALLOW_V = 96 * 1024 * 8;  // the boundary's limit for allow-lists (a V-bit mask of 96 KB once; the slices need none)
constexpr int HEAD_BITS = 4;   // mask bits ahead of the slice's groups: the up to three columns before a row's first aligned group

template <typename T> __device__ __forceinline__ float up(T v);
template <> __device__ __forceinline__ float up<float>(float v) { return v; }
template <> __device__ __forceinline__ float up<uint16_t>(uint16_t v) { return __uint_as_float((uint32_t)v << 16); }

// Four consecutive elements, as one load where the address allows it.
typedef float f32x4 __attribute__((ext_vector_type(4)));
template <typename T, bool VEC> __device__ __forceinline__ f32x4 load4(const T* p) {
  if constexpr (VEC && sizeof(T) == 4) return *reinterpret_cast<const f32x4*>(p);
  else if constexpr (VEC) {
    const uint2 w = *reinterpret_cast<const uint2*>(p);
    return f32x4{__uint_as_float(w.x << 16), __uint_as_float(w.x & 0xFFFF0000u), __uint_as_float(w.y << 16), __uint_as_float(w.y & 0xFFFF0000u)};
  } else return f32x4{up<T>(p[0]), up<T>(p[1]), up<T>(p[2]), up<T>(p[3])};
}

// One workgroup per slice of a row (a few rows then still reach the whole chip; one workgroup per row
// read and wrote one element per thread and step, 167 us for 32 rows of 128,256 bfloat16 columns where
// this takes 12).  Bound: memory, one read and one write of the logits.  Groups of four columns are
// aligned to the output, whose stores are 16 bytes whatever the row stride; `VEC` says that the
// input's groups are aligned too.  If the row has an allow-list, every slice scans it and keeps its own
// columns as a mask in LDS.  The bias entries of the slice follow.  Entries that name the same column add
// up in list order: the thread of a column's first entry walks the rest of the list for it, so
// the float32 additions happen in the order the list gives.
template <typename T, bool VEC>
__global__ __launch_bounds__(CT) void constraints_kernel(const T* logits, int64_t V, int64_t stride,
                                                         const int64_t* __restrict__ bias_ptr, const int32_t* __restrict__ bias_ids,
                                                         const float* __restrict__ bias_vals, const int64_t* __restrict__ allow_ptr,
                                                         const int32_t* __restrict__ allow_ids, float* out, int64_t out_stride) {
  __shared__ uint32_t mask[CSL / 32 + 1];
  __shared__ __align__(16) int32_t sid[BCAP];
  const int tid = threadIdx.x;
  const int64_t row = blockIdx.x;
  const T* src = logits + row * stride;
  float* dst = out + row * out_stride;
  int64_t a0 = 0, a1 = 0, b0 = 0, b1 = 0;
  if (allow_ptr) { a0 = allow_ptr[row]; a1 = allow_ptr[row + 1]; }
  if (bias_ptr) { b0 = bias_ptr[row]; b1 = bias_ptr[row + 1]; }
  // columns before the first 16-byte aligned output address belong to the first slice
  const int64_t head = min(V, (int64_t)((0u - (unsigned)(reinterpret_cast<uintptr_t>(dst) >> 2)) & 3u));
  const bool masked = a1 > a0;  // a row without entries has no allow-list: every column stays
  const int64_t nb = b1 - b0;
  const bool staged = nb > 0 && nb <= BCAP;
  if (staged) for (int i = tid; i < ((int)nb + 3) / 4 * 4; i += CT) sid[i] = i < (int)nb ? bias_ids[b0 + i] : -1;
  // (one slice per workgroup for every row the grid's second dimension can hold)
  for (int64_t sl = blockIdx.y; sl * CSL < V; sl += gridDim.y) {
    const int64_t s0 = head + sl * CSL;                       // first grouped column of the slice
    const int64_t c0 = sl == 0 ? 0 : s0;                      // the slice is [c0, c1)
    const int64_t c1 = min(V, s0 + CSL);
    if (c0 >= c1) break;
    const int64_t bit0 = s0 - HEAD_BITS;                      // column of mask bit 0
    const T* sp = src + s0;
    float* dp = dst + s0;
    const int n_grp = (int)(c1 > s0 ? (c1 - s0) / 4 : 0);
    f32x4 z[CG];  // requested before the lists: their way through memory is the longer one
#pragma unroll
    for (int u = 0; u < CG; ++u) if (tid + u * CT < n_grp) z[u] = load4<T, VEC>(sp + 4 * (tid + u * CT));
    __syncthreads();                                          // (the mask of the slice before is no longer read)
    if (masked) {
      for (int w = tid; w < CSL / 32 + 1; w += CT) mask[w] = 0u;
      __syncthreads();
      for (int64_t i = a0 + tid; i < a1; i += AG * CT) {
        int id[AG];
#pragma unroll
        for (int k = 0; k < AG; ++k) id[k] = i + k * CT < a1 ? allow_ids[i + k * CT] : -1;
#pragma unroll
        for (int k = 0; k < AG; ++k) {
          if (id[k] >= c0 && id[k] < c1) {  // (an id outside the vocabulary is in no slice)
            const int bit = (int)(id[k] - bit0);
            atomicOr(&mask[bit >> 5], 1u << (bit & 31));
          }
        }
      }
      __syncthreads();
    }
    auto allowed = [&](int bit) { return (mask[bit >> 5] >> (bit & 31)) & 1u; };
#pragma unroll
    for (int u = 0; u < CG; ++u) {
      const int g = tid + u * CT;
      if (g >= n_grp) continue;
      if (masked) {
        const int bit = HEAD_BITS + 4 * g;  // four bits of one word
        const uint32_t nib = mask[bit >> 5] >> (bit & 31);
        z[u].x = (nib & 1u) ? z[u].x : -INFINITY; z[u].y = (nib & 2u) ? z[u].y : -INFINITY;
        z[u].z = (nib & 4u) ? z[u].z : -INFINITY; z[u].w = (nib & 8u) ? z[u].w : -INFINITY;
      }
      *reinterpret_cast<f32x4*>(dp + 4 * g) = z[u];
    }
    {  // the columns outside the groups: before the first one, and behind the row's last
      const int n_head = (int)(min(s0, c1) - c0), n_tail = (int)max(c1 - (s0 + 4 * n_grp), (int64_t)0);
      if (tid < n_head + n_tail) {
        const int64_t v = tid < n_head ? c0 + tid : s0 + 4 * n_grp + (tid - n_head);
        const float z = up<T>(src[v]);
        dst[v] = (masked && !allowed((int)(v - bit0))) ? -INFINITY : z;
      }
    }
    if (nb <= 0) continue;
    __syncthreads();  // the slice is written before its bias entries read it back
    for (int64_t i = tid; i < nb; i += CT) {
      const int id = staged ? sid[i] : bias_ids[b0 + i];
      if (id < c0 || id >= c1) continue;
      float acc = dst[id];
      bool first = true;
      auto entry = [&](int64_t j, int other) {  // in list order, one float32 rounding per entry
        if (other != id) return;
        if (j < i) first = false;
        else acc = acc + bias_vals[b0 + j];
      };
      if (staged) {
        for (int j = 0; j < (int)nb && first; j += 4) {  // (places behind the list hold an id that no entry has)
          const int4 q = *reinterpret_cast<const int4*>(sid + j);
          entry(j, q.x); entry(j + 1, q.y); entry(j + 2, q.z); entry(j + 3, q.w);
        }
      } else {
        for (int64_t j = 0; j < nb && first; ++j) entry(j, bias_ids[b0 + j]);
      }
      if (first) dst[id] = acc;
    }
  }
}

}  // namespace constraints
}  // namespace simple

extern "C" int simple_apply_logit_constraints(const void* logits_dev, int64_t B, int64_t V, int dtype, int64_t row_stride_elems,
                                              const int64_t* bias_ptr_dev, const int32_t* bias_ids_dev, const float* bias_vals_dev,
                                              const int64_t* allow_ptr_dev, const int32_t* allow_ids_dev,
                                              float* out_dev, int64_t out_stride_elems, void* hip_stream) {
  using namespace simple::constraints;
  if (B < 0 || V <= 0 || row_stride_elems < V || out_stride_elems < V) return SIMPLE_EINVAL;
  if (dtype != SIMPLE_F32 && dtype != SIMPLE_BF16) return SIMPLE_EINVAL;
  if ((bias_ptr_dev && (!bias_ids_dev || !bias_vals_dev)) || (allow_ptr_dev && !allow_ids_dev)) return SIMPLE_EINVAL;
  if (B == 0) return SIMPLE_OK;
  if (!logits_dev || !out_dev) return SIMPLE_EINVAL;
  if (B > (int64_t)0x7FFFFFFF) return SIMPLE_EINVAL;
  if (allow_ptr_dev && V > MAX_ALLOW_V) return SIMPLE_ECAPACITY;
  hipStream_t st = (hipStream_t)hip_stream;
  const int64_t n_sl = (V + CSL - 1) / CSL;  // (a row's slices start up to three columns in: the last one still covers its end)
  const dim3 grid((unsigned)B, (unsigned)(n_sl < 65535 ? n_sl : 65535));
  // the input's groups start where the output's do: aligned when both matrices start aligned and keep the same phase from row to row
  const size_t esz = (dtype == SIMPLE_F32) ? 4 : 2;
  const bool vec = ((uintptr_t)out_dev & 15u) == 0 && ((uintptr_t)logits_dev & (4 * esz - 1)) == 0 &&
                   ((row_stride_elems ^ out_stride_elems) & 3) == 0;
  auto launch = [&](auto kernel, auto* src) {
    hipLaunchKernelGGL(kernel, grid, dim3(CT), 0, st, src, V, row_stride_elems, bias_ptr_dev, bias_ids_dev, bias_vals_dev, allow_ptr_dev,
                       allow_ids_dev, out_dev, out_stride_elems);
  };
  if (dtype == SIMPLE_F32) {
    if (vec) launch(constraints_kernel<float, true>, (const float*)logits_dev);
    else launch(constraints_kernel<float, false>, (const float*)logits_dev);
  } else {
    if (vec) launch(constraints_kernel<uint16_t, true>, (const uint16_t*)logits_dev);
    else launch(constraints_kernel<uint16_t, false>, (const uint16_t*)logits_dev);
  }
  return hipGetLastError() == hipSuccess ? SIMPLE_OK : SIMPLE_EDEVICE;
}
