// Layout helpers around the Newton-Schulz workspace: copies between caller
// matrices and the zero-padded bf16 working layout, the copy in with the sums of
// squares for the Frobenius scale of Alg. PolarNS.
#include "common.h"

#include <algorithm>

namespace {

constexpr int TPB = 256;

// Both copies work on groups of four entries of a row, one per thread: rows and matrices of odd length make the caller's
// side unaligned, the working side always is aligned.
static_assert(SM_MOM_CHUNK == 4 * TPB, "a workgroup covers one chunk of partial sums");

struct copy_args {
  const void* src;
  void* dst;
  long long n;           // entries of a matrix on the caller's side
  long long groups;      // groups of four of a matrix
  long long stride;      // entries between matrices on the working side
  const float* scale;
  float* partial;
  int cols, ld, per_row;
  sm_div by_row;         // by per_row
};

// Group t of a matrix: where it lies on the caller's and on the working side, and how many entries it has.
__device__ __forceinline__ int copy_group(const copy_args& a, long long t, long long& flat, long long& padded) {
  long long r;
  int c;
  sm_row_of(a.by_row, a.per_row, t, r, c);
  c *= 4;
  flat = r * a.cols + c;
  padded = r * a.ld + c;
  return min(4, a.cols - c);
}

template <int DT>
__device__ __forceinline__ f32x4 load_group(const void* src, long long at, int live) {
  f32x4 v = {0.f, 0.f, 0.f, 0.f};
  if (DT == SM_F32) {
    const float* s = reinterpret_cast<const float*>(src) + at;
    if (live == 4) return __builtin_nontemporal_load(reinterpret_cast<const f32x4_u*>(s));
#pragma unroll
    for (int k = 0; k < 3; ++k)
      if (k < live) v[k] = s[k];
  } else {
    const bf16_t* s = reinterpret_cast<const bf16_t*>(src) + at;
    if (live == 4) {
      const bf16x4 h = __builtin_nontemporal_load(reinterpret_cast<const bf16x4_u*>(s));
#pragma unroll
      for (int k = 0; k < 4; ++k) v[k] = (float)h[k];
    } else {
#pragma unroll
      for (int k = 0; k < 3; ++k)
        if (k < live) v[k] = (float)s[k];
    }
  }
  return v;
}

template <int DT>
__global__ void __launch_bounds__(TPB) sm_copy_in_kernel(const copy_args a) {
  __shared__ float red[4];
  const int b = blockIdx.y;
  const long long t = (long long)blockIdx.x * TPB + threadIdx.x;
  float ss = 0.f;
  if (t < a.groups) {
    long long flat, padded;
    const int live = copy_group(a, t, flat, padded);
    const f32x4 v = load_group<DT>(a.src, (long long)b * a.n + flat, live);
    ss = (v[0] * v[0] + v[1] * v[1]) + (v[2] * v[2] + v[3] * v[3]);
    const bf16x4 h = {(bf16_t)v[0], (bf16_t)v[1], (bf16_t)v[2], (bf16_t)v[3]};  // zeros beyond the row's end
    *reinterpret_cast<bf16x4*>(reinterpret_cast<bf16_t*>(a.dst) + (long long)b * a.stride + padded) = h;
  }
  if (a.partial) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) ss += __shfl_down(ss, off, 64);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = ss;
    __syncthreads();
    if (threadIdx.x == 0) a.partial[(long long)b * gridDim.x + blockIdx.x] = (red[0] + red[1]) + (red[2] + red[3]);
  }
}

template <int DT>
__global__ void __launch_bounds__(TPB) sm_copy_out_kernel(const copy_args a) {
  const int b = blockIdx.y;
  const long long t = (long long)blockIdx.x * TPB + threadIdx.x;
  if (t >= a.groups) return;
  long long flat, padded;
  const int live = copy_group(a, t, flat, padded);
  const bf16x4 h = __builtin_nontemporal_load(
      reinterpret_cast<const bf16x4*>(reinterpret_cast<const bf16_t*>(a.src) + (long long)b * a.stride + padded));
  f32x4 v = {(float)h[0], (float)h[1], (float)h[2], (float)h[3]};
  if (a.scale) {
    const float s = a.scale[b];
#pragma unroll
    for (int k = 0; k < 4; ++k) v[k] *= s;
  }
  const long long at = (long long)b * a.n + flat;
  if (DT == SM_F32) {
    float* d = reinterpret_cast<float*>(a.dst) + at;
    if (live == 4) {
      *reinterpret_cast<f32x4_u*>(d) = v;
    } else {
#pragma unroll
      for (int k = 0; k < 3; ++k)
        if (k < live) d[k] = v[k];
    }
  } else {
    bf16_t* d = reinterpret_cast<bf16_t*>(a.dst) + at;
    const bf16x4 o = {(bf16_t)v[0], (bf16_t)v[1], (bf16_t)v[2], (bf16_t)v[3]};
    if (live == 4) {
      *reinterpret_cast<bf16x4_u*>(d) = o;
    } else {
#pragma unroll
      for (int k = 0; k < 3; ++k)
        if (k < live) d[k] = o[k];
    }
  }
}

copy_args copy_setup(const void* src, void* dst, int rows, int cols, int ld, long long stride) {
  copy_args a;
  a.src = src;
  a.dst = dst;
  a.n = (long long)rows * cols;
  a.per_row = (cols + 3) / 4;
  a.groups = (long long)rows * a.per_row;
  a.stride = stride;
  a.scale = nullptr;
  a.partial = nullptr;
  a.cols = cols;
  a.ld = ld;
  a.by_row = sm_div_by((unsigned)a.per_row);
  return a;
}

}  // namespace

int sm_launch_copy_in(signmuon_ctx* ctx, const void* src, int dtype, int batch, int rows, int cols, bf16_t* dst,
                      int ld, long long dst_stride, float* partial) {
  copy_args a = copy_setup(src, dst, rows, cols, ld, dst_stride);
  a.partial = partial;
  const dim3 grid((unsigned)((a.groups + TPB - 1) / TPB), batch);
  if (partial && (long long)grid.x != sm_mom_chunks(rows, cols, ld)) return sm_fail(ctx, SM_EINVAL, "internal: copy chunks");
  sm_launch_scope sc(ctx, SM_K_OTHER);
  if (dtype == SM_F32)
    hipLaunchKernelGGL(sm_copy_in_kernel<SM_F32>, grid, dim3(TPB), 0, ctx->stream, a);
  else
    hipLaunchKernelGGL(sm_copy_in_kernel<SM_BF16>, grid, dim3(TPB), 0, ctx->stream, a);
  SM_HIP(ctx, hipGetLastError());
  return SM_OK;
}

int sm_launch_copy_out(signmuon_ctx* ctx, const bf16_t* src, int ld, long long src_stride, int batch, int rows,
                       int cols, void* dst, int dtype, const float* scale) {
  copy_args a = copy_setup(src, dst, rows, cols, ld, src_stride);
  a.scale = scale;
  const dim3 grid((unsigned)((a.groups + TPB - 1) / TPB), batch);
  sm_launch_scope sc(ctx, SM_K_OTHER);
  if (dtype == SM_F32)
    hipLaunchKernelGGL(sm_copy_out_kernel<SM_F32>, grid, dim3(TPB), 0, ctx->stream, a);
  else
    hipLaunchKernelGGL(sm_copy_out_kernel<SM_BF16>, grid, dim3(TPB), 0, ctx->stream, a);
  SM_HIP(ctx, hipGetLastError());
  return SM_OK;
}
