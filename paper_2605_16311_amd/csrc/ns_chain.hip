// Newton-Schulz recurrence of small matrices (s <= 256, padded): the whole run of s x s products of a segment in one
// launch, one workgroup per matrix, every matrix of the run on chip.
//
// A product of the recurrence waits for the one before it.  As one launch per product a set of small matrices is bound
// by what a launch costs besides its arithmetic: start and drain, the first slice's way from memory, the write-out and
// the next launch's read of it (5 to 8 us per product at s = 256, of which matrix instructions are 0.5).  Here a
// workgroup keeps its matrix for the whole run: two matrices lie in LDS as operands of the current product, two more in
// registers, and products are separated by barriers.
//
// Storage.  Symmetric half-precision matrices as packed 32 x 32 blocks on and above the diagonal: block (r, c), r <= c,
// is 2 KB of row-major entries at index c (c + 1) / 2 + r; 72 KB at s = 256.  A block row of an operand is read through
// the symmetry: block (r, k) as stored for r <= k, otherwise as the transpose of block (k, r).
//
// Split.  Ten waves.  The matrix is a 4 x 4 grid of super-blocks of SB x SB blocks (SB = 1 for s <= 128, 2 above); six
// waves take a super-block above the diagonal each, four a diagonal one (of which only the blocks on and above the
// diagonal are computed): 4 or 3 accumulators of v_mfma_f32_32x32x16_f16 per wave.  (Two waves with two diagonal ones
// each were the last by far, waiting for the LDS once per three matrix instructions: 9100 cycles per product at s = 256
// where the others took 4500.  With a test per term and not per block and term: 40 polar factors of 192 x 192, K = 5,
// 77 -> 63 us, 256 of 256 x 256 136 -> 122.)  A wave always writes
// the same blocks, so what it adds to a product (a multiple of A, of P or of the matrix it overwrites) it has in
// registers or in its own blocks in LDS; the sum is taken in float32 and rounded once.
//
// LDS layout of a block: 32 rows of 64 bytes, 16-byte chunk c of row r at slot c ^ ((r >> 2) & 3): sixteen lanes that
// read a column of chunks cover all banks; a transposing read takes four whole rows.
#include "common.h"

#include <algorithm>

namespace sm_chain {

constexpr int WAVES = 10, NTH = WAVES * 64;
// Wave w takes super-block off_diagonal(w) of those above the diagonal, or diagonal(w): numbered so that each SIMD (w mod
// 4) has 8 to 10 blocks at SB = 2.
__device__ __forceinline__ bool on_diagonal(int wv) { return wv == 4 || wv == 5 || wv >= 8; }
__device__ __forceinline__ int off_diagonal(int wv) { return wv < 4 ? wv : wv - 2; }
__device__ __forceinline__ int diagonal(int wv) { return wv < 6 ? wv - 4 : wv - 6; }
typedef __attribute__((ext_vector_type(8))) _Float16 f16x8;
typedef __attribute__((ext_vector_type(4))) _Float16 f16x4;
typedef __attribute__((ext_vector_type(4))) short s16x4;
typedef __attribute__((ext_vector_type(8))) short s16x8;
#define LDS_PTR(p) ((__attribute__((address_space(3))) void*)(p))

__device__ __forceinline__ int block_index(int r, int c) { return c * (c + 1) / 2 + r; }

// Fragment of k-step ks (0, 1): lane (row = lane & 31, g = lane >> 5) receives entries 16 ks + 8 g .. + 7 of its row.
struct frag_lane {
  int kc[2], tr_lo[2], tr_hi[2];
  __device__ __forceinline__ void init(int lane) {
    const int fr = lane & 31, fg = lane >> 5, i = lane & 15, g16 = lane >> 4;
    const int c16 = 2 * (g16 & 1) + ((i & 3) >> 1);
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      kc[ks] = fr * 64 + (((2 * ks + fg) ^ ((fr >> 2) & 3)) << 4);
      const int k = 16 * ks + 8 * (g16 >> 1) + (i >> 2);
      tr_lo[ks] = k * 64 + ((c16 ^ ((k >> 2) & 3)) << 4) + (i & 1) * 8;
      tr_hi[ks] = (k + 4) * 64 + ((c16 ^ (((k + 4) >> 2) & 3)) << 4) + (i & 1) * 8;
    }
  }
  __device__ __forceinline__ f16x8 transposed(const unsigned char* block, int ks) const {
    const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(block + tr_lo[ks]));
    const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(block + tr_hi[ks]));
    const s16x8 v = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
    return __builtin_bit_cast(f16x8, v);
  }
  // of block (r, kb) of a packed matrix, stored (r <= kb) or as the transpose of block (kb, r)
  template <bool STORED>
  __device__ __forceinline__ f16x8 get(const unsigned char* m, int r, int kb, int ks) const {
    if constexpr (STORED) return *reinterpret_cast<const f16x8*>(m + block_index(r, kb) * 2048 + kc[ks]);
    else return transposed(m + block_index(kb, r) * 2048, ks);
  }
};

// Blocks of a wave: NU of them, block u at (row[u], col) = (r, c), computed from its super-blocks.
template <int SB, bool DIAG>
struct wave_blocks {
  static constexpr int NU = DIAG ? SB * (SB + 1) / 2 : SB * SB;
  int I, J;  // super-block (I, J)
  __device__ __forceinline__ wave_blocks(int wv) {
    if (!DIAG) {
      const int w = off_diagonal(wv);
      I = w < 3 ? 0 : w < 5 ? 1 : 2;
      J = w < 3 ? w + 1 : w < 5 ? w - 1 : 3;
    } else {
      I = J = diagonal(wv);
    }
  }
  __device__ __forceinline__ void at(int u, int& r, int& c) const {
    if (!DIAG) {
      r = SB * I + u / SB;
      c = SB * J + u % SB;
    } else {
      const int j = u < 1 ? 0 : u < 3 ? 1 : 2;
      r = SB * I + u - j * (j + 1) / 2;
      c = SB * I + j;
    }
  }
};

// acc = X Y for super-block (I, J), or (DIAG) for the super-block (I, I), over the whole short side.
// No barrier: the operands do not change meanwhile.  Everything about a fragment's place and form (stored or
// transposed) is fixed at compile time, so the reads run ahead of the matrix instructions; choosing the form at run
// time put a branch and a wait for the LDS in front of every read (s = 256: 11 us per product, 7 without).
template <int SB, int I, int J, bool DIAG, bool SQUARE, int NU>
__device__ __forceinline__ void multiply_at(f32x16 (&acc)[NU], const unsigned char* X, const unsigned char* Y, const frag_lane& fl) {
#pragma unroll
  for (int u = 0; u < NU; ++u)
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[u][v] = 0.f;
#define MMA(u, a, b) acc[u] = __builtin_amdgcn_mfma_f32_32x32x16_f16(b, a, acc[u], 0, 0, 0)
#define FRAG(M, r, kb, ks) ((kb) >= (r) ? fl.get<true>(M, r, kb, ks) : fl.get<false>(M, r, kb, ks))
#pragma unroll
  for (int kb = 0; kb < 4 * SB; ++kb)
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      if constexpr (!DIAG) {
        f16x8 fa[SB], fb[SB];
#pragma unroll
        for (int i = 0; i < SB; ++i) fa[i] = FRAG(X, SB * I + i, kb, ks);
#pragma unroll
        for (int i = 0; i < SB; ++i) fb[i] = FRAG(Y, SB * J + i, kb, ks);
#pragma unroll
        for (int r = 0; r < SB; ++r)
#pragma unroll
          for (int c = 0; c < SB; ++c) MMA(r * SB + c, fa[r], fb[c]);
      } else {
        f16x8 fa[SB], fb[SB];
#pragma unroll
        for (int i = 0; i < SB; ++i) fa[i] = FRAG(X, SB * I + i, kb, ks);
#pragma unroll
        for (int i = 0; i < SB; ++i) fb[i] = SQUARE ? fa[i] : FRAG(Y, SB * I + i, kb, ks);
#pragma unroll
        for (int c = 0; c < SB; ++c)
#pragma unroll
          for (int r = 0; r <= c; ++r) MMA(c * (c + 1) / 2 + r, fa[r], fb[c]);
      }
    }
#undef FRAG
#undef MMA
}

template <int SB, bool DIAG, int NU>
__device__ __forceinline__ void multiply(f32x16 (&acc)[NU], const unsigned char* X, const unsigned char* Y, int wv, const frag_lane& fl) {
  if constexpr (!DIAG) {
    switch (off_diagonal(wv)) {
      case 0: multiply_at<SB, 0, 1, false, false>(acc, X, Y, fl); break;
      case 1: multiply_at<SB, 0, 2, false, false>(acc, X, Y, fl); break;
      case 2: multiply_at<SB, 0, 3, false, false>(acc, X, Y, fl); break;
      case 3: multiply_at<SB, 1, 2, false, false>(acc, X, Y, fl); break;
      case 4: multiply_at<SB, 1, 3, false, false>(acc, X, Y, fl); break;
      default: multiply_at<SB, 2, 3, false, false>(acc, X, Y, fl);
    }
  } else if (X == Y) {
    switch (diagonal(wv)) {
      case 0: multiply_at<SB, 0, 0, true, true>(acc, X, Y, fl); break;
      case 1: multiply_at<SB, 1, 1, true, true>(acc, X, Y, fl); break;
      case 2: multiply_at<SB, 2, 2, true, true>(acc, X, Y, fl); break;
      default: multiply_at<SB, 3, 3, true, true>(acc, X, Y, fl);
    }
  } else {
    switch (diagonal(wv)) {
      case 0: multiply_at<SB, 0, 0, true, false>(acc, X, Y, fl); break;
      case 1: multiply_at<SB, 1, 1, true, false>(acc, X, Y, fl); break;
      case 2: multiply_at<SB, 2, 2, true, false>(acc, X, Y, fl); break;
      default: multiply_at<SB, 3, 3, true, false>(acc, X, Y, fl);
    }
  }
}

// A wave's blocks of one matrix in registers, as its accumulators are: a lane has row fr, columns 8 vg + 4 fg .. + 3 of
// a block.
template <int NU>
struct kept {
  f16x4 v[NU][4];
};

// An op read from LDS, in scalar registers.
__device__ __forceinline__ chain_op uniform_op(const chain_op* p) {
  chain_op o = *p;
  int* w = reinterpret_cast<int*>(&o);
#pragma unroll
  for (int i = 0; i < (int)(sizeof(chain_op) / 4); ++i) w[i] = __builtin_amdgcn_readfirstlane(w[i]);
  return o;
}

// The run, on the waves above (DIAG false) or on the diagonal; see chain_op.
template <int SB, bool DIAG>
__device__ __forceinline__ void chain(const chain_args& a, const chain_class& C, long long at, int nb,
                                      unsigned char* L0, unsigned char* L1, const chain_op* ops) {
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const wave_blocks<SB, DIAG> wb(wv);
  constexpr int NU = wave_blocks<SB, DIAG>::NU;
  f32x16 acc[NU];
  kept<NU> A, P;
  // f(block number, block row, block column, LDS byte offset of the lane's piece 0; piece vg is the offset ^ (vg << 4))
  auto for_blocks = [&](auto f) {
    int lane = threadIdx.x & 63;
    asm volatile("" : "+v"(lane));  // worked out here each time, not carried through the products in registers
    const int fr = lane & 31, fg = lane >> 5, own = fr * 64 + (((fr >> 2) & 3) << 4) + fg * 8;
#pragma unroll
    for (int u = 0; u < NU; ++u) {
      int r, c;
      wb.at(u, r, c);
      if (c < nb) f(u, r, c, block_index(r, c) * 2048 + own, fr, fg);  // r <= c
    }
  };
  auto put = [&](unsigned char* L, const kept<NU>& m) {
    for_blocks([&](int u, int, int, int b, int, int) {
#pragma unroll
      for (int vg = 0; vg < 4; ++vg) *reinterpret_cast<f16x4*>(L + (b ^ (vg << 4))) = m.v[u][vg];
    });
  };
  for_blocks([&](int u, int, int, int b, int, int) {
#pragma unroll
    for (int vg = 0; vg < 4; ++vg) A.v[u][vg] = *reinterpret_cast<const f16x4*>(L0 + (b ^ (vg << 4)));
  });
#pragma unroll
  for (int u = 0; u < NU; ++u)
#pragma unroll
    for (int vg = 0; vg < 4; ++vg) P.v[u][vg] = f16x4{0, 0, 0, 0};
#pragma clang loop unroll(disable)
  for (int o = 0; o < a.n_ops; ++o) {
    const chain_op op = uniform_op(ops + o);
    if (op.pre) {
      if (op.pre & 1) put(L0, A);
      if (op.pre & 2) put(L0, P);
      if (op.pre & 4) put(L1, P);
      __syncthreads();
    }
    {
      int lane = threadIdx.x & 63;
      asm volatile("" : "+v"(lane));
      frag_lane fl;
      fl.init(lane);
      multiply<SB, DIAG>(acc, op.x ? L1 : L0, op.y ? L1 : L0, wv, fl);
    }
    // one pass over the blocks per term that there is (a test per block and term took as long as the terms)
    if (op.alpha != 1.f) {
#pragma unroll
      for (int u = 0; u < NU; ++u)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[u][v] *= op.alpha;
    }
    if (op.ca != 0.f) {
#pragma unroll
      for (int u = 0; u < NU; ++u)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[u][v] = fmaf((float)A.v[u][v >> 2][v & 3], op.ca, acc[u][v]);
    }
    if (op.cp != 0.f) {
#pragma unroll
      for (int u = 0; u < NU; ++u)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[u][v] = fmaf((float)P.v[u][v >> 2][v & 3], op.cp, acc[u][v]);
    }
    if (op.cl != 0.f) {
      for_blocks([&](int u, int, int, int b, int, int) {
#pragma unroll
        for (int vg = 0; vg < 4; ++vg) {
          const f16x4 e = *reinterpret_cast<const f16x4*>(L1 + (b ^ (vg << 4)));
#pragma unroll
          for (int k = 0; k < 4; ++k) acc[u][4 * vg + k] = fmaf((float)e[k], op.cl, acc[u][4 * vg + k]);
        }
      });
    }
    if (DIAG && op.diag != 0.f) {
      for_blocks([&](int u, int r, int c, int, int fr, int fg) {
        if (r == c) {
#pragma unroll
          for (int v = 0; v < 16; ++v)
            if (fr == 8 * (v >> 2) + 4 * fg + (v & 3)) acc[u][v] += op.diag;
        }
      });
    }
    __syncthreads();  // every wave is done with both operands
    if (o + 1 < a.n_ops) {  // (the last result leaves from acc)
      kept<NU> h;
#pragma unroll
      for (int u = 0; u < NU; ++u)
#pragma unroll
        for (int vg = 0; vg < 4; ++vg)
          h.v[u][vg] = f16x4{(_Float16)acc[u][4 * vg], (_Float16)acc[u][4 * vg + 1], (_Float16)acc[u][4 * vg + 2], (_Float16)acc[u][4 * vg + 3]};
      if (op.put >= 0) put(op.put ? L1 : L0, h);
      if (op.keep & 1) A = h;
      if (op.keep & 2) P = h;
      if (op.put >= 0) __syncthreads();
    }
  }
  // the result leaves in bf16 as a whole row-major matrix; the mirrored blocks are transposed through the wave's share
  // of L0
  unsigned char* scratch = L0 + wv * 2048;
  unsigned char* out = C.out + at;
  for_blocks([&](int u, int r, int c, int b, int fr, int fg) {
    const int own = b - block_index(r, c) * 2048;
#pragma unroll
    for (int vg = 0; vg < 4; ++vg) {
      const bf16x4 h = {(bf16_t)acc[u][4 * vg], (bf16_t)acc[u][4 * vg + 1], (bf16_t)acc[u][4 * vg + 2], (bf16_t)acc[u][4 * vg + 3]};
      *reinterpret_cast<bf16x4*>(out + ((long long)(32 * r + fr) * C.s + 32 * c + 8 * vg + 4 * fg) * 2) = h;
      if (r != c) *reinterpret_cast<bf16x4*>(scratch + (own ^ (vg << 4))) = h;
    }
    if (r != c) {
      frag_lane fl;
      fl.init(fr + 32 * fg);
#pragma unroll
      for (int ks = 0; ks < 2; ++ks)
        *reinterpret_cast<f16x8*>(out + ((long long)(32 * c + fr) * C.s + 32 * r + 16 * ks + 8 * fg) * 2) = fl.transposed(scratch, ks);
    }
  });
}

template <int SB>
__global__ void __launch_bounds__(NTH) sm_ns_chain_kernel(const chain_args a) {
  constexpr int BLOCKS = 4 * SB * (4 * SB + 1) / 2;
  __shared__ __attribute__((aligned(1024))) unsigned char L0[BLOCKS * 2048], L1[BLOCKS * 2048];
  // the ops of the run: from the kernel arguments each would cost a trip to host memory when its turn comes
  __shared__ __attribute__((aligned(16))) chain_op ops[SM_CHAIN_MAX_OPS];
  constexpr int WORDS = SM_CHAIN_MAX_OPS * sizeof(chain_op) / 4;
  static_assert(WORDS <= NTH, "one word per thread");
  if (threadIdx.x < WORDS) reinterpret_cast<int*>(ops)[threadIdx.x] = reinterpret_cast<const int*>(a.op)[threadIdx.x];
  const int ci = sm_find(a.begin, a.n, blockIdx.x);
  const chain_class& C = a.c[ci];
  const int nb = C.s / 32;
  const long long at = (long long)(blockIdx.x - a.begin.v[ci]) * C.s * C.s * 2;
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // A_0: wave-load L brings half L & 1 of block L >> 1, each lane the chunk that belongs in its slot
  const unsigned char* in = C.in + at;
  const __amdgpu_buffer_rsrc_t ra = __builtin_amdgcn_make_buffer_rsrc(const_cast<unsigned char*>(in), 0, 0x7FFFFFFF, 0x00020000);
  const int voff = (lane >> 2) * 64 + (((lane & 3) ^ ((lane >> 4) & 3)) << 4);
  for (int L = wv; L < nb * (nb + 1); L += WAVES) {
    const int vo = voff, so = L * 1024;
    __builtin_amdgcn_raw_ptr_buffer_load_lds(ra, LDS_PTR(L0 + L * 1024), 16, vo, so, 0, 0);
  }
  // what the matrix does not fill reads as zero in both
  for (int w = threadIdx.x + nb * (nb + 1) / 2 * 128; w < BLOCKS * 128; w += NTH) {
    reinterpret_cast<u32x4*>(L0)[w] = u32x4{0u, 0u, 0u, 0u};
    reinterpret_cast<u32x4*>(L1)[w] = u32x4{0u, 0u, 0u, 0u};
  }
  __builtin_amdgcn_s_waitcnt(0x0070);
  __syncthreads();
  if (on_diagonal(wv)) chain<SB, true>(a, C, at, nb, L0, L1, ops);
  else chain<SB, false>(a, C, at, nb, L0, L1, ops);
}

}  // namespace sm_chain
using namespace sm_chain;

int sm_launch_chain(signmuon_ctx* ctx, chain_args& a, int blocks) {
  int most = 0;
  for (int i = 0; i < a.n; ++i) {
    if (a.c[i].s % 64 || a.c[i].s < 64 || a.c[i].s > SM_CHAIN_MAX_S) return sm_fail(ctx, SM_EINVAL, "internal: chain size");
    most = std::max(most, a.c[i].s);
  }
  if (a.n < 1 || a.n_ops < 1 || blocks < 1) return sm_fail(ctx, SM_EINVAL, "internal: chain arguments");
  if ((ctx->profiling >> SM_K_NS_SMALL) & 1u) {
    for (int i = 0; i < a.n; ++i) {
      const double s = a.c[i].s, mats = (i + 1 < a.n ? a.begin.v[i + 1] : blocks) - a.begin.v[i];
      double area = 0.0;  // the 32 x 32 blocks on and above the diagonal, clipped to the logical matrix
      for (int c = 0; c < a.c[i].su; c += 32) area += (double)std::min(32, a.c[i].su - c) * std::min(c + 32, a.c[i].su);
      ctx->work_flop[SM_K_NS_SMALL] += 2.0 * area * a.c[i].su * mats * a.n_ops;
      ctx->work_dense[SM_K_NS_SMALL] += 2.0 * s * s * s * mats * a.n_ops;
      ctx->work_bytes[SM_K_NS_SMALL] += 2.0 * (s * (s + 32) / 2 + s * s) * mats;  // A_0 packed, P whole
    }
  }
  sm_launch_scope sc(ctx, SM_K_NS_SMALL);
  const dim3 grid(blocks), block(NTH);
  if (most <= 128) hipLaunchKernelGGL(sm_ns_chain_kernel<1>, grid, block, 0, ctx->stream, a);
  else hipLaunchKernelGGL(sm_ns_chain_kernel<2>, grid, block, 0, ctx->stream, a);
  SM_HIP(ctx, hipGetLastError());
  return SM_OK;
}
