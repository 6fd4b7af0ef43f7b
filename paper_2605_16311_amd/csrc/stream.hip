// HBM-bound kernels of the Sign-Muon step: momentum (a1), sign extraction and
// packing (a5), majority vote (a6) with the fused update (a8), and the update
// after a local polar step.  All are pure streaming passes: every byte is read
// once with 16-byte (or 4-byte broadcast) coalesced accesses and written once.
#include "common.h"

#include <type_traits>

namespace {

constexpr int TPB = 256;

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off, 64);
  return v;
}

// Sum over the 256 threads of a workgroup, fixed order; result valid in thread 0.
__device__ __forceinline__ float block_sum(float v, float* lds4) {
  v = wave_sum(v);
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  if (lane == 0) lds4[wv] = v;
  __syncthreads();
  float r = 0.f;
  if (threadIdx.x == 0) r = (lds4[0] + lds4[1]) + (lds4[2] + lds4[3]);
  return r;
}

// sign decision of Alg. 3's encoding note, x >= 0 by IEEE comparison, taken on
// the bit pattern so that it does not depend on the denormal mode:
// true for +0 .. +inf and for -0, false for negatives and every NaN.
__device__ __forceinline__ unsigned ge0_f32(unsigned u) { return (u <= 0x7F800000u) | (u == 0x80000000u); }
__device__ __forceinline__ unsigned ge0_bf16(unsigned h) { return (h <= 0x7F80u) | (h == 0x8000u); }

// ------------------------------------------------------------------ momentum
// start: byte k is the block that holds workgroup (k << shift) of the launch, so that a workgroup finds its
// block in a step or two instead of comparing all starts (workgroups are short: that would show).  Bytes are
// taken out of words: there is no scalar byte load, and a vector load of the arguments goes to host memory.
struct mom_args {
  int n, M;
  float beta, omb, wd;
  int shift;
  sm_starts<SM_MOM_MAX_GROUP> begin;
  unsigned start[16];
  sm_mom_desc d[SM_MOM_MAX_GROUP];
};
static_assert(sizeof(mom_args) <= 4096, "kernel arguments are limited to 4 KB");

__device__ __forceinline__ float mom_one(float m, float g, float w, const mom_args& a, bool has_wd) {
  if (has_wd) g = __fadd_rn(g, __fmul_rn(a.wd, w));
  return __fadd_rn(__fmul_rn(a.beta, m), __fmul_rn(a.omb, g));
}

// A thread owns four consecutive entries, of one row where the rows of x are padded (then the group that ends a row
// also writes x's zeros up to the next multiple of four).  Rows and workers of odd length make the vectors unaligned,
// which costs a ninth line per wave and load; one path serves every size (the scalar one it replaces, with a 64-bit
// division per entry, took 61 us where the traffic is worth 28: 1000x2047 and smaller blocks, three workers).
__global__ void __launch_bounds__(TPB) sm_momentum_kernel(const mom_args a) {
  static_assert(SM_MOM_CHUNK == TPB * 4, "one group of four entries per thread");
  __shared__ float red[4];
  int bi = 0;
  if (a.n > 1) {
    const unsigned k = blockIdx.x >> a.shift;
    bi = (a.start[k >> 2] >> (8 * (k & 3))) & 0xFFu;
  }
  while (bi + 1 < a.n && (int)blockIdx.x >= a.begin.v[bi + 1]) ++bi;
  const sm_mom_desc& D = a.d[bi];
  const int local = blockIdx.x - a.begin.v[bi];
  const int p = local / D.chunks, ch = local - p * D.chunks;
  const long long d = D.d;
  const bool has_wd = (D.w != nullptr) && (a.wd != 0.f);
  long long i = (long long)ch * SM_MOM_CHUNK + threadIdx.x * 4;  // first entry of the group
  long long xi = i;
  int live = 4;
  if (D.quads.shift) {
    long long r;
    int c;
    sm_row_of(D.quads, (D.cols + 3) >> 2, (long long)ch * TPB + threadIdx.x, r, c);
    c *= 4;
    i = r * D.cols + c;
    xi = r * ((D.cols + 63) & ~63) + c;
    live = min(4, D.cols - c);
  }
  if (i >= d) live = 0;
  else if (d - i < live) live = (int)(d - i);
  float ss = 0.f;
  if (live > 0) {
    float* mom = D.mom + (long long)p * d + i;
    const float* grad = D.grad + (long long)p * d + i;
    f32x4 m = {0.f, 0.f, 0.f, 0.f};
    if (live == 4) {
      m = __builtin_nontemporal_load(reinterpret_cast<const f32x4_u*>(mom));
      const f32x4 g = __builtin_nontemporal_load(reinterpret_cast<const f32x4_u*>(grad));
      f32x4 ww = {0.f, 0.f, 0.f, 0.f};
      if (has_wd) ww = *reinterpret_cast<const f32x4_u*>(D.w + i);
#pragma unroll
      for (int k = 0; k < 4; ++k) m[k] = mom_one(m[k], g[k], ww[k], a, has_wd);
      // neither the momentum nor its bf16 copy is read again before it has left the caches
      __builtin_nontemporal_store(m, reinterpret_cast<f32x4_u*>(mom));
    } else {
#pragma unroll
      for (int k = 0; k < 3; ++k)
        if (k < live) {
          m[k] = mom_one(mom[k], grad[k], has_wd ? D.w[i + k] : 0.f, a, has_wd);
          mom[k] = m[k];
        }
    }
    ss = (m[0] * m[0] + m[1] * m[1]) + (m[2] * m[2] + m[3] * m[3]);
    if (D.x) {
      bf16_t* x = D.x + (long long)p * D.x_stride + xi;
      const bf16x4 h = {(bf16_t)m[0], (bf16_t)m[1], (bf16_t)m[2], (bf16_t)m[3]};
      if (live == 4 || D.quads.shift) {
        __builtin_nontemporal_store(h, reinterpret_cast<bf16x4_u*>(x));
      } else {
#pragma unroll
        for (int k = 0; k < 3; ++k)
          if (k < live) x[k] = h[k];
      }
    }
  }
  if (D.partial) {
    const float tot = block_sum(ss, red);
    if (threadIdx.x == 0) D.partial[(long long)p * D.chunks + ch] = tot;
  }
}

// Sum of an item's partial sums of squares, fixed order; result valid in thread 0.  One workgroup per item, so what bounds
// it is the latency of its loads, one after the other (seven to ten for the partial sums of a 768-wide block, 172 for those
// of 4096 x 11008, by 256 threads in a loop that adds as it loads): 1024 threads have eight loads in flight each.  Momentum
// of eight workers' 768 x 2304 with its norms: 37.2 -> 36.2 us.
constexpr int TPS = 1024, SUM_AHEAD = 8;
__device__ __forceinline__ float sum_partials(const float* __restrict__ src, int chunks) {
  __shared__ float red[TPS / 64];
  float s = 0.f;
  for (int base = 0; base < chunks; base += TPS * SUM_AHEAD) {
    float x[SUM_AHEAD];
#pragma unroll
    for (int k = 0; k < SUM_AHEAD; ++k) x[k] = src[min(base + k * TPS + (int)threadIdx.x, chunks - 1)];
#pragma unroll
    for (int k = 0; k < SUM_AHEAD; ++k) s += base + k * TPS + (int)threadIdx.x < chunks ? x[k] : 0.f;
  }
  s = wave_sum(s);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
  __syncthreads();
  s = threadIdx.x < TPS / 64 ? red[threadIdx.x] : 0.f;
#pragma unroll
  for (int off = TPS / 128; off > 0; off >>= 1) s += __shfl_down(s, off, 64);
  return s;
}

// sumsq[i] = sum of partial[i*chunks .. +chunks); one workgroup per i.
__global__ void __launch_bounds__(TPS) sm_reduce_partials_kernel(const float* partial, int chunks, float* sumsq) {
  const float tot = sum_partials(partial + (long long)blockIdx.x * chunks, chunks);
  if (threadIdx.x == 0) sumsq[blockIdx.x] = tot;
}

struct sigma_args {
  int n;
  float eps;
  sm_sigma_desc d[SM_SIGMA_MAX_GROUP];
  sm_starts<SM_SIGMA_MAX_GROUP> begin;
};

// One workgroup per item of every class of the table.
__global__ void __launch_bounds__(TPS) sm_sigma_group_kernel(const sigma_args a) {
  int i;
  const sm_sigma_desc& D = a.d[sm_entry(a.begin, a.n, blockIdx.x, i)];
  if (D.mode == 0) {
    const float tot = sum_partials(D.partial + (long long)i * D.chunks, D.chunks);
    if (threadIdx.x == 0) {
      if (D.sig) D.sig[i] = tot;
      D.inv[i] = 1.0f / fmaxf(sqrtf(tot), a.eps);
    }
  } else if (threadIdx.x == 0) {
    D.inv[i] = 1.0f / fmaxf(D.sig[i], a.eps);
  }
}

// ------------------------------------------------------------------ sign pack
// One launch covers a table of matrices (all workers of each): workgroup -> (matrix, worker, chunk).
struct sp_args {
  int n;
  int pad_;
  sm_starts<SM_SP_MAX_GROUP> begin;
  sm_sp_desc d[SM_SP_MAX_GROUP];
};

template <int DT>
__device__ __forceinline__ unsigned ge0_at(const void* u, long long i) {
  return DT == SM_BF16 ? ge0_bf16(reinterpret_cast<const unsigned short*>(u)[i])
                       : ge0_f32(reinterpret_cast<const unsigned*>(u)[i]);
}

// Entry e of the flattened matrix in the source, which has padded rows (ROWS) or is flat; room: entries left in its row.
template <bool ROWS>
__device__ __forceinline__ long long sp_source(const sm_sp_desc& D, long long e, int& room) {
  if (!ROWS) {
    room = 0x7FFFFFFF;
    return e;
  }
  long long r;
  int c;
  sm_row_of(D.by_cols, D.cols, e, r, c);
  room = D.cols - c;
  return r * D.ld + c;
}

// Bits of entries e0 .. e0 + E - 1 one at a time: the group that ends a matrix, or one that straddles rows of a
// padded source.  Bits beyond entry n - 1 are zero.
template <int DT, int E, bool ROWS>
__device__ __forceinline__ unsigned sp_slow(const sm_sp_desc& D, const void* u, long long e0) {
  unsigned bits = 0;
  for (int k = 0; k < E; ++k) {
    if (e0 + k >= D.n) break;
    int room;
    bits |= ge0_at<DT>(u, sp_source<ROWS>(D, e0 + k, room)) << k;
  }
  return bits;
}

template <int DT>
__device__ __forceinline__ const void* sp_row(const sm_sp_desc& D, int b) {
  return DT == SM_BF16 ? (const void*)(reinterpret_cast<const unsigned short*>(D.u) + (long long)b * D.batch_stride)
                       : (const void*)(reinterpret_cast<const unsigned*>(D.u) + (long long)b * D.batch_stride);
}

// 1-bit output: a thread turns 8 entries into a byte, SP_UNROLL times; all loads are issued before the first use, and
// the bytes of four neighbouring lanes leave as one 32-bit store (byte stores cost a full store slot each).  Rows of
// the source may start at any element (odd lengths), rows of the output at any multiple of 8 bytes.
constexpr int SP_UNROLL = 2;

template <int DT, bool ROWS>
__global__ void __launch_bounds__(TPB) sm_sign_pack_bits_kernel(const sp_args a) {
  const int di = sm_find(a.begin, a.n, blockIdx.x);
  const sm_sp_desc& D = a.d[di];
  const int local = blockIdx.x - a.begin.v[di];
  const int b = local / D.blocks_per_row, bx = local - b * D.blocks_per_row;
  const long long n = D.n, bytes_per_row = 8 * ((n + 63) / 64);  // a multiple of 8: a 4-lane group is in range as a whole
  const void* u = sp_row<DT>(D, b);
  unsigned char* o = reinterpret_cast<unsigned char*>(D.out) + (long long)b * D.out_stride;
  const long long q0 = ((long long)bx * SP_UNROLL) * TPB + threadIdx.x;
  u32x4 v0[SP_UNROLL], v1[SP_UNROLL];
  bool whole[SP_UNROLL];
#pragma unroll
  for (int j = 0; j < SP_UNROLL; ++j) {
    const long long e0 = (q0 + (long long)j * TPB) * 8;
    v0[j] = v1[j] = u32x4{0u, 0u, 0u, 0u};
    whole[j] = false;
    if (e0 + 8 <= n) {
      int room;
      const long long src = sp_source<ROWS>(D, e0, room);
      whole[j] = room >= 8;
      if (whole[j]) {
        if (DT == SM_BF16) {
          v0[j] = __builtin_nontemporal_load(reinterpret_cast<const u32x4_u*>(reinterpret_cast<const unsigned short*>(u) + src));
        } else {
          v0[j] = __builtin_nontemporal_load(reinterpret_cast<const u32x4_u*>(reinterpret_cast<const unsigned*>(u) + src));
          v1[j] = __builtin_nontemporal_load(reinterpret_cast<const u32x4_u*>(reinterpret_cast<const unsigned*>(u) + src + 4));
        }
      }
    }
  }
#pragma unroll
  for (int j = 0; j < SP_UNROLL; ++j) {
    const long long q = q0 + (long long)j * TPB;  // byte index
    unsigned bits = 0;
    if (whole[j]) {
      if (DT == SM_BF16) {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          bits |= ge0_bf16(v0[j][k] & 0xFFFFu) << (2 * k);
          bits |= ge0_bf16(v0[j][k] >> 16) << (2 * k + 1);
        }
      } else {
#pragma unroll
        for (int k = 0; k < 4; ++k) bits |= (ge0_f32(v0[j][k]) << k) | (ge0_f32(v1[j][k]) << (k + 4));
      }
    } else {
      bits = sp_slow<DT, 8, ROWS>(D, u, q * 8);
    }
    bits |= __shfl_down(bits, 1, 64) << 8;
    bits |= __shfl_down(bits, 2, 64) << 16;
    if ((threadIdx.x & 3) == 0 && q < bytes_per_row) __builtin_nontemporal_store(bits, reinterpret_cast<unsigned*>(o + q));
  }
}

// Four signs as int8: +1 = 0x01, -1 = 0xFF.
__device__ __forceinline__ unsigned pm1_bytes(unsigned bits) {
  unsigned v = 0;
#pragma unroll
  for (int k = 0; k < 4; ++k) v |= (((bits >> k) & 1u) ? 0x01u : 0xFFu) << (8 * k);
  return v;
}

// int8 output: a thread turns 16 bytes of the source (8 bf16 or 4 f32 entries) into as many signs, SP8_UNROLL times,
// loads first.  Rows of source and output may start at any element.
constexpr int SP8_UNROLL = 4;

template <int DT, bool ROWS>
__global__ void __launch_bounds__(TPB) sm_sign_pack_int8_kernel(const sp_args a) {
  constexpr int E = (DT == SM_BF16) ? 8 : 4;
  const int di = sm_find(a.begin, a.n, blockIdx.x);
  const sm_sp_desc& D = a.d[di];
  const int local = blockIdx.x - a.begin.v[di];
  const int b = local / D.blocks_per_row, bx = local - b * D.blocks_per_row;
  const long long n = D.n;
  const void* u = sp_row<DT>(D, b);
  unsigned char* o = reinterpret_cast<unsigned char*>(D.out) + (long long)b * D.out_stride;
  const long long q0 = ((long long)bx * SP8_UNROLL) * TPB + threadIdx.x;
  u32x4 v[SP8_UNROLL];
  bool whole[SP8_UNROLL];
#pragma unroll
  for (int j = 0; j < SP8_UNROLL; ++j) {
    const long long e0 = (q0 + (long long)j * TPB) * E;
    v[j] = u32x4{0u, 0u, 0u, 0u};
    whole[j] = false;
    if (e0 + E <= n) {
      int room;
      const long long src = sp_source<ROWS>(D, e0, room);
      whole[j] = room >= E;
      if (whole[j])
        v[j] = __builtin_nontemporal_load(reinterpret_cast<const u32x4_u*>(
            DT == SM_BF16 ? (const void*)(reinterpret_cast<const unsigned short*>(u) + src)
                          : (const void*)(reinterpret_cast<const unsigned*>(u) + src)));
    }
  }
#pragma unroll
  for (int j = 0; j < SP8_UNROLL; ++j) {
    const long long e0 = (q0 + (long long)j * TPB) * E;
    if (e0 >= n) break;
    if (whole[j]) {
      unsigned bits = 0;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        if (DT == SM_BF16)
          bits |= (ge0_bf16(v[j][k] & 0xFFFFu) << (2 * k)) | (ge0_bf16(v[j][k] >> 16) << (2 * k + 1));
        else
          bits |= ge0_f32(v[j][k]) << k;
      }
      if (DT == SM_BF16)
        *reinterpret_cast<u32x2_u*>(o + e0) = u32x2{pm1_bytes(bits), pm1_bytes(bits >> 4)};
      else
        *reinterpret_cast<u32_u*>(o + e0) = pm1_bytes(bits);
    } else {
      const unsigned bits = sp_slow<DT, E, ROWS>(D, u, e0);
      for (int k = 0; k < E && e0 + k < n; ++k) o[e0 + k] = ((bits >> k) & 1u) ? 0x01 : 0xFF;
    }
  }
}

// ------------------------------------------------------------------ vote
// Voted bits only.  Bit-sliced counting: the M words of a position are added into
// PLANES binary counter planes with ripple carries (M < 2^PLANES), then the planes
// are compared with the threshold ceil(M/2) bit-serially from the top plane down.
// Adds the set bits of `x` into the bit-sliced counter `plane` (ripple carry).
template <int PLANES, typename W>
__device__ __forceinline__ void planes_add(W (&plane)[PLANES], W x) {
#pragma unroll
  for (int k = 0; k < PLANES; ++k) {
    const W t = plane[k] & x;
    plane[k] ^= x;
    x = t;
  }
}

// Adds eight words at once: full adders down to one carry into plane 3, then one ripple.  For the many planes of 256
// workers and more, where eight ripples are 16 operations per plane: bits from 300 workers, 0.1 / 1 / 17 M entries, by
// ripples 179 / 158 / 505 us, so 68 / 57 / 125 (the first by the latency of 38 rounds of loads).
template <int PLANES, typename W>
__device__ __forceinline__ void planes_add8(W (&plane)[PLANES], const W (&x)[8]) {
  if constexpr (PLANES <= 8) {
#pragma unroll
    for (int q = 0; q < 8; ++q) planes_add<PLANES>(plane, x[q]);
  } else {
    // sum <- sum + a + b of one weight; returns the carry
    auto add = [](W& sum, W a, W b) {
      const W d = sum ^ a, carry = (sum & a) | (d & b);
      sum = d ^ b;
      return carry;
    };
    const W two0 = add(plane[0], x[0], x[1]), two1 = add(plane[0], x[2], x[3]);
    const W four0 = add(plane[1], two0, two1);
    const W two2 = add(plane[0], x[4], x[5]), two3 = add(plane[0], x[6], x[7]);
    const W four1 = add(plane[1], two2, two3);
    W eight = add(plane[2], four0, four1);
#pragma unroll
    for (int k = 3; k < PLANES; ++k) {
      const W t = plane[k] & eight;
      plane[k] ^= eight;
      eight = t;
    }
  }
}

// Bit mask of the positions whose count is >= T.
template <int PLANES, typename W>
__device__ __forceinline__ W planes_ge(const W (&plane)[PLANES], unsigned T) {
  W gt = 0, eq = ~(W)0;
#pragma unroll
  for (int k = PLANES - 1; k >= 0; --k) {
    const W tb = ((T >> k) & 1u) ? ~(W)0 : (W)0;
    gt |= eq & plane[k] & ~tb;
    eq &= ~(plane[k] ^ tb);
  }
  return gt | eq;
}

// Workers are read eight at a time: all eight loads of a group are issued before the first is
// added, so a thread keeps 8 x 16 bytes in flight (rows beyond M read as zero words, which
// count nothing).
constexpr int VOTE_GROUP = 8;  // as many as planes_add8 takes
constexpr int VOTE8_GROUP = 4;  // with 16 bytes per load and 16 sums: eight cost the registers of every other wave

// f(number of workers, first worker) over workers [first, end) in groups of G, the number a constant in each group: the
// last group is not padded, so a thread does no arithmetic for workers that are not there.
template <int G, typename F>
__device__ __forceinline__ void for_workers(int first, int end, F f) {
  int p = first;
  for (; p + G <= end; p += G) f(std::integral_constant<int, G>(), p);
  switch (end - p) {
    case 1: f(std::integral_constant<int, 1>(), p); break;
    case 2: f(std::integral_constant<int, 2>(), p); break;
    case 3: f(std::integral_constant<int, 3>(), p); break;
    case 4: f(std::integral_constant<int, 4>(), p); break;
    case 5: f(std::integral_constant<int, 5>(), p); break;
    case 6: f(std::integral_constant<int, 6>(), p); break;
    case 7: f(std::integral_constant<int, 7>(), p); break;
    default: break;
  }
}

// A thread owns VB_PAIRS pairs of 64-bit words, TPB pairs apart (rows are 8-byte aligned with any stride: a
// pair is read with one 16-byte load only where row base and stride allow it).  Measured on 85 M entries, M = 8:
// one pair per thread 17.3 us, two 18.6 us, four 22.3 us.
constexpr int VB_PAIRS = 1;

template <int PLANES>
__global__ void __launch_bounds__(TPB) sm_vote_bits_kernel(const unsigned long long* __restrict__ signs, int M,
                                                           long long words, long long stride_words,
                                                           long long n, unsigned long long* __restrict__ voted) {
  typedef __attribute__((ext_vector_type(2))) unsigned long long u64x2;
  const bool vec_ok = ((stride_words & 1) == 0) && ((reinterpret_cast<uintptr_t>(signs) & 15) == 0);
  long long w0[VB_PAIRS];
  unsigned long long p0[VB_PAIRS][PLANES], p1[VB_PAIRS][PLANES];
#pragma unroll
  for (int r = 0; r < VB_PAIRS; ++r) {
    w0[r] = (((long long)blockIdx.x * VB_PAIRS + r) * TPB + threadIdx.x) * 2;
#pragma unroll
    for (int k = 0; k < PLANES; ++k) p0[r][k] = p1[r][k] = 0;
  }
  if (w0[0] >= words) return;
  for (int pb = 0; pb < M; pb += VOTE_GROUP) {
    unsigned long long a[VB_PAIRS][VOTE_GROUP], b[VB_PAIRS][VOTE_GROUP];
#pragma unroll
    for (int r = 0; r < VB_PAIRS; ++r) {
      const bool live = w0[r] < words, pair = w0[r] + 1 < words;
#pragma unroll
      for (int q = 0; q < VOTE_GROUP; ++q) {
        a[r][q] = b[r][q] = 0;
        if (live && pb + q < M) {
          const unsigned long long* src = signs + (long long)(pb + q) * stride_words + w0[r];
          if (vec_ok && pair) {
            const u64x2 v = __builtin_nontemporal_load(reinterpret_cast<const u64x2*>(src));
            a[r][q] = v[0];
            b[r][q] = v[1];
          } else {
            a[r][q] = __builtin_nontemporal_load(src);
            if (pair) b[r][q] = __builtin_nontemporal_load(src + 1);
          }
        }
      }
    }
#pragma unroll
    for (int r = 0; r < VB_PAIRS; ++r) {
      planes_add8<PLANES>(p0[r], a[r]);
      planes_add8<PLANES>(p1[r], b[r]);
    }
  }
  const unsigned T = (unsigned)((M + 1) / 2);  // vote = (count >= T)
  const bool out_vec = (reinterpret_cast<uintptr_t>(voted) & 15) == 0;
#pragma unroll
  for (int r = 0; r < VB_PAIRS; ++r) {
    if (w0[r] >= words) break;
    const bool pair = w0[r] + 1 < words;
    unsigned long long v[2] = {planes_ge<PLANES>(p0[r], T), planes_ge<PLANES>(p1[r], T)};
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const long long rem = n - (w0[r] + h) * 64;
      if (rem < 64) v[h] &= (rem <= 0) ? 0ull : ((1ull << rem) - 1ull);
    }
    if (pair && out_vec) {
      const u64x2 o = {v[0], v[1]};
      __builtin_nontemporal_store(o, reinterpret_cast<u64x2*>(voted + w0[r]));
    } else {
      voted[w0[r]] = v[0];
      if (pair) voted[w0[r] + 1] = v[1];
    }
  }
}

typedef sm_vote_desc vote_x_args;
struct vote_g_args {
  int n;
  int pad_;
  sm_starts<SM_VOTE_MAX_GROUP> begin;
  sm_vote_desc d[SM_VOTE_MAX_GROUP];
};
static_assert(sizeof(vote_g_args) <= 4096, "kernel arguments are limited to 4 KB");

// Stores of up to four consecutive results; `live` of them exist.
__device__ __forceinline__ void step4(float* w, float lr, const f32x4 old, unsigned bits, int live) {
  f32x4 o;
#pragma unroll
  for (int k = 0; k < 4; ++k) o[k] = __fsub_rn(old[k], __fmul_rn(lr, ((bits >> k) & 1u) ? 1.0f : -1.0f));
  if (live == 4) {
    __builtin_nontemporal_store(o, reinterpret_cast<f32x4_u*>(w));
  } else {
#pragma unroll
    for (int k = 0; k < 3; ++k)
      if (k < live) w[k] = o[k];
  }
}
__device__ __forceinline__ f32x4 load4(const float* w, int live) {
  f32x4 o = {0.f, 0.f, 0.f, 0.f};
  if (live == 4) {
    o = __builtin_nontemporal_load(reinterpret_cast<const f32x4_u*>(w));
  } else {
#pragma unroll
    for (int k = 0; k < 3; ++k)
      if (k < live) o[k] = w[k];
  }
  return o;
}
__device__ __forceinline__ void counts4(int32_t* c, const i32x4 v, int live) {
  if (live == 4) {
    *reinterpret_cast<i32x4_u*>(c) = v;
  } else {
#pragma unroll
    for (int k = 0; k < 3; ++k)
      if (k < live) c[k] = v[k];
  }
}
__device__ __forceinline__ unsigned pm1_bf16(unsigned two) {
  return ((two & 1u) ? 0x3F80u : 0xBF80u) | ((two & 2u) ? 0x3F800000u : 0xBF800000u);
}
// four voted entries in format vfmt at entry `at` of the output
__device__ __forceinline__ void voted4(void* voted, int vfmt, long long at, unsigned bits, int live) {
  if (vfmt == SM_VOTE_INT8) {
    unsigned char* o = reinterpret_cast<unsigned char*>(voted) + at;
    const unsigned v = pm1_bytes(bits);
    if (live == 4) {
      *reinterpret_cast<u32_u*>(o) = v;
    } else {
      for (int k = 0; k < live; ++k) o[k] = (unsigned char)(v >> (8 * k));
    }
  } else if (vfmt == SM_VOTE_BF16) {
    unsigned short* o = reinterpret_cast<unsigned short*>(voted) + at;
    const u32x2 v = {pm1_bf16(bits), pm1_bf16(bits >> 2)};
    if (live == 4) {
      *reinterpret_cast<u32x2_u*>(o) = v;
    } else {
      for (int k = 0; k < live; ++k) o[k] = (unsigned short)(v[k >> 1] >> (16 * (k & 1)));
    }
  } else {
    float* o = reinterpret_cast<float*>(voted) + at;
    f32x4 v;
#pragma unroll
    for (int k = 0; k < 4; ++k) v[k] = ((bits >> k) & 1u) ? 1.0f : -1.0f;
    if (live == 4) {
      *reinterpret_cast<f32x4_u*>(o) = v;
    } else {
#pragma unroll
      for (int k = 0; k < 3; ++k)
        if (k < live) o[k] = v[k];
    }
  }
}

// Voted bits from int8 signs: a thread sums 8 consecutive entries over the workers and makes a byte of them; the bytes
// of four lanes leave as one 32-bit store.
__global__ void __launch_bounds__(TPB) sm_vote_int8_bits_kernel(const signed char* __restrict__ signs, int M,
                                                                long long n, long long stride_bytes,
                                                                unsigned char* __restrict__ voted,
                                                                long long bytes_out) {
  const long long q = (long long)blockIdx.x * TPB + threadIdx.x;
  const long long e0 = q * 8;
  int c[8] = {0, 0, 0, 0, 0, 0, 0, 0};
  unsigned bits = 0;
  if (e0 + 8 <= n) {
#pragma unroll 4
    for (int p = 0; p < M; ++p) {
      const u32x2 v = __builtin_nontemporal_load(reinterpret_cast<const u32x2_u*>(signs + (long long)p * stride_bytes + e0));
#pragma unroll
      for (int k = 0; k < 8; ++k) c[k] += (int)(signed char)(v[k >> 2] >> (8 * (k & 3)));
    }
#pragma unroll
    for (int k = 0; k < 8; ++k) bits |= (c[k] >= 0 ? 1u : 0u) << k;
  } else {
    for (int k = 0; k < 8 && e0 + k < n; ++k) {
      int t = 0;
      for (int p = 0; p < M; ++p) t += signs[(long long)p * stride_bytes + e0 + k];
      bits |= (t >= 0 ? 1u : 0u) << k;
    }
  }
  bits |= __shfl_down(bits, 1, 64) << 8;
  bits |= __shfl_down(bits, 2, 64) << 16;
  if ((threadIdx.x & 3) == 0 && q < bytes_out) *reinterpret_cast<unsigned*>(voted + q) = bits;  // bytes_out % 8 == 0
}

// ------------------------------------------------------------------ update after a local polar step
struct upd_args {
  int n;
  int pad_;
  sm_starts<SM_UPD_MAX_GROUP> begin;
  sm_upd_desc d[SM_UPD_MAX_GROUP];
};

// A workgroup owns UPD_ITERS * TPB groups of four entries, each inside a row (the last group of a row may be short),
// UPD_ITERS per thread; all loads are issued before the first store.
constexpr int UPD_ITERS = 4;
constexpr int UPD_CHUNK = UPD_ITERS * TPB;  // groups

__global__ void __launch_bounds__(TPB) sm_update_kernel(const upd_args g) {
  const int di = sm_find(g.begin, g.n, blockIdx.x);
  const sm_upd_desc& D = g.d[di];
  float* __restrict__ w = D.w;
  const bf16_t* __restrict__ d = D.d;
  const int cols = D.cols, ld = D.ld;
  const float step = D.kappa ? __fmul_rn(D.step, D.kappa[0]) : D.step;
  const int q = (cols + 3) >> 2;
  const long long groups = (long long)D.rows * q;
  const long long base = (long long)(blockIdx.x - g.begin.v[di]) * UPD_CHUNK + threadIdx.x;
  bf16x4 h[UPD_ITERS];
  f32x4 wv[UPD_ITERS];
  long long at[UPD_ITERS];
  int live[UPD_ITERS];
#pragma unroll
  for (int it = 0; it < UPD_ITERS; ++it) {
    const long long t = base + it * TPB;
    h[it] = bf16x4{0, 0, 0, 0};
    wv[it] = f32x4{0.f, 0.f, 0.f, 0.f};
    at[it] = 0;
    live[it] = 0;
    if (t < groups) {
      long long r;
      int c;
      sm_row_of(D.quads, q, t, r, c);
      c *= 4;
      at[it] = r * cols + c;
      live[it] = min(4, cols - c);
      h[it] = __builtin_nontemporal_load(reinterpret_cast<const bf16x4*>(d + r * ld + c));
      wv[it] = load4(w + at[it], live[it]);
    }
  }
#pragma unroll
  for (int it = 0; it < UPD_ITERS; ++it) {
    if (live[it] == 0) break;
#pragma unroll
    for (int k = 0; k < 4; ++k) wv[it][k] = __fsub_rn(wv[it][k], __fmul_rn(step, (float)h[it][k]));
    if (live[it] == 4) {
      __builtin_nontemporal_store(wv[it], reinterpret_cast<f32x4_u*>(w + at[it]));
    } else {
#pragma unroll
      for (int k = 0; k < 3; ++k)
        if (k < live[it]) w[at[it] + k] = wv[it][k];
    }
  }
}

}  // namespace

// =================================================================== host side
int sm_launch_momentum(signmuon_ctx* ctx, const sm_mom_desc* descs, int n, int M, float beta, float wd) {
  int done = 0;
  while (done < n) {
    const int g = std::min(n - done, SM_MOM_MAX_GROUP);
    mom_args a;
    sm_starts_clear(a.begin);
    a.n = g;
    a.M = M;
    a.beta = beta;
    a.omb = 1.0f - beta;
    a.wd = wd;
    long long blocks = 0;
    for (int i = 0; i < g; ++i) {
      a.d[i] = descs[done + i];
      a.begin.v[i] = (int)blocks;
      blocks += (long long)M * a.d[i].chunks;
    }
    if (blocks > 0x7FFFFFFFLL) return sm_fail(ctx, SM_EUNSUPPORTED, "momentum: too many entries for one launch");
    a.shift = 0;
    while ((blocks >> a.shift) >= 64) ++a.shift;
    for (unsigned& w : a.start) w = 0;
    for (int k = 0, bi = 0; k < 64; ++k) {
      while (bi + 1 < g && ((long long)k << a.shift) >= a.begin.v[bi + 1]) ++bi;
      a.start[k >> 2] |= (unsigned)bi << (8 * (k & 3));
    }
    if (blocks > 0) {
      sm_launch_scope sc(ctx, SM_K_MOMENTUM);
      hipLaunchKernelGGL(sm_momentum_kernel, dim3((unsigned)blocks), dim3(TPB), 0, ctx->stream, a);
    }
    SM_HIP(ctx, hipGetLastError());
    done += g;
  }
  return SM_OK;
}

int sm_launch_reduce_partials(signmuon_ctx* ctx, const float* partial, int chunks, int count, float* sumsq) {
  sm_launch_scope sc(ctx, SM_K_OTHER);
  hipLaunchKernelGGL(sm_reduce_partials_kernel, dim3(count), dim3(TPS), 0, ctx->stream, partial, chunks, sumsq);
  SM_HIP(ctx, hipGetLastError());
  return SM_OK;
}

int sm_launch_sigma_group(signmuon_ctx* ctx, const sm_sigma_desc* descs, int n, float eps) {
  int done = 0;
  while (done < n) {
    const int g = std::min(n - done, SM_SIGMA_MAX_GROUP);
    sigma_args a;
    sm_starts_clear(a.begin);
    a.n = g;
    a.eps = eps;
    int blocks = 0;
    for (int i = 0; i < g; ++i) {
      a.d[i] = descs[done + i];
      a.begin.v[i] = blocks;
      blocks += a.d[i].count;
    }
    if (blocks > 0) {
      sm_launch_scope sc(ctx, SM_K_OTHER);
      hipLaunchKernelGGL(sm_sigma_group_kernel, dim3(blocks), dim3(TPS), 0, ctx->stream, a);
    }
    SM_HIP(ctx, hipGetLastError());
    done += g;
  }
  return SM_OK;
}

int sm_launch_sign_pack_group(signmuon_ctx* ctx, const sm_sp_desc* descs, int n, int dtype, int fmt, int M) {
  int done = 0;
  while (done < n) {
    const int g = std::min(n - done, SM_SP_MAX_GROUP);
    sp_args a;
    sm_starts_clear(a.begin);
    a.n = g;
    a.pad_ = 0;
    // entries per workgroup
    const int per_block = TPB * (fmt == SM_SIGN_1BIT ? 8 * SP_UNROLL : (dtype == SM_BF16 ? 8 : 4) * SP8_UNROLL);
    long long blocks = 0;
    bool rows = false;
    for (int i = 0; i < g; ++i) {
      sm_sp_desc& D = a.d[i];
      D = descs[done + i];
      D.by_cols = sm_div_by((unsigned)D.cols);
      rows = rows || D.ld != D.cols;
      D.blocks_per_row = (int)(((D.n + 63) / 64 * 64 + per_block - 1) / per_block);
      a.begin.v[i] = (int)blocks;
      blocks += (long long)D.blocks_per_row * M;
    }
    if (blocks > 0x7FFFFFFFLL) return sm_fail(ctx, SM_EUNSUPPORTED, "sign pack: too many entries for one launch");
    if (blocks > 0) {
      const dim3 grid((unsigned)blocks), block(TPB);
      sm_launch_scope sc(ctx, SM_K_SIGN_PACK);
#define SP_LAUNCH(KERNEL, DT)                                                                                  \
  if (rows) hipLaunchKernelGGL((KERNEL<DT, true>), grid, block, 0, ctx->stream, a);                            \
  else hipLaunchKernelGGL((KERNEL<DT, false>), grid, block, 0, ctx->stream, a)
      if (fmt == SM_SIGN_1BIT && dtype == SM_BF16) { SP_LAUNCH(sm_sign_pack_bits_kernel, SM_BF16); }
      else if (fmt == SM_SIGN_1BIT) { SP_LAUNCH(sm_sign_pack_bits_kernel, SM_F32); }
      else if (dtype == SM_BF16) { SP_LAUNCH(sm_sign_pack_int8_kernel, SM_BF16); }
      else { SP_LAUNCH(sm_sign_pack_int8_kernel, SM_F32); }
#undef SP_LAUNCH
    }
    SM_HIP(ctx, hipGetLastError());
    done += g;
  }
  return SM_OK;
}

int sm_launch_sign_pack(signmuon_ctx* ctx, const void* u, int dtype, int batch, long long n, int fmt, void* out,
                        long long out_stride_bytes) {
  sm_sp_desc D;
  D.u = u;
  D.out = out;
  D.n = n;
  D.batch_stride = n;
  D.out_stride = out_stride_bytes;
  D.cols = D.ld = (int)n;
  D.blocks_per_row = 0;
  D.pad_ = 0;
  return sm_launch_sign_pack_group(ctx, &D, 1, dtype, fmt, batch);
}

int sm_launch_vote(signmuon_ctx* ctx, const sm_vote_args& v) {
  const long long n = v.n;
  const bool want_bits = v.voted && v.vfmt == SM_VOTE_BITS;
  const bool want_expand = v.counts || v.w || (v.voted && v.vfmt != SM_VOTE_BITS);
  if (want_bits) {
    sm_launch_scope sc(ctx, SM_K_VOTE);
    if (v.fmt == SM_SIGN_1BIT) {
      const long long words = (n + 63) / 64;
      const dim3 grid((unsigned)(((words + 1) / 2 + TPB * VB_PAIRS - 1) / (TPB * VB_PAIRS)));  // VB_PAIRS word pairs per thread
      const unsigned long long* sp = reinterpret_cast<const unsigned long long*>(v.signs);
      unsigned long long* vp = reinterpret_cast<unsigned long long*>(v.voted);
      if (v.M < 8)
        hipLaunchKernelGGL(sm_vote_bits_kernel<3>, grid, dim3(TPB), 0, ctx->stream, sp, v.M, words, v.stride_bytes / 8, n, vp);
      else if (v.M < 32)
        hipLaunchKernelGGL(sm_vote_bits_kernel<5>, grid, dim3(TPB), 0, ctx->stream, sp, v.M, words, v.stride_bytes / 8, n, vp);
      else if (v.M < 256)
        hipLaunchKernelGGL(sm_vote_bits_kernel<8>, grid, dim3(TPB), 0, ctx->stream, sp, v.M, words, v.stride_bytes / 8, n, vp);
      else
        hipLaunchKernelGGL(sm_vote_bits_kernel<31>, grid, dim3(TPB), 0, ctx->stream, sp, v.M, words, v.stride_bytes / 8, n, vp);
    } else {
      const long long bytes_out = 8 * ((n + 63) / 64);
      hipLaunchKernelGGL(sm_vote_int8_bits_kernel, dim3((unsigned)((bytes_out + TPB - 1) / TPB)), dim3(TPB), 0,
                         ctx->stream, reinterpret_cast<const signed char*>(v.signs), v.M, n, v.stride_bytes,
                         reinterpret_cast<unsigned char*>(v.voted), bytes_out);
    }
    SM_HIP(ctx, hipGetLastError());
  }
  if (want_expand) {
    sm_vote_desc a;
    a.signs = v.signs;
    a.n = n;
    a.stride_bytes = v.stride_bytes;
    a.voted = (v.voted && v.vfmt != SM_VOTE_BITS) ? v.voted : nullptr;
    a.counts = v.counts;
    a.w = v.w;
    a.lr = v.lr_scaled;
    a.M = v.M;
    a.vfmt = v.vfmt;
    a.cols = a.sld = a.ld = 0;
    return sm_launch_vote_group(ctx, &a, 1, v.fmt);
  }
  return SM_OK;
}

// Expanding vote over 1-bit signs: a lane takes one 32-bit word of every worker's buffer, counted bit-sliced
// (PLANES binary counter planes, M < 2^PLANES) and compared with ceil(M/2) as in sm_vote_bits_kernel.  The 2048 votes
// of a wave are then spread over its lanes so that every store (and every load of W) covers consecutive addresses:
// lane l writes 8 consecutive bf16 per store, and takes 4 consecutive weights or counts at a time.  The loads of eight
// workers, and the eight loads of W, are in flight together (fused W update on 85 M entries, M = 8: 125 us; two or four
// runs of words per wave: 136 us).
// ROWS: the signs are rows of sld entries, so a word also has a row and a number of entries that count; the flat
// outputs then start at any element.  Otherwise one run of n entries, whose last word may be partial.
template <int PLANES, bool ROWS>
__global__ void __launch_bounds__(TPB) sm_vote_wide_kernel(const vote_g_args g) {
  const int di = sm_find(g.begin, g.n, blockIdx.x);
  const vote_x_args& a = g.d[di];
  const long long words = (a.n + 31) >> 5;
  const int lane = threadIdx.x & 63;
  const long long w0 = (long long)(blockIdx.x - g.begin.v[di]) * TPB + (threadIdx.x & ~63);  // the wave's first word
  if (w0 >= words) return;
  const long long stride_w = a.stride_bytes >> 2;
  const unsigned* sbase = reinterpret_cast<const unsigned*>(a.signs) + w0 + lane;
  const bool in = w0 + lane < words;
  unsigned plane[PLANES];
#pragma unroll
  for (int k = 0; k < PLANES; ++k) plane[k] = 0;
  for (int pb = 0; pb < a.M; pb += VOTE_GROUP) {
    unsigned x[VOTE_GROUP];
#pragma unroll
    for (int q = 0; q < VOTE_GROUP; ++q) {
      x[q] = 0;
      if (in && pb + q < a.M) x[q] = __builtin_nontemporal_load(sbase + (long long)(pb + q) * stride_w);
    }
    planes_add8<PLANES>(plane, x);
  }
  const unsigned v = planes_ge<PLANES>(plane, (unsigned)((a.M + 1) / 2));
  int row = 0, live = 0;  // of the lane's own word
  if (ROWS && in) {
    long long r;
    int c;
    sm_row_of(a.by_row, a.sld >> 5, w0 + lane, r, c);
    row = (int)r;
    live = min(32, a.cols - 32 * c);
  }
  // entries that count in word t of the wave, and where its first entry lies in a flat output
  auto live_of = [&](int t) {
    if (ROWS) return __shfl(live, t, 64);
    const long long rem = a.n - 32 * (w0 + t);
    return (int)(rem < 0 ? 0 : rem > 32 ? 32 : rem);
  };
  auto flat_of = [&](int t) {
    const long long e = 32 * (w0 + t);
    return ROWS ? e - (long long)__shfl(row, t, 64) * (a.sld - a.cols) : e;
  };
  if (a.voted && a.vfmt == SM_VOTE_BF16) {
    const bool padded = ROWS && a.ld == a.sld;
    unsigned short* o = reinterpret_cast<unsigned short*>(a.voted);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      // chunk 64 k + lane of the wave's 256 chunks of 8 entries: byte (lane & 3) of word 16 k + lane / 4
      const int t = 16 * k + (lane >> 2), e = 8 * (lane & 3);
      const unsigned bits = (__shfl(v, t, 64) >> e) & 0xFFu;
      const int lv = live_of(t) - e;
      const long long flat = flat_of(t) + e;
      u32x4 h;
#pragma unroll
      for (int q = 0; q < 4; ++q) h[q] = pm1_bf16(bits >> (2 * q));
      if (padded) {
#pragma unroll
        for (int q = 0; q < 4; ++q) h[q] &= (2 * q < lv ? 0xFFFFu : 0u) | (2 * q + 1 < lv ? 0xFFFF0000u : 0u);
        if (w0 + t < words) *reinterpret_cast<u32x4*>(o + 32 * (w0 + t) + e) = h;
      } else if (lv >= 8) {
        *reinterpret_cast<u32x4_u*>(o + flat) = h;
      } else if (lv > 0) {
        for (int q = 0; q < lv; ++q) o[flat + q] = (unsigned short)(pm1_bf16(bits >> q));
      }
    }
  } else if (a.voted) {
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const int t = 8 * k + (lane >> 3), e = 4 * (lane & 7);
      const unsigned bits = (__shfl(v, t, 64) >> e) & 0xFu;
      const int lv = live_of(t) - e;
      const long long flat = flat_of(t) + e;
      if (lv > 0) voted4(a.voted, a.vfmt, flat, bits, min(lv, 4));
    }
  }
  if (a.counts) {
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const int t = 8 * k + (lane >> 3), e = 4 * (lane & 7);
      i32x4 c = {0, 0, 0, 0};
#pragma unroll
      for (int b = 0; b < PLANES; ++b) {
        const unsigned x = __shfl(plane[b], t, 64) >> e;
#pragma unroll
        for (int q = 0; q < 4; ++q) c[q] += (int)((x >> q) & 1u) << b;
      }
      const int lv = live_of(t) - e;
      const long long flat = flat_of(t) + e;
      if (lv > 0) counts4(a.counts + flat, c, min(lv, 4));
    }
  }
  if (a.w) {
    f32x4 wv[8];
    int lv[8];
    long long at[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const int t = 8 * k + (lane >> 3), e = 4 * (lane & 7);
      lv[k] = min(live_of(t) - e, 4);
      at[k] = flat_of(t) + e;
      wv[k] = load4(a.w + at[k], lv[k]);
    }
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const unsigned bits = (__shfl(v, 8 * k + (lane >> 3), 64) >> (4 * (lane & 7))) & 0xFu;
      if (lv[k] > 0) step4(a.w + at[k], a.lr, wv[k], bits, lv[k]);
    }
  }
}

// Expanding vote over int8 signs, one thread = 16 consecutive entries (one 16-byte load per worker, one worker at a
// time), for matrices of n % 16 == 0 entries in 16-byte aligned rows, votes int8 or flat bf16: where the signs are nearly
// all of the bytes, one stream after the other is the better order on rows a power of two apart (counts alone, 32
// workers of 8.4 M entries: 52 us, 60 in sm_vote_int8_kernel; of 10 M entries 70 and 66).
__global__ void __launch_bounds__(TPB) sm_vote_int8_wide_kernel(const vote_g_args g) {
  const int di = sm_find(g.begin, g.n, blockIdx.x);
  const vote_x_args& a = g.d[di];
  const long long t = (long long)(blockIdx.x - g.begin.v[di]) * TPB + threadIdx.x;
  const long long e0 = t * 16;
  if (e0 >= a.n) return;
  int c[16];
#pragma unroll
  for (int k = 0; k < 16; ++k) c[k] = 0;
  const unsigned char* base = reinterpret_cast<const unsigned char*>(a.signs) + e0;
  for (int p = 0; p < a.M; ++p) {
    const u32x4 v = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(base + (long long)p * a.stride_bytes));
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int k = 0; k < 4; ++k) c[4 * q + k] += (int)(signed char)(v[q] >> (8 * k));
  }
  unsigned bits = 0;
#pragma unroll
  for (int k = 0; k < 16; ++k) bits |= (c[k] >= 0 ? 1u : 0u) << k;
  if (a.counts) {
#pragma unroll
    for (int q = 0; q < 4; ++q)
      *reinterpret_cast<i32x4*>(a.counts + e0 + 4 * q) = i32x4{c[4 * q], c[4 * q + 1], c[4 * q + 2], c[4 * q + 3]};
  }
  if (a.w) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      f32x4* w = reinterpret_cast<f32x4*>(a.w + e0 + 4 * q);
      f32x4 o = *w;
#pragma unroll
      for (int k = 0; k < 4; ++k) o[k] = __fsub_rn(o[k], __fmul_rn(a.lr, c[4 * q + k] >= 0 ? 1.0f : -1.0f));
      *w = o;
    }
  }
  if (!a.voted) return;
  if (a.vfmt == SM_VOTE_INT8) {
    u32x4 o;
#pragma unroll
    for (int q = 0; q < 4; ++q) o[q] = pm1_bytes(bits >> (4 * q));
    *reinterpret_cast<u32x4*>(reinterpret_cast<unsigned char*>(a.voted) + e0) = o;
  } else {
    bf16_t* ob = reinterpret_cast<bf16_t*>(a.voted) + e0;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      u32x4 o;
#pragma unroll
      for (int q = 0; q < 4; ++q) o[q] = pm1_bf16(bits >> (8 * h + 2 * q));
      *reinterpret_cast<u32x4*>(ob + 8 * h) = o;
    }
  }
}

// Group t of four entries of the source: how many of them count, and where the first lies in a flat output.
template <bool ROWS>
__device__ __forceinline__ void vote_place(const vote_x_args& a, long long t, int& live, long long& at) {
  live = 0;
  at = 4 * t;
  if (4 * t >= a.n) return;
  if (ROWS) {
    long long r;
    int q;
    sm_row_of(a.by_row, a.sld >> 2, t, r, q);
    live = max(0, min(4, a.cols - 4 * q));
    at = r * a.cols + 4 * q;
  } else {
    live = (int)(a.n - 4 * t < 4 ? a.n - 4 * t : 4);
  }
}

// All outputs of group t, which lies inside the source; wv: its weights, where there are any.
template <bool ROWS>
__device__ __forceinline__ void vote_out(const vote_x_args& a, long long t, int live, long long at, unsigned bits,
                                         const i32x4& counts, const f32x4& wv) {
  if (a.voted && ROWS && a.ld == a.sld) {  // bf16 with padded rows: zeros beyond cols
    const u32x2 h = {pm1_bf16(bits) & ((0 < live ? 0xFFFFu : 0u) | (1 < live ? 0xFFFF0000u : 0u)),
                     pm1_bf16(bits >> 2) & ((2 < live ? 0xFFFFu : 0u) | (3 < live ? 0xFFFF0000u : 0u))};
    *reinterpret_cast<u32x2*>(reinterpret_cast<unsigned short*>(a.voted) + 4 * t) = h;
  }
  if (live == 0) return;
  if (a.voted && !(ROWS && a.ld == a.sld)) voted4(a.voted, a.vfmt, at, bits, live);
  if (a.counts) counts4(a.counts + at, counts, live);
  if (a.w) step4(a.w + at, a.lr, wv, bits, live);
}

// Expanding vote, a lane takes GROUPS times four entries, a workgroup's width apart: no exchange between lanes, so the
// chain from the signs to the results is short, and accesses of every output are consecutive across lanes.  1 bit: the
// entries' bits out of every worker's word (eight lanes read the same one), counted in the four bytes of a register, 248
// workers at most before the bytes are taken out.  us, one group (four where it says so) / the other form of the
// transport (sm_vote_wide_kernel, sm_vote_int8_kernel):
//   1 bit, bf16 votes + counts + update   0.26 M entries, M = 16   4.9 / 7.5      4 M, M = 1 (four)   10.1 / 13.0
//                                         33 M, M = 8   73 / 76                   33 M, M = 32   134 / 94
//   1 bit, counts                         33 M, M = 8   25 / 32                   1 bit, bf16 votes   8 M, M = 8   7.9 / 6.2
//   int8, counts                          33 M, M = 8   60 / 75                   4 M, M = 16   18.9 / 17.3
//   int8, f32 votes                       2 M, M = 8   4.5 / 5.5                  4 M, M = 32   31.5 / 30.2
// ROWS as in sm_vote_wide_kernel.
template <int FMT, bool ROWS, int GROUPS>
__global__ void __launch_bounds__(TPB) sm_vote_narrow_kernel(const vote_g_args g) {
  constexpr int AHEAD = GROUPS > 1 ? 4 : VOTE_GROUP;  // workers in flight
  const int di = sm_find(g.begin, g.n, blockIdx.x);
  const vote_x_args& a = g.d[di];
  const long long first = (long long)(blockIdx.x - g.begin.v[di]) * TPB * GROUPS;
  const long long t0 = first + threadIdx.x;
  i32x4 c[GROUPS];
#pragma unroll
  for (int j = 0; j < GROUPS; ++j) c[j] = i32x4{0, 0, 0, 0};
  // whole: every group of the workgroup lies inside the buffer with all four entries
  auto count = [&](auto whole) {
    bool full[GROUPS];
#pragma unroll
    for (int j = 0; j < GROUPS; ++j) full[j] = decltype(whole)::value || 4 * (t0 + j * TPB) + (FMT == SM_SIGN_1BIT ? 1 : 4) <= a.n;
    if (FMT == SM_SIGN_1BIT) {
      const unsigned* base = reinterpret_cast<const unsigned*>(a.signs) + (t0 >> 3);
      const int sh = 4 * (int)(t0 & 7);
      const long long stride_w = a.stride_bytes >> 2;
      for (int p0 = 0; p0 < a.M; p0 += 31 * VOTE_GROUP) {
        unsigned acc[GROUPS] = {};
        for_workers<AHEAD>(p0, min(a.M, p0 + 31 * VOTE_GROUP), [&](auto number, int p) {
          constexpr int N = decltype(number)::value;
          unsigned x[GROUPS][N];
#pragma unroll
          for (int j = 0; j < GROUPS; ++j)
#pragma unroll
            for (int q = 0; q < N; ++q) x[j][q] = full[j] ? base[(long long)(p + q) * stride_w + j * (TPB / 8)] : 0u;
#pragma unroll
          for (int j = 0; j < GROUPS; ++j)
#pragma unroll
            for (int q = 0; q < N; ++q) acc[j] += (((x[j][q] >> sh) & 0xFu) * 0x00204081u) & 0x01010101u;
        });
#pragma unroll
        for (int j = 0; j < GROUPS; ++j)
#pragma unroll
          for (int k = 0; k < 4; ++k) c[j][k] += (int)((acc[j] >> (8 * k)) & 0xFFu);
      }
    } else {
      const signed char* src = reinterpret_cast<const signed char*>(a.signs) + 4 * t0;
      for_workers<AHEAD>(0, a.M, [&](auto number, int p) {
        constexpr int N = decltype(number)::value;
        unsigned x[GROUPS][N];
#pragma unroll
        for (int q = 0; q < N; ++q)
#pragma unroll
          for (int j = 0; j < GROUPS; ++j)
            x[j][q] = full[j] ? __builtin_nontemporal_load(reinterpret_cast<const u32_u*>(src + (long long)(p + q) * a.stride_bytes + 4 * j * TPB)) : 0u;
#pragma unroll
        for (int j = 0; j < GROUPS; ++j)
#pragma unroll
          for (int q = 0; q < N; ++q)
#pragma unroll
            for (int k = 0; k < 4; ++k) c[j][k] += (int)(signed char)(x[j][q] >> (8 * k));
      });
#pragma unroll
      for (int j = 0; j < GROUPS; ++j)
        if (!full[j] && 4 * (t0 + j * TPB) < a.n)  // up to three entries at the end of the buffer
          for (int p = 0; p < a.M; ++p)
#pragma unroll
            for (int k = 0; k < 3; ++k)
              if (4 * (t0 + j * TPB) + k < a.n) c[j][k] += src[(long long)p * a.stride_bytes + 4 * j * TPB + k];
    }
  };
  int live[GROUPS];
  long long at[GROUPS];
  f32x4 wv[GROUPS];
  auto weights = [&]() {
#pragma unroll
    for (int j = 0; j < GROUPS; ++j) {
      vote_place<ROWS>(a, t0 + j * TPB, live[j], at[j]);
      if (a.w) wv[j] = load4(a.w + at[j], live[j]);
    }
  };
  if (GROUPS == 1) weights();  // requested before the signs; with four groups after them (6.2 M, M = 4, all outputs: 22.5 / 17.8 us)
  if (4 * (first + GROUPS * TPB) <= a.n) count(std::true_type());
  else count(std::false_type());
  if (GROUPS > 1) weights();
#pragma unroll
  for (int j = 0; j < GROUPS; ++j) {
    const long long t = t0 + j * TPB;
    if (4 * t >= a.n) break;
    unsigned bits = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) bits |= ((FMT == SM_SIGN_1BIT ? 2 * c[j][k] >= a.M : c[j][k] >= 0) ? 1u : 0u) << k;
    vote_out<ROWS>(a, t, live[j], at[j], bits, c[j], wv[j]);
  }
}

// Expanding vote over int8 signs for many workers and entries (at least 16 of them).  A wave takes 1024 consecutive
// entries: a lane sums 16 of them (one 16-byte load per worker, four workers in flight), the int32 sums change owners
// through the wave's 4 KB of LDS, and a lane then has four groups of four entries, 256 apart, so that the accesses of
// weights and counts are consecutive across lanes.  The weights are requested before the signs.  The lane at the end of
// the buffer reads its last 16 bytes and shifts out what lies before its own entries.  ROWS as in sm_vote_wide_kernel.
template <bool ROWS>
__global__ void __launch_bounds__(TPB) sm_vote_int8_kernel(const vote_g_args g) {
  __shared__ __attribute__((aligned(16))) unsigned char sums[TPB * 64];
  const int di = sm_find(g.begin, g.n, blockIdx.x);
  const vote_x_args& a = g.d[di];
  const int lane = threadIdx.x & 63;
  const long long run = ((long long)(blockIdx.x - g.begin.v[di]) * TPB + (threadIdx.x & ~63)) * 16;
  if (run >= a.n) return;  // the wave as a whole
  f32x4 wv[4];
  int live[4];
  long long at[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    vote_place<ROWS>(a, run / 4 + 64 * k + lane, live[k], at[k]);
    if (a.w) wv[k] = load4(a.w + at[k], live[k]);
  }
  int c[16];
#pragma unroll
  for (int k = 0; k < 16; ++k) c[k] = 0;
  const long long e0 = run + 16 * lane;
  const int past = e0 + 16 <= a.n ? 0 : e0 >= a.n ? 16 : (int)(e0 + 16 - a.n);  // entries of the lane beyond the buffer
  if (past < 16) {
    const signed char* src = reinterpret_cast<const signed char*>(a.signs) + e0 - past;
    for_workers<VOTE8_GROUP>(0, a.M, [&](auto count, int p) {
      constexpr int N = decltype(count)::value;
      u32x4 v[N];
#pragma unroll
      for (int q = 0; q < N; ++q)
        v[q] = __builtin_nontemporal_load(reinterpret_cast<const u32x4_u*>(src + (long long)(p + q) * a.stride_bytes));
      if (past) {
#pragma unroll
        for (int q = 0; q < N; ++q)
          v[q] = __builtin_bit_cast(u32x4, __builtin_bit_cast(unsigned __int128, v[q]) >> (8 * past));
      }
#pragma unroll
      for (int q = 0; q < N; ++q)
#pragma unroll
        for (int k = 0; k < 16; ++k) c[k] += (int)(signed char)(v[q][k >> 2] >> (8 * (k & 3)));
    });
  }
  // lane l's sums of entries 16 l + 4 j .. + 3 at byte 64 l + 16 (j ^ (l / 4 mod 4)): no bank conflicts either way
  unsigned char* share = sums + (threadIdx.x & ~63) * 64;
#pragma unroll
  for (int j = 0; j < 4; ++j)
    *reinterpret_cast<i32x4*>(share + 64 * lane + 16 * (j ^ ((lane >> 2) & 3))) = i32x4{c[4 * j], c[4 * j + 1], c[4 * j + 2], c[4 * j + 3]};
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const long long t = run / 4 + 64 * k + lane;
    const i32x4 s = *reinterpret_cast<const i32x4*>(share + 1024 * k + 64 * (lane >> 2) + 16 * ((lane & 3) ^ ((lane >> 4) & 3)));
    unsigned bits = 0;
#pragma unroll
    for (int q = 0; q < 4; ++q) bits |= (s[q] >= 0 ? 1u : 0u) << q;
    if (4 * t >= a.n) break;
    vote_out<ROWS>(a, t, live[k], at[k], bits, s, wv[k]);
  }
}

int sm_launch_vote_group(signmuon_ctx* ctx, const sm_vote_desc* descs, int n, int fmt) {
  int done = 0;
  while (done < n) {
    const int g = std::min(n - done, SM_VOTE_MAX_GROUP);
    vote_g_args a;
    sm_starts_clear(a.begin);
    a.n = g;
    a.pad_ = 0;
    bool rows = false, counts = false;
    int max_m = 0;
    long long entries = 0, shortest = 16;
    const long long one_round = (long long)ctx->n_cu * 4 * 8 * 64 * 4;
    bool whole = true, votes_alone = true;  // what sm_vote_int8_wide_kernel needs
    for (int i = 0; i < g; ++i) {
      const sm_vote_desc& d = descs[done + i];
      rows = rows || d.sld != 0;
      counts = counts || d.counts;
      entries += d.n;
      shortest = std::min(shortest, d.n);
      max_m = std::max(max_m, d.M);
      votes_alone = votes_alone && !d.w && !d.counts;
      whole = whole && !d.sld && d.n % 16 == 0 && d.stride_bytes % 16 == 0 && sm_aligned(d.signs, 16) && sm_aligned(d.voted, 16) &&
              sm_aligned(d.w, 16) && sm_aligned(d.counts, 16) && (!d.voted || d.vfmt == SM_VOTE_INT8 || d.vfmt == SM_VOTE_BF16);
    }
    // Four entries per lane (sm_vote_narrow_kernel, figures there) where the launch is one round of its waves, eight per
    // SIMD: latency counts.  Beyond, 1-bit signs take it with counts, which the wide form has to gather from other
    // lanes plane by plane, until the eightfold reads of the words outweigh that (between 16 and 32 workers); int8 signs
    // up to 8 workers, above which requests of four bytes bound it.  Whole int8 matrices go 16 entries per lane for
    // votes alone, and for any output where many workers' signs outweigh it.
    const bool wide8 = fmt == SM_SIGN_INT8 && whole && (votes_alone || (max_m >= 16 && entries >= 2 * one_round));
    const bool narrow = fmt == SM_SIGN_1BIT ? entries <= one_round || (counts && max_m < 32)
                                            : !wide8 && (max_m <= 8 || entries <= one_round || shortest < 16);
    // Four groups per lane where few workers leave a lane few loads.  int8, int8 votes + counts, one group / four, us:
    // 6.2 M entries, M = 1 / 4 / 6 / 8: 9.8 / 7.5, 14.0 / 10.7, 14.4 / 13.9, 17.1 / 16.9; 12 M: 17.0 / 14.7, 25.6 / 22.0,
    // 25.1 / 26.5, 29.1 / 30.9.  1 bit, counts, 6.2 M, M = 6 / 8: 8.7 / 7.5, 7.6 / 7.6.
    const bool few = narrow && max_m < 8 && entries > one_round;
    long long blocks = 0;
    for (int i = 0; i < g; ++i) {
      sm_vote_desc& D = a.d[i];
      D = descs[done + i];
      if (rows) {
        // a flat matrix among padded ones has rows of whole words: rows without padding
        if (!D.sld) D.sld = D.ld = D.cols;
        if (D.cols < 1 || D.sld % 64 || D.n % D.cols) return sm_fail(ctx, SM_EINVAL, "internal: vote rows");
        D.n = D.n / D.cols * D.sld;  // entries of the source
        D.by_row = sm_div_by((unsigned)(fmt == SM_SIGN_1BIT && !narrow ? D.sld / 32 : D.sld / 4));
      }
      a.begin.v[i] = (int)blocks;
      const long long per_wg = narrow ? 4 * TPB * (few ? 4 : 1) : fmt == SM_SIGN_1BIT ? 32 * TPB : 16 * TPB;
      blocks += (D.n + per_wg - 1) / per_wg;
    }
    if (blocks > 0x7FFFFFFFLL) return sm_fail(ctx, SM_EUNSUPPORTED, "vote: too many entries for one launch");
    if (blocks > 0) {
      sm_launch_scope sc(ctx, SM_K_VOTE);
      const dim3 grid((unsigned)blocks), block(TPB);
#define VOTE_WIDE(PLANES)                                                                                     \
  if (rows) hipLaunchKernelGGL((sm_vote_wide_kernel<PLANES, true>), grid, block, 0, ctx->stream, a);          \
  else hipLaunchKernelGGL((sm_vote_wide_kernel<PLANES, false>), grid, block, 0, ctx->stream, a)
#define VOTE_NARROW(FMT, GROUPS)                                                                               \
  if (rows) hipLaunchKernelGGL((sm_vote_narrow_kernel<FMT, true, GROUPS>), grid, block, 0, ctx->stream, a);   \
  else hipLaunchKernelGGL((sm_vote_narrow_kernel<FMT, false, GROUPS>), grid, block, 0, ctx->stream, a)
      if (narrow && fmt == SM_SIGN_1BIT) {
        if (few) { VOTE_NARROW(SM_SIGN_1BIT, 4); }
        else { VOTE_NARROW(SM_SIGN_1BIT, 1); }
      } else if (narrow) {
        if (few) { VOTE_NARROW(SM_SIGN_INT8, 4); }
        else { VOTE_NARROW(SM_SIGN_INT8, 1); }
      } else if (fmt == SM_SIGN_1BIT) {
        if (max_m < 8) { VOTE_WIDE(3); }
        else if (max_m < 32) { VOTE_WIDE(5); }
        else if (max_m < 256) { VOTE_WIDE(8); }
        else { VOTE_WIDE(31); }
      } else if (wide8) {
        hipLaunchKernelGGL(sm_vote_int8_wide_kernel, grid, block, 0, ctx->stream, a);
      } else if (rows) {
        hipLaunchKernelGGL((sm_vote_int8_kernel<true>), grid, block, 0, ctx->stream, a);
      } else {
        hipLaunchKernelGGL((sm_vote_int8_kernel<false>), grid, block, 0, ctx->stream, a);
      }
#undef VOTE_WIDE
#undef VOTE_NARROW
    }
    SM_HIP(ctx, hipGetLastError());
    done += g;
  }
  return SM_OK;
}

int sm_launch_update_group(signmuon_ctx* ctx, const sm_upd_desc* descs, int n) {
  int done = 0;
  while (done < n) {
    const int g = std::min(n - done, SM_UPD_MAX_GROUP);
    upd_args a;
    sm_starts_clear(a.begin);
    a.n = g;
    a.pad_ = 0;
    long long blocks = 0;
    for (int i = 0; i < g; ++i) {
      a.d[i] = descs[done + i];
      a.begin.v[i] = (int)blocks;
      const int q = (a.d[i].cols + 3) / 4;
      a.d[i].quads = sm_div_by((unsigned)q);
      blocks += ((long long)a.d[i].rows * q + UPD_CHUNK - 1) / UPD_CHUNK;
    }
    if (blocks > 0) {
      sm_launch_scope sc(ctx, SM_K_UPDATE);
      hipLaunchKernelGGL(sm_update_kernel, dim3((unsigned)blocks), dim3(TPB), 0, ctx->stream, a);
    }
    SM_HIP(ctx, hipGetLastError());
    done += g;
  }
  return SM_OK;
}

