// Internal declarations shared by the HIP sources of libsignmuon (gfx950 only).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <string>
#include <vector>

#include "../../include/signmuon.h"

typedef __bf16 bf16_t;
typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) unsigned u32x4;
typedef __attribute__((ext_vector_type(2))) unsigned u32x2;
typedef __attribute__((ext_vector_type(4))) int i32x4;

// ---------------------------------------------------------------- context
struct sm_event_pair {
  hipEvent_t a, b;
};

struct signmuon_ctx {
  hipStream_t stream = nullptr;
  int device = 0;
  std::string last_error;

  // Workspaces: one growable device arena each, sub-allocated by a cached Newton-Schulz plan
  // (shape classes + offsets).  Slot SM_WS_STEP serves signmuon_step, SM_WS_NS signmuon_polar_ns,
  // so that calls of the two interleave without replanning.  `arena` is the arena of the slot
  // in use by the running call.
  struct workspace {
    void* arena = nullptr;
    size_t bytes = 0;
    struct ns_plan* plan = nullptr;
  } ws[2];
  void* arena = nullptr;
  // small scratch of the standalone entry points (partial sums of signmuon_momentum)
  void* aux = nullptr;
  size_t aux_bytes = 0;

  // device address of the library's static scratch array on this context's device
  // (signmuon_momentum_noalloc); fixed size SM_STATIC_SCRATCH_BYTES
  void* static_scratch = nullptr;

  // tuning switches (signmuon_set_option)
  int opt[SM_OPT_COUNT] = {};
  int n_cu = 256;  // compute units of the device
  int gemm_flip = 0;  // parity of the GEMM launches so far: every other launch walks its tile ranges backwards

  // timing taps
  unsigned profiling = 0;  // bit k set: launches of kernel class k are bracketed with events
  std::vector<sm_event_pair> ev_pool;        // every pair ever created
  size_t ev_used = 0;                        // pairs handed out since the last reset
  std::vector<std::pair<int, size_t>> ev_log;  // (kernel class, pool index)
  double work_flop[SM_K_COUNT] = {};         // flops of the output tiles that timed GEMM launches compute (logical sizes)
  double work_dense[SM_K_COUNT] = {};        // 2 M N K of the same products as written
  double work_bytes[SM_K_COUNT] = {};        // their operand + result bytes
};

int sm_fail(signmuon_ctx* ctx, int code, const std::string& msg);
int sm_hip_fail(signmuon_ctx* ctx, hipError_t e, const char* what);

#define SM_HIP(ctx, call)                                        \
  do {                                                           \
    hipError_t e__ = (call);                                     \
    if (e__ != hipSuccess) return sm_hip_fail(ctx, e__, #call);  \
  } while (0)

// Scoped launch bracket: records an event pair around a launch when profiling.
struct sm_launch_scope {
  signmuon_ctx* ctx;
  int klass;
  long idx = -1;
  sm_launch_scope(signmuon_ctx* c, int k);
  ~sm_launch_scope();
};

constexpr size_t SM_STATIC_SCRATCH_BYTES = SM_NOALLOC_SCRATCH_BYTES;
constexpr int SM_WS_STEP = 0, SM_WS_NS = 1;
// Ensures the arena of workspace `slot` holds at least `bytes` and makes it the current arena;
// contents (and the slot's plan) are lost when it grows.
int sm_arena_reserve(signmuon_ctx* ctx, int slot, size_t bytes);
// Ensures the auxiliary scratch holds at least `bytes`.
int sm_aux_reserve(signmuon_ctx* ctx, size_t bytes);

static inline int64_t sm_round_up(int64_t x, int64_t m) { return (x + m - 1) / m * m; }
static inline bool sm_aligned(const void* p, size_t a) { return (reinterpret_cast<uintptr_t>(p) % a) == 0; }

// ---------------------------------------------------------------- descriptor tables
// Grouped launches carry their table in the kernel arguments, which lie in host memory: every cache line of it
// that a compute unit reads costs about a microsecond, one after the other where an address depends on what the
// line before it held.  A workgroup finds its entry from the entries' first workgroups, which therefore stand side
// by side (unused ones INT_MAX) and are compared sixteen at a time; walking the descriptors themselves took 6.8 us
// per launch of 24 entries against 3.2 us.
template <int N>
struct sm_starts {
  static_assert(N % 16 == 0, "compared sixteen at a time");
  int v[N];
};
template <int N>
static inline void sm_starts_clear(sm_starts<N>& s) {
  for (int i = 0; i < N; ++i) s.v[i] = 0x7FFFFFFF;
}
// Largest i with v[i] <= bx, among the first n entries (v[0] <= bx).
template <int N>
__device__ __forceinline__ int sm_find(const sm_starts<N>& s, int n, int bx) {
  if (n == 1) return 0;
  int at = 0;
  for (int i = 0; i < n; i += 16) {
#pragma unroll
    for (int k = 0; k < 16; ++k) at = (bx >= s.v[i + k]) ? i + k : at;
  }
  return at;
}

// The same, and the workgroup's number within the entry.  A table of one entry needs no line of starts; where it often
// is one, the descriptors stand before the starts, so that the first lies next to n (copies and PowerIter alone on one
// 256 x 1024 matrix: 1.10 of the time with starts inside the descriptors where the starts were first and read, 1.04 so).
template <int N>
__device__ __forceinline__ int sm_entry(const sm_starts<N>& s, int n, int bx, int& local) {
  local = bx;
  if (n == 1) return 0;
  const int i = sm_find(s, n, bx);
  local -= s.v[i];
  return i;
}

// ---------------------------------------------------------------- unaligned vectors, division
// Vectors of which only the elements are aligned: a row of odd length starts anywhere, and global memory takes
// 8- and 16-byte accesses at any address of this part.
typedef f32x4 f32x4_u __attribute__((aligned(4)));
typedef u32x4 u32x4_u __attribute__((aligned(1)));
typedef u32x2 u32x2_u __attribute__((aligned(1)));
typedef unsigned u32_u __attribute__((aligned(1)));
typedef bf16x4 bf16x4_u __attribute__((aligned(2)));
typedef i32x4 i32x4_u __attribute__((aligned(4)));

// Division of 0 <= n < 2^31 by a divisor the host knows: multiply and shift (64-bit division is a call of some
// hundred instructions, which is what bounded the copies of rows of odd length).
struct sm_div {
  unsigned mul, shift;
};
static inline sm_div sm_div_by(unsigned d) {
  unsigned s = 0;
  while ((1ull << s) < d) ++s;
  return sm_div{(unsigned)(((1ull << (31 + s)) + d - 1) / d), 31 + s};
}
__device__ __forceinline__ unsigned sm_quot(const sm_div& v, unsigned n) {
  return (unsigned)(((unsigned long long)n * v.mul) >> v.shift);
}
// Row and column of entry `at` (any size) of rows of d entries (v = sm_div_by(d)).
__device__ __forceinline__ void sm_row_of(const sm_div& v, int d, long long at, long long& row, int& col) {
  if (at < 0x7FFFFFFFLL) {
    const unsigned q = sm_quot(v, (unsigned)at);
    row = q;
    col = (int)((unsigned)at - q * (unsigned)d);
  } else {
    row = at / d;
    col = (int)(at - row * d);
  }
}

// ---------------------------------------------------------------- streaming kernels (stream.hip)
// Descriptor of one weight block for the grouped momentum launch.
struct sm_mom_desc {
  float* mom;          // [M][d]
  const float* grad;   // [M][d]
  const float* w;      // [d] or null
  bf16_t* x;           // [M] bf16 copies, flat or with padded rows, or null
  float* partial;      // [M][chunks] per-chunk sums of squares, or null
  long long d;         // rows*cols
  long long x_stride;  // elements between workers in x
  int cols;            // row length
  int chunks;          // chunks per worker (sm_mom_chunks)
  sm_div quads;        // by the number of 4-entry groups per row where the rows of x are padded to whole 64 entries;
                       // shift 0: x is as flat as mom
};
// Chunks of SM_MOM_CHUNK entries per worker.  A matrix that goes into padded rows (ld != cols) is cut into groups
// of four entries row by row, so that a group never straddles rows; otherwise it is one flat run.
static inline long long sm_mom_chunks(long long rows, long long cols, long long ld) {
  const long long n = (ld == cols) ? rows * cols : rows * ((cols + 3) / 4 * 4);
  return (n + 1024 - 1) / 1024;
}
constexpr int SM_MOM_MAX_GROUP = 48;  // blocks per launch: the table rides in the kernel arguments (4 KB at most)
constexpr int SM_MOM_CHUNK = 1024;  // elements per workgroup: one 16-byte piece per thread (short-lived workgroups
                                    // keep the four streams of the momentum update close together in memory)

int sm_launch_momentum(signmuon_ctx* ctx, const sm_mom_desc* descs, int n, int M, float beta, float wd);
// sumsq[i] = sum_j partial[i*chunks + j], i < count (fixed order)
int sm_launch_reduce_partials(signmuon_ctx* ctx, const float* partial, int chunks, int count, float* sumsq);
// Inverse scales over a table of matrix classes, one launch: per class `count` items with
//   mode 0: sig (if not null) = sum of the item's `chunks` partial sums of squares, inv = 1 / max(sqrt(sig), eps)
//   mode 1: inv = 1 / max(sig, eps)
struct sm_sigma_desc {
  const float* partial;
  float* sig;
  float* inv;
  int chunks, count, mode;
};
constexpr int SM_SIGMA_MAX_GROUP = 64;
int sm_launch_sigma_group(signmuon_ctx* ctx, const sm_sigma_desc* descs, int n, float eps);

// Grouped sign pack: one launch over a table of matrices, `M` workers each.
struct sm_sp_desc {
  const void* u;            // [M][rows][ld]
  void* out;                // M rows of out_stride bytes
  long long n;              // rows * cols
  long long batch_stride;   // elements between workers in u
  long long out_stride;     // bytes
  int cols, ld;             // ld == cols: u is flat
  sm_div by_cols;           // filled by the launcher
  int blocks_per_row;       // filled by the launcher
  int pad_;
};
constexpr int SM_SP_MAX_GROUP = 48;
int sm_launch_sign_pack_group(signmuon_ctx* ctx, const sm_sp_desc* descs, int n, int dtype, int fmt, int M);

// Grouped vote with expanded outputs (+ fused update): one launch over a table of matrices.  The signs of a worker
// are rows of `sld` entries of which `cols` count, sld a multiple of 64, or (sld == 0) one run of n entries.
struct sm_vote_desc {
  const void* signs;
  long long n, stride_bytes;  // n: rows * cols
  void* voted;       // non-bit formats only (SM_VOTE_INT8/BF16/F32), or null
  int32_t* counts;   // flat, or null
  float* w;          // flat, or null
  float lr;
  int M, vfmt;
  int cols, sld;
  int ld;            // row length of voted: sld (then the columns beyond cols are written as zeros; bf16 only) or cols
  sm_div by_row;     // by the words (sm_vote_wide_kernel) or groups of four (the others) of a row of sld; filled by the launcher
};
constexpr int SM_VOTE_MAX_GROUP = 48;
int sm_launch_vote_group(signmuon_ctx* ctx, const sm_vote_desc* descs, int n, int fmt);

// Grouped update after a local polar step: w[r][c] -= step * d[r][ld]
struct sm_upd_desc {
  float* w;
  const bf16_t* d;
  const float* kappa;  // optional device scalar multiplied into step
  int rows, cols, ld;
  float step;
  sm_div quads;        // by the 4-entry groups of a row; filled by the launcher
};
constexpr int SM_UPD_MAX_GROUP = 64;
int sm_launch_update_group(signmuon_ctx* ctx, const sm_upd_desc* descs, int n);

// sign pack of a flat source: u[batch][n] -> rows of bits or int8
int sm_launch_sign_pack(signmuon_ctx* ctx, const void* u, int dtype, int batch, long long n, int fmt, void* out,
                        long long out_stride_bytes);

struct sm_vote_args {
  const void* signs;
  int fmt, M;
  long long n, stride_bytes;
  void* voted;
  int vfmt;          // SM_VOTE_*
  int32_t* counts;
  float* w;
  float lr_scaled;
};
int sm_launch_vote(signmuon_ctx* ctx, const sm_vote_args& a);

// ---------------------------------------------------------------- layout helpers (layout.hip)
// dst[b][rows_p][ld] (bf16, padding not touched) <- src[b][rows][cols] (f32 or bf16); with partial also the sums of
// squares of the source per chunk, partial[b * sm_mom_chunks(rows, cols, ld) + chunk]
int sm_launch_copy_in(signmuon_ctx* ctx, const void* src, int dtype, int batch, int rows, int cols,
                      bf16_t* dst, int ld, long long dst_stride, float* partial);
// dst[b][rows][cols] (f32 or bf16) <- scale[b] * src[b][rows][ld]; scale may be null
int sm_launch_copy_out(signmuon_ctx* ctx, const bf16_t* src, int ld, long long src_stride, int batch, int rows,
                       int cols, void* dst, int dtype, const float* scale);

// ---------------------------------------------------------------- GEMM (ns_gemm.hip)
// C[b] = rnd(rnd(alpha * scale[b]^scale_pow * (A' * B'^T) + diag * I) + gamma * R[b]),
//        A' = opA[b] + a_diag I,  B' = opB[b] + b_diag I
// opA is M x K, opB is N x K, C and R are [M][ldc]; M, N, K multiples of 64; fp32 accumulation.
// With a symmetric output R must be symmetric too.  The identity shifts need half-precision
// K-contiguous operands.
// Matrices hold 16-bit elements: bf16, or IEEE half where in_f16 (A, B) / out_f16 (C) say
// so (r_f16 for R); the pointer type is bf16_t either way.
struct sm_gemm_prob {
  const bf16_t* A;
  const bf16_t* B;
  bf16_t* C;
  const bf16_t* R;       // or null
  float* scale;          // [batch], see sm_gemm_args::scale_mode
  long long sA, sB, sC;  // batch strides in elements (C and R share sC)
  int M, N, K;
  int lda, ldb, ldc;
  int batch;
  int tiles_m, tiles_n;  // filled by the launcher, like the next
  sm_div by_item;        // by the tiles of a batch item (the mate's among them)
  int layout;            // bit 0: A stored [K][M] (lda = its row length), bit 1: B stored [K][N]
  // Optional sign output of a general (non-symmetric) bf16 product: the signs (x >= 0) of the
  // leading sign_rows x sign_ld part of C[b], packed row by row (sign_ld a multiple of 64) into
  // sign_out + b * sign_stride as in signmuon_sign_pack.  C may then be null.
  // (A Gram launch with SM_SCALE_PARTIAL has its [batch][sign_rows] partial sums of squares here: one place for both, as
  // a table of 24 problems just fits the kernel arguments.)
  void* sign_out;
  long long sign_stride;
  int sign_rows, sign_ld;
  int sign_fmt;
  // Index (> own index) of a second problem of equal M, N, K and batch whose tiles are dealt item by
  // item right after this problem's (item b of this one, item b of the mate, item b + 1, ...), so
  // that operands the two share are read from HBM once; 0 = none.  The mate owns no tiles itself.
  int mate;
  // logical (unpadded) M, N, K, for the work accounting of the timing taps; 0 = as M, N, K.  A general product also
  // writes zeros to the entries of C beyond mu x nu, whatever the product has there (0 * NaN where an operand is not
  // finite): the padding of the working layout reads as zero for every later call.
  int mu, nu, ku;
  float scale_value;  // SM_SCALE_VALUE
};
// Inverse scale of a GEMM's item, taken by the kernel itself: a launch for it costs as much as a product of small matrices.
constexpr int SM_SCALE_INV = 0;      // scale[b]
constexpr int SM_SCALE_SIG = 1;      // 1 / max(scale[b], eps)
constexpr int SM_SCALE_VALUE = 2;    // scale_value, the same for every item
constexpr int SM_SCALE_PARTIAL = 3;  // Gram matrices: 1 / max(sqrt(sum of the item's partial sums), eps), also written to scale[b]
constexpr int SM_GEMM_MAX_PROB = 24;
constexpr int SM_GEMM_STARTS = 32;
struct sm_gemm_args {
  int n_prob;
  int per_xcd_wgs;   // workgroups per XCD; filled by the launcher, like the next two
  int reverse;       // an XCD walks its range of the tile list from the end (every other launch)
  int total_tiles;
  int scale_pow;     // 0, 1 or 2
  int scale_mode;    // SM_SCALE_*: what scale[b] of the formula is
  float eps;
  int direct;        // a general product writes to a caller's matrices of mu x nu (ldc = nu a multiple of 8): 1 bf16, 2 float32
  float alpha, gamma, diag;
  float a_diag, b_diag;  // 0 = none
  int in_f16, out_f16, r_f16;
  int sym_store;     // bit 0: the operands hold valid data only in their 256 x 256 blocks on and above the diagonal
                     // (symmetric matrices; half precision, M == N == K); bit 1: write the output that way; bit 2:
                     // write the output as packed 32 x 32 blocks on and above the diagonal (ns_chain.hip)
  int xcd_begin[9];  // XCD x owns tiles [xcd_begin[x], xcd_begin[x + 1]) of the tile list
  sm_starts<SM_GEMM_STARTS> tile_begin;  // first tile of every problem; filled by the launcher
  sm_gemm_prob p[SM_GEMM_MAX_PROB];
};
static_assert(sizeof(sm_gemm_args) <= 4096, "kernel arguments are limited to 4 KB");
// Output tiles of a launch at tile sizes 64, 128 and 256 and its longest K; the tile size and LDS stages it gets.
struct sm_tile_count {
  double tiles[3] = {0, 0, 0};
  int longest = 0;
  void add(int M, int N, int K, int batch, bool sym);
};
int sm_gemm_tile(const signmuon_ctx* ctx, const sm_tile_count& c);
int sm_gemm_stages(const signmuon_ctx* ctx, const sm_tile_count& c);
// One grouped launch over the problem table.  sym: every problem's output is symmetric (M == N;
// layout 0 or 3): only the upper triangle of tiles is computed and stored mirrored.  Otherwise
// layout 0 or 2.  Half-precision operands need sym and layout 0.  klass is the profiling class
// the launch is booked under.
int sm_launch_gemm(signmuon_ctx* ctx, sm_gemm_args& args, bool sym, int klass);

// ---------------------------------------------------------------- chain of s x s products (ns_chain.hip)
// From A_0 (half precision, packed 32 x 32 blocks) to P_K (bf16, whole row-major matrix), one workgroup per matrix.
// Two matrices are in LDS (0: A_0 at first, and 1) and two in registers (A: A_0 at first, and P).  An op does, in order:
// pre (bits: 1 LDS 0 <- A, 2 LDS 0 <- P, 4 LDS 1 <- P); c = alpha X Y + ca A + cp P + cl (LDS 1) + diag I with X, Y the
// LDS matrices x, y; LDS put <- c (put >= 0); keep (bits: 1 A <- c, 2 P <- c).  The last op's c is the result.
constexpr int SM_CHAIN_MAX_S = 256;
struct chain_class {
  const unsigned char* in;  // of the class's first matrix; s * s 16-bit elements per matrix
  unsigned char* out;
  int s, su;                // padded and logical side (the latter for the work accounting alone)
};
struct chain_op {
  int x, y, pre, put, keep;
  float alpha, ca, cp, cl, diag;
};
constexpr int SM_CHAIN_MAX_CLASSES = 64, SM_CHAIN_MAX_OPS = 10;
struct chain_args {
  sm_starts<SM_CHAIN_MAX_CLASSES> begin;  // first workgroup of every class
  int n, n_ops;
  chain_op op[SM_CHAIN_MAX_OPS];
  chain_class c[SM_CHAIN_MAX_CLASSES];
};
static_assert(sizeof(chain_args) <= 4096, "kernel arguments are limited to 4 KB");
int sm_launch_chain(signmuon_ctx* ctx, chain_args& a, int blocks);

// ---------------------------------------------------------------- power iteration (poweriter.hip)
// sigma[item] = PowerIter(X[item], P, eps, v0[item]) for the `items` matrices of each table entry.
struct sm_pi_desc {
  const bf16_t* x;      // [items][rows][ld], zero beyond cols in every row
  long long stride;     // elements between matrices
  const float* v0;      // [items] start vectors of cols floats, v0_stride floats apart
  long long v0_stride;
  float* u;             // scratch [items][up]
  float* v;             // scratch [items][ld]
  float* part;          // scratch [items][chunks][ld]
  float* sigma;         // [items]
  int rows, cols, ld;   // ld a multiple of 64
  int up;               // rows rounded up to a multiple of 8
  int items;
  int chunks;           // ceil(rows / SM_PI_ROW_CHUNK)
};
constexpr int SM_PI_MAX_GROUP = 40;
constexpr int SM_PI_ROW_CHUNK = 128;
constexpr int SM_PI_FUSED_ROWS = 64;       // rows per workgroup of the fused pass
constexpr int SM_PI_FUSED_MAX_LD = 4096;   // widest matrix (padded columns) the fused pass holds in registers
int sm_launch_power_iter_group(signmuon_ctx* ctx, const sm_pi_desc* descs, int n, int P, float eps);
