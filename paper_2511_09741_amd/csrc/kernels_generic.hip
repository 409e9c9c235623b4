// Shape-generic kernels: fp32 arithmetic on fp32 or bf16 storage, any dimensions.  They carry the
// fp32 configuration (head_dim 16, widths that fit no bf16 MFMA tile) and every bf16 shape the MFMA
// kernels do not take.  The layers they serve are small: what bounds them is the latency of a launch
// and of the loads behind it, so a launch does as much as it can and has all of its loads in flight early.
#include <type_traits>

#include "dev_common.h"
#include "taw_internal.h"

namespace taw {

// =============================================================================== GEMM
// C[m,n] (=|+=) sum_k A(m,k) B(k,n) (+ R[m,n]) on the fp32 matrix instruction (16x16x4, IEEE fp32 products and sums), operands
// straight from memory into registers: of 16 consecutive k, lane group g = lane >> 4 loads k = 4g .. 4g + 3 (one load of four
// values, at any alignment, where the operand is contiguous along k) and matrix instruction i multiplies the four k = 4g + i, the same for both operands.
//   SPLIT: a workgroup owns 16 x 16 outputs, its four wavefronts a quarter of K each, summed through LDS in wavefront order: every
//     load of a short contraction is in flight at once, and a 128 x 64 result has 32 workgroups.
//   otherwise: a workgroup owns 64 x 64, each wavefront 32 x 32 over all of K: more products per load, for results that fill the chip; an
//     operand contiguous along the result is loaded two columns at a time (1024 x 4096 x 1024 TN in bf16: 200 -> 133 us; one 2-byte load per value
//     was slower there than the staged tiles below).
// (32 x 32 tiles staged through LDS 16 k at a time, one exposed load latency per 16 k, took 6 - 30 us for the products of a
// 64-wide layer with 128 tokens; these take 2 - 5.)
namespace gen {

struct Args {
  int64_t M, N, K;
  const void* A;
  int64_t lda;
  const void* B;
  int64_t ldb;
  void* C;
  int64_t ldc;
  int accumulate;
  const void* R;
  int64_t ldr;
  int tiles_n, blocks;        // tiles along n, workgroups in all
  const float* table;         // kRope: [S][d/2][2] (cos, sin); columns below rot_cols are rotated, row r at position r % S
  int S, d;
  int64_t rot_cols;
  const void* gu;             // kSwigluBwd: [M][2N] gate | up
  void* C2;                   // kSwigluFwd: silu(gate) up, [M][N]; C is [M][2N] gate | up and B has 2N rows
};
enum { kPlain = 0, kRope = 1, kSwigluFwd = 2, kSwigluBwd = 3 };

// N consecutive values from an address aligned to one of them only: as wide a load as the device takes there
template <typename T, int N> struct Run { T v[N]; };
template <int N, typename T> __device__ __forceinline__ Run<T, N> load_run(const T* p) {
  Run<T, N> r;
  __builtin_memcpy(&r, p, sizeof(r));
  return r;
}

// the four values k .. k + 3 of one row (KC) or column of an operand; those at or beyond K are 0 and not read
template <typename T, bool KC>
__device__ __forceinline__ f32x4_t operand4(const T* mat, int64_t ld, int64_t idx, int64_t k, int64_t K) {
  f32x4_t v;
  if (KC && k + 4 <= K) {
    const Run<T, 4> r = load_run<4>(mat + idx * ld + k);
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = (float)r.v[i];
  } else {
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = k + i < K ? (float)(KC ? mat[idx * ld + k + i] : mat[(k + i) * ld + idx]) : 0.f;
  }
  return v;
}
// the same of the two columns idx, idx + 1 of an operand contiguous along them, of which the last two, `last` and last + 1, are read where idx
// lies beyond them (idx = last + 1, the last column alone, then comes first)
template <typename T>
__device__ __forceinline__ void operand4x2(f32x4_t& v0, f32x4_t& v1, const T* mat, int64_t ld, int64_t idx, int64_t last, int64_t k, int64_t K) {
  const bool beyond = idx > last;
  const T* p = mat + (beyond ? last : idx);
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    Run<T, 2> r{{(T)0.f, (T)0.f}};
    if (k + i < K) r = load_run<2>(p + (k + i) * ld);
    v0[i] = (float)(beyond ? r.v[1] : r.v[0]);
    v1[i] = (float)r.v[1];
  }
}

// one output (and, kSwigluFwd, its partner of the up half) leaves; lanes l, l ^ 1 hold columns 2j, 2j + 1 of one row
template <typename TC, int EPI>
__device__ __forceinline__ void finish(const Args& g, int64_t row, int64_t col, float v, float v2) {
  if constexpr (EPI == kRope) {
    const float w = __shfl_xor(v, 1, 64);
    if (col < g.rot_cols && row < g.M) {
      // 32-bit remainders (token counts and widths fit): 64-bit ones, once per output of a 64 x 64 tile, were 33 KB of code
      const float* tb = g.table + (int64_t)((unsigned)row % (unsigned)g.S) * g.d + ((unsigned)col % (unsigned)g.d) / 2 * 2;
      v = col & 1 ? w * tb[1] + v * tb[0] : v * tb[0] - w * tb[1];
    }
  }
  if (row >= g.M || col >= g.N) return;
  TC* C = static_cast<TC*>(g.C);
  if constexpr (EPI == kSwigluFwd) {
    TC* c = C + row * g.ldc + col;
    c[0] = (TC)v;
    c[g.N] = (TC)v2;
    v = (float)(TC)v;          // the backward sees the stored gate and up: so does this product
    v2 = (float)(TC)v2;
    static_cast<TC*>(g.C2)[row * g.N + col] = (TC)(v / (1.0f + __expf(-v)) * v2);
    return;
  }
  if constexpr (EPI == kSwigluBwd) {
    v = (float)(TC)v;          // the gradient of a, in its storage type
    const TC* gu = static_cast<const TC*>(g.gu) + row * 2 * g.N + col;
    const float gg = (float)gu[0], uu = (float)gu[g.N], sig = 1.0f / (1.0f + __expf(-gg));
    TC* c = C + row * g.ldc + col;
    c[0] = (TC)(v * uu * sig * (1.0f + gg * (1.0f - sig)));
    c[g.N] = (TC)(v * gg * sig);
    return;
  }
  if (g.R) v += (float)static_cast<const TC*>(g.R)[row * g.ldr + col];
  TC* c = C + row * g.ldc + col;
  if (g.accumulate) v += (float)*c;
  *c = (TC)v;
}

// FORM: kSplit, or the number of chains of a 64 x 64 tile
constexpr int kSplit = 0;
template <typename TI, typename TC, int MODE, int FORM, int EPI>
__device__ __forceinline__ void body(const Args& g, int block, float* red) {
  constexpr bool SPLIT = FORM == kSplit;
  constexpr bool A_KC = MODE != GEMM_TN, B_KC = MODE == GEMM_NT;
  constexpr int R = SPLIT ? 1 : 2, NB = EPI == kSwigluFwd ? 2 : 1;        // R x R matrix tiles per wavefront; NB: B panels
  constexpr int U = SPLIT ? 4 : 2;                                        // groups of 16 k whose loads are in flight together
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, l16 = lane & 15, g4 = 4 * (lane >> 4);
  const int tm = block / g.tiles_n, tn = block - tm * g.tiles_n;
  const int64_t m0 = (int64_t)tm * (SPLIT ? 16 : 64) + (SPLIT ? 0 : 32 * (wave >> 1));
  const int64_t n0 = (int64_t)tn * (SPLIT ? 16 : 64) + (SPLIT ? 0 : 32 * (wave & 1));
  int64_t k0 = 0, k1 = g.K;
  if (SPLIT) {
    const int64_t part = (g.K + 63) / 64 * 16;
    k0 = wave * part;
    k1 = k0 + part < g.K ? k0 + part : g.K;
  }
  const TI* A = static_cast<const TI*>(g.A);
  const TI* B = static_cast<const TI*>(g.B);
  // Rows and columns of the result this lane loads the operands of: those outside it read its last one.  Of the 32 rows (columns) of a
  // wavefront, matrix tile i has 16 i .. 16 i + 15 where they are loaded along k, and every second one where the operand is contiguous along
  // them: then one load of two adjacent values serves both tiles.
  constexpr bool A_PAIR = !SPLIT && !A_KC, B_PAIR = !SPLIT && !B_KC;
  int64_t ar[R], bc[R];
#pragma unroll
  for (int i = 0; i < R; ++i) {
    ar[i] = m0 + 16 * i + l16 < g.M ? m0 + 16 * i + l16 : g.M - 1;
    bc[i] = n0 + 16 * i + l16 < g.N ? n0 + 16 * i + l16 : g.N - 1;
  }
  // NA accumulators per output, matrix instruction e of a group adding to accumulator e % NA
  constexpr int NA = SPLIT ? 1 : FORM;
  static_assert(NA == 1 || NA == 4, "one accumulator, or one per matrix instruction of a group");
  f32x4_t acc[NA][NB][R][R];
#pragma unroll
  for (int n = 0; n < NA; ++n)
#pragma unroll
    for (int q = 0; q < NB; ++q)
#pragma unroll
      for (int i = 0; i < R; ++i)
#pragma unroll
        for (int j = 0; j < R; ++j) acc[n][q][i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  for (int64_t k = k0; k < k1; k += 16 * U) {
    f32x4_t a[U][R], b[U][NB][R];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int64_t kk = k + 16 * u + g4;
      if constexpr (A_PAIR) operand4x2<TI>(a[u][0], a[u][1], A, g.lda, m0 + 2 * l16, g.M - 2, kk, k1);
      if constexpr (B_PAIR) operand4x2<TI>(b[u][0][0], b[u][0][1], B, g.ldb, n0 + 2 * l16, g.N - 2, kk, k1);
#pragma unroll
      for (int i = 0; i < R; ++i) {
        if constexpr (!A_PAIR) a[u][i] = operand4<TI, A_KC>(A, g.lda, ar[i], kk, k1);
        if constexpr (!B_PAIR) {
#pragma unroll
          for (int q = 0; q < NB; ++q) b[u][q][i] = operand4<TI, B_KC>(B, g.ldb, bc[i] + q * g.N, kk, k1);
        }
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int q = 0; q < NB; ++q)
#pragma unroll
          for (int i = 0; i < R; ++i)
#pragma unroll
            for (int j = 0; j < R; ++j) acc[e % NA][q][i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[u][i][e], b[u][q][j][e], acc[e % NA][q][i][j], 0, 0, 0);
  }
  // accumulator register r of lane l: row 4 (l >> 4) + r, column l & 15
  if constexpr (SPLIT) {
#pragma unroll
    for (int q = 0; q < NB; ++q)
#pragma unroll
      for (int r = 0; r < 4; ++r) red[((q * 4 + wave) * 16 + g4 + r) * 16 + l16] = acc[0][q][0][0][r];
    __syncthreads();
    float v[2] = {0.f, 0.f};
#pragma unroll
    for (int q = 0; q < NB; ++q)
#pragma unroll
      for (int w = 0; w < 4; ++w) v[q] += red[(q * 4 + w) * 256 + threadIdx.x];
    finish<TC, EPI>(g, m0 + (threadIdx.x >> 4), n0 + l16, v[0], v[1]);
  } else {
#pragma unroll
    for (int i = 0; i < R; ++i)
#pragma unroll
      for (int j = 0; j < R; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          auto sum = [&](int q) {
            float v = acc[0][q][i][j][r];
            if constexpr (NA == 4) v = (v + acc[1][q][i][j][r]) + (acc[2][q][i][j][r] + acc[3][q][i][j][r]);
            return v;
          };
          finish<TC, EPI>(g, m0 + (A_PAIR ? 2 * (g4 + r) + i : 16 * i + g4 + r), n0 + (B_PAIR ? 2 * l16 + j : 16 * j + l16), sum(0), sum(NB - 1));
        }
  }
}

template <typename TI, typename TC, int MODE, int FORM, int EPI>
__global__ void __launch_bounds__(256) gemm_kernel(Args g) {
  __shared__ float red[FORM == kSplit ? (EPI == kSwigluFwd ? 2 : 1) * 1024 : 1];
  body<TI, TC, MODE, FORM, EPI>(g, (int)blockIdx.x, red);
}
// weight gradient (TN, fp32) and input gradient (NN) of a linear in one grid
template <typename T, int EPI>
__global__ void __launch_bounds__(256) gemm_dual_kernel(Args g0, Args g1) {
  __shared__ float red[1024];
  if ((int)blockIdx.x < g0.blocks) body<T, float, GEMM_TN, kSplit, kPlain>(g0, (int)blockIdx.x, red);
  else body<T, T, GEMM_NN, kSplit, EPI>(g1, (int)blockIdx.x - g0.blocks, red);
}

constexpr int64_t kSplitTiles = 4096;      // the paired backward splits up to this many 16 x 16 tiles of either product, and results of no more sum in four chains

// Splitting pays while its workgroups, one per 16 x 16 tile, are few: us split / 64 x 64 (fp32, NT): 400 x 750 x 250 (1175 tiles) 6.5 / 10.7, 1024 x 512 x 512
// (2048) 17 / 18, 1024 x 1024 x 256 (4096) 18 / 12; with a short contraction a workgroup is mostly overhead: 4096 x 64 x 64 (1024) 4.6 / 5.6,
// 4096 x 176 x 64 (2816) 8.4 / 6.2.  A tile of 64 x 64 loads pairs of rows or columns, of which a single one has none.
inline int64_t small_tiles(const Args& g) { return ((g.M + 15) / 16) * ((g.N + 15) / 16); }
inline bool take_split(const Args& g) { return g.M < 2 || g.N < 2 || small_tiles(g) <= (g.K <= 128 ? 1536 : 2048); }
// The 64 x 64 form adds up all of K.  Up to kSplitTiles it does so in four chains, which round off as little as the four quarters of the split form
// (layer of 3 x 400 tokens, 256 wide, I = 768: weight gradients 4.0e-7 from fp64 in both, 4.9e-7 with one chain); grids beyond are bound by how many
// wavefronts a SIMD holds, and four chains' registers cost them up to half (4096 x 1024 x 1024 NT in bf16 154 us with one chain, 169 with four).
inline bool take_chains(const Args& g) { return small_tiles(g) <= kSplitTiles; }
inline void tile_up(Args& g, bool split) {
  const int t = split ? 16 : 64;
  g.tiles_n = (int)((g.N + t - 1) / t);
  g.blocks = (int)((g.M + t - 1) / t) * g.tiles_n;
}
inline Args make(int64_t M, int64_t N, int64_t K, const void* A, int64_t lda, const void* B, int64_t ldb, void* C, int64_t ldc, int accumulate,
                 const void* R, int64_t ldr) {
  return Args{M, N, K, A, lda, B, ldb, C, ldc, accumulate, R, ldr, 0, 0, nullptr, 1, 2, 0, nullptr, nullptr};
}

template <typename TI, typename TC, int MODE, int EPI>
int launch(Args g, hipStream_t st) {
  const bool split = take_split(g);
  tile_up(g, split);
#define TAW_GEN(FORM) hipLaunchKernelGGL((gemm_kernel<TI, TC, MODE, FORM, EPI>), dim3((unsigned)g.blocks), dim3(256), 0, st, g)
  if (split) TAW_GEN(kSplit); else if (take_chains(g)) TAW_GEN(4); else TAW_GEN(1);
#undef TAW_GEN
  return (int)hipGetLastError();
}
template <typename TI, typename TC>
int launch_mode(int mode, const Args& g, hipStream_t st) {
  if (mode == GEMM_NT) return launch<TI, TC, GEMM_NT, kPlain>(g, st);
  if (mode == GEMM_NN) return launch<TI, TC, GEMM_NN, kPlain>(g, st);
  return launch<TI, TC, GEMM_TN, kPlain>(g, st);
}

}  // namespace gen

int launch_gemm_generic(int dtype, int mode, int64_t M, int64_t N, int64_t K, const void* A, int64_t lda,
                        const void* B, int64_t ldb, void* C, int64_t ldc, int c_dtype, int accumulate,
                        const void* R, int64_t ldr, hipStream_t st) {
  if (M == 0 || N == 0) return 0;
  const gen::Args g = gen::make(M, N, K, A, lda, B, ldb, C, ldc, accumulate, R, ldr);
  if (dtype == DT_F32) return gen::launch_mode<float, float>(mode, g, st);
  return c_dtype == DT_BF16 ? gen::launch_mode<bf16_t, bf16_t>(mode, g, st) : gen::launch_mode<bf16_t, float>(mode, g, st);
}

int launch_gemm_generic_rope(int dtype, int64_t M, int64_t N, int64_t K, const void* A, int64_t lda, const void* B, int64_t ldb, void* C,
                             int64_t ldc, const float* table, int S, int d, int64_t rot_cols, hipStream_t st) {
  gen::Args g = gen::make(M, N, K, A, lda, B, ldb, C, ldc, 0, nullptr, 0);
  g.table = table; g.S = S; g.d = d; g.rot_cols = rot_cols;
  return dtype == DT_F32 ? gen::launch<float, float, GEMM_NT, gen::kRope>(g, st) : gen::launch<bf16_t, bf16_t, GEMM_NT, gen::kRope>(g, st);
}

int launch_gemm_generic_swiglu(int dtype, int64_t T, int64_t I, int64_t K, const void* A, int64_t lda, const void* W, int64_t ldw, void* gu, void* a,
                               hipStream_t st) {
  gen::Args g = gen::make(T, I, K, A, lda, W, ldw, gu, 2 * I, 0, nullptr, 0);
  g.C2 = a;
  return dtype == DT_F32 ? gen::launch<float, float, GEMM_NT, gen::kSwigluFwd>(g, st) : gen::launch<bf16_t, bf16_t, GEMM_NT, gen::kSwigluFwd>(g, st);
}

bool gemm_generic_linear_bwd_supported(int64_t T, int64_t N, int64_t K) {
  const int64_t t = (T + 15) / 16, n = (N + 15) / 16, k = (K + 15) / 16;
  return t * k <= gen::kSplitTiles && n * k <= gen::kSplitTiles;
}
int launch_gemm_generic_linear_bwd(int dtype, int64_t T, int64_t N, int64_t K, const void* dy, const void* W, const void* x, void* dx, float* G,
                                   int accumulate, const void* gu, hipStream_t st) {
  gen::Args g0 = gen::make(N, K, T, dy, N, x, K, G, K, accumulate, nullptr, 0);
  gen::Args g1 = gen::make(T, K, N, dy, N, W, K, dx, gu ? 2 * K : K, 0, nullptr, 0);
  g1.gu = gu;
  gen::tile_up(g0, true);
  gen::tile_up(g1, true);
  const dim3 grid((unsigned)(g0.blocks + g1.blocks));
#define TAW_GEN(T_, EPI) hipLaunchKernelGGL((gen::gemm_dual_kernel<T_, gen::EPI>), grid, dim3(256), 0, st, g0, g1)
#define TAW_GEN_T(T_) do { if (gu) TAW_GEN(T_, kSwigluBwd); else TAW_GEN(T_, kPlain); } while (0)
  if (dtype == DT_F32) TAW_GEN_T(float); else TAW_GEN_T(bf16_t);
#undef TAW_GEN_T
#undef TAW_GEN
  return (int)hipGetLastError();
}

// =============================================================================== attention, narrow heads
// head_dim <= 32: one wavefront per (batch, head, row), a lane per row of the other side (keys of a query, queries of a key), which
// it keeps in registers: DP = head_dim rounded up to 8, 16 or 32 values, loaded in fours at any alignment (head_dim is even), so a wavefront has 64 rows
// in flight and no serial chain over the sequence.  Each lane sums over its own rows; the DP sums then meet by halves: at step b a
// lane keeps the half its bit b names and receives the other lane's, until lane l holds element l % DP.  (A loop over those steps is not
// unrolled, and every access to the row becomes a search through its registers: 33 and 100 KB of code for the two kernels at 32
// values instead of 7 and 14, most of it fetched once per wavefront: 16 sequences of 64 tokens, 8 heads of 24, forward / backward
// 64 / 195 us, with them 15 / 45.)
// FULL: d == DP, no value to leave out and no branch per load (backward at 3 sequences of 1000 tokens, 8 heads of 8 in bf16: 264 us with, 227 without)
template <bool FULL, typename T, int DP>
__device__ __forceinline__ void load_row(float (&v)[DP], const T* p, int d) {
#pragma unroll
  for (int i = 0; i < DP; i += 4) {
    gen::Run<T, 4> r{{(T)0.f, (T)0.f, (T)0.f, (T)0.f}};
    if (FULL || i + 4 <= d) {
      r = gen::load_run<4>(p + i);
    } else if (i < d) {
      const gen::Run<T, 2> h = gen::load_run<2>(p + i);
      r.v[0] = h.v[0];
      r.v[1] = h.v[1];
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) v[i + e] = (float)r.v[e];
  }
}
template <int DP> __device__ __forceinline__ float dot_row(const float (&a)[DP], const float (&b)[DP]) {
  float s = 0.f;
#pragma unroll
  for (int i = 0; i < DP; ++i) s += a[i] * b[i];
  return s;
}
template <int N, int DP> __device__ __forceinline__ void sum_halves(float (&v)[DP], int lane) {
  if constexpr (N > 0) {
    const bool up = (lane & N) != 0;
#pragma unroll
    for (int i = 0; i < N; ++i) {
      const float mine = up ? v[N + i] : v[i], other = up ? v[i] : v[N + i];
      v[i] = mine + __shfl_xor(other, N, 64);
    }
    sum_halves<N / 2>(v, lane);
  }
}
template <int DP> __device__ __forceinline__ float sum_lanes(float (&v)[DP], int lane) {
  sum_halves<DP / 2>(v, lane);
#pragma unroll
  for (int n = DP; n < 64; n *= 2) v[0] += __shfl_xor(v[0], n, 64);
  return v[0];
}

// the wavefront's (batch, head, row); a launch has fewer than 2^26 of them (2^32 work-items), so 32-bit divisions do
struct NarrowRow {
  int b, h, t;
};
__device__ __forceinline__ NarrowRow narrow_row(int S, int nh) {
  const unsigned gid = blockIdx.x * 4u + (unsigned)__builtin_amdgcn_readfirstlane(threadIdx.x >> 6), pair = gid / (unsigned)S, b = pair / (unsigned)nh;
  return NarrowRow{(int)b, (int)(pair - b * (unsigned)nh), (int)(gid - pair * (unsigned)S)};
}

// No more wavefronts on a SIMD than the rows they stream (a cache line each, read in pieces) leave room for in the L1 cache: 3 sequences of
// 1000 tokens, 8 heads of 10 in fp32, forward 184 us without the limit, 99 with; 1000 tokens, 4 heads of 8, backward 62 and 50.
template <typename T, int DP, bool FULL>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, DP == 32 ? 3 : 4))) attn_fwd_narrow_kernel(const T* __restrict__ qkv, T* __restrict__ o, float* __restrict__ lse, int B, int S,
                                                              int nh, int d) {
  const int lane = threadIdx.x & 63;
  const NarrowRow row = narrow_row(S, nh);
  if (row.b >= B) return;
  const int t = row.t, h = row.h, b = row.b;
  const int64_t H = (int64_t)nh * d, ld = 3 * H;
  const T* qbase = qkv + (int64_t)b * S * ld + (int64_t)h * d;
  const float scale = 1.0f / sqrtf((float)d);
  float q[DP], acc[DP], m = -INFINITY, z = 0.f;
  load_row<FULL>(q, qbase + (int64_t)t * ld, d);
#pragma unroll
  for (int i = 0; i < DP; ++i) acc[i] = 0.f;
  for (int u = lane; u <= t; u += 64) {
    float k[DP], v[DP];
    const T* kv = qbase + (int64_t)u * ld;
    load_row<FULL>(k, kv + H, d);
    load_row<FULL>(v, kv + 2 * H, d);
    // a key whose score overflowed to -inf has weight 0, also where the lane has seen no other yet (expf(-inf + inf) is NaN)
    const float s = dot_row(q, k) * scale, mn = fmaxf(m, s);
    const float keep = m == -INFINITY ? 0.f : expf(m - mn), p = s == -INFINITY ? 0.f : expf(s - mn);
    m = mn;
    z = z * keep + p;
#pragma unroll
    for (int i = 0; i < DP; ++i) acc[i] = acc[i] * keep + p * v[i];
  }
  const float mt = wave_max(m), keep = expf(m - mt);        // lanes without a key: exp(-inf) = 0
  z = wave_sum(z * keep);
#pragma unroll
  for (int i = 0; i < DP; ++i) acc[i] *= keep;
  const float r = sum_lanes(acc, lane) * (1.0f / z);
  if (lane < d) o[((int64_t)b * S + t) * H + (int64_t)h * d + lane] = (T)r;
  if (lane == 0) lse[((int64_t)b * nh + h) * S + t] = mt + logf(z);
}

// blockIdx.y = 0: dq of a query; 1: dk, dv of a key (along y, since a launch takes fewer than 2^32 work-items along x).  D[t] = dO[t] . o[t] is formed where it is needed.  The gradients of
// rotated q and k are rotated back before they leave where a table is given.
template <typename T, int DP, bool FULL>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 5))) attn_bwd_narrow_kernel(const T* __restrict__ qkv, const T* __restrict__ o, const T* __restrict__ dO,
                                                              const float* __restrict__ lse, T* __restrict__ dqkv, int B, int S, int nh, int d,
                                                              const float* __restrict__ rope) {
  const int lane = threadIdx.x & 63;
  const bool keys = blockIdx.y != 0;
  const NarrowRow row = narrow_row(S, nh);
  if (row.b >= B) return;
  const int t = row.t, h = row.h, b = row.b;
  const int64_t H = (int64_t)nh * d, ld = 3 * H;
  const T* qbase = qkv + (int64_t)b * S * ld + (int64_t)h * d;
  const int64_t ooff = (int64_t)b * S * H + (int64_t)h * d;
  const float* L = lse + ((int64_t)b * nh + h) * S;
  const float scale = 1.0f / sqrtf((float)d);
  auto leave = [&](float v, int64_t part, bool rotate) {
    if (rope && rotate) {
      const float w = __shfl_xor(v, 1, 64);
      if (lane < d) {
        const float* tb = rope + ((int64_t)t * (d / 2) + lane / 2) * 2;
        v = lane & 1 ? v * tb[0] - w * tb[1] : v * tb[0] + w * tb[1];
      }
    }
    if (lane < d) dqkv[((int64_t)b * S + t) * ld + part * H + (int64_t)h * d + lane] = (T)v;
  };
  float x[DP], y[DP], acc[DP], acc2[DP];
#pragma unroll
  for (int i = 0; i < DP; ++i) { acc[i] = 0.f; acc2[i] = 0.f; }
  if (!keys) {        // x = q[t], y = dO[t]
    load_row<FULL>(x, qbase + (int64_t)t * ld, d);
    load_row<FULL>(y, dO + ooff + (int64_t)t * H, d);
    load_row<FULL>(acc2, o + ooff + (int64_t)t * H, d);
    const float Dt = dot_row(y, acc2), Lt = L[t];
    for (int u = lane; u <= t; u += 64) {
      float k[DP], v[DP];
      const T* kv = qbase + (int64_t)u * ld;
      load_row<FULL>(k, kv + H, d);
      load_row<FULL>(v, kv + 2 * H, d);
      const float ds = expf(dot_row(x, k) * scale - Lt) * (dot_row(y, v) - Dt);
#pragma unroll
      for (int i = 0; i < DP; ++i) acc[i] += ds * k[i];
    }
    leave(sum_lanes(acc, lane) * scale, 0, true);
  } else {            // x = k[t], y = v[t]
    load_row<FULL>(x, qbase + (int64_t)t * ld + H, d);
    load_row<FULL>(y, qbase + (int64_t)t * ld + 2 * H, d);
    for (int u = t + lane; u < S; u += 64) {
      float q[DP], g[DP], ov[DP];
      load_row<FULL>(q, qbase + (int64_t)u * ld, d);
      load_row<FULL>(g, dO + ooff + (int64_t)u * H, d);
      load_row<FULL>(ov, o + ooff + (int64_t)u * H, d);
      const float p = expf(dot_row(q, x) * scale - L[u]), ds = p * (dot_row(g, y) - dot_row(g, ov));
#pragma unroll
      for (int i = 0; i < DP; ++i) {
        acc[i] += ds * q[i];
        acc2[i] += p * g[i];
      }
    }
    leave(sum_lanes(acc, lane) * scale, 1, true);
    leave(sum_lanes(acc2, lane), 2, false);
  }
}

// =============================================================================== attention, any head
// One wavefront per (batch, head, row).  Scores of the row live in LDS (S floats per wavefront).
constexpr int kNarrowHead = 32;      // wider rows would not fit a lane's registers
constexpr int kGenAttnMaxS = 4096;  // backward: 4 wavefronts x 2 arrays x 4096 x 4 B = 128 KiB of LDS
bool attn_generic_supported(int S, int d) { return S >= 1 && S <= kGenAttnMaxS && d >= 2; }

template <typename T>
__device__ __forceinline__ float dot_d(const T* a, const T* b, int d) {
  float s = 0.f;
  for (int i = 0; i < d; ++i) s += (float)a[i] * (float)b[i];
  return s;
}

// o[t] = sum_{u<=t} softmax_u(q[t].k[u]/sqrt(d)) v[u];  lse[t] = log sum_u exp(score)
template <typename T>
__global__ void __launch_bounds__(256) attn_fwd_generic_kernel(const T* __restrict__ qkv, T* __restrict__ o,
                                                               float* __restrict__ lse, int B, int S, int nh, int d) {
  extern __shared__ float lds[];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  float* p = lds + (size_t)wave * S;
  const int64_t gid = (int64_t)blockIdx.x * 4 + wave;  // (b, h, t)
  const int64_t total = (int64_t)B * nh * S;
  if (gid >= total) return;
  const int t = (int)(gid % S);
  const int h = (int)((gid / S) % nh);
  const int b = (int)(gid / ((int64_t)S * nh));
  const int64_t H = (int64_t)nh * d, ld = 3 * H;
  const T* qrow = qkv + ((int64_t)b * S + t) * ld + (int64_t)h * d;
  const T* kbase = qkv + (int64_t)b * S * ld + H + (int64_t)h * d;
  const T* vbase = kbase + H;
  const float scale = 1.0f / sqrtf((float)d);
  float m = -INFINITY;
  for (int u = lane; u <= t; u += 64) {
    const float s = dot_d(qrow, kbase + (int64_t)u * ld, d) * scale;
    p[u] = s;
    m = fmaxf(m, s);
  }
  m = wave_max(m);
  float z = 0.f;
  for (int u = lane; u <= t; u += 64) {
    const float e = expf(p[u] - m);
    p[u] = e;
    z += e;
  }
  z = wave_sum(z);
  if (lane == 0) lse[((int64_t)b * nh + h) * S + t] = m + logf(z);
  const float inv = 1.0f / z;
  // LDS writes above are read by other lanes of the same wavefront below
  __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0)
  __builtin_amdgcn_wave_barrier();
  T* orow = o + ((int64_t)b * S + t) * H + (int64_t)h * d;
  for (int i = lane; i < d; i += 64) {
    float acc = 0.f;
    for (int u = 0; u <= t; ++u) acc += p[u] * (float)vbase[(int64_t)u * ld + i];
    orow[i] = (T)(acc * inv);
  }
}

// dq[t] = (1/sqrt d) sum_{u<=t} dS[t,u] k[u],  dS = P (dP - D),  P = exp(score - lse),  dP = do[t].v[u]
template <typename T>
__global__ void __launch_bounds__(256) attn_bwd_dq_generic_kernel(const T* __restrict__ qkv, const T* __restrict__ dO,
                                                                  const float* __restrict__ lse, const float* __restrict__ D,
                                                                  T* __restrict__ dqkv, int B, int S, int nh, int d) {
  extern __shared__ float lds[];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  float* ds = lds + (size_t)wave * S;
  const int64_t gid = (int64_t)blockIdx.x * 4 + wave;
  const int64_t total = (int64_t)B * nh * S;
  if (gid >= total) return;
  const int t = (int)(gid % S);
  const int h = (int)((gid / S) % nh);
  const int b = (int)(gid / ((int64_t)S * nh));
  const int64_t H = (int64_t)nh * d, ld = 3 * H;
  const T* qrow = qkv + ((int64_t)b * S + t) * ld + (int64_t)h * d;
  const T* kbase = qkv + (int64_t)b * S * ld + H + (int64_t)h * d;
  const T* vbase = kbase + H;
  const T* dorow = dO + ((int64_t)b * S + t) * H + (int64_t)h * d;
  const float scale = 1.0f / sqrtf((float)d);
  const float L = lse[((int64_t)b * nh + h) * S + t];
  const float Dt = D[((int64_t)b * nh + h) * S + t];
  for (int u = lane; u <= t; u += 64) {
    const float s = dot_d(qrow, kbase + (int64_t)u * ld, d) * scale;
    const float pr = expf(s - L);
    const float dP = dot_d(dorow, vbase + (int64_t)u * ld, d);
    ds[u] = pr * (dP - Dt);
  }
  __builtin_amdgcn_s_waitcnt(0xc07f);
  __builtin_amdgcn_wave_barrier();
  T* dqrow = dqkv + ((int64_t)b * S + t) * ld + (int64_t)h * d;
  for (int i = lane; i < d; i += 64) {
    float acc = 0.f;
    for (int u = 0; u <= t; ++u) acc += ds[u] * (float)kbase[(int64_t)u * ld + i];
    dqrow[i] = (T)(acc * scale);
  }
}

// dv[u] = sum_{t>=u} P[t,u] do[t];  dk[u] = (1/sqrt d) sum_{t>=u} dS[t,u] q[t]
template <typename T>
__global__ void __launch_bounds__(256) attn_bwd_dkv_generic_kernel(const T* __restrict__ qkv, const T* __restrict__ dO,
                                                                   const float* __restrict__ lse, const float* __restrict__ D,
                                                                   T* __restrict__ dqkv, int B, int S, int nh, int d) {
  extern __shared__ float lds[];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  float* pp = lds + (size_t)wave * 2 * S;
  float* ds = pp + S;
  const int64_t gid = (int64_t)blockIdx.x * 4 + wave;
  const int64_t total = (int64_t)B * nh * S;
  if (gid >= total) return;
  const int u = (int)(gid % S);
  const int h = (int)((gid / S) % nh);
  const int b = (int)(gid / ((int64_t)S * nh));
  const int64_t H = (int64_t)nh * d, ld = 3 * H;
  const T* qbase = qkv + (int64_t)b * S * ld + (int64_t)h * d;
  const T* krow = qbase + H + (int64_t)u * ld;
  const T* vrow = krow + H;
  const T* dobase = dO + (int64_t)b * S * H + (int64_t)h * d;
  const float* Lb = lse + ((int64_t)b * nh + h) * S;
  const float* Db = D + ((int64_t)b * nh + h) * S;
  const float scale = 1.0f / sqrtf((float)d);
  for (int t = u + lane; t < S; t += 64) {
    const float s = dot_d(qbase + (int64_t)t * ld, krow, d) * scale;
    const float pr = expf(s - Lb[t]);
    const float dP = dot_d(dobase + (int64_t)t * H, vrow, d);
    pp[t - u] = pr;
    ds[t - u] = pr * (dP - Db[t]);
  }
  __builtin_amdgcn_s_waitcnt(0xc07f);
  __builtin_amdgcn_wave_barrier();
  T* dkrow = dqkv + ((int64_t)b * S + u) * ld + H + (int64_t)h * d;
  T* dvrow = dkrow + H;
  for (int i = lane; i < d; i += 64) {
    float ak = 0.f, av = 0.f;
    for (int t = u; t < S; ++t) {
      ak += ds[t - u] * (float)qbase[(int64_t)t * ld + i];
      av += pp[t - u] * (float)dobase[(int64_t)t * H + i];
    }
    dkrow[i] = (T)(ak * scale);
    dvrow[i] = (T)av;
  }
}

template <typename T>
static int attn_fwd_generic_t(int B, int S, int nh, int d, const T* qkv, T* o, float* lse, hipStream_t st) {
  const int64_t total = (int64_t)B * nh * S;
  if (total == 0) return 0;
  const size_t lds = (size_t)4 * S * sizeof(float);
  TAW_SET_LDS_LIMIT_ONCE((attn_fwd_generic_kernel<T>), (size_t)4 * kGenAttnMaxS * sizeof(float));
  hipLaunchKernelGGL((attn_fwd_generic_kernel<T>), dim3((unsigned)((total + 3) / 4)), dim3(256), lds, st, qkv, o, lse, B, S, nh, d);
  return (int)hipGetLastError();
}

template <typename T>
static int attn_fwd_narrow_t(int B, int S, int nh, int d, const T* qkv, T* o, float* lse, hipStream_t st) {
  const dim3 grid((unsigned)(((int64_t)B * nh * S + 3) / 4));
#define TAW_NARROW(DP, FULL) hipLaunchKernelGGL((attn_fwd_narrow_kernel<T, DP, FULL>), grid, dim3(256), 0, st, qkv, o, lse, B, S, nh, d)
  if (d == 8) TAW_NARROW(8, true); else if (d == 16) TAW_NARROW(16, true); else if (d == 32) TAW_NARROW(32, true);
  else if (d < 8) TAW_NARROW(8, false); else if (d < 16) TAW_NARROW(16, false); else TAW_NARROW(32, false);
#undef TAW_NARROW
  return (int)hipGetLastError();
}

int launch_attn_fwd_generic(int dtype, int B, int S, int nh, int d, const void* qkv, void* o, float* lse, hipStream_t st) {
  if (d <= kNarrowHead) {
    if (dtype == DT_BF16) return attn_fwd_narrow_t<bf16_t>(B, S, nh, d, (const bf16_t*)qkv, (bf16_t*)o, lse, st);
    return attn_fwd_narrow_t<float>(B, S, nh, d, (const float*)qkv, (float*)o, lse, st);
  }
  if (dtype == DT_BF16) return attn_fwd_generic_t<bf16_t>(B, S, nh, d, (const bf16_t*)qkv, (bf16_t*)o, lse, st);
  return attn_fwd_generic_t<float>(B, S, nh, d, (const float*)qkv, (float*)o, lse, st);
}

template <typename T>
static int attn_bwd_generic_t(int B, int S, int nh, int d, const T* qkv, const T* dO, const float* lse, const float* D,
                              T* dqkv, hipStream_t st) {
  const int64_t total = (int64_t)B * nh * S;
  if (total == 0) return 0;
  const unsigned grid = (unsigned)((total + 3) / 4);
  size_t lds = (size_t)4 * S * sizeof(float);
  TAW_SET_LDS_LIMIT_ONCE((attn_bwd_dq_generic_kernel<T>), (size_t)4 * kGenAttnMaxS * sizeof(float));
  hipLaunchKernelGGL((attn_bwd_dq_generic_kernel<T>), dim3(grid), dim3(256), lds, st, qkv, dO, lse, D, dqkv, B, S, nh, d);
  int rc = (int)hipGetLastError();
  if (rc) return rc;
  lds *= 2;
  TAW_SET_LDS_LIMIT_ONCE((attn_bwd_dkv_generic_kernel<T>), (size_t)8 * kGenAttnMaxS * sizeof(float));
  hipLaunchKernelGGL((attn_bwd_dkv_generic_kernel<T>), dim3(grid), dim3(256), lds, st, qkv, dO, lse, D, dqkv, B, S, nh, d);
  return (int)hipGetLastError();
}

template <typename T>
static int attn_bwd_narrow_t(int B, int S, int nh, int d, const T* qkv, const T* o, const T* dO, const float* lse, T* dqkv, const float* rope, hipStream_t st) {
  const dim3 grid((unsigned)(((int64_t)B * nh * S + 3) / 4), 2);
#define TAW_NARROW(DP, FULL) hipLaunchKernelGGL((attn_bwd_narrow_kernel<T, DP, FULL>), grid, dim3(256), 0, st, qkv, o, dO, lse, dqkv, B, S, nh, d, rope)
  if (d == 8) TAW_NARROW(8, true); else if (d == 16) TAW_NARROW(16, true); else if (d == 32) TAW_NARROW(32, true);
  else if (d < 8) TAW_NARROW(8, false); else if (d < 16) TAW_NARROW(16, false); else TAW_NARROW(32, false);
#undef TAW_NARROW
  return (int)hipGetLastError();
}

int launch_attn_bwd_generic(int dtype, int B, int S, int nh, int d, const void* qkv, const void* o, const void* dO,
                            const float* lse, float* D, void* dqkv, const float* rope, hipStream_t st) {
  if (d <= kNarrowHead) {
    if (dtype == DT_BF16)
      return attn_bwd_narrow_t<bf16_t>(B, S, nh, d, (const bf16_t*)qkv, (const bf16_t*)o, (const bf16_t*)dO, lse, (bf16_t*)dqkv, rope, st);
    return attn_bwd_narrow_t<float>(B, S, nh, d, (const float*)qkv, (const float*)o, (const float*)dO, lse, (float*)dqkv, rope, st);
  }
  const int64_t H = (int64_t)nh * d;
  int rc = launch_attn_rowdot(dtype, B, S, nh, d, o, H, dO, H, D, st);
  if (rc) return rc;
  rc = dtype == DT_BF16 ? attn_bwd_generic_t<bf16_t>(B, S, nh, d, (const bf16_t*)qkv, (const bf16_t*)dO, lse, D, (bf16_t*)dqkv, st)
                        : attn_bwd_generic_t<float>(B, S, nh, d, (const float*)qkv, (const float*)dO, lse, D, (float*)dqkv, st);
  if (rc || !rope) return rc;
  return launch_rope(dtype, B, S, (int)(2 * H), d, dqkv, 3 * H, rope, 1, st);
}

}  // namespace taw
