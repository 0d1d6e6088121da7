// Direct solve of the Kernel-SHAP regression for small player counts:
// popcount Gram matrix + blocked Cholesky, all accumulation in fp64.
//
// Paper, "Distributed Shapley Computations": the direct method forms
// G = M^T W M and r = M^T W y and solves G phi = r. Here the efficiency
// decomposition (f(N) = phi_0 + sum phi_i) is imposed exactly: with
// delta = y_1 - y_0, psi = phi - delta/n, P = I - 11^T/n and
// t_i = y_i - y_0 - (delta/n)|S_i|, psi solves (P G P + gamma 11^T/n) psi = P c,
// c = M^T W t, and any gamma > 0 leaves psi orthogonal to 1.
//
// G[a][b] = sum_i w_i z_ia z_ib is computed from the transposed bit matrix: a
// 64-row word whose rows share one weight contributes w * popcount(col_a & col_b);
// a word that straddles weight classes is a dense 64-row contraction on the matrix cores.
#include <stdlib.h>

#include "internal.h"
#include "small_game.h"
#include "solve_common.h"

namespace {

constexpr int kThreads = 256;
constexpr int kTile = 64;
constexpr int kChunk = 32;  // 64-row words per LDS chunk

// which rows enter the sums, with which weight and right-hand-side coefficient.
// Paired rows (2r, 2r+1 complementary, one weight w): z z^T + zc zc^T = 2 z z^T - z 1^T - 1 z^T + 11^T and
// t z + tc zc = (t - tc) z + tc 1; the terms with 1 vanish under the projection P, so only the small
// member is used, with weight 2w and coefficient w (t_2r - t_2r+1). Otherwise every row is used.
__device__ __forceinline__ float used_row_weight(const float* w, int64_t r, int paired) {
  const int64_t i = paired ? 2 * r : r;
  const float wi = w[i];
  return i < 2 ? 0.f : paired ? 2.0f * wi : wi;  // the two constraint rows carry no weight
}

__global__ void used_row_rhs_kernel(const float* wc, const double* t, int64_t R, int paired, double* gc) {
  const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= R) return;
  gc[r] = paired ? (double)wc[2 * r] * (t[2 * r] - t[2 * r + 1]) : (double)wc[r] * t[r];
}

// How the column-wise Gram kernel treats a word of 64 rows (`uni`): 1 = one weight (popcount), 0 = mixed weights and sparse rows
// (walk the set bits of the AND), 2 = mixed weights and dense rows (matrix cores), 3 = none of its rows is left to it. The density
// is read off the first row of the word (rows are ordered by size): with a fraction p of the columns set, a pair of
// columns shares about 64 p^2 rows of the word, and walking them costs more than the fixed-price contraction from p of
// about 0.08 on (measured).
constexpr float kDenseFraction = 0.08f;

// ---- sparse rows: row-wise outer products -------------------------------------------------------
// A row with s of n columns set touches s^2 entries of G, while the column-wise kernel pays for all
// n^2/2 pairs of columns whatever the row holds; up to a density of about a tenth the row-wise form is the
// cheaper one, and in a Kernel-SHAP sample most rows are far sparser than that. Rows are split by their
// own popcount: sparse ones go to gram_rows_kernel, the others stay with the column-wise kernel
// (`keep` holds their bits per 64-row word).
//   Zc[cb][r] = word cb of row r (zero for a kept row): the 64 columns of a tile side for all rows, contiguous.
//   wq[r]     = weight of row r in fixed point, w_r * 2^e with e chosen so that the sum of all weights stays
//               below 2^62: every entry of G is a sum over a subset of the rows, so the integer sums cannot
//               overflow, they are exact, and they do not depend on the order of the atomic additions.
constexpr int kSparseDivisor = 12;  // rows with at most n / 12 columns set are sparse (measured optimum: flat from 8 to 16)

// The used rows' weights gw and scale[0] = 2^e (0 if they are not all finite and non-negative: then every row is kept). One
// workgroup; what bounds it is the latency of its loads, so that each of its threads has eight under way.
constexpr int kWeightThreads = 1024;
__global__ __launch_bounds__(kWeightThreads) void gram_weights_kernel(const float* w, int64_t R, int paired, float* gw, double* scale) {
  constexpr int kAhead = 8;
  __shared__ double sh[kWeightThreads / 64];
  const int tid = threadIdx.x;
  double a = 0.0;
  int b = 0;
  for (int64_t i0 = tid; i0 < R; i0 += kAhead * kWeightThreads) {
    float v[kAhead];
#pragma unroll
    for (int u = 0; u < kAhead; ++u) {
      const int64_t i = i0 + u * kWeightThreads;
      v[u] = used_row_weight(w, i < R ? i : R - 1, paired);
    }
#pragma unroll
    for (int u = 0; u < kAhead; ++u) {
      const int64_t i = i0 + u * kWeightThreads;
      if (i >= R) break;
      gw[i] = v[u];
      if (!(v[u] >= 0.f) || v[u] > 3.0e38f) b = 1;
      a += (double)v[u];
    }
  }
  a = ds_wave_sum(a);
  if ((tid & 63) == 0) sh[tid >> 6] = a;
  const int anyb = __syncthreads_or(b);
  if (tid == 0) {
    double x = 0.0;
    for (int i = 0; i < kWeightThreads / 64; ++i) x += sh[i];
    double sc = 0.0;
    if (!anyb && x > 0.0 && x < 1e300) {
      int e;
      frexp(x, &e);  // x < 2^e
      sc = ldexp(1.0, 61 - e);
    }
    scale[0] = sc;
  }
}

// Sparse or kept, for every used row, and from that what the column-wise kernel does with the words of 64 rows: a workgroup takes the
// rows of a word, each wave four of them with their loads in flight together. (As a kernel of a wave per row, one that
// read the rows' weights back word by word, and two that cleared and summed for them, it took 42 us at 10,000 rows of 1,010 columns; the
// two kernels here take 11.)
constexpr int kClassWaves = 16;
constexpr int64_t kClassGridX = 1 << 14;   // workgroups in x direction, the rest in y: 2^32 threads in one direction (2^28 rows) are refused
__global__ __launch_bounds__(64 * kClassWaves) void gram_row_class_kernel(const uint64_t* Z, int64_t R, int64_t W, int64_t n,
                                                                          int64_t row_step, const float* gw, const double* scale,
                                                                          int sparse_divisor, float dense_fraction, uint64_t* Zc,
                                                                          unsigned long long* keep, unsigned long long* wq, float* wu,
                                                                          int32_t* uni) {
  constexpr int kRows = 64 / kClassWaves;
  __shared__ int set[64];   // columns set in a row of the word
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t wd = (int64_t)blockIdx.y * gridDim.x + blockIdx.x, r0 = wd * 64 + wave * kRows;
  if (wd * 64 >= R) return;
  const double sc = scale[0];
  const uint64_t* zr[kRows];
  int c[kRows];
#pragma unroll
  for (int u = 0; u < kRows; ++u) {
    zr[u] = Z + (r0 + u < R ? r0 + u : R - 1) * row_step * W;
    c[u] = 0;
  }
  uint64_t z0[kRows];   // the first 64 words stay in registers for the copy
  for (int64_t x0 = 0; x0 < W; x0 += 64) {
    uint64_t z[kRows];
#pragma unroll
    for (int u = 0; u < kRows; ++u) z[u] = zr[u][x0 + lane < W ? x0 + lane : W - 1];
#pragma unroll
    for (int u = 0; u < kRows; ++u) {
      if (x0 == 0) z0[u] = z[u];
      c[u] += x0 + lane < W ? __popcll(z[u]) : 0;
    }
  }
  for (int o = 32; o > 0; o >>= 1)
#pragma unroll
    for (int u = 0; u < kRows; ++u) c[u] += __shfl_xor(c[u], o, 64);
#pragma unroll
  for (int u = 0; u < kRows; ++u) {
    const int64_t r = r0 + u;
    if (lane == 0) set[wave * kRows + u] = c[u];
    if (r >= R) continue;
    const bool sparse = sc > 0.0 && (int64_t)c[u] * sparse_divisor <= n;
    if (lane < W) Zc[lane * R + r] = sparse ? z0[u] : 0ull;
    for (int64_t x = 64 + lane; x < W; x += 64) Zc[x * R + r] = sparse ? zr[u][x] : 0ull;
    if (lane == 0) wq[r] = sparse ? (unsigned long long)llrint((double)gw[r] * sc) : 0ull;
  }
  __syncthreads();
  if (wave > 0) return;
  const int64_t r = wd * 64 + lane;
  const int mine = set[lane];
  const bool kept = r < R && !(sc > 0.0 && (int64_t)mine * sparse_divisor <= n);
  const unsigned long long km = __ballot(kept);
  const int fb = km ? __ffsll((long long)km) - 1 : 0;   // the first kept row stands for the word
  const float wr = gw[r < R ? r : R - 1], first = __shfl(wr, fb, 64);
  const int same = __ballot(kept && wr != first) == 0ull;
  if (lane == 0) {
    keep[wd] = km;
    wu[wd] = km ? first : 0.f;
    uni[wd] = !km ? 3 : same ? 1 : (float)set[fb] > dense_fraction * (float)n ? 2 : 0;
  }
}

// One 64x64 tile of G per workgroup (lower tiles); streams the two column-block words of every row.
__device__ __forceinline__ void gram_rows_tile(const uint64_t* Zc, const unsigned long long* wq, int64_t R, int64_t n,
                                               const double* scale, double* G, int ta, int tb, unsigned long long* acc) {
  const int tid = threadIdx.x;
  for (int i = tid; i < kTile * kTile; i += kThreads) acc[i] = 0ull;
  __syncthreads();
  const uint64_t* Ac = Zc + (size_t)ta * R;
  const uint64_t* Bc = Zc + (size_t)tb * R;
  constexpr int kRowsPerStep = 8;  // rows per step: their loads are in flight together (addresses clamped, not skipped)
  for (int64_t r0 = tid; r0 < R; r0 += kRowsPerStep * kThreads) {
    uint64_t av[kRowsPerStep], bv[kRowsPerStep];
    unsigned long long wvv[kRowsPerStep];
#pragma unroll
    for (int u = 0; u < kRowsPerStep; ++u) {
      const int64_t r = r0 + (int64_t)u * kThreads, rc = r < R ? r : R - 1;
      av[u] = Ac[rc];
      bv[u] = Bc[rc];
      wvv[u] = wq[rc];
    }
#pragma unroll
    for (int u = 0; u < kRowsPerStep; ++u) {
      if (r0 + (int64_t)u * kThreads >= R || av[u] == 0ull || bv[u] == 0ull) continue;
      const unsigned long long wv = wvv[u];
      uint64_t am = av[u];
      while (am) {
        const int a = __ffsll((long long)am) - 1;
        am &= am - 1;
        uint64_t bm = bv[u];
        while (bm) {
          const int b = __ffsll((long long)bm) - 1;
          bm &= bm - 1;
          atomicAdd(&acc[a * kTile + b], wv);
        }
      }
    }
  }
  __syncthreads();
  const double sc = scale[0];
  const double inv = sc > 0.0 ? 1.0 / sc : 0.0;
  for (int i = tid; i < kTile * kTile; i += kThreads) {
    const int64_t a = (int64_t)ta * kTile + (i >> 6), b = (int64_t)tb * kTile + (i & 63);
    if (a < n && b < n) {
      G[a * n + b] = (double)acc[i] * inv;
    }
  }
}

__global__ __launch_bounds__(kThreads) void gram_rows_kernel(const uint64_t* Zc, const unsigned long long* wq, int64_t R,
                                                             int64_t n, const double* scale, double* G) {
  if (blockIdx.x > blockIdx.y) return;
  __shared__ unsigned long long acc[kTile * kTile];
  gram_rows_tile(Zc, wq, R, n, scale, G, blockIdx.y, blockIdx.x, acc);
}

// A tile's share of the row sums of G, of which only the lower tiles are kept (diagonal tiles whole): part[t][a] = sum of G[a][b] over the
// 64 columns b of tile column t. The tile T (values past n zero) gives the row sums of its rows and, below the diagonal, the column sums
// that stand for the tile above it. (Stored on both sides, the tiles above the diagonal as 8-byte pieces, and summed by row afterwards: 6,007
// columns: 1,624 us for the Gram kernels, the sums and the system matrix, now 1,425.)
__device__ __forceinline__ void gram_tile_sums(const double (*T)[kTile + 1], int ta, int tb, int64_t n, double* part) {
  const int tid = threadIdx.x, i = tid & 63;
  if (tid >= 128 || (tid >= 64 && ta == tb)) return;
  const bool cols = tid >= 64;
  double s = 0.0;
#pragma unroll 16
  for (int k = 0; k < kTile; ++k) s += cols ? T[k][i] : T[i][k];
  const int64_t a = (int64_t)(cols ? tb : ta) * kTile + i;
  if (a < n) part[(int64_t)(cols ? ta : tb) * n + a] = s;
}

// One 64x64 tile of G per workgroup and slice of the row words (split-K); each slice writes the lower tiles of its own partial
// matrix, summed later in a fixed order. A single slice leaves the tile's sums in `part` (else nullptr).
// A word of 64 rows that share one weight costs an AND and a popcount per pair of columns. A word that
// straddles weight classes (most words past the first few classes: a class soon has fewer than 64 rows)
// either walks the set bits of the AND (sparse rows) or, when its rows are dense, is treated as the small
// dense contraction it is, sum_r (w_r z_ra) z_rb, on the matrix cores. The fp32 weight is split into three
// bfloat16 pieces (w = w1 + w2 + w3 to 24 bits; a bit is exactly 0 or 1 in bfloat16), so the contraction runs
// as three v_mfma_f32_32x32x16_bf16 per 16 rows with fp32 accumulation, many times the rate of the fp32
// instruction: lane l supplies A[m = l%32][k = 8*(l/32) + j] = piece of row r * bit r of column m's word and
// B[k][n = l%32] = bit r of column n's word, r = 16 kb + k, j < 8 (two values per register). Operands are
// made with look-ups: a 16-entry LDS table (whose entries lie in banks of their own, which those of a byte's would not) turns
// four bits into the two registers of 16-bit masks (or of bfloat16 ones for B), which the packed weight pieces are ANDed with.
// (Eight rows at a time with v_mfma_f32_32x32x8bf16_1k, the same 32 cycles each: 6,007 columns, 20,000 rows 1,050 us, now 877.) Each wave owns a 32x32 quadrant of the
// tile (accumulator register i of lane l is D[8*(i/4) + 4*(l/32) + i%4][l%32]). Both paths add up in fp32
// within a chunk of 32 words and in fp64 across chunks.
// The sparse rows' part is in slice 0 already (`rows_apart`: gram_rows_kernel, whose own launch holds more workgroups per compute unit), or
// it is the launch's last slice: where the tiles of one triangle do not fill the GPU, both kinds run together
// (1,010 columns, 10,000 rows: 48 + 51 us apart, 76 together).
typedef float gram_f16_t __attribute__((ext_vector_type(16)));
typedef __bf16 gram_b8_t __attribute__((ext_vector_type(8)));
typedef unsigned int gram_u4_t __attribute__((ext_vector_type(4)));
typedef unsigned int gram_u2_t __attribute__((ext_vector_type(2)));

__device__ __forceinline__ uint32_t bf16_bits_rn(float x) {  // nearest-even bfloat16 of a finite float, as 16 bits
  uint32_t u = __float_as_uint(x);
  u += 0x7FFFu + ((u >> 16) & 1u);
  return u >> 16;
}
// 16-bit lane masks of two bits: bit 0 -> low half, bit 1 -> high half
__device__ __forceinline__ uint32_t pair_mask(uint32_t two_bits) {
  return ((0u - (two_bits & 1u)) & 0xFFFFu) | ((0u - ((two_bits >> 1) & 1u)) & 0xFFFF0000u);
}

__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2, 4))) void gram_kernel(const uint64_t* Zt, int64_t n, int64_t k, int64_t KW,
                                                        const float* w, const float* wu, const int32_t* uni,
                                                        const uint64_t* keep, double* Gp, int64_t words_per_slice, int rows_apart,
                                                        const uint64_t* Zc, const unsigned long long* wq, const double* scale,
                                                        double* part) {
  const int ta = blockIdx.y, tb = blockIdx.x;
  if (tb > ta) return;
  // As | Bs during the accumulation; reused as one 64 x 65 fp64 tile when the two paths are merged
  __shared__ __attribute__((aligned(16))) uint64_t raw[2 * kTile * (kChunk + 1)];
  static_assert(sizeof(uint64_t) * 2 * kTile * (kChunk + 1) >= sizeof(double) * kTile * (kTile + 1), "merge tile must fit");
  uint64_t (*As)[kChunk + 1] = (uint64_t (*)[kChunk + 1])raw;
  uint64_t (*Bs)[kChunk + 1] = (uint64_t (*)[kChunk + 1])(raw + kTile * (kChunk + 1));
  __shared__ float wrow[kChunk * 64];
  __shared__ __align__(16) gram_u2_t wpk[3][kChunk * 16];  // weight pieces as bfloat16, rows 4j..4j+3 of a word per entry
  __shared__ gram_u2_t tabA[16], tabB[16];   // four bits -> 16-bit masks / bfloat16 ones (two registers)
  __shared__ float wus[kChunk];
  __shared__ int unis[kChunk];
  if (!rows_apart && blockIdx.z == gridDim.z - 1) {
    static_assert(sizeof(uint64_t) * kTile * kTile <= sizeof(raw), "the accumulators of the sparse rows must fit");
    gram_rows_tile(Zc, wq, k, n, scale, Gp + (size_t)blockIdx.z * n * n, ta, tb, (unsigned long long*)raw);
    return;
  }
  const int tid = threadIdx.x, tx = tid & 15, ty = tid >> 4;
  const int lane = tid & 63, wave = tid >> 6, half = lane >> 5, l32 = lane & 31;
  if (tid < 16) {
    const gram_u2_t m = {pair_mask(tid & 3u), pair_mask((uint32_t)tid >> 2)};
    tabA[tid] = m;
    tabB[tid] = gram_u2_t{m.x & 0x3F803F80u, m.y & 0x3F803F80u};
  }
  const int wi = (wave >> 1) * 32, wj = (wave & 1) * 32;
  const int64_t a0 = (int64_t)ta * kTile, b0 = (int64_t)tb * kTile;
  double* G = Gp + (size_t)blockIdx.z * n * n;
  const int64_t wbeg = (int64_t)blockIdx.z * words_per_slice;
  const int64_t wend = wbeg + words_per_slice < KW ? wbeg + words_per_slice : KW;
  double acc[4][4];   // popcount path: elements (ty + 16 i, tx + 16 j)
  double accm[16];    // matrix-core path: elements (wi + 8*(i/4) + 4*half + i%4, wj + l32)
  for (int i = 0; i < 4; ++i)
    for (int j = 0; j < 4; ++j) {
      acc[i][j] = 0.0;
      accm[4 * i + j] = 0.0;
    }
  for (int64_t wd0 = wbeg; wd0 < wend; wd0 += kChunk) {
    {  // a chunk none of whose rows is kept (all sparse: done by the row-wise kernel) is not even loaded
      const int64_t wd = wd0 + (tid & (kChunk - 1));
      const bool any = wd < wend && keep[wd] != 0ull;
      if (!__syncthreads_or(any)) continue;
    }
    // Everything the chunk needs from global memory is fetched into registers first (addresses clamped instead of
    // skipped) and only then stored to LDS: a loop that loads and stores element by element pays one memory latency
    // per element, about twenty per chunk.
    {
      constexpr int kZ = kTile * kChunk / kThreads;  // mask words per thread and operand
      constexpr int kWr = kChunk * 64 / kThreads;    // row weights per thread
      constexpr int kWp = kChunk * 16 / kThreads;    // groups of four rows per thread
      static_assert(kThreads % kChunk == 0, "a thread stays in one word column of the chunk");
      uint64_t za[kZ], zb[kZ];
      float wr_[kWr], w4[kWp][4];
      const int cz = tid % kChunk;  // this thread's word of the chunk (the same for all its elements)
      const int64_t wdz = wd0 + cz < wend ? wd0 + cz : wend - 1;
      const uint64_t kp = keep[wdz];
#pragma unroll
      for (int u = 0; u < kZ; ++u) {
        const int r = (tid + u * kThreads) / kChunk;
        const int64_t ra = a0 + r < n ? a0 + r : n - 1, rb = b0 + r < n ? b0 + r : n - 1;
        za[u] = Zt[ra * KW + wdz];
        zb[u] = Zt[rb * KW + wdz];
      }
#pragma unroll
      for (int u = 0; u < kWr; ++u) {
        const int64_t i = wd0 * 64 + tid + u * kThreads;
        wr_[u] = w[i < k ? i : k - 1];
      }
#pragma unroll
      for (int u = 0; u < kWp; ++u)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const int64_t i = wd0 * 64 + 4 * (int64_t)(tid + u * kThreads) + j;
          w4[u][j] = w[i < k ? i : k - 1];
        }
#pragma unroll
      for (int u = 0; u < kZ; ++u) {
        const int idx = tid + u * kThreads, r = idx / kChunk, c = idx - r * kChunk;
        const bool in = wd0 + c < wend;
        As[r][c] = (a0 + r < n && in) ? (za[u] & kp) : 0ull;  // kept rows only
        Bs[r][c] = (b0 + r < n && in) ? zb[u] : 0ull;
      }
#pragma unroll
      for (int u = 0; u < kWr; ++u) {
        const int idx = tid + u * kThreads;
        wrow[idx] = wd0 * 64 + idx < k ? wr_[u] : 0.f;
      }
#pragma unroll
      for (int u = 0; u < kWp; ++u) {  // rows 4 idx .. 4 idx + 3 of the chunk
        const int idx = tid + u * kThreads;
        uint32_t pc[3][4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const int64_t i = wd0 * 64 + 4 * (int64_t)idx + j;
          float rest = i < k ? w4[u][j] : 0.f;
#pragma unroll
          for (int p = 0; p < 3; ++p) {
            pc[p][j] = bf16_bits_rn(rest);
            rest -= __uint_as_float(pc[p][j] << 16);  // exact: the piece shares the leading bits of `rest`
          }
        }
#pragma unroll
        for (int p = 0; p < 3; ++p) wpk[p][idx] = gram_u2_t{pc[p][0] | (pc[p][1] << 16), pc[p][2] | (pc[p][3] << 16)};
      }
    }
    if (tid < kChunk) {
      const int64_t wd = wd0 + tid;
      wus[tid] = wd < wend ? wu[wd] : 0.f;
      unis[tid] = wd < wend ? uni[wd] : 1;
    }
    __syncthreads();
    float f[4][4];
    for (int i = 0; i < 4; ++i)
      for (int j = 0; j < 4; ++j) f[i][j] = 0.f;
    gram_f16_t fm0, fm1;
#pragma unroll
    for (int i = 0; i < 16; ++i) { fm0[i] = 0.f; fm1[i] = 0.f; }
    for (int c = 0; c < kChunk; ++c) {
      if (unis[c] == 1) {
        uint64_t av[4], bv[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          av[i] = As[ty + 16 * i][c];
          bv[i] = Bs[tx + 16 * i][c];
        }
        const float wv = wus[c];
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int j = 0; j < 4; ++j) f[i][j] += wv * (float)__popcll(av[i] & bv[j]);
      } else if (unis[c] == 3) {
        // no kept row in this word
      } else if (unis[c] == 2) {
        // rows 16 kb + 8 half + j, j < 8: a byte of each column word per step (pre-shifted by 8 half)
        const uint64_t aw = As[wi + l32][c] >> (8 * half), bw = Bs[wj + l32][c] >> (8 * half);
        const gram_u4_t* w1 = (const gram_u4_t*)(wpk[0] + c * 16) + half;
        const gram_u4_t* w2 = (const gram_u4_t*)(wpk[1] + c * 16) + half;
        const gram_u4_t* w3 = (const gram_u4_t*)(wpk[2] + c * 16) + half;
#pragma unroll
        for (int kb = 0; kb < 4; ++kb) {
          const uint32_t x = (uint32_t)(aw >> (16 * kb)), y = (uint32_t)(bw >> (16 * kb));
          const gram_u2_t a0 = tabA[x & 15u], a1 = tabA[(x >> 4) & 15u], b0 = tabB[y & 15u], b1 = tabB[(y >> 4) & 15u];
          const gram_u4_t am = {a0.x, a0.y, a1.x, a1.y};
          const gram_b8_t bo = __builtin_bit_cast(gram_b8_t, gram_u4_t{b0.x, b0.y, b1.x, b1.y});
          const gram_b8_t p1 = __builtin_bit_cast(gram_b8_t, w1[2 * kb] & am);
          const gram_b8_t p2 = __builtin_bit_cast(gram_b8_t, w2[2 * kb] & am);
          const gram_b8_t p3 = __builtin_bit_cast(gram_b8_t, w3[2 * kb] & am);
          fm0 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(p1, bo, fm0, 0, 0, 0);
          fm1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(p2, bo, fm1, 0, 0, 0);
          fm1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(p3, bo, fm1, 0, 0, 0);
        }
      } else {
        uint64_t av[4], bv[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          av[i] = As[ty + 16 * i][c];
          bv[i] = Bs[tx + 16 * i][c];
        }
        const float* wr = wrow + c * 64;
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            uint64_t m = av[i] & bv[j];
            float sum = 0.f;
            while (m) {
              sum += wr[__ffsll((long long)m) - 1];
              m &= m - 1;
            }
            f[i][j] += sum;
          }
      }
    }
    for (int i = 0; i < 4; ++i)
      for (int j = 0; j < 4; ++j) acc[i][j] += (double)f[i][j];
#pragma unroll
    for (int i = 0; i < 16; ++i) accm[i] += (double)fm0[i] + (double)fm1[i];
  }
  // merge: the matrix-core quadrants pass through LDS into the popcount path's element order
  __syncthreads();
  double (*Ts)[kTile + 1] = (double (*)[kTile + 1])raw;
#pragma unroll
  for (int i = 0; i < 16; ++i) Ts[wi + 8 * (i / 4) + 4 * half + (i % 4)][wj + l32] = accm[i];
  __syncthreads();
  // slice 0 already holds the lower tiles of the sparse rows' part, if that had a launch of its own (else it is the last slice): all of a
  // thread's entries are fetched before the first store (one memory latency instead of sixteen; addresses clamped instead of skipped)
  double prev[4][4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int64_t a = a0 + ty + 16 * i, b = b0 + tx + 16 * j;
      prev[i][j] = rows_apart && blockIdx.z == 0 ? G[(a < n ? a : n - 1) * n + (b < n ? b : n - 1)] : 0.0;
    }
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int64_t a = a0 + ty + 16 * i, b = b0 + tx + 16 * j;
      const bool in = a < n && b < n;
      const double v = acc[i][j] + Ts[ty + 16 * i][tx + 16 * j] + prev[i][j];
      if (in) G[a * n + b] = v;
      if (part) Ts[ty + 16 * i][tx + 16 * j] = in ? v : 0.0;   // (this thread's own element)
    }
  if (!part) return;
  __syncthreads();
  gram_tile_sums(Ts, ta, tb, n, part);
}

// G = sum of the slices (into slice 0), and the tiles' sums: one workgroup per lower tile
__global__ __launch_bounds__(kThreads) void sum_slices_kernel(double* Gp, int64_t n, int slices, double* part) {
  const int ta = blockIdx.y, tb = blockIdx.x;
  if (tb > ta) return;
  __shared__ double T[kTile][kTile + 1];
  constexpr int kPer = kTile * kTile / kThreads;
  double v[kPer];
  for (int z = 0; z < slices; ++z) {   // (a slice's loads in flight together; addresses clamped)
    double g[kPer];
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
      const int idx = threadIdx.x + u * kThreads;
      const int64_t a = (int64_t)ta * kTile + (idx >> 6), b = (int64_t)tb * kTile + (idx & 63);
      g[u] = Gp[(size_t)z * n * n + (a < n ? a : n - 1) * n + (b < n ? b : n - 1)];
    }
#pragma unroll
    for (int u = 0; u < kPer; ++u) v[u] = z == 0 ? g[u] : v[u] + g[u];
  }
#pragma unroll
  for (int u = 0; u < kPer; ++u) {
    const int idx = threadIdx.x + u * kThreads;
    const int64_t a = (int64_t)ta * kTile + (idx >> 6), b = (int64_t)tb * kTile + (idx & 63);
    const bool in = a < n && b < n;
    if (in) Gp[a * n + b] = v[u];
    T[idx >> 6][idx & 63] = in ? v[u] : 0.0;
  }
  __syncthreads();
  gram_tile_sums(T, ta, tb, n, part);
}

// m[a] = mean of row a of G
__global__ void row_means_kernel(const double* part, int64_t n, int tiles, double* m) {
  const int64_t a = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (a >= n) return;
  double s = 0.0;
#pragma unroll 8
  for (int t = 0; t < tiles; ++t) s += part[(int64_t)t * n + a];
  m[a] = s / (double)n;
}

// single block: stats[0] = mu (grand mean of G), stats[1] = trace(G); clears the factorisation's flag
__global__ __launch_bounds__(kThreads) void stats_kernel(const double* G, const double* m, int64_t n, double* stats, int* flag) {
  __shared__ double sh[2][kThreads];
  double a = 0, b = 0;
  for (int64_t i = threadIdx.x; i < n; i += kThreads) {
    a += m[i];
    b += G[i * n + i];
  }
  sh[0][threadIdx.x] = a;
  sh[1][threadIdx.x] = b;
  __syncthreads();
  if (threadIdx.x == 0) {
    double x = 0, yv = 0;
    for (int i = 0; i < kThreads; ++i) {
      x += sh[0][i];
      yv += sh[1][i];
    }
    stats[0] = x / (double)n;
    stats[1] = yv;
    *flag = 0;
  }
}

// The system lives in one (n+1) x ld array M: rows 0..n-1 = A = P G P + gamma 11^T / n (lower triangle
// is what the factorisation reads), row n = the right-hand side c - mean(c). Factorising with row n
// carried along as an ordinary sub-diagonal row leaves L^-1 rhs in it (the forward solve comes for free).
// gamma = trace(PGP)/(n-1) keeps the added direction at the scale of the other eigenvalues.
// pivot_floor: the smallest pivot the factorisation accepts, relative to the mean diagonal entry of A: a pivot
// that exact arithmetic would make zero (a direction the sampled rows do not determine) comes out of fp64
// as about n * 2^-52 times the scale, with either sign; 256 n 2^-52 sits well above that and far below the
// pivots of a determined system.
// Lower tiles only, one workgroup each; the first 64 columns also go to P (row r at P[64 r ..]), the panel of the first fused step.
__global__ __launch_bounds__(kThreads) void build_matrix_kernel(const double* G, const double* m, const double* stats, int64_t n, int64_t ld,
                                                                double* M, double* P, double* pivot_floor) {
  const int ta = blockIdx.y, tb = blockIdx.x;
  if (tb > ta) return;
  const double mu = stats[0];
  const double tr = stats[1] - (double)n * mu;
  double gamma = tr / (double)(n > 1 ? n - 1 : 1);
  if (!(gamma > 0.0)) gamma = 1.0;
  const int tid = threadIdx.x;
  if (ta == 0 && tid == 0) *pivot_floor = 256.0 * (double)n * 0x1p-52 * ((tr > 0.0 ? tr : 0.0) + gamma) / (double)n;
  constexpr int kPer = kTile * kTile / kThreads;
  const int64_t b = (int64_t)tb * kTile + (tid & 63), bc = b < n ? b : n - 1;
  const double mb = m[bc];
  double g[kPer], ma[kPer];
#pragma unroll
  for (int u = 0; u < kPer; ++u) {
    const int64_t a = (int64_t)ta * kTile + (tid >> 6) + u * (kThreads / 64), ac = a < n ? a : n - 1;
    g[u] = G[ac * n + bc];
    ma[u] = m[ac];
  }
#pragma unroll
  for (int u = 0; u < kPer; ++u) {
    const int64_t a = (int64_t)ta * kTile + (tid >> 6) + u * (kThreads / 64);
    if (a >= n || b >= n) continue;
    const double v = g[u] - ma[u] - mb + mu + gamma / (double)n;
    M[a * ld + b] = v;
    if (tb == 0) P[a * kTile + b] = v;
  }
}

// row n of M (and of P, its first 64 columns) = c - mean(c); single block
__global__ __launch_bounds__(kThreads) void build_rhs_kernel(const double* c, int64_t n, int64_t ld, double* M, double* P) {
  __shared__ double sh[kThreads];
  double a = 0;
  for (int64_t i = threadIdx.x; i < n; i += kThreads) a += c[i];
  sh[threadIdx.x] = a;
  __syncthreads();
  if (threadIdx.x == 0) {
    double x = 0;
    for (int i = 0; i < kThreads; ++i) x += sh[i];
    sh[0] = x / (double)n;
  }
  __syncthreads();
  const double mean = sh[0];
  for (int64_t i = threadIdx.x; i < n; i += kThreads) {
    M[n * ld + i] = c[i] - mean;
    if (i < kTile) P[n * kTile + i] = c[i] - mean;
  }
}

// ---------------- blocked Cholesky (lower, in place, fp64) ----------------
constexpr int NB = 64;
constexpr int64_t kSuperCols = 256;  // columns of a super-panel (large trailing matrices)

// 1/sqrt(p) for 1e-30 < p < 1e30: single-precision seed, two Newton steps r += r (1/2 - (p/2) r^2) in double (a
// short dependent chain; the library routine costs several times more per step of a sequential loop)
__device__ __forceinline__ double fast_rsqrt(double p) {
  double r = (double)__frsqrt_rn((float)p);  // relative error about 1e-7
  const double hp = 0.5 * p;
  r = fma(r, fma(-hp * r, r, 0.5), r);        // -> 1e-14
  r = fma(r, fma(-hp * r, r, 0.5), r);        // -> below one ulp
  return r;
}

typedef double double4_t __attribute__((ext_vector_type(4)));

// acc (+)= A[64 x 64] * B[64 x 64]^T for 64x64 tiles held in LDS with row pitch NB+1, on the fp64
// matrix cores. Each of the four waves owns a 32x32 quadrant = 2x2 tiles of v_mfma_f64_16x16x4f64:
// lane l supplies A[i = l%16][k = l/16] and B^T[k = l/16][j = l%16] = B[j][k]; its four results are
// D[4*r + l/16][l%16], r = 0..3.
__device__ __forceinline__ void tile_nt_mfma(const double (*A)[NB + 1], const double (*B)[NB + 1], double4_t (&acc)[2][2]) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int wi = (wave >> 1) * 32, wj = (wave & 1) * 32;
  const int l16 = lane & 15, lk = lane >> 4;
  const double* pa0 = &A[wi + l16][lk];
  const double* pa1 = &A[wi + 16 + l16][lk];
  const double* pb0 = &B[wj + l16][lk];
  const double* pb1 = &B[wj + 16 + l16][lk];
  // the operands of the next step are read from LDS before this step's products are issued
  double a0 = pa0[0], a1 = pa1[0], b0 = pb0[0], b1 = pb1[0];
#pragma unroll
  for (int k0 = 0; k0 < NB; k0 += 4) {
    double na0 = 0.0, na1 = 0.0, nb0 = 0.0, nb1 = 0.0;
    if (k0 + 4 < NB) {
      na0 = pa0[k0 + 4];
      na1 = pa1[k0 + 4];
      nb0 = pb0[k0 + 4];
      nb1 = pb1[k0 + 4];
    }
    acc[0][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(a0, b0, acc[0][0], 0, 0, 0);
    acc[0][1] = __builtin_amdgcn_mfma_f64_16x16x4f64(a0, b1, acc[0][1], 0, 0, 0);
    acc[1][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(a1, b0, acc[1][0], 0, 0, 0);
    acc[1][1] = __builtin_amdgcn_mfma_f64_16x16x4f64(a1, b1, acc[1][1], 0, 0, 0);
    a0 = na0;
    a1 = na1;
    b0 = nb0;
    b1 = nb1;
  }
}

// acc[j] = A[64 x 64] * L[64 x 64]^T for a lower triangular L (both in LDS), subtile (wave, j) of 16 x 16: column block j takes
// the k up to its own end only, and a wave owns a row of subtiles, so that the waves have the same 40 of 64 products.
__device__ __forceinline__ void tile_nt_lower_mfma(const double (*A)[NB + 1], const double (*L)[NB + 1], double4_t (&acc)[4]) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int l16 = lane & 15, lk = lane >> 4;
  const double* pa = &A[16 * wave + l16][lk];
  const double* pl = &L[l16][lk];
#pragma unroll
  for (int k0 = 0; k0 < NB; k0 += 4) {
    const double av = pa[k0];
#pragma unroll
    for (int j = 0; j < 4; ++j)
      if (16 * j + 15 >= k0) acc[j] = __builtin_amdgcn_mfma_f64_16x16x4f64(av, pl[16 * j * (NB + 1) + k0], acc[j], 0, 0, 0);
  }
}

// A 64 x 64 tile from global memory into LDS (row pitch NB+1) in two halves, so that a kernel can have the loads of
// all its tiles in flight before the first LDS store: written as one loop that loads and stores element by element
// (the bounds checks make every load a branch of its own), each of a thread's 16 elements costs a memory latency.
// Element (r, c) is src[(row0 + r) * stride + col0 + c], valid for row0 + r < row_limit and c < ncols, zero otherwise;
// out-of-range elements are read from a clamped address. row_limit and ncols are at least 1.
struct TileRegs {
  double v[kTile * NB / kThreads];
};
__device__ __forceinline__ void tile_fetch(TileRegs& t, const double* src, int64_t stride, int64_t row0, int64_t row_limit,
                                           int64_t col0, int ncols) {
#pragma unroll
  for (int u = 0; u < kTile * NB / kThreads; ++u) {
    const int idx = threadIdx.x + u * kThreads, r = idx >> 6, c = idx & 63;
    const int64_t rr = row0 + r < row_limit ? row0 + r : row_limit - 1;
    t.v[u] = src[rr * stride + col0 + (c < ncols ? c : ncols - 1)];
  }
}
__device__ __forceinline__ void tile_put(double (*T)[NB + 1], const TileRegs& t, int64_t row0, int64_t row_limit, int ncols) {
#pragma unroll
  for (int u = 0; u < kTile * NB / kThreads; ++u) {
    const int idx = threadIdx.x + u * kThreads, r = idx >> 6, c = idx & 63;
    T[r][c] = (row0 + r < row_limit && c < ncols) ? t.v[u] : 0.0;
  }
}

// M[r][c] -= acc over a wave's NI x NJ matrix-core tiles at (i0 + wi, c0 + wj), lower triangle and in-bounds
// entries only; P, if not null, also receives the new values of the tile's column block (row r at P[r * 64 ..]).
// All loads of a tile row are issued before the first store: written as `M[..] -= acc` under its bounds check,
// every entry becomes a load, a wait and a store of its own, one memory latency each. The loads are made safe
// by clamping the address instead of skipping them.
template <int NI, int NJ>
__device__ __forceinline__ void tile_sub_store(double* M, int64_t ld, int64_t rows_total, int64_t n, int64_t i0, int64_t c0,
                                               int wi, int wj, const double4_t (&acc)[NI][NJ], double* P) {
  const int lane = threadIdx.x & 63, l16 = lane & 15, lk = lane >> 4;
#pragma unroll
  for (int i = 0; i < NI; ++i) {
    double cur[NJ][4];
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
      for (int r4 = 0; r4 < 4; ++r4) {
        const int64_t r = i0 + wi + 16 * i + 4 * r4 + lk, c = c0 + wj + 16 * j + l16;
        const int64_t rs = r < rows_total ? r : rows_total - 1, cs = c < n ? c : n - 1;
        cur[j][r4] = M[rs * ld + cs];
      }
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
      for (int r4 = 0; r4 < 4; ++r4) {
        const int64_t r = i0 + wi + 16 * i + 4 * r4 + lk, c = c0 + wj + 16 * j + l16;
        if (r < rows_total && c < n && c <= r) {
          const double v = cur[j][r4] - acc[i][j][r4];
          M[r * ld + c] = v;
          if (P) P[r * NB + (c - c0)] = v;
        }
      }
  }
}

// value of `v` in lane `src` (a compile-time constant after unrolling) for the whole wave, through two scalar registers
__device__ __forceinline__ double wave_bcast(double v, int src) {
  const int lo = __builtin_amdgcn_readlane(__double2loint(v), src);
  const int hi = __builtin_amdgcn_readlane(__double2hiint(v), src);
  return __hiloint2double(hi, lo);
}

constexpr int kSub = 16;  // sub-block of the diagonal block: one matrix-core tile

// One wave eliminates the 16 x 16 block D = S[o.., o..] and, alongside, the identity: what it leaves is the factor
// and its inverse up to the scaling by 1/sqrt(pivot), which the other waves apply where they use them,
//   L[i][k] = S[o+i][o+k] r_k,   Linv[k][c] = XT[c][k] r_k,   r_k = 1/sqrt(d_k),   d_k = S[o+k][o+k].
// A lone wave issues one instruction every few cycles whatever the instruction is, so the loop holds nothing that
// can be done elsewhere: no square root, no pivot check, no stores to global memory.
// Lane l < 16 keeps row l of D (columns up to l matter), lane 16 + l keeps column l of the inverse (the upper half
// of the wave repeats the lower). With d the pivot of column j and p = 1/d, L[i][j] L[k][j] = S[i][j] S[k][j] p:
// lane i subtracts (S[i][j] p) col[k] from its entry of column k > j, where col[] is column j as updated so far;
// the same column moves the forward substitution L X = I on, X[k][c] -= col[k] (X[j][c] p), so one multiply-add per k
// serves both halves. What bounds the loop is the chain from pivot to pivot: reciprocal, p, the next column's entry.
// The two values it needs, the pivot and col[j + 1], reach all lanes through scalar registers; the rest of the column
// travels through LDS (two buffers; reads of one address by all lanes are a broadcast), which takes longer than a step, so
// the updates with it are a step late: they fill the wait for the next reciprocal. (With every update waiting for its
// column: 2,500 cycles a block; now 2,360.) I16 is a 16 x 16 identity.
__device__ __forceinline__ void eliminate_sub_block(double (*S)[NB + 1], int o, double (*XT)[kSub + 1],
                                                    const double (*I16)[kSub + 1], double* col) {
  const int lane = threadIdx.x & 63, l = lane & 15, slot = lane & 31;
  const bool inv = (lane & 16) != 0;
  double* mine = inv ? &XT[l][0] : &S[o + l][o];
  const double* init = inv ? &I16[l][0] : mine;
  double v[kSub];
#pragma unroll
  for (int k = 0; k < kSub; ++k) v[k] = init[k];
  // The column's store and loads are written as instructions: the loads of a column have to be issued right
  // behind its store, so that they return under the step that follows, and the compiler's scheduler
  // puts them next to their first use instead. LDS answers a wave in order, so the compiler's own counting of its
  // LDS accesses stays on the safe side. Between a load and the wait below its destination registers are in flight,
  // which the compiler does not know: tests/test_isa_lds_reads.py checks the generated code for any use in between.
  typedef double pair_t __attribute__((ext_vector_type(2)));
  const unsigned col_lds = (unsigned)(size_t)(__attribute__((address_space(3))) double*)col;  // byte address in LDS
  const unsigned slot_lds = col_lds + 8u * slot;
  pair_t q[kSub / 2];
  asm volatile("ds_write_b64 %0, %1" ::"v"(slot_lds), "v"(v[0]) : "memory");
#pragma unroll
  for (int h = 0; h < kSub / 2; ++h) asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(q[h]) : "v"(col_lds), "n"(16 * h));
  // The order below is the order of issue (sched_barrier): the late updates go where the chain waits.
#define DS_HERE __builtin_amdgcn_sched_barrier(0)
  double c[kSub];      // column j - 1, whose updates of the columns from j + 1 on are still to be made, and ...
  double late = 0.0;   // ... its p
#pragma unroll
  for (int j = 0; j + 1 < kSub; ++j) {
    int at = j + 1;    // next late update
    auto update = [&](int count) {
      if (j > 0) {
#pragma unroll
        for (int i = 0; i < count; ++i)
          if (at < kSub) {
            v[at] = fma(-late, c[at], v[at]);
            ++at;
          }
      }
      DS_HERE;
    };
    const double d = wave_bcast(v[j], j);
    double x = __builtin_amdgcn_rcp(d);   // 1/d for 1e-30 < d < 1e30: seed (about 24 bits), then x (1 + e + e^2) with e = 1 - d x
    DS_HERE;
    const double next = wave_bcast(v[j], j + 1);
    update(3);
    double e = fma(-d, x, 1.0);
    update(1);
    e = fma(e, e, e);
    update(1);
    x = fma(x, e, x);
    update(1);
    const double p = v[j] * x;
    update(1);
    v[j + 1] = fma(-p, next, v[j + 1]);
    update(kSub);
    if (j + 2 < kSub) {
      // column j is here (q[h] for h below (j + 2) / 2 were not loaded and pass through unchanged)
      asm volatile("s_waitcnt lgkmcnt(0)"
                   : "+v"(q[0]), "+v"(q[1]), "+v"(q[2]), "+v"(q[3]), "+v"(q[4]), "+v"(q[5]), "+v"(q[6]), "+v"(q[7]));
#pragma unroll
      for (int h = (j + 2) / 2; h < kSub / 2; ++h) {
        c[2 * h] = q[h].x;
        c[2 * h + 1] = q[h].y;
      }
      late = p;
    }
    if (j + 3 < kSub) {  // column j + 1 is complete: send it on its way
      asm volatile("ds_write_b64 %0, %1 offset:%2" ::"v"(slot_lds), "v"(v[j + 1]), "n"(((j + 1) & 1) * 256) : "memory");
#pragma unroll
      for (int h = (j + 2) / 2; h < kSub / 2; ++h)
        asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(q[h]) : "v"(col_lds), "n"(((j + 1) & 1) * 256 + 16 * h));
    }
    DS_HERE;
  }
#undef DS_HERE
  asm volatile("" ::: "memory");
#pragma unroll
  for (int k = 0; k < kSub; ++k) mine[k] = v[k];
}

// sum_k A(m, k) B(k, n) over a 16 x 16 x 16 product on the fp64 matrix cores, added to acc: A(m, k) = Ap[m * ars + k * acs]
// and B(k, n) = Bp[k * brs + n * bcs]; lane l holds D[4 r + l / 16][l % 16], r = 0..3.
__device__ __forceinline__ double4_t sub_block_mma(const double* Ap, int ars, int acs, const double* Bp, int brs, int bcs,
                                                   double4_t acc) {
  const int lane = threadIdx.x & 63, l16 = lane & 15, lk = lane >> 4;
#pragma unroll
  for (int kk = 0; kk < kSub; kk += 4) {
    const double av = Ap[l16 * ars + (kk + lk) * acs];
    const double bv = Bp[(kk + lk) * brs + l16 * bcs];
    acc = __builtin_amdgcn_mfma_f64_16x16x4f64(av, bv, acc, 0, 0, 0);
  }
  return acc;
}
__device__ __forceinline__ double4_t sub_block_load(const double (*T)[NB + 1], int r0, int c0) {
  const int lane = threadIdx.x & 63, l16 = lane & 15, lk = lane >> 4;
  double4_t v;
#pragma unroll
  for (int r = 0; r < 4; ++r) v[r] = T[r0 + 4 * r + lk][c0 + l16];
  return v;
}
__device__ __forceinline__ void sub_block_store(double (*T)[NB + 1], int r0, int c0, double4_t v) {
  const int lane = threadIdx.x & 63, l16 = lane & 15, lk = lane >> 4;
#pragma unroll
  for (int r = 0; r < 4; ++r) T[r0 + 4 * r + lk][c0 + l16] = v[r];
}

// Factor the nb x nb diagonal block at j0 (lower factor L, in place) and invert the factor: Linv (NB x NB,
// identity-padded) goes to linv_out. One workgroup of four waves; the block S and the inverse Y live in the two
// LDS tiles the caller hands over. The block is taken as 4 x 4 sub-blocks of 16, left-looking; for block column b
//   A. S_ib -= sum_{k<b} L_ik L_bk^T for i >= b, and T_bj = sum_{j<=k<b} L_bk Y_kj for j < b   (4 tasks, one a wave),
//   B. one wave eliminates S_bb and the identity beside it (the only sequential part: 16 columns),
//   C. L_ib = S_ib Linv_bb^T for i > b, Y_bj = -Linv_bb T_bj for j < b, and the scaled L_bb and Y_bb = Linv_bb
//      (4 tasks, one a wave; this is where the square roots are taken and the pivots are checked),
// where Y follows the forward substitution L Y = I block row by block row. The terms of A that do not wait for block column
// b - 1 are formed while the wave of B eliminates (by the other three, in registers), so that A itself is one product a wave.
// (A took 910, 1,350 and 1,820 cycles for b = 1..3, now 820 each; the whole block 24,600, now 22,900.) A and C are 16 x 16 x 16
// products on the fp64 matrix cores; results go to global memory as they appear. A pivot that is not positive (or not a number, or
// below the relative floor stored next to the flag, or above 1e30) raises the flag; nothing is repaired, the caller discards a flagged factorisation.
// `pend`: optional 64 x 64 tile (LDS, pitch NB+1; may be the tile Y) holding the rows of this block in the panel
// just finished; its outer product is the one trailing update the block has not received yet and is subtracted
// first.
// The diagonal block's ten lower 16 x 16 subtiles (the others are not looked at) are dealt to the four waves, subtile t to
// wave t % 4: DiagRegs holds a wave's entries, matrix-core layout, identity beyond row or column nb. A caller with other
// work to do first loads them early, so that they arrive under that work.
struct DiagRegs {
  double4_t v[3];
};
constexpr int kDiagTiles = 10;
__device__ __forceinline__ void diag_subtile(int t, int& r0, int& c0) {
  const int i = t >= 6 ? 3 : t >= 3 ? 2 : t >= 1 ? 1 : 0;
  r0 = kSub * i;
  c0 = kSub * (t - i * (i + 1) / 2);
}
__device__ __forceinline__ void load_diag_block(const double* M, int64_t ld, int64_t j0, int nb, DiagRegs& mt) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
  for (int u = 0; u < 3; ++u) {
    const int t = wave + 4 * u;
    if (t >= kDiagTiles) break;
    int r0, c0;
    diag_subtile(t, r0, c0);
#pragma unroll
    for (int r4 = 0; r4 < 4; ++r4) {
      const int r = r0 + 4 * r4 + (lane >> 4), c = c0 + (lane & 15);
      const bool in = r < nb && c < nb;
      const double m = M[(j0 + (in ? r : 0)) * ld + j0 + (in ? c : 0)];
      mt.v[u][r4] = in ? m : (r == c ? 1.0 : 0.0);
    }
  }
}

__device__ __forceinline__ void chol_diag_body(double* M, int64_t ld, int64_t j0, int nb, double* linv_out, int* flag,
                                               const double (*pend)[NB + 1], double (*S)[NB + 1], double (*Y)[NB + 1],
                                               const DiagRegs& mt) {
  __shared__ double XT[kSub][kSub + 1];
  __shared__ double I16[kSub][kSub + 1];
  __shared__ __align__(16) double col[2 * 32];  // two buffers for the column in flight
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int l16 = lane & 15, lk = lane >> 4;
  {
    double4_t v[3];
#pragma unroll
    for (int u = 0; u < 3; ++u) {
      v[u] = mt.v[u];
      const int t = wave + 4 * u;
      if (pend && t < kDiagTiles) {   // rows past nb of the tile are zero, so the identity padding stays as it is
        int r0, c0;
        diag_subtile(t, r0, c0);
        double4_t acc = double4_t{0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int k0 = 0; k0 < NB; k0 += 4)
          acc = __builtin_amdgcn_mfma_f64_16x16x4f64(pend[r0 + l16][k0 + lk], pend[c0 + l16][k0 + lk], acc, 0, 0, 0);
        v[u] -= acc;
      }
    }
    if (pend) __syncthreads();  // every wave has read `pend` before Y (possibly the same tile) is written
#pragma unroll
    for (int u = 0; u < 3; ++u) {
      const int t = wave + 4 * u;
      if (t < kDiagTiles) {
        int r0, c0;
        diag_subtile(t, r0, c0);
        sub_block_store(S, r0, c0, v[u]);
      }
    }
    I16[tid >> 4][tid & 15] = (tid >> 4) == (tid & 15) ? 1.0 : 0.0;
    // the sub-blocks of Linv above the diagonal are zero; the others are written as they are computed
    for (int idx = tid; idx < NB * NB; idx += kThreads)
      if (((idx & 63) >> 4) > (idx >> 10)) linv_out[idx] = 0.0;
  }
  __syncthreads();
  constexpr int nsb = NB / kSub;
  const double4_t zero = double4_t{0.0, 0.0, 0.0, 0.0};
  double4_t early = zero;   // waves 1..3: the terms k < b - 1 of this wave's task in A
  for (int b = 0; b < nsb; ++b) {
    const int o = b * kSub;
    // tasks of A: wave 0 takes T_b,b-1 (one term only), waves 1 .. the column's S_ib, then the row's other T_bj
    if (b > 0) {  // A
      const int kb = (b - 1) * kSub;
      if (wave > 0 && wave - 1 < nsb - b) {
        const int i = b + wave - 1;  // (m, n): sum_kk S[16 i + m][16 k + kk] S[16 b + n][16 k + kk]
        const double4_t acc = sub_block_mma(&S[i * kSub][kb], NB + 1, 1, &S[o][kb], 1, NB + 1, early);
        sub_block_store(S, i * kSub, o, sub_block_load(S, i * kSub, o) - acc);
      } else {
        const int j = wave > 0 ? wave - 1 - (nsb - b) : b - 1;  // (m, n): sum_kk S[o + m][16 k + kk] Y[16 k + kk][16 j + n]
        sub_block_store(Y, o, j * kSub, sub_block_mma(&S[o][kb], NB + 1, 1, &Y[kb][j * kSub], NB + 1, 1, early));
      }
      __syncthreads();
    }
    if (wave == 0) {
      eliminate_sub_block(S, o, XT, I16, col);  // B
    } else if (b + 1 < nsb) {   // the next A's terms k < b
      const int b1 = b + 1, i = b1 + wave - 1, j = wave - 1 - (nsb - b1);
      early = zero;
      if (wave - 1 < nsb - b1) {
        for (int k = 0; k < b; ++k)
          early = sub_block_mma(&S[i * kSub][k * kSub], NB + 1, 1, &S[b1 * kSub][k * kSub], 1, NB + 1, early);
      } else {
        for (int k = j; k < b; ++k)
          early = sub_block_mma(&S[b1 * kSub][k * kSub], NB + 1, 1, &Y[k * kSub][j * kSub], NB + 1, 1, early);
      }
    }
    __syncthreads();
    {  // C
      const double d = S[o + l16][o + l16];
      const double rl = fast_rsqrt(d);  // r of this lane's column; r of row m is lane m's
      if (wave < nsb - 1 - b) {
        const int i = b + 1 + wave;  // L_ib(m, n) = r_n sum_k S_ib(m, k) XT(k, n)
        const double4_t xv = sub_block_mma(&S[i * kSub][o], NB + 1, 1, &XT[0][0], kSub + 1, 1, zero) * rl;
        sub_block_store(S, i * kSub, o, xv);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int row = i * kSub + 4 * r + lk;
          if (row < nb) M[(j0 + row) * ld + j0 + o + l16] = xv[r];
        }
      } else if (wave < nsb - 1) {
        const int j = wave - (nsb - 1 - b);  // Y_bj(m, n) = -r_m sum_k XT(k, m) T(k, n)
        const double4_t tv = sub_block_mma(&XT[0][0], 1, kSub + 1, &Y[o][j * kSub], NB + 1, 1, zero);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const double yv = -tv[r] * __shfl(rl, 4 * r + lk);
          Y[o + 4 * r + lk][j * kSub + l16] = yv;
          linv_out[(o + 4 * r + lk) * NB + j * kSub + l16] = yv;
        }
      } else {
        if (!(d > *(const double*)(flag + 2) && d < 1e30)) atomicExch(flag, 1);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int m = 4 * r + lk;  // row of the sub-block, column l16
          const double x = XT[l16][m] * __shfl(rl, m);
          Y[o + m][o + l16] = x;
          linv_out[(o + m) * NB + o + l16] = x;
          if (l16 <= m && o + m < nb) M[(j0 + o + m) * ld + j0 + o + l16] = S[o + m][o + l16] * rl;
        }
      }
    }
    __syncthreads();
  }
}

// a >= b of the p-th pair
__device__ __forceinline__ void small_pair(int p, int& a, int& b) {
  a = (int)((sqrtf(8.f * (float)p + 1.f) - 1.f) * 0.5f);
  while (a * (a + 1) / 2 > p) --a;
  while ((a + 1) * (a + 2) / 2 <= p) ++a;
  b = p - a * (a + 1) / 2;
}

// The system matrix of a game of at most 64 players from the parts of its counts (as sum_slices, row_means, stats and build_matrix form
// it), one workgroup; S, mean: its LDS. The elimination follows in the same kernel, a launch fewer.
__device__ __forceinline__ void small_system(const double* part, int parts, int n, int* flag, double (&S)[kTile][NB + 1],
                                             double (&mean)[NB], DiagRegs& mt) {
  constexpr int kAhead = 16;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, pairs = n * (n + 1) / 2;
  for (int p = tid; p < pairs; p += kThreads) {
    double sum = 0.0;
    for (int i0 = 0; i0 < parts; i0 += kAhead) {   // (all of a step's loads in flight; past the end the last part is read again)
      double v[kAhead];
#pragma unroll
      for (int u = 0; u < kAhead; ++u) v[u] = part[(size_t)(i0 + u < parts ? i0 + u : parts - 1) * pairs + p];
#pragma unroll
      for (int u = 0; u < kAhead; ++u) sum += i0 + u < parts ? v[u] : 0.0;
    }
    int a, b;
    small_pair(p, a, b);
    S[a][b] = sum;
    S[b][a] = sum;
  }
  __syncthreads();
  if (tid < n) {
    double sum = 0.0;
    for (int b = 0; b < n; ++b) sum += S[tid][b];
    mean[tid] = sum / (double)n;
  }
  __syncthreads();
  double mu = 0.0, tr = 0.0;
  for (int i = 0; i < n; ++i) {
    mu += mean[i];
    tr += S[i][i];
  }
  mu /= (double)n;
  tr -= (double)n * mu;
  double gamma = tr / (double)(n > 1 ? n - 1 : 1);
  if (!(gamma > 0.0)) gamma = 1.0;
  if (tid == 0) {
    *flag = 0;
    *(double*)(flag + 2) = 256.0 * (double)n * 0x1p-52 * ((tr > 0.0 ? tr : 0.0) + gamma) / (double)n;   // see build_matrix_kernel
    __threadfence_block();
  }
#pragma unroll
  for (int u = 0; u < 3; ++u) {
    const int t = wave + 4 * u;
    if (t >= kDiagTiles) break;
    int r0, c0;
    diag_subtile(t, r0, c0);
#pragma unroll
    for (int r4 = 0; r4 < 4; ++r4) {
      const int r = r0 + 4 * r4 + (lane >> 4), c = c0 + (lane & 15);
      mt.v[u][r4] = r < n && c < n ? S[r][c] - mean[r] - mean[c] + mu + gamma / (double)n : (r == c ? 1.0 : 0.0);
    }
  }
  __syncthreads();   // every wave has read the sums before the block's tile is written
}

// part (or nullptr: the block lies in M): the counts of a small game
__global__ __launch_bounds__(kThreads) void chol_diag_kernel(double* M, int64_t ld, int64_t j0, int nb, double* linv_out,
                                                             int* flag, const double* part, int parts) {
  __shared__ double S[kTile][NB + 1];
  __shared__ double Y[kTile][NB + 1];
  __shared__ double mean[NB];
  DiagRegs mt;
  if (part) small_system(part, parts, nb, flag, S, mean, mt);
  else load_diag_block(M, ld, j0, nb, mt);
  chol_diag_body(M, ld, j0, nb, linv_out, flag, nullptr, S, Y, mt);
}

// rows below the diagonal block: X = A21 L11^-T = A21 Linv^T, a 64x64 product per workgroup
__global__ __launch_bounds__(kThreads) void chol_panel_kernel(double* M, int64_t ld, int64_t rows_total, int64_t j0,
                                                              int nb, const double* linv) {
  __shared__ double As[kTile][NB + 1];
  __shared__ double Ls[NB][NB + 1];
  const int64_t i0 = j0 + nb + (int64_t)blockIdx.x * kTile;
  {
    TileRegs ta, tl;
    tile_fetch(ta, M, ld, i0, rows_total, j0, nb);
    tile_fetch(tl, linv, NB, 0, NB, 0, NB);
    tile_put(As, ta, i0, rows_total, nb);
    tile_put(Ls, tl, 0, NB, NB);
  }
  __syncthreads();
  double4_t acc[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) acc[j] = double4_t{0.0, 0.0, 0.0, 0.0};
  tile_nt_lower_mfma(As, Ls, acc);
  {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int r4 = 0; r4 < 4; ++r4) {
        const int64_t r = i0 + 16 * wave + 4 * r4 + (lane >> 4);
        const int c = 16 * j + (lane & 15);
        if (r < rows_total && c < nb) M[r * ld + j0 + c] = acc[j][r4];
      }
  }
}

// trailing update A22 -= L21 L21^T on the lower tiles (rows up to rows_total, columns below n).
// The workgroup of the first diagonal tile does more: that tile is the next diagonal block, so it applies the
// tile's update in registers and factorises it straight away (and stores its inverse), while the other
// workgroups are still updating the rest of the trailing matrix. The next step then starts at its panel.
// (FUSE = false: plain update of every tile; used while the trailing matrix is large, where the registers of
// the factorisation would halve the number of resident update workgroups for no gain.)
template <bool FUSE>
__global__ __launch_bounds__(kThreads) void chol_update_kernel(double* M, int64_t ld, int64_t rows_total, int64_t n,
                                                               int64_t j0, int nb, double* linv_next, int* flag) {
  const int ti = blockIdx.y, tj = blockIdx.x;
  if (tj > ti) return;
  __shared__ double Li[kTile][NB + 1];
  __shared__ double Lj[kTile][NB + 1];
  const int64_t base = j0 + nb;
  const int64_t i0 = base + (int64_t)ti * kTile, c0 = base + (int64_t)tj * kTile;
  DiagRegs mt;  // the next diagonal block (its workgroup only), on its way with the operands
  if (FUSE && ti == 0 && tj == 0) load_diag_block(M, ld, base, (int)(n - base < NB ? n - base : NB), mt);
  {
    TileRegs ta, tb;
    tile_fetch(ta, M, ld, i0, rows_total, j0, nb);
    tile_fetch(tb, M, ld, c0, n, j0, nb);
    tile_put(Li, ta, i0, rows_total, nb);
    tile_put(Lj, tb, c0, n, nb);
  }
  __syncthreads();
  if (FUSE && ti == 0 && tj == 0) {  // Lj holds the rows of the next diagonal block in this panel (zero past column n)
    // a short last block shares its tile with the right-hand-side row, which still needs this update
    if (rows_total > n && n - base < NB && (int64_t)threadIdx.x < n - base) {
      const int rr = (int)(n - base), c = threadIdx.x;
      double sum = 0.0;
      for (int k = 0; k < NB; ++k) sum += Li[rr][k] * Lj[c][k];
      M[n * ld + base + c] -= sum;
    }
    __syncthreads();  // the row above has read Li, which becomes the block's tile
    chol_diag_body(M, ld, base, (int)(n - base < NB ? n - base : NB), linv_next, flag, Lj, Li, Lj, mt);
    return;
  }
  double4_t acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) acc[i][j] = double4_t{0.0, 0.0, 0.0, 0.0};
  tile_nt_mfma(Li, Lj, acc);
  {
    const int wave = threadIdx.x >> 6;
    tile_sub_store<2, 2>(M, ld, rows_total, n, i0, c0, (wave >> 1) * 32, (wave & 1) * 32, acc, nullptr);
  }
}

// One launch per 64-column step: panel solve, update of the block columns ahead (all of them while the trailing matrix is small, those of
// the super-panel, gridDim.x of them, before) and factorisation of the next diagonal block together. Every workgroup (ti, tj), tj <= ti, first
// solves its own two 64-row pieces of the panel, X = A Linv^T, instead of waiting for a launch that does so
// (twice the arithmetic of the update itself, on workgroups that would otherwise be idle), then updates its tile;
// the workgroup of the first diagonal tile factorises that tile instead, as in chol_update_kernel<true>.
// The rows of the panel as the step before left them come from Pcur (row r of the matrix at Pcur[r * 64 ..]), not
// from M: the workgroups of tile column 0 store the solved panel to M while others may still be reading, and they
// store their updated tile, the next step's panel, to Pnext as well.
__global__ __launch_bounds__(kThreads) void chol_step_kernel(double* M, int64_t ld, int64_t rows_total, int64_t n, int64_t j0,
                                                             const double* linv, double* linv_next, int* flag,
                                                             const double* Pcur, double* Pnext) {
  const int ti = blockIdx.y, tj = blockIdx.x;
  if (tj > ti) return;
  __shared__ double Li[kTile][NB + 1];
  __shared__ double Lj[kTile][NB + 1];
  __shared__ double Ls[NB][NB + 1];
  const int64_t base = j0 + NB;
  const int64_t i0 = base + (int64_t)ti * kTile, c0 = base + (int64_t)tj * kTile;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int wi = (wave >> 1) * 32, wj = (wave & 1) * 32;
  DiagRegs mt;  // the next diagonal block (first diagonal tile only), on its way while the panel is solved
  if (ti == 0) load_diag_block(M, ld, base, (int)(n - base < NB ? n - base : NB), mt);
  {
    TileRegs ta, tb, tl;
    tile_fetch(ta, Pcur, NB, i0, rows_total, 0, NB);
    tile_fetch(tl, linv, NB, 0, NB, 0, NB);
    if (ti != tj) tile_fetch(tb, Pcur, NB, c0, rows_total, 0, NB);  // tj < ti: all 64 rows lie above row i0 <= n
    tile_put(Li, ta, i0, rows_total, NB);
    tile_put(Ls, tl, 0, NB, NB);
    if (ti != tj) tile_put(Lj, tb, c0, rows_total, NB);
  }
  __syncthreads();
  double4_t xi[4], xj[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) xi[j] = xj[j] = double4_t{0.0, 0.0, 0.0, 0.0};
  tile_nt_lower_mfma(Li, Ls, xi);
  if (ti != tj) tile_nt_lower_mfma(Lj, Ls, xj);
  __syncthreads();
#pragma unroll
  for (int j = 0; j < 4; ++j)
#pragma unroll
    for (int r4 = 0; r4 < 4; ++r4) {
      const int r = 16 * wave + 4 * r4 + (lane >> 4), c = 16 * j + (lane & 15);
      const double x = xi[j][r4];
      Li[r][c] = x;
      // on a diagonal tile Lj is the same piece without the right-hand-side row (row n of the matrix)
      Lj[r][c] = ti != tj ? xj[j][r4] : (c0 + r < n ? x : 0.0);
      if (tj == 0 && i0 + r < rows_total) M[(i0 + r) * ld + j0 + c] = x;
    }
  __syncthreads();
  if (ti == 0) {  // tj == 0 too: the next diagonal block
    // a short last block shares its tile with the right-hand-side row, which still needs this update
    if (rows_total > n && n - base < NB && (int64_t)threadIdx.x < n - base) {
      const int rr = (int)(n - base), c = threadIdx.x;
      double sum = 0.0;
      for (int k = 0; k < NB; ++k) sum += Li[rr][k] * Lj[c][k];
      M[n * ld + base + c] -= sum;
    }
    __syncthreads();  // the row above has read Li, which becomes the block's tile
    chol_diag_body(M, ld, base, (int)(n - base < NB ? n - base : NB), linv_next, flag, Lj, Li, Ls, mt);
    return;
  }
  double4_t acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) acc[i][j] = double4_t{0.0, 0.0, 0.0, 0.0};
  tile_nt_mfma(Li, Lj, acc);
  tile_sub_store<2, 2>(M, ld, rows_total, n, i0, c0, wi, wj, acc, tj == 0 ? Pnext : nullptr);
}

// rows [row0, rows_total) of the 64 columns at j0 -> P (row r at P[r * 64 ..]): the panel of a first fused step behind others
__global__ void copy_panel_kernel(const double* M, int64_t ld, int64_t rows_total, int64_t row0, int64_t j0, int64_t n, double* P) {
  const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t r = row0 + (idx >> 6);
  const int c = (int)(idx & 63);
  if (r < rows_total) P[r * NB + c] = j0 + c < n ? M[r * ld + j0 + c] : 0.0;
}

// Trailing update of a whole super-panel: A22 -= L21 L21^T with L21 = the KW columns starting at J, on the lower part of
// the matrix from row/column `base` = J + KW on. A tile stays in registers across the columns of the super-panel, so it
// is read and written once per super-panel instead of once per 64 columns. Two kernels share it.
//
// The next super-panel's own columns: 64x64 tiles (block columns 0 .. gridDim.x - 1), which fill the GPU, and the
// workgroup of the first one goes on to factorise it, as in chol_update_kernel<true>; the first block column also goes to P, the
// panel of the fused step that follows. The next chunk of the two operands is
// fetched into registers while the matrix cores work on the current one.
template <int KW>  // known at compile time, so that the chunk loop unrolls (column offsets become immediates and the
                   // accumulators stay where the matrix cores want them)
__global__ __launch_bounds__(kThreads) void chol_update_next_kernel(double* M, int64_t ld, int64_t rows_total, int64_t n, int64_t J,
                                                                    int64_t base, double* linv_next, int* flag, double* P) {
  const int ti = blockIdx.y, tj = blockIdx.x;
  if (tj > ti) return;
  __shared__ double Li[kTile][NB + 1];
  __shared__ double Lj[kTile][NB + 1];
  const int tid = threadIdx.x;
  const int64_t i0 = base + (int64_t)ti * kTile, c0 = base + (int64_t)tj * kTile;
  constexpr int kPer = kTile * NB / kThreads;
  double pi[kPer], pj[kPer];
  // Rows past the end of the matrix are read from the last valid row instead of being zeroed: such a row of an
  // operand only reaches rows (or columns) of the tile that are never stored. The row addresses are formed once.
  const double* rowi[kPer];
  const double* rowj[kPer];
#pragma unroll
  for (int u = 0; u < kPer; ++u) {
    const int idx = tid + u * kThreads, r = idx >> 6, c = idx & 63;
    rowi[u] = M + (i0 + r < rows_total ? i0 + r : rows_total - 1) * ld + J + c;
    rowj[u] = M + (c0 + r < n ? c0 + r : n - 1) * ld + J + c;
  }
  auto fetch = [&](int kc) {
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
      pi[u] = rowi[u][kc];
      pj[u] = rowj[u][kc];
    }
  };
  double4_t acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) acc[i][j] = double4_t{0.0, 0.0, 0.0, 0.0};
  fetch(0);
  DiagRegs mt;   // the next diagonal block (its workgroup only)
#pragma unroll
  for (int kc = 0; kc < KW; kc += NB) {
    __syncthreads();
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
      const int idx = tid + u * kThreads, r = idx >> 6, c = idx & 63;
      Li[r][c] = pi[u];
      Lj[r][c] = pj[u];
    }
    __syncthreads();
    if (kc + NB < KW) fetch(kc + NB);
    else if (ti == 0) load_diag_block(M, ld, base, NB, mt);
    tile_nt_mfma(Li, Lj, acc);
  }
  if (ti == 0) {   // the next diagonal block (the super-panels leave at least 64 columns)
    __syncthreads();   // every wave has read Li and Lj
    const int wi = (tid >> 7) * 32, wj = ((tid >> 6) & 1) * 32;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j) sub_block_store(Li, wi + 16 * i, wj + 16 * j, acc[i][j]);
    __syncthreads();
#pragma unroll
    for (int u = 0; u < 3; ++u) {
      const int t = (tid >> 6) + 4 * u;
      if (t < kDiagTiles) {
        int r0, q0;
        diag_subtile(t, r0, q0);
        mt.v[u] -= sub_block_load(Li, r0, q0);
      }
    }
    __syncthreads();   // Li becomes the block's tile
    chol_diag_body(M, ld, base, NB, linv_next, flag, nullptr, Li, Lj, mt);
    return;
  }
  const int wave = tid >> 6;
  tile_sub_store<2, 2>(M, ld, rows_total, n, i0, c0, (wave >> 1) * 32, (wave & 1) * 32, acc, tj == 0 ? P : nullptr);
}

// The rest of the matrix, 128x128 tiles from row/column `base` on (T rows of tiles), a 32x64 piece of one to each of
// eight waves. One workgroup fills a compute unit, so the kernel pipelines on its own: the operands' next step is on its
// way while the matrix cores work on the current one, the tile's old values under the last step, the next tile's first
// step under this tile's stores. A tile takes 37 us, 30 of them the products (the matrix cores alone need 28.5), the rest
// is the tile's way in and out: 51 TFLOP/s over 946 tiles on 256 compute units, against 44 of 64 x 64 tiles. Two workgroups
// of four waves on a unit reach more (30 us a tile), but the diagonal block's lone wave beside them then takes six times
// as long; a whole unit to a workgroup leaves kWideSpare units to the chain.
constexpr int kWideThreads = 512;
constexpr int kWideTile = 128;
constexpr int kWideK = 32;                 // columns per step, two buffers
constexpr int kWidePitch = kWideK + 2;     // doubles per LDS row: the 32 lanes of half a wave read from all 64 banks
constexpr int kWidePut = 24;               // column of a step after which the next one's operands go to LDS
constexpr int kWideSpare = 32;             // compute units left to the chain on the side stream
constexpr int kWideStrip = 4;              // tile rows walked together

// the p-th lower tile of T rows of tiles, in strips of kWideStrip rows, column by column inside a strip: workgroups with
// neighbouring p share operands
__device__ __forceinline__ void wide_tile_of(int p, int T, int& ti, int& tj) {
  int r0 = 0, h = 0;
  for (;; r0 += kWideStrip) {
    h = T - r0 < kWideStrip ? T - r0 : kWideStrip;
    const int count = h * (r0 + 1) + h * (h - 1) / 2;
    if (p < count) break;
    p -= count;
  }
  if (p < h * (r0 + 1)) {
    tj = p / h;
    ti = r0 + p % h;
    return;
  }
  p -= h * (r0 + 1);
  int j = 1;
  for (; p >= h - j; ++j) p -= h - j;
  tj = r0 + j;
  ti = r0 + j + p;
}

template <int KW>
__global__ __launch_bounds__(kWideThreads, 2) void chol_update_wide_kernel(double* M, int64_t ld, int64_t rows_total, int64_t n,
                                                                           int64_t J, int64_t base, int T, int tiles) {
  __shared__ __align__(16) double Ls[2][2][kWideTile * kWidePitch];   // [buffer][rows, columns of the tile]
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int l16 = lane & 15, lk = lane >> 4;
  const int wi = (wave >> 1) * 32, wj = (wave & 1) * 64;
  typedef double pair_t __attribute__((ext_vector_type(2)));
  constexpr int kPer = kWideTile * kWideK / 2 / kWideThreads;   // 16-byte pieces per thread and operand
  constexpr int kRowsPer = kWideThreads / (kWideK / 2);         // rows per pass
  const int pr = tid / (kWideK / 2), pc = (tid % (kWideK / 2)) * 2;
  int64_t i0, c0;
  int ti, tj;
  const char *basei, *basej;   // one base per operand and 32-bit offsets from it
  uint32_t offi[kPer], offj[kPer];
  pair_t pi[kPer], pj[kPer];
  auto fetch = [&](int kc) {
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
      pi[u] = *(const pair_t*)(basei + (offi[u] + (uint32_t)kc * 8u));
      pj[u] = *(const pair_t*)(basej + (offj[u] + (uint32_t)kc * 8u));
    }
  };
  auto put = [&](int buf) {
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
      *(pair_t*)&Ls[buf][0][(pr + u * kRowsPer) * kWidePitch + pc] = pi[u];
      *(pair_t*)&Ls[buf][1][(pr + u * kRowsPer) * kWidePitch + pc] = pj[u];
    }
  };
  auto start = [&](int p) {   // the p-th tile, its first step requested
    wide_tile_of(p, T, ti, tj);
    i0 = base + (int64_t)ti * kWideTile;
    c0 = base + (int64_t)tj * kWideTile;
    basei = (const char*)(M + i0 * ld + J);
    // (a last tile that holds the right-hand-side row only has no columns of its own; it is not stored)
    const int64_t cs = c0 < n ? c0 : n - 1;
    basej = (const char*)(M + cs * ld + J);
    const int last_i = (int)(rows_total - 1 - i0 < kWideTile ? rows_total - 1 - i0 : kWideTile);
    const int last_j = (int)(n - 1 - cs < kWideTile ? n - 1 - cs : kWideTile);
#pragma unroll
    for (int u = 0; u < kPer; ++u) {   // (rows past the end: as in chol_update_next_kernel)
      const int r = pr + u * kRowsPer;
      offi[u] = ((uint32_t)(r < last_i ? r : last_i) * (uint32_t)ld + (uint32_t)pc) * 8u;
      offj[u] = ((uint32_t)(r < last_j ? r : last_j) * (uint32_t)ld + (uint32_t)pc) * 8u;
    }
    fetch(0);
  };
  // consecutive workgroups go to the eight XCDs in turn: each XCD takes a run of neighbouring tiles
  const int G = (int)gridDim.x, bid = (int)blockIdx.x;
  int p = (G & 7) == 0 ? (bid & 7) * (G >> 3) + (bid >> 3) : bid;
  if (p >= tiles) return;
  start(p);
  for (;;) {
    double4_t acc[2][4], cur[2][4];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j) acc[i][j] = double4_t{0.0, 0.0, 0.0, 0.0};
    const bool live = ti != tj || wj < wi + 32;   // (a piece above the diagonal has nothing to do)
    put(0);   // (every wave is past the barrier that ended the tile before)
    __syncthreads();
#pragma unroll
    for (int kc = 0; kc < KW; kc += kWideK) {
      const int buf = (kc / kWideK) & 1;
      const bool last = kc + kWideK >= KW;
      if (!last) {
        fetch(kc + kWideK);
      } else {
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int r4 = 0; r4 < 4; ++r4) {
            const int64_t r = i0 + wi + 16 * i + 4 * r4 + lk, rs = r < rows_total ? r : rows_total - 1;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
              const int64_t c = c0 + wj + 16 * j + l16;
              cur[i][j][r4] = M[rs * ld + (c < n ? c : n - 1)];
            }
          }
      }
      const double* pa = &Ls[buf][0][(wi + l16) * kWidePitch + lk];
      const double* pb = &Ls[buf][1][(wj + l16) * kWidePitch + lk];
      double av[2][2], bv[2][4];
      auto operands = [&](int k0) {
        const int q = (k0 >> 2) & 1;
#pragma unroll
        for (int i = 0; i < 2; ++i) av[q][i] = pa[i * 16 * kWidePitch + k0];
#pragma unroll
        for (int j = 0; j < 4; ++j) bv[q][j] = pb[j * 16 * kWidePitch + k0];
      };
      operands(0);
#pragma unroll
      for (int k0 = 0; k0 < kWideK; k0 += 4) {
        const int q = (k0 >> 2) & 1;
        if (k0 + 4 < kWideK) operands(k0 + 4);
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int j = 0; j < 4; ++j) acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[q][i], bv[q][j], acc[i][j], 0, 0, 0);
        if (k0 == kWidePut && !last) put(buf ^ 1);
      }
      __syncthreads();
    }
    const int64_t si = i0 + wi, sj = c0 + wj;
    p += G;
    const bool more = p < tiles;
    if (more) start(p);
    if (live) {
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int r4 = 0; r4 < 4; ++r4) {
          const int64_t r = si + 16 * i + 4 * r4 + lk;
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            const int64_t c = sj + 16 * j + l16;
            if (r < rows_total && c < n && c <= r) M[r * ld + c] = cur[i][j][r4] - acc[i][j][r4];
          }
        }
    }
    if (!more) return;
  }
}


// Triangular solves with the factor, kSolveBlocks * 64 unknowns per launch (BLOCKS blocks of 64 from column J on). Every workgroup
// solves the launch's unknowns itself from the stored inverses of the diagonal blocks, then takes their contribution off
// its own 64 entries of v that are still to be solved. What bounds them is latency: a chain of launches, in each eight dependent
// products of a 64 x 64 tile with a vector. All of a thread's matrix entries (8 per tile, 14 tiles) are therefore requested before the
// first product, and partial sums stay in registers until their block's turn. Sums have a fixed order.
constexpr int64_t kFuseMaxRows = 2048;
constexpr int kSolveBlocks = 4;                    // diagonal blocks per launch
constexpr int kSolveThreads = 512;
constexpr int kSolvePer = NB * NB / kSolveThreads; // entries of a 64 x 64 tile per thread: one output, eight terms

// sum over the eight neighbouring lanes that share lane / 8, in all of them
__device__ __forceinline__ double sum_of_8_lanes(double a) {
#define DS_DPP_ADD(ctrl)                                                                          \
  a += __hiloint2double(__builtin_amdgcn_update_dpp(0, __double2hiint(a), ctrl, 0xf, 0xf, false), \
                        __builtin_amdgcn_update_dpp(0, __double2loint(a), ctrl, 0xf, 0xf, false))
  DS_DPP_ADD(0xb1);    // quad_perm [1,0,3,2]
  DS_DPP_ADD(0x4e);    // quad_perm [2,3,0,1]
  DS_DPP_ADD(0x141);   // row_half_mirror
#undef DS_DPP_ADD
  return a;
}

// L x = v from the front, out = x (for a factorisation that ran without the right-hand side as its row n). Eight neighbouring lanes
// share a row of a tile, 16 bytes each at a time, and fold its sum by three DPP moves.
template <int BLOCKS>
__global__ __launch_bounds__(kSolveThreads) void chol_forward_kernel(const double* M, int64_t ld, int64_t n, int64_t J,
                                                                     const double* linv, double* v, double* out) {
  __shared__ __align__(16) double xs[NB];
  __shared__ __align__(16) double ys[BLOCKS][NB];
  typedef double pair_t __attribute__((ext_vector_type(2)));
  const int tid = threadIdx.x, o = tid >> 3, q = tid & 7;   // row of a tile, share of its columns
  struct Terms { pair_t a[kSolvePer / 2]; };
  auto fetch = [&](Terms& t, const double* A, int64_t stride, int64_t row0, int64_t rows, int64_t col0) {
    // (rows past n are read from row n - 1; their sums are not used)
    const double* row = A + (row0 + o < rows ? row0 + o : rows - 1) * stride + col0 + 2 * q;
#pragma unroll
    for (int i = 0; i < kSolvePer / 2; ++i) t.a[i] = *(const pair_t*)(row + 16 * i);
  };
  auto dot = [&](const Terms& t, const double* x) {
    double s = 0.0;
#pragma unroll
    for (int i = 0; i < kSolvePer / 2; ++i) {
      const pair_t w = *(const pair_t*)(x + 16 * i + 2 * q);
      s += t.a[i].x * w.x;
      s += t.a[i].y * w.y;
    }
    return s;
  };
  Terms inv[BLOCKS], in[BLOCKS][BLOCKS], rest[BLOCKS];
  double rhs[BLOCKS], acc[BLOCKS];
  const int64_t j0 = J + BLOCKS * NB + (int64_t)blockIdx.x * NB;
  const bool more = j0 < n;   // (the last launch: workgroup 0 only, no entries left)
#pragma unroll
  for (int b = 0; b < BLOCKS; ++b) {
    fetch(inv[b], linv + (size_t)(J / NB + b) * NB * NB, NB, 0, NB, 0);
    const int64_t at = J + b * NB + o;
    rhs[b] = at < n ? v[at] : 0.0;
    acc[b] = 0.0;
#pragma unroll
    for (int c = b + 1; c < BLOCKS; ++c) fetch(in[b][c], M, ld, J + c * NB, n, J + b * NB);
  }
#pragma unroll
  for (int b = 0; b < BLOCKS; ++b) {
    const int64_t at = J + b * NB + o;
    const double x = at < n ? rhs[b] - (b > 0 ? sum_of_8_lanes(acc[b]) : 0.0) : 0.0;
    if (q == 0) xs[o] = x;
    __syncthreads();
    const double y = sum_of_8_lanes(dot(inv[b], xs));
    if (q == 0) ys[b][o] = y;
    if (q == 0 && blockIdx.x == 0 && at < n) out[at] = y;
    if (more) fetch(rest[b], M, ld, j0, n, J + b * NB);   // (the remaining steps hide it)
    __syncthreads();
#pragma unroll
    for (int c = b + 1; c < BLOCKS; ++c) acc[c] += dot(in[b][c], ys[b]);
  }
  if (!more) return;
  double sum = 0.0;
#pragma unroll
  for (int b = 0; b < BLOCKS; ++b) sum += dot(rest[b], ys[b]);
  sum = sum_of_8_lanes(sum);
  if (q == 0 && j0 + o < n) v[j0 + o] -= sum;
}

// L^T psi = v from the end, phi = psi + (y1 - y0)/n. A wave reads whole rows of a tile (lane = column), and the eight waves'
// partial sums meet in LDS: lanes that share a column, as in the forward solve, would read 64 bytes of a row each (a launch then
// takes 20 us instead of 10).
template <int BLOCKS>
__global__ __launch_bounds__(kSolveThreads) void chol_back_kernel(const double* M, int64_t ld, int64_t n, int64_t J,
                                                                  const double* linv, double* v, const float* y01, float* phi) {
  constexpr int kWavesHere = kSolveThreads / NB;
  __shared__ double xs[NB];
  __shared__ double ys[BLOCKS][NB];
  __shared__ double part[kWavesHere][NB];
  const int tid = threadIdx.x, c = tid & (NB - 1), g = tid / NB;   // column of a tile, first of its rows
  struct Terms { double a[kSolvePer]; };
  auto fetch = [&](Terms& t, const double* A, int64_t stride, int64_t row0, int64_t rows, int64_t col0) {
#pragma unroll
    for (int i = 0; i < kSolvePer; ++i) {   // (rows past n are read from row n - 1 and meet zeros)
      const int64_t r = row0 + g + kWavesHere * i;
      t.a[i] = A[(r < rows ? r : rows - 1) * stride + col0 + c];
    }
  };
  auto dot = [&](const Terms& t, const double* x) {
    double s = 0.0;
#pragma unroll
    for (int i = 0; i < kSolvePer; ++i) s += t.a[i] * x[g + kWavesHere * i];
    return s;
  };
  auto folded = [&]() {   // the first wave: the sum of the partial sums of its lane's column
    double s = 0.0;
#pragma unroll
    for (int w = 0; w < kWavesHere; ++w) s += part[w][c];
    return s;
  };
  Terms inv[BLOCKS], in[BLOCKS][BLOCKS], rest[BLOCKS];
  double rhs[BLOCKS], acc[BLOCKS];
  const int64_t j0 = (int64_t)blockIdx.x * NB;
  const bool more = j0 < J;   // (the last launch: workgroup 0 only, no entries left)
#pragma unroll
  for (int b = BLOCKS - 1; b >= 0; --b) {
    fetch(inv[b], linv + (size_t)(J / NB + b) * NB * NB, NB, 0, NB, 0);   // (identity-padded, zero above the diagonal)
    rhs[b] = J + b * NB + c < n ? v[J + b * NB + c] : 0.0;
    acc[b] = 0.0;
#pragma unroll
    for (int k = b - 1; k >= 0; --k) fetch(in[b][k], M, ld, J + b * NB, n, J + k * NB);
  }
  const double shift = ((double)y01[1] - (double)y01[0]) / (double)n;
#pragma unroll
  for (int b = BLOCKS - 1; b >= 0; --b) {
    if (b < BLOCKS - 1) {
      part[g][c] = acc[b];
      __syncthreads();
    }
    if (g == 0) xs[c] = b < BLOCKS - 1 ? rhs[b] - folded() : rhs[b];
    __syncthreads();
    part[g][c] = dot(inv[b], xs);
    if (more) fetch(rest[b], M, ld, J + b * NB, n, j0);   // (the remaining steps hide it)
    __syncthreads();
    if (g == 0) {
      const double s = folded();
      ys[b][c] = s;
      const int64_t at = J + b * NB + c;
      if (blockIdx.x == 0 && at < n) phi[at] = (float)(s + shift);
    }
    __syncthreads();
#pragma unroll
    for (int k = b - 1; k >= 0; --k) acc[k] += dot(in[b][k], ys[b]);
  }
  if (!more) return;
  double sum = 0.0;
#pragma unroll
  for (int b = BLOCKS - 1; b >= 0; --b) sum += dot(rest[b], ys[b]);
  part[g][c] = sum;
  __syncthreads();
  if (g == 0) v[j0 + c] -= folded();
}

inline float dense_fraction(const ds_ctx* ctx) {
  return ctx->tuning.gram_dense_fraction > 0.f ? ctx->tuning.gram_dense_fraction : kDenseFraction;
}
inline int sparse_divisor(const ds_ctx* ctx) {
  return ctx->tuning.gram_sparse_div >= 1 ? ctx->tuning.gram_sparse_div : kSparseDivisor;
}

// ---------------- games of at most 64 players ----------------
// One mask word per row and one diagonal block: four launches in place of fourteen, each of which costs its start and a
// trip through memory for a few kilobytes of matrix (an explanation of 12 players, 4,096 coalitions: 324 us; now 232). Sums of the weights themselves
// in fp64, in a fixed order; a pair of players costs six instructions per row. A solve alone, us, fourteen launches and four:
//   13 players    4,096 rows 149, 69    80,000 267, 82     400,000 760, 130     1,600,000 2,560, 317
//   33 players    4,096 rows 150, 73    80,000 275, 132    400,000 768, 363     1,600,000 2,604, 1,229
//   64 players    4,096 rows 154, 92    80,000 299, 201    400,000 878, 639     1,600,000 3,020, 2,272
// The line is drawn by the players alone, as more do not fit one block. Near it and with many rows, the 64 workgroups of these kernels are
// too few: 65 players, which the general kernels take, 200,000 rows 344 (64 players: 363), 400,000 568 (639), 1,600,000 1,837 (2,273).
constexpr int kSmallChunk = 512;    // rows per step
constexpr int kSmallParts = 64;     // workgroups at most, each with a part of the rows

// part[blockIdx.x][p] = sum of the weights of this workgroup's rows that hold both players of pair p (the threads' shares: small_game.h).
__global__ __launch_bounds__(kSmallThreads) void small_gram_kernel(const uint64_t* Z, const float* w, int64_t R, int paired, int n,
                                                                   double* part) {
  __shared__ uint64_t zs[kSmallChunk];
  __shared__ double ws[kSmallChunk];
  __shared__ double red[kSmallThreads];
  const int tid = threadIdx.x, pairs = n * (n + 1) / 2;
  const ds_small_share mine = ds_small_share_of(pairs, tid);
  const int width = mine.width, groups = mine.groups, t = mine.at;
  uint64_t mask[kSmallPerThread];
  double acc[kSmallPerThread];
#pragma unroll
  for (int u = 0; u < kSmallPerThread; ++u) {
    const int p = t + u * width;
    int a = 0, b = 0;
    small_pair(p < pairs ? p : 0, a, b);
    mask[u] = (1ull << a) | (1ull << b);
    acc[u] = 0.0;
  }
  const int64_t per = (R + gridDim.x - 1) / gridDim.x;
  const int64_t first = per * blockIdx.x, last = first + per < R ? first + per : R;
  for (int64_t r0 = first; r0 < last; r0 += kSmallChunk) {
    const int count = (int)(last - r0 < kSmallChunk ? last - r0 : kSmallChunk);
    __syncthreads();
    if (tid < count) {
      zs[tid] = Z[(r0 + tid) * (paired ? 2 : 1)];
      ws[tid] = (double)used_row_weight(w, r0 + tid, paired);
    }
    __syncthreads();
    if (ds_small_adds(mine))
      for (int i = mine.group; i < count; i += groups) {
        const uint64_t z = zs[i];
        const double wi = ws[i];
#pragma unroll
        for (int u = 0; u < kSmallPerThread; ++u)
          if (u * width < pairs) acc[u] += (z & mask[u]) == mask[u] ? wi : 0.0;
      }
  }
  if (groups > 1) {
    red[tid] = acc[0];
    __syncthreads();
  }
  if (!ds_small_stores(mine)) return;
  for (int i = 1; i < groups; ++i) acc[0] += red[i * width + t];
#pragma unroll
  for (int u = 0; u < kSmallPerThread; ++u)
    if (t + u * width < pairs) part[(size_t)blockIdx.x * pairs + t + u * width] = acc[u];
}

// cpart[blockIdx.x][a] = sum over this workgroup's rows that hold player a of the right-hand side's coefficients
// (used_row_rhs_kernel on row_prep's values)
__global__ __launch_bounds__(kSmallThreads) void small_rhs_kernel(const uint64_t* Z, const float* w, const float* y, int64_t R,
                                                                  int paired, int n, double* cpart) {
  __shared__ uint64_t zs[kSmallChunk];
  __shared__ double gs[kSmallChunk];
  __shared__ double red[kSmallThreads / 64][64];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const double f0 = (double)y[0], slope = ((double)y[1] - (double)y[0]) / (double)n;
  const uint64_t all = n < 64 ? (1ull << n) - 1ull : ~0ull;
  const int64_t per = (R + gridDim.x - 1) / gridDim.x;
  const int64_t first = per * blockIdx.x, last = first + per < R ? first + per : R;
  double acc = 0.0;
  for (int64_t r0 = first; r0 < last; r0 += kSmallChunk) {
    const int count = (int)(last - r0 < kSmallChunk ? last - r0 : kSmallChunk);
    __syncthreads();
    if (tid < count) {
      const int64_t i = (r0 + tid) * (paired ? 2 : 1);
      const uint64_t z = Z[i];
      const int size = __popcll(z & all);
      auto t = [&](int64_t row, int members) { return row < 2 ? 0.0 : (double)y[row] - f0 - slope * (double)members; };
      const double wi = i < 2 ? 0.0 : (double)w[i];
      zs[tid] = z;
      gs[tid] = paired ? wi * (t(i, size) - t(i + 1, n - size)) : wi * t(i, size);
    }
    __syncthreads();
    for (int i = wave; i < count; i += kSmallThreads / 64) acc += (zs[i] >> lane) & 1ull ? gs[i] : 0.0;
  }
  red[wave][lane] = acc;
  __syncthreads();
  if (wave > 0) return;
  for (int i = 1; i < kSmallThreads / 64; ++i) acc += red[i][lane];
  cpart[(size_t)blockIdx.x * 64 + lane] = acc;
}

// right-hand side from its parts, forward and back substitution by the inverse of the one block, phi: one workgroup
__global__ __launch_bounds__(kThreads) void small_solve_kernel(const double* cpart, int parts, int n, const double* linv,
                                                               const float* y01, float* phi) {
  constexpr int kPer = NB * NB / kThreads;
  __shared__ double xs[2][NB];
  __shared__ double part[kThreads / NB][NB];
  const int tid = threadIdx.x, c = tid & (NB - 1), g = tid / NB;
  double li[kPer];   // rows g, g + 4, .. of column c
#pragma unroll
  for (int i = 0; i < kPer; ++i) li[i] = linv[(g + (kThreads / NB) * i) * NB + c];
  double sum = 0.0;
  for (int i = g; i < parts; i += kThreads / NB) sum += cpart[(size_t)i * 64 + c];
  part[g][c] = sum;
  __syncthreads();
  if (g == 0) {   // the first wave: c - mean(c)
    double x = 0.0;
    for (int i = 0; i < kThreads / NB; ++i) x += part[i][c];
    x = c < n ? x : 0.0;
    const double mean = ds_wave_sum(x) / (double)n;
    xs[0][c] = c < n ? x - mean : 0.0;
  }
  __syncthreads();
  // y = Linv x: a wave's rows one after the other, folded over its lanes
#pragma unroll
  for (int i = 0; i < kPer; ++i) {
    const double v = ds_wave_sum(li[i] * xs[0][c]);
    if (c == 0) xs[1][g + (kThreads / NB) * i] = v;
  }
  __syncthreads();
  double s = 0.0;   // psi = Linv^T y
#pragma unroll
  for (int i = 0; i < kPer; ++i) s += li[i] * xs[1][g + (kThreads / NB) * i];
  part[g][c] = s;
  __syncthreads();
  if (g == 0 && c < n) {
    double v = 0.0;
    for (int i = 0; i < kThreads / NB; ++i) v += part[i][c];
    phi[c] = (float)(v + ((double)y01[1] - (double)y01[0]) / (double)n);
  }
}

inline unsigned nblocks(int64_t n, int per) { return (unsigned)((n + per - 1) / per); }

// workgroups of the small games' two passes over the rows
inline unsigned small_parts(int64_t R) {
  const int64_t parts = (R + 63) / 64;
  return (unsigned)(parts < 1 ? 1 : parts > kSmallParts ? kSmallParts : parts);
}

struct GramDims {
  int64_t R, RW, ld, nblk;
  int slices;       // of the column-wise part, and one more of the sparse rows unless they have a launch of their own
  int rows_apart;
  int64_t words_per_slice;
};

GramDims gram_dims(int64_t n, int64_t k, int paired, int num_cus) {
  GramDims d;
  d.R = paired ? k / 2 : k;
  d.RW = (d.R + 63) / 64;
  d.ld = (n + 1 + 7) & ~(int64_t)7;
  d.nblk = (n + NB - 1) / NB;
  const int64_t tiles = (n + kTile - 1) / kTile;
  const int64_t lower = tiles * (tiles + 1) / 2;
  if (num_cus > 256) num_cus = 256;
  int64_t s = (2 * (int64_t)num_cus + lower - 1) / lower;
  const int64_t chunks = (d.RW + kChunk - 1) / kChunk;
  if (s > chunks) s = chunks;
  if (s > 16) s = 16;
  if (s < 1) s = 1;
  const int64_t cps = (chunks + s - 1) / s;  // chunks per slice
  d.words_per_slice = cps * kChunk;
  d.slices = (int)((chunks + cps - 1) / cps);
  d.rows_apart = lower > num_cus;
  if (!d.rows_apart) ++d.slices;
  return d;
}

}  // namespace

// row sums of G by tile columns
static size_t gram_sums_bytes(int64_t n) { return (size_t)((n + kTile - 1) / kTile) * n * 8; }

// the parts of the sums of a game of at most 64 players: per pair of players, and per player
static constexpr size_t small_bytes = (size_t)kSmallParts * kSmallPairs * 8;

// rows of a 64-column panel, one buffer (the fused steps of the factorisation keep two)
static size_t panel_bytes(int64_t n) { return (size_t)(n + 1) * NB * 8; }

size_t ds_gram_arena_bytes(int64_t n, int64_t k) {
  const GramDims d = gram_dims(n, k, 0, 256);  // the unpaired layout is the larger one
  const GramDims dp = gram_dims(n, k, 1, 256);
  const size_t slices = (size_t)(d.slices > dp.slices ? d.slices : dp.slices) + 1;  // +1: CU counts differ a little
  return (n <= kSmallMax ? 2 * ds_align(small_bytes) : 0) + ds_align(gram_sums_bytes(n)) + ds_align((size_t)n * d.RW * 8) + ds_align(slices * (size_t)n * n * 8) + ds_align((size_t)(n + 1) * d.ld * 8) +
         ds_align((size_t)d.nblk * NB * NB * 8) + 2 * ds_align(panel_bytes(n)) + 2 * ds_align(k * 4) + 2 * ds_align(k * 8) + ds_align(k * 4) +
         ds_align(k * 8) + ds_align(d.RW * 4) * 2 + 4 * ds_align(n * 8) + 8192 +
         ds_align((size_t)((n + 63) / 64) * d.R * 8 + 8) + ds_align((size_t)d.RW * 8 + 8) + ds_align((size_t)d.R * 8 + 8) + 256;
}

// The buffers of all parts, from one contiguous region of the arena.
int ds_gram_alloc(ds_ctx* ctx, int64_t n, int64_t k, int paired, ds_gram_state* gs) {
  if (paired && (k & 1)) return ds_fail(ctx, DS_EINVAL, "paired rows need an even row count");
  const int64_t W = (n + 63) / 64;
  const GramDims d = gram_dims(n, k, paired, ctx->num_cus);
  const int64_t R = d.R, RW = d.RW, ld = d.ld;
  gs->n = n; gs->k = k; gs->R = R; gs->RW = RW; gs->ld = ld; gs->nblk = d.nblk; gs->paired = paired;
  gs->Zt = (uint64_t*)ds_arena_alloc(ctx, (size_t)n * RW * 8);
  gs->slices = d.slices; gs->rows_apart = d.rows_apart; gs->words_per_slice = d.words_per_slice;
  gs->Gp = (double*)ds_arena_alloc(ctx, n <= kSmallMax ? small_bytes : (size_t)d.slices * n * n * 8);
  gs->M = (double*)ds_arena_alloc(ctx, (size_t)(n + 1) * ld * 8);
  gs->linv = (double*)ds_arena_alloc(ctx, (size_t)d.nblk * NB * NB * 8);
  gs->panel[0] = (double*)ds_arena_alloc(ctx, panel_bytes(n));
  gs->panel[1] = (double*)ds_arena_alloc(ctx, panel_bytes(n));
  gs->gw = (float*)ds_arena_alloc(ctx, R * 4);
  gs->wu = (float*)ds_arena_alloc(ctx, RW * 4);
  gs->uni = (int32_t*)ds_arena_alloc(ctx, RW * 4);
  gs->m = (double*)ds_arena_alloc(ctx, n * 8);
  gs->sums = (double*)ds_arena_alloc(ctx, gram_sums_bytes(n));
  gs->stats = (double*)ds_arena_alloc(ctx, 64);
  gs->Zc = (uint64_t*)ds_arena_alloc(ctx, (size_t)W * R * 8 + 8);
  gs->keep = (uint64_t*)ds_arena_alloc(ctx, (size_t)RW * 8 + 8);
  gs->wq = (uint64_t*)ds_arena_alloc(ctx, (size_t)R * 8 + 8);
  gs->gscale = (double*)ds_arena_alloc(ctx, 64);
  gs->sz = (int32_t*)ds_arena_alloc(ctx, k * 4);
  gs->wc = (float*)ds_arena_alloc(ctx, k * 4);
  gs->t = (double*)ds_arena_alloc(ctx, n <= kSmallMax ? small_bytes : k * 8);
  gs->sqw = (double*)ds_arena_alloc(ctx, k * 8);
  gs->gc = (double*)ds_arena_alloc(ctx, R * 8);
  gs->c = (double*)ds_arena_alloc(ctx, n * 8);
  gs->flag = (int*)ds_arena_alloc(ctx, 64);
  if (!gs->Zt || !gs->Gp || !gs->M || !gs->linv || !gs->panel[0] || !gs->panel[1] || !gs->gw || !gs->wu || !gs->uni || !gs->m ||
      !gs->sums || !gs->stats || !gs->Zc || !gs->keep || !gs->wq || !gs->gscale || !gs->sz || !gs->wc || !gs->t || !gs->sqw || !gs->gc || !gs->c ||
      !gs->flag)
    return ds_fail(ctx, DS_EINTERNAL, "gram: arena exhausted");
  return DS_OK;
}

// Part 1: everything that does not need the model outputs y (Gram matrix, projection, system matrix, first diagonal block).
// It may run on another stream than part 3, concurrently with the masked inference.
int ds_gram_begin(ds_ctx* ctx, ds_gram_state* gs, const uint64_t* Z, const float* w) {
  hipStream_t st = ctx->stream;
  const int64_t n = gs->n, R = gs->R, RW = gs->RW, ld = gs->ld, W = (n + 63) / 64;
  const int paired = gs->paired;
  gs->formed = n > kSmallMax ? ctx->kev[3] : nullptr;   // (the event of the mark below)
  if (n <= kSmallMax) {
    const unsigned parts = small_parts(R);
    DS_TRY(ds_kernel_mark(ctx, 1, 0));
    hipLaunchKernelGGL(small_gram_kernel, dim3(parts), dim3(kSmallThreads), 0, st, Z, w, R, paired, (int)n, gs->Gp);
    DS_TRY(ds_kernel_mark(ctx, 1, 1));
    DS_TRY(ds_kernel_mark(ctx, 2, 0));
    hipLaunchKernelGGL(chol_diag_kernel, dim3(1), dim3(kThreads), 0, st, gs->M, ld, (int64_t)0, (int)n, gs->linv, gs->flag, (const double*)gs->Gp,
                       (int)parts);
    DS_HIP(ctx, hipGetLastError());
    return ds_kernel_mark(ctx, 2, 1);
  }
  float *gw = gs->gw, *wu = gs->wu;
  int32_t* uni = gs->uni;
  double *Gp = gs->Gp, *m = gs->m, *stats = gs->stats, *gscale = gs->gscale;
  uint64_t *Zc = gs->Zc, *keep = gs->keep, *wq = gs->wq;
  DS_TRY(ds_bit_transpose(ctx, Z, R, n, W, 0, paired ? 2 : 1, gs->Zt));
  // sparse rows: row-wise outer products; the rest (bits in `keep`) column-wise
  const int64_t row_step = paired ? 2 : 1;
  hipLaunchKernelGGL(gram_weights_kernel, dim3(1), dim3(kWeightThreads), 0, st, w, R, paired, gw, gscale);
  const int64_t class_y = (RW + kClassGridX - 1) / kClassGridX;
  hipLaunchKernelGGL(gram_row_class_kernel, dim3((unsigned)((RW + class_y - 1) / class_y), (unsigned)class_y), dim3(64 * kClassWaves), 0, st, Z, R, W, n, row_step, gw, gscale,
                     sparse_divisor(ctx), dense_fraction(ctx), Zc, (unsigned long long*)keep, (unsigned long long*)wq, wu, uni);
  const unsigned tiles = nblocks(n, kTile);
  DS_TRY(ds_kernel_mark(ctx, 1, 0));
  if (gs->rows_apart)
    hipLaunchKernelGGL(gram_rows_kernel, dim3(tiles, tiles), dim3(kThreads), 0, st, Zc, (const unsigned long long*)wq, R, n,
                       gscale, Gp);
  hipLaunchKernelGGL(gram_kernel, dim3(tiles, tiles, gs->slices), dim3(kThreads), 0, st, gs->Zt, n, R, RW, gw, wu, uni, keep,
                     Gp, gs->words_per_slice, gs->rows_apart, Zc, (const unsigned long long*)wq, gscale,
                     gs->slices == 1 ? gs->sums : nullptr);
  DS_TRY(ds_kernel_mark(ctx, 1, 1));
  if (gs->slices > 1) hipLaunchKernelGGL(sum_slices_kernel, dim3(tiles, tiles), dim3(kThreads), 0, st, Gp, n, gs->slices, gs->sums);
  hipLaunchKernelGGL(row_means_kernel, dim3(nblocks(n, 64)), dim3(64), 0, st, gs->sums, n, (int)tiles, m);
  hipLaunchKernelGGL(stats_kernel, dim3(1), dim3(kThreads), 0, st, Gp, m, n, stats, gs->flag);
  hipLaunchKernelGGL(build_matrix_kernel, dim3(tiles, tiles), dim3(kThreads), 0, st, Gp, m, stats, n, ld, gs->M, gs->panel[0],
                     (double*)(gs->flag + 2));
  // the first diagonal block does not involve the right-hand side either: factorised here, off the path that waits
  // for the model outputs
  hipLaunchKernelGGL(chol_diag_kernel, dim3(1), dim3(kThreads), 0, st, gs->M, ld, (int64_t)0, (int)(n < NB ? n : NB), gs->linv,
                     gs->flag, (const double*)nullptr, 0);
  DS_HIP(ctx, hipGetLastError());
  return DS_OK;
}

// Part 2: the factorisation on ctx->stream (and, where the trailing matrix is large, the side stream). rows_total = n + 1: row n of
// the matrix carries the right-hand side along, which leaves L^-1 rhs in it. rows_total = n: the factor alone; mid, if
// not null, is recorded behind the last full group of kSolveBlocks blocks that is not the last group at all.
static int gram_factor(ds_ctx* ctx, const ds_gram_state* gs, int64_t rows_total, hipEvent_t mid) {
  hipStream_t st = ctx->stream;
  const int64_t n = gs->n, ld = gs->ld;
  double* M = gs->M;
  double* linv = gs->linv;
  const int64_t mid_at = (gs->nblk - 1) / kSolveBlocks * kSolveBlocks * NB;
  DS_TRY(ds_kernel_mark(ctx, 2, 0));
  // While the trailing matrix is large the blocks are taken four at a time (a super-panel of 256 columns):
  // inside it the updates reach only the super-panel's own columns, and the rest of the trailing matrix is
  // updated once with all 256 columns. Below kFuseMaxRows trailing rows: one block per step, the update
  // factorising the next diagonal block on the way.
  // The super-panels run one ahead on the side stream: the columns of the next super-panel are updated first and its
  // chain of small launches (fused steps on its own columns; panels and updates apart: six games of 1,175 to 6,007 10.3 ms, now 10.1) goes on behind
  // them, while the main stream updates the rest of the matrix. Every tile still meets the super-panels in their order:
  // the next super-panel's columns wait for the rest of the update before (join_ev), the rest for them (fork_ev).
  hipStream_t chain = st;
  bool rest_queued = false;   // an update of the rest is under way on the main stream, join_ev behind it
  bool diag_done = true;  // the first diagonal block was factorised with the system matrix (ds_gram_begin)
  bool panel_ready = true;   // gs->panel[pbuf] holds the rows of the current panel (the first one's since it was built)
  int pbuf = 0;
  int64_t j0 = 0;
  while (j0 < n) {
    if (mid && j0 == mid_at) DS_HIP(ctx, hipEventRecord(mid, st));   // (the launch before has left block j0 factorised)
    const bool super = rows_total - j0 - kSuperCols > kFuseMaxRows && n - j0 >= kSuperCols + NB;
    if (super) {
      if (chain == st) {   // the first one
        chain = ctx->side;
        DS_HIP(ctx, hipEventRecord(ctx->fork_ev, st));
        DS_HIP(ctx, hipStreamWaitEvent(chain, ctx->fork_ev, 0));
      }
      for (int b = 0; b < kSuperCols / NB; ++b) {
        const int64_t jb = j0 + (int64_t)b * NB;
        double* li = linv + (size_t)(jb / NB) * NB * NB;
        // the launch before has factorised the diagonal block on the way
        const unsigned tt = nblocks(rows_total - jb - NB, kTile);
        const unsigned inside = (unsigned)(kSuperCols / NB - 1 - b);  // block columns of the super-panel still ahead
        if (inside > 0) {
          hipLaunchKernelGGL(chol_step_kernel, dim3(inside, tt), dim3(kThreads), 0, chain, M, ld, rows_total, n, jb, li, li + (size_t)NB * NB,
                             gs->flag, gs->panel[pbuf], gs->panel[pbuf ^ 1]);
          pbuf ^= 1;
        } else {
          hipLaunchKernelGGL(chol_panel_kernel, dim3(tt), dim3(kThreads), 0, chain, M, ld, rows_total, jb, NB, li);
        }
      }
      const int64_t base = j0 + kSuperCols;
      if (rest_queued) DS_HIP(ctx, hipStreamWaitEvent(chain, ctx->join_ev, 0));
      hipLaunchKernelGGL(chol_update_next_kernel<(int)kSuperCols>, dim3((unsigned)(kSuperCols / NB), nblocks(rows_total - base, kTile)),
                         dim3(kThreads), 0, chain, M, ld, rows_total, n, j0, base, linv + (size_t)(base / NB) * NB * NB, gs->flag, gs->panel[pbuf]);
      DS_HIP(ctx, hipEventRecord(ctx->fork_ev, chain));
      DS_HIP(ctx, hipStreamWaitEvent(st, ctx->fork_ev, 0));
      const int64_t tw = (rows_total - base - kSuperCols + kWideTile - 1) / kWideTile;   // (kFuseMaxRows rows are left at least)
      const int64_t tiles = tw * (tw + 1) / 2, slots = ctx->num_cus > 2 * kWideSpare ? ctx->num_cus - kWideSpare : ctx->num_cus;
      hipLaunchKernelGGL(chol_update_wide_kernel<(int)kSuperCols>, dim3((unsigned)(tiles < slots ? tiles : slots)), dim3(kWideThreads), 0, st,
                         M, ld, rows_total, n, j0, base + kSuperCols, (int)tw, (int)tiles);
      DS_HIP(ctx, hipEventRecord(ctx->join_ev, st));
      rest_queued = true;
      j0 += kSuperCols;
      continue;   // (diag_done stays true)
    }
    if (chain != st) {   // behind the last super-panel everything is on the main stream again
      DS_HIP(ctx, hipEventRecord(ctx->fork_ev, chain));
      DS_HIP(ctx, hipStreamWaitEvent(st, ctx->fork_ev, 0));
      chain = st;
    }
    const int nb = (int)(n - j0 < NB ? n - j0 : NB);
    double* li = linv + (size_t)(j0 / NB) * NB * NB;
    // a diagonal block has a launch of its own only if the update before it did not factorise it already
    if (!diag_done) hipLaunchKernelGGL(chol_diag_kernel, dim3(1), dim3(kThreads), 0, st, M, ld, j0, nb, li, gs->flag,
                                       (const double*)nullptr, 0);
    diag_done = false;
    const int64_t rest = rows_total - j0 - nb;
    // One launch per step where its workgroups, one to a compute unit, run in a single round; above that the panel's own
    // launch is the cheaper one (2,048 rows: 53 us in one launch, 24 in two; 1,408 rows: 24 and 22).
    const int64_t step_tiles = nblocks(rest, kTile);
    if (n - j0 - nb > 0 && rest <= kFuseMaxRows && step_tiles * (step_tiles + 1) / 2 <= ctx->num_cus) {  // nb == NB here
      const unsigned tt = (unsigned)step_tiles;
      if (!panel_ready) {
        hipLaunchKernelGGL(copy_panel_kernel, dim3(nblocks(rest * NB, 256)), dim3(256), 0, st, M, ld, rows_total, j0 + NB, j0, n,
                           gs->panel[pbuf]);
        panel_ready = true;
      }
      hipLaunchKernelGGL(chol_step_kernel, dim3(tt, tt), dim3(kThreads), 0, st, M, ld, rows_total, n, j0, li,
                         li + (size_t)NB * NB, gs->flag, gs->panel[pbuf], gs->panel[pbuf ^ 1]);
      pbuf ^= 1;
      diag_done = true;
      j0 += nb;
      continue;
    }
    panel_ready = false;
    if (rest > 0) hipLaunchKernelGGL(chol_panel_kernel, dim3(nblocks(rest, kTile)), dim3(kThreads), 0, st, M, ld, rows_total, j0, nb, li);
    if (n - j0 - nb > 0) {
      const unsigned tt = nblocks(rest, kTile);
      if (rest <= kFuseMaxRows) {
        hipLaunchKernelGGL(chol_update_kernel<true>, dim3(tt, tt), dim3(kThreads), 0, st, M, ld, rows_total, n, j0, nb,
                           li + (size_t)NB * NB, gs->flag);
        diag_done = true;
      } else {
        hipLaunchKernelGGL(chol_update_kernel<false>, dim3(tt, tt), dim3(kThreads), 0, st, M, ld, rows_total, n, j0, nb,
                           (double*)nullptr, gs->flag);
      }
    }
    j0 += nb;
  }
  DS_HIP(ctx, hipGetLastError());
  return ds_kernel_mark(ctx, 2, 1);
}

// one launch of a triangular solve: `blocks` blocks from column J on, `pieces` blocks of 64 entries still to be solved
static void launch_forward(hipStream_t st, int blocks, int64_t pieces, const ds_gram_state* gs, int64_t J, double* v, double* out) {
  static_assert(kSolveBlocks == 4, "one instance per number of blocks");
  void (*const kern)(const double*, int64_t, int64_t, int64_t, const double*, double*, double*) =
      blocks == 4 ? chol_forward_kernel<4> : blocks == 3 ? chol_forward_kernel<3> : blocks == 2 ? chol_forward_kernel<2> : chol_forward_kernel<1>;
  hipLaunchKernelGGL(kern, dim3((unsigned)(pieces > 0 ? pieces : 1)), dim3(kSolveThreads), 0, st, gs->M, gs->ld, gs->n, J, gs->linv, v, out);
}
static void launch_back(hipStream_t st, int blocks, int64_t pieces, const ds_gram_state* gs, int64_t J, double* v, const float* y01,
                        float* phi) {
  void (*const kern)(const double*, int64_t, int64_t, int64_t, const double*, double*, const float*, float*) =
      blocks == 4 ? chol_back_kernel<4> : blocks == 3 ? chol_back_kernel<3> : blocks == 2 ? chol_back_kernel<2> : chol_back_kernel<1>;
  hipLaunchKernelGGL(kern, dim3((unsigned)(pieces > 0 ? pieces : 1)), dim3(kSolveThreads), 0, st, gs->M, gs->ld, gs->n, J, gs->linv, v, y01,
                     phi);
}

// Whether a factorisation may run beside the inference, ahead of the right-hand side: no super-panels, whose wide updates fill the
// GPU and want the main stream.
bool ds_gram_ahead_applies(int64_t n) { return n - kSuperCols <= kFuseMaxRows; }

// Part 2 without the right-hand side (ds_gram_ahead_applies); `mid` as for gram_factor.
int ds_gram_factor_ahead(ds_ctx* ctx, const ds_gram_state* gs, hipEvent_t mid) {
  return gs->n <= kSmallMax ? DS_OK : gram_factor(ctx, gs, gs->n, mid);   // (ds_gram_begin has factorised a single block)
}

static int gram_check(ds_ctx* ctx, const ds_gram_state* gs) {
  DS_HIP(ctx, hipMemcpyAsync(ctx->h_mail, gs->flag, sizeof(int), hipMemcpyDeviceToHost, ctx->stream));
  DS_HIP(ctx, hipStreamSynchronize(ctx->stream));
  if (*(int*)ctx->h_mail != 0)
    return ds_fail(ctx, DS_ESINGULAR, "Cholesky met a non-positive pivot: the sampled rows do not determine all %lld players", (long long)gs->n);
  return DS_OK;
}

// Part 3: right-hand side from y, factorisation (unless it runs ahead on another stream: `mid` and `done` are its events), back
// substitution.
int ds_gram_finish(ds_ctx* ctx, const ds_gram_state* gs, const uint64_t* Z, const float* w, const float* y, float* phi,
                   int defer_check, hipEvent_t mid, hipEvent_t done) {
  hipStream_t st = ctx->stream;
  const int64_t n = gs->n, k = gs->k, R = gs->R, RW = gs->RW, ld = gs->ld;
  if (n <= kSmallMax) {
    const unsigned parts = small_parts(R);
    hipLaunchKernelGGL(small_rhs_kernel, dim3(parts), dim3(kSmallThreads), 0, st, Z, w, y, R, gs->paired, (int)n, gs->t);
    if (done) DS_HIP(ctx, hipStreamWaitEvent(st, done, 0));
    hipLaunchKernelGGL(small_solve_kernel, dim3(1), dim3(kThreads), 0, st, gs->t, (int)parts, (int)n, gs->linv, y, phi);
    DS_HIP(ctx, hipGetLastError());
    return defer_check ? DS_OK : gram_check(ctx, gs);
  }
  DS_TRY(ds_row_prep(ctx, Z, k, n, gs->paired, w, y, gs->sz, gs->t, gs->sqw, gs->wc));
  hipLaunchKernelGGL(used_row_rhs_kernel, dim3(nblocks(R, 256)), dim3(256), 0, st, gs->wc, gs->t, R, gs->paired, gs->gc);
  DS_TRY(ds_bit_spmv(ctx, gs->Zt, n, R, RW, 0, 1, gs->gc, gs->c));  // c_j = sum over the rows containing j of gc
  hipLaunchKernelGGL(build_rhs_kernel, dim3(1), dim3(kThreads), 0, st, gs->c, n, ld, gs->M, gs->panel[0]);
  DS_HIP(ctx, hipGetLastError());
  double* const rhs = gs->M + n * ld;
  double* v = rhs;   // L^-1 rhs
  if (done) {
    v = gs->c;       // (the sums have gone into the right-hand side)
    const int64_t groups = (gs->nblk + kSolveBlocks - 1) / kSolveBlocks;
    for (int64_t g = 0; g < groups; ++g) {
      if (g == 0 && groups > 1) DS_HIP(ctx, hipStreamWaitEvent(st, mid, 0));
      if (g == groups - 1) DS_HIP(ctx, hipStreamWaitEvent(st, done, 0));
      const int64_t first = g * kSolveBlocks, last = first + kSolveBlocks < gs->nblk ? first + kSolveBlocks : gs->nblk;
      launch_forward(st, (int)(last - first), gs->nblk - last, gs, first * NB, rhs, v);
    }
  } else {
    DS_TRY(gram_factor(ctx, gs, n + 1, nullptr));
  }
  for (int64_t last = gs->nblk; last > 0;) {   // blocks first .. last - 1 per launch
    const int64_t first = (last - 1) / kSolveBlocks * kSolveBlocks;
    launch_back(st, (int)(last - first), first, gs, first * NB, v, y, phi);
    last = first;
  }
  DS_HIP(ctx, hipGetLastError());
  return defer_check ? DS_OK : gram_check(ctx, gs);   // (deferred: the caller reads gs->flag back with its own results)
}

int ds_solve_gram_chol(ds_ctx* ctx, int64_t n, int64_t k, const uint64_t* Z, const float* w, const float* y, int paired,
                       float* phi) {
  ds_gram_state gs;
  DS_TRY(ds_gram_alloc(ctx, n, k, paired, &gs));
  DS_TRY(ds_gram_begin(ctx, &gs, Z, w));
  return ds_gram_finish(ctx, &gs, Z, w, y, phi, 0, nullptr, nullptr);
}
