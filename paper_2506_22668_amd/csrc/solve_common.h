// Helpers shared by the two least-squares solvers (internal).
#pragma once
#include "internal.h"

// sz[i] = |S_i|, t[i] = y_i - y_0 - ((y_1-y_0)/n)|S_i| (0 for the two constraint rows),
// sqw[i] = sqrt(w_i), wc[i] = w_i (both 0 for the two constraint rows); paired (k even): row 2r+1 is row 2r's complement
// and is not read
int ds_row_prep(ds_ctx* ctx, const uint64_t* Z, int64_t k, int64_t n, int paired, const float* w, const float* y, int32_t* sz,
                double* t, double* sqw, float* wc);
// out[cols x ceil(rows/64)] = transpose of the rows row_first + i*row_step (i < rows) of `in`; out_stride: words from one row of
// `out` to the next, ceil(rows/64) unless given
int ds_bit_transpose(ds_ctx* ctx, const uint64_t* in, int64_t rows, int64_t cols, int64_t in_stride, int64_t row_first,
                     int64_t row_step, uint64_t* out, int64_t out_stride = 0);
// the same transpose of the rows i * row_step (i < rows), laid out by blocks of 64 of them: out[b * 64*ceil(cols/64) + j] =
// bits of column j in the rows 64b .. 64b+63 of that selection (rows past the last and columns past `cols` read as zero)
int ds_bit_transpose_blocks(ds_ctx* ctx, const uint64_t* in, int64_t rows, int64_t cols, int64_t in_stride, int64_t row_step,
                            uint64_t* out);
// out[i] = sum of x[j] over the set bits j < cols of row (row_first + i*row_step) of B, i < rows (fp64)
int ds_bit_spmv(ds_ctx* ctx, const uint64_t* B, int64_t rows, int64_t cols, int64_t stride, int64_t row_first,
                int64_t row_step, const double* x, double* out);
// ---- products of the CGLS matrix of a large game in fixed point (exact integer sums) ----
// The fixed point of a vector is 2^-54 of its largest entry, from the partial maxima of |x| (bit patterns, max_parts[0..parts), at most
// 1,024; left by the kernel that wrote x, or by ds_vec_absmax); scal[0] becomes the power of two that scales integer
// results back. The sparse rows' product comes first and leaves the digits for the dense rows' product on the way; without sparse
// rows ds_mm_quantize does.
//
// Dense rows on the matrix cores (x split into digits); out = (addend or 0) + result. A plan fixes
// the launch shape and the scratch of one (rows, cols) shape: ds_bit_spmv_mm_ws_bytes bytes at `ws`, which
// ds_bit_spmv_mm_prepare initialises (on ctx->stream).
struct ds_mm_plan {
  int64_t rows, cols, row_groups, n_chunks, groups, cpg;
  int64_t even_wgs;  // workgroups of an even cut (groups: the slots of a row group's sums); 0: a workgroup per row group and column group
  int8_t* D;         // the vector's digits, chunk by chunk
  longlong2* partial;  // [groups][rows]: a row's sum in units of the vector's fixed point is 2^24 x + y
};
size_t ds_bit_spmv_mm_ws_bytes(const ds_ctx* ctx, int64_t rows, int64_t cols);
int ds_bit_spmv_mm_prepare(ds_ctx* ctx, int64_t rows, int64_t cols, void* ws, ds_mm_plan* plan);
int ds_vec_absmax(ds_ctx* ctx, const double* x, int64_t len, unsigned long long* max_parts, int parts);
int ds_mm_quantize(ds_ctx* ctx, const ds_mm_plan* plan, const double* x, const unsigned long long* max_parts, int parts, double* scal);
// out == nullptr: the per-group digit sums are left for the caller's own kernel to add up (ds_mm_sum below)
int ds_bit_spmv_mm_product(ds_ctx* ctx, const ds_mm_plan* plan, const uint64_t* B, int64_t stride, int64_t row_first,
                           int64_t row_step, const double* scal, const double* addend, double* out);

// Sparse rows as 2-D tiles of (row, column) entries: one list serves both products. Built from the index lists of the
// rows (off = exclusive prefix sums of the row sizes, idx = ascending columns); rows must not hold more than
// max_row_size entries. ws: ds_tile_ws_bytes bytes. The plan keeps `idx`'s memory (the entries end up there) and
// `off` is free after the call.
struct ds_tile_plan {
  int64_t rows, cols, nnz;
  int32_t nrb, ncb, nga, gf, cpg;   // row blocks, column chunks, adjoint row-block groups, forward chunk groups (of cpg)
  int sh_f, sh_a;                   // bits dropped (rounded) from the 2^-54-scaled integers so that the sums fit 63 bits
  int32_t *rb_start, *ga_start, *tile_off;
  uint32_t* ent;
  long long* partial;
};
size_t ds_tile_ws_bytes(const ds_ctx* ctx, int64_t rows, int64_t cols, int64_t nnz);
int ds_tile_build(ds_ctx* ctx, int64_t rows, int64_t cols, int64_t nnz, int64_t max_row_size, const int32_t* off,
                  int32_t* idx, void* ws, ds_tile_plan* plan);
// forward: out[r] = sum of x[c] over the entries of row r (x: cols entries);
// adjoint: out[c] = sum of x[r] over the entries of column c (x: rows entries)
// planes (or nullptr): the dense rows' plan, whose digits of x_planes are made on the way
// out == nullptr: the per-group partial vectors are left for the caller's own kernel to add up (ds_tile_sum below)
int ds_tile_spmv(ds_ctx* ctx, const ds_tile_plan* plan, int adjoint, const double* x, const unsigned long long* max_parts, int parts,
                 const ds_mm_plan* planes, const double* x_planes, double* scal, double* out);

// Where the integer results of one product lie before they are added up, for kernels that consume them directly
// (groups == 0: that part of the matrix is empty).
struct ds_fixed_view {
  const long long* tile_partial;  // [tile_groups][tile_len]
  int64_t tile_len;
  int tile_groups, tile_sh;
  const longlong2* mm_partial;    // [mm_groups][mm_rows]
  int64_t mm_rows;
  int mm_groups;
};
static inline ds_fixed_view ds_fixed_view_of(const ds_tile_plan* t, const ds_mm_plan* m, int adjoint) {
  ds_fixed_view v;
  const bool has_t = t && t->rows > 0 && t->nnz > 0, has_m = m && m->rows > 0;
  v.tile_partial = has_t ? t->partial : nullptr;
  v.tile_len = has_t ? (adjoint ? t->cols : t->rows) : 0;
  v.tile_groups = has_t ? (adjoint ? t->nga : t->gf) : 0;
  v.tile_sh = has_t ? (adjoint ? t->sh_a : t->sh_f) : 0;
  v.mm_partial = has_m ? m->partial : nullptr;
  v.mm_rows = has_m ? m->rows : 0;
  v.mm_groups = has_m ? (int)m->groups : 0;
  return v;
}
#ifdef __HIPCC__
// ---- the vectors of the products in fixed point ----
// the largest m of a workgroup, in every thread; wm: a word of LDS per wave, of the call's own
template <int THREADS>
__device__ __forceinline__ void ds_block_max(unsigned long long& m, unsigned long long* wm) {
  for (int o = 32; o > 0; o >>= 1) {
    const unsigned long long t = __shfl_xor(m, o, 64);
    m = t > m ? t : m;
  }
  if ((threadIdx.x & 63) == 0) wm[threadIdx.x >> 6] = m;
  __syncthreads();
#pragma unroll
  for (int i = 0; i < THREADS / 64; ++i) m = wm[i] > m ? wm[i] : m;
}
struct ds_fixed_point {
  int f;         // x 2^f is below 2^54 in magnitude
  bool finite;   // a vector with a non-finite entry: zeros, and NaN for the way back (the products are NaN everywhere)
  __device__ __forceinline__ long long of(double x) const { return finite ? __double2ll_rn(ldexp(x, f)) : 0ll; }
  __device__ __forceinline__ double back() const { return finite ? ldexp(1.0, -f) : __longlong_as_double(0x7ff8000000000000ll); }
};
// Every workgroup goes through the partial maxima itself: with one atomic per workgroup on a single slot instead, the
// kernel that wrote the vector spent 8 us on a thousand atomics.
template <int THREADS>
__device__ __forceinline__ ds_fixed_point ds_fixed_point_of(const unsigned long long* max_parts, int parts) {
  __shared__ unsigned long long wm[THREADS / 64];
  unsigned long long m = 0;
  for (int i = threadIdx.x; i < parts; i += THREADS) m = max_parts[i] > m ? max_parts[i] : m;
  ds_block_max<THREADS>(m, wm);
  const double mx = __longlong_as_double((long long)m);
  ds_fixed_point fp;
  fp.finite = mx < __longlong_as_double(0x7ff0000000000000ll);
  int e = 0;
  if (fp.finite && mx > 0.0) frexp(mx, &e);   // mx < 2^e
  fp.f = 54 - e;
  return fp;
}
// The digits that the dense rows' product reads (described there). A half operand, 16 columns, is a thread's share: 96 bits of every
// plane. Half operand id: (chunk, 128 columns, j, half); its columns are 4 apart.
constexpr int kMmChunk = 1024;                       // columns per step of the product
constexpr int kMmDigits = 14;                        // base 16
constexpr int kMmPlanes = kMmDigits + 1;             // and the plane of ones
constexpr int kMmOperand = 24;                       // bytes of a lane's B operand: 32 elements of six bits
constexpr int kMmPlaneBytes = kMmChunk * 6 / 8;      // of a chunk: [512 columns][lane group of 128][j] operands
constexpr int kMmChunkBytes = kMmPlanes * kMmPlaneBytes;
constexpr int kMmHalf = 16;
constexpr int kMmHalves1024 = kMmChunk / kMmHalf;    // of a chunk
__device__ __forceinline__ int64_t ds_mm_half_column(int64_t id) { return (id >> 3) * 128 + ((id & 1) << 6) + ((id >> 1) & 3); }
__device__ __forceinline__ void ds_mm_half_operand(const double* x, int64_t n, int64_t id, double (&xv)[kMmHalf]) {
  const int64_t col0 = ds_mm_half_column(id);
#pragma unroll
  for (int i = 0; i < kMmHalf; ++i) {
    const int64_t col = col0 + 4 * i;
    xv[i] = x[col < n ? col : n - 1];
  }
}
__device__ __forceinline__ void ds_mm_store_digits(const double (&xv)[kMmHalf], int64_t n, int64_t id, const ds_fixed_point& fp, int8_t* D) {
  const int64_t col0 = ds_mm_half_column(id);
  unsigned long long q[kMmHalf];
#pragma unroll
  for (int i = 0; i < kMmHalf; ++i) q[i] = col0 + 4 * i < n ? (unsigned long long)(fp.of(xv[i]) + (1ll << 54)) : 0ull;
  uint32_t* const out = (uint32_t*)(D + (id >> 6) * kMmChunkBytes + ((id >> 3) & 7) * (4 * kMmOperand) + ((id >> 1) & 3) * kMmOperand +
                                    (id & 1) * (kMmOperand / 2));
#pragma unroll
  for (int d = 0; d < kMmPlanes; ++d) {
    uint32_t w[3] = {0u, 0u, 0u};
#pragma unroll
    for (int i = 0; i < kMmHalf; ++i) {
      const uint32_t digit = d < kMmDigits ? (uint32_t)(q[i] >> (4 * d)) & 15u : (col0 + 4 * i < n ? 1u : 0u);
      const int at = 6 * i, sh = at & 31;
      w[at >> 5] |= digit << sh;
      if (sh > 28) w[(at >> 5) + 1] |= digit >> (32 - sh);
    }
#pragma unroll
    for (int u = 0; u < 3; ++u) out[d * (kMmPlaneBytes / 4) + u] = w[u];
  }
}

// The sums over the groups are exact integers, so they may be split over T lanes in any way: lane `sub` (0 <= sub < T)
// adds the groups sub, sub + T, ... (four loads in flight), the lanes' integers are added, and one rounding ends it.
// tile product, entry i: the groups as two 32-bit halves, so that the total may exceed 63 bits
__device__ __forceinline__ void ds_tile_sum_part(const long long* partial, int64_t len, int groups, int64_t i, int sub, int T,
                                                 long long& hi, long long& lo) {
  int g = sub;
  for (; g + 3 * T < groups; g += 4 * T) {
    const long long* q = partial + (int64_t)g * len + i;
    const int64_t st = (int64_t)T * len;
    const long long p0 = q[0], p1 = q[st], p2 = q[2 * st], p3 = q[3 * st];
    hi += (p0 >> 32) + (p1 >> 32) + (p2 >> 32) + (p3 >> 32);
    lo += (p0 & 0xffffffffll) + (p1 & 0xffffffffll) + (p2 & 0xffffffffll) + (p3 & 0xffffffffll);
  }
  for (; g < groups; g += T) {
    const long long p = partial[(int64_t)g * len + i];
    hi += p >> 32;
    lo += p & 0xffffffffll;
  }
}
// ... times 2^sh
__device__ __forceinline__ double ds_tile_sum_finish(long long hi, long long lo, int sh) {
  return ((double)hi * 4294967296.0 + (double)lo) * (double)(1ll << sh);
}
__device__ __forceinline__ double ds_tile_sum(const long long* partial, int64_t len, int groups, int sh, int64_t i) {
  long long hi = 0, lo = 0;
  ds_tile_sum_part(partial, len, groups, i, 0, 1, hi, lo);
  return ds_tile_sum_finish(hi, lo, sh);
}
// matrix-core product, row r: 2^24 hi + lo
__device__ __forceinline__ void ds_mm_sum_part(const longlong2* partial, int64_t rows, int groups, int64_t r, int sub, int T,
                                               long long& hi, long long& lo) {
  int g = sub;
  for (; g + 3 * T < groups; g += 4 * T) {
    const longlong2* p = partial + (int64_t)g * rows + r;
    const int64_t st = (int64_t)T * rows;
    const longlong2 a = p[0], b = p[st], c = p[2 * st], d = p[3 * st];
    hi += a.x + b.x + c.x + d.x;
    lo += a.y + b.y + c.y + d.y;
  }
  for (; g < groups; g += T) {
    const longlong2 a = partial[(int64_t)g * rows + r];
    hi += a.x;
    lo += a.y;
  }
}
__device__ __forceinline__ double ds_mm_sum_finish(long long hi, long long lo) { return (double)hi * 16777216.0 + (double)lo; }
__device__ __forceinline__ double ds_mm_sum(const longlong2* partial, int64_t rows, int groups, int64_t r) {
  long long hi = 0, lo = 0;
  ds_mm_sum_part(partial, rows, groups, r, 0, 1, hi, lo);
  return ds_mm_sum_finish(hi, lo);
}
// 64 x 64 bits, a row per lane, transposed: bit i of lane j = bit j of lane i. Six rounds of swapping bit blocks with the
// lane 32, 16, ... 1 away.
__device__ __forceinline__ uint64_t ds_transpose64_in_wave(uint64_t x, int lane) {
  const uint64_t masks[6] = {0x00000000FFFFFFFFull, 0x0000FFFF0000FFFFull, 0x00FF00FF00FF00FFull,
                             0x0F0F0F0F0F0F0F0Full, 0x3333333333333333ull, 0x5555555555555555ull};
#pragma unroll
  for (int s = 0; s < 6; ++s) {
    const int j = 32 >> s;
    const uint64_t m = masks[s];
    const uint32_t lo = (uint32_t)__shfl_xor((int)(uint32_t)x, j, 64), hi = (uint32_t)__shfl_xor((int)(uint32_t)(x >> 32), j, 64);
    const uint64_t t = ((uint64_t)hi << 32) | lo;
    // rows whose index has bit j clear keep their low bit blocks and take the partner's low blocks as their high
    // ones; the others keep their high blocks and take the partner's high blocks as their low ones
    x = (lane & j) ? (((t >> j) & m) | (x & ~m)) : ((x & m) | ((t & m) << j));
  }
  return x;
}
#endif

// index lists of the set bits of rows (off = exclusive prefix sums of the row sizes)
int ds_rows_to_csr(ds_ctx* ctx, const uint64_t* B, int64_t rows, int64_t cols, int64_t stride, int64_t row_first,
                   int64_t row_step, const int32_t* off, int32_t* idx);

// Sum of a over the 64 lanes, the same value in every lane: the additions of `for (o = 32; o > 0; o >>= 1) a +=
// __shfl_xor(a, o, 64)`, to the bit, without its LDS round trips (two ds_bpermute per step and double, each a wait of
// some 100 cycles). Lanes 32 and 16 away are reached by the half and row swaps; from there on the values repeat
// within a row of 16, so that rotations stand in for the lanes 8 and 4 away.
__device__ __forceinline__ double ds_wave_sum(double a) {
  auto swapped = [](double v, bool half, double& w) {
    typedef unsigned u2 __attribute__((ext_vector_type(2)));
    const unsigned lo = (unsigned)__double2loint(v), hi = (unsigned)__double2hiint(v);
    const u2 l = half ? __builtin_amdgcn_permlane32_swap(lo, lo, false, false) : __builtin_amdgcn_permlane16_swap(lo, lo, false, false);
    const u2 h = half ? __builtin_amdgcn_permlane32_swap(hi, hi, false, false) : __builtin_amdgcn_permlane16_swap(hi, hi, false, false);
    w = __hiloint2double((int)h.y, (int)l.y);
    return __hiloint2double((int)h.x, (int)l.x);
  };
  double b;
  a = swapped(a, true, b);    // a, b: the pair {x[l], x[l ^ 32]} in one order or the other
  a += b;
  a = swapped(a, false, b);
  a += b;
#define DS_DPP_ADD(ctrl)                                                                                              \
  a += __hiloint2double(__builtin_amdgcn_update_dpp(0, __double2hiint(a), ctrl, 0xf, 0xf, false),                     \
                        __builtin_amdgcn_update_dpp(0, __double2loint(a), ctrl, 0xf, 0xf, false))
  DS_DPP_ADD(0x128);   // row_ror:8
  DS_DPP_ADD(0x124);   // row_ror:4
  DS_DPP_ADD(0x4e);    // quad_perm [2,3,0,1]
  DS_DPP_ADD(0xb1);    // quad_perm [1,0,3,2]
#undef DS_DPP_ADD
  return a;
}
