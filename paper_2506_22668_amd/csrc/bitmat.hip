// Helpers on bit-packed mask matrices shared by the two solvers: per-row
// regression targets and the bit-matrix transpose.
#include "internal.h"
#include "solve_common.h"
#include "mm_split.h"

namespace {
constexpr int kThreads = 256;

// One wave per row (paired: per pair of rows 2r, 2r+1, of which only the first is read, the other being its
// complement): size |S_i| = popcount, target t_i = y_i - y_0 - (delta/n)|S_i| (the regression re-centred on the
// efficiency constraint), sqrt(w_i), and w_i itself with the two constraint rows zeroed. Bound by the read of the mask
// matrix (60,000 paired rows of 300,007 players: 425 us when both were read, at
// 5.3 TB/s; now about half).
__global__ __launch_bounds__(kThreads) void row_prep_kernel(const uint64_t* Z, int64_t k, int64_t W, int64_t n, int paired,
                                                            const float* w, const float* y, int32_t* sz, double* t,
                                                            double* sqw, float* wc) {
  const int lane = threadIdx.x & 63;
  const int64_t wave = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
  const int64_t nwaves = ((int64_t)gridDim.x * blockDim.x) >> 6;
  const double f0 = (double)y[0], delta = (double)y[1] - (double)y[0];
  const uint64_t tail = (n & 63) ? ((1ull << (n & 63)) - 1ull) : ~0ull;
  const int per = paired ? 2 : 1;
  for (int64_t i0 = wave * per; i0 < k; i0 += nwaves * per) {
    int c = 0;
    for (int64_t wd = lane; wd < W; wd += 64) c += __popcll(Z[i0 * W + wd] & (wd == W - 1 ? tail : ~0ull));
    for (int o = 32; o > 0; o >>= 1) c += __shfl_xor(c, o, 64);
    if (lane < per) {
      const int64_t i = i0 + lane;
      const int ci = lane == 0 ? c : (int)n - c;
      sz[i] = ci;
      t[i] = i < 2 ? 0.0 : (double)y[i] - f0 - (delta / (double)n) * (double)ci;
      sqw[i] = i < 2 ? 0.0 : sqrt((double)w[i]);
      wc[i] = i < 2 ? 0.f : w[i];
    }
  }
}

// Transpose a bit matrix: in[rows x Win words] (row stride in_stride words, rows taken as row_first + i*row_step)
// -> out[cols x Wout words], Wout = ceil(rows/64); bit i of out row j = bit j of in row i.
// A workgroup of 512 threads takes a tile of 512 rows x 512 columns through LDS: every row is read in 64 contiguous
// bytes and every output row written in 64 contiguous bytes (one wave per 64x64 block with 8-byte accesses, the first
// version, left most of every cache line unused: 0.3 TB/s). Each wave transposes eight of the tile's 64x64 blocks in
// registers: lane = row, six rounds of swapping bit blocks with the lane 32, 16, ... 1 away.
constexpr int kTrThreads = 512;
constexpr int kTrPitch = 9;  // 64-bit words per LDS row of 8: lanes that read one word column of 64 rows spread over the banks

__global__ __launch_bounds__(kTrThreads) void bit_transpose_kernel(const uint64_t* in, int64_t rows, int64_t cols,
                                                                   int64_t in_stride, int64_t row_first, int64_t row_step,
                                                                   uint64_t* out, int64_t Wout, int64_t tiles_c, int block_major) {
  __shared__ uint64_t tin[512 * kTrPitch];
  __shared__ uint64_t tout[512 * kTrPitch];
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const int64_t Win = (cols + 63) / 64;
  const int64_t tr = blockIdx.x / tiles_c, tc = blockIdx.x % tiles_c;   // consecutive workgroups walk along a row block
  const int64_t r0 = tr * 512, w0 = tc * 8;
  // load: 8 lanes per row (64 contiguous bytes), 64 rows per step
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    const int r = k * 64 + (t >> 3), w = t & 7;
    uint64_t v = 0;
    if (r0 + r < rows && w0 + w < Win) v = in[(row_first + (r0 + r) * row_step) * in_stride + w0 + w];
    tin[r * kTrPitch + w] = v;
  }
  __syncthreads();
  // wave `wave` transposes the blocks (row block rbi, word column wave) for the eight row blocks
#pragma unroll
  for (int rbi = 0; rbi < 8; ++rbi) {
    const uint64_t x = ds_transpose64_in_wave(tin[(rbi * 64 + lane) * kTrPitch + wave], lane);
    tout[(wave * 64 + lane) * kTrPitch + rbi] = x;   // lane = column within the word column, word = row block
  }
  __syncthreads();
  if (block_major) {
    // out[row block][column] (Win * 64 columns per row block): a wave writes the 64 columns of one row block, 512
    // contiguous bytes
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const int c = k * 64 + lane, w = wave;
      const int64_t col = w0 * 64 + c, ow = tr * 8 + w;
      if (col < Win * 64 && ow < Wout) out[ow * (Win * 64) + col] = tout[c * kTrPitch + w];
    }
    return;
  }
  // store: 8 lanes per output row (64 contiguous bytes)
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    const int c = k * 64 + (t >> 3), w = t & 7;
    const int64_t col = w0 * 64 + c, ow = tr * 8 + w;
    if (col < cols && ow < Wout) out[col * Wout + ow] = tout[c * kTrPitch + w];
  }
}
// out[i] = sum over the set bits j of row i of x[j] (fp64).
// The vector is staged through LDS in chunks of 8192 columns, so the one gather per set bit is an
// LDS read instead of an L2 transaction; the matrix is streamed once, each (row, chunk) segment
// being 1 KB of contiguous words. A wave owns 16 rows and keeps their partial sums in registers
// across all chunks (one cross-lane reduction per row at the very end); per chunk it first loads
// the two words of each of its rows into registers (16 independent row loads in flight), then walks
// their set bits. The LDS copy is pitched 65 doubles per 64-column word to spread the banks.
constexpr int kSpmvChunkWords = 128;
constexpr int kSpmvRowsPerWave = 16;
constexpr int kSpmvPitch = 65;

__global__ __launch_bounds__(kThreads) void bit_spmv_kernel(const uint64_t* B, int64_t rows, int64_t cols, int64_t stride,
                                                            int64_t row_first, int64_t row_step, const double* x,
                                                            double* out) {
  __shared__ double xs[kSpmvChunkWords * kSpmvPitch];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int64_t Wc = (cols + 63) / 64;
  const uint64_t tail = (cols & 63) ? ((1ull << (cols & 63)) - 1ull) : ~0ull;
  // blocks walk the rows from the end: mask rows are sorted by size, so the long (dense) rows start first
  const int64_t row0 = (int64_t)(gridDim.x - 1 - blockIdx.x) * (kSpmvRowsPerWave * (kThreads / 64)) + (int64_t)wave * kSpmvRowsPerWave;
  double acc[kSpmvRowsPerWave];
#pragma unroll
  for (int i = 0; i < kSpmvRowsPerWave; ++i) acc[i] = 0.0;
  const double* xa = xs + (2 * lane) * kSpmvPitch;
  const double* xb = xs + (2 * lane + 1) * kSpmvPitch;
  for (int64_t c0 = 0; c0 < Wc; c0 += kSpmvChunkWords) {
    __syncthreads();
    for (int i = tid; i < kSpmvChunkWords * 64; i += kThreads) {
      const int64_t col = c0 * 64 + i;
      xs[(i >> 6) * kSpmvPitch + (i & 63)] = col < cols ? x[col] : 0.0;
    }
    __syncthreads();
    const int64_t wa = c0 + 2 * lane, wb = wa + 1;
    uint64_t w0[kSpmvRowsPerWave], w1[kSpmvRowsPerWave];
#pragma unroll
    for (int i = 0; i < kSpmvRowsPerWave; ++i) {
      const int64_t r = row0 + i;
      w0[i] = 0ull;
      w1[i] = 0ull;
      if (r < rows) {
        const uint64_t* p = B + (row_first + r * row_step) * stride;
        if (wa < Wc) w0[i] = p[wa] & (wa == Wc - 1 ? tail : ~0ull);  // padding bits name no column
        if (wb < Wc) w1[i] = p[wb] & (wb == Wc - 1 ? tail : ~0ull);
      }
    }
    // four rows (eight words) are walked together so that eight LDS reads are in flight
#pragma unroll
    for (int i = 0; i < kSpmvRowsPerWave; i += 4) {
      uint64_t m[8] = {w0[i], w1[i], w0[i + 1], w1[i + 1], w0[i + 2], w1[i + 2], w0[i + 3], w1[i + 3]};
      double s[8] = {0, 0, 0, 0, 0, 0, 0, 0};
      while (m[0] | m[1] | m[2] | m[3] | m[4] | m[5] | m[6] | m[7]) {
        double v[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) {
          const bool live = m[q] != 0ull;
          const int bit = live ? __ffsll((long long)m[q]) - 1 : 0;
          const double xv = (q & 1) ? xb[bit] : xa[bit];
          v[q] = live ? xv : 0.0;
          m[q] &= m[q] - 1;  // 0 stays 0
        }
#pragma unroll
        for (int q = 0; q < 8; ++q) s[q] += v[q];
      }
      acc[i] += s[0] + s[1];
      acc[i + 1] += s[2] + s[3];
      acc[i + 2] += s[4] + s[5];
      acc[i + 3] += s[6] + s[7];
    }
  }
#pragma unroll
  for (int i = 0; i < kSpmvRowsPerWave; ++i) {
    double s = acc[i];
    for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
    if (lane == 0 && row0 + i < rows) out[row0 + i] = s;
  }
}


// Few rows (the tiled kernel above would leave most of the GPU idle): one wave per row, lanes over words.
__global__ __launch_bounds__(kThreads) void bit_spmv_rows_kernel(const uint64_t* B, int64_t rows, int64_t cols, int64_t stride,
                                                                 int64_t row_first, int64_t row_step, const double* x,
                                                                 double* out) {
  const int lane = threadIdx.x & 63;
  const int64_t wave = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
  const int64_t nwaves = ((int64_t)gridDim.x * blockDim.x) >> 6;
  const int64_t Wc = (cols + 63) / 64;
  const uint64_t tail = (cols & 63) ? ((1ull << (cols & 63)) - 1ull) : ~0ull;
  for (int64_t i = wave; i < rows; i += nwaves) {
    const uint64_t* row = B + (row_first + i * row_step) * stride;
    double acc = 0.0;
    for (int64_t wd = lane; wd < Wc; wd += 128) {
      uint64_t w0 = row[wd] & (wd == Wc - 1 ? tail : ~0ull);
      uint64_t w1 = wd + 64 < Wc ? (row[wd + 64] & (wd + 64 == Wc - 1 ? tail : ~0ull)) : 0ull;
      const double* x0 = x + wd * 64;
      const double* x1 = x0 + 64 * 64;
      double a0 = 0.0, a1 = 0.0;
      while (w0 | w1) {  // four bits of either word per step: eight gathers in flight (same order of additions)
        double v0[4], v1[4];
        bool l0[4], l1[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          l0[u] = w0 != 0ull;
          l1[u] = w1 != 0ull;
          v0[u] = x0[l0[u] ? __ffsll((long long)w0) - 1 : 0];
          v1[u] = *(l1[u] ? x1 + (__ffsll((long long)w1) - 1) : x0);  // x1 may lie past the end when w1 is empty
          w0 &= w0 - 1;
          w1 &= w1 - 1;
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          a0 += l0[u] ? v0[u] : 0.0;
          a1 += l1[u] ? v1[u] : 0.0;
        }
      }
      acc += a0 + a1;
    }
    for (int o = 32; o > 0; o >>= 1) acc += __shfl_xor(acc, o, 64);
    if (lane == 0) out[i] = acc;
  }
}

// ---- dense rows: product on the fp4 x fp6 matrix cores --------------------------------------
// out[i] = sum over set bits j of row i of x[j], for rows dense enough that one look-up or one
// gather per set bit (or per byte of mask) costs more than streaming the bits. The product is a
// (rows x cols 0/1 matrix) . (cols x 14 matrix of base-16 digits of x): exact integer arithmetic, carried by
// floating-point formats that hold these integers exactly.
//  * x is scaled by a power of two so that max|x| < 2^54 and rounded to integers (the same 2^-54 relative step for
//    every entry); 2^54 is added, so that the 14 digits are 0..15 and a digit is its own code in fp6 (e2m3: the magnitude
//    codes 0..15 are the multiples of 1/8). A fifteenth plane of ones counts the columns, to take the 2^54s off again.
//  * A operand of v_mfma_scale_f32_16x16x128_f8f6f4 = 16 rows x 128 columns of mask bits as fp4. A lane holds 32 nibbles
//    of one row, which come from the lane's four 32-bit mask words by ONE AND each: word & (0x11111111 << j) leaves
//    bit j of every nibble in place, the fp4 (e2m1) codes 1, 2, 4 are 1/2, 1, 2, and bit 3, the sign, is shifted down to
//    code 4. The instruction's block scales (2, 1, 1/2, 1/2 and 8 for the digits) make every product digit x bit, so that
//    operand j multiplies the columns {4i + j} and all four share one accumulator. Lane l supplies row (column of B)
//    l % 16 and the k from 32 (l / 16) on; digits are stored in the order that matches: within 128 columns, operand j's
//    element 8 w + i is column 32 w + 4 i + j, six bits each, 24 bytes.
//  * Sums of up to 2^20 digits stay below 2^24 and are exact in the fp32 accumulators.
//  * The planes of a 1024-column chunk are staged in LDS once per workgroup and read by all of its waves.
//  * A wave owns 64 rows (four 16-row tiles); per chunk every row is visited with 128 contiguous
//    bytes (two 16-byte loads per lane and tile), requested two chunks ahead.
// (On the int8 instruction, seven base-256 digits against bytes of one bit: half as many columns per instruction of the
// same 16 cycles, twice the ANDs, four accumulators for the four places of a bit, which left no registers for a second
// chunk on its way. The products of 99,981 players, 117 MB each: 37.5 us on average, now 32.5 in the loop and 29 alone, of which the
// loads take 21; 300,007 players, 318 MB: 86.5 on average, now 81.)
// The digit sums of a row are put together as two exact integers (2^24 hi + lo); those of its column groups are added up and rescaled by
// whoever reads them, so the result does not depend on the grouping.
typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v8i __attribute__((ext_vector_type(8)));
typedef float v4f __attribute__((ext_vector_type(4)));
constexpr int kMmTiles = 4;                          // 16-row tiles per wave
constexpr int kMmWaves = 4;                          // waves per workgroup
constexpr int kMmThreads = 64 * kMmWaves;
constexpr int kMmWaveRows = 16 * kMmTiles;
constexpr int kMmRows = kMmWaveRows * kMmWaves;      // rows per workgroup
constexpr int kMmHalves = kMmChunk / 512;            // 64-byte pieces of a row per chunk
constexpr int kMmSums = 8;                           // sums of a row in LDS: seven base-256 digits, the count
constexpr int kMmSumBytes = 16;                      // and in memory: hi, lo
constexpr int kMmSumPitch = kMmSums + 1;
// LDS image of a chunk: the four operands of a lane group in 128 bytes, planes 8 bytes further, so that the 32 lanes of half a
// wave read 8 bytes each from all 64 banks
constexpr int kMmGroupPitch = 128;
constexpr int kMmPlanePitch = kMmHalves * 4 * kMmGroupPitch + 8;
constexpr int64_t kMmMaxGroupCols = 1 << 20;         // 2^20 columns * 15 < 2^24: exact in fp32

// max_parts[block] = bit pattern of the block's max |x| (non-negative doubles order like their bit patterns)
__global__ __launch_bounds__(256) void absmax_kernel(const double* x, int64_t n, unsigned long long* max_parts) {
  __shared__ unsigned long long wm[4];
  unsigned long long m = 0;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
    const unsigned long long b = (unsigned long long)__double_as_longlong(x[i]) & 0x7fffffffffffffffull;
    m = b > m ? b : m;
  }
  ds_block_max<256>(m, wm);
  if (threadIdx.x == 0) max_parts[blockIdx.x] = m;
}

// The digits of a vector whose game has no sparse rows (else tile_spmv_kernel makes them on the side): one thread per half operand.
__global__ __launch_bounds__(256) void quantize_kernel(const double* x, int64_t n, int64_t chunks, const unsigned long long* max_parts,
                                                       int parts, int8_t* D, double* scal) {
  const int64_t id = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  double xv[kMmHalf];
  if (id < chunks * kMmHalves1024) ds_mm_half_operand(x, n, id, xv);   // (does not wait for the maximum)
  const ds_fixed_point fp = ds_fixed_point_of<256>(max_parts, parts);
  if (id == 0) scal[0] = fp.back();
  if (id < chunks * kMmHalves1024) ds_mm_store_digits(xv, n, id, fp, D);
}

// A workgroup's units (a chunk of a row group each) are consecutive, row group by row group: cut evenly (even_units = their
// total: mm_split.h; a plan clears the slots that nobody writes), or `groups` to a row group (even_units = 0). The mask words of
// the two units ahead are on their way while one is used, across row groups too. Every load is issued unconditionally (behind the last
// unit, of one cache line): a conditional one would make the wait for the current words a wait for all of them.
__global__ __launch_bounds__(kMmThreads, 2) void bit_spmv_mm_kernel(const uint64_t* B, int64_t rows, int64_t cols, int64_t stride,
                                                                    int64_t row_first, int64_t row_step, const int8_t* D,
                                                                    longlong2* partial, int64_t even_units, int64_t groups,
                                                                    int64_t chunks_per_group, int64_t n_chunks) {
  __shared__ __align__(16) int8_t Bs[2][kMmPlanes * kMmPlanePitch];
  __shared__ int sums[kMmWaves][kMmWaveRows * kMmSumPitch];
  typedef int v2i __attribute__((ext_vector_type(2)));
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r16 = lane & 15, g = lane >> 4;
  const int64_t Wc = (cols + 63) / 64;
  const int64_t G = gridDim.x, bid = blockIdx.x;
  int64_t rg, c;       // row group and chunk of the current unit
  int64_t left;        // units from it on
  int64_t slot = 0;    // where this workgroup's sums of the row group go
  if (even_units > 0) {
    const int64_t u0 = ds_mm_even_begin(bid, G, even_units);
    left = ds_mm_even_begin(bid + 1, G, even_units) - u0;
    rg = u0 / n_chunks;
    c = u0 - rg * n_chunks;
    slot = bid - ds_mm_even_owner(rg * n_chunks, G, even_units);   // (a later row group's first workgroup is this one)
  } else {
    const int64_t row_groups = G / groups;   // (consecutive workgroups: consecutive row groups of one column group)
    slot = bid / row_groups;
    rg = bid - slot * row_groups;
    c = slot * chunks_per_group;
    left = c + chunks_per_group < n_chunks ? chunks_per_group : n_chunks - c;
  }
  const int64_t row_bytes = row_step * stride * 8;
  const char* Bb = (const char*)(B + row_first * stride);
  const uint32_t lane_off = (uint32_t)r16 * (uint32_t)row_bytes;   // the host keeps 16 * row_bytes below 2^32
  v4f acc[kMmTiles];
  auto clear = [&]() {
#pragma unroll
    for (int t = 0; t < kMmTiles; ++t) acc[t] = v4f{0.f, 0.f, 0.f, 0.f};
  };
  // Rows past the end are read from a live row and never stored. Words past the row's end meet zero digits; the 16 bytes that
  // would cross it are read 8 bytes earlier and moved into place where they are used (`fix`). (One 16-byte load per lane, tile and
  // half: as two 8-byte loads the same bytes took twice the requests and the kernel ran 17 % slower.)
  typedef uint32_t u4a8 __attribute__((ext_vector_type(4), aligned(8)));   // rows are 8-byte aligned
  struct Words { u4a8 a[kMmTiles][kMmHalves]; };
  const int64_t last_pair = Wc > 1 ? Wc - 2 : 0;   // (a single word: the caller's rows have 8 bytes more behind the last)
  auto load_a = [&](Words& w, int64_t group, int64_t chunk, bool live) {
    const int64_t wave_row0 = (group * kMmWaves + wave) * kMmWaveRows;
#pragma unroll
    for (int t = 0; t < kMmTiles; ++t) {
      const int64_t r_t = wave_row0 + 16 * t;
      const char* base = live ? Bb + (r_t < rows ? r_t : rows - 1) * row_bytes : Bb;   // uniform over the wave
      const uint32_t lo = live && r_t + r16 < rows ? lane_off : 0u;
#pragma unroll
      for (int h = 0; h < kMmHalves; ++h) {
        const int64_t w0 = chunk * (kMmChunk / 64) + h * 8 + g * 2;
        w.a[t][h] = *(const u4a8*)(base + (lo + (live ? (uint32_t)(w0 < last_pair ? w0 : last_pair) * 8u : 0u)));
      }
    }
  };
  auto fix = [&](Words& w, int64_t chunk) {
#pragma unroll
    for (int h = 0; h < kMmHalves; ++h) {
      const bool odd = chunk * (kMmChunk / 64) + h * 8 + g * 2 == Wc - 1 && Wc > 1;   // this lane's first word is the row's last
#pragma unroll
      for (int t = 0; t < kMmTiles; ++t) {
        w.a[t][h].x = odd ? w.a[t][h].z : w.a[t][h].x;
        w.a[t][h].y = odd ? w.a[t][h].w : w.a[t][h].y;
      }
    }
  };
  // staging of a chunk's digit planes, 16 bytes at a time: piece p of a plane is a sixth of a lane group's operands
  constexpr int kPieces = kMmChunkBytes / 16, kStage = (kPieces + kMmThreads - 1) / kMmThreads, kPlanePieces = kMmPlaneBytes / 16;
  int st_src[kStage], st_dst[kStage];
#pragma unroll
  for (int u = 0; u < kStage; ++u) {
    const int p = tid + u * kMmThreads < kPieces ? tid + u * kMmThreads : tid;   // (past the end: the thread's first piece again)
    const int plane = p / kPlanePieces, in = p - plane * kPlanePieces, group = in / (4 * kMmOperand / 16);
    st_src[u] = p * 16;
    st_dst[u] = plane * kMmPlanePitch + group * kMmGroupPitch + (in - group * (4 * kMmOperand / 16)) * 16;
  }
  v4i st[kStage];
  auto stage_load = [&](int64_t chunk) {
    const int8_t* const src = D + chunk * kMmChunkBytes;
#pragma unroll
    for (int u = 0; u < kStage; ++u) st[u] = *(const v4i*)(src + st_src[u]);
  };
  auto stage_store = [&](int buf) {
#pragma unroll
    for (int u = 0; u < kStage; ++u) {   // (planes start at multiples of 8 bytes)
      *(v2i*)&Bs[buf][st_dst[u]] = v2i{st[u].x, st[u].y};
      *(v2i*)&Bs[buf][st_dst[u] + 8] = v2i{st[u].z, st[u].w};
    }
  };
  const int b_off = (r16 < kMmPlanes ? r16 : kMmPlanes - 1) * kMmPlanePitch + g * kMmGroupPitch;   // (column 15 is not looked at)
  constexpr int kOne = 0x7f;   // block scale 2^0
  const int scale_a[4] = {kOne + 1, kOne, kOne - 1, kOne - 1}, scale_b = kOne + 3;
  auto multiply = [&](const Words& w, int buf) {
    const int8_t* bs = &Bs[buf][b_off];
    v2i bq[2][4][3];
    auto operands = [&](int h) {
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int u = 0; u < 3; ++u) bq[h & 1][j][u] = *(const v2i*)(bs + h * 4 * kMmGroupPitch + j * kMmOperand + u * 8);
    };
    operands(0);
#pragma unroll
    for (int h = 0; h < kMmHalves; ++h) {
      if (h + 1 < kMmHalves) operands(h + 1);
#pragma unroll
      for (int t = 0; t < kMmTiles; ++t) {
        const u4a8 x = w.a[t][h];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const uint32_t m = j < 3 ? 0x11111111u << j : 0x44444444u;
          const u4a8 y = j < 3 ? x : x >> 1;
          const v8i av = {(int)(y.x & m), (int)(y.y & m), (int)(y.z & m), (int)(y.w & m), 0, 0, 0, 0};
          const v2i* const q = bq[h & 1][j];
          const v8i bv = {q[0].x, q[0].y, q[1].x, q[1].y, q[2].x, q[2].y, 0, 0};
          acc[t] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(av, bv, acc[t], 4, 2, 0, scale_a[j], 0, scale_b);   // fp4, fp6 e2m3
        }
      }
    }
  };
  // Lane (plane r16, lane group g) holds rows 4g + v of every tile. Two neighbouring digits make a base-256 one, and through LDS a
  // lane gets all those of a row: 16 contiguous bytes a lane go to memory. (Stored as eight 32-bit sums a row from the lanes
  // that have them, 32 bytes at a time, the sums of 300,007 rows cost 13 us of 78.)
  auto store_sums = [&]() {
    int* const mine = sums[wave];
#pragma unroll
    for (int t = 0; t < kMmTiles; ++t)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int digit = (int)acc[t][v];
        const int high = __builtin_amdgcn_update_dpp(0, digit, 0xf5, 0xf, 0xf, false);   // quad_perm [1,1,3,3]: the next plane's
        if ((r16 & 1) == 0) mine[(16 * t + 4 * g + v) * kMmSumPitch + (r16 >> 1)] = r16 < kMmDigits ? digit + 16 * high : digit;
      }
    const int64_t row = (rg * kMmWaves + wave) * kMmWaveRows + lane;
    const int* const q = mine + lane * kMmSumPitch;
    longlong2 out;   // sum_d 256^d S[d] - 2^54 count = 2^24 x + y
    out.x = (((long long)q[6] * 256 + q[5]) * 256 + q[4]) * 256 + q[3] - ((long long)q[7] << 30);
    out.y = ((long long)q[2] * 256 + q[1]) * 256 + q[0];
    if (row < rows) partial[slot * rows + row] = out;
  };
  Words w0, w1, w2;
  int64_t rg1 = rg, c1 = c;   // the next unit, then the one behind it; both stay on a live one behind the last
  auto advance = [&](int64_t& group, int64_t& chunk) {
    const bool wrap = chunk + 1 == n_chunks;
    group = wrap ? group + 1 : group;
    chunk = wrap ? 0 : chunk + 1;
  };
  // one unit from `cur`; `next` takes the words of the one behind the next. False behind the last.
  auto unit = [&](Words& cur, Words& next, int buf) {
    int64_t rg2 = rg1, c2 = c1;
    advance(rg2, c2);
    stage_load(left > 1 ? c1 : c);
    load_a(next, rg2, c2, left > 2);
    if (c == n_chunks - 1 && (Wc & 1)) fix(cur, c);
    multiply(cur, buf);
    if (c == n_chunks - 1 || left == 1) {
      store_sums();
      clear();
      slot = 0;
    }
    if (left == 1) return false;
    stage_store(buf ^ 1);
    __syncthreads();   // every wave is done with Bs[buf]; Bs[buf ^ 1] is complete
    rg = rg1;
    c = c1;
    rg1 = rg2;
    c1 = c2;
    --left;
    return true;
  };
  advance(rg1, c1);
  stage_load(c);
  load_a(w0, rg, c, true);
  load_a(w1, rg1, c1, left > 1);
  clear();
  stage_store(0);
  __syncthreads();
  for (;;) {   // (the words' three buffers and LDS's two in turn)
    if (!unit(w0, w2, 0)) break;
    if (!unit(w1, w0, 1)) break;
    if (!unit(w2, w1, 0)) break;
    if (!unit(w0, w2, 1)) break;
    if (!unit(w1, w0, 0)) break;
    if (!unit(w2, w1, 1)) break;
  }
}

// out[r] = (addend[r] or 0) + scal[0] * sum_d 256^d * (sum over the column groups of digit sum d)
__global__ __launch_bounds__(256) void mm_reduce_kernel(const longlong2* partial, int64_t rows, int groups, const double* scal,
                                                        const double* addend, double* out) {
  const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= rows) return;
  const double val = ds_mm_sum(partial, rows, groups, r) * scal[0];
  out[r] = addend ? addend[r] + val : val;
}

// ---- sparse rows: index lists (the input of the tile build) ------------------------------------
// idx[off[i] .. off[i+1]) = ascending columns of the set bits of row i; one wave per row
__global__ __launch_bounds__(kThreads) void rows_to_csr_kernel(const uint64_t* B, int64_t rows, int64_t cols, int64_t stride,
                                                               int64_t row_first, int64_t row_step, const int32_t* off,
                                                               int32_t* idx) {
  const int lane = threadIdx.x & 63;
  const int64_t wave = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
  const int64_t nwaves = ((int64_t)gridDim.x * blockDim.x) >> 6;
  const int64_t Wc = (cols + 63) / 64;
  const uint64_t tail = (cols & 63) ? ((1ull << (cols & 63)) - 1ull) : ~0ull;
  for (int64_t i = wave; i < rows; i += nwaves) {
    const uint64_t* row = B + (row_first + i * row_step) * stride;
    int32_t base = off[i];
    for (int64_t w0 = 0; w0 < Wc; w0 += 64) {
      const int64_t wd = w0 + lane;
      uint64_t word = wd < Wc ? row[wd] : 0ull;
      if (wd == Wc - 1) word &= tail;
      const int cnt = __popcll(word);
      int pre = cnt;  // inclusive scan over the lanes
      for (int o = 1; o < 64; o <<= 1) {
        const int v = __shfl_up(pre, o, 64);
        if (lane >= o) pre += v;
      }
      int32_t at = base + pre - cnt;
      while (word) {
        idx[at++] = (int32_t)(wd * 64 + __ffsll((long long)word) - 1);
        word &= word - 1;
      }
      base += __shfl(pre, 63, 64);
    }
  }
}

}  // namespace

int ds_bit_spmv(ds_ctx* ctx, const uint64_t* B, int64_t rows, int64_t cols, int64_t stride, int64_t row_first,
                int64_t row_step, const double* x, double* out) {
  if (rows <= 0) return DS_OK;
  const int64_t rows_per_block = kSpmvRowsPerWave * (kThreads / 64);
  const int64_t blocks = (rows + rows_per_block - 1) / rows_per_block;
  if (blocks < (int64_t)ctx->num_cus) {
    hipLaunchKernelGGL(bit_spmv_rows_kernel, dim3((unsigned)((rows * 64 + kThreads - 1) / kThreads)), dim3(kThreads), 0,
                       ctx->stream, B, rows, cols, stride, row_first, row_step, x, out);
    DS_HIP(ctx, hipGetLastError());
    return DS_OK;
  }
  hipLaunchKernelGGL(bit_spmv_kernel, dim3((unsigned)blocks), dim3(kThreads), 0, ctx->stream, B, rows, cols, stride,
                     row_first, row_step, x, out);
  DS_HIP(ctx, hipGetLastError());
  return DS_OK;
}

int ds_row_prep(ds_ctx* ctx, const uint64_t* Z, int64_t k, int64_t n, int paired, const float* w, const float* y, int32_t* sz,
                double* t, double* sqw, float* wc) {
  const int64_t W = (n + 63) / 64;
  int64_t blocks = ((paired ? k / 2 : k) * 64 + kThreads - 1) / kThreads;
  if (blocks > (int64_t)ctx->num_cus * 16) blocks = (int64_t)ctx->num_cus * 16;
  hipLaunchKernelGGL(row_prep_kernel, dim3((unsigned)blocks), dim3(kThreads), 0, ctx->stream, Z, k, W, n, paired, w, y, sz, t, sqw, wc);
  DS_HIP(ctx, hipGetLastError());
  return DS_OK;
}

int ds_bit_transpose(ds_ctx* ctx, const uint64_t* in, int64_t rows, int64_t cols, int64_t in_stride, int64_t row_first,
                     int64_t row_step, uint64_t* out, int64_t out_stride) {
  const int64_t Wout = out_stride > 0 ? out_stride : (rows + 63) / 64, Win = (cols + 63) / 64;
  const int64_t tiles_r = (rows + 511) / 512, tiles_c = (Win + 7) / 8;
  if (tiles_r < 1 || tiles_c < 1) return DS_OK;
  if (tiles_r * tiles_c > 0x7fffffffLL) return ds_fail(ctx, DS_EINVAL, "bit matrix too large to transpose");
  hipLaunchKernelGGL(bit_transpose_kernel, dim3((unsigned)(tiles_r * tiles_c)), dim3(kTrThreads), 0, ctx->stream, in, rows, cols,
                     in_stride, row_first, row_step, out, Wout, tiles_c, 0);
  DS_HIP(ctx, hipGetLastError());
  return DS_OK;
}

int ds_bit_transpose_blocks(ds_ctx* ctx, const uint64_t* in, int64_t rows, int64_t cols, int64_t in_stride, int64_t row_step,
                            uint64_t* out) {
  const int64_t Wout = (rows + 63) / 64, Win = (cols + 63) / 64;
  const int64_t tiles_r = (rows + 511) / 512, tiles_c = (Win + 7) / 8;
  if (tiles_r < 1 || tiles_c < 1) return DS_OK;
  if (tiles_r * tiles_c > 0x7fffffffLL) return ds_fail(ctx, DS_EINVAL, "bit matrix too large to transpose");
  hipLaunchKernelGGL(bit_transpose_kernel, dim3((unsigned)(tiles_r * tiles_c)), dim3(kTrThreads), 0, ctx->stream, in, rows, cols,
                     in_stride, (int64_t)0, row_step, out, Wout, tiles_c, 1);
  DS_HIP(ctx, hipGetLastError());
  return DS_OK;
}

static void mm_shape(const ds_ctx* ctx, int64_t rows, int64_t cols, ds_mm_plan* p) {
  p->rows = rows;
  p->cols = cols;
  p->row_groups = (rows + kMmRows - 1) / kMmRows;
  p->n_chunks = (cols + kMmChunk - 1) / kMmChunk;
  const ds_mm_split c = ds_mm_choose_split(ctx->num_cus, rows, p->row_groups, p->n_chunks, kMmMaxGroupCols / kMmChunk, 2 * kMmSumBytes);
  const ds_mm_even e = ds_mm_choose_even(ctx->num_cus, rows, p->row_groups, p->n_chunks, kMmMaxGroupCols / kMmChunk, kMmSumBytes, c);
  p->cpg = c.cpg;
  p->groups = e.wgs > 0 ? e.slots : c.groups;
  p->even_wgs = e.wgs;
}

size_t ds_bit_spmv_mm_ws_bytes(const ds_ctx* ctx, int64_t rows, int64_t cols) {
  ds_mm_plan p;
  mm_shape(ctx, rows, cols, &p);
  return ds_align((size_t)p.n_chunks * kMmChunkBytes) + ds_align((size_t)p.groups * rows * kMmSumBytes);
}

int ds_bit_spmv_mm_prepare(ds_ctx* ctx, int64_t rows, int64_t cols, void* ws, ds_mm_plan* plan) {
  mm_shape(ctx, rows, cols, plan);
  char* p = (char*)ws;
  plan->D = (int8_t*)p;
  plan->partial = (longlong2*)(p + ds_align((size_t)plan->n_chunks * kMmChunkBytes));
  if (plan->even_wgs > 0)   // (slots of a row group that no workgroup reaches)
    DS_HIP(ctx, hipMemsetAsync(plan->partial, 0, (size_t)plan->groups * rows * kMmSumBytes, ctx->stream));
  return DS_OK;
}

int ds_vec_absmax(ds_ctx* ctx, const double* x, int64_t len, unsigned long long* max_parts, int parts) {
  hipLaunchKernelGGL(absmax_kernel, dim3((unsigned)parts), dim3(256), 0, ctx->stream, x, len, max_parts);
  DS_HIP(ctx, hipGetLastError());
  return DS_OK;
}

int ds_mm_quantize(ds_ctx* ctx, const ds_mm_plan* p, const double* x, const unsigned long long* max_parts, int parts, double* scal) {
  const int64_t threads = p->n_chunks * kMmHalves1024;
  hipLaunchKernelGGL(quantize_kernel, dim3((unsigned)((threads + 255) / 256)), dim3(256), 0, ctx->stream, x, p->cols, p->n_chunks, max_parts,
                     parts, p->D, scal);
  DS_HIP(ctx, hipGetLastError());
  return DS_OK;
}

int ds_bit_spmv_mm_product(ds_ctx* ctx, const ds_mm_plan* p, const uint64_t* B, int64_t stride, int64_t row_first,
                           int64_t row_step, const double* scal, const double* addend, double* out) {
  if (p->rows <= 0) return DS_OK;
  if (row_step * stride * 8 * 16 >= ((int64_t)1 << 32))
    return ds_fail(ctx, DS_EINTERNAL, "matrix-core product: rows of %lld bytes are too far apart", (long long)(row_step * stride * 8));
  const int64_t wgs = p->even_wgs > 0 ? p->even_wgs : p->row_groups * p->groups;
  hipLaunchKernelGGL(bit_spmv_mm_kernel, dim3((unsigned)wgs), dim3(kMmThreads), 0, ctx->stream, B, p->rows, p->cols, stride,
                     row_first, row_step, p->D, p->partial, p->even_wgs > 0 ? p->row_groups * p->n_chunks : (int64_t)0, p->groups,
                     p->cpg, p->n_chunks);
  if (out)
    hipLaunchKernelGGL(mm_reduce_kernel, dim3((unsigned)((p->rows + 255) / 256)), dim3(256), 0, ctx->stream, p->partial, p->rows,
                       (int)p->groups, scal, addend, out);
  DS_HIP(ctx, hipGetLastError());
  return DS_OK;
}

int ds_rows_to_csr(ds_ctx* ctx, const uint64_t* B, int64_t rows, int64_t cols, int64_t stride, int64_t row_first,
                   int64_t row_step, const int32_t* off, int32_t* idx) {
  if (rows <= 0) return DS_OK;
  int64_t blocks = (rows * 64 + kThreads - 1) / kThreads;
  if (blocks > (int64_t)ctx->num_cus * 16) blocks = (int64_t)ctx->num_cus * 16;
  hipLaunchKernelGGL(rows_to_csr_kernel, dim3((unsigned)blocks), dim3(kThreads), 0, ctx->stream, B, rows, cols, stride,
                     row_first, row_step, off, idx);
  DS_HIP(ctx, hipGetLastError());
  return DS_OK;
}
