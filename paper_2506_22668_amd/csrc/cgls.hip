// Conjugate gradients for least squares on the bit-packed mask matrix.
//
// Paper, Alg. 1 (CGLS on sqrt(W) M with a 1D row layout; here one GPU holds all
// rows, so the two all-reduces of the algorithm are plain device reductions). The
// iteration is the standard Hestenes-Stiefel form (the step ratio is
// |s_i|^2/|s_(i-1)|^2), started from zero, on the matrix sqrt(W) Z P with
// P = I - 11^T/n, so the iterate stays orthogonal to 1 and, when the problem is
// rank-deficient, converges to the minimum-norm solution.
//
// Both products walk set bits only. With complementary pairs (rows 2r, 2r+1 with
// one weight) only the small member of each pair is read:
//   forward:  d_r = sum_{j in S_r} u_j;  v_2r = a_r d_r,  v_2r+1 = a_r (sum(u) - d_r)
//   adjoint:  s = P sum_r a_r (r_2r - r_2r+1) z_r          (constants vanish under P)
// and the adjoint runs the same row kernel on a transposed copy of the small rows.
// Without the pairing promise every row is walked and the transpose holds all rows.
// All vectors and sums are fp64 (fp64 adds run at the rate of unpacked fp32 here).
#include "internal.h"
#include "solve_common.h"

namespace {

constexpr int kThreads = 256;
constexpr int kRed = 1024;  // blocks (and partials) of every reduction, at most

__device__ __forceinline__ void block_reduce2(double a, double b, double* pa, double* pb) {
  __shared__ double sh[2][kThreads / 64];
  for (int o = 32; o > 0; o >>= 1) {
    a += __shfl_xor(a, o, 64);
    b += __shfl_xor(b, o, 64);
  }
  if ((threadIdx.x & 63) == 0) {
    sh[0][threadIdx.x >> 6] = a;
    sh[1][threadIdx.x >> 6] = b;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    double x = 0, y = 0;
    for (int i = 0; i < kThreads / 64; ++i) {
      x += sh[0][i];
      y += sh[1][i];
    }
    *pa = x;
    *pb = y;
  }
  __syncthreads();
}

// scalars (device doubles): 0 gamma, 1 delta, 2 theta, 3 beta, 4 sum(u), 5 mean(s_raw), 6 gamma_new, 7 gamma0,
// 8 done (0/1), 9 iterations completed, 10 relative residual at the last test
// partial sums: four arrays of kRed doubles, one per reduction of the loop (|v|^2, sum(s), |Ps|^2, sum(u)), so
// that a kernel can read the partials of the reduction before it while writing those of its own
struct Vecs {
  int64_t n, k, R;   // R = rows of the forward matrix (pairs or rows)
  int paired;
  const double* sqw; // [k]
  double *x, *u, *s, *r, *v, *d, *h;  // n, n, n, k, k, R, R
  double* scal;
  double* part;      // [4 * kRed]
  // fixed-point products only (else null): where the kernel that writes u (h) leaves its workgroups' max |u| (max |h|)
  // for the next forward (adjoint) product, which then needs no pass of its own over the vector. An iteration that has
  // stopped leaves vector and maxima alone.
  unsigned long long *max_u, *max_h;
  // fixed-point products inside the loop (fused != 0): the products leave their integer partial sums, and the loop's
  // kernel that reads d (s) first adds them up itself and scales them by scal_f[0] (scal_a[0]). Forward: the rows [0, Rs) come from the tiles, the rest from the matrix cores; adjoint: both parts
  // cover all n entries and are added, tiles first.
  int fused;
  int64_t Rs;
  ds_fixed_view fwd, adj;
  const double *scal_f, *scal_a;
};

// T lanes (a power of two, consecutive lanes of a wave, `sub` = the lane's place among them) add up one entry together:
// each takes every T-th group, the integers are added across the lanes, and all T lanes return the same value
template <int T>
__device__ __forceinline__ double mm_result(const ds_fixed_view& v, int64_t r, int sub) {
  long long hi = 0, lo = 0;
  ds_mm_sum_part(v.mm_partial, v.mm_rows, v.mm_groups, r, sub, T, hi, lo);
#pragma unroll
  for (int o = 1; o < T; o <<= 1) {
    hi += __shfl_xor(hi, o, 64);
    lo += __shfl_xor(lo, o, 64);
  }
  return ds_mm_sum_finish(hi, lo);
}
template <int T>
__device__ __forceinline__ double tile_result(const ds_fixed_view& v, int64_t i, int sub) {
  long long hi = 0, lo = 0;
  ds_tile_sum_part(v.tile_partial, v.tile_len, v.tile_groups, i, sub, T, hi, lo);
#pragma unroll
  for (int o = 1; o < T; o <<= 1) {
    hi += __shfl_xor(hi, o, 64);
    lo += __shfl_xor(lo, o, 64);
  }
  return ds_tile_sum_finish(hi, lo, v.tile_sh);
}
template <int T>
__device__ __forceinline__ double forward_result(const Vecs& a, double sc, int64_t i, int sub) {
  if (i < a.Rs) return a.fwd.tile_groups ? tile_result<T>(a.fwd, i, sub) * sc : 0.0;
  return mm_result<T>(a.fwd, i - a.Rs, sub) * sc;
}
template <int T>
__device__ __forceinline__ double adjoint_result(const Vecs& a, double sc, int64_t j, int sub) {
  const double mm = a.adj.mm_groups ? mm_result<T>(a.adj, j, sub) * sc : 0.0;
  if (!a.adj.tile_groups) return mm;
  const double tl = tile_result<T>(a.adj, j, sub) * sc;
  return a.adj.mm_groups ? tl + mm : tl;
}

// the workgroup's part of max |x| into max_parts[blockIdx.x] (every thread of the workgroup must call this)
__device__ __forceinline__ void publish_absmax(unsigned long long m, unsigned long long* max_parts) {
  __shared__ unsigned long long wm[kThreads / 64];
  ds_block_max<kThreads>(m, wm);
  if (threadIdx.x == 0) max_parts[blockIdx.x] = m;
  __syncthreads();
}
__device__ __forceinline__ unsigned long long abs_bits(double x) {
  return (unsigned long long)__double_as_longlong(x) & 0x7fffffffffffffffull;
}
// r = sqrt(w) t ; h from r
__global__ void init_r_kernel(Vecs a, const double* t) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < a.k) a.r[i] = a.sqw[i] * t[i];
}
__global__ void make_h_kernel(Vecs a) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= a.R) return;
  a.h[i] = a.paired ? a.sqw[2 * i] * (a.r[2 * i] - a.r[2 * i + 1]) : a.sqw[i] * a.r[i];
}

// sum of nparts (<= kRed) partials by one wave, in a fixed order; every lane gets the result
__device__ __forceinline__ double wave_sum_partials(const double* part, int nparts) {
  double s = 0.0;
  for (int i = threadIdx.x; i < nparts; i += 64) s += part[i];
  for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
  return s;
}

// partial sums of the raw adjoint (for its mean)
__global__ __launch_bounds__(kThreads) void s_sum_kernel(Vecs a) {
  double s1 = 0;
  for (int64_t j = (int64_t)blockIdx.x * kThreads + threadIdx.x; j < a.n; j += (int64_t)gridDim.x * kThreads) s1 += a.s[j];
  double dummy;
  block_reduce2(s1, 0.0, &a.part[blockIdx.x], &dummy);
}

__global__ void fin_mean_kernel(Vecs a, int nparts) {
  const double s1 = wave_sum_partials(a.part, nparts);
  if (threadIdx.x == 0) a.scal[5] = s1 / (double)a.n;
}

// s <- P s (subtract the mean in place) and partial |P s|^2. Two passes on purpose:
// the raw adjoint carries a large common offset, and sum(s^2) - n mean^2 would cancel.
__global__ __launch_bounds__(kThreads) void s_center_kernel(Vecs a) {
  const double mean = a.scal[5];
  double s2 = 0;
  for (int64_t j = (int64_t)blockIdx.x * kThreads + threadIdx.x; j < a.n; j += (int64_t)gridDim.x * kThreads) {
    const double v = a.s[j] - mean;
    a.s[j] = v;
    s2 += v * v;
  }
  double dummy;
  block_reduce2(s2, 0.0, &a.part[blockIdx.x], &dummy);
}

// gamma_new = |P s|^2 and beta; the first call sets gamma0 and beta = theta = 0
__global__ void fin_gamma_kernel(Vecs a, int nparts, int first) {
  const double g = wave_sum_partials(a.part, nparts);
  if (threadIdx.x != 0) return;
  a.scal[6] = g;
  if (first) {
    a.scal[7] = g;
    a.scal[3] = 0.0;
    a.scal[2] = 0.0;
  } else {
    a.scal[3] = a.scal[0] > 0.0 ? g / a.scal[0] : 0.0;
  }
}

// x += theta u ; u = s + beta u (s already projected) ; partial sum(u)
__global__ __launch_bounds__(kThreads) void update_xu_kernel(Vecs a) {
  const double th = a.scal[2], beta = a.scal[3];
  double acc = 0;
  for (int64_t j = (int64_t)blockIdx.x * kThreads + threadIdx.x; j < a.n; j += (int64_t)gridDim.x * kThreads) {
    const double uo = a.u[j];
    a.x[j] += th * uo;
    const double un = a.s[j] + beta * uo;
    a.u[j] = un;
    acc += un;
  }
  double dummy;
  block_reduce2(acc, 0.0, &a.part[blockIdx.x], &dummy);
}

__global__ void fin_u_kernel(Vecs a, int nparts) {
  const double s = wave_sum_partials(a.part, nparts);
  if (threadIdx.x == 0) {
    a.scal[4] = s;
    a.scal[0] = a.scal[6];
  }
}

// ---- the loop's kernels: every reduction is finished by the kernel that needs its result (each workgroup
// adds the same partials in the same order, workgroup 0 records the scalar), and the stopping rule of the
// iteration is evaluated on the device, so that the host only looks every few iterations. Once `done` is set
// the state that the result is made of (x, u, theta) is left alone by everything that still runs. ----
constexpr int kPartV = 0, kPartS = 1, kPartG = 2, kPartU = 3;

// all threads of the workgroup get the sum of their values (lanes first, then waves)
__device__ __forceinline__ double block_sum(double s) {
  __shared__ double bs[kThreads / 64];
  for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
  __syncthreads();
  if ((threadIdx.x & 63) == 0) bs[threadIdx.x >> 6] = s;
  __syncthreads();
  double t = bs[0];
  for (int i = 1; i < kThreads / 64; ++i) t += bs[i];
  return t;
}
// all threads of the workgroup get the sum of the nparts partials of array `which`
// (every workgroup adds them in the same order: thread t takes the partials t, t + kThreads, ..., then lanes, then waves)
__device__ __forceinline__ double block_sum_partials(const Vecs& a, int which, int nparts) {
  const double* part = a.part + which * kRed;
  double s = 0.0;
  for (int i = threadIdx.x; i < nparts; i += kThreads) s += part[i];
  return block_sum(s);
}

// v from d (after finishing sum(u) and moving gamma_new to gamma); partial |v|^2. T lanes per row (1 unless fused).
template <int T>
__global__ __launch_bounds__(kThreads) void loop_make_v_kernel(Vecs a, int parts_u) {
  const double U = block_sum_partials(a, kPartU, parts_u);
  if (blockIdx.x == 0 && threadIdx.x == 0 && a.scal[8] == 0.0) {
    a.scal[4] = U;
    a.scal[0] = a.scal[6];
  }
  const double sc = a.fused ? a.scal_f[0] : 0.0;
  double acc = 0.0;
  const int sub = threadIdx.x & (T - 1);
  for (int64_t i = ((int64_t)blockIdx.x * kThreads + threadIdx.x) / T; i < a.R; i += (int64_t)gridDim.x * (kThreads / T)) {
    const double d = a.fused ? forward_result<T>(a, sc, i, sub) : a.d[i];
    if (sub == 0) {   // (all T lanes hold the same d)
      if (a.paired) {
        const double w = a.sqw[2 * i];
        const double v0 = w * d, v1 = w * (U - d);
        a.v[2 * i] = v0;
        a.v[2 * i + 1] = v1;
        acc += v0 * v0 + v1 * v1;
      } else {
        const double v0 = a.sqw[i] * d;
        a.v[i] = v0;
        acc += v0 * v0;
      }
    }
  }
  double dummy;
  block_reduce2(acc, 0.0, &a.part[kPartV * kRed + blockIdx.x], &dummy);
}

// delta = |v|^2, theta = gamma / delta; r -= theta v, then h. A direction in the null space (delta = 0)
// ends the iteration with theta = 0.
__global__ __launch_bounds__(kThreads) void loop_update_r_kernel(Vecs a, int parts_v) {
  const double delta = block_sum_partials(a, kPartV, parts_v);
  const bool done = a.scal[8] != 0.0;
  const double gamma = a.scal[0];
  const bool null_dir = !(delta > 0.0);
  const double th = null_dir ? 0.0 : gamma / delta;
  if (done) return;
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    a.scal[1] = delta;
    a.scal[2] = th;
    if (null_dir) {
      a.scal[8] = 1.0;
      a.scal[9] += 1.0;
    }
  }
  unsigned long long hm = 0;
  for (int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x; i < a.R; i += (int64_t)gridDim.x * kThreads) {
    double hn;
    if (a.paired) {
      const double r0 = a.r[2 * i] - th * a.v[2 * i], r1 = a.r[2 * i + 1] - th * a.v[2 * i + 1];
      a.r[2 * i] = r0;
      a.r[2 * i + 1] = r1;
      hn = a.sqw[2 * i] * (r0 - r1);
    } else {
      const double r0 = a.r[i] - th * a.v[i];
      a.r[i] = r0;
      hn = a.sqw[i] * r0;
    }
    a.h[i] = hn;
    const unsigned long long b = abs_bits(hn);
    hm = b > hm ? b : hm;
  }
  if (a.max_h) publish_absmax(hm, a.max_h);
}

// how many of n entries workgroup b of a grid of `grid` takes that stride over them, `per` to a workgroup at a time
__device__ __forceinline__ uint32_t block_entries(uint32_t n, uint32_t per, uint32_t grid, uint32_t b) {
  const uint32_t turn = per * grid, left = n % turn, first = per * b;
  return n / turn * per + (left > first ? (left - first < per ? left - first : per) : 0);
}

// s; per workgroup the sum S of its entries and the sum M of their squared distances from their own mean. Together,
// |P s|^2 = sum of M + count (S / count - mean)^2: nothing cancels, as sum(s^2) - n mean^2 would (see s_center_kernel), and there is
// no second launch behind the mean of all. (A kernel that waited for it and wrote P s: an iteration of 113 us at 99,981 players, now 109.)
template <int T>
__global__ __launch_bounds__(kThreads) void loop_s_sum_kernel(Vecs a) {
  const int64_t first = ((int64_t)blockIdx.x * kThreads + threadIdx.x) / T, step = (int64_t)gridDim.x * (kThreads / T);
  const int sub = threadIdx.x & (T - 1);
  double s1 = 0, v0 = 0;   // v0: the first entry, the only one of all but the largest games
  if (a.fused) {
    const double sc = a.scal_a[0];
    for (int64_t j = first; j < a.n; j += step) {
      const double v = adjoint_result<T>(a, sc, j, sub);
      if (sub == 0) {
        a.s[j] = v;
        s1 += v;
        if (j == first) v0 = v;
      }
    }
  } else {
    for (int64_t j = first; j < a.n; j += step) {
      const double v = a.s[j];
      s1 += v;
      if (j == first) v0 = v;
    }
  }
  const double sum = block_sum(s1);
  const double mean = sum / block_entries((uint32_t)a.n, kThreads / T, gridDim.x, blockIdx.x);
  double s2 = 0;
  if (sub == 0)
    for (int64_t j = first; j < a.n; j += step) {
      const double v = (j == first ? v0 : a.s[j]) - mean;
      s2 += v * v;
    }
  s2 = block_sum(s2);
  if (threadIdx.x == 0) {
    a.part[kPartS * kRed + blockIdx.x] = sum;
    a.part[kPartG * kRed + blockIdx.x] = s2;
  }
}

// end of an iteration: gamma_new = |P s|^2, the stopping rule, and (if the iteration goes on and do_update)
// x += theta u, u = P s + beta u with the partial sums of the new u. The partials are those of loop_s_sum_kernel, `per` entries
// to a workgroup at a time.
__global__ __launch_bounds__(kThreads) void loop_update_xu_kernel(Vecs a, int parts, int per, double tol, int do_update) {
  constexpr int kMine = kRed / kThreads;
  double ps[kMine], pm[kMine], s1 = 0;
#pragma unroll
  for (int i = 0; i < kMine; ++i) {
    const int b = threadIdx.x + i * kThreads;
    ps[i] = b < parts ? a.part[kPartS * kRed + b] : 0.0;
    pm[i] = b < parts ? a.part[kPartG * kRed + b] : 0.0;
    s1 += ps[i];
  }
  const double mean = block_sum(s1) / (double)a.n;
  double g = 0;
#pragma unroll
  for (int i = 0; i < kMine; ++i) {
    const int b = threadIdx.x + i * kThreads;
    if (b >= parts) continue;
    const double count = block_entries((uint32_t)a.n, per, parts, b), away = ps[i] / count - mean;
    g += pm[i] + count * (away * away);
  }
  g = block_sum(g);
  if (a.scal[8] != 0.0) return;
  const double gamma = a.scal[0], gamma0 = a.scal[7];
  const double rel = sqrt(g) / sqrt(gamma0);
  const bool stop = rel <= tol;
  const double beta = gamma > 0.0 ? g / gamma : 0.0;
  const double th = a.scal[2];
  __syncthreads();  // every thread has read the scalars before workgroup 0 changes them
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    a.scal[9] += 1.0;
    a.scal[10] = rel;
    if (stop) a.scal[8] = 1.0;
    else if (do_update) {
      a.scal[3] = beta;
      a.scal[6] = g;
    }
  }
  if (stop || !do_update) return;
  double acc = 0;
  unsigned long long um = 0;
  for (int64_t j = (int64_t)blockIdx.x * kThreads + threadIdx.x; j < a.n; j += (int64_t)gridDim.x * kThreads) {
    const double uo = a.u[j];
    a.x[j] += th * uo;
    const double un = (a.s[j] - mean) + beta * uo;
    a.u[j] = un;
    acc += un;
    const unsigned long long b = abs_bits(un);
    um = b > um ? b : um;
  }
  if (a.max_u) publish_absmax(um, a.max_u);
  double dummy;
  block_reduce2(acc, 0.0, &a.part[kPartU * kRed + blockIdx.x], &dummy);
}

// x += theta u only (last step, u not needed any more)
__global__ void final_x_kernel(Vecs a, const float* y, float* phi) {
  const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= a.n) return;
  const double delta = (double)y[1] - (double)y[0];
  phi[j] = (float)(a.x[j] + a.scal[2] * a.u[j] + delta / (double)a.n);
}

inline unsigned nblocks(int64_t n, int per) { return (unsigned)((n + per - 1) / per); }

// ---- hybrid storage of the small members (paired rows, sorted by size) ----
// cnt[r] = size of the small member of pair r; mail[0] = rows with cnt <= thr, mail[1] = 1 if not ascending
__global__ void pair_sizes_kernel(const int32_t* sz, int64_t R, int32_t thr, int32_t* cnt, int64_t* mail) {
  const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= R) return;
  const int32_t c = sz[2 * r];
  cnt[r] = c;
  if (c <= thr) atomicAdd((unsigned long long*)&mail[0], 1ull);
  if (r > 0 && sz[2 * (r - 1)] > c) atomicExch((unsigned long long*)&mail[1], 1ull);
}

// ---- small games: an iteration in two launches ----
// With a few thousand players and rows an iteration of the loop above is six launches of 3 to 11 us that each
// start by finishing the reduction of the one before, so what bounds it is the chain of launches. Here every
// workgroup redoes the vector work of all n (R) entries itself, straight into the LDS copy that its products gather
// from (a few dozen KB per workgroup, from L2), and only the owner of a slice writes it back. What is left is
//   forward: mean and |P s|^2 of the last adjoint, the stopping rule, x and u | d = (rows) u
//   adjoint: |v|^2 and theta, the residual, h                                 | s = (rows)^T h
// A kernel never writes what another workgroup of it may still read: u and the residual alternate between two
// buffers, the scalars between two records (forward reads the adjoint's and writes its own, and the other way
// round). Every operation, and the order of every sum, is that of the loop above (a sum over a vector goes lane by
// lane within 64 entries, then 64 by 64 within 256, then over the 256s), so the results are the same to the bit: CGLS
// turns the last bit of a product into the sixth digit of a score within 200 steps of a badly conditioned game.
// 3,001 players, 4,000 pairs, 200 iterations: 7.55 -> 3.84 ms (5.68 with the lanes' sums through LDS instead of
// ds_wave_sum; 7.17 with a workgroup on consecutive rows, whose dense end then sets the time).
constexpr int kSmallThreads = 1024;
constexpr int64_t kSmallPlayers = 4096;  // at most this many players ...
constexpr int64_t kSmallRows = 8192;     // ... and rows of the forward matrix (pairs, or rows): an LDS copy of 65 KB
constexpr int kSmallPitch = 65;          // doubles per 64-column word of the LDS copy: words start in different banks

enum SmallScalar { kGamma, kTheta, kDone, kIters, kRel, kGamma0, kSumU, kBufU, kSmallScalars };

struct SmallArgs {
  int n, R;
  int64_t Wf, stride_f, Wa;        // forward: rows of Z, Wf words of each, stride_f words apart; adjoint: Wa words per row
  const uint64_t *Z, *Zt;
  const double *sqw, *t;           // [k]
  double *x, *s, *d;
  double *u[2], *r[2];
  double *rec_f, *rec_a;           // scalar records of the two kernels
  double tol;
};

// Sum over a vector of up to N * kSmallThreads entries, entry tid + N' * kSmallThreads in v[N'] (zero past its end), in
// every thread. part: LDS, 16 N doubles of its own. One barrier.
template <int N>
__device__ __forceinline__ double small_sum(const double (&v)[N], double* part) {
  const int tid = threadIdx.x, lane = tid & 63;
#pragma unroll
  for (int i = 0; i < N; ++i) {
    const double a = ds_wave_sum(v[i]);
    if (lane == 0) part[i * (kSmallThreads / 64) + (tid >> 6)] = a;
  }
  __syncthreads();
  double p = 0.0;
  if (lane < N * (kSmallThreads / 256)) {
#pragma unroll
    for (int i = 0; i < 4; ++i) p += part[4 * lane + i];
  }
  return ds_wave_sum(p);
}

// index of the lowest set bit, 0xffffffff if there is none (what the instruction gives; __ffs adds a select)
__device__ __forceinline__ uint32_t first_bit(uint32_t x) {
  uint32_t r;
  asm("v_ffbl_b32 %0, %1" : "=v"(r) : "v"(x));
  return r;
}
// Sum of x[j] over the set bits j of w in ascending order; x[64] is zero (the spare entry of the pitch). What bounds the
// products is the instructions per set bit, so a bit costs one find-first per half, one three-way minimum that sends
// an empty word to the zero entry, and the 64-bit w & (w - 1); eight LDS reads are in flight.
__device__ __forceinline__ double small_word_sum(uint64_t w, const double* x) {
  double a = 0.0;
  while (w) {
    double v[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const uint32_t lo = first_bit((uint32_t)w), hi = first_bit((uint32_t)(w >> 32)) | 32u;
      const uint32_t bit = lo < hi ? lo : hi;
      v[q] = x[bit < 64u ? bit : 64u];
      w &= w - 1;  // 0 stays 0
    }
#pragma unroll
    for (int q = 0; q < 8; ++q) a += v[q];
  }
  return a;
}
// Sum of xs (pitched in LDS) over the set bits of one row of at most 128 words: a wave, lanes over words; w0 and w1 are
// the lane's words (word `lane` and word 64 + `lane`, zero past the row's end).
template <bool TWO>
__device__ __forceinline__ double small_row_sum(uint64_t w0, uint64_t w1, const double* xs) {
  const int lane = threadIdx.x & 63;
  double acc = small_word_sum(w0, xs + lane * kSmallPitch);
  if (TWO) acc += small_word_sum(w1, xs + (64 + lane) * kSmallPitch);
  return ds_wave_sum(acc);
}
__device__ __forceinline__ uint64_t small_word(const uint64_t* row, int64_t wd, int64_t W, int64_t cols) {
  if (wd >= W) return 0ull;
  return row[wd] & (wd == W - 1 && (cols & 63) ? ((1ull << (cols & 63)) - 1ull) : ~0ull);
}

// mode 0: a step; 1: the first one (u = s, x = 0); 2: only the stopping rule (one workgroup). ub: which u is current.
template <bool PAIRED, int N>   // N * kSmallThreads >= n
__global__ __launch_bounds__(kSmallThreads) void small_forward_kernel(SmallArgs a, int ub, int mode) {
  extern __shared__ double us[];
  __shared__ double part[3][N * (kSmallThreads / 64)];
  const int tid = threadIdx.x, lane = tid & 63;
  // rows ascend by size: a workgroup takes rows a grid apart, so that the dense ones are spread over all of them
  const int wave0 = (tid >> 6) * (int)gridDim.x + (int)blockIdx.x, waves = (int)gridDim.x * (kSmallThreads / 64);
  // everything that does not depend on another load is requested first
  const uint64_t* const row0 = a.Z + (int64_t)(wave0 < a.R ? wave0 : a.R - 1) * a.stride_f;
  uint64_t w0 = small_word(row0, lane, a.Wf, a.n);
  double sv[N], uo[N];
#pragma unroll
  for (int i = 0; i < N; ++i) {
    const int j = tid + i * kSmallThreads;
    sv[i] = j < a.n ? a.s[j] : 0.0;
    uo[i] = j < a.n && mode != 1 ? a.u[ub][j] : 0.0;
  }
  if (tid < (int)a.Wf) us[tid * kSmallPitch + 64] = 0.0;
  const double gamma = a.rec_a[kGamma], theta = a.rec_a[kTheta], gamma0 = a.rec_a[kGamma0];
  if (a.rec_a[kDone] != 0.0) {
    if (blockIdx.x == 0 && tid < kSmallScalars) a.rec_f[tid] = a.rec_a[tid];
    return;
  }
  const double mean = small_sum<N>(sv, part[0]) / (double)a.n;
  double sq[N];
#pragma unroll
  for (int i = 0; i < N; ++i) {
    const int j = tid + i * kSmallThreads;
    sv[i] = sv[i] - mean;
    sq[i] = j < a.n ? sv[i] * sv[i] : 0.0;
  }
  const double g = small_sum<N>(sq, part[1]);
  const double rel = mode == 1 ? 1.0 : sqrt(g) / sqrt(gamma0);
  const bool stop = mode == 1 ? !(g > 0.0) : rel <= a.tol;
  const bool step = mode == 1 || (!stop && mode != 2);   // (u_0 = s_0 is part of the result even if nothing follows)
  const double beta = mode == 1 || !(gamma > 0.0) ? 0.0 : g / gamma;
  double U = 0.0;
  if (step) {
#pragma unroll
    for (int i = 0; i < N; ++i) {
      const int j = tid + i * kSmallThreads;
      sv[i] = j < a.n ? sv[i] + beta * uo[i] : 0.0;
      if (j < a.n) us[(j >> 6) * kSmallPitch + (j & 63)] = sv[i];
    }
    U = small_sum<N>(sv, part[2]);   // (its barrier also completes us for the products)
  }
  if (blockIdx.x == 0 && tid == 0) {
    a.rec_f[kGamma] = step ? g : gamma;
    a.rec_f[kTheta] = theta;
    a.rec_f[kDone] = stop ? 1.0 : 0.0;
    a.rec_f[kIters] = a.rec_a[kIters] + (mode == 1 ? 0.0 : 1.0);
    a.rec_f[kRel] = rel;
    a.rec_f[kGamma0] = mode == 1 ? g : gamma0;
    a.rec_f[kSumU] = U;
    a.rec_f[kBufU] = (double)(step ? ub ^ 1 : ub);
  }
  if (!step) return;
  for (int i = wave0; i < a.R; i += waves) {
    if (i != wave0) w0 = small_word(a.Z + (int64_t)i * a.stride_f, lane, a.Wf, a.n);
    const double d = small_row_sum<false>(w0, 0ull, us);
    if (lane == 0) a.d[i] = d;
  }
  // the slice of x and u that this workgroup owns
  const int per = (a.n + (int)gridDim.x - 1) / (int)gridDim.x, own0 = (int)blockIdx.x * per, own1 = own0 + per;
#pragma unroll
  for (int i = 0; i < N; ++i) {
    const int j = tid + i * kSmallThreads;
    if (j < a.n && j >= own0 && j < own1) {
      a.x[j] = mode == 1 ? 0.0 : a.x[j] + theta * uo[i];
      a.u[ub ^ 1][j] = sv[i];
    }
  }
}

// first: the residual is still the right-hand side's, no step to take off it. rb: which residual is current.
template <bool PAIRED, int N>   // N * kSmallThreads >= R
__global__ __launch_bounds__(kSmallThreads) void small_adjoint_kernel(SmallArgs a, int rb, int first) {
  extern __shared__ double hs[];
  __shared__ double part[N * (kSmallThreads / 64)];
  const int tid = threadIdx.x, lane = tid & 63;
  // rows ascend by size: a workgroup takes rows a grid apart, so that the dense ones are spread over all of them
  const int wave0 = (tid >> 6) * (int)gridDim.x + (int)blockIdx.x, waves = (int)gridDim.x * (kSmallThreads / 64);
  const uint64_t* const row0 = a.Zt + (int64_t)(wave0 < a.n ? wave0 : a.n - 1) * a.Wa;
  uint64_t w0 = small_word(row0, lane, a.Wa, a.R), w1 = small_word(row0, 64 + lane, a.Wa, a.R);
  if (tid < (int)a.Wa) hs[tid * kSmallPitch + 64] = 0.0;
  double d[N], w[N], r0[N], r1[N];
#pragma unroll
  for (int i = 0; i < N; ++i) {
    const int q = tid + i * kSmallThreads;
    const bool in = q < a.R;
    w[i] = in ? a.sqw[PAIRED ? 2 * q : q] : 0.0;
    d[i] = in && !first ? a.d[q] : 0.0;
    r1[i] = 0.0;
    if (first) {
      r0[i] = in ? w[i] * a.t[PAIRED ? 2 * q : q] : 0.0;
      if (PAIRED && in) r1[i] = a.sqw[2 * q + 1] * a.t[2 * q + 1];
    } else {
      r0[i] = in ? a.r[rb][PAIRED ? 2 * q : q] : 0.0;
      if (PAIRED && in) r1[i] = a.r[rb][2 * q + 1];
    }
  }
  double theta = 0.0;
  if (!first) {
    const double gamma = a.rec_f[kGamma], U = a.rec_f[kSumU];
    if (a.rec_f[kDone] != 0.0) {
      if (blockIdx.x == 0 && tid < kSmallScalars) a.rec_a[tid] = a.rec_f[tid];
      return;
    }
    double vv[N];
#pragma unroll
    for (int i = 0; i < N; ++i) {
      const double v0 = w[i] * d[i], v1 = w[i] * (U - d[i]);
      vv[i] = PAIRED ? v0 * v0 + v1 * v1 : v0 * v0;
    }
    const double delta = small_sum<N>(vv, part);
    const bool null_dir = !(delta > 0.0);   // a direction in the null space ends the iteration with theta = 0
    theta = null_dir ? 0.0 : gamma / delta;
    if (blockIdx.x == 0 && tid < kSmallScalars)
      a.rec_a[tid] = tid == kTheta ? theta : tid == kDone ? (null_dir ? 1.0 : 0.0) : tid == kIters && null_dir ? a.rec_f[tid] + 1.0 : a.rec_f[tid];
    if (null_dir) return;
#pragma unroll
    for (int i = 0; i < N; ++i) {
      r0[i] -= theta * (w[i] * d[i]);
      if (PAIRED) r1[i] -= theta * (w[i] * (U - d[i]));
    }
  } else if (blockIdx.x == 0 && tid < kSmallScalars) {
    a.rec_a[tid] = 0.0;
  }
  const int per = (a.R + (int)gridDim.x - 1) / (int)gridDim.x, own0 = (int)blockIdx.x * per, own1 = own0 + per;
#pragma unroll
  for (int i = 0; i < N; ++i) {
    const int q = tid + i * kSmallThreads;
    if (q < a.R) {
      hs[(q >> 6) * kSmallPitch + (q & 63)] = w[i] * (PAIRED ? r0[i] - r1[i] : r0[i]);
      if (q >= own0 && q < own1) {
        a.r[rb ^ 1][PAIRED ? 2 * q : q] = r0[i];
        if (PAIRED) a.r[rb ^ 1][2 * q + 1] = r1[i];
      }
    }
  }
  __syncthreads();
  for (int j = wave0; j < a.n; j += waves) {
    if (j != wave0) {
      const uint64_t* row = a.Zt + (int64_t)j * a.Wa;
      w0 = small_word(row, lane, a.Wa, a.R);
      w1 = small_word(row, 64 + lane, a.Wa, a.R);
    }
    const double sj = a.Wa > 64 ? small_row_sum<true>(w0, w1, hs) : small_row_sum<false>(w0, 0ull, hs);
    if (lane == 0) a.s[j] = sj;
  }
}

// the last step's x += theta u is folded into the output (theta is 0 if no step was taken)
__global__ void small_final_kernel(SmallArgs a, const double* rec, const float* y, float* phi) {
  const int j = (int)(blockIdx.x * blockDim.x + threadIdx.x);
  if (j >= a.n) return;
  const double delta = (double)y[1] - (double)y[0];
  phi[j] = (float)(a.x[j] + rec[kTheta] * a.u[(int)rec[kBufU]][j] + delta / (double)a.n);
}

constexpr int64_t kHybridMinPlayers = 4096;  // below this the plain bit walk is already cheap
constexpr int32_t kDenseDiv = 64;            // pair rows with more than n / 64 players are multiplied as bitmaps

// The loop of the small games: see the kernels above. Zt: the transposed copy of the forward matrix's rows.
template <bool PAIRED>
int solve_small(ds_ctx* ctx, const SmallArgs& a, int grid, int max_iter, const float* y, float* phi, int* iters_out,
                double* relres_out, bool* converged_out) {
  hipStream_t st = ctx->stream;
  const unsigned lds_f = (unsigned)(a.Wf * kSmallPitch * 8), lds_a = (unsigned)(a.Wa * kSmallPitch * 8);
  static_assert(kSmallPlayers <= 4 * kSmallThreads && kSmallRows <= 8 * kSmallThreads, "entries per thread");
  void (*const fwd)(SmallArgs, int, int) = a.n <= 2 * kSmallThreads ? small_forward_kernel<PAIRED, 2> : small_forward_kernel<PAIRED, 4>;
  void (*const adj)(SmallArgs, int, int) = a.R <= 2 * kSmallThreads   ? small_adjoint_kernel<PAIRED, 2>
                                           : a.R <= 4 * kSmallThreads ? small_adjoint_kernel<PAIRED, 4>
                                                                      : small_adjoint_kernel<PAIRED, 8>;
  if (lds_a > 48 * 1024) DS_HIP(ctx, hipFuncSetAttribute((const void*)adj, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_a));
  int ub = 0, rb = 0;   // (a run that has stopped leaves both buffers alone: the record says which u is the last)
  auto adjoint = [&](int first) {
    hipLaunchKernelGGL(adj, dim3(grid), dim3(kSmallThreads), lds_a, st, a, rb, first);
    rb ^= 1;
  };
  auto forward = [&](int mode) {
    hipLaunchKernelGGL(fwd, dim3(mode == 2 ? 1 : grid), dim3(kSmallThreads), lds_f, st, a, ub, mode);
    ub ^= 1;
  };
  adjoint(1);
  forward(1);
  DS_TRY(ds_kernel_mark(ctx, 3, 0));
  // The scalars come back every kBurst iterations and are looked at while the next burst is already queued: what runs
  // after the iteration that stopped only copies them on.
  constexpr int kBurst = 16;
  hipEvent_t seen[2] = {ctx->fork2_ev, ctx->join2_ev};
  int launched = 0, bursts = 0, looked = 0;
  const double* rec = nullptr;
  auto look = [&]() -> int {
    DS_HIP(ctx, hipEventSynchronize(seen[looked & 1]));
    rec = (const double*)(ctx->h_mail + 16 * (looked & 1));
    ++looked;
    return DS_OK;
  };
  while (launched < max_iter && !(rec && rec[kDone] != 0.0)) {
    const int burst = max_iter - launched < kBurst ? max_iter - launched : kBurst;
    for (int b = 0; b < burst; ++b) {
      adjoint(0);
      forward(launched + b + 1 == max_iter ? 2 : 0);   // the last iteration allowed takes no further step
    }
    launched += burst;
    DS_HIP(ctx, hipGetLastError());
    DS_HIP(ctx, hipMemcpyAsync(ctx->h_mail + 16 * (bursts & 1), a.rec_f, kSmallScalars * 8, hipMemcpyDeviceToHost, st));
    DS_HIP(ctx, hipEventRecord(seen[bursts & 1], st));
    ++bursts;
    if (bursts - looked == 2) DS_TRY(look());
  }
  while (looked < bursts) DS_TRY(look());
  DS_TRY(ds_kernel_mark(ctx, 3, 1));
  hipLaunchKernelGGL(small_final_kernel, dim3(nblocks(a.n, 256)), dim3(256), 0, st, a, a.rec_f, y, phi);
  DS_HIP(ctx, hipGetLastError());
  DS_HIP(ctx, hipStreamSynchronize(st));
  *iters_out = (int)rec[kIters];
  *relres_out = rec[kGamma0] > 0.0 ? rec[kRel] : 0.0;
  *converged_out = rec[kDone] != 0.0;
  return DS_OK;
}

}  // namespace

size_t ds_cgls_arena_bytes(int64_t n, int64_t k) {
  const int64_t KW = (k + 63) / 64;
  // The hybrid storage never exceeds 1.5 x the plain transposed bitmap: the transposed bitmap of the dense pair rows
  // is at most half of it, and the index lists of the sparse rows (needed while their tiles are built) and the tile
  // entries take 4 bytes per set bit of rows with at most n/32 of them each. Plus offsets, the scratch of the two
  // matrix-core products (digit planes, per-group digit sums) and of the tile products (per-group partial vectors,
  // tile counters).
  const size_t tile_scratch = ds_align((size_t)(2 * (k / 32768) + 160) * n * 8) + ds_align((size_t)32 * k * 8) +
                              ds_align((size_t)(k / 8192 + 160) * (n / 8192 + 2) * 8);
  const size_t hybrid = 3 * ds_align((size_t)n * KW * 8) + 4 * ds_align((n + 2) * 4) + 2 * ds_align((k + 2) * 4) +
                        ds_align(112 * (size_t)(n > k ? n : k)) + ((size_t)80 << 20) + tile_scratch +
                        4 * ds_scan_arena_bytes(n > k ? n + 1 : k + 1);
  return hybrid + 2 * ds_align(k * 4) + 7 * ds_align(k * 8) + 5 * ds_align(n * 8) + 131072 + 2 * kRed * 8;
}

int ds_solve_cgls_impl(ds_ctx* ctx, int64_t n, int64_t k, const uint64_t* Z, const float* w, const float* y, int paired,
                       double tol, int max_iter, float* phi, int* iters_out, double* relres_out) {
  hipStream_t st = ctx->stream;
  const int64_t W = (n + 63) / 64;
  if (paired && (k & 1)) return ds_fail(ctx, DS_EINVAL, "paired rows need an even row count");
  const int64_t R = paired ? k / 2 : k;
  const int64_t RW = (R + 63) / 64;
  if (tol <= 0) tol = 1e-6;
  if (max_iter <= 0) max_iter = (int)(n < 10000 ? n : 10000);

  int32_t* sz = (int32_t*)ds_arena_alloc(ctx, k * 4);
  float* wc = (float*)ds_arena_alloc(ctx, k * 4);
  double* t = (double*)ds_arena_alloc(ctx, k * 8);
  Vecs a;
  a.n = n; a.k = k; a.R = R; a.paired = paired;
  double* sqw = (double*)ds_arena_alloc(ctx, k * 8);
  a.sqw = sqw;
  a.r = (double*)ds_arena_alloc(ctx, k * 8);
  a.v = (double*)ds_arena_alloc(ctx, k * 8);
  a.d = (double*)ds_arena_alloc(ctx, R * 8);
  a.h = (double*)ds_arena_alloc(ctx, R * 8);
  a.x = (double*)ds_arena_alloc(ctx, n * 8);
  a.u = (double*)ds_arena_alloc(ctx, n * 8);
  a.s = (double*)ds_arena_alloc(ctx, n * 8);
  a.scal = (double*)ds_arena_alloc(ctx, 128);
  a.part = (double*)ds_arena_alloc(ctx, 4 * kRed * 8);
  if (!sz || !wc || !t || !sqw || !a.r || !a.v || !a.d || !a.h || !a.x || !a.u || !a.s || !a.scal || !a.part)
    return ds_fail(ctx, DS_EINTERNAL, "cgls: arena exhausted");

  DS_TRY(ds_row_prep(ctx, Z, k, n, paired, w, y, sz, t, sqw, wc));

  // Few players and few rows (from kHybridMinPlayers on the fixed-point products take over; more rows do not fit the
  // LDS copy): an iteration in two launches.
  static_assert(kHybridMinPlayers <= kSmallPlayers, "the small kernels hold one word of a forward row per lane");
  if (n < kHybridMinPlayers && R <= kSmallRows) {
    uint64_t* Zt = (uint64_t*)ds_arena_alloc(ctx, (size_t)n * RW * 8);
    double* u1 = (double*)ds_arena_alloc(ctx, n * 8);
    double* rec = (double*)ds_arena_alloc(ctx, 256);
    if (!Zt || !u1 || !rec) return ds_fail(ctx, DS_EINTERNAL, "cgls: arena exhausted");
    DS_TRY(ds_bit_transpose(ctx, Z, R, n, W, 0, paired ? 2 : 1, Zt));
    DS_HIP(ctx, hipMemsetAsync(rec, 0, 256, st));
    SmallArgs q;
    q.n = (int)n; q.R = (int)R;
    q.Wf = W; q.stride_f = paired ? 2 * W : W; q.Wa = RW;
    q.Z = Z; q.Zt = Zt;
    q.sqw = sqw; q.t = t;
    q.x = a.x; q.s = a.s; q.d = a.d;
    q.u[0] = a.u; q.u[1] = u1;
    q.r[0] = a.r; q.r[1] = a.v;
    q.rec_f = rec; q.rec_a = rec + 16;
    q.tol = tol;
    ctx->cgls_bytes_per_iter = 2.0 * (double)R * (double)W * 8.0;
    const int64_t longest = n > R ? n : R;
    int64_t grid = (longest + kSmallThreads / 64 - 1) / (kSmallThreads / 64);
    if (grid > ctx->num_cus) grid = ctx->num_cus;
    int it = 0;
    double rel = 0.0;
    bool converged = false;
    DS_TRY(paired ? solve_small<true>(ctx, q, (int)grid, max_iter, y, phi, &it, &rel, &converged)
                  : solve_small<false>(ctx, q, (int)grid, max_iter, y, phi, &it, &rel, &converged));
    if (iters_out) *iters_out = it;
    if (relres_out) *relres_out = rel;
    if (!converged) return ds_fail(ctx, DS_ENOTCONV, "CGLS reached max_iter=%d with relative residual %.3e (tol %.1e)", max_iter, rel, tol);
    return DS_OK;
  }

  // ---- storage for the two products ----
  // Paired, size-sorted rows of a large game: the small members with at most n/div players become
  // (row, column) entries in 2-D tiles that serve both products through LDS, the denser tail stays a
  // bitmap (rows of Z itself, plus a transposed copy) and is multiplied on the matrix cores; both
  // in fixed point with exact integer sums. Otherwise: plain bitmap and its transpose, set bits walked
  // one by one in fp64.
  bool hybrid = false;
  int64_t Rs = 0, Rd = 0, RdW = 0, RdS = 0, nnz_s = 0;
  uint64_t *Zt = nullptr, *Ztd = nullptr;
  ds_mm_plan mm_f = {}, mm_a = {};   // dense rows: forward (Rd x n) and adjoint (n x Rd) products
  ds_tile_plan tiles = {};           // sparse rows: one entry list for both products
  double *scal_f = nullptr, *scal_a = nullptr;  // [0] scale of the forward / adjoint product's integers
  if (paired && n >= kHybridMinPlayers && n < ((int64_t)1 << 28)) {   // (the matrix-core product addresses rows with 32 bits)
    int32_t* cnt = (int32_t*)ds_arena_alloc(ctx, (R + 1) * 4);
    if (!cnt) return ds_fail(ctx, DS_EINTERNAL, "cgls: arena exhausted");
    DS_HIP(ctx, hipMemsetAsync(ctx->d_mail, 0, 4 * sizeof(int64_t), st));
    const int32_t dense_div = ctx->tuning.cgls_dense_div >= 32 ? ctx->tuning.cgls_dense_div : kDenseDiv;   // below 32 the index lists outgrow the bitmap
    const int32_t thr = (int32_t)(n / dense_div);
    hipLaunchKernelGGL(pair_sizes_kernel, dim3(nblocks(R, 256)), dim3(256), 0, st, sz, R, thr, cnt, ctx->d_mail);
    DS_TRY(ds_mail_fetch(ctx, 4));
    if (ctx->h_mail[1] == 0) {
      hybrid = true;
      Rs = ctx->h_mail[0];
      Rd = R - Rs;
      RdW = (Rd + 63) / 64;
      // rows of the transposed bitmap start at cache lines where that makes them at most an eighth longer (300,007 rows of 133 words,
      // the adjoint product alone: 84 -> 76 us)
      RdS = (RdW + 15) & ~(int64_t)15;
      if (8 * RdS > 9 * RdW) RdS = RdW;
      int32_t* csr_off = (int32_t*)ds_arena_alloc(ctx, (Rs + 2) * 4);
      if (!csr_off) return ds_fail(ctx, DS_EINTERNAL, "cgls: arena exhausted");
      DS_HIP(ctx, hipMemsetAsync(cnt + Rs, 0, 4, st));  // the scan's last slot: total
      DS_TRY(ds_scan_exclusive_i32(ctx, cnt, csr_off, Rs + 1, ctx->d_mail + 2));
      DS_TRY(ds_mail_fetch(ctx, 4));
      nnz_s = ctx->h_mail[2];
      if (nnz_s > 0x7fff0000LL) return ds_fail(ctx, DS_EINTERNAL, "cgls: too many set bits in the sparse rows (%lld)", (long long)nnz_s);
      Ztd = (uint64_t*)ds_arena_alloc(ctx, (size_t)n * (RdS > 0 ? RdS : 1) * 8 + 8);   // (rows of one word are read in pairs)
      void* ws_f = ds_arena_alloc(ctx, ds_bit_spmv_mm_ws_bytes(ctx, Rd, n));
      void* ws_a = ds_arena_alloc(ctx, ds_bit_spmv_mm_ws_bytes(ctx, n, Rd));
      void* ws_t = ds_arena_alloc(ctx, ds_tile_ws_bytes(ctx, Rs, n, nnz_s));
      scal_f = (double*)ds_arena_alloc(ctx, 256 + 2 * kRed * 8);   // scalars, then max_u and max_h
      int32_t* csr_idx = (int32_t*)ds_arena_alloc(ctx, (nnz_s + 1) * 4);   // (index lists; the tile build keeps the memory)
      if (!Ztd || !ws_f || !ws_a || !ws_t || !scal_f || !csr_idx) return ds_fail(ctx, DS_EINTERNAL, "cgls: arena exhausted");
      scal_a = scal_f + 16;
      DS_HIP(ctx, hipMemsetAsync(scal_f, 0, 256, st));
      if (Rd > 0) {
        DS_TRY(ds_bit_spmv_mm_prepare(ctx, Rd, n, ws_f, &mm_f));
        DS_TRY(ds_bit_spmv_mm_prepare(ctx, n, Rd, ws_a, &mm_a));
        DS_TRY(ds_bit_transpose(ctx, Z, Rd, n, W, 2 * Rs, 2, Ztd, RdS));
      }
      if (Rs > 0) {
        DS_TRY(ds_rows_to_csr(ctx, Z, Rs, n, W, 0, 2, csr_off, csr_idx));
        DS_TRY(ds_tile_build(ctx, Rs, n, nnz_s, thr > 1 ? thr : 1, csr_off, csr_idx, ws_t, &tiles));
      }
      DS_HIP(ctx, hipGetLastError());
    }
  }
  if (!hybrid) {
    Zt = (uint64_t*)ds_arena_alloc(ctx, (size_t)n * RW * 8);
    if (!Zt) return ds_fail(ctx, DS_EINTERNAL, "cgls: arena exhausted");
    DS_TRY(ds_bit_transpose(ctx, Z, R, n, W, 0, paired ? 2 : 1, Zt));
  }
  // Hybrid layout: the vector is brought into fixed point by the tile product; the sparse rows' tiles and the dense
  // rows' bitmap are multiplied one after the other (side by side on two streams they only competed for memory
  // bandwidth and the iteration took 8 % longer), the dense product adding the sparse result in the adjoint.
  const unsigned red_n = nblocks(n, kThreads) < (unsigned)kRed ? nblocks(n, kThreads) : (unsigned)kRed;
  const unsigned red_r = nblocks(R, kThreads) < (unsigned)kRed ? nblocks(R, kThreads) : (unsigned)kRed;
  a.max_u = hybrid ? (unsigned long long*)(scal_f + 32) : nullptr;
  a.max_h = hybrid ? a.max_u + kRed : nullptr;
  // with_absmax = 0: the kernel that wrote the vector has left its workgroups' maxima
  // d (sv) == nullptr: the integer partial sums are left for the loop's kernels
  auto forward = [&](const double* u, double* d, int with_absmax) -> int {  // d = (rows) . u
    if (!hybrid) return ds_bit_spmv(ctx, Z, R, n, W, 0, paired ? 2 : 1, u, d);
    if (with_absmax) DS_TRY(ds_vec_absmax(ctx, u, n, a.max_u, (int)red_n));
    DS_TRY(ds_tile_spmv(ctx, &tiles, 0, u, a.max_u, (int)red_n, &mm_f, u, scal_f, d));
    if (Rd > 0) DS_TRY(ds_bit_spmv_mm_product(ctx, &mm_f, Z, W, 2 * Rs, 2, scal_f, nullptr, d ? d + Rs : nullptr));
    return DS_OK;
  };
  auto adjoint = [&](const double* h, double* sv, int with_absmax) -> int {  // s = (rows)^T . h
    if (!hybrid) return ds_bit_spmv(ctx, Zt, n, R, RW, 0, 1, h, sv);
    if (with_absmax) DS_TRY(ds_vec_absmax(ctx, h, R, a.max_h, (int)red_r));
    DS_TRY(ds_tile_spmv(ctx, &tiles, 1, h, a.max_h, (int)red_r, &mm_a, h + Rs, scal_a, sv));
    if (Rd > 0) DS_TRY(ds_bit_spmv_mm_product(ctx, &mm_a, Ztd, RdS, 0, 1, scal_a, sv && Rs > 0 ? sv : nullptr, sv));
    return DS_OK;
  };
  a.fused = hybrid ? 1 : 0;
  a.Rs = Rs;
  a.fwd = ds_fixed_view_of(&tiles, &mm_f, 0);
  a.adj = ds_fixed_view_of(&tiles, &mm_a, 1);
  a.scal_f = scal_f;
  a.scal_a = scal_a;
  // what one iteration must read of the matrix: the bitmap rows of both orientations and 4 bytes per tile entry, twice
  ctx->cgls_bytes_per_iter = hybrid ? 2.0 * ((double)Rd * (double)W * 8.0 + 4.0 * (double)nnz_s)
                                    : 2.0 * (double)R * (double)W * 8.0;
  DS_HIP(ctx, hipMemsetAsync(a.x, 0, n * 8, st));
  DS_HIP(ctx, hipMemsetAsync(a.u, 0, n * 8, st));
  DS_HIP(ctx, hipMemsetAsync(a.scal, 0, 128, st));

  // lanes per entry in the two kernels that add up the products' partial sums: short vectors take 4 or 16, so that
  // enough loads are in flight
  auto lanes_for = [&](int64_t len) { return !hybrid ? 1 : len * 16 <= 262144 ? 16 : len * 4 <= 262144 ? 4 : 1; };
  const int lanes_v = lanes_for(R), lanes_s = lanes_for(n);
  const unsigned grid_v = nblocks(R * lanes_v, kThreads) < (unsigned)kRed ? nblocks(R * lanes_v, kThreads) : (unsigned)kRed;
  const unsigned grid_s = nblocks(n * lanes_s, kThreads) < (unsigned)kRed ? nblocks(n * lanes_s, kThreads) : (unsigned)kRed;
  auto launch_make_v = [&]() {
    if (lanes_v == 16) hipLaunchKernelGGL(loop_make_v_kernel<16>, dim3(grid_v), dim3(kThreads), 0, st, a, (int)red_n);
    else if (lanes_v == 4) hipLaunchKernelGGL(loop_make_v_kernel<4>, dim3(grid_v), dim3(kThreads), 0, st, a, (int)red_n);
    else hipLaunchKernelGGL(loop_make_v_kernel<1>, dim3(grid_v), dim3(kThreads), 0, st, a, (int)red_n);
  };
  auto launch_s_sum = [&]() {
    if (lanes_s == 16) hipLaunchKernelGGL(loop_s_sum_kernel<16>, dim3(grid_s), dim3(kThreads), 0, st, a);
    else if (lanes_s == 4) hipLaunchKernelGGL(loop_s_sum_kernel<4>, dim3(grid_s), dim3(kThreads), 0, st, a);
    else hipLaunchKernelGGL(loop_s_sum_kernel<1>, dim3(grid_s), dim3(kThreads), 0, st, a);
  };

  // s_0 = P A^T r_0, u_0 = s_0
  hipLaunchKernelGGL(init_r_kernel, dim3(nblocks(k, 256)), dim3(256), 0, st, a, t);
  hipLaunchKernelGGL(make_h_kernel, dim3(nblocks(R, 256)), dim3(256), 0, st, a);
  DS_TRY(adjoint(a.h, a.s, 1));
  hipLaunchKernelGGL(s_sum_kernel, dim3(red_n), dim3(kThreads), 0, st, a);
  hipLaunchKernelGGL(fin_mean_kernel, dim3(1), dim3(64), 0, st, a, (int)red_n);
  hipLaunchKernelGGL(s_center_kernel, dim3(red_n), dim3(kThreads), 0, st, a);
  hipLaunchKernelGGL(fin_gamma_kernel, dim3(1), dim3(64), 0, st, a, (int)red_n, 1);
  {
    Vecs au = a;  // the partial sums of u live in their own array (the loop's first kernel adds them up)
    au.part = a.part + kPartU * kRed;
    hipLaunchKernelGGL(update_xu_kernel, dim3(red_n), dim3(kThreads), 0, st, au);  // theta = beta = 0: u = s
    hipLaunchKernelGGL(fin_u_kernel, dim3(1), dim3(64), 0, st, au, (int)red_n);
  }
  DS_HIP(ctx, hipGetLastError());
  DS_HIP(ctx, hipMemcpyAsync(ctx->h_mail, a.scal, 64, hipMemcpyDeviceToHost, st));
  DS_HIP(ctx, hipStreamSynchronize(st));
  const double gamma0 = ((double*)ctx->h_mail)[7];
  int it = 0;
  double rel = gamma0 > 0 ? 1.0 : 0.0;
  bool converged = !(gamma0 > 0);
  DS_TRY(ds_kernel_mark(ctx, 3, 0));
  // The stopping rule runs on the device; the host reads the scalars back every kCheckEvery iterations
  // (kernels queued after the iteration that stopped leave the result alone).
  constexpr int kCheckEvery = 8;
  int launched = 0;
  while (!converged && launched < max_iter) {
    const int burst = max_iter - launched < kCheckEvery ? max_iter - launched : kCheckEvery;
    for (int b = 0; b < burst; ++b) {
      DS_TRY(forward(a.u, hybrid ? nullptr : a.d, launched + b == 0 ? 1 : 0));   // (the first u comes from the set-up, not from the loop's kernel)
      launch_make_v();
      hipLaunchKernelGGL(loop_update_r_kernel, dim3(red_r), dim3(kThreads), 0, st, a, (int)grid_v);
      DS_TRY(adjoint(a.h, hybrid ? nullptr : a.s, 0));
      launch_s_sum();
      // the last iteration allowed takes no further step: it only evaluates the stopping rule
      hipLaunchKernelGGL(loop_update_xu_kernel, dim3(red_n), dim3(kThreads), 0, st, a, (int)grid_s, kThreads / lanes_s, tol,
                         launched + b + 1 < max_iter ? 1 : 0);
    }
    launched += burst;
    DS_HIP(ctx, hipGetLastError());
    DS_HIP(ctx, hipMemcpyAsync(ctx->h_mail, a.scal, 128, hipMemcpyDeviceToHost, st));
    DS_HIP(ctx, hipStreamSynchronize(st));
    const double* sc = (const double*)ctx->h_mail;
    it = (int)sc[9];
    if (sc[10] > 0.0 || it > 0) rel = sc[10] > 0.0 ? sc[10] : rel;
    if (sc[8] != 0.0) converged = true;
  }
  DS_TRY(ds_kernel_mark(ctx, 3, 1));
  // the last step's x += theta u is folded into the output (theta is 0 if no step was taken)
  hipLaunchKernelGGL(final_x_kernel, dim3(nblocks(n, 256)), dim3(256), 0, st, a, y, phi);
  DS_HIP(ctx, hipGetLastError());
  DS_HIP(ctx, hipStreamSynchronize(st));
  if (iters_out) *iters_out = it;
  if (relres_out) *relres_out = rel;
  if (!converged) {
    ds_fail(ctx, DS_ENOTCONV, "CGLS reached max_iter=%d with relative residual %.3e (tol %.1e)", max_iter, rel, tol);
    return DS_ENOTCONV;
  }
  return DS_OK;
}
