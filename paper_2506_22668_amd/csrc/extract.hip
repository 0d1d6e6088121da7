// k-hop computational-graph extraction on the device.
//
// Paper, "Computational graph": an L-layer GNN's prediction for v depends only on
// v's 1..L-hop neighbours and the edges among them; that induced sub-graph G_c(v)
// is what the explanation works on, and its edges are the players. The steps here:
// level-synchronous BFS along CSR rows (in-neighbours), local ids in ascending
// (hop, global id) order by prefix sums, induced sub-CSR by ordered wave
// compaction, player ids in ascending global (a, b) order, and a gather of the
// feature rows.
#include "internal.h"

namespace {

constexpr int kThreads = 256;
constexpr int kScanItems = 8;                       // per thread
constexpr int kScanTile = kThreads * kScanItems;    // per block

// ---------------- exclusive prefix sum (int32), three phases ----------------

__device__ __forceinline__ int block_reduce_sum(int v, int* sh) {
  for (int o = 32; o > 0; o >>= 1) v += __shfl_down(v, o, 64);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if (lane == 0) sh[wave] = v;
  __syncthreads();
  int total = 0;
  for (int i = 0; i < kThreads / 64; ++i) total += sh[i];
  __syncthreads();
  return total;
}

__global__ __launch_bounds__(kThreads) void scan_tile_sums(const int32_t* in, int64_t count, int32_t* tile_sums) {
  __shared__ int sh[kThreads / 64];
  const int64_t base = (int64_t)blockIdx.x * kScanTile;
  int s = 0;
  for (int i = 0; i < kScanItems; ++i) {
    const int64_t idx = base + (int64_t)i * kThreads + threadIdx.x;
    if (idx < count) s += in[idx];
  }
  const int total = block_reduce_sum(s, sh);
  if (threadIdx.x == 0) tile_sums[blockIdx.x] = total;
}

// single block: exclusive scan of the tile sums in place; total -> mail slot
__global__ __launch_bounds__(kThreads) void scan_tile_offsets(int32_t* tile_sums, int64_t tiles, int64_t* total_out) {
  __shared__ int sh[kThreads];
  __shared__ long long carry;
  if (threadIdx.x == 0) carry = 0;
  __syncthreads();
  for (int64_t base = 0; base < tiles; base += kThreads) {
    const int64_t idx = base + threadIdx.x;
    const int v = idx < tiles ? tile_sums[idx] : 0;
    sh[threadIdx.x] = v;
    __syncthreads();
    for (int o = 1; o < kThreads; o <<= 1) {  // Hillis-Steele inclusive scan
      int add = threadIdx.x >= o ? sh[threadIdx.x - o] : 0;
      __syncthreads();
      sh[threadIdx.x] += add;
      __syncthreads();
    }
    const long long c = carry;
    if (idx < tiles) tile_sums[idx] = (int32_t)(c + sh[threadIdx.x] - v);
    __syncthreads();
    if (threadIdx.x == kThreads - 1) carry = c + sh[kThreads - 1];
    __syncthreads();
  }
  if (threadIdx.x == 0 && total_out) *total_out = carry;
}

__global__ __launch_bounds__(kThreads) void scan_apply(const int32_t* in, int32_t* out, int64_t count,
                                                       const int32_t* tile_offsets) {
  __shared__ int sh[kThreads];
  const int64_t base = (int64_t)blockIdx.x * kScanTile + (int64_t)threadIdx.x * kScanItems;
  int v[kScanItems];
  int s = 0;
  for (int i = 0; i < kScanItems; ++i) {
    v[i] = (base + i < count) ? in[base + i] : 0;
    s += v[i];
  }
  sh[threadIdx.x] = s;
  __syncthreads();
  for (int o = 1; o < kThreads; o <<= 1) {
    int add = threadIdx.x >= o ? sh[threadIdx.x - o] : 0;
    __syncthreads();
    sh[threadIdx.x] += add;
    __syncthreads();
  }
  int run = tile_offsets[blockIdx.x] + sh[threadIdx.x] - s;
  for (int i = 0; i < kScanItems; ++i) {
    if (base + i < count) out[base + i] = run;
    run += v[i];
  }
}

// short inputs: the whole exclusive scan in one launch. Every thread owns a contiguous run of items: it sums
// them, the 1024 run sums are scanned in LDS, and the thread then walks its run again (out may alias in: a
// run is read and written by its owner only, after every first pass is over).
constexpr int kSmallScanThreads = 1024;
constexpr int64_t kSmallScanMax = 4096;  // beyond a few items per thread the strided runs cost more than two extra launches
__global__ __launch_bounds__(kSmallScanThreads) void scan_small_kernel(const int32_t* in, int32_t* out, int64_t count,
                                                                       int64_t* total_out) {
  __shared__ int sh[kSmallScanThreads];
  const int tid = threadIdx.x;
  const int64_t per = (count + kSmallScanThreads - 1) / kSmallScanThreads;
  const int64_t b = (int64_t)tid * per, e = b + per < count ? b + per : count;
  int s = 0;
  for (int64_t i = b; i < e; ++i) s += in[i];
  sh[tid] = s;
  __syncthreads();
  for (int o = 1; o < kSmallScanThreads; o <<= 1) {  // Hillis-Steele inclusive scan of the run sums
    const int add = tid >= o ? sh[tid - o] : 0;
    __syncthreads();
    sh[tid] += add;
    __syncthreads();
  }
  int run = sh[tid] - s;
  for (int64_t i = b; i < e; ++i) {
    const int v = in[i];
    out[i] = run;
    run += v;
  }
  if (tid == kSmallScanThreads - 1 && total_out) *total_out = sh[tid];
}

}  // namespace

size_t ds_scan_arena_bytes(int64_t count) {
  const int64_t tiles = (count + kScanTile - 1) / kScanTile;
  return ds_align((tiles + 1) * sizeof(int32_t));
}

// out may alias in. The grand total goes to mail slot `total_mail_slot` (device side) if not null.
int ds_scan_exclusive_i32(ds_ctx* ctx, const int32_t* in, int32_t* out, int64_t count, int64_t* total_mail_slot) {
  if (count <= 0) {
    if (total_mail_slot) DS_HIP(ctx, hipMemsetAsync(total_mail_slot, 0, sizeof(int64_t), ctx->stream));
    return DS_OK;
  }
  if (count <= kSmallScanMax) {
    hipLaunchKernelGGL(scan_small_kernel, dim3(1), dim3(kSmallScanThreads), 0, ctx->stream, in, out, count, total_mail_slot);
    DS_HIP(ctx, hipGetLastError());
    return DS_OK;
  }
  const int64_t tiles = (count + kScanTile - 1) / kScanTile;
  int32_t* tile_sums = (int32_t*)ds_arena_alloc(ctx, (tiles + 1) * sizeof(int32_t));
  if (!tile_sums) return ds_fail(ctx, DS_EINTERNAL, "scan: arena exhausted");
  hipLaunchKernelGGL(scan_tile_sums, dim3((unsigned)tiles), dim3(kThreads), 0, ctx->stream, in, count, tile_sums);
  hipLaunchKernelGGL(scan_tile_offsets, dim3(1), dim3(kThreads), 0, ctx->stream, tile_sums, tiles, total_mail_slot);
  hipLaunchKernelGGL(scan_apply, dim3((unsigned)tiles), dim3(kThreads), 0, ctx->stream, in, out, count, tile_sums);
  DS_HIP(ctx, hipGetLastError());
  return DS_OK;
}

namespace {

// ---------------- CSR validation ----------------
__global__ void validate_csr_kernel(const int64_t* row_ptr, const int32_t* col, int64_t N, int64_t nnz, int* bad) {
  const int lane = threadIdx.x & 63;
  const int64_t wave = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
  const int64_t nwaves = ((int64_t)gridDim.x * blockDim.x) >> 6;
  for (int64_t i = wave; i < N; i += nwaves) {
    const int64_t a = row_ptr[i], b = row_ptr[i + 1];
    if (a > b || a < 0 || b > nnz) {
      if (lane == 0) atomicExch(bad, 1);
      continue;
    }
    for (int64_t e = a + lane; e < b; e += 64) {
      const int32_t c = col[e];
      if (c < 0 || c >= N || (e > a && col[e - 1] >= c)) atomicExch(bad, 2);
    }
  }
}

// ---------------- BFS ----------------
__global__ void fill_i32(int32_t* p, int64_t count, int32_t v) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < count) p[i] = v;
}

// mail layout (int64 slots): [0..7] level counts, [8] nnz_c, [9] players, [10] error, [11] members, [12] the hop before which
// ball_small_kernel gave up, [13] the frontier it leaves, [40..47] CSR entries of the rows within h hops
__global__ void bfs_seed(int32_t* dist, int32_t* frontier, int64_t* mail, int64_t target) {
  dist[target] = 0;
  frontier[0] = (int32_t)target;
  for (int i = 0; i < 16; ++i) mail[i] = 0;
  mail[0] = 1;
}

__global__ __launch_bounds__(kThreads) void bfs_visit(const int64_t* row_ptr, const int32_t* col, int32_t* dist,
                                                      const int32_t* frontier, int32_t* next, int64_t* mail, int level) {
  const int lane = threadIdx.x & 63;
  const int64_t wave = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
  const int64_t nwaves = ((int64_t)gridDim.x * blockDim.x) >> 6;
  const int64_t count = mail[level - 1];
  unsigned long long* next_count = (unsigned long long*)&mail[level];
  for (int64_t f = wave; f < count; f += nwaves) {
    const int64_t i = frontier[f];
    const int64_t a = row_ptr[i], b = row_ptr[i + 1];
    for (int64_t e = a + lane; e < b; e += 64) {
      const int32_t j = col[e];
      if (atomicCAS(&dist[j], -1, level) == -1) {
        const unsigned long long pos = atomicAdd(next_count, 1ull);
        next[pos] = j;
      }
    }
  }
}

// flags over the expanded index space h*N + g (local order = hop, then global id)
__global__ void member_flags(const int32_t* dist, int64_t N, int levels, int32_t* level_flag, int32_t* member_flag) {
  const int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (g >= N) return;
  const int d = dist[g];
  member_flag[g] = d >= 0 ? 1 : 0;
  for (int h = 0; h < levels; ++h) level_flag[(int64_t)h * N + g] = (d == h) ? 1 : 0;
}

struct GraphOut {
  int32_t* row_ptr;
  int32_t* col;
  int32_t* eid;
  int2* pl;
  int64_t* node_gid;
  int32_t* hop;
  float* Xc;
};

__global__ void assign_nodes(const int32_t* dist, const int32_t* lid_scan, const int32_t* rank_scan, int64_t N,
                             int64_t* node_gid, int32_t* hop, int32_t* lid_of_rank) {
  const int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (g >= N) return;
  const int d = dist[g];
  if (d < 0) return;
  const int32_t lid = lid_scan[(int64_t)d * N + g];
  node_gid[lid] = g;
  hop[lid] = d;
  lid_of_rank[rank_scan[g]] = lid;
}

// one wave per member (in global-id rank order): count induced entries and upper entries
__global__ __launch_bounds__(kThreads) void count_entries(const int64_t* row_ptr, const int32_t* col, const int32_t* dist,
                                                          const int64_t* node_gid, const int32_t* lid_of_rank, const int64_t* members,
                                                          int32_t* cnt_all_lid, int32_t* cnt_all_rank, int32_t* cnt_up_rank) {
  const int64_t V = *members;
  const int lane = threadIdx.x & 63;
  const int64_t wave = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
  const int64_t nwaves = ((int64_t)gridDim.x * blockDim.x) >> 6;
  for (int64_t rk = wave; rk < V; rk += nwaves) {
    const int32_t lid = lid_of_rank[rk];
    const int64_t g = node_gid[lid];
    const int64_t a = row_ptr[g], b = row_ptr[g + 1];
    int all = 0, up = 0;
    for (int64_t e = a + lane; e < b; e += 64) {
      const int32_t j = col[e];
      if (j != g && dist[j] >= 0) {
        ++all;
        if (j > g) ++up;
      }
    }
    for (int o = 32; o > 0; o >>= 1) {
      all += __shfl_down(all, o, 64);
      up += __shfl_down(up, o, 64);
    }
    if (lane == 0) {
      cnt_all_lid[lid] = all;
      cnt_all_rank[rk] = all;
      cnt_up_rank[rk] = up;
    }
  }
}

// one wave per member: ordered compaction of its row into the local CSR, player ids
// for the entries this row owns (undirected: neighbours with larger global id;
// directed: every entry), and the member's own entries of the per-node arrays and its feature row. The local id of node j at
// hop d is lid[d * lid_stride + j].
__global__ __launch_bounds__(kThreads) void fill_entries(const int64_t* row_ptr, const int32_t* col, const int32_t* dist,
                                                         const int32_t* lid_scan, int64_t lid_stride, const int32_t* lid_of_rank,
                                                         const int32_t* player_start_rank, const int32_t* row_start,
                                                         const int64_t* node_gid, const int32_t* hop, const float* X, int d0,
                                                         int64_t V, int directed, GraphOut out) {
  const int lane = threadIdx.x & 63;
  const int64_t wave = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
  const int64_t nwaves = ((int64_t)gridDim.x * blockDim.x) >> 6;
  const unsigned long long lt = (1ull << lane) - 1ull;
  for (int64_t rk = wave; rk < V; rk += nwaves) {
    const int32_t lid = lid_of_rank[rk];
    const int64_t g = node_gid[lid];
    const int64_t a = row_ptr[g], b = row_ptr[g + 1];
    int32_t pos = row_start[lid];
    if (lane == 0) {
      out.row_ptr[lid] = pos;
      out.node_gid[lid] = g;
      out.hop[lid] = hop[lid];
      if (rk == 0) out.row_ptr[V] = row_start[V];
    }
    int32_t ppos = player_start_rank[rk];
    for (int64_t e0 = a; e0 < b; e0 += 64) {
      const int64_t e = e0 + lane;
      int32_t j = -1, d = -1;
      if (e < b) {
        j = col[e];
        d = dist[j];
      }
      const bool in = (j >= 0) && (j != g) && (d >= 0);
      const bool own = in && (directed || j > g);
      const unsigned long long m_in = __ballot(in), m_own = __ballot(own);
      if (in) {
        const int32_t jl = lid_scan[(int64_t)d * lid_stride + j];
        const int32_t at = pos + __popcll(m_in & lt);
        out.col[at] = jl;
        int32_t p = -1;
        if (own) {
          p = ppos + __popcll(m_own & lt);
          out.pl[p] = directed ? make_int2(jl, lid) : make_int2(lid, jl);
        }
        out.eid[at] = p;
      }
      pos += __popcll(m_in);
      ppos += __popcll(m_own);
    }
    constexpr int kAhead = 4;
    for (int f0 = lane; f0 < d0; f0 += 64 * kAhead) {   // (its loads in flight together; past the end the last feature is read again)
      float x[kAhead];
#pragma unroll
      for (int u = 0; u < kAhead; ++u) x[u] = X[g * d0 + (f0 + 64 * u < d0 ? f0 + 64 * u : d0 - 1)];
#pragma unroll
      for (int u = 0; u < kAhead; ++u)
        if (f0 + 64 * u < d0) out.Xc[(int64_t)lid * d0 + f0 + 64 * u] = x[u];
    }
  }
}

// undirected: entries (row b, neighbour a) with gid(a) < gid(b) look their player
// up in a's owned range (ascending in the global id of the far end). unmatched: host memory, set if one has none.
__global__ void backfill_entries(GraphOut out, const int32_t* rank_scan, const int32_t* player_start_rank, int64_t V,
                                 volatile int64_t* unmatched) {
  const int lane = threadIdx.x & 63;
  const int64_t wave = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
  const int64_t nwaves = ((int64_t)gridDim.x * blockDim.x) >> 6;
  for (int64_t t = wave; t < V; t += nwaves) {
    const int64_t g = out.node_gid[t];
    for (int32_t e = out.row_ptr[t] + lane; e < out.row_ptr[t + 1]; e += 64) {
      if (out.eid[e] >= 0) continue;
      const int32_t al = out.col[e];
      const int64_t ag = out.node_gid[al];
      const int32_t rk = rank_scan[ag];
      int32_t lo = player_start_rank[rk], hi = player_start_rank[rk + 1];
      int32_t found = -1;
      while (lo < hi) {
        const int32_t mid = (lo + hi) >> 1;
        const int64_t bg = out.node_gid[out.pl[mid].y];
        if (bg == g) {
          found = mid;
          break;
        }
        if (bg < g) lo = mid + 1; else hi = mid;
      }
      if (found < 0) *unmatched = 1;
      out.eid[e] = found < 0 ? 0 : found;
    }
  }
}

// ---------------- small graphs: the ball in one workgroup ----------------
//
// Everything up to the sizes of the computational graph is a chain of nineteen launches that do nothing for most of their
// 3 - 5 us, and two round trips. One workgroup with a thread per 64 nodes keeps the nodes of every hop as a bitmap in LDS: a
// claim is an atomic OR, and the rank of a node among those of its hop is a prefix sum of popcounts, so that nothing has to be
// sorted; two more launches count the entries. ds_extract of 16 players in 10,000 nodes: 135 -> 52 us; 3,000 players in
// 60,000 nodes, 1,000 rows visited: 155 -> 104 us. Bound by the latency of the visited rows, which one workgroup has to itself:
// past the limits below it hands over the hops it has (slot 12), the whole GPU visits the others, and the nodes are numbered by a
// workgroup to 1,024 of them, each of which counts all the others for itself.
// ds_extract of 4,000 players, 1,200 rows in hop 2, 160 -> 102 us (the scans of the general kernels behind a workgroup that gave up: 190);
// 62,000 players, 800 rows in hop 1, 375 -> 343 us (407).
constexpr int kBallThreads = 1024;
constexpr int64_t kBallNodes = 64 * kBallThreads;   // a thread to a word of the bitmaps
constexpr int kBallRows = 1024;                     // rows visited per hop, a thread to each
constexpr int kBallEntries = 16384;                 // entries of all rows visited
constexpr int kBallWaves = kBallThreads / 64;

size_t ball_lds_bytes(int64_t N, int levels) {
  const size_t words = (size_t)((N + 63) / 64);
  return words * (size_t)(levels + 1) * 12 + (size_t)kBallRows * 20 + 16;
}

// inclusive sum over the wave
__device__ __forceinline__ int wave_scan(int v) {
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int up = __shfl_up(v, o, 64);
    if ((int)(threadIdx.x & 63) >= o) v += up;
  }
  return v;
}

__global__ __launch_bounds__(kBallThreads) void ball_small_kernel(const int64_t* row_ptr, const int32_t* col, int64_t N, int hops,
                                                                  int32_t target, int32_t* dist, int32_t* lid, int32_t* rank,
                                                                  int64_t* node_gid, int32_t* hop, int32_t* lid_of_rank,
                                                                  int64_t* mail, unsigned long long* maps_out) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem_ball[];
  __shared__ int wave_sums[DS_MAX_HOPS + 2][kBallWaves];
  __shared__ int totals[DS_MAX_HOPS + 2];
  __shared__ int claimed, entries;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int levels = hops + 1, words = (int)((N + 63) / 64);
  unsigned long long* const maps = (unsigned long long*)smem_ball;   // one per hop, then all members
  unsigned long long* const all = maps + levels * words;
  int64_t* const row_at = (int64_t*)(all + words);
  int* const row_len = (int*)(row_at + kBallRows);
  int* cur = row_len + kBallRows;
  int* next = cur + kBallRows;
  int* const before = next + kBallRows;   // [map][word]: nodes of the map in the words before
  for (int i = tid; i < words * (levels + 1); i += kBallThreads) maps[i] = 0ull;
  __syncthreads();
  if (tid == 0) {
    maps[target >> 6] = all[target >> 6] = 1ull << (target & 63);
    cur[0] = target;
    entries = 0;
  }
  int count = 1, left = 0;   // left: the hop before which it gives up
  for (int h = 1; h <= hops; ++h) {
    __syncthreads();   // `cur` is complete, the counters have been read
    if (tid == 0) claimed = 0;
    if (tid < count) {
      const int g = cur[tid];
      const int64_t a = row_ptr[g], len = row_ptr[g + 1] - a;
      row_at[tid] = a;
      row_len[tid] = (int)(len < kBallEntries + 1 ? len : kBallEntries + 1);
      atomicAdd(&entries, row_len[tid]);
    }
    __syncthreads();
    if (entries > kBallEntries) {
      left = h;
      break;
    }
    for (int f = wave; f < count; f += kBallWaves) {
      const int32_t* row = col + row_at[f];
      for (int e = lane; e < row_len[f]; e += 64) {
        const int j = row[e];
        const unsigned long long bit = 1ull << (j & 63);
        if (atomicOr(&all[j >> 6], bit) & bit) continue;
        atomicOr(&maps[h * words + (j >> 6)], bit);
        if (h < hops) {
          const int pos = atomicAdd(&claimed, 1);
          if (pos < kBallRows) next[pos] = j;
        }
      }
    }
    __syncthreads();
    if (h < hops) count = claimed;
    if (count > kBallRows) {
      left = h + 1;
      break;
    }
    int* const t = cur;
    cur = next;
    next = t;
  }
  if (left) {   // (no members: the kernels queued behind this one have nothing to do)
    for (int i = tid; i < words * left; i += kBallThreads) maps_out[i] = maps[i];
    if (tid < 16) mail[tid] = tid == left - 1 ? count : tid == 12 ? left : 0;
    return;
  }
  for (int q = 0; q <= levels; ++q) {
    const int c = tid < words ? __popcll(maps[q * words + tid]) : 0;
    const int incl = wave_scan(c);
    if (tid < words) before[q * words + tid] = incl - c;
    if (lane == 63) wave_sums[q][wave] = incl;
  }
  __syncthreads();
  if (tid <= levels) {
    int v[kBallWaves], run = 0;
#pragma unroll
    for (int w = 0; w < kBallWaves; ++w) v[w] = wave_sums[tid][w];
#pragma unroll
    for (int w = 0; w < kBallWaves; ++w) {
      wave_sums[tid][w] = run;
      run += v[w];
    }
    totals[tid] = run;
  }
  __syncthreads();
  if (tid < 16) mail[tid] = tid < levels ? totals[tid] : tid == 11 ? totals[levels] : 0;
  for (int g = tid; g < (int)N; g += kBallThreads) {
    const int w = g >> 6;
    const unsigned long long bit = 1ull << (g & 63), members = all[w];
    if (!(members & bit)) {
      dist[g] = -1;
      continue;
    }
    int d = 0, first = 0;   // local ids ascend by hop, then by global id
    while (!(maps[d * words + w] & bit)) first += totals[d++];
    const int l = first + wave_sums[d][w >> 6] + before[d * words + w] + __popcll(maps[d * words + w] & (bit - 1ull));
    const int rk = wave_sums[levels][w >> 6] + before[levels * words + w] + __popcll(members & (bit - 1ull));
    dist[g] = d;
    lid[g] = l;
    rank[g] = rk;
    node_gid[l] = g;
    hop[l] = d;
    lid_of_rank[rk] = l;
  }
}

// `levels` bitmaps of hops -> distances (-1: none), and the nodes of the last of them as the frontier of bfs_visit
__global__ void ball_unpack_kernel(const unsigned long long* maps, int64_t N, int levels, int32_t* dist, int32_t* frontier, int64_t* mail) {
  const int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x, words = (N + 63) / 64;
  if (g >= N) return;
  int d = -1;
  for (int q = 0; q < levels; ++q)
    if ((maps[q * words + (g >> 6)] >> (g & 63)) & 1ull) d = q;
  dist[g] = d;
  if (d == levels - 1) frontier[atomicAdd((unsigned long long*)&mail[13], 1ull)] = (int32_t)g;
}

// ball_small_kernel's numbering from the distances, a workgroup to 1,024 nodes: each counts the nodes of every hop among all nodes and
// among those before its own (a byte per hop and thread: 64 nodes at most)
__global__ __launch_bounds__(kBallThreads) void ball_rank_kernel(const int32_t* dist, int64_t N, int levels, int32_t* lid, int32_t* rank,
                                                                 int64_t* node_gid, int32_t* hop, int32_t* lid_of_rank, int64_t* mail) {
  __shared__ unsigned long long sums[kBallWaves][4];
  __shared__ int own[DS_MAX_HOPS + 2][kBallWaves];     // this workgroup's nodes of a hop (of any, last), by wave
  __shared__ int total[DS_MAX_HOPS + 1], first[DS_MAX_HOPS + 2];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int n = (int)N, base = (int)blockIdx.x * kBallThreads, g = base + tid;
  unsigned long long before = 0ull, all = 0ull;
  auto count = [&](int i, int d) {
    if (d < 0) return;
    all += 1ull << (8 * d);
    if (i < base) before += 1ull << (8 * d);
  };
  for (int i = 4 * tid; i < n; i += 4 * kBallThreads) {
    if (i + 3 < n) {
      const int4 d = *(const int4*)(dist + i);
      count(i, d.x);
      count(i + 1, d.y);
      count(i + 2, d.z);
      count(i + 3, d.w);
    } else {
      for (int u = i; u < n; ++u) count(u, dist[u]);
    }
  }
  // (64 lanes: 16 bits to a hop, the even and the odd ones apart)
  const unsigned long long even = 0x00ff00ff00ff00ffull;
  unsigned long long part[4] = {all & even, (all >> 8) & even, before & even, (before >> 8) & even};
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    for (int o = 32; o > 0; o >>= 1) part[i] += __shfl_xor(part[i], o, 64);
    if (lane == 0) sums[wave][i] = part[i];
  }
  const int d = g < n ? dist[g] : -1;
  const unsigned long long lt = (1ull << lane) - 1ull, members = __ballot(d >= 0);
  int in_hop = 0;   // nodes of the same hop in the wave before this lane
  for (int q = 0; q < levels; ++q) {
    const unsigned long long m = __ballot(d == q);
    if (d == q) in_hop = __popcll(m & lt);
    if (lane == 0) own[q][wave] = __popcll(m);
  }
  if (lane == 0) own[levels][wave] = __popcll(members);
  __syncthreads();
  if (tid < levels) {
    int t = 0, f = 0;
    for (int w = 0; w < kBallWaves; ++w) {
      t += (int)(sums[w][tid & 1] >> (16 * (tid >> 1))) & 0xffff;
      f += (int)(sums[w][2 + (tid & 1)] >> (16 * (tid >> 1))) & 0xffff;
    }
    total[tid] = t;
    first[tid] = f;
  }
  __syncthreads();
  if (tid <= levels) {   // exclusive sums over the waves, from the nodes before this workgroup's on
    int run = 0;
    if (tid < levels) {
      run = first[tid];
    } else {
      for (int q = 0; q < levels; ++q) run += first[q];
    }
    for (int w = 0; w < kBallWaves; ++w) {
      const int c = own[tid][w];
      own[tid][w] = run;
      run += c;
    }
  }
  if (blockIdx.x == 0 && tid < 16) {
    int v = 0;
    if (tid < levels) v = total[tid];
    else if (tid == 11)
      for (int q = 0; q < levels; ++q) v += total[q];
    mail[tid] = v;
  }
  __syncthreads();
  if (d < 0) return;
  int l = own[d][wave] + in_hop;   // local ids ascend by hop, then by global id
  for (int q = 0; q < d; ++q) l += total[q];
  const int rk = own[levels][wave] + __popcll(members & lt);
  lid[g] = l;
  rank[g] = rk;
  node_gid[l] = g;
  hop[l] = d;
  lid_of_rank[rk] = l;
}

// the members' entry and player counts into row and player starts (V + 1 each, in place), their totals and the entries of every
// ball: one workgroup, which leaves the mailbox with the host too (a copy behind it would be one more launch to wait for)
__global__ __launch_bounds__(kBallThreads) void ball_rows_kernel(int32_t* row_start, int32_t* player_start, int64_t* mail, int64_t* host_mail) {
  __shared__ int sums[2][kBallWaves];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int V = (int)mail[11];
  int ball[8], acc = 0;
#pragma unroll
  for (int h = 0; h < 8; ++h) {
    acc += (int)mail[h];
    ball[h] = acc;
  }
  int at_row = 0, at_player = 0;
  for (int base = 0; base <= V; base += kBallThreads) {
    const int i = base + tid;
    const int a = i < V ? row_start[i] : 0, b = i < V ? player_start[i] : 0;
    const int ia = wave_scan(a), ib = wave_scan(b);
    if (lane == 63) {
      sums[0][wave] = ia;
      sums[1][wave] = ib;
    }
    __syncthreads();
    int ea = at_row + ia - a, eb = at_player + ib - b;
#pragma unroll
    for (int w = 0; w < kBallWaves; ++w) {
      const int sa = sums[0][w], sb = sums[1][w];
      if (w < wave) {
        ea += sa;
        eb += sb;
      }
      at_row += sa;
      at_player += sb;
    }
    if (i <= V) {
      row_start[i] = ea;
      player_start[i] = eb;
#pragma unroll
      for (int h = 0; h < 8; ++h)
        if (ball[h] == i) mail[40 + h] = ea;
    }
    __syncthreads();
  }
  if (tid == 0) {
    mail[8] = at_row;
    mail[9] = at_player;
  }
  __syncthreads();
  if (tid < 48) host_mail[tid] = mail[tid];
}

// the same for many members, a workgroup to 1,024 of them, each of which sums the counts before its own for itself; into other
// arrays, the counts being read by all
__global__ __launch_bounds__(kBallThreads) void ball_rows_wide_kernel(const int32_t* row_count, const int32_t* player_count, int32_t* row_start,
                                                                      int32_t* player_start, int64_t* mail) {
  __shared__ int sums[2][kBallWaves], own[2][kBallWaves];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int V = (int)mail[11], base = (int)blockIdx.x * kBallThreads, i = base + tid;
  if (base > V) return;
  int sa = 0, sb = 0;
  for (int j = 4 * tid; j < base; j += 4 * kBallThreads) {
    const int4 a = *(const int4*)(row_count + j), b = *(const int4*)(player_count + j);
    sa += a.x + a.y + a.z + a.w;
    sb += b.x + b.y + b.z + b.w;
  }
  const int a = i < V ? row_count[i] : 0, b = i < V ? player_count[i] : 0;
  sa = wave_scan(sa);
  sb = wave_scan(sb);
  const int ia = wave_scan(a), ib = wave_scan(b);
  if (lane == 63) {
    sums[0][wave] = sa;
    sums[1][wave] = sb;
    own[0][wave] = ia;
    own[1][wave] = ib;
  }
  __syncthreads();
  int ea = ia - a, eb = ib - b;
#pragma unroll
  for (int w = 0; w < kBallWaves; ++w) {
    ea += sums[0][w] + (w < wave ? own[0][w] : 0);
    eb += sums[1][w] + (w < wave ? own[1][w] : 0);
  }
  if (i > V) return;
  row_start[i] = ea;
  player_start[i] = eb;
  int ball = 0;
  for (int h = 0; h < 8; ++h) {
    ball += (int)mail[h];
    if (ball == i) mail[40 + h] = ea;
  }
  if (i == V) {
    mail[8] = ea;
    mail[9] = eb;
  }
}

inline unsigned blocks_for(int64_t n, int per = kThreads) { return (unsigned)((n + per - 1) / per); }

}  // namespace

int ds_validate_csr(ds_ctx* ctx) {
  ds_arena_reset(ctx);
  DS_TRY(ds_arena_reserve(ctx, 4096));
  int* bad = (int*)ds_arena_alloc(ctx, 256);
  DS_HIP(ctx, hipMemsetAsync(bad, 0, sizeof(int), ctx->stream));
  DS_HIP(ctx, hipMemcpyAsync(ctx->h_mail, ctx->row_ptr, sizeof(int64_t), hipMemcpyDeviceToHost, ctx->stream));
  DS_HIP(ctx, hipMemcpyAsync(ctx->h_mail + 1, ctx->row_ptr + ctx->N, sizeof(int64_t), hipMemcpyDeviceToHost, ctx->stream));
  DS_HIP(ctx, hipStreamSynchronize(ctx->stream));
  if (ctx->h_mail[0] != 0 || ctx->h_mail[1] < 0)
    return ds_fail(ctx, DS_EINVAL, "row_ptr[0] must be 0 and row_ptr[N] >= 0");
  ctx->nnz = ctx->h_mail[1];
  if (ctx->N > 0) {
    hipLaunchKernelGGL(validate_csr_kernel, dim3(ctx->num_cus * 8), dim3(kThreads), 0, ctx->stream, ctx->row_ptr,
                       ctx->col, ctx->N, ctx->nnz, bad);
    DS_HIP(ctx, hipGetLastError());
  }
  DS_HIP(ctx, hipMemcpyAsync(ctx->h_mail, bad, sizeof(int), hipMemcpyDeviceToHost, ctx->stream));
  DS_HIP(ctx, hipStreamSynchronize(ctx->stream));
  const int code = *(int*)ctx->h_mail;
  ds_arena_reset(ctx);
  if (code == 1) return ds_fail(ctx, DS_EINVAL, "row_ptr is not monotone within [0, nnz]");
  if (code == 2) return ds_fail(ctx, DS_EINVAL, "col has an id outside [0, N) or a row that is not strictly ascending");
  return DS_OK;
}

namespace {
__global__ void zero_three_kernel(int32_t* a, int32_t* b, int32_t* c) {
  if (threadIdx.x == 0) {
    *a = 0;
    *b = 0;
    *c = 0;
  }
}
struct BallSizes { int32_t v[8]; };
// out[h] = row_ptr[ball[h]]: the CSR entries of the rows within h hops
__global__ void ball_entries_kernel(const int32_t* row_ptr, BallSizes b, int64_t* out) {
  if (threadIdx.x < 8) out[threadIdx.x] = row_ptr[b.v[threadIdx.x]];
}
}  // namespace

int ds_extract_impl(ds_ctx* ctx, int64_t target, int hops, int directed, ds_cgraph** out_cg) {
  if (!ctx->row_ptr) return ds_fail(ctx, DS_EINVAL, "ds_set_graph has not been called");
  if (!ctx->X) return ds_fail(ctx, DS_EINVAL, "ds_set_features has not been called");
  if (target < 0 || target >= ctx->N) return ds_fail(ctx, DS_EINVAL, "target %lld outside [0, %lld)", (long long)target, (long long)ctx->N);
  if (hops < 1 || hops > DS_MAX_HOPS) return ds_fail(ctx, DS_EINVAL, "hops must be in [1, %d]", DS_MAX_HOPS);
  const int64_t N = ctx->N;
  const int levels = hops + 1;
  hipStream_t st = ctx->stream;

  // phase 1 temporaries, all O(N)
  ds_arena_reset(ctx);
  size_t need = ds_align((N + 1) * 4) * 16 + ds_align((size_t)levels * N * 4) +
                ds_scan_arena_bytes((int64_t)levels * N) + 4 * ds_scan_arena_bytes(N + 1) + 65536;
  DS_TRY(ds_arena_reserve(ctx, need));
  int64_t* mail = ctx->d_mail;
  int64_t V = 0, ball[8] = {0};
  auto ball_sizes = [&]() -> int {   // from the level counts and the member count in the mailbox
    V = ctx->h_mail[11];
    int64_t acc = 0;
    for (int h = 0; h <= hops; ++h) {
      acc += ctx->h_mail[h];
      ball[h] = acc;
    }
    if (acc != V) return ds_fail(ctx, DS_EINTERNAL, "extract: level counts (%lld) disagree with member count (%lld)", (long long)acc, (long long)V);
    return DS_OK;
  };
  int32_t *dist = nullptr, *rank_scan = nullptr, *lid_scan = nullptr, *lid_of_rank = nullptr, *hop_tmp = nullptr, *rowptr_tmp = nullptr;
  int32_t *cnt_all_rank = nullptr, *cnt_up_rank = nullptr;
  int64_t *node_gid_tmp = nullptr, lid_stride = N;
  // phase 2 temporaries, one entry for each of up to v nodes
  auto member_arrays = [&](int64_t v) {
    node_gid_tmp = (int64_t*)ds_arena_alloc(ctx, v * 8);
    hop_tmp = (int32_t*)ds_arena_alloc(ctx, v * 4);
    lid_of_rank = (int32_t*)ds_arena_alloc(ctx, v * 4);
    rowptr_tmp = (int32_t*)ds_arena_alloc(ctx, (v + 1) * 4);
    cnt_all_rank = (int32_t*)ds_arena_alloc(ctx, (v + 1) * 4);
    cnt_up_rank = (int32_t*)ds_arena_alloc(ctx, (v + 1) * 4);
    return node_gid_tmp && hop_tmp && lid_of_rank && rowptr_tmp && cnt_all_rank && cnt_up_rank;
  };
  const bool small = N <= kBallNodes;
  if (small) {
    dist = (int32_t*)ds_arena_alloc(ctx, N * 4);
    rank_scan = (int32_t*)ds_arena_alloc(ctx, N * 4);
    lid_scan = (int32_t*)ds_arena_alloc(ctx, N * 4);
    int32_t* cur = (int32_t*)ds_arena_alloc(ctx, N * 4);
    int32_t* nxt = (int32_t*)ds_arena_alloc(ctx, N * 4);
    unsigned long long* maps = (unsigned long long*)ds_arena_alloc(ctx, (size_t)(N + 63) / 64 * levels * 8);
    if (!dist || !rank_scan || !lid_scan || !cur || !nxt || !maps || !member_arrays(N)) return ds_fail(ctx, DS_EINTERNAL, "extract: arena exhausted");
    const size_t lds = ball_lds_bytes(N, levels);
    if (lds > 48 * 1024)
      DS_HIP(ctx, hipFuncSetAttribute((const void*)ball_small_kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
    hipLaunchKernelGGL(ball_small_kernel, dim3(1), dim3(kBallThreads), lds, st, ctx->row_ptr, ctx->col, N, hops, (int32_t)target, dist,
                       lid_scan, rank_scan, node_gid_tmp, hop_tmp, lid_of_rank, mail, maps);
    hipLaunchKernelGGL(count_entries, dim3(ctx->num_cus * 2), dim3(kThreads), 0, st, ctx->row_ptr, ctx->col, dist, node_gid_tmp, lid_of_rank,
                       mail + 11, rowptr_tmp, cnt_all_rank, cnt_up_rank);
    hipLaunchKernelGGL(ball_rows_kernel, dim3(1), dim3(kBallThreads), 0, st, rowptr_tmp, directed ? cnt_all_rank : cnt_up_rank, mail,
                       ctx->h_mail);
    DS_HIP(ctx, hipGetLastError());
    DS_HIP(ctx, hipStreamSynchronize(st));
    if (ctx->h_mail[12] != 0) {   // more than one workgroup's work
      int h = (int)ctx->h_mail[12];
      hipLaunchKernelGGL(ball_unpack_kernel, dim3(blocks_for(N)), dim3(kThreads), 0, st, maps, N, h, dist, cur, mail);
      for (; h <= hops; ++h) {
        hipLaunchKernelGGL(bfs_visit, dim3(ctx->num_cus * 4), dim3(kThreads), 0, st, ctx->row_ptr, ctx->col, dist, cur, nxt, mail, h);
        int32_t* t = cur; cur = nxt; nxt = t;
      }
      hipLaunchKernelGGL(ball_rank_kernel, dim3(blocks_for(N, kBallThreads)), dim3(kBallThreads), 0, st, dist, N, levels, lid_scan, rank_scan,
                         node_gid_tmp, hop_tmp, lid_of_rank, mail);
      hipLaunchKernelGGL(count_entries, dim3(ctx->num_cus * 8), dim3(kThreads), 0, st, ctx->row_ptr, ctx->col, dist, node_gid_tmp, lid_of_rank,
                         mail + 11, rowptr_tmp, cnt_all_rank, cnt_up_rank);
      int32_t* const rows_out = (int32_t*)ds_arena_alloc(ctx, (N + 1) * 4);
      int32_t* const players_out = (int32_t*)ds_arena_alloc(ctx, (N + 1) * 4);
      if (!rows_out || !players_out) return ds_fail(ctx, DS_EINTERNAL, "extract: arena exhausted");
      hipLaunchKernelGGL(ball_rows_wide_kernel, dim3(blocks_for(N + 1, kBallThreads)), dim3(kBallThreads), 0, st, rowptr_tmp,
                         directed ? cnt_all_rank : cnt_up_rank, rows_out, players_out, mail);
      rowptr_tmp = rows_out;
      cnt_all_rank = cnt_up_rank = players_out;
      DS_HIP(ctx, hipGetLastError());
      DS_TRY(ds_mail_fetch(ctx, 48));
    }
    DS_TRY(ball_sizes());
    lid_stride = 0;
  }
  const auto wave_blocks = [&]() { return (unsigned)((V * 64 + kThreads - 1) / kThreads < (int64_t)ctx->num_cus * 8 ? (V * 64 + kThreads - 1) / kThreads : (int64_t)ctx->num_cus * 8); };
  if (!small) {
    dist = (int32_t*)ds_arena_alloc(ctx, N * 4);
    int32_t* fr_a = (int32_t*)ds_arena_alloc(ctx, N * 4);
    int32_t* fr_b = (int32_t*)ds_arena_alloc(ctx, N * 4);
    rank_scan = (int32_t*)ds_arena_alloc(ctx, N * 4);
    lid_scan = (int32_t*)ds_arena_alloc(ctx, (size_t)levels * N * 4);
    if (!dist || !fr_a || !fr_b || !rank_scan || !lid_scan) return ds_fail(ctx, DS_EINTERNAL, "extract: arena exhausted");

    hipLaunchKernelGGL(fill_i32, dim3(blocks_for(N)), dim3(kThreads), 0, st, dist, N, -1);
    hipLaunchKernelGGL(bfs_seed, dim3(1), dim3(1), 0, st, dist, fr_a, mail, target);
    int32_t *cur = fr_a, *nxt = fr_b;
    for (int h = 1; h <= hops; ++h) {
      hipLaunchKernelGGL(bfs_visit, dim3(ctx->num_cus * 4), dim3(kThreads), 0, st, ctx->row_ptr, ctx->col, dist, cur, nxt, mail, h);
      int32_t* t = cur; cur = nxt; nxt = t;
    }
    hipLaunchKernelGGL(member_flags, dim3(blocks_for(N)), dim3(kThreads), 0, st, dist, N, levels, lid_scan, rank_scan);
    DS_HIP(ctx, hipGetLastError());
    DS_TRY(ds_scan_exclusive_i32(ctx, lid_scan, lid_scan, (int64_t)levels * N, nullptr));
    DS_TRY(ds_scan_exclusive_i32(ctx, rank_scan, rank_scan, N, mail + 11));
    DS_TRY(ds_mail_fetch(ctx, 16));
    DS_TRY(ball_sizes());
    if (V > 0x7ffffff0LL) return ds_fail(ctx, DS_EINVAL, "computational graph too large");

    // grow and redo would invalidate live buffers; the reserve above is sized by N >= V, so add headroom instead
    if (!member_arrays(V)) return ds_fail(ctx, DS_EINTERNAL, "extract: arena exhausted (phase 2)");
    hipLaunchKernelGGL(assign_nodes, dim3(blocks_for(N)), dim3(kThreads), 0, st, dist, lid_scan, rank_scan, N, node_gid_tmp, hop_tmp, lid_of_rank);
    hipLaunchKernelGGL(zero_three_kernel, dim3(1), dim3(64), 0, st, rowptr_tmp + V, cnt_all_rank + V, cnt_up_rank + V);
    hipLaunchKernelGGL(count_entries, dim3(wave_blocks()), dim3(kThreads), 0, st, ctx->row_ptr, ctx->col, dist, node_gid_tmp, lid_of_rank, mail + 11, rowptr_tmp, cnt_all_rank, cnt_up_rank);
    DS_HIP(ctx, hipGetLastError());
    DS_TRY(ds_scan_exclusive_i32(ctx, rowptr_tmp, rowptr_tmp, V + 1, mail + 8));
    int32_t* starts = directed ? cnt_all_rank : cnt_up_rank;
    DS_TRY(ds_scan_exclusive_i32(ctx, starts, starts, V + 1, mail + 9));
    BallSizes bs;   // number of CSR entries in the rows of every ball (rows are ordered by hop)
    for (int h = 0; h < 8; ++h) bs.v[h] = (int32_t)ball[h <= hops ? h : hops];
    hipLaunchKernelGGL(ball_entries_kernel, dim3(1), dim3(64), 0, st, rowptr_tmp, bs, mail + 40);
    DS_HIP(ctx, hipGetLastError());
    DS_HIP(ctx, hipMemcpyAsync(ctx->h_mail + 40, mail + 40, 8 * sizeof(int64_t), hipMemcpyDeviceToHost, st));
    DS_TRY(ds_mail_fetch(ctx, 16));
  }
  int32_t* const player_start = directed ? cnt_all_rank : cnt_up_rank;
  const int64_t nnz_c = ctx->h_mail[8];
  const int64_t n = ctx->h_mail[9];
  if (nnz_c > 0x7ffffff0LL) return ds_fail(ctx, DS_EINVAL, "computational graph has too many entries");
  if (!directed && nnz_c != 2 * n)
    return ds_fail(ctx, DS_EINVAL, "CSR is not symmetric inside the computational graph (entries %lld, pairs %lld): undirected players need both directions", (long long)nnz_c, (long long)n);

  // the computational graph itself: one allocation
  ds_cgraph* cg = new ds_cgraph();
  memset(cg, 0, sizeof(*cg));
  cg->owner = ctx;
  const int d0 = ctx->d0, d1 = ds_first_width(ctx);
  const int att_heads = ctx->model_kind == DS_MODEL_GAT && ctx->L > 0 ? ctx->gat.heads[0] : 0;
  size_t off = 0;
  auto carve = [&](size_t bytes) { size_t o = off; off += ds_align(bytes); return o; };
  const size_t o_rp = carve((V + 1) * 4), o_col = carve(nnz_c * 4 + 4), o_eid = carve(nnz_c * 4 + 4);
  const size_t o_pl = carve(n * 8 + 8), o_gid = carve(V * 8), o_hop = carve(V * 4);
  const size_t o_x = carve((size_t)V * d0 * 4), o_p = carve((size_t)V * (d1 > 0 ? d1 : 1) * 4);
  const size_t o_pred = carve(256);
  const size_t o_att = carve((size_t)V * att_heads * 8 + 8);
  if (ctx->cg_spare && ctx->cg_spare_bytes >= off) {
    cg->block = ctx->cg_spare;
    cg->block_bytes = ctx->cg_spare_bytes;
    ctx->cg_spare = nullptr;
    ctx->cg_spare_bytes = 0;
  } else {
    cg->block_bytes = off;
    if (hipMalloc(&cg->block, off) != hipSuccess) {
      (void)hipGetLastError();
      delete cg;
      return ds_fail(ctx, DS_ENOMEM, "extract: cannot allocate %zu bytes for the computational graph", off);
    }
  }
  char* base = (char*)cg->block;
  cg->row_ptr = (int32_t*)(base + o_rp);
  cg->col = (int32_t*)(base + o_col);
  cg->eid = (int32_t*)(base + o_eid);
  cg->pl = (int2*)(base + o_pl);
  cg->node_gid = (int64_t*)(base + o_gid);
  cg->hop = (int32_t*)(base + o_hop);
  cg->Xc = (float*)(base + o_x);
  cg->P = (float*)(base + o_p);
  cg->d_pred = (int32_t*)(base + o_pred);
  cg->att = (float*)(base + o_att);
  cg->pred_class = -1;
  cg->d0 = d0;
  cg->d1 = d1;
  cg->att_heads = att_heads;
  for (int h = 0; h < 8; ++h) cg->ball_entries[h] = ctx->h_mail[40 + h];
  cg->info.num_players = n;
  cg->info.num_nodes = V;
  cg->info.num_entries = nnz_c;
  cg->info.target = target;
  cg->info.hops = hops;
  cg->info.directed = directed;
  for (int h = 0; h < 8; ++h) cg->info.ball[h] = h <= hops ? ball[h] : ball[hops];
  ctx->graphs.push_back(cg);
  *out_cg = cg;

  ctx->h_mail[10] = 0;   // (nothing is under way: the sizes have been read)
  GraphOut go{cg->row_ptr, cg->col, cg->eid, cg->pl, cg->node_gid, cg->hop, cg->Xc};
  hipLaunchKernelGGL(fill_entries, dim3(wave_blocks()), dim3(kThreads), 0, st, ctx->row_ptr, ctx->col, dist, lid_scan, lid_stride, lid_of_rank,
                     player_start, rowptr_tmp, node_gid_tmp, hop_tmp, ctx->X, d0, V, directed, go);
  if (!directed && nnz_c > 0)
    hipLaunchKernelGGL(backfill_entries, dim3(wave_blocks()), dim3(kThreads), 0, st, go, rank_scan, player_start, V, ctx->h_mail + 10);
  DS_HIP(ctx, hipGetLastError());
  DS_HIP(ctx, hipStreamSynchronize(st));
  ds_arena_reset(ctx);
  if (ctx->h_mail[10] != 0) {
    ds_cgraph_free(ctx, cg);
    *out_cg = nullptr;
    return ds_fail(ctx, DS_EINVAL, "CSR is not symmetric inside the computational graph: an entry has no reverse entry");
  }
  return DS_OK;
}
