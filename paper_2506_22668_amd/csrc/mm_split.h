// How the matrix-core product of the bit-packed rows (bitmat.hip) is cut into the shares of its workgroups. For host and, the shares of an
// even cut, device.
#pragma once
#include <stdint.h>
#ifdef __HIPCC__
#define DS_MM_FN __host__ __device__ inline
#else
#define DS_MM_FN inline
#endif

struct ds_mm_split {
  int64_t cpg, groups;   // chunks per column group; column groups
};

// Column groups: a workgroup per row group and column group. Two workgroups fit a compute unit, so a launch runs in rounds of up
// to 2 x CUs of them. Every split is priced and the cheapest taken. A round costs, per chunk of its groups, 2.6 us with two
// workgroups on a unit, also where only some units hold two, and 1.6 with at most one on each: a workgroup waits for the
// latency of its loads and, where two share a unit, for the other. A group's digit sums (`sum_bytes` a row) are written
// and read once more by whoever adds them up: 1 us per MB. The three figures were fitted to the product on the int8 instruction, with 32
// bytes of sums a row, and the caller still states 32 where a row has 16. Their order of the splits holds for the present kernel: with
// the number of groups of either product of eleven games swept, and the even cut below, what is chosen was within 1.5 % of the
// fastest CGLS iteration but for two (us per iteration; tests/test_mm_split.py has the sweeps):
//   500,009 x 15,102: 562, one column group 542;  100,428 x 3,414: 75.4, one column group 73.8
inline double ds_mm_price(int64_t num_cus, int64_t wgs, int64_t chunks, int64_t sums) {
  const int64_t cap = 2 * num_cus, rest = wgs % cap;
  const double per_chunk = 2.6 * (double)(wgs / cap) + (rest == 0 ? 0.0 : rest <= num_cus ? 1.6 : 2.6);
  return (double)chunks * per_chunk + (double)sums * 1.0e-6;
}

inline ds_mm_split ds_mm_choose_split(int64_t num_cus, int64_t rows, int64_t row_groups, int64_t n_chunks, int64_t max_cpg,
                                      int64_t sum_bytes) {
  const int64_t cap = 2 * num_cus, rg = row_groups > 0 ? row_groups : 1;
  int64_t g_hi = (10 * cap + rg - 1) / rg;
  if (g_hi > n_chunks) g_hi = n_chunks;
  ds_mm_split best = {n_chunks > 0 ? n_chunks : 1, 1};
  double best_us = -1.0;
  for (int64_t g = 1; g <= g_hi; ++g) {
    int64_t cpg = (n_chunks + g - 1) / g;
    if (cpg > max_cpg) cpg = max_cpg;
    if (cpg < 1) cpg = 1;
    const int64_t groups = (n_chunks + cpg - 1) / cpg;
    const double us = ds_mm_price(num_cus, rg * groups, cpg, groups * rows * sum_bytes);
    if (best_us < 0.0 || us < best_us) {
      best_us = us;
      best.cpg = cpg;
      best.groups = groups;
    }
  }
  return best;
}

// The same work cut evenly: the units (a chunk of a row group each) of all row groups in one line, row group by row group; workgroup b of
// `wgs` takes units ds_mm_even_begin(b) to ds_mm_even_begin(b + 1) of u. A row group's sums then come from up to `slots` workgroups: each
// leaves its own in the slot that counts the workgroups from the row group's first one on.
struct ds_mm_even {
  int64_t wgs, slots;    // wgs == 0: the column groups are cheaper
};

DS_MM_FN int64_t ds_mm_even_begin(int64_t b, int64_t wgs, int64_t units) { return b * units / wgs; }
// the workgroup that holds unit x
DS_MM_FN int64_t ds_mm_even_owner(int64_t x, int64_t wgs, int64_t units) { return ((x + 1) * wgs - 1) / units; }

// A workgroup to a compute unit, 1.6 to 1.8 us a unit (with two: 3.2 to 4.1). A workgroup that holds a row group whole meets no more than
// two others' ends, so that what a cut within row groups costs is the second slot's sums (1 us per MB, as above). Taken where its price
// is below that of the column groups at the same cost of a unit; no more of one row group than the accumulators hold. (us per iteration, best
// number of column groups and even: 34,177 x 99,981 283, 276; 10,253 x 99,981 116.5, 116.3; 9,410 x 300,007 251, 249.)
inline ds_mm_even ds_mm_choose_even(int64_t num_cus, int64_t rows, int64_t row_groups, int64_t n_chunks, int64_t max_cpg,
                                    int64_t sum_bytes, const ds_mm_split& split) {
  const double unit_us = 1.8;
  ds_mm_even best = {0, 0};
  const int64_t units = row_groups * n_chunks, wgs = units < num_cus ? units : num_cus;
  if (units < 1) return best;
  const int64_t per = (units + wgs - 1) / wgs, rounds = (row_groups * split.groups + num_cus - 1) / num_cus;
  if ((per < n_chunks ? per : n_chunks) > max_cpg) return best;
  int64_t slots = 1;
  for (int64_t g = 0; g < row_groups; ++g) {
    const int64_t s = ds_mm_even_owner((g + 1) * n_chunks - 1, wgs, units) - ds_mm_even_owner(g * n_chunks, wgs, units) + 1;
    if (s > slots) slots = s;
  }
  const double sums = (double)(rows * sum_bytes) * 1.0e-6;
  if (unit_us * (double)per + sums * (double)slots < unit_us * (double)(rounds * split.cpg) + sums * (double)split.groups) {
    best.wgs = wgs;
    best.slots = slots;
  }
  return best;
}
