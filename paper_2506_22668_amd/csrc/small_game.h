// How the workgroups of small_gram_kernel (gram_chol.hip) share the pairs of players of a game of at most 64. For host and device.
#pragma once
#ifdef __HIPCC__
#define DS_SMALL_FN __host__ __device__ __forceinline__
#else
#define DS_SMALL_FN inline
#endif

constexpr int kSmallMax = 64;         // players
constexpr int kSmallThreads = 1024;
constexpr int kSmallPairs = kSmallMax * (kSmallMax + 1) / 2;
constexpr int kSmallPerThread = (kSmallPairs + kSmallThreads - 1) / kSmallThreads;

// The threads form `groups` groups of `width`, (at least) one thread to a pair, which take the rows in turn: thread `at` of its group
// has the pairs at, at + width, ... Whole waves that are left over (32 to 43 players: one group of 576 to 960) count as one
// more group, which takes no rows.
struct ds_small_share {
  int width, groups, group, at;
};
DS_SMALL_FN ds_small_share ds_small_share_of(int pairs, int tid) {
  ds_small_share s;
  s.width = pairs < kSmallThreads ? (pairs + 63) & ~63 : kSmallThreads;
  s.groups = kSmallThreads / s.width;
  s.group = tid / s.width;
  s.at = tid - s.group * s.width;
  return s;
}
DS_SMALL_FN bool ds_small_adds(const ds_small_share& s) { return s.group < s.groups; }
// the first group adds the others' sums to its own and stores them
DS_SMALL_FN bool ds_small_stores(const ds_small_share& s) { return s.group == 0; }
