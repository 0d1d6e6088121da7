// Host side of the sampling plan: how many mask rows, which coalition sizes, and
// the regression weight of each size class.
//
// Follows the paper's sample-distribution equation (rho_s = (n-1)/(s(n-s)),
// k_s proportional to rho_s) and its complementary pairing. A pair class s
// (1 <= s <= floor(n/2)) holds the sizes (s, n-s); its mass is 2*rho_s, or rho_s
// when 2s == n. The K sampled pairs are split by cumulative rounding so that the
// classes sum to K exactly and pairs are laid out by ascending size. A row of
// size s weighs rho_s / (number of emitted rows of size s), so each represented
// size carries its whole kernel mass; under enumeration this is the Shapley
// kernel weight itself. (Option: every sampled row weighs 1 instead, the
// importance-sampling form, since the allocation already follows rho_s.)
//
// Every operation that decides an integer is a single IEEE double + * / or floor
// (no fused multiply-add: build with -ffp-contract=off), so the boundaries are
// reproducible bit for bit.
#include <cmath>

#include "internal.h"

static double rho_mass(int64_t n, int64_t s) {
  return (double)(n - 1) / ((double)s * (double)(n - s));
}

extern "C" int ds_sample_plan(int64_t n, int64_t n_samples, int64_t* k_out, int32_t* enumerated_out) {
  if (n < 0 || n_samples < 0) return DS_EINVAL;
  int enumerate = (n <= DS_ENUM_MAX_PLAYERS && n_samples >= ((int64_t)1 << n)) ? 1 : 0;
  int64_t k = enumerate ? ((int64_t)1 << n) : 2 * (n_samples / 2);
  if (k_out) *k_out = k;
  if (enumerated_out) *enumerated_out = enumerate;
  return DS_OK;
}

ds_plan::~ds_plan() {
  if (!owner) return;
  ds_plan_memory& kept = owner->plan_memory;
  if (b.capacity() > kept.b.capacity()) b.swap(kept.b);
  if (wtab.capacity() > kept.wtab.capacity()) wtab.swap(kept.wtab);
}

// What bounds the plan of a large game: divisions, one addition after another, and the page faults of three fresh tables of n / 2
// entries. The tables' memory stays with the context; the masses are divided block by block in front of their sum, two at a
// time, so that one block's additions run beside the next one's divisions (blocks of 8, 16, 32, 64: 304, 279, 175, 280 us of 200,006
// classes; on another machine, with fresh tables, 32.3, 32.3, 29.8, 30.7 of 5,000 and 6.5, 6.6, 6.2, 6.6 ms of 500,087). The plan of 400,013 players, which the sampler waits for: about 0.5 ms, now 0.3.
constexpr int32_t kBlock = 32;

int ds_make_plan(ds_ctx* ctx, int64_t n, int64_t n_samples, ds_plan* plan, int weighting, int saturate) {
  if (n < 2) return ds_fail(ctx, DS_EINVAL, "sampling needs at least 2 players (n=%lld)", (long long)n);
  if (n > 0x7fffffffLL) return ds_fail(ctx, DS_EINVAL, "too many players (n=%lld)", (long long)n);
  int32_t enumerate;
  int64_t k;
  ds_sample_plan(n, n_samples, &k, &enumerate);
  if (!enumerate && n_samples < 4)
    return ds_fail(ctx, DS_EINVAL, "n_samples must be at least 4 (got %lld)", (long long)n_samples);
  plan->n = n;
  plan->k = k;
  plan->K = k / 2 - 1;
  plan->H = n / 2;
  plan->enumerate = enumerate;
  const int64_t H = plan->H, K = plan->K;
  std::vector<double> own;
  const bool keep = ctx && H < kPlanKept;
  if (keep && !plan->owner) {
    plan->owner = ctx;
    plan->b.swap(ctx->plan_memory.b);
    plan->wtab.swap(ctx->plan_memory.wtab);
  }
  plan->wtab.resize(H + 1);
  plan->b.resize(H + 1);
  plan->enum_upto = 0;
  if (saturate && weighting != DS_WEIGHT_CLASS_MASS)
    return ds_fail(ctx, DS_EINVAL, "saturated size classes need the class-mass weighting");
  if (enumerate) {
    plan->b.assign(H + 1, 0);
    plan->wtab[0] = 0.0f;
    double binom = 1.0;  // C(n, s), exact in double for n <= 24
    for (int64_t s = 1; s <= H; ++s) {
      binom = binom * (double)(n - s + 1) / (double)s;
      plan->wtab[s] = (float)(rho_mass(n, s) / binom);
    }
    return DS_OK;
  }
  // Option `saturate`: a class that is allotted at least as many pairs as it has coalitions (q_s >= C(n, s)) is
  // enumerated (every s-subset once) and the pairs this frees go to the classes that are left, by the same
  // cumulative rounding; the test moves on to the next class (C(n, s) grows and the allotment shrinks with s, so
  // the enumerated classes are 1..enum_upto). The class 2s == n is never enumerated this way.
  std::vector<double>& masses = keep ? ctx->plan_memory.c : own;
  if (masses.size() < (size_t)(H + 1)) masses.resize(H + 1);
  double* const c = masses.data();
  int64_t* const b = plan->b.data();
  b[0] = 0;
  int64_t enum_upto = 0, used = 0, cap_prev = 1;  // cap_prev = C(n, enum_upto)
  for (;;) {
    const double top = (double)(n - 1);
    const int32_t n32 = (int32_t)n, last = (int32_t)H - (2 * H == n ? 1 : 0);   // (the class of n / 2 alone counts once)
    double acc = 0.0;
    int32_t s0 = (int32_t)enum_upto + 1;
    for (; s0 + kBlock - 1 <= last; s0 += kBlock) {
      double mass[kBlock];
      for (int32_t i = 0; i < kBlock; ++i) mass[i] = 2.0 * (top / ((double)(s0 + i) * (double)(n32 - s0 - i)));
      for (int32_t i = 0; i < kBlock; ++i) {
        acc = acc + mass[i];
        c[s0 + i] = acc;
      }
    }
    for (int64_t s = s0; s <= H; ++s) {
      const double r = rho_mass(n, s);
      acc = acc + ((2 * s == n) ? r : 2.0 * r);
      c[s] = acc;
    }
    const double T = acc, pairs = (double)(K - used);
    // rounded down (nothing is negative), by the conversion: floor() is a call here
    if (K < 0x7fffffff)
      for (int64_t s = enum_upto + 1; s < H; ++s) b[s] = used + (int64_t)(int32_t)(pairs * (c[s] / T) + 0.5);
    else
      for (int64_t s = enum_upto + 1; s < H; ++s) b[s] = used + (int64_t)(pairs * (c[s] / T) + 0.5);
    b[H] = K;
    const int64_t s1 = enum_upto + 1;
    if (!saturate || s1 > H || 2 * s1 >= n) break;
    const __int128 cap = (__int128)cap_prev * (__int128)(n - s1 + 1) / (__int128)s1;  // C(n, s1), exact
    if (cap > (__int128)(plan->b[s1] - used)) break;
    enum_upto = s1;
    used += (int64_t)cap;
    cap_prev = (int64_t)cap;
    plan->b[s1] = used;
  }
  plan->enum_upto = enum_upto;
  float* const wtab = plan->wtab.data();
  wtab[0] = 0.0f;
  int64_t before = 0;
  for (int64_t s = 1; s <= H; ++s) {
    int64_t m = b[s] - before;
    before = b[s];
    if (m <= 0) {   // (most classes of a large game)
      wtab[s] = 0.0f;
      continue;
    }
    if (2 * s == n) m *= 2;
    wtab[s] = weighting == DS_WEIGHT_UNIFORM ? 1.0f : (float)(rho_mass(n, s) / (double)m);
  }
  return DS_OK;
}

extern "C" int ds_plan_tables(int64_t n, int64_t n_samples, int64_t* b, float* wtab) {
  return ds_plan_tables_ex(n, n_samples, nullptr, b, wtab, nullptr);
}

extern "C" int ds_plan_tables_ex(int64_t n, int64_t n_samples, const ds_options* opts, int64_t* b, float* wtab,
                                 int64_t* enum_upto) {
  if (n < 2 || n > 0x7fffffffLL || n_samples < 0) return DS_EINVAL;
  ds_plan plan;
  int rc = ds_make_plan(nullptr, n, n_samples, &plan, opts ? opts->weighting : DS_WEIGHT_CLASS_MASS, opts ? opts->saturate : 0);
  if (enum_upto) *enum_upto = plan.enum_upto;
  if (rc != DS_OK) return rc;
  for (int64_t s = 0; s <= plan.H; ++s) {
    if (b) b[s] = plan.b[s];
    if (wtab) wtab[s] = plan.wtab[s];
  }
  return DS_OK;
}
