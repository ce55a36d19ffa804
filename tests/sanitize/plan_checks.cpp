// Checks of the workspace plan: regions that share memory, over sizes at the
// edges of every rounding.  Includes the host file for its internal plan.
#include "arckv_host.cpp"

#include <stdio.h>

using namespace arckv;

static int failures = 0;
#define CHECK_THAT(cond, ...)                         \
  do {                                                \
    if (!(cond)) {                                    \
      printf("FAIL line %d: %s: ", __LINE__, #cond);  \
      printf(__VA_ARGS__);                            \
      printf("\n");                                   \
      ++failures;                                     \
    }                                                 \
  } while (0)

static void check(int B, int T, int n, int t, int dtype, int64_t P) {
  const arckv_problem p = {B, T, n, 128, dtype, 0.0f};
  const Dims d = make_dims(&p, t);
  const Plan pl = make_plan(d, P);
#define AT "B %d T %d n %d t %d dtype %d P %lld", B, T, n, t, dtype, (long long)P
  // the parts of h: after h, before what follows the solve's vectors
  CHECK_THAT(pl.hpart >= pl.h + P * d.tp * 8, AT);
  CHECK_THAT(pl.hpart + P * (kPhicRanges - 1) * d.tp * 8 <= pl.rprev, AT);
  // the lists of the later passes end where E^T ends
  const int64_t ppk = pool_per_key(d), dcap = pass_d_capacity(d.Tp, ppk);
  CHECK_THAT(ppk >= 8, AT);
  CHECK_THAT(pl.psim >= pl.Et && pl.ditem + P * (dcap + 2) * 4 <= pl.U, AT);
  CHECK_THAT(pl.pool >= pl.psim + P * 2 * query_ranges(d.n, d.T) * ppk * d.Tp * 8, AT);
  CHECK_THAT(pl.dkey >= pl.pool + P * ppk * d.Tp * 4, AT);
  CHECK_THAT(ppk * d.Tp <= INT32_MAX, AT);   // pool offsets are int32
  // the parts of the anchors' norms in the first partials' place
  CHECK_THAT(d.MT * d.Tp / d.tp >= 1 && pl.part1 + P * d.MT * d.Tp * 8 <= pl.part2, AT);
  // the solves' scratch in the residual's X^T
  CHECK_THAT(pl.XT + P * d.tp * kHeadDimH * 4 <= pl.Pm, AT);
}

int main() {
  // the pool's counter adds up to T t candidates
  static_assert(sizeof(*AssignLists{}.pcnt) == 8, "a pool counter of 64 bits");
  for (int dtype : {ARCKV_F32, ARCKV_BF16})
    for (int B : {1, 3, 256})
      for (int T : {1, 255, 256, 257, 15001, 16383, 16384, 131072})
        for (int n : {1, 128, 129, 256, 257, 1920, 1921, 4096, 8192})
          for (int t : {1, 256, 257, 1639, 26214})
            if (t <= T)
              for (int64_t P : {(int64_t)1, (int64_t)(B + 1) / 2, (int64_t)B}) check(B, T, n, t, dtype, P);
  printf("%s: %d failures\n", failures ? "FAILED" : "ok", failures);
  return failures ? 1 : 0;
}
