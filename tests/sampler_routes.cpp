// CPU check of the sampler's dispatch at shapes where both sides of a line were
// measured: the form that a call takes, and the waves it runs.
#include <cstdio>

#include "../paper_2501_18456_amd/csrc/gather_plan.hpp"

using namespace bmdca;

static int failures = 0;
#define CHECK(cond)                               \
  do {                                            \
    if (!(cond)) {                                \
      std::printf("FAIL line %d: %s\n", __LINE__, #cond); \
      ++failures;                                 \
    }                                             \
  } while (0)

int main() {
  // heat-bath, few chains on 256 CUs: a workgroup per chain or the staged form
  auto few = [](int64_t N, int L, int q) { return gather_few(N, L, q, 256); };
  for (int q : {2, 3, 4}) {
    CHECK(few(1280, 200, q) && !few(1281, 200, q));
    CHECK(few(1030, 230, q) && !few(1280, 230, q));
    CHECK(few(1024, 300, q) && !few(1030, 300, q));
    CHECK(few(770, 400, q) && !few(1024, 400, q));
    CHECK(few(768, 512, q) && !few(900, 512, q) && !few(1280, 512, q));
  }
  CHECK(few(1280, 512, 5) && few(1280, 300, 8) && !few(1281, 300, 8));
  CHECK(few(2816, 120, 21) && !few(2817, 120, 21));
  // Metropolis by free-running waves: the waves that hold chains, and token rows
  // of chains of 16 lanes an odd number apart
  auto mh = [](int64_t N, int L, int q) {
    const GatherShape g = gather_plan(N, L, q, 256, 128, false);
    return gather_free(g, q, true) ? free_shape(g, q, true) : FreeShape{};
  };
  CHECK(mh(358, 512, 4).nw == 1 && mh(1024, 250, 8).nw == 1 && mh(2048, 250, 8).nw == 3);
  CHECK(mh(2500, 250, 8).nw == 3 && mh(4096, 250, 8).nw == 4);
  CHECK(mh(9000, 511, 3).nw == 9 && mh(9000, 511, 3).m4 % 2 == 1);
  for (int L : {250, 323, 512}) CHECK(mh(358, L, 2).m4 % 2 == 1 && mh(358, L, 8).m4 % 2 == 1);
  // heat-bath, many waves: barriers or free-running waves
  auto free = [](int waves, int L, int q) {
    const GatherShape g = gather_plan(256 * 8 * waves, L, q, 256);
    CHECK(g.waves == waves);
    return gather_free(g, q, false);
  };
  CHECK(!free(9, 200, 4) && !free(13, 150, 3) && free(8, 200, 4) && free(9, 80, 4));
  CHECK(!free(14, 80, 4) && free(13, 120, 4) && free(13, 60, 4) && free(13, 200, 2));
  CHECK(!free(12, 70, 8) && free(11, 70, 8) && !free(13, 100, 5) && free(13, 250, 5));
  CHECK(!free(13, 50, 9) && free(12, 50, 9) && free(13, 80, 9) && free(13, 50, 16));
  std::printf("%d failures\n", failures);
  return failures == 0 ? 0 : 1;
}
