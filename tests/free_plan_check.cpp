// CPU check of the launch shapes of the gather sampler's other two forms, for
// every planned shape that takes them:
//   - free-running waves: the LDS holds ring, tokens and counters; the 1 KB
//     loads of a chunk stay in its slot; every (chain, site) has a token byte of
//     its own; the dwords a lane reads for its positions are those bytes, and
//     what it reads past them lies in the token or counter area;
//   - a workgroup per chain: loads, row, block, table and token indices stay in
//     the buffers the launch allocates.
// Exit status 0 when all hold.
#include <cstdio>
#include <vector>

#include "../paper_2501_18456_amd/csrc/gather_plan.hpp"

using namespace bmdca;

static int failures = 0;
#define CHECK(cond, ...)                                                                  \
  do {                                                                                    \
    if (!(cond)) {                                                                        \
      if (failures++ < 20) {                                                              \
        std::printf("FAIL %s: N=%lld L=%d q=%d: ", #cond, (long long)N, L, q);            \
        std::printf(__VA_ARGS__);                                                         \
        std::printf("\n");                                                                \
      }                                                                                   \
      return;                                                                             \
    }                                                                                     \
  } while (0)

static constexpr size_t kLdsCu = 160 * 1024;

static void check_free(int64_t N, int L, int q, const GatherShape& g, bool mh) {
  const FreeShape f = free_shape(g, q, mh);
  const int S = gather_s(q, g.lpc), QP = gather_qp(q), CPW = 64 / g.lpc;
  const int CPB = f.nw * CPW, loaders = f.waves - f.nw;
  CHECK(f.nw >= 1 && CPB >= g.cpb, "nw %d cpb %d", f.nw, g.cpb);
  CHECK(f.waves <= kGMaxWaves && loaders >= 1 && loaders <= kGLoaders, "waves %d nw %d", f.waves,
        f.nw);
  const size_t ring = (size_t)4 * g.slot * 4, tok = (size_t)4 * S * f.m4 * CPB;
  const size_t counters = 4 * (kGMaxWaves + 1);
  CHECK(f.lds <= kLdsCu && ring + tok + counters <= f.lds, "ring %zu tokens %zu lds %zu", ring, tok,
        f.lds);
  const size_t chunk = (size_t)g.jc * q * QP * 4;
  CHECK((chunk + 1023) / 1024 * 1024 <= (size_t)g.slot * 4, "chunk %zu slot %d", chunk, g.slot);
  CHECK(g.jc % (4 * S) == 0 && g.nchunk * g.jc >= L, "jc %d", g.jc);
  CHECK(!f.tq || (f.m4 % 4 == 0 && g.jc / S % 16 == 0), "tq m4 %d jc %d", f.m4, g.jc);

  // the kernel's byte of site j of chain cb, and the one its layout writes
  auto off = [&](int j, int cb) -> size_t {
    const int m = j / S;
    if (f.tq) return (size_t)(((j % S) * (f.m4 / 4) + (m >> 4)) * CPB + cb) * 16 + (m & 15);
    if (mh) return (size_t)(((j % S) * f.m4 + (m >> 2)) * CPB + cb) * 4 + (m & 3);
    return (size_t)((j % S) * CPB + cb) * f.m4 * 4 + m;
  };
  auto put = [&](int uu, int mq, int cb) -> size_t {  // dword of positions 4 mq .. of group uu
    if (f.tq) return (size_t)((uu * (f.m4 / 4) + (mq >> 2)) * CPB + cb) * 4 + (mq & 3);
    if (mh) return (size_t)(uu * f.m4 + mq) * CPB + cb;
    return (size_t)(uu * CPB + cb) * f.m4 + mq;
  };
  static std::vector<int> owner;  // 1 + the site and chain of a byte, in this shape
  owner.assign(tok, 0);
  for (int cb : {0, 1, CPB / 2, CPB - 1}) {
    if (cb >= CPB || (cb == 1 && CPB / 2 == 1) || (cb == CPB / 2 && cb == 0)) continue;
    if (cb == CPB / 2 && (cb == CPB - 1 || cb == 0)) continue;
    for (int j = 0; j < L; ++j) {
      const size_t o = off(j, cb);
      CHECK(o < tok, "token %zu of %zu (site %d chain %d)", o, tok, j, cb);
      const int id = 1 + j * CPB + cb;
      CHECK(owner[o] == 0 || owner[o] == id, "sites share a byte (site %d chain %d)", j, cb);
      owner[o] = id;
      const int m = j / S;
      CHECK(o / 4 == put(j % S, m >> 2, cb) && o % 4 == (size_t)(m & 3), "site %d chain %d", j, cb);
    }
    for (int k = 0; k < S * f.m4; ++k)
      CHECK(put(k / f.m4, k % f.m4, cb) < tok / 4, "written dword %d of chain %d", k, cb);
  }
  // row reads: the last position's last row, its last quad
  const int jcs = g.jc / S;
  const int64_t last = ((int64_t)(S * (jcs - 1) + S - 1) * q + (q - 1)) * QP + QP - 1;
  CHECK(last < g.slot, "row read %lld slot %d", (long long)last, g.slot);
  if (mh) return;
  // heat-bath token reads: 16 positions at a time, the first of the next chunk ahead
  const int jcl = std::min(jcs, (((L - (g.nchunk - 1) * g.jc + S - 1) / S) + 3) & ~3);
  for (int k = 0; k < g.nchunk; ++k) {
    const int nv = k + 1 < g.nchunk ? jcs : jcl;
    CHECK(nv % 4 == 0 && nv >= 4, "positions %d", nv);
    for (int r = 0; r < nv; r += 16)
      for (int u : {0, S - 1})
        for (int cb : {0, CPB - 1}) {
          const int d0 = (k * jcs + r) >> 2;
          const size_t first = f.tq ? (size_t)16 * (u * (f.m4 / 4) * CPB + cb) + (size_t)d0 * CPB * 4
                                    : (size_t)4 * ((u * CPB + cb) * f.m4 + d0);
          CHECK(!f.tq || (d0 % 4 == 0 && first % 16 == 0), "aligned reads, d0 %d", d0);
          CHECK(first + 16 <= tok + (f.tq ? 0 : counters), "read %zu of %zu", first, tok);
          for (int e = 0; e < std::min(16, nv - r); ++e) {
            const int j = S * (k * jcs + r + e) + u;
            if (j < L) CHECK(first + e == off(j, cb), "position %d of site %d", e, j);
            CHECK(first + e < tok, "position %d read at %zu", e, first + e);
          }
        }
  }
}

static void check_few(int64_t N, int L, int q, const FewShape& f) {
  const int QP = gather_qp(q), NQ = QP / 4, S = gather_s(q, 8), D = f.waves - 1;
  const int nit = (L * NQ + 63) / 64, nb = (q * NQ + 63) / 64;
  CHECK(f.waves == 2 || f.waves == 3, "waves %d", f.waves);
  CHECK(f.fits >= 1 && f.lds <= kLdsCu, "lds %zu", f.lds);
  const size_t wavef = (size_t)f.rowf + D * nb * 256 + 64 + 32;
  CHECK(4 * (f.waves * wavef + (size_t)nit * 64 + 4) + L <= f.lds, "lds %zu", f.lds);
  CHECK(nit * 256 <= f.rowf, "row loads %d of %d", nit * 256, f.rowf);
  CHECK(L * NQ <= nit * 64 && (q - 1) * QP + QP - 1 < nb * 256 && QP <= 32, "table, blocks");
  // positions a lane reads of a site group, as the kernel walks them
  const int Lr = (L + S - 1) / S;
  int most = 0;
  auto ld = [&](int r) { most = std::max(most, r + 7); };
  auto two = [&](int r, bool more) {
    ld(r + 8);
    if (more) ld(r + 16);
  };
  auto seg = [&](int r0, int r1) {
    int r = r0;
    if (r + 8 <= r1) {
      ld(r);
      for (; r + 24 <= r1; r += 16) two(r, true);
      if (r + 16 <= r1) {
        two(r, false);
        r += 16;
      } else {
        r += 8;
      }
    }
    if (r < r1) ld(r);
  };
  for (int q1 = 0; q1 < Lr; ++q1) {
    seg(0, q1);
    for (int q2 : {0, q1 / 2, q1 > 0 ? q1 - 1 : 0}) {
      seg(0, q2);
      seg(q2, q1);
    }
    most = std::max(most, q1);
    ld(q1 + 1);
    int r = q1 + 1;
    for (; r + 16 < Lr; r += 16) two(r, true);
    if (r + 8 < Lr) two(r, false);
  }
  CHECK((most + 1) * S * QP <= f.rowf, "position %d of %d floats", most, f.rowf);
}

int main() {
  std::vector<int> Ls;
  for (int L = 1; L <= 40; ++L) Ls.push_back(L);
  for (int L : {50, 64, 80, 99, 100, 101, 127, 128, 150, 200, 250, 257, 300, 323, 385, 400, 511, 512})
    Ls.push_back(L);
  int shapes = 0;
  for (int q = 2; q <= 32; ++q)
    for (int L : Ls)
      for (int64_t n : {1, 7, 100, 1000, 1500, 4096, 10000, 20000, 26000, 30000, 40000, 100000})
        for (int64_t c : {256, 32}) {
          const FewShape few = few_plan(n, L, q, c);
          if (gather_few(n, L, q, c)) check_few(n, L, q, few), ++shapes;
          for (int cap : {128, kGShareChains})
            for (bool mh : {false, true}) {
              const GatherShape g = gather_plan(n, L, q, c, cap, !mh);
              if (!gather_free(g, q, mh)) continue;
              check_free(n, L, q, g, mh);
              ++shapes;
            }
        }
  std::printf("%d shapes checked, %d failures\n", shapes, failures);
  return failures == 0 ? 0 : 1;
}
