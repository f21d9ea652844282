// Launch shape of the gather-form Gibbs sampler: chains per workgroup,
// lanes per chain, chunk length, LDS ring and load counts.  Plain host C++
// (the constexpr helpers are also used by the kernels), so that a CPU
// program can check every planned shape against the kernel's index ranges.
#pragma once

#include <algorithm>
#include <cstddef>
#include <cstdint>

namespace bmdca {

constexpr int64_t gp_ceil(int64_t a, int64_t b) { return (a + b - 1) / b; }

constexpr int kGMaxWaves = 16;   // waves per workgroup at most
constexpr int kGMinWaves = 4;    // and at least
// Chains per workgroup at most for a launch on a share of the CUs (grouped
// training of 64 models over 8 lanes: caps of 32, 64 and 128 chains measured
// 909, 575 and 1163 ms per epoch).
constexpr int kGShareChains = 64;
constexpr size_t kGLds = 160 * 1024 - 256;
constexpr size_t kGAlign = 128;  // chunk boundaries on whole cache lines of the run

// Row pitch of Jt: q rounded up to a multiple of 4 floats (16-byte quads).
constexpr int gather_qp(int q) { return (q + 3) & ~3; }
// Lanes per quad group: quads per row rounded up to a power of two.
constexpr int gather_v(int q) {
  return gather_qp(q) / 4 <= 1 ? 1 : gather_qp(q) / 4 <= 2 ? 2 : gather_qp(q) / 4 <= 4 ? 4 : 8;
}
// Site groups per chain of `lpc` lanes (8 or 16; a narrow chain, one lane
// per quad of its row, has one).
constexpr int gather_s(int q, int lpc) { return lpc >= gather_v(q) ? lpc / gather_v(q) : 1; }

struct GatherShape {
  int lpc;        // lanes per chain (8 or 16)
  int waves;      // waves per workgroup
  int cpb;        // chains per workgroup
  int jc;         // sites per chunk (multiple of 4 S)
  int nchunk;     // chunks per site
  int m4;         // token dwords per (chain, site group)
  int ahead;      // chunks in flight (ring = ahead + 1 slots)
  int items;      // 1 KB loads per loading wave per chunk: 8, 16 or 31, a template
                  // parameter so that every wait is an immediate (31 keeps two
                  // younger chunks within vmcnt's range)
  int nload;      // loading waves (waves 0..nload-1; wave w loads blocks w*items ...)
  int slot;       // floats per ring slot (nload * items KB)
  size_t lds;     // dynamic LDS bytes
  unsigned blocks;
  int pair;       // gather_pair() of the shape; read by no kernel
};

// Token bytes per chain.
inline size_t gather_tok_bytes(int L, int q, int lpc) {
  const int S = gather_s(q, lpc);
  return (size_t)S * (size_t)gp_ceil(gp_ceil(L, S), 4) * 4;
}

// Shape for `cpb` chains per workgroup and a ring of `nslot` slots; waves = 0
// if it does not fit.  `align` asks for chunks on 256-byte boundaries.
inline GatherShape gather_shape_n(int L, int q, int cpb, int nslot, int lpc, bool align) {
  GatherShape g{};
  const int S = gather_s(q, lpc);
  const size_t site_row = (size_t)q * gather_qp(q) * sizeof(float);  // bytes per site of a chunk
  // at least 4 waves, one per SIMD, to spread the chunk loads and barriers
  g.lpc = lpc;
  g.waves = std::max<int>(kGMinWaves, (int)gp_ceil(cpb, 64 / lpc));
  if (g.waves < 1 || g.waves > kGMaxWaves) return GatherShape{};
  const size_t tok = gather_tok_bytes(L, q, lpc) * (size_t)(g.waves * (64 / lpc));
  if (tok >= kGLds) return GatherShape{};
  const size_t per_slot = std::min((kGLds - tok) / nslot, (size_t)31 * g.waves * 1024);
  // Chunks are a multiple of 4 S sites (4 token positions per lane, one
  // token dword) and of kGAlign bytes: a chunk that starts off a 128-byte
  // boundary of the run makes every load of it misaligned.  Aligned and not, in
  // free-running waves, ms, 3 sweeps: q = 19, L = 300, 6000 chains, 16- and
  // 20-site chunks, 7.96 and 8.45, 10 000 chains 8.63 and 8.95; q = 17, L = 100,
  // 24- and 20-site chunks, 5 sweeps, 1.77 and 1.73 (few chunk lengths are
  // affected: rows of q = 21 or 13 are aligned by the token rule alone).  A
  // 256-byte rule costs steps for nothing: at q = 21 it takes 8-site chunks
  // where 12 fit (with barriers at L = 512: 64 chunk-steps per site instead of
  // 43; 39.6 against 25.0 ms per sweep for 10 000 chains on 32 CUs).
  int step = 4 * S;
  while (align && ((size_t)step * site_row) % kGAlign != 0) step += 4 * S;
  const int lcap = (int)gp_ceil(L, 4 * S) * 4 * S;
  // the largest chunk whose padded slots and tokens fit (a chunk of the
  // whole run needs no alignment)
  for (int jc = std::min((int)(per_slot / site_row) / (4 * S) * (4 * S), lcap); jc >= 4 * S;
       jc -= 4 * S) {
    g.nchunk = (int)gp_ceil(L, jc);
    g.jc = (int)gp_ceil(gp_ceil(L, g.nchunk), 4 * S) * 4 * S;  // balanced chunks
    if (g.nchunk > 1) g.jc = (int)gp_ceil(g.jc, step) * step;
    if (g.jc > jc) continue;
    g.nchunk = (int)gp_ceil(L, g.jc);
    g.m4 = (int)gp_ceil(gp_ceil(L, S), 4);
    g.ahead = nslot - 1;
    g.cpb = cpb;
    const int nblk = (int)gp_ceil((size_t)g.jc * site_row, 1024);
    for (int it : {8, 16, 31}) {  // the least padding that the waves can load
      if ((nslot - 2) * it > 63) continue;  // vmcnt range of the younger chunks
      g.items = it;
      g.nload = (int)gp_ceil(nblk, it);
      g.slot = g.nload * it * 256;
      g.lds = (size_t)nslot * g.slot * sizeof(float) + tok;
      if (g.nload <= g.waves && g.lds <= kGLds) return g;
    }
  }
  return GatherShape{};
}

// A ring of 4 slots: three chunks in flight.  Measured with barriers at L =
// 100..512, q = 21: 3 slots (larger chunks, two in flight) take 1.4-1.8x as
// long per sweep, 5, 6 or 8 slots (smaller chunks, more steps) 1.5-2.5x (not
// measured in free-running waves).
inline GatherShape gather_shape(int L, int q, int cpb, int lpc) {
  const GatherShape g = gather_shape_n(L, q, cpb, 4, lpc, true);
  // unaligned chunks only where no aligned shape fits (q = 25 or 27 at large
  // L, or large L with many chains' tokens in the LDS)
  return g.waves ? g : gather_shape_n(L, q, cpb, 4, lpc, false);
}

// Lanes per chain (8 or 16): a function of q and the draw alone, never of
// the chain count or the CU share, because the FP32 summation order of a
// chain's local fields follows its lanes -- with this rule a chain draws the
// same bits in bmdca_gibbs, in a grouped epoch on a CU share and in a merged
// bmdca_gibbs_streams launch.  So the lanes are part of the results, and stay
// whatever a kernel would favour: 8, and 16 for Metropolis at q <= 8 (rows of
// at most two quads).  They were taken from a form with barriers: 16 lanes cost
// 1.9x at q = 21, where the per-wave step overhead doubles; at q = 5, L = 400,
// 10 000 chains the heat bath took 23.6 ms per 10 sweeps with 8 and 28.2 with
// 16, Metropolis 27.2 and 24.0.
constexpr int gather_lanes(int q, bool small) { return (gather_v(q) <= 2 && !small) ? 16 : 8; }

// Narrow heat-bath chains: rows of 5, 6 or 7 quads (q = 17..28) can also run
// with one lane per quad, 12, 10 or 9 chains per wave instead of 8, so no
// lane of the row gathers idles (q = 21: 6 of 8 lanes would).  Each lane adds
// its quad over the positions in the same order as in an 8-lane chain, and
// the draw's cross-lane steps keep the 8-lane association order, so a narrow
// chain draws the same bits as an 8-lane one (checked over whole runs): the
// choice may follow the launch shape.  The planner takes it where it saves
// waves and still leaves at least kGNarrowWaves, two per SIMD.  Free-running
// waves, 8 lanes -> narrow, ms, 3 sweeps of q = 21, with 8 narrow waves or more:
// 18 000 chains (9 waves -> 8) L = 60 0.62 -> 0.61, L = 100 1.54 -> 1.47, L =
// 256 9.26 -> 7.93, L = 512 42.7 -> 34.6; 30 000 (15 -> 12) 0.80 -> 0.77, 2.11
// -> 1.93, 13.0 -> 11.1, 58.2 -> 47.0; 24 000 (12 -> 10), the weakest, 0.65 ->
// 0.71, 1.66 -> 1.77, 10.0 -> 10.1, 45.4 -> 43.5; q = 17, L = 100 15-18%
// faster, q = 25, L = 256 even to 17% faster.  With fewer: 16 384 (8 -> 7)
// 0.48 -> 0.59, 1.26 -> 1.44, 7.30 -> 7.85, 33.6 -> 34.2, 12 000 (6 -> 5) 0.47
// -> 0.53, 1.18 -> 1.31, 6.60 -> 6.76, 27.1 -> 27.0, 10 000 (5 -> 4) 0.47 ->
// 0.50, 1.16 -> 1.18, 6.39 -> 6.08, 27.1 -> 27.0: a wave that is there to hide
// another's draw is worth more than the idle lanes.
constexpr int kGNarrowWaves = 8;
constexpr int gather_narrow_lanes(int q, bool small) {
  return (small && gather_v(q) == 8 && gather_qp(q) / 4 < 8) ? gather_qp(q) / 4 : 0;
}

// Whether a plan's chunk-steps would be worth pairing in the form with barriers:
// the ring of 4 slots refilled two chunks at a time, one wait and one barrier per
// two steps, two chunks in flight instead of three.  No kernel reads it: the form
// with barriers runs plans of many waves, pairs always, and free-running waves
// have no steps to pair.  A launch on a share of the CUs pairs as well; it runs
// Metropolis of q <= 8 in plans of 16 waves, ms unpaired -> paired: 32 CUs, q = 5,
// 2048 chains L = 100 2.95 -> 2.76, L = 400 38.9 -> 37.7, q = 4, L = 200, 1024
// chains on 16 CUs 11.6 -> 11.2; epochs of 32 models at q = 5 55.2 -> 52.5, q = 8
// 66.3 -> 64.3, q = 4 98.8 -> 91.3, of 64 models 113.5 -> 108.4.
constexpr int kGPairChains = 32;
constexpr double kGPairCacheBytes = 256.0 * 1024 * 1024;
inline int gather_pair(int L, int q, int cpb) {
  const double jt = (double)L * L * q * gather_qp(q) * sizeof(float);
  return (cpb >= kGPairChains && (jt <= kGPairCacheBytes || cpb >= 2 * kGPairChains)) ? 1 : 0;
}

// Chains per workgroup for chains of `lpc` lanes: spread the chains over the
// CUs (one workgroup per CU at a time) in as few rounds as the largest
// workgroup that fits allows.
inline GatherShape gather_plan_lanes(int64_t N, int L, int q, int64_t cus, int cap, int lpc) {
  const int cpw = 64 / lpc;  // chains per wave
  int cmax = std::min(cap, kGMaxWaves * cpw);
  while (cmax > cpw && gather_shape(L, q, cmax, lpc).waves == 0) cmax -= cpw;
  const int64_t rounds = gp_ceil(N, cus * cmax);
  const int cpb = (int)std::min<int64_t>(cmax, gp_ceil(N, rounds * cus));
  GatherShape g = gather_shape(L, q, cpb, lpc);
  g.blocks = (unsigned)gp_ceil(N, (int64_t)cpb);
  g.pair = g.waves > 0 ? gather_pair(L, q, g.cpb) : 0;
  return g;
}

inline GatherShape gather_plan(int64_t N, int L, int q, int64_t cus, int cap = kGMaxWaves * 8,
                               bool small = true) {
  GatherShape g = gather_plan_lanes(N, L, q, cus, cap, gather_lanes(q, small));
  const int nl = gather_narrow_lanes(q, small);
  if (nl > 0 && g.waves > kGNarrowWaves) {
    const GatherShape n = gather_plan_lanes(N, L, q, cus, cap, nl);
    if (n.waves >= kGNarrowWaves && n.waves < g.waves && n.blocks <= g.blocks) g = n;
  }
  return g;
}

// Free-running waves wherever a wave is left to load: plans of 16 waves (more
// than 120 chains per workgroup in 8 lanes, 60 in 16) keep the barriers, which
// need no wave of their own.  Barriers -> free at either end of the range, ms:
// q = 12, L = 50, 6000 chains, 5 sweeps, 0.43 -> 0.33; q = 5, L = 400, 20 000
// chains, 3 sweeps, 6.88 -> 6.58; 15 waves, one more loading: q = 16, L = 100,
// 30 000 chains, 3 sweeps, 1.74 -> 1.37, q = 9, L = 60, 5 sweeps 0.89 -> 0.89,
// Metropolis q = 21, L = 100, 10 sweeps 5.02 -> 4.38.
// The barriers also keep heat-bath plans of many waves and 3 to 12 states whose
// sites are one chunk each of other than whole groups of 16 positions a lane (the
// free form reads their tokens by single dwords): from 9 waves on of q <= 4 and 20
// positions, 12 of q <= 8, else 13.  Barriers and free there, ms, 3 sweeps: q = 4,
// L = 200, 13 waves 1.34 and 1.54, 9 waves 1.10 and 1.18, L = 80, 14 waves 0.37 and
// 0.40, q = 8, L = 70, 12 waves 0.40 and 0.43; with fewer waves, fewer positions or
// whole groups the free form is even or faster (q = 4, L = 200, 8 waves 1.05 and
// 0.95, L = 120, 13 waves 0.61 and 0.62, 12 waves 0.55 and 0.52).  Over 3250 shapes
// of 7 to 15 waves a call takes at most 6% longer than by barriers, 0.90 of their
// time in the mean.
constexpr int kGLoaders = 2;
inline bool gather_free(const GatherShape& gs, int q, bool mh) {
  const int positions = gs.jc / gather_s(q, gs.lpc);
  if (!mh && q >= 3 && q <= 12 && gs.nchunk == 1 && positions >= 12 && positions % 16 != 0 &&
      gs.waves >= (q <= 4 && positions >= 20 ? 9 : q <= 8 ? 12 : 13))
    return false;
  return gs.waves < kGMaxWaves;
}

// Waves, token layout and LDS of the free-running form of a plan.
struct FreeShape {
  int nw;      // waves that hold chains; the others load
  int waves;   // waves per workgroup
  bool tq;     // tokens of 16 positions side by side
  int m4;      // token dwords per (chain, site group)
  size_t lds;  // dynamic LDS bytes
};

// Tokens of a heat-bath chain: in chunks of whole groups of 16 positions a
// lane's 16 tokens side by side, one 16-byte read; else all of a site group's
// side by side, an odd number of dwords apart from the next chain's.  Against
// dwords interleaved over the chains (four reads, each address clamped), as
// Metropolis has them: q = 5, L = 400, 10 000 chains, 5 sweeps 7.12 -> 6.74
// ms, q = 12, L = 200 3.65 -> 3.49, q = 25, L = 150, 3 sweeps 3.77 -> 3.46;
// Metropolis q = 21, L = 256 would take 3.9 ms for 3.6.  Interleaved dwords of a
// chain of 16 lanes (16 or 8 site groups) are an odd number of rows of chains
// apart too: with 4 or 8 the lanes of a chain read few banks (q = 2, L = 512, 1000
// chains, one sweep 2.01 ms, 1.74 with the next rule, 1.54 with both).
//
// Waves: a plan has at least four, for the loads, but here a chains' wave without
// chains only polls and reads LDS beside those that have some.  Chains of 16 lanes
// take what holds them, and three for two waves' chains (even or up to 5% faster
// than two): q = 8, L = 250, one sweep, 358 chains 680 -> 519 us, 2048 643 -> 581.
// (In 8 lanes 0.86 to 1.05 of the time, and heat-bath sweeps of few chains have a
// form of their own.)
// The loading waves come beside the plan's; the counters (chunks consumed by
// each wave, chunks complete) lie behind the tokens, kGLds leaves 256 bytes for
// them.
inline FreeShape free_shape(const GatherShape& gs, int q, bool mh) {
  FreeShape f{};
  const int S = gather_s(q, gs.lpc), m4q = (int)gp_ceil(gs.m4, 4) * 4;
  const size_t col = (size_t)S * 4 * (gs.waves * (64 / gs.lpc));  // bytes of a token dword of all
  const int need = (int)gp_ceil(gs.cpb, 64 / gs.lpc);
  f.nw = gs.lpc != 16 ? gs.waves : need == 2 ? 3 : need;
  f.waves = std::min(f.nw + kGLoaders, kGMaxWaves);
  f.tq = !mh && gs.jc / S % 16 == 0 && gs.lds + (m4q - gs.m4) * col <= kGLds;
  const bool odd = (!mh || gs.lpc == 16) && gs.m4 % 2 == 0 && gs.lds + col <= kGLds;
  f.m4 = f.tq ? m4q : gs.m4 + (odd ? 1 : 0);
  f.lds = gs.lds + (f.m4 - gs.m4) * col + 4 * (kGMaxWaves + 1);
  return f;
}

// ---------------------------------------------------------------------------
// A workgroup per chain (sampler_few.hip).
// ---------------------------------------------------------------------------
constexpr int64_t kGFewPerCu = 16;  // workgroups per CU counted on at most

struct FewShape {
  int waves;      // 2 or 3
  int rowf;       // floats of a row buffer
  size_t lds;     // dynamic LDS bytes
  int64_t fits;   // workgroups per CU (0: the LDS does not hold one)
};

inline FewShape few_shape(int L, int q, int waves) {
  const int qp = gather_qp(q), nq = qp / 4, S = gather_s(q, 8);
  const int nit = (int)gp_ceil(L * nq, 64), nb = (int)gp_ceil(q * nq, 64);
  const int lr = (int)gp_ceil(L, S) + 9;  // positions read, past the last one too
  FewShape f{};
  f.waves = waves;
  f.rowf = std::max(nit * 256, lr * S * qp);
  const size_t wavef = (size_t)f.rowf + (waves - 1) * nb * 256 + 96;
  f.lds = sizeof(float) * (waves * wavef + nit * 64 + 4) + (size_t)gp_ceil(L, 16) * 16;
  f.fits = std::min<int64_t>(kGFewPerCu, (int64_t)(kGLds / f.lds));
  return f;
}

// Three waves for one or two chains per CU (L = 100, q = 21, 128 chains: 0.85
// us a visit, 0.94 with two waves; 1024 chains 1.71 and 1.22), and where a CU
// takes so few workgroups of two that the chains come in several rounds (L =
// 400, 1024 chains: 7.8 and 9.0).
inline FewShape few_plan(int64_t N, int L, int q, int64_t cus) {
  const FewShape f3 = few_shape(L, q, 3), f2 = few_shape(L, q, 2);
  if (N <= cus * std::min<int64_t>(2, f3.fits)) return f3;
  return (f3.fits > 0 && f2.fits <= 3 && N > cus * f2.fits) ? f3 : f2;
}

// Chains per CU up to which a workgroup per chain is the faster form.  The
// gather form's visit costs at least its staging, L q QP floats, whatever the
// number of chains (up to 24 per CU); here it costs the chains' rows.  Measured,
// us per visit, here and there: q = 21, L = 120: 2.2 and 3.9 with 1280 chains,
// 3.6 and 3.9 with 2816, 4.5 and 3.9 with 3328; L = 300 (one workgroup per CU)
// 7.3 and 8.9 with 1280, 10.2 and 8.9 with 1792; q = 12, L = 120: 1.8 and 2.4
// with 2304, L = 300: 4.5 and 4.9 with 1792, 6.2 and 5.0 with 2304; q = 5, L =
// 120: 0.9 and 1.2 with 1280, L = 300: 2.1 and 2.4 with 1280, 2.7 and 2.4 with
// 1536; q = 32, L = 120: 5.5 and 6.1 with 3072, 8.1 and 6.2 with 4608.
// Of q <= 4 the staging is cheap (16 bytes a site and state) and the chains' rows
// grow with L, so the line falls with it, from 5 chains per CU at 200 sites to 3
// at 512; us a sweep here and there, q = 2: L = 200 200 and 220 with 1280, L = 230
// 232 and 253 with 1030, 286 and 253 with 1280, L = 300 384 and 399 with 1024, 458
// and 398 with 1030, L = 400 595 and 638 with 770, 693 and 640 with 1024, L = 512
// 829 and 877 with 768, 1003 and 877 with 900.
inline bool gather_few(int64_t N, int L, int q, int64_t cus) {
  const FewShape f = few_plan(N, L, q, cus);
  if (f.fits == 0) return false;
  if (q <= 4 && 5 * N * L > cus * (8 * L + 3600)) return false;
  const int64_t most = q <= 8 ? 5 : q <= 16 ? 8 : q <= 24 ? 11 : 13;
  return N <= cus * (f.fits > 1 ? most : most / 2 + 1);
}

}  // namespace bmdca
