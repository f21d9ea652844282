// Downstream scores of a trained model (adabmDCA 2.0, Sec. 4):
//   - energies of a batch of sequences, Eq. (1) (Sec. 4.3);
//   - single-mutant energy differences from the wild type's local fields
//     (Sec. 4.4);
//   - zero-sum-gauge Frobenius norms with the average-product correction,
//     Eq. (13) (Sec. 4.2).
#include "common.hpp"
#include "internal.hpp"

namespace bmdca {

// ---------------------------------------------------------------------------
// Energy of a batch, Eq. (1), tiled over sequences and coupling tiles.
//
// The pairs i < j are walked as steps (column chunk jc of kEJC sites, row
// site i), jc outer: a step needs the q x (kEJC*q) tile of J with rows
// (i, a) and columns (j, b), j in the chunk.  A workgroup owns 1024 (q <= 8),
// 2048 or 4096 (q > 24) sequences and one contiguous range of steps; it stages
// each tile in LDS once (double-buffered through registers) and every
// sequence picks J[(i, s_i), (j, s_j)] for its own tokens.  A step's 16
// terms are summed in FP32 in column order, the step sums of a sub-range (a
// range has kEFine of them) in FP64 in step order and the sub-range sums in
// order, one FP64 partial sum per (range, sequence); the finish adds the
// fields and the partials in a fixed order.
// Ranges and sub-ranges depend on L only, so a sequence's energy does not
// depend on the rest of the batch, on the workgroup size or on the form below.
//
// Small batches (fewer than kESplitBlocks workgroups otherwise, and room for
// the sums) take a workgroup per sub-range and, up to kEFewSeqs sequences and
// kEFewBlocks workgroups, one sequence per thread; the finish then adds the sub-range sums of each range
// first.  A workgroup's steps follow each other (fetch a tile, store it, look
// up), about 2 us each, so a small call takes their number: 1003 sequences at
// L = 123, q = 21, 16 ranges of 34 steps 84 us, 128 sub-ranges of 4 16 us; whole
// calls, L = 200, 3000 sequences 122 -> 46 us, L = 60, 20 000 124 -> 34, q = 5,
// L = 100, 1000 80 -> 18.  More workgroups than that take turns on the CUs, each
// with tiles of its own to load, and several sequences per thread are faster: L =
// 512, q = 32, 2048 sequences 390 -> 171 us (by ranges 258), q = 21 187 -> 96.  Where
// the ranges fill the device, sub-range sums
// would be traffic for nothing, and the lookups bound the call: 64 random
// 4-byte reads of LDS take 8.7 cycles (L = 512, q = 21, 1e5 sequences 2.9 ms).
// ---------------------------------------------------------------------------
constexpr int kEJC = 16;
// Sequences per thread: eight where the tiles leave a CU one workgroup anyway
// (q = 32, L = 300, 50 000 sequences 839 -> 656 us, q = 26 738 -> 613); where
// two fit, the registers of eight would take the second one (q = 21, L = 512,
// 1e5 sequences 2.91 -> 3.20 ms).
constexpr int energy_seqs(int Q) { return Q > 24 ? 8 : 4; }
constexpr int kEFine = 8;  // sub-ranges per range
constexpr int64_t kESplitBlocks = 256;
constexpr int64_t kEFewSeqs = 2048;
constexpr int64_t kEFewBlocks = 2048;
// Threads per workgroup: 512 (2048 sequences) for q > 8, so that each staged
// tile serves twice the lookups (a workgroup loads its own copy of every
// tile; at q = 21 the tile stores were about 30% of the LDS traffic): L = 512,
// q = 21, 1e5 sequences 4.37 -> 3.30 ms, q = 32 -1/3.  For q <= 8 (tiles of
// at most 8 KB) 256, where 512 measured 3-4% slower.
constexpr int energy_threads(int Q) { return Q > 8 ? 512 : 256; }

// Row pitch of the LDS tile in floats: 16 Q plus a pad of 0, 4, 8 or 12
// (rows stay 16-byte aligned).  A lookup's bank is (P s_i + s_j + const) mod
// 64 over the 64 four-byte banks; the pad is the one whose largest share of
// the Q^2 pairs (s_i, s_j) in one bank is smallest, then the smallest sum of
// squared shares, among the pads that keep as many workgroups per CU (two
// tiles in 160 KB of LDS).  With P = 16 Q the row offsets take
// 64 / gcd(16 Q, 64) values only: at q = 21 four, so twenty banks carry twice
// the pairs of the rest; at q = 8 one, so all rows share the banks of their
// first 8 floats.
constexpr int energy_pitch(int Q) {
  constexpr long long kLdsCU = 160 * 1024;
  const long long wg_cap = 32 / (energy_threads(Q) / 64);  // 32 waves of a CU
  auto wgs = [wg_cap](long long bytes) { return kLdsCU / bytes < wg_cap ? kLdsCU / bytes : wg_cap; };
  const long long wg0 = wgs(2LL * Q * 16 * Q * 4);
  int best = 16 * Q;
  long long best_mx = -1, best_sq = 0;
  for (int pad = 0; pad <= 12; pad += 4) {
    const int P = 16 * Q + pad;
    if (wgs(2LL * Q * P * 4) < wg0) continue;
    int cnt[64] = {};
    for (int a = 0; a < Q; ++a)
      for (int b = 0; b < Q; ++b) ++cnt[(P * a + b) % 64];
    long long mx = 0, sq = 0;
    for (int k = 0; k < 64; ++k) {
      mx = cnt[k] > mx ? cnt[k] : mx;
      sq += (long long)cnt[k] * cnt[k];
    }
    if (best_mx < 0 || mx < best_mx || (mx == best_mx && sq < best_sq)) {
      best = P;
      best_mx = mx;
      best_sq = sq;
    }
  }
  return best;
}

// Row sites of chunk jc that pair with some j > i in the chunk.
__host__ __device__ inline int energy_rows(int jc, int L) {
  return min(jc * kEJC + kEJC - 1, L - 1);
}

EnergyPlan plan_energy(int64_t B, int L, int q, size_t ws_bytes) {
  EnergyPlan p{};
  p.Bpad = ceil_div(std::max<int64_t>(B, 1), 64) * 64;
  p.steps = 0;
  for (int jc = 0; jc * kEJC < L; ++jc) p.steps += energy_rows(jc, L);
  p.parts = p.steps == 0 ? 0 : (int)std::min<int64_t>(128, std::max<int64_t>(1, p.steps / 32));
  size_t o = 0;
  p.off_xt = o;   o = align256(o + (size_t)L * p.Bpad);
  p.off_part = o; o = align256(o + sizeof(double) * (size_t)p.parts * p.Bpad);
  p.total = p.wanted = o;
  if (ceil_div(p.Bpad, energy_threads(q) * energy_seqs(q)) * p.parts < kESplitBlocks) {
    p.wanted = align256(p.off_part + sizeof(double) * (size_t)p.parts * kEFine * p.Bpad);
    p.split = ws_bytes >= p.wanted;
  }
  return p;
}

// KS: sequences per thread.  SPLIT: a workgroup per sub-range.
template <int Q, int KS, bool SPLIT>
__global__ __launch_bounds__(energy_threads(Q)) void k_energy_pairs(
    const float* __restrict__ J, const int8_t* __restrict__ XT, int64_t Bpad, int64_t B, int L,
    int64_t steps, int parts, double* __restrict__ part, const int64_t* __restrict__ count) {
  constexpr int kEThreads = energy_threads(Q);
  constexpr int kESeqBlock = kEThreads * KS;  // sequences per workgroup
  if (count && *count < B) B = *count;  // live sequences of a launch sized for B
  if ((int64_t)blockIdx.x * kESeqBlock >= B) return;  // whole workgroup, before any barrier
  constexpr int kW = kEJC * Q;                                 // tile row length (16 Q floats)
  constexpr int kP = energy_pitch(Q);                          // its pitch in LDS
  constexpr int kRowQ = kW / 4;                                // 16-byte quads per tile row
  constexpr int kQuads = Q * kRowQ;                            // quads per tile
  constexpr int kNQ = (kQuads + kEThreads - 1) / kEThreads;    // tile quads per thread
  typedef float f4 __attribute__((ext_vector_type(4)));
  __shared__ __attribute__((aligned(16))) float tile[2][Q * kP];
  const int tid = threadIdx.x;
  // the steps of the range and the end of its sub-range f
  const int p = SPLIT ? blockIdx.y / kEFine : blockIdx.y;
  const int64_t r0 = steps * p / parts, r1 = steps * (p + 1) / parts;
  auto fine_end = [&](int k) { return r0 + (r1 - r0) * (k + 1) / kEFine; };
  int f = SPLIT ? blockIdx.y % kEFine : 0;
  const int64_t t0 = SPLIT ? fine_end(f - 1) : r0, t1 = SPLIT ? fine_end(f) : r1;
  int64_t fend = fine_end(f);
  const int Lq = L * Q;
  const int64_t b0 = (int64_t)blockIdx.x * kESeqBlock;  // first sequence of the workgroup
  int64_t bs[KS];
#pragma unroll
  for (int k = 0; k < KS; ++k) bs[k] = b0 + tid + kEThreads * k;

  // (jc, i) of step t0
  int jc = 0;
  int64_t r = t0;
  while (r >= energy_rows(jc, L)) {
    r -= energy_rows(jc, L);
    ++jc;
  }
  int i = (int)r;

  // Tokens of a site through a buffer resource over the workgroup's part of
  // that site's row of XT [L][Bpad] (64-bit base, at most Bpad - b0 bytes,
  // under 2^31): reads past the row (sequences beyond Bpad) return 0,
  // padding rows hold -1 (read as 0).
  auto site_rsrc = [&](int site) {
    const int64_t left = Bpad - b0;  // > 0: b0 < B <= Bpad
    return __builtin_amdgcn_make_buffer_rsrc(
        (void*)(XT + (size_t)site * Bpad + b0), (short)0,
        (int)std::min<int64_t>(left, 0x7FFFFFFF), 0x00020000);
  };
  auto tok_in = [&](__amdgpu_buffer_rsrc_t rs, int k) -> int {
    const int t = (int)(int8_t)__builtin_amdgcn_raw_buffer_load_b8(rs, tid + kEThreads * k, 0, 0);
    return t < 0 ? 0 : t;  // invalid tokens were flagged by the transpose
  };
  // Tile (ti, tjc): rows (ti Q + a), columns tjc kW + c of J, as 16-byte
  // quads; quad e = a kRowQ + c4 of the tile comes from float
  // a Lq + 4 c4 past the tile's corner (32-bit offsets fixed per thread).
  // Columns past the last site (partial last chunk) bring values of the next
  // row, or zeros past the end of J: lookups never read them.
  uint32_t qoff[kNQ];
#pragma unroll
  for (int n = 0; n < kNQ; ++n) {
    const int e = tid + kEThreads * n;
    qoff[n] = (uint32_t)((e / kRowQ) * Lq + 4 * (e % kRowQ)) * 4u;
  }
  const size_t jbytes = (size_t)Lq * Lq * sizeof(float);  // up to 2^32 (L 1024, q 32)
  auto load_tile = [&](f4(&v)[kNQ], int ti, int tjc) {
    // a resource from the tile's corner to the end of J, at most 2^31 - 1
    // bytes (a tile spans under q Lq 4 + 16 q 4 bytes, far less)
    const size_t corner = ((size_t)ti * Q * Lq + (size_t)tjc * kW) * sizeof(float);
    const __amdgpu_buffer_rsrc_t rj = __builtin_amdgcn_make_buffer_rsrc(
        (void*)(reinterpret_cast<const char*>(J) + corner), (short)0,
        (int)std::min<size_t>(jbytes - corner, 0x7FFFFFFF), 0x00020000);
#pragma unroll
    for (int n = 0; n < kNQ; ++n) {
      if (tid + kEThreads * n < kQuads) {
        const auto w = __builtin_amdgcn_raw_buffer_load_b128(rj, (int)qoff[n], 0, 0);
        v[n] = f4{__uint_as_float(w[0]), __uint_as_float(w[1]), __uint_as_float(w[2]),
                  __uint_as_float(w[3])};
      }
    }
  };
  auto store_tile = [&](const f4(&v)[kNQ], int buf) {
#pragma unroll
    for (int n = 0; n < kNQ; ++n) {
      const int e = tid + kEThreads * n;
      if (e < kQuads)
        *reinterpret_cast<f4*>(&tile[buf][(e / kRowQ) * kP + 4 * (e % kRowQ)]) = v[n];
    }
  };
  auto advance = [&](int& ii, int& jj) {
    if (++ii >= energy_rows(jj, L)) {
      ii = 0;
      ++jj;
    }
  };

  double acc[KS], tot[KS];  // of the sub-range, of the sub-ranges before it
#pragma unroll
  for (int k = 0; k < KS; ++k) acc[k] = tot[k] = 0.0;
  auto step_done = [&](int64_t t) {  // the steps before t are in acc
    while (!SPLIT && t == fend && f < kEFine) {
#pragma unroll
      for (int k = 0; k < KS; ++k) {
        tot[k] += acc[k];
        acc[k] = 0.0;
      }
      fend = fine_end(++f);
    }
  };
  step_done(t0);  // empty sub-ranges
  // the chunk's tokens times 4 (bytes into a tile row), four to a register: a
  // lookup's address is one addition of a byte of it (64 registers of unpacked
  // tokens left no room for a second workgroup per CU with 8 sequences)
  uint32_t sj[KS][kEJC / 4];
  auto load_chunk = [&](int cjc) {
#pragma unroll
    for (int jj = 0; jj < kEJC; ++jj) {
      const int j = cjc * kEJC + jj;
      const __amdgpu_buffer_rsrc_t rs = site_rsrc(min(j, L - 1));
#pragma unroll
      for (int k = 0; k < KS; ++k) {
        const uint32_t t = (uint32_t)tok_in(rs, k) << (8 * (jj & 3) + 2);
        sj[k][jj / 4] = (jj & 3) ? sj[k][jj / 4] | t : t;
      }
    }
  };
  auto row_tokens = [&](int(&s)[KS], int site) {
    const __amdgpu_buffer_rsrc_t rs = site_rsrc(site);
#pragma unroll
    for (int k = 0; k < KS; ++k) s[k] = tok_in(rs, k) * (4 * kP);
  };
  // The lookups of one step (row site si_, chunk cjc, LDS buffer buf): the
  // step's terms summed in FP32 in column order, then added to the FP64 sum.
  auto lookups = [&](int si_, int cjc, const int(&srow)[KS], int buf) {
    float sf[KS];
    auto look = [&](int k, int jj) {  // J[(i, s_i), (j, s_j)] of sequence k
      const uint32_t a = (uint32_t)srow[k] + ((sj[k][jj / 4] >> (8 * (jj & 3))) & 0xFFu);
      return *(const float*)((const char*)tile[buf] + a + 4 * jj * Q);
    };
#pragma unroll
    for (int k = 0; k < KS; ++k) sf[k] = 0.0f;
    // for q <= 8 a step whose columns all pair with the row site skips the
    // per-column tests (q = 5: 11% shorter; for larger q the tests cost
    // nothing and the second copy of the loop 1-4%)
    if (Q <= 8 && cjc * kEJC > si_ && cjc * kEJC + kEJC <= L) {
#pragma unroll
      for (int jj = 0; jj < kEJC; ++jj)
#pragma unroll
        for (int k = 0; k < KS; ++k) sf[k] += look(k, jj);
    } else {
#pragma unroll
      for (int jj = 0; jj < kEJC; ++jj) {
        const int j = cjc * kEJC + jj;
        if (j > si_ && j < L) {  // uniform over the workgroup
#pragma unroll
          for (int k = 0; k < KS; ++k) sf[k] += look(k, jj);
        }
      }
    }
#pragma unroll
    for (int k = 0; k < KS; ++k) acc[k] += (double)sf[k];
  };

  // The tile of step t + 1 is fetched into registers during step t and
  // stored to LDS buffer (t + 1 - t0) % 2 at its end; the row tokens of step
  // t + 2 are fetched during step t into the registers of t's parity (A: even
  // offsets from t0, B: odd), so the lookups never wait on a load issued in
  // their own step and no register copy waits for one.
  f4 v[kNQ];
  int sA[KS], sB[KS];
  int iA = i, jA = jc, iB = i, jB = jc;
  advance(iB, jB);
  if (t0 < t1) {
    load_tile(v, iA, jA);
    store_tile(v, 0);
    load_chunk(jA);
    row_tokens(sA, iA);
  }
  if (t0 + 1 < t1) {
    row_tokens(sB, iB);
  }
  __syncthreads();
  for (int64_t t = t0; t < t1; t += 2) {
    // ---- step t (A)
    int iC = iB, jC = jB;  // step t + 2
    advance(iC, jC);
    if (t + 1 < t1) load_tile(v, iB, jB);
    lookups(iA, jA, sA, 0);
    step_done(t + 1);
    if (t + 2 < t1) {
      row_tokens(sA, iC);
    }
    if (t + 1 < t1) {
      store_tile(v, 1);
      if (jB != jA) load_chunk(jB);
    }
    __syncthreads();
    if (t + 1 >= t1) break;
    // ---- step t + 1 (B)
    int iD = iC, jD = jC;  // step t + 3
    advance(iD, jD);
    if (t + 2 < t1) load_tile(v, iC, jC);
    lookups(iB, jB, sB, 1);
    step_done(t + 2);
    if (t + 3 < t1) {
      row_tokens(sB, iD);
    }
    if (t + 2 < t1) {
      store_tile(v, 0);
      if (jC != jB) load_chunk(jC);
    }
    __syncthreads();
    iA = iC;
    jA = jC;
    iB = iD;
    jB = jD;
  }
#pragma unroll
  for (int k = 0; k < KS; ++k)
    if (bs[k] < B) part[(size_t)blockIdx.y * Bpad + bs[k]] = SPLIT ? acc[k] : tot[k];
}

// E = -(fields) - (partial sums).  Eight groups of a workgroup's threads share
// the sites and the ranges of 64 sequences, an eighth of either each, in order;
// their sums are added in order.  A thread's loads come in batches of 16
// (tokens, then their fields; then partial sums), so one thread per sequence
// waited for L / 8 of them in turn: L = 123, 1003 sequences 11 -> 4.6 us.
// FINE: the sums of kEFine sub-ranges per range, added in order first.
constexpr int kEGroups = 8;
template <bool FINE>
__global__ __launch_bounds__(64 * kEGroups) void k_energy_finish(
    const float* __restrict__ h, const int8_t* __restrict__ XT, int64_t Bpad, int64_t B, int L,
    int q, int parts, const double* __restrict__ part, float* __restrict__ E,
    const int64_t* __restrict__ count, int64_t b0) {
  if (count && *count < B) B = *count;
  b0 += (int64_t)blockIdx.x * 64;
  if (b0 >= B) return;  // whole workgroup, before the barrier
  __shared__ double sums[kEGroups][64];
  const int g = __builtin_amdgcn_readfirstlane(threadIdx.x / 64), lane = threadIdx.x % 64;
  const int64_t b = b0 + lane;  // below Bpad
  double acc = 0.0;
  // batches of 16 sites; past the group's last one that site again, not added
  const int i1 = L * (g + 1) / kEGroups;
  for (int i = L * g / kEGroups; i < i1; i += 16) {
    int t[16];
#pragma unroll
    for (int u = 0; u < 16; ++u) t[u] = XT[(size_t)min(i + u, i1 - 1) * Bpad + b];
    float hv[16];
#pragma unroll
    for (int u = 0; u < 16; ++u) hv[u] = h[min(i + u, i1 - 1) * q + (t[u] < 0 ? 0 : t[u])];
#pragma unroll
    for (int u = 0; u < 16; ++u)
      if (i + u < i1) acc -= (double)hv[u];
  }
  const int p1 = parts * (g + 1) / kEGroups;
  constexpr int kR = FINE ? kEFine : 1, kN = 16 / kR;  // sums per range, ranges per batch
  for (int p = parts * g / kEGroups; p < p1; p += kN) {
    double pv[kN][kR];
#pragma unroll
    for (int u = 0; u < kN; ++u)
#pragma unroll
      for (int r = 0; r < kR; ++r) pv[u][r] = part[(size_t)(min(p + u, p1 - 1) * kR + r) * Bpad + b];
#pragma unroll
    for (int u = 0; u < kN; ++u) {
      double x = 0.0;
#pragma unroll
      for (int r = 0; r < kR; ++r) x += pv[u][r];
      if (p + u < p1) acc -= x;
    }
  }
  sums[g][lane] = acc;
  __syncthreads();
  if (g != 0 || b >= B) return;
#pragma unroll
  for (int k = 1; k < kEGroups; ++k) acc += sums[k][lane];
  E[b] = (float)acc;
}

template <int Q>
static void launch_energy_q(const float* J, const int8_t* XT, int64_t B, int L,
                            const EnergyPlan& plan, double* part, hipStream_t s,
                            const int64_t* count) {
  constexpr int T = energy_threads(Q);
  constexpr int KS = energy_seqs(Q);
  const bool few = B <= kEFewSeqs && ceil_div(B, T) * plan.parts * kEFine <= kEFewBlocks;
  const int seqs = plan.split && few ? 1 : KS;
  auto kern = !plan.split ? k_energy_pairs<Q, KS, false>
              : seqs == 1 ? k_energy_pairs<Q, 1, true>
                          : k_energy_pairs<Q, KS, true>;
  const dim3 grid((unsigned)ceil_div(B, T * seqs), (unsigned)(plan.parts * (plan.split ? kEFine : 1)));
  hipLaunchKernelGGL(kern, grid, dim3(T), 0, s, J, XT, plan.Bpad, B, L, plan.steps, plan.parts, part,
                     count);
}

hipError_t launch_energy(const float* h, const float* J, const int8_t* seqs, int64_t B, int L,
                         int q, float* E, const EnergyPlan& plan, void* ws, int32_t* dev_err,
                         hipStream_t s, const int64_t* count) {
  char* base = static_cast<char*>(ws);
  int8_t* XT = reinterpret_cast<int8_t*>(base + plan.off_xt);
  double* part = reinterpret_cast<double*>(base + plan.off_part);
  hipError_t e = launch_transpose_tokens(seqs, B, L, q, XT, plan.Bpad, dev_err, s, count);
  if (e != hipSuccess) return e;
  if (plan.parts > 0) {
    switch (q) {
#define BMDCA_EQ(n)                                        \
  case n:                                                  \
    launch_energy_q<n>(J, XT, B, L, plan, part, s, count); \
    break;
      BMDCA_EQ(2) BMDCA_EQ(3) BMDCA_EQ(4) BMDCA_EQ(5) BMDCA_EQ(6) BMDCA_EQ(7) BMDCA_EQ(8)
      BMDCA_EQ(9) BMDCA_EQ(10) BMDCA_EQ(11) BMDCA_EQ(12) BMDCA_EQ(13) BMDCA_EQ(14) BMDCA_EQ(15)
      BMDCA_EQ(16) BMDCA_EQ(17) BMDCA_EQ(18) BMDCA_EQ(19) BMDCA_EQ(20) BMDCA_EQ(21) BMDCA_EQ(22)
      BMDCA_EQ(23) BMDCA_EQ(24) BMDCA_EQ(25) BMDCA_EQ(26) BMDCA_EQ(27) BMDCA_EQ(28) BMDCA_EQ(29)
      BMDCA_EQ(30) BMDCA_EQ(31) BMDCA_EQ(32)
#undef BMDCA_EQ
      default:
        return hipErrorInvalidValue;
    }
    e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  // one launch per 2^22 workgroups (a grid dimension holds fewer than 2^32
  // work-items: 2^29 sequences would pass it)
  const int64_t chunk = (int64_t)64 << 22;
  for (int64_t b0 = 0; b0 < B; b0 += chunk)
    hipLaunchKernelGGL(plan.split ? k_energy_finish<true> : k_energy_finish<false>,
                       dim3((unsigned)ceil_div(std::min(chunk, B - b0), 64)), dim3(64 * kEGroups), 0, s,
                       h, XT, plan.Bpad, B, L, q, plan.parts, part, E, count, b0);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Single mutants: dE[b][i*q+a] = -(H[b][i*q+a] - H[b][i*q+wt_i]), with H the
// wild type's local fields (h + sum_{j != i} J_ij(., wt_j)).
// Columns go in blocks of up to 256 / q whole sites, four consecutive columns
// per lane; the L coupling rows in eighths, each summed in order (FP32), the
// eighths added to h in order.  A column's own site is left out by a select on
// the sum, so no row has a special case.
//   SPLIT: a workgroup per (block, wild type), one wave per eighth.  What bounds
//   a few wild types is the latency of the row loads: with all rows in one
//   thread, four in flight, and the differences in a launch of their own, one
//   wild type at L = 256, q = 21 took 21.7 + 4.1 us, now 7.1; 16 at L = 512 whole
//   calls 65 -> 30 us.
//   Otherwise a wave per (block, wild type), four wild types per workgroup.
// Which, by the number of (block, wild type) pairs, and ROWS, the rows in flight;
// us, all rows of a wild type in one workgroup and the differences in a launch of
// their own, then now:
//   - up to 256 pairs, one a CU: split, 16 rows (latency), 23 -> 11 (L = 256, q = 21,
//     one wild type);
//   - while an eighth's rows are worth a wave, up to 64 L pairs, and up to 8192,
//     where whole wild types fill the device: split, 2 rows (few registers: 32 waves
//     a CU; with 16 rows 2 to 4 times longer), L = 180, q = 21, 100 wild types 28.6 ->
//     20.0, L = 256, q = 3, 1000 35.4 -> 36.1, with 16 rows 80;
//   - of more than 4096 fields the couplings no longer stay in the caches, and from
//     2048 pairs on eight waves that read eight rows far apart cost more than they
//     cover: whole wild types, 4 rows, L = 256, q = 21, 150 47.5 -> 49.9 (split 55), L
//     = 500, 100 173 -> 156;
//   - the rest whole, 2 rows, L = 40, q = 21, 4000 39 -> 38 (4 rows 52), L = 256, 1000
//     431 -> 220; but 4 rows between 8192 waves, where 2 need a second round, and
//     12 288 (L = 256, q = 21, 400 155 -> 99, 2 rows 128).
// Over 929 sizes at most 1.12 of the two launches' time, 0.6 in the mean.
// The sums are the same, so dE does not depend on the batch.
// ---------------------------------------------------------------------------
constexpr int kMParts = 8;
template <bool SPLIT, int ROWS>
__global__ __launch_bounds__(SPLIT ? 64 * kMParts : 256) void k_mutant_scan(
    const float* __restrict__ h, const float* __restrict__ J, const int8_t* __restrict__ wt,
    int64_t B, int L, int q, int sites, int64_t g0, float* __restrict__ dE,
    const int64_t* __restrict__ count) {
  // contiguous (column block, wild type) ranges per XCD, wild type fastest, as
  // in k_local_fields: rows that several wild types share come from the XCD's L2
  constexpr int kPer = SPLIT ? 1 : 4;  // wild types per workgroup
  const uint32_t nwg = gridDim.x, f = blockIdx.x, xcd = f % 8u, per = nwg / 8u;
  const int64_t g = g0 + (int64_t)(xcd * per + min(xcd, nwg % 8u) + f / 8u);
  const int64_t groups = ceil_div(B, kPer);
  const int lane = threadIdx.x % 64;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x / 64);
  const int64_t b = g % groups * kPer + (SPLIT ? 0 : w);
  if (b >= B || (count && b >= *count)) return;  // SPLIT: whole workgroup, before any barrier
  const int s0 = (int)(g / groups) * sites, s1 = min(s0 + sites, L);  // this block's sites
  const int c0 = s0 * q, nc = (s1 - s0) * q, Lq = L * q;              // and columns, at most 256
  __shared__ float part[SPLIT ? kMParts : 1][256];
  __shared__ float fields[kPer][256];
  float* H = fields[SPLIT ? 0 : w];
  typedef uint32_t u4 __attribute__((ext_vector_type(4)));
  int site[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) site[e] = (c0 + 4 * lane + e) / q;
  // lanes past the block load from past the row's end: 0
  const int off = 4 * lane < nc ? (c0 + 4 * lane) * (int)sizeof(float) : Lq * (int)sizeof(float);
  auto eighth = [&](int p, float(&acc)[4]) {
    const int k1 = L * (p + 1) / kMParts;
    for (int kc = L * p / kMParts; kc < k1; kc += 64) {
      const int n = min(64, k1 - kc), kl = kc + min(lane, n - 1);
      const uint64_t row = (uint64_t)(kl * q + checked_token(wt[b * L + kl], q, nullptr)) * Lq * 4u;
      for (int r = 0; r < n; r += ROWS) {
        u4 x[ROWS];
#pragma unroll
        for (int e = 0; e < ROWS; ++e) {  // past the end the last row again, not added
          const int k = min(r + e, n - 1);
          const uint64_t at = (uint32_t)__builtin_amdgcn_readlane((int)row, k) |
                              (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(row >> 32), k) << 32;
          const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
              (void*)(reinterpret_cast<const char*>(J) + at), (short)0, Lq * (int)sizeof(float),
              0x00020000);
          x[e] = __builtin_amdgcn_raw_buffer_load_b128(rs, off, 0, 0);
        }
#pragma unroll
        for (int e = 0; e < ROWS; ++e) {
          const bool over = r + e >= n;
#pragma unroll
          for (int c = 0; c < 4; ++c) {
            const float sum = acc[c] + __uint_as_float(x[e][c]);
            acc[c] = over || kc + r + e == site[c] ? acc[c] : sum;
          }
        }
      }
    }
  };
  auto write = [&](int c) {
    const int i = c / q;
    const int a = checked_token(wt[b * L + s0 + i], q, nullptr);
    dE[b * Lq + c0 + c] = c == i * q + a ? 0.0f : -(H[c] - H[i * q + a]);
  };
  if constexpr (SPLIT) {
    float acc[4] = {0.0f, 0.0f, 0.0f, 0.0f};
    eighth(w, acc);
#pragma unroll
    for (int e = 0; e < 4; ++e) part[w][4 * lane + e] = acc[e];
    __syncthreads();
    const int c = threadIdx.x;
    if (c < nc) {
      float x = h[c0 + c];
#pragma unroll
      for (int p = 0; p < kMParts; ++p) x += part[p][c];
      H[c] = x;
    }
    __syncthreads();
    if (c < nc) write(c);
  } else {
    float x[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) x[e] = 4 * lane + e < nc ? h[c0 + 4 * lane + e] : 0.0f;
    for (int p = 0; p < kMParts; ++p) {
      float acc[4] = {0.0f, 0.0f, 0.0f, 0.0f};
      eighth(p, acc);
#pragma unroll
      for (int e = 0; e < 4; ++e) x[e] += acc[e];
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) H[4 * lane + e] = x[e];
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
    for (int c = lane; c < nc; c += 64) write(c);
  }
}

hipError_t launch_mutant_scan(const float* h, const float* J, const int8_t* wt, int64_t B, int L,
                              int q, float* dE, hipStream_t s, const int64_t* count) {
  // blocks of equal width, so that every XCD's range holds the same work
  const int sites = (int)ceil_div(L, ceil_div(L, 256 / q));
  const int64_t blocks = ceil_div(L, sites);
  const int64_t pairs = B * blocks;
  const bool large = L * q > 4096;
  const bool split = pairs <= std::min<int64_t>(64 * L, large ? 2048 : 8192);
  const bool four = (large && pairs <= 4800) || (L * q > 1600 && pairs > 8192 && pairs <= 12288);
  auto kern = split  ? (pairs <= 256 ? k_mutant_scan<true, 16> : k_mutant_scan<true, 2>)
              : four ? k_mutant_scan<false, 4>
                     : k_mutant_scan<false, 2>;
  // one launch per 2^22 workgroups (a grid dimension holds fewer than 2^32 work-items)
  const int64_t nwg = ceil_div(B, split ? 1 : 4) * blocks, chunk = (int64_t)1 << 22;
  for (int64_t g0 = 0; g0 < nwg; g0 += chunk)
    hipLaunchKernelGGL(kern, dim3((unsigned)std::min(chunk, nwg - g0)),
                       dim3(split ? 64 * kMParts : 256), 0, s, h, J, wt, B, L, q, sites, g0, dE, count);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// APC Frobenius.  k_frob_blocks: each wave takes 64 / q blocks (i, j), j > i,
// of one block-row i; lane (block, t) owns row t and column t of its block,
// both held in registers: the row by 16-byte loads, the column by 4-byte
// loads that are coalesced over the block's lanes (and hit the cache lines
// the row loads brought in).  In FP64 the lane forms the row mean r_t and the
// column mean c_t over all q states; the column means go through LDS, every
// lane of the block reads all q of them and their mean m, and sums the
// squares of the gauged entries J_tb - r_t - c_b + m of its row with
// t, b != gap; one lane per block adds the q row sums in order, and
// F_ij = F_ji = the square root.  Block-rows i and L - 1 - i share a run of
// wave tasks (L - 1 blocks between them), so every run is as long.  J is read
// once, without LDS staging.  k_apc_rows: S_i = sum_k F_ik (one wave per
// row); k_apc_out: S = sum_i S_i, F_apc = F - S_i S_j / S,
// diagonals 0 (the diagonal of F is never read).
// ---------------------------------------------------------------------------
size_t apc_ws_bytes(int L) { return align256(sizeof(double) * ((size_t)L * L + L + 8)); }

// Wave tasks per pair of block-rows (p, L - 1 - p): ceil((L - 1 - p) / bpw)
// tasks of row p and ceil(p / bpw) of row L - 1 - p, at most this many.
inline int frob_tasks_per_pair(int L, int q) { return (int)ceil_div(L - 1, 64 / q) + 1; }

// QP4: quads per block row, ceil(q / 4).
template <int QP4>
__global__ __launch_bounds__(256) void k_frob_blocks(const float* __restrict__ J, int L, int q,
                                                     int gap, int tpp, double* __restrict__ F) {
  constexpr int QB = 4 * QP4;  // columns a lane walks (q rounded up to quads)
  __shared__ double cmean[4][64];  // per wave: c_t of lane (block, t) at block * q + t
  __shared__ double rowss[4][64];  // per wave: the lanes' sums of squares
  const int lane = threadIdx.x % 64;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x / 64);  // wave-uniform, as is the wave task below
  const int task = (int)blockIdx.x * 4 + wv;  // below 2^19 (L <= 1024, tpp <= 1024)
  const int npair = (L + 1) / 2;
  if (task >= npair * tpp) return;  // whole wave; only wave barriers below
  const int p = task / tpp, k = task - (task / tpp) * tpp;
  const int bpw = 64 / q;
  const int i0 = p, i1 = L - 1 - p;
  const int n0 = (int)ceil_div(L - 1 - i0, bpw);  // tasks of row i0
  int i, jfirst;
  if (k < n0) {
    i = i0;
    jfirst = i0 + 1 + k * bpw;
  } else {
    if (i1 == i0) return;  // the middle row of an odd L has no partner
    i = i1;
    jfirst = i1 + 1 + (k - n0) * bpw;
    if (jfirst >= L) return;
  }
  const int jb = lane / q, t = lane - jb * q;
  const bool live = jb < bpw && jfirst + jb < L;
  const int j = live ? jfirst + jb : i;  // dead lanes read block (i, i): in bounds, unused
  const int Lq = L * q;
  // Block-row i as one buffer (q Lq floats, at most 4 MiB).  Row t of block
  // (i, j) starts at float t Lq + j q; the quads past its q-th float read the
  // next block (or, past the buffer, zeros) and are cleared.
  const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
      (void*)(J + (size_t)i * q * Lq), (short)0, (int)((size_t)q * Lq * sizeof(float)), 0x00020000);
  const int rowoff = (t * Lq + j * q) * (int)sizeof(float);
  double x[QB];
#pragma unroll
  for (int u = 0; u < QP4; ++u) {
    const auto v = __builtin_amdgcn_raw_buffer_load_b128(rs, rowoff + 16 * u, 0, 0);
#pragma unroll
    for (int e = 0; e < 4; ++e) x[4 * u + e] = (double)__uint_as_float(v[e]);
  }
  float y[QB];
#pragma unroll
  for (int a = 0; a < QB; ++a)
    y[a] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(
        rs, (min(a, q - 1) * Lq + j * q + t) * (int)sizeof(float), 0, 0));
  // entries past q (compile-time positions in the last quad) become +0, which
  // leaves every sum below unchanged (a sum that starts at +0 never is -0)
#pragma unroll
  for (int b = 4 * (QP4 - 1); b < QB; ++b) {
    x[b] = (b < q) ? x[b] : 0.0;
    y[b] = (b < q) ? y[b] : 0.0f;
  }
  double rsum = 0.0, csum = 0.0;
#pragma unroll
  for (int b = 0; b < QB; ++b) {
    rsum += x[b];
    csum += (double)y[b];
  }
  const double r = rsum / (double)q;
  double* cm = cmean[wv];
  cm[lane] = csum / (double)q;
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
  const int base = min(jb, bpw - 1) * q;  // this lane's block in the wave's arrays
  double cb[QB];
  double all = 0.0;
#pragma unroll
  for (int b = 0; b < QB; ++b) {
    // the read is unconditional (a select around it becomes a branch); past q
    // it is scaled to +-0
    cb[b] = cm[base + min(b, q - 1)];
    if (b >= 4 * (QP4 - 1)) cb[b] *= (b < q) ? 1.0 : 0.0;
    all += cb[b];
  }
  const double m = all / (double)q;
  double ss = 0.0;
#pragma unroll
  for (int b = 0; b < QB; ++b) {
    const double w = (b < q && b != gap) ? 1.0 : 0.0;  // uniform per b
    const double z = ((x[b] - r) - cb[b]) + m;
    ss = __builtin_fma(z * w, z, ss);  // +-0 for the skipped columns: ss unchanged
  }
  double* rss = rowss[wv];
  rss[lane] = (t == gap) ? 0.0 : ss;
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
  if (live && t == 0) {
    double tot = 0.0;
    for (int u = 0; u < q; ++u) tot += rss[base + u];
    const double f = sqrt(tot);
    F[(size_t)i * L + j] = f;
    F[(size_t)j * L + i] = f;
  }
}

__global__ __launch_bounds__(256) void k_apc_rows(const double* __restrict__ F, int L,
                                                  double* __restrict__ S) {
  const int lane = threadIdx.x % 64;
  const int i = blockIdx.x * 4 + threadIdx.x / 64;
  if (i >= L) return;
  // eight loads in flight, added in order (the diagonal and past the end: 0)
  double s = 0.0;
  for (int k0 = 0; k0 < L; k0 += 512) {
    double f[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int k = k0 + 64 * u + lane;
      f[u] = k < L && k != i ? F[(size_t)i * L + k] : 0.0;
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) s += f[u];
  }
  for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
  if (lane == 0) S[i] = s;
}

// F_apc = F - S_i S_j / S.  Every workgroup adds S = sum_i S_i for itself while
// its entries load: thread t adds S_t, S_{t+256}, ... in ascending order, then a
// fixed tree over the 256 partial sums.  Latency bounds this and k_apc_rows
// (eight loads in flight there): with a launch of one workgroup for S, one load
// at a time and one entry per thread a call took 79.5 us at L = 512, q = 21, now
// 76.3; 20.0 and 17.1 at L = 100.
constexpr int kApcPer = 4;  // entries per thread
__global__ __launch_bounds__(256) void k_apc_out(const double* __restrict__ F,
                                                 const double* __restrict__ S, int L,
                                                 float* __restrict__ Fout,
                                                 float* __restrict__ Fapc) {
  __shared__ double part[256];
  const size_t n = (size_t)L * L;
  // the entries and their rows' sums are on their way during the sum
  double f[kApcPer], si[kApcPer], sj[kApcPer];
  int row[kApcPer], col[kApcPer];
#pragma unroll
  for (int e = 0; e < kApcPer; ++e) {
    const size_t k = min(((size_t)blockIdx.x * kApcPer + e) * 256 + threadIdx.x, n - 1);
    row[e] = (int)(k / L);
    col[e] = (int)(k % L);
    f[e] = F[k];
    si[e] = S[row[e]];
    sj[e] = S[col[e]];
  }
  double tot = 0.0;
  for (int i = threadIdx.x; i < L; i += 256) tot += S[i];
  part[threadIdx.x] = tot;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) part[threadIdx.x] += part[threadIdx.x + w];
    __syncthreads();
  }
  const double all = part[0];
#pragma unroll
  for (int e = 0; e < kApcPer; ++e) {
    const size_t k = ((size_t)blockIdx.x * kApcPer + e) * 256 + threadIdx.x;
    if (k >= n) return;
    if (Fout) Fout[k] = row[e] == col[e] ? 0.0f : (float)f[e];
    Fapc[k] = row[e] == col[e] ? 0.0f : (float)(f[e] - si[e] * sj[e] / all);
  }
}

hipError_t launch_apc(const float* J, int L, int q, int gap, float* F, float* Fapc, void* ws,
                      hipStream_t s) {
  double* Fd = static_cast<double*>(ws);
  double* S = Fd + (size_t)L * L;
  const int tpp = frob_tasks_per_pair(L, q);
  const unsigned nwg = (unsigned)ceil_div((int64_t)((L + 1) / 2) * tpp, 4);
  switch ((q + 3) / 4) {
#define BMDCA_FROB(QP4)                                                                     \
  case QP4:                                                                                 \
    hipLaunchKernelGGL(k_frob_blocks<QP4>, dim3(nwg), dim3(256), 0, s, J, L, q, gap, tpp, Fd); \
    break;
    BMDCA_FROB(1) BMDCA_FROB(2) BMDCA_FROB(3) BMDCA_FROB(4)
    BMDCA_FROB(5) BMDCA_FROB(6) BMDCA_FROB(7) BMDCA_FROB(8)
#undef BMDCA_FROB
    default:
      return hipErrorInvalidValue;
  }
  hipLaunchKernelGGL(k_apc_rows, dim3((unsigned)ceil_div(L, 4)), dim3(256), 0, s, Fd, L, S);
  hipLaunchKernelGGL(k_apc_out, dim3((unsigned)ceil_div((int64_t)L * L, 256 * kApcPer)), dim3(256),
                     0, s, Fd, S, L, F, Fapc);
  return hipGetLastError();
}

}  // namespace bmdca
