// Heat-bath sweeps of few chains (adabmDCA 2.0, Sec. 2.1): a workgroup per
// chain, coupling rows fetched for that chain alone.  Same draws as the gather
// form.
#include "gather_kernel.hpp"

namespace bmdca {

// ---------------------------------------------------------------------------
// With few chains per CU the gather form's time is the staging: every
// workgroup streams site i's whole block run (L q QP floats) through LDS for
// the handful of rows its chains read (L = 200, q = 21, 100 chains: 9.4 us per
// visit, whatever the chain count).  Here a workgroup owns one chain and
// fetches only the L rows (j, s_j) it needs, straight from J.
//
// What bounds a visit then is one serial chain: the field sum runs over j in
// the gather kernel's order (ascending within each of its S site groups, one
// dependent add per row), the draw follows, and the next site's sum needs the
// drawn state.  Only the rows from that state's on, though: W = 2 or 3 waves
// take the visits in turn, and while one adds its last rows and draws, the
// next has its rows loaded and everything before the row still unknown added.
//
//   - tab[] holds the byte offset in J of every 16-byte quad of the chain's
//     rows; a wave's rows go to its own LDS buffer by direct buffer->LDS
//     loads, 64 quads each, row j at j * QP floats.  (Successive sites read
//     the same rows q floats further on: half of them on lines that the
//     previous visit brought into the caches.)
//   - when a wave loads for visit t (right after its visit t - W) the states
//     of the W - 1 visits before t are unknown: it loads the whole q x q blocks
//     of (this site, those sites) as well and picks the row when the state is
//     published.  The row of the site itself (the diagonal block of J, ignored
//     by contract) is cleared.
//   - lane (u, a) = u * 4V + a adds state a over the sites j = u, u + S, ...,
//     the order of the gather kernel's 8-lane chain (S site groups of V
//     quads); then an exchange through LDS gives lane p the quad p that lane
//     p of such a chain holds, and the draw is that kernel's, step by step, so
//     a chain draws the same bits as there.
//   - a drawn state is published in pub[t % 4] as (t, state); the other waves
//     of the workgroup poll it.  A slot is reused four visits later, after the
//     visits t + 1 .. t + 3 that read it have been drawn.
// ---------------------------------------------------------------------------
typedef float few_f4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) float lds_f;
typedef __attribute__((address_space(3))) few_f4 lds_f4;
typedef __attribute__((address_space(3))) uint32_t lds_u;
typedef __attribute__((address_space(3))) unsigned char lds_b;

template <int Q, int W>
__global__ __launch_bounds__(64 * W) void k_gibbs_few(
    const float* __restrict__ h, const float* __restrict__ J, int8_t* __restrict__ chains,
    int64_t N, int L, int rowf, int sweeps, uint32_t k0, uint32_t k1, uint64_t sweep_offset,
    float beta, unsigned long long* flips_out, int32_t* dev_err,
    const uint64_t* __restrict__ epoch, const int32_t* __restrict__ run,
    const ChainStream* __restrict__ streams, const int64_t* __restrict__ count) {
  if (run && *run == 0) return;
  if (count && *count < N) N = *count;
  const int64_t c = blockIdx.x;
  if (c >= N) return;  // whole workgroup, before any barrier
  if (epoch) sweep_offset += *epoch * (uint64_t)sweeps;
  constexpr int QP = gather_qp(Q), NQ = QP / 4, V = gather_v(Q), S = gather_s(Q, 8);
  constexpr int vL = (Q - 1) / 4, eL = (Q - 1) % 4;  // lane and slot of state q-1
  constexpr int NB = (Q * NQ + 63) / 64;             // loads of a q x q block
  constexpr int D = W - 1;                           // states unknown when a visit is loaded
  constexpr uint32_t kPast = 0x80000000u;            // past the end of J: reads 0
  extern __shared__ __attribute__((aligned(16))) unsigned char g_smem[];
  const int lane = threadIdx.x & 63;
  const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int nit = (L * NQ + 63) / 64;  // loads of a visit's rows
  const int wavef = rowf + D * NB * 256 + 64 + 32;  // floats of a wave's buffers
  lds_f* smem = (lds_f*)g_smem;
  lds_f* rows = smem + wid * wavef;         // [rowf]
  lds_f* blk = rows + rowf;                 // [D][NB * 256]
  lds_f* hbuf = blk + D * NB * 256;         // [64]
  lds_f* xch = hbuf + 64;                   // [32]
  lds_u* tab = (lds_u*)(smem + W * wavef);  // [nit * 64]
  lds_u* pub = tab + nit * 64;              // [4]
  lds_b* tok = (lds_b*)(pub + 4);           // [L]
  uint32_t cid = (uint32_t)c;
  if (streams) {
    const ChainStream st = streams[c];
    k0 = (uint32_t)st.seed;
    k1 = (uint32_t)(st.seed >> 32);
    cid = st.chain;
    sweep_offset += st.sweep_offset;
  }
  const uint32_t Lq = (uint32_t)(L * Q);
  const uint32_t jbytes = Lq * Lq * 4u;  // at most 2^30 (L <= 512, q <= 32)

  // rows past L (up to whole groups of positions) stay zero
  for (int k = lane; k < rowf; k += 64) rows[k] = 0.0f;
  for (int e = L * NQ + (int)threadIdx.x; e < nit * 64; e += 64 * W) tab[e] = kPast;
  for (int j = threadIdx.x; j < L; j += 64 * W) {
    const int t = checked_token(chains[c * L + j], Q, dev_err);
    tok[j] = (unsigned char)t;
    for (int v = 0; v < NQ; ++v)
      tab[j * NQ + v] = ((uint32_t)(j * Q + t) * Lq + 4u * v) * 4u;
  }
  if (threadIdx.x < 4) pub[threadIdx.x] = ~0u;
  __syncthreads();

  uint32_t boff[NB];  // this lane's quads of a q x q block, from its corner
#pragma unroll
  for (int n = 0; n < NB; ++n) {
    const int e = 64 * n + lane, b = e / NQ, v = e % NQ;
    boff[n] = b < Q ? ((uint32_t)b * Lq + 4u * v) * 4u : kPast;
  }
  auto rsrc = [&](uint32_t first) {  // J from float `first` on
    return __builtin_amdgcn_make_buffer_rsrc((void*)(J + first), (short)0,
                                             (int)(jbytes - first * 4u), 0x00020000);
  };
  // the site d visits before site i's
  auto back = [&](int i, int d) {
    int r = i - d;
    while (r < 0) r += L;
    return r;
  };
  // Loads of a visit to site i: the rows by the offsets in tab, the blocks of
  // the D sites before it, h_i one state per lane.
  auto issue = [&](int i) {
    const __amdgpu_buffer_rsrc_t rs = rsrc((uint32_t)(i * Q));
    auto some = [&](int it, auto n_c) {
      constexpr int n = decltype(n_c)::value;
      uint32_t off[n];
#pragma unroll
      for (int e = 0; e < n; ++e) off[e] = tab[64 * (it + e) + lane];
#pragma unroll
      for (int e = 0; e < n; ++e)
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (lds_void_t*)(rows + 256 * (it + e)), 16,
                                                 (int)off[e], 0, 0, 0);
    };
    int it = 0;
    for (; it + 8 <= nit; it += 8) some(it, std::integral_constant<int, 8>{});
    if (nit & 4) { some(it, std::integral_constant<int, 4>{}); it += 4; }
    if (nit & 2) { some(it, std::integral_constant<int, 2>{}); it += 2; }
    if (nit & 1) some(it, std::integral_constant<int, 1>{});
#pragma unroll
    for (int d = 1; d <= D; ++d) {
      const __amdgpu_buffer_rsrc_t rb = rsrc((uint32_t)(back(i, d) * Q) * Lq + (uint32_t)(i * Q));
#pragma unroll
      for (int n = 0; n < NB; ++n)
        __builtin_amdgcn_raw_ptr_buffer_load_lds(
            rb, (lds_void_t*)(blk + ((d - 1) * NB + n) * 256), 16, (int)boff[n], 0, 0, 0);
    }
    const __amdgpu_buffer_rsrc_t rh = __builtin_amdgcn_make_buffer_rsrc(
        (void*)(h + i * Q), (short)0, (int)((Lq - (uint32_t)(i * Q)) * 4u), 0x00020000);
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rh, (lds_void_t*)hbuf, 4, 4 * lane, 0, 0, 0);
  };

  const int Lr = (L + S - 1) / S;  // positions per site group
  const int p = lane & 7, v = p % V;
  const int ua = (lane & 31) / (4 * V), aa = min((lane & 31) % (4 * V), QP - 1);
  const lds_f* rp = rows + ua * QP + aa;  // position r at r * S * QP
  constexpr int kPos = S * QP;
  const int64_t Tn = (int64_t)sweeps * L;
  unsigned long long nflip = 0;
  // state drawn at visit t (site r); the initial state before the first visit
  auto drawn = [&](int64_t t, int r) -> int {
    if (t < 0) return __builtin_amdgcn_readfirstlane((int)tok[r]);
    const volatile lds_u* pv = pub + (t & 3);
    uint32_t w;
    do {
      w = (uint32_t)__builtin_amdgcn_readfirstlane((int)*pv);
    } while ((w >> 8) != ((uint32_t)t & 0xFFFFFFu));
    return (int)(w & 255u);
  };
  int i = wid % L;
  int sw = wid / L;  // sweep of visit t
  if (wid < Tn) issue(i);
  for (int64_t t = wid; t < Tn; t += W) {
    const uint32_t sg = (uint32_t)(sweep_offset + (uint64_t)sw);
    const uint4 rnd = philox4x32_10(make_uint4((uint32_t)i >> 2, sg, cid, 0u), k0, k1);
    const float uni = word_to_uniform(pick_word(rnd, i & 3));
    const int r1 = back(i, 1), q1 = r1 / S;  // the site drawn last, and its position
    compiler_fence();
    wait_vm_lgkm0<0>();
    compiler_fence();
    if (lane < QP) rows[i * QP + lane] = 0.0f;
    compiler_fence();

    // ---- state a of site group u over the positions [0, Lr) in order
    float acc1 = 0.0f;
    auto ld = [&](float(&z)[8], int r) {
#pragma unroll
      for (int e = 0; e < 8; ++e) z[e] = rp[(r + e) * kPos];
    };
    auto ad = [&](const float(&z)[8]) {
#pragma unroll
      for (int e = 0; e < 8; ++e) acc1 += z[e];
    };
    // x holds positions r..r+7: adds them and the 8 after them, each group
    // read while the one before it is added; then x holds r+16..r+23
    auto two = [&](float(&x)[8], float(&y)[8], int r, bool more) {
      ld(y, r + 8);
      __builtin_amdgcn_sched_barrier(0);
      ad(x);
      if (more) ld(x, r + 16);
      __builtin_amdgcn_sched_barrier(0);
      ad(y);
    };
    // positions [r0, r1e), exactly
    auto seg = [&](int r0, int r1e) {
      float x[8], y[8];
      int r = r0;
      if (r + 8 <= r1e) {
        ld(x, r);
        for (; r + 24 <= r1e; r += 16) two(x, y, r, true);
        if (r + 16 <= r1e) {
          two(x, y, r, false);
          r += 16;
        } else {
          ad(x);
          r += 8;
        }
      }
      if (r < r1e) {
        ld(x, r);
#pragma unroll
        for (int e = 0; e < 7; ++e) acc1 += r + e < r1e ? x[e] : 0.0f;
      }
    };
    int r = 0;
    if constexpr (D == 2) {
      // (site 1 of a sweep: the row before last is the last one, r2 > r1 = 0)
      const int r2 = back(i, 2), q2 = r2 / S;
      const bool before = r2 < r1;
      if (before) {
        seg(0, q2);
        r = q2;
      }
      const int s2 = drawn(t - 2, r2);
      if (r2 != i && lane < QP) rows[r2 * QP + lane] = blk[NB * 256 + s2 * QP + lane];
      compiler_fence();
      if (before) {
        seg(q2, q1);
        r = q1;
      }
    } else {
      seg(0, q1);
      r = q1;
    }
    // from the unknown row's position on, its first 8 positions read ahead
    float z0 = rp[r * kPos], x[8], y[8];
    ld(x, r + 1);
    const few_f4 hc = *(const lds_f4*)(hbuf + 4 * v);
    const int s1 = drawn(t - 1, r1);
    __builtin_amdgcn_s_setprio(3);  // the other waves wait for this one's draw
    const int told = tok[i];
    const float xb = blk[s1 * QP + aa];
    if (r1 != i && ua == r1 % S) z0 = xb;
    acc1 += z0;
    ++r;
    for (; r + 16 < Lr; r += 16) two(x, y, r, true);
    if (r + 8 < Lr)  // positions past Lr are zero rows
      two(x, y, r, false);
    else if (r < Lr)
      ad(x);
    if (lane < 32) xch[lane] = acc1;
    compiler_fence();
    few_f4 acc = *(const lds_f4*)(xch + 4 * p);
    compiler_fence();

    // ---- the gather kernel's draw for an 8-lane chain, on every 8 lanes
#pragma unroll
    for (int e = 0; e < 4; ++e) acc[e] = combine_sites<V, 8>(acc[e]);
    float l[4];
    float mx = -INFINITY;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const bool ok = v < NQ && 4 * v + e < Q;
      l[e] = ok ? beta * (hc[e] + acc[e]) : -INFINITY;
      mx = fmaxf(mx, l[e]);
    }
    mx = group_max<V>(mx);
    float P[4];
    float run_sum = 0.0f;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const bool ok = v < NQ && 4 * v + e < Q;
      run_sum += ok ? __expf(l[e] - mx) : 0.0f;
      P[e] = run_sum;
    }
    const float inc = group_scan<V>(run_sum, v);
    float excl = V > 1 ? dpp_f<kDppShr1>(inc) : 0.0f;
    if (v == 0) excl = 0.0f;
    const float Stot = group_bcast<V, vL>(excl + P[eL], v);  // S_{q-1}
    const float uz = uni * Stot;
    int cnt = 0;
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (v < NQ && 4 * v + e < Q - 1 && excl + P[e] <= uz) ++cnt;
    cnt = __builtin_amdgcn_readfirstlane(group_sum<V>(cnt));
    // what the other waves read after they see the state goes first (a wave's
    // LDS operations are in order)
    if (lane < NQ) tab[i * NQ + lane] = ((uint32_t)(i * Q + cnt) * Lq + 4u * lane) * 4u;
    if (lane == 0) tok[i] = (unsigned char)cnt;
    compiler_fence();
    if (lane == 0) *(volatile lds_u*)(pub + (t & 3)) = ((uint32_t)t << 8) | (uint32_t)cnt;
    compiler_fence();
    __builtin_amdgcn_s_setprio(0);
    nflip += cnt != told ? 1 : 0;
    i += W;
    while (i >= L) {
      i -= L;
      ++sw;
    }
    // the buffers' reads are done (their sums were used) before they are loaded again
    if (t + W < Tn) issue(i);
  }
  __syncthreads();
  for (int j = threadIdx.x; j < L; j += 64 * W) chains[c * L + j] = (int8_t)tok[j];
  if (flips_out && lane == 0 && nflip) atomicAdd(flips_out, nflip);
}

template <int Q, int W>
static hipError_t launch_few_qw(const float* J, const GatherArgs& a, const FewShape& f) {
  auto kern = k_gibbs_few<Q, W>;
  const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)f.lds);
  if (e != hipSuccess) return e;
  const DevCtl& ctl = *a.ctl;
  hipLaunchKernelGGL(kern, dim3((unsigned)a.N), dim3(64 * W), f.lds, a.s, a.h, J, a.chains, a.N,
                     a.L, f.rowf, a.sweeps, (uint32_t)a.seed, (uint32_t)(a.seed >> 32),
                     a.sweep_offset, a.beta, a.flips_out, a.dev_err, ctl.epoch, ctl.active,
                     ctl.streams, ctl.count);
  return hipGetLastError();
}

template <int Q>
static hipError_t launch_few_q(const float* J, const GatherArgs& a, int64_t cus) {
  const FewShape f = few_plan(a.N, a.L, Q, cus);
  return f.waves == 3 ? launch_few_qw<Q, 3>(J, a, f) : launch_few_qw<Q, 2>(J, a, f);
}

hipError_t launch_gather_few(int q, const float* J, const GatherArgs& a, int64_t cus) {
  switch (q) {
#define BMDCA_GQ(n) \
  case n:           \
    return launch_few_q<n>(J, a, cus);
    BMDCA_GQ(2) BMDCA_GQ(3) BMDCA_GQ(4) BMDCA_GQ(5) BMDCA_GQ(6) BMDCA_GQ(7) BMDCA_GQ(8)
    BMDCA_GQ(9) BMDCA_GQ(10) BMDCA_GQ(11) BMDCA_GQ(12) BMDCA_GQ(13) BMDCA_GQ(14) BMDCA_GQ(15)
    BMDCA_GQ(16) BMDCA_GQ(17) BMDCA_GQ(18) BMDCA_GQ(19) BMDCA_GQ(20) BMDCA_GQ(21) BMDCA_GQ(22)
    BMDCA_GQ(23) BMDCA_GQ(24) BMDCA_GQ(25) BMDCA_GQ(26) BMDCA_GQ(27) BMDCA_GQ(28) BMDCA_GQ(29)
    BMDCA_GQ(30) BMDCA_GQ(31) BMDCA_GQ(32)
#undef BMDCA_GQ
    default:
      return hipErrorInvalidValue;
  }
}

}  // namespace bmdca
