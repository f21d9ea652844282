// Gather-form sampler whose waves run free (adabmDCA 2.0, Sec. 2.1): the
// draws and the LDS layout of gather_kernel.hpp with a loading wave and
// counters in the place of the barriers.
#pragma once
#include "gather_kernel.hpp"

namespace bmdca {

// ---------------------------------------------------------------------------
// In gather_kernel.hpp every wave meets a barrier per chunk-step (or per two)
// and the waves that hold chains also issue the loads.  A step there takes
// about 1700 cycles at q = 21 with 24 chains on a CU as with 80: the barrier
// lines every wave up with the slowest, so LDS reads, draws and load issue do
// not cover each other, and half of a wave's instructions are load issue and
// bookkeeping.  Here the chains' waves only wait for data:
//
//   - one more wave loads.  It waits until every wave has consumed the chunk
//     that a slot holds, loads the slot, and publishes in LDS how many chunks
//     are complete (chunk t - 1 once chunk t is on its way);
//   - a chains' wave reads that count only when it has used up the chunks that
//     it knows to be complete, and counts the chunks it has consumed in LDS (a
//     wave's LDS operations are in order, so the count follows its reads).
//
// So waves may be up to three chunks apart and one's draw is covered by the
// others' reads.  Every wait ends: all waves of a workgroup are resident, the
// loader waits for chunks that are published, the others for chunks that it
// loads next.  h_i comes by a vector load a visit ahead: without scalar loads
// in the loop the waits of the LDS reads stay exact.  Sums and draws are those
// of gather_kernel.hpp, so chains draw the same bits.
//
// What bounds it: up to 40 chains per CU the latency of a wave's own row reads
// and adds (24 chains and 80 chains differ by a quarter), above that the LDS
// reads.  Chunks in flight: publishing one chunk later (three in flight, two
// loading waves) cost 5-15%, as the waves' slack is worth more; polls with a
// sleep between cost 2-6%; twelve lanes per chain (two states each) -6 to
// +20%.  Barriers -> free, ms, 256 CUs: q = 21, L = 100, 10 sweeps, N = 6000
// 5.40 -> 4.21, 10 000 5.22 -> 4.45, 18 000 5.49 -> 5.34; L = 256, 3 sweeps,
// N = 6000 8.97 -> 6.68, 20 000 8.94 -> 8.54; L = 512, 1 sweep, N = 10 000
// 11.69 -> 9.24, 20 000 24.5 -> 19.0; q = 25, L = 150, 3 sweeps, N = 6000
// 8.95 -> 5.49; Metropolis q = 21, 10 sweeps, L = 100, N = 10 000 3.90 -> 3.34,
// L = 127, N = 8191 5.74 -> 4.68.
// ---------------------------------------------------------------------------

// LDS by byte address.
__device__ __forceinline__ uint32_t lds_addr(const float* p) {
  return (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const float*)p;
}
__device__ __forceinline__ uint32_t lds_dword(uint32_t a) {
  return *(__attribute__((address_space(3))) const uint32_t*)(uintptr_t)a;
}
__device__ __forceinline__ uint32_t lds_dword_now(uint32_t a) {  // read again on every call
  return *(volatile __attribute__((address_space(3))) const uint32_t*)(uintptr_t)a;
}
__device__ __forceinline__ void lds_put(uint32_t a, uint32_t x) {
  *(volatile __attribute__((address_space(3))) uint32_t*)(uintptr_t)a = x;
}
// f(integral_constant 0), ..., f(integral_constant N - 1)
template <int N, class F>
__device__ __forceinline__ void unroll_n(F&& f) {
  if constexpr (N > 0) {
    unroll_n<N - 1>(f);
    f(std::integral_constant<int, N - 1>{});
  }
}

template <int Q, int LPC, bool MH, int MAXW>
__global__ __launch_bounds__(MAXW * 64) void k_gibbs_free(
    const float* __restrict__ h, const float* __restrict__ Jt, int8_t* __restrict__ chains,
    int64_t N, int L, int jc, int nchunk, int m4, int slot, int cpb,
    int sweeps, uint32_t k0, uint32_t k1, uint64_t sweep_offset, float beta,
    unsigned long long* flips_out, int32_t* dev_err, const uint64_t* __restrict__ epoch,
    const int32_t* __restrict__ run, const ChainStream* __restrict__ streams,
    const int64_t* __restrict__ count) {
  if (run && *run == 0) return;  // whole grid leaves before any barrier
  // With a live count (a launch sized for N chains of which the first *count
  // are live) the workgroups take chains strided by the grid, chain
  // cb * gridDim.x + blockIdx.x, so a partly filled arena still spreads its
  // live chains over every workgroup; otherwise each takes a contiguous range.
  if (count) {
    const int64_t live = *count;
    if (live < N) N = live;
  }
  if ((count ? (int64_t)blockIdx.x : (int64_t)blockIdx.x * cpb) >= N)
    return;  // no live chain: whole workgroup, before any barrier
  if (epoch) sweep_offset += *epoch * (uint64_t)sweeps;
  constexpr int QP = gather_qp(Q), NQ = QP / 4, V = gather_v(Q), S = gather_s(Q, LPC);
  constexpr int vL = (Q - 1) / 4, eL = (Q - 1) % 4;  // lane and slot of state q-1
  typedef float fv __attribute__((ext_vector_type(4)));
  extern __shared__ __attribute__((aligned(16))) unsigned char g_smem[];
  // chains per wave: 64 / LPC (narrow chains: the last 64 % LPC lanes of a
  // wave hold no chain)
  constexpr int CPW = 64 / LPC;
  constexpr bool kNarrow = LPC < 8;
  // the last wave loads, the others hold the chains
  const int T = blockDim.x - 64, nw = T / 64, CPB = kNarrow ? nw * CPW : T / LPC;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wid = __builtin_amdgcn_readfirstlane(tid >> 6);  // wave-uniform
  const int p = kNarrow ? lane % LPC : lane & (LPC - 1), u = p / V, v = p % V;
  const bool lane_ok = !kNarrow || lane < CPW * LPC;
  const int cb = kNarrow ? wid * CPW + lane / LPC : tid / LPC;
  constexpr int nslot = 4;
  float* ring = reinterpret_cast<float*>(g_smem);                             // [nslot][slot]
  uint32_t* tokw = reinterpret_cast<uint32_t*>(ring + (size_t)nslot * slot);  // [S][m4][CPB]
  unsigned char* tokb = reinterpret_cast<unsigned char*>(tokw);
  const int64_t c =
      count ? (int64_t)cb * gridDim.x + blockIdx.x : (int64_t)blockIdx.x * cpb + cb;
  const bool has_chain = lane_ok && cb < cpb && wid < nw;
  const bool active = has_chain && (c < N);
  const bool reader = has_chain && v < NQ;
  uint32_t cid = (uint32_t)c;
  if (streams && active) {
    const ChainStream st = streams[c];
    k0 = (uint32_t)st.seed;
    k1 = (uint32_t)(st.seed >> 32);
    cid = st.chain;
    sweep_offset += st.sweep_offset;
  }
  // byte offset in the chain's token area of the token of site j (32-bit arithmetic)
  auto tok_off = [&](int j) -> uint32_t {
    const int m = j / S;
    return (uint32_t)((((j % S) * m4 + (m >> 2)) * CPB + cb) * 4 + (m & 3));
  };
  auto tok_at = [&](int j) -> unsigned char* {
    const int m = j / S;
    return tokb + ((size_t)((j % S) * m4 + (m >> 2)) * CPB + cb) * 4 + (m & 3);
  };

  // dword k = (site group, 4 positions)
  for (int k = lane_ok && wid < nw ? p : S * m4; k < S * m4; k += LPC) {
    const int uu = k / m4, mq = k % m4;
    uint32_t w = 0;
    for (int e = 0; e < 4; ++e) {
      const int j = S * (4 * mq + e) + uu;
      int t = 0;
      if (active && j < L) t = checked_token(chains[c * L + j], Q, dev_err);
      w |= (uint32_t)t << (8 * e);
    }
    tokw[k * CPB + cb] = w;
  }

  const uint32_t site_bytes = (uint32_t)((size_t)L * Q * QP * sizeof(float));
  const uint32_t chunk_bytes = (uint32_t)((size_t)jc * Q * QP * sizeof(float));
  const uint32_t slot_bytes = (uint32_t)slot * 4u, ring_bytes = (uint32_t)nslot * slot_bytes;
  const uint32_t jt_bytes = (uint32_t)L * site_bytes;  // at most 2^30
  const uint32_t last_chunk = site_bytes - (uint32_t)(nchunk - 1) * chunk_bytes;
  // counters behind the tokens: chunks consumed by each wave, and chunks
  // complete in LDS (mod 2^32, compared by their difference)
  const uint32_t done0 = lds_addr(ring) + ring_bytes + 4u * (uint32_t)(S * m4 * CPB);
  const uint32_t ready0 = done0 + 4u * kGMaxWaves;
  if (tid <= kGMaxWaves) lds_put(done0 + 4u * tid, 0u);
  __syncthreads();
  if (wid == nw) {
    // ---- the loading wave.  Chunk k of site i: bytes [k*chunk_bytes, +slot
    // bytes) of the site's run, read through a resource that ends with the run
    // (the hardware returns 0 past it), as 1 KB blocks, lane l the 16 bytes at
    // 16 l of each; four blocks share a base (a load's immediate offset moves
    // both of its addresses).  Bytes past the chunk land in the slot's padding.
    const int n = (int)gp_ceil(chunk_bytes, 1024), rem = n & 3, quads = n >> 2;
    const uint32_t done_l = done0 + 4u * min(lane, nw - 1);
    const int64_t Tn = (int64_t)sweeps * L * nchunk;
    uint32_t poff = 0, pleft = site_bytes, psl = lds_addr(ring);  // offset in Jt, bytes left of
    const uint32_t ring_end = psl + ring_bytes;                   // the run, slot
    int pk = 0;
    auto publish = [&](int64_t complete) {
      compiler_fence();
      if (lane == 0) lds_put(ready0, (uint32_t)complete);
      compiler_fence();
    };
    for (int64_t t = 0; t < Tn; ++t) {
      if (t >= nslot) {  // the slot's last chunk, t - 4, must be consumed by every wave
        while (!__all((int)(lds_dword_now(done_l) - (uint32_t)(t - nslot + 1)) >= 0)) {
        }
      }
      compiler_fence();
      const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
          (void*)(reinterpret_cast<const char*>(Jt) + poff), (short)0, (int)pleft, 0x00020000);
      uint32_t dst = psl;
      int vo = 16 * lane;
      for (int it = 0; it < rem; ++it, dst += 1024, vo += 1024)
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (lds_void_t*)(uintptr_t)dst, 16, vo, 0, 0, 0);
      for (int it = 0; it < quads; ++it, dst += 4096, vo += 4096)
        unroll_n<4>([&](auto e) {
          __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (lds_void_t*)(uintptr_t)dst, 16, vo, 0,
                                                   1024 * decltype(e)::value, 0);
        });
      psl += slot_bytes;
      if (psl == ring_end) psl -= ring_bytes;
      if (++pk < nchunk) {
        poff += chunk_bytes;
        pleft -= chunk_bytes;
      } else {
        pk = 0;
        pleft = site_bytes;
        poff += last_chunk;
        if (poff == jt_bytes) poff = 0;
      }
      if (t >= 1) {
        // Chunk t - 1 and all before it are in LDS once at most n loads are
        // out; the wait's count is an immediate, so the next lower of 32, 16
        // and 0 (a switch over every n cost 4%: the chains' waves wait here).
        if (n >= 32)
          __builtin_amdgcn_s_waitcnt(0x8f70);
        else if (n >= 16)
          __builtin_amdgcn_s_waitcnt(0x4f70);
        else
          __builtin_amdgcn_s_waitcnt(0x0f70);
        publish(t);
      }
    }
    wait_vm_lgkm0<0>();
    publish(Tn);
  }

  fv acc = (fv)(0.0f);
  float hq[4] = {};
  unsigned long long nflip = 0;
  // one Philox call gives the words of 4 consecutive sites (heat-bath draw)
  // or 2 (Metropolis); sites are drawn in order from i = 0 every sweep
  uint4 rnd = make_uint4(0u, 0u, 0u, 0u);
  // Metropolis visit state: current and proposed state, uniform, and this
  // lane's part of H_i(a') - H_i(a)
  int mh_old = 0, mh_prop = 0;
  float mh_u = 0.0f, mh_d = 0.0f;
  // tokens of the next chunk-step's first two positions of this lane, read
  // one step ahead (software pipeline), and their sites
  uint32_t mh_nsv[2] = {0u, 0u};
  int mh_nj[2] = {0, 0};
  const int jcs = jc / S;  // positions per lane per chunk (multiple of 4)
  uint32_t csl = 0;   // ring slot of the current chunk, in bytes
  uint32_t nth = 0, complete = 0;  // chunks consumed; chunks known to be in LDS
  // heat-bath draw: the four token dwords the next chunk-step's first group
  // of 16 positions starts with, read one step ahead (software pipeline).
  // In the 16-wave instantiation (128 VGPRs) only with one site group
  // (q > 16): with several, the four live registers cost more in spills than
  // the pipeline saves.
  constexpr bool kPipeTok = !MH && (S == 1 || MAXW <= kGMidWaves);
  // four token dwords of this lane's sites from dword d0 on (past the last:
  // the last again)
  const uint32_t twl =
      lds_addr(reinterpret_cast<const float*>(tokw)) + 4u * (uint32_t)(u * m4 * CPB + cb);
  const uint32_t tstep = 4u * (uint32_t)CPB;
  auto tokens = [&](auto& tk, auto n_c, int d0) {
    constexpr int n = decltype(n_c)::value;
    if (d0 + n <= m4) {
      const uint32_t a = twl + (uint32_t)d0 * tstep;
#pragma unroll
      for (int d = 0; d < n; ++d) tk[d] = lds_dword(a + d * tstep);
    } else {
#pragma unroll
      for (int d = 0; d < n; ++d) tk[d] = lds_dword(twl + (uint32_t)min(d0 + d, m4 - 1) * tstep);
    }
  };
  using four = std::integral_constant<int, 4>;
  uint32_t g_tok[4] = {0u, 0u, 0u, 0u};
  if (kPipeTok && reader) tokens(g_tok, four{}, 0);  // tokens written above by this wave
  if (MH) {  // tokens of the first chunk-step (written above by this wave)
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      mh_nj[e] = min(min(p + LPC * e, jc - 1), L - 1);
      mh_nsv[e] = (uint32_t)tokb[tok_off(mh_nj[e])];
    }
  }
  const __amdgpu_buffer_rsrc_t rh =
      __builtin_amdgcn_make_buffer_rsrc((void*)h, (short)0, L * Q * 4, 0x00020000);
  auto load_h = [&](int site) {  // values past the row are masked in the draw
    return __builtin_amdgcn_raw_buffer_load_b128(rh, (site * Q + 4 * v) * 4, 0, 0);
  };
  auto hnext = load_h(0);
  for (int sw = 0; wid < nw && sw < sweeps; ++sw)
  for (int i = 0; i < L; ++i)
  for (int k = 0; k < nchunk; ++k) {
    while ((int)(complete - nth) <= 0)
      complete = (uint32_t)__builtin_amdgcn_readfirstlane((int)lds_dword_now(ready0));
    compiler_fence();
    if (MH && k == 0) {
      // proposal and uniform of this visit; lane 0 starts the difference
      // with h_i(a') - h_i(a)
      const uint32_t sg = (uint32_t)(sweep_offset + (uint64_t)sw);
      if ((i & 1) == 0)
        rnd = philox4x32_10(make_uint4((uint32_t)i >> 1, sg, cid, 3u), k0, k1);
      const uint32_t wp = pick_word(rnd, 2 * (i & 1));
      mh_u = word_to_uniform(pick_word(rnd, 2 * (i & 1) + 1));
      mh_old = (int)*tok_at(i);
      mh_prop = (mh_old + 1 + (int)(((uint64_t)wp * (uint64_t)(Q - 1)) >> 32)) % Q;
      // h_i by scalar loads of the whole row (uniform addresses), then a lane
      // select: a per-lane vector load here would share the counter of the
      // chunk loads in flight and make the wave wait for all of them
      float hs[Q];
#pragma unroll
      for (int a = 0; a < Q; ++a) hs[a] = h[i * Q + a];
      float hp = 0.0f, ho = 0.0f;
#pragma unroll
      for (int a = 0; a < Q; ++a) {
        hp = a == mh_prop ? hs[a] : hp;
        ho = a == mh_old ? hs[a] : ho;
      }
      mh_d = p == 0 ? hp - ho : 0.0f;
    }
    if (!MH && k == 0) {
      // h_i for this lane's quad, loaded a visit ahead (a chain's wave has no
      // other vector memory operations in flight)
#pragma unroll
      for (int e = 0; e < 4; ++e) hq[e] = __uint_as_float(hnext[e]);
      hnext = load_h(i + 1 < L ? i + 1 : 0);
    }
    // ---- this lane's sites of the chunk: j = k*jc + S*r + u, r < jc/S,
    // token positions m0 + r.  The rows of j = i (zero block) and of j >= L
    // (past the end of the run, loaded as zeros) add nothing, so every
    // position is added unconditionally; positions past the last token dword
    // read any valid token.  Groups of 16 positions: 4 token loads, 16 row
    // loads, the adds (a tail group loads only its positions).
    if (MH && has_chain) {
      // Metropolis needs two entries of each row: the chain's lanes split
      // the chunk's sites (lane p: positions p, p + LPC, ...) and add
      // J_ij(a', s_j) - J_ij(a, s_j); the row of j = i is the zero block.
      // Two positions at a time, without branches: both token reads, then
      // the four entry reads.  Positions past the chunk are clamped and not
      // added; sites past the run read a valid token (clamped to L - 1) and
      // find a zero row (the slot holds zeros past the run end).
      const float* cb0 = reinterpret_cast<const float*>(g_smem + csl);
      const int j0 = k * jc;
      const int nr = (jc + LPC - 1) / LPC;  // positions per lane, uniform
      for (int r0 = 0; r0 < nr; r0 += 2) {
        uint32_t sv[2];
        int jlv[2];
        bool ok[2];
#pragma unroll
        for (int e = 0; e < 2; ++e) {
          const int jl = p + LPC * (r0 + e);
          ok[e] = jl < jc;
          jlv[e] = ok[e] ? jl : jc - 1;
          sv[e] = r0 == 0 ? mh_nsv[e] : (uint32_t)tokb[tok_off(min(j0 + jlv[e], L - 1))];
        }
#pragma unroll
        for (int e = 0; e < 2; ++e) {
          const float* row = cb0 + __umul24((uint32_t)(jlv[e] * Q) + sv[e], (uint32_t)QP);
          const float x = row[mh_prop] - row[mh_old];
          mh_d += ok[e] ? x : 0.0f;
        }
      }
    }
    if (MH) {
      // read the tokens the next chunk-step starts with (same site, next
      // chunk; or the next site's first chunk)
      const int nk = k + 1 < nchunk ? k + 1 : 0;
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        const int jl = min(p + LPC * e, jc - 1);
        mh_nj[e] = min(nk * jc + jl, L - 1);
        mh_nsv[e] = (uint32_t)tokb[tok_off(mh_nj[e])];
      }
    }
    if (!MH && reader) {
      const float* jb = reinterpret_cast<const float*>(g_smem + csl) + 4 * v;
      const int m0 = k * jcs;  // multiple of 4
      auto group = [&](int r0, bool tail) {
        // a tail with several site groups (q <= 16, long chunks) skips the
        // loads past its positions; with one (q > 16, at most 16 positions
        // lost) it loads clamped rows, the faster code at protein scale
        constexpr bool kSkip = S > 1;
        uint32_t tk[4];
        if (kPipeTok && r0 == 0) {  // read one step ahead
#pragma unroll
          for (int d = 0; d < 4; ++d) tk[d] = g_tok[d];
        } else {
          tokens(tk, four{}, (m0 + r0) >> 2);
        }
        // six row reads in flight ahead of the adds (a fixed order: left to
        // itself the compiler puts all sixteen first)
        constexpr int kAhead = 6;
        fv x[16];
        auto read_row = [&](int e) {
          const int s = (int)((tk[e >> 2] >> (8 * (e & 3))) & 0xFF);
          // row offset s * QP by a 24-bit multiply (full rate; a 32-bit
          // integer multiply issues at a quarter of the rate)
          const uint32_t so = __umul24((uint32_t)s, (uint32_t)QP);
          if (kSkip) {
            if (!tail || r0 + e < jcs)  // wave-uniform
              x[e] = *reinterpret_cast<const fv*>(jb + (S * (r0 + e) + u) * Q * QP + so);
          } else {
            const int r = tail ? min(r0 + e, jcs - 1) : r0 + e;
            x[e] = *reinterpret_cast<const fv*>(jb + (S * r + u) * Q * QP + so);
          }
        };
#pragma unroll
        for (int e = 0; e < kAhead; ++e) read_row(e);
        if (!tail) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          if (e + kAhead < 16) read_row(e + kAhead);
          if (!tail || r0 + e < jcs) acc += x[e];
          if (!tail && e + kAhead < 16) __builtin_amdgcn_sched_barrier(0);
        }
      };
      if (QP < 24 && QP != 16 && jcs % 16 != 0) {
        // Rows of 1-3 or 5 quads (q <= 12, q = 17..20) in chunks whose
        // positions per lane are not a multiple of 16: groups of a
        // compile-time length over the
        // positions of this chunk that can hold a site j < L (a multiple of
        // 4, at most jcs; the rest, past the run in a site's last chunk, are
        // zero rows, and adding +0 to a sum that started at +0 changes no
        // bit), with no clamped or skipped reads in the tail group.  Measured
        // per 10 sweeps: q = 5, L = 400: 23.2 -> 17.4 ms; q = 12, L = 200:
        // 14.5 -> 11.2; q = 17, L = 150: 15.6 -> 10.9.  Where the positions
        // are a multiple of 16 (q = 8, L = 60; q = 13, L = 130) this form was
        // 2-4% slower, so those take the group below; with both forms in the
        // kernel the compiler scheduled the common group of 16-float rows
        // (q = 13..16) worse (5% at q = 13, L = 130), and for rows of 6-8
        // quads (q = 21) the new form itself read 10-13% slower, so those
        // instantiations keep the group below alone.
        const int nv = min(jcs, (((L - k * jc + S - 1) / S) + 3) & ~3);
        auto tgroup = [&](int r1, auto n_c) {
          constexpr int n = decltype(n_c)::value;
          uint32_t tk[n / 4];
          if (kPipeTok && r1 == 0) {
#pragma unroll
            for (int d = 0; d < n / 4; ++d) tk[d] = g_tok[d];
          } else {
            tokens(tk, std::integral_constant<int, n / 4>{}, (m0 + r1) >> 2);
          }
          fv x[n];
#pragma unroll
          for (int e = 0; e < n; ++e) {
            const uint32_t so = __umul24((tk[e >> 2] >> (8 * (e & 3))) & 0xFFu, (uint32_t)QP);
            x[e] = *reinterpret_cast<const fv*>(jb + (S * (r1 + e) + u) * Q * QP + so);
          }
#pragma unroll
          for (int e = 0; e < n; ++e) acc += x[e];
        };
        int r1 = 0;
        for (; r1 + 16 <= nv; r1 += 16) tgroup(r1, std::integral_constant<int, 16>{});
        if (nv - r1 == 12)
          tgroup(r1, std::integral_constant<int, 12>{});
        else if (nv - r1 == 8)
          tgroup(r1, std::integral_constant<int, 8>{});
        else if (nv - r1 == 4)
          tgroup(r1, std::integral_constant<int, 4>{});
      } else {
        int r0 = 0;
        for (; r0 + 16 <= jcs; r0 += 16) group(r0, false);
        if (r0 < jcs) group(r0, true);
      }
      if (kPipeTok) {
        // the next chunk-step's first token dwords (same site's next chunk,
        // or the next site's first chunk)
        tokens(g_tok, four{}, k + 1 < nchunk ? (m0 + jcs) >> 2 : 0);
      }
    }

    // (a wave's LDS operations are in order: its reads come before this)
    compiler_fence();
    ++nth;
    if (lane == 0) lds_put(done0 + 4u * wid, nth);
    compiler_fence();
    if (k == nchunk - 1) {
      // ---- combine the S site groups, draw, store the token
      if constexpr (MH) {
        float d = group_fsum<8>(mh_d);  // H_i(a') - H_i(a), in every lane of the chain
        if (LPC == 16) d += dpp_f<kDppRor8>(d);
        const bool acc_mh = mh_u < expf(beta * d);
        if (acc_mh) {
          // the next step's tokens were read before this change
#pragma unroll
          for (int e = 0; e < 2; ++e)
            if (mh_nj[e] == i) mh_nsv[e] = (uint32_t)mh_prop;
        }
        if (p == 0 && has_chain && acc_mh) {
          if (active) ++nflip;
          *tok_at(i) = (unsigned char)mh_prop;
        }
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[e] = combine_sites<V, LPC>(acc[e]);
        const uint32_t sg = (uint32_t)(sweep_offset + (uint64_t)sw);
        float l[4];
        float mx = -INFINITY;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const bool ok = v < NQ && 4 * v + e < Q;
          l[e] = ok ? beta * (hq[e] + acc[e]) : -INFINITY;
          mx = fmaxf(mx, l[e]);
        }
        const int nbase = lane - p;  // first lane of the chain (narrow chains)
        if constexpr (kNarrow)
          mx = narrow_max<LPC>(mx, nbase);
        else
          mx = group_max<V>(mx);
        float P[4];
        float run_sum = 0.0f;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const bool ok = v < NQ && 4 * v + e < Q;
          run_sum += ok ? __expf(l[e] - mx) : 0.0f;
          P[e] = run_sum;
        }
        // inclusive scan of the quad sums over v; exclusive = shifted by one
        float inc, excl, Stot;
        if constexpr (kNarrow) {
          inc = narrow_scan(run_sum, lane, v);
          excl = __shfl(inc, lane - 1, kWave);
          if (v == 0) excl = 0.0f;
          Stot = __shfl(excl + P[eL], nbase + vL, kWave);  // S_{q-1}
        } else {
          inc = group_scan<V>(run_sum, v);
          excl = V > 1 ? dpp_f<kDppShr1>(inc) : 0.0f;
          if (v == 0) excl = 0.0f;
          Stot = group_bcast<V, vL>(excl + P[eL], v);  // S_{q-1}
        }
        if ((i & 3) == 0)
          rnd = philox4x32_10(make_uint4((uint32_t)i >> 2, sg, cid, 0u), k0, k1);
        const float uz = word_to_uniform(pick_word(rnd, i & 3)) * Stot;
        int cnt = 0;
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (v < NQ && 4 * v + e < Q - 1 && excl + P[e] <= uz) ++cnt;
        if constexpr (kNarrow)
          cnt = narrow_sum<LPC>(cnt, nbase);
        else
          cnt = group_sum<V>(cnt);
        // every lane of the chain drew the same state: patch the token of
        // site i in the dwords read ahead for the next site's first chunk
        if (kPipeTok && reader && u == i % S) {
          const int mi = i / S;
#pragma unroll
          for (int d = 0; d < 4; ++d)
            if (min(d, m4 - 1) == (mi >> 2))
              g_tok[d] =
                  (g_tok[d] & ~(0xFFu << (8 * (mi & 3)))) | ((uint32_t)cnt << (8 * (mi & 3)));
        }
        if (p == 0 && has_chain) {
          unsigned char* tp = tok_at(i);
          if (active && cnt != (int)*tp) ++nflip;
          *tp = (unsigned char)cnt;
        }
      }
      acc = (fv)(0.0f);
    }
    csl += slot_bytes;
    if (csl == ring_bytes) csl = 0;
  }
  __syncthreads();
  if (active)
    for (int j = p; j < L; j += LPC) chains[c * L + j] = (int8_t)*tok_at(j);
  if (flips_out) {
    unsigned long long tot = nflip;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) tot += __shfl_xor(tot, o, kWave);
    if (lane == 0 && tot) atomicAdd(flips_out, tot);
  }
}


// The loading wave comes beside the plan's waves; its counters lie behind the
// plan's LDS (kGLds leaves 256 bytes).
template <int Q, bool MH, int MAXW>
hipError_t launch_free_shape(const GatherShape& gs, const GatherArgs& a) {
  constexpr int LP = gather_lanes(Q, !MH), LN = gather_narrow_lanes(Q, !MH);
  if (gs.ahead != 3 || gs.waves + 1 > MAXW || gs.slot > 40 * 256) return hipErrorInvalidValue;
  auto kern = k_gibbs_free<Q, LP, MH, MAXW>;
  if (gs.lpc != LP) {
    if constexpr (LN > 0) {
      if (gs.lpc != LN) return hipErrorInvalidValue;
      kern = k_gibbs_free<Q, LN, MH, MAXW>;
    } else {
      return hipErrorInvalidValue;
    }
  }
  const size_t lds = gs.lds + 4 * (kGMaxWaves + 1);
  const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (e != hipSuccess) return e;
  const DevCtl& ctl = *a.ctl;
  hipLaunchKernelGGL(kern, dim3(gs.blocks), dim3((gs.waves + 1) * 64), lds, a.s, a.h, a.Jt,
                     a.chains,
                     a.N, a.L, gs.jc, gs.nchunk, gs.m4, gs.slot, gs.cpb, a.sweeps, (uint32_t)a.seed,
                     (uint32_t)(a.seed >> 32), a.sweep_offset, a.beta, a.flips_out, a.dev_err,
                     ctl.epoch, ctl.active, ctl.streams, ctl.count);
  return hipGetLastError();
}

// 12 waves leave 168 registers per lane, 16 leave 128.
template <int Q, bool MH>
hipError_t launch_free_waves(const GatherShape& gs, const GatherArgs& a) {
  if constexpr (!MH) {
    if (gs.waves + 1 <= kGMidWaves) return launch_free_shape<Q, MH, kGMidWaves>(gs, a);
  }
  return launch_free_shape<Q, MH, kGMaxWaves>(gs, a);
}

}  // namespace bmdca
