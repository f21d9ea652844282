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
//   - up to kGLoaders more waves load, each every second chunk.  One waits
//     until every wave has consumed the chunk that its slot holds, loads the
//     slot, waits for the loads and counts the chunk complete in LDS, in order;
//   - a chains' wave reads that count only when it has used up the chunks that
//     it knows to be complete, and counts the chunks it has consumed in LDS (a
//     wave's LDS operations are in order, so the count follows its reads).
//
// So waves may be up to three chunks apart and one's draw is covered by the
// others' reads.  Every wait ends: all waves of a workgroup are resident, a
// loader waits for chunks that are complete or its partner's to come, the
// others for chunks that the loaders fetch next.  h_i comes by a vector load at
// the start of the visit: without scalar loads in the loop the waits of the LDS
// reads stay exact.  Sums and draws are those of gather_kernel.hpp, so chains
// draw the same bits.
//
// What bounds it: up to 60 chains per CU a wave's own instructions, one a row
// for the address, one read, one wait and four adds (24 chains and 80 differ by
// a third); above that the LDS, whose reads of random rows conflict (8.6 cycles
// for 64 lanes where 4 would do); at L = 512 the loads.  Tried: a switch over
// every load count in the loader's wait (4% slower: the chains' waves wait
// there), polls with a sleep between (2-6%), publishing a chunk later with more
// in flight (5-15%), one loader (2-25%), three (even), twelve lanes per chain
// of two states each (-7 to +20%), one lane for both quads of a row of q = 5..8
// (+3 to +30%), reads going on over the ends of groups and chunks (+30%), four
// or eight row reads ahead instead of six (even).
// Barriers -> free, ms, 256 CUs: q = 21, L = 100, 10 sweeps, 10 000 chains 5.22
// -> 3.78; L = 256, 3 sweeps, 6000 chains 8.95 -> 5.71, 20 000 8.94 -> 7.6; L =
// 512, 1 sweep, 10 000 11.7 -> 9.1, 20 000 24.4 -> 12.3; q = 25, L = 150, 3
// sweeps, 6000 chains 8.85 -> 3.42; q = 12, L = 200, 5 sweeps, 10 000 4.37 ->
// 3.70; q = 5, L = 400, 3 sweeps, 6000 4.82 -> 3.77; Metropolis q = 21, 10
// sweeps, L = 100, 10 000 3.90 -> 3.0, L = 127, 8191 5.73 -> 4.0.
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
// a wave-uniform value, kept in a scalar register
__device__ __forceinline__ uint32_t scalar(uint32_t x) {
  return (uint32_t)__builtin_amdgcn_readfirstlane((int)x);
}
// f(integral_constant 0), ..., f(integral_constant N - 1)
template <int N, class F>
__device__ __forceinline__ void unroll_n(F&& f) {
  if constexpr (N > 0) {
    unroll_n<N - 1>(f);
    f(std::integral_constant<int, N - 1>{});
  }
}

// Metropolis of q <= 8 runs two workgroups per CU where the chains take several
// rounds (at most 60 chains and 15 to 16 waves each), if its registers allow 8
// waves a SIMD: q = 4 and 8 took a few more than the 64 by themselves (q = 4, L =
// 120, 25 000 chains, 3 sweeps 1.56 -> 1.32 ms; bound to 64, q = 5 would take 6%
// longer).
constexpr int free_simd_waves(int Q, bool mh) { return mh && (Q == 4 || Q == 8) ? 8 : 4; }

template <int Q, int LPC, bool MH, bool TQ>
__global__ __launch_bounds__(kGMaxWaves * 64, free_simd_waves(Q, MH)) void k_gibbs_free(
    const float* __restrict__ h, const float* __restrict__ Jt, int8_t* __restrict__ chains,
    int64_t N, int L, int jc, int nchunk, int m4, int slot, int cpb, int nw,
    int sweeps, uint32_t k0, uint32_t k1, uint64_t sweep_offset, float beta,
    unsigned long long* flips_out, int32_t* dev_err, const uint64_t* __restrict__ epoch,
    const int32_t* __restrict__ run, const ChainStream* __restrict__ streams,
    const int64_t* __restrict__ count) {
  if (run && *run == 0) return;  // whole grid leaves before any barrier
  // With a live count (a launch sized for N chains of which the first *count
  // are live) the workgroups take chains strided by the grid, chain
  // cb * nblk + blk, so a partly filled arena still spreads its live chains over
  // every workgroup; otherwise each takes a contiguous range.
  const uint32_t nblk = gridDim.x * gridDim.y, blk = blockIdx.y * gridDim.x + blockIdx.x;
  if (count) {
    const int64_t live = *count;
    if (live < N) N = live;
  }
  if ((count ? (int64_t)blk : (int64_t)blk * cpb) >= N)
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
  // the last waves load, the others hold the chains
  const int CPB = nw * CPW, loaders = (int)blockDim.x / 64 - nw;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wid = __builtin_amdgcn_readfirstlane(tid >> 6);  // wave-uniform
  // lanes without a chain (the last 64 % LPC of narrow chains) go along with
  // the last one that has one, lanes past the row's quads (v >= NQ) with the
  // last quad: their reads cost nothing and no lane mask is set in the loop
  const bool lane_ok = !kNarrow || lane < CPW * LPC;
  const int gl = kNarrow ? min(lane, CPW * LPC - 1) : lane;
  const int p = gl % LPC, u = p / V, v = p % V;
  const int cb = wid * CPW + gl / LPC;
  constexpr int nslot = 4;
  float* ring = reinterpret_cast<float*>(g_smem);                             // [nslot][slot]
  uint32_t* tokw = reinterpret_cast<uint32_t*>(ring + (size_t)nslot * slot);
  unsigned char* tokb = reinterpret_cast<unsigned char*>(tokw);
  const int64_t c = count ? (int64_t)cb * nblk + blk : (int64_t)blk * cpb + cb;
  const bool has_chain = lane_ok && cb < cpb && wid < nw;
  const bool active = has_chain && (c < N);
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
    if (TQ) return (uint32_t)((((j % S) * (m4 / 4) + (m >> 4)) * CPB + cb) * 16 + (m & 15));
    if (MH) return (uint32_t)((((j % S) * m4 + (m >> 2)) * CPB + cb) * 4 + (m & 3));
    return (uint32_t)(((j % S) * CPB + cb) * m4 * 4 + m);
  };
  auto tok_at = [&](int j) -> unsigned char* { return tokb + tok_off(j); };

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
    tokw[TQ   ? ((uu * (m4 / 4) + (mq >> 2)) * CPB + cb) * 4 + (mq & 3)
         : MH ? k * CPB + cb
              : (uu * CPB + cb) * m4 + mq] = w;
  }

  const uint32_t site_bytes = (uint32_t)((size_t)L * Q * QP * sizeof(float));
  const uint32_t chunk_bytes = (uint32_t)((size_t)jc * Q * QP * sizeof(float));
  const uint32_t slot_bytes = (uint32_t)slot * 4u, ring_bytes = (uint32_t)nslot * slot_bytes;
  // counters behind the tokens: chunks consumed by each wave, and chunks
  // complete in LDS (mod 2^32, compared by their difference)
  const uint32_t done0 = lds_addr(ring) + ring_bytes + 4u * (uint32_t)(S * m4 * CPB);
  const uint32_t ready0 = done0 + 4u * kGMaxWaves;
  if (tid <= kGMaxWaves) lds_put(done0 + 4u * tid, 0u);
  __syncthreads();
  if (wid >= nw) {
    // ---- a loading wave: chunks t = wid - nw, then every loaders-th.  Chunk
    // k of site i: bytes [k*chunk_bytes, +slot bytes) of the site's run, read
    // through a resource that ends with the run (the hardware returns 0 past
    // it), as 1 KB blocks, lane l the 16 bytes at 16 l of each; four blocks
    // share a base (a load's immediate offset moves both of its addresses).
    // Bytes past the chunk land in the slot's padding.
    const int n = (int)gp_ceil(chunk_bytes, 1024), rem = n & 3, quads = n >> 2;
    const uint32_t done_l = done0 + 4u * min(lane, nw - 1);
    const int64_t Tn = (int64_t)sweeps * L * nchunk;
    auto publish = [&](uint32_t chunks) {
      compiler_fence();
      if (lane == 0) lds_put(ready0, chunks);
      compiler_fence();
    };
    int pi = 0, pk = wid - nw;  // site and chunk
    for (int64_t t = wid - nw; t < Tn; t += loaders, pk += loaders) {
      while (pk >= nchunk) {
        pk -= nchunk;
        if (++pi == L) pi = 0;
      }
      const uint32_t off = (uint32_t)pk * chunk_bytes;
      const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
          (void*)(reinterpret_cast<const char*>(Jt) + (uint32_t)pi * site_bytes + off), (short)0,
          (int)(site_bytes - off), 0x00020000);
      uint32_t dst = lds_addr(ring) + (uint32_t)(t & (nslot - 1)) * slot_bytes;
      int vo = 16 * lane;
      if (t >= nslot) {  // the slot's last chunk, t - 4, must be consumed by every wave
        while (!__all((int)(lds_dword_now(done_l) - (uint32_t)(t - nslot + 1)) >= 0)) {
        }
      }
      compiler_fence();
      for (int it = 0; it < rem; ++it, dst += 1024, vo += 1024)
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (lds_void_t*)(uintptr_t)dst, 16, vo, 0, 0, 0);
      for (int it = 0; it < quads; ++it, dst += 4096, vo += 4096)
        unroll_n<4>([&](auto e) {
          __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (lds_void_t*)(uintptr_t)dst, 16, vo, 0,
                                                   1024 * decltype(e)::value, 0);
        });
      if (loaders > 1) {
        wait_vm_lgkm0<0>();  // chunk t is in LDS; the count moves in order
        while (scalar(lds_dword_now(ready0)) != (uint32_t)t) {
        }
        publish((uint32_t)t + 1u);
      } else {
        // alone: chunk t - 1 is in LDS once at most n loads are out (the
        // count is an immediate, so the next lower of 32, 16 and 0)
        if (n >= 32)
          wait_vm_lgkm0<32>();
        else if (n >= 16)
          wait_vm_lgkm0<16>();
        else
          wait_vm_lgkm0<0>();
        publish((uint32_t)t);
      }
    }
    if (loaders == 1) {
      wait_vm_lgkm0<0>();
      publish((uint32_t)Tn);
    }
  }

  fv acc = (fv)(0.0f);
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
  // positions of a site's last chunk that can hold a site j < L (a multiple
  // of 4; the rest are zero rows, and adding +0 to a sum that started at +0
  // changes no bit)
  const int jcl = min(jcs, (((L - (nchunk - 1) * jc + S - 1) / S) + 3) & ~3);
  uint32_t csl = 0;                // ring slot of the current chunk, in bytes
  uint32_t nth = 0, complete = 0;  // chunks consumed; chunks known to be in LDS
  // heat-bath draw: the token dwords the next chunk-step's first group of 16
  // positions starts with, read one step ahead (past the last: the last again)
  typedef uint32_t u4 __attribute__((ext_vector_type(4)));
  const uint32_t twl = lds_addr(reinterpret_cast<const float*>(tokw)) +
                       (TQ ? 16u * (uint32_t)(u * (m4 / 4) * CPB + cb)
                           : 4u * (uint32_t)((u * CPB + cb) * m4));
  auto tokens = [&](int d0) -> u4 {
    if constexpr (TQ) {
      return *(__attribute__((address_space(3))) const u4*)(uintptr_t)(
          twl + (uint32_t)(d0 * CPB * 4));
    } else {
      const uint32_t a = twl + 4u * (uint32_t)d0;
      return u4{lds_dword(a), lds_dword(a + 4), lds_dword(a + 8), lds_dword(a + 12)};
    }
  };
  u4 g_tok = {0u, 0u, 0u, 0u};
  if (!MH && wid < nw) g_tok = tokens(0);  // tokens written above by this wave
  if (MH && wid < nw) {  // tokens of the first chunk-step (written above by this wave)
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      mh_nj[e] = min(min(p + LPC * e, jc - 1), L - 1);
      mh_nsv[e] = (uint32_t)tokb[tok_off(mh_nj[e])];
    }
  }
  // Adds the rows of n positions whose tokens are in tk, the first at LDS
  // address a.  Six reads are in flight ahead of the adds, in a fixed order:
  // left to itself the compiler puts all sixteen first.  Token byte times row
  // length plus base is one dot product with a constant that has the row length
  // (at most 128 bytes) in that byte.
  auto rows = [&](auto n_c, u4 tk, uint32_t a) {
    constexpr int n = decltype(n_c)::value, kAhead = n < 6 ? n : 6;
    fv x[n];
    auto read_row = [&](int e) {
      const uint32_t at = __builtin_amdgcn_udot4(tk[e >> 2], (4u * QP) << (8 * (e & 3)), a, false);
      x[e] = *(__attribute__((address_space(3))) const fv*)(uintptr_t)(
          at + (uint32_t)(S * e * Q * QP * 4));
    };
#pragma unroll
    for (int e = 0; e < kAhead; ++e) read_row(e);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int e = 0; e < n; ++e) {
      if (e + kAhead < n) read_row(e + kAhead);
      acc += x[e];
      if (e + kAhead < n) __builtin_amdgcn_sched_barrier(0);
    }
  };
  const uint32_t row0 =
      lds_addr(ring) + 16u * (uint32_t)min(v, NQ - 1) + (uint32_t)(u * Q * QP * 4);
  const __amdgpu_buffer_rsrc_t rh =
      __builtin_amdgcn_make_buffer_rsrc((void*)h, (short)0, L * Q * 4, 0x00020000);
  auto load_h = [&](int site) {  // values past the row are masked in the draw
    return __builtin_amdgcn_raw_buffer_load_b128(rh, (site * Q + 4 * v) * 4, 0, 0);
  };
  auto hq = load_h(0);
  constexpr int kRowRegs = MH ? (Q + LPC - 1) / LPC : 0;
  uint32_t mh_h[kRowRegs + 1];
  auto load_row = [&](int site) {  // lane p the states p, p + LPC, ... (past the end: 0)
#pragma unroll
    for (int e = 0; e < kRowRegs; ++e)
      mh_h[e] = __builtin_amdgcn_raw_buffer_load_b32(rh, (site * Q + p + LPC * e) * 4, 0, 0);
  };
  if (MH) load_row(0);
  for (int sw = 0; wid < nw && sw < sweeps; ++sw) {
    for (int i = 0; i < L; ++i) {
      if (MH) {
        // proposal and uniform of this visit; lane 0 starts the difference
        // with h_i(a') - h_i(a)
        const uint32_t sg = (uint32_t)(sweep_offset + (uint64_t)sw);
        if ((i & 1) == 0)
          rnd = philox4x32_10(make_uint4((uint32_t)i >> 1, sg, cid, 3u), k0, k1);
        const uint32_t wp = pick_word(rnd, 2 * (i & 1));
        mh_u = word_to_uniform(pick_word(rnd, 2 * (i & 1) + 1));
        mh_old = (int)*tok_at(i);
        mh_prop = (mh_old + 1 + (int)(((uint64_t)wp * (uint64_t)(Q - 1)) >> 32)) % Q;
        // the chain's lanes hold h_i, loaded a visit ahead
        float hp = 0.0f, ho = 0.0f;
#pragma unroll
        for (int e = 0; e < kRowRegs; ++e) {
          const float x = __uint_as_float(mh_h[e]);
          const float xp = __shfl(x, (lane & ~(LPC - 1)) + (mh_prop & (LPC - 1)), kWave);
          const float xo = __shfl(x, (lane & ~(LPC - 1)) + (mh_old & (LPC - 1)), kWave);
          hp = mh_prop / LPC == e ? xp : hp;
          ho = mh_old / LPC == e ? xo : ho;
        }
        mh_d = p == 0 ? hp - ho : 0.0f;
        load_row(i + 1 < L ? i + 1 : 0);
      }
      // h_i for this lane's quad, used at the draw
      if (!MH) hq = load_h(i);
      // ---- the chunks of site i.  This lane's sites of chunk k: j = k*jc + S*r
      // + u, r < jc/S.  The row of j = i is the zero block: every position is
      // added unconditionally.
      for (int k = 0; k < nchunk; ++k) {
        while ((int)(complete - nth) <= 0)
          complete = scalar(lds_dword_now(ready0));
        compiler_fence();
        if (MH) {
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
        if (!MH) {
          const int nv = k + 1 < nchunk ? jcs : jcl;  // multiple of 4
          const uint32_t a0 = row0 + csl;
          int r = 0;
          u4 tk = g_tok;
          for (; r + 16 <= nv; r += 16) {
            if (r > 0) tk = tokens((k * jcs + r) >> 2);
            rows(std::integral_constant<int, 16>{}, tk, a0 + (uint32_t)(r * (S * Q * QP * 4)));
          }
          if (r < nv) {
            if (r > 0) tk = tokens((k * jcs + r) >> 2);
            const uint32_t a = a0 + (uint32_t)(r * (S * Q * QP * 4));
            if (nv - r == 12)
              rows(std::integral_constant<int, 12>{}, tk, a);
            else if (nv - r == 8)
              rows(std::integral_constant<int, 8>{}, tk, a);
            else
              rows(std::integral_constant<int, 4>{}, tk, a);
          }
          // the next chunk-step's first token dwords (same site's next chunk, or
          // the next site's first chunk)
          g_tok = tokens(k + 1 < nchunk ? ((k + 1) * jcs) >> 2 : 0);
        }

        // (a wave's LDS operations are in order: its reads come before this)
        compiler_fence();
        nth = MH ? nth + 1 : scalar(nth + 1);
        if (lane == 0) lds_put(done0 + 4u * wid, nth);
        compiler_fence();
        csl += slot_bytes;
        if (csl == ring_bytes) csl = 0;
        if (!MH) csl = scalar(csl);  // (MH: its addresses come out longer that way)
      }
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
          l[e] = ok ? beta * (__uint_as_float(hq[e]) + acc[e]) : -INFINITY;
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
        if (u == i % S) {
          const int mi = i / S;
#pragma unroll
          for (int d = 0; d < 4; ++d)
            if (d == (mi >> 2))
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

template <int Q, bool MH>
hipError_t launch_free_shape(const GatherShape& gs, const GatherArgs& a) {
  constexpr int LP = gather_lanes(Q, !MH), LN = gather_narrow_lanes(Q, !MH);
  if (gs.ahead != 3 || gs.waves >= kGMaxWaves) return hipErrorInvalidValue;
  const FreeShape fs = free_shape(gs, Q, MH);
  auto pick = [&](auto lanes) {
    constexpr int LL = decltype(lanes)::value;
    if constexpr (!MH) {
      if (fs.tq) return k_gibbs_free<Q, LL, MH, true>;
    }
    return k_gibbs_free<Q, LL, MH, false>;
  };
  auto kern = pick(std::integral_constant<int, LP>{});
  if (gs.lpc != LP) {
    if constexpr (LN > 0) {
      if (gs.lpc != LN) return hipErrorInvalidValue;
      kern = pick(std::integral_constant<int, LN>{});
    } else {
      return hipErrorInvalidValue;
    }
  }
  const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)fs.lds);
  if (e != hipSuccess) return e;
  const DevCtl& ctl = *a.ctl;
  // 2^21 workgroups a row of the grid (a dimension holds fewer than 2^32
  // work-items, and the loading waves are work-items too)
  const unsigned gx = std::min(gs.blocks, 1u << 21);
  const dim3 grid(gx, (unsigned)gp_ceil(gs.blocks, gx));
  hipLaunchKernelGGL(kern, grid, dim3(fs.waves * 64), fs.lds, a.s, a.h, a.Jt, a.chains, a.N,
                     a.L, gs.jc, gs.nchunk, fs.m4, gs.slot, gs.cpb, fs.nw, a.sweeps,
                     (uint32_t)a.seed, (uint32_t)(a.seed >> 32), a.sweep_offset, a.beta, a.flips_out, a.dev_err,
                     ctl.epoch, ctl.active, ctl.streams, ctl.count);
  return hipGetLastError();
}

}  // namespace bmdca
