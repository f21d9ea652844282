// Importance weights of Eq. (7) (adabmDCA 2.0, Sec. 2.3, step p.2):
// N^(m) = #{n : identical positions of rows m and n >= T}, w = 1 / N^(m).
//
// Exact counts by bit slices: the token at every position is split into P =
// ceil(log2 q) bit planes of ceil(L/32) 32-bit words per row.  Two rows differ
// at a position iff some plane differs there, so
//   mismatches = sum_w popcount(OR_p (plane_p[m][w] XOR plane_p[n][w]))
// and identical positions = L - mismatches (padding bits are 0 in both rows).
// That is P + 1 operations per pair and word on the vector units; almost all
// pairs of an alignment are far from similar, though, and a bound shows it:
// the matrix cores compare a short code of every row first (k_count_similar),
// and only the pairs that the code leaves open are compared by planes.  Each
// unordered pair is looked at once and counted for both rows.  Counts are
// exact integers.
#include "common.hpp"
#include "internal.hpp"

#include <type_traits>

namespace bmdca {

constexpr int kRwThreads = 256;
constexpr int kMaxPlanes = 5;  // q <= 32
constexpr int kRwTile = 256;   // rows and columns of a tile of pairs
// Truth table of (a ^ b) | c for v_bitop3_b32(a, b, c): bit (4a + 2b + c).
#ifndef BMDCA_XOR_OR_TABLE
#define BMDCA_XOR_OR_TABLE 0xBE
#endif
constexpr unsigned kXorOr = BMDCA_XOR_OR_TABLE;

static int planes_for(int q) {
  int p = 0;
  while ((1 << p) < q) ++p;
  return std::max(p, 1);
}

// Code of a row: +-1 per position and dimension, 4-bit floats (e2m1: 0x2 = 1,
// 0xA = -1, 0 past L), 32 positions per 16-byte unit.
//   one dimension:    bit 0 of the token; the dot product of two codes is
//                     L - 2 d, d positions with another bit 0;
//   three dimensions: bits 0 and 1 and their XOR; 3 L - 4 d, d positions with
//                     another pair of bits.
// Either way d <= mismatches.  For unrelated rows d is about 1/2 (one
// dimension) or 3/4 (three) of the mismatches; short rows take three, where
// the margin of one would be a few standard deviations.
constexpr int rw_dims(int W) { return W <= 4 ? 3 : 1; }
constexpr int rw_units(int W) { return (rw_dims(W) * W + 1) / 2 * 2; }  // whole 64-element steps

ReweightPlan plan_reweight(int64_t M, int L, int q) {
  ReweightPlan r{};
  r.planes = planes_for(q);
  r.words = (int)ceil_div(L, 32);
  r.Mpad = ceil_div(M, kRwTile) * kRwTile;
  size_t o = 0;
  r.off_planes = o;
  o = align256(o + sizeof(uint32_t) * (size_t)r.Mpad * kMaxPlanes * r.words);
  r.off_codes = o;
  o = align256(o + 16 * (size_t)rw_units(r.words) * r.Mpad);
  r.off_red = o;
  o = align256(o + sizeof(double) * kRwRed);
  r.total = o;
  return r;
}

// 32 bits -> 16 bytes of +-1 codes, the first `live` of them (0 after that).
__device__ __forceinline__ uint4 code_unit(uint32_t bits, int live) {
  uint32_t w[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    uint32_t x = (bits >> (8 * k)) & 0xFFu;  // spread 8 bits to bit 3 of 8 nibbles
    x = (x | (x << 12)) & 0x000F000Fu;
    x = (x | (x << 6)) & 0x03030303u;
    x = (x | (x << 3)) & 0x11111111u;
    x = (x << 3) | 0x22222222u;
    const int n = min(max(live - 8 * k, 0), 8);
    w[k] = n == 8 ? x : x & ((1u << (4 * n)) - 1u);
  }
  return make_uint4(w[0], w[1], w[2], w[3]);
}

// planes[m][p][w]: bit t of word w = bit p of the token at position 32w + t;
// codes[unit][m]: the row's code, dimension by dimension (unit = dim * W + w;
// an odd last unit and the rows past M are zero).  n_sim[m] = 1 (the row
// itself).
__global__ void k_encode_rows(const int8_t* __restrict__ msa, int64_t M, int64_t Mpad, int L, int q,
                              int P, int W, uint32_t* __restrict__ planes,
                              uint4* __restrict__ codes, int32_t* __restrict__ n_sim,
                              int32_t* dev_err) {
  const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t m = idx / W;
  const int w = (int)(idx % W);
  if (m >= Mpad) return;
  uint32_t bits[kMaxPlanes] = {0, 0, 0, 0, 0};
  const int live = m < M ? min(32, L - 32 * w) : 0;
  const int8_t* src = msa + m * L + 32 * w;
  auto put = [&](int t, int8_t x) {
    const int tok = checked_token(x, q, dev_err);
#pragma unroll
    for (int p = 0; p < kMaxPlanes; ++p) bits[p] |= (uint32_t)((tok >> p) & 1) << t;
  };
  if (live == 32) {
    int8_t x[32];
    __builtin_memcpy(x, src, 32);
#pragma unroll
    for (int t = 0; t < 32; ++t) put(t, x[t]);
  } else {
    for (int t = 0; t < live; ++t) put(t, src[t]);
  }
  if (m < M)
    for (int p = 0; p < P; ++p) planes[((size_t)m * kMaxPlanes + p) * W + w] = bits[p];
  const int dims = rw_dims(W);
  codes[(size_t)w * Mpad + m] = code_unit(bits[0], live);
  if (dims == 3) {
    codes[(size_t)(W + w) * Mpad + m] = code_unit(bits[1], live);
    codes[(size_t)(2 * W + w) * Mpad + m] = code_unit(bits[0] ^ bits[1], live);
  }
  if (w == 0) {
    if (rw_units(W) != dims * W) codes[(size_t)(dims * W) * Mpad + m] = make_uint4(0, 0, 0, 0);
    if (m < M) n_sim[m] = 1;
  }
}

// Pair counts over unordered pairs m < n, in tiles of 256 x 256 pairs on or
// above the diagonal.  A work item is a run of `chunk` tiles of the block-rows
// p and S - 1 - p (S + 1 tiles between them, so every run is as long).
//
// A tile first goes through the matrix cores: a wave holds the codes of 64
// rows, the tile's 256 columns are staged in LDS (units of 16 bytes column by
// column: 512-byte runs per half wave), and 32x32x64 products of 4-bit floats
// (exact integers in FP32) give the dot products.  Pairs with a dot product of
// at least `thr`, mismatches possibly <= maxmis, are appended to a list in
// LDS, compared by planes one per lane when the list is half full and at the
// end of the run.  A tile with more open pairs than the list holds (a tight
// family) is compared by planes as a whole, and so are the run's later tiles;
// `filter` = 0 (thresholds so low that the bound says nothing) does that from
// the start.
//
// Measured, M = 100 000, L = 256, q = 21: 0.45 ms (7.87 ms when every pair was
// compared by planes, 52 vector operations each).  The products alone take
// 0.25 ms (4 x 32 cycles per 1024 pairs; with more column blocks per tile the
// time grows by that); the rest is the maxima (17 operations per 1024
// products), staging and barriers, which two or three workgroups per CU
// overlap (with two buffers fewer fit a CU: 12-60% longer by L).
//
// Tiles compared by planes are bound by the vector operations, P + 1 a word.
// What kept them from it, M = 100 000 rows of one close family, L = 100, q = 21,
// ms: 7.65 with the rows loaded and counted tile by tile, 64 columns at a time
// and a 64-bit compare a pair; 4.35 with rows and counts kept over a run, 256
// columns, the next one read ahead and 32 bits; 4.15 with four rows a thread
// where their planes leave room (L = 30 1.18 -> 1.06), 3.57 with a third
// workgroup on the CU.  (Every pair by planes, without the matrix cores: 3.68.)
typedef __attribute__((address_space(3))) void rw_lds_t;
typedef int rw_i4 __attribute__((ext_vector_type(4)));
typedef int rw_i8 __attribute__((ext_vector_type(8)));
typedef float rw_f16 __attribute__((ext_vector_type(16)));

template <int P, int W>
__global__ __launch_bounds__(kRwThreads, 2) void k_count_similar(
    const uint32_t* __restrict__ planes, const uint4* __restrict__ codes, int64_t Mpad, int64_t M,
    int maxmis, float thr, int filter, int chunk, int32_t* __restrict__ n_sim) {
  constexpr int U = rw_units(W), UC = U / 2;
  // rows per thread of the plane compare: what its registers hold
  constexpr int R = P * W <= 20 ? 4 : P * W <= 40 ? 2 : 1;
  constexpr int kCodes = U * kRwTile * 16;  // a tile's column codes
  // columns it stages at a time, each with its counts by the 4 / R waves of other
  // rows: as many as fit where the codes were
  constexpr int kColBytes = P * W * 4 + 4 / R * 4;
  constexpr int kCols = kRwTile * kColBytes <= kCodes ? kRwTile : kRwTile / 2;
  static_assert(kCols * kColBytes <= kCodes, "the plane compare's columns");
  __shared__ __attribute__((aligned(16))) unsigned char buf[kCodes];
  // The list, 2% of a tile's pairs: the row in its block-row; the column after the
  // first of the tile `base` or, in the second block-row (kSecond), after its first
  // from there on.  Four bytes a pair; at W = 4, the longest code, three, so that
  // three workgroups fit a CU there too.
  constexpr int kList = 1504, kSecond = 0x8000, kListTiles = kSecond / kRwTile;
  constexpr bool kThree = W == 4;
  __shared__ uint32_t list[kThree ? 1 : kList];
  __shared__ uint8_t list_row[kThree ? kList : 1];
  __shared__ uint16_t list_col[kThree ? kList : 1];
  __shared__ int nlist;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wid = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int S = (int)(Mpad / kRwTile);
  const int nch = (S + 1 + chunk - 1) / chunk;
  const int p0 = (int)(blockIdx.x / (unsigned)nch);
  const int c0 = (int)(blockIdx.x % (unsigned)nch) * chunk, c1 = min(c0 + chunk, S + 1);
  if (tid == 0) nlist = 0;

  // mismatches of rows m and n by planes
  auto mismatches = [&](int64_t m, int64_t n) {
    const uint32_t* a = planes + (size_t)m * kMaxPlanes * W;
    const uint32_t* b = planes + (size_t)n * kMaxPlanes * W;
    int mis = 0;
#pragma unroll 4
    for (int w = 0; w < W; ++w) {
      uint32_t d = a[w] ^ b[w];
#pragma unroll
      for (int p = 1; p < P; ++p) d |= a[p * W + w] ^ b[p * W + w];
      mis += __popc(d);
    }
    return mis;
  };
  // tile s of the run: block-row and block-column; false past the run's last
  auto tile = [&](int s, int& rb, int& st) {
    rb = p0;
    st = p0 + s;
    if (st < S) return s < c1;
    rb = S - 1 - p0;
    st = rb + s - (S - p0);
    return s < c1 && rb != p0;  // the middle block-row of an odd S has no partner
  };
  // the list's pairs, one per lane (all threads; the list is complete)
  int base = c0;
  // first listed column of the first and the second block-row
  auto first_col = [&](bool second) -> int64_t {
    const int st = second ? S - 1 - p0 + max(base - (S - p0), 0) : p0 + base;
    return (int64_t)st * kRwTile;
  };
  auto flush = [&]() {
    const int n = nlist;
    const int64_t f0 = first_col(false), f1 = first_col(true);
    for (int e = tid; e < n; e += kRwThreads) {
      const int c = kThree ? list_col[e] : list[e] & 0xFFFF;
      const int r = kThree ? list_row[e] : list[e] >> 16;
      const int64_t m = (c & kSecond ? (int64_t)(S - 1 - p0) * kRwTile : (int64_t)p0 * kRwTile) + r;
      const int64_t k = (c & kSecond ? f1 - kSecond : f0) + c;
      if (mismatches(m, k) <= maxmis) {
        atomicAdd(n_sim + m, 1);
        atomicAdd(n_sim + k, 1);
      }
    }
    __syncthreads();
    if (tid == 0) nlist = 0;
    __syncthreads();
  };
  // Every pair of the run's tiles from s on, by planes: R rows per thread in
  // registers, loaded once per block-row; kCols columns at a time in LDS
  // (broadcast reads; short ones are on their way while the column before is
  // compared), an R-th of them per wave.  Rows are counted in registers, a wave's
  // columns one per lane.  (A row past M has no column after it.)
  auto by_planes = [&](int s) {
    constexpr int PW = P * W, kWaveCols = kCols / R;  // columns per wave
    uint32_t* sh = reinterpret_cast<uint32_t*>(buf);
    int* colcnt = reinterpret_cast<int*>(sh + kCols * PW);
    // rows r0 + kStep r of the tile, columns c0w .. of the staged ones
    constexpr int kStep = kRwTile / R, kParts = 4 / R;
    const int r0 = tid & (kStep - 1);
    const int part = wid & (kParts - 1), c0w = wid / kParts * kWaveCols;
    int rb, st;
    bool more = tile(s, rb, st);
    while (more) {
      const int row = rb;
      const int64_t m0 = (int64_t)rb * kRwTile;
      uint32_t mine[R][PW];
      int count[R];
#pragma unroll
      for (int r = 0; r < R; ++r) {
        const int64_t m = m0 + r0 + kStep * r;
        count[r] = 0;
#pragma unroll
        for (int k = 0; k < PW; ++k)
          mine[r][k] = m < M ? planes[(size_t)m * kMaxPlanes * W + k] : 0u;
      }
      for (; more && rb == row; more = tile(++s, rb, st)) {
        const int64_t n0 = (int64_t)st * kRwTile;
        for (int b = 0; b < kRwTile; b += kCols) {
          const int nload = (int)std::min<int64_t>(kCols, M - (n0 + b));
          if (nload <= 0) break;  // uniform
          __syncthreads();
          for (int k = tid; k < nload * PW; k += kRwThreads) {
            const int nl = k / PW, pw = k % PW;
            sh[k] = planes[(size_t)(n0 + b + nl) * kMaxPlanes * W + pw];
          }
          __syncthreads();
          // DIAG: the tile of the rows themselves, columns after the row only
          auto compare = [&](auto diag) {
            constexpr bool DIAG = decltype(diag)::value;
            for (int g = c0w; g < c0w + kWaveCols; g += 64) {  // a column per lane
              const int g1 = min(min(g + 64, c0w + kWaveCols), nload);
              int mycol = 0;
              auto column = [&](const uint32_t(&o)[PW], int nl) {
                int wc = 0;
#pragma unroll
                for (int r = 0; r < R; ++r) {
                  int mism = 0;
#pragma unroll
                  for (int w = 0; w < W; ++w) {
                    // d = OR_p (mine_p ^ other_p), one three-input bit operation per plane
                    uint32_t d = mine[r][w] ^ o[w];
#pragma unroll
                    for (int p = 1; p < P; ++p)
                      d = __builtin_amdgcn_bitop3_b32(mine[r][p * W + w], o[p * W + w], d, kXorOr);
                    mism += __popc(d);
                  }
                  const bool sim = mism <= maxmis && (!DIAG || r0 + kStep * r < b + nl);
                  count[r] += sim ? 1 : 0;
                  wc += __popcll(__ballot(sim));
                }
                mycol = lane == nl - g ? wc : mycol;
              };
              auto read = [&](uint32_t(&o)[PW], int nl) {  // past the last: the last again
                const uint32_t* src = sh + min(nl, g1 - 1) * PW;
#pragma unroll
                for (int k = 0; k < PW; ++k) o[k] = src[k];
              };
              if (g < g1) {
                if constexpr (PW <= 20) {
                  uint32_t x[PW], y[PW];
                  read(x, g);
                  int nl = g;
                  for (; nl + 2 <= g1; nl += 2) {
                    read(y, nl + 1);
                    column(x, nl);
                    read(x, nl + 2);
                    column(y, nl + 1);
                  }
                  if (nl < g1) column(x, nl);
                } else {
                  for (int nl = g; nl < g1; ++nl) {
                    uint32_t x[PW];
                    read(x, nl);
                    column(x, nl);
                  }
                }
              }
              if (g + lane < c0w + kWaveCols) colcnt[part * kCols + g + lane] = mycol;
            }
          };
          if (st == row)
            compare(std::true_type{});
          else
            compare(std::false_type{});
          __syncthreads();
          if (tid < nload) {
            int c = 0;
#pragma unroll
            for (int k = 0; k < kParts; ++k) c += colcnt[k * kCols + tid];
            if (c > 0) atomicAdd(n_sim + n0 + b + tid, c);
          }
        }
      }
#pragma unroll
      for (int r = 0; r < R; ++r)
        if (count[r] > 0) atomicAdd(n_sim + m0 + r0 + kStep * r, count[r]);
    }
  };
  rw_i4 a[2][UC];
  // block-column st's codes into LDS by direct loads
  auto fetch = [&](int st) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
          (void*)(codes + (size_t)u * Mpad + (int64_t)st * kRwTile + 64 * wid), (short)0, 1024,
          0x00020000);
      __builtin_amdgcn_raw_ptr_buffer_load_lds(
          rs, (rw_lds_t*)(buf + 16 * (u * kRwTile + 64 * wid)), 16, 16 * lane, 0, 0, 0);
    }
  };
  // columns 32 cb .. of the staged tile; their products with the wave's rows
  auto columns = [&](rw_i4(&b)[UC], int cb) {
#pragma unroll
    for (int kc = 0; kc < UC; ++kc)
      b[kc] = *reinterpret_cast<const rw_i4*>(
          buf + 16 * ((2 * kc + (lane >> 5)) * kRwTile + 32 * cb + (lane & 31)));
  };
  auto products = [&](const rw_i4(&b)[UC], rw_f16(&acc)[2]) {
#pragma unroll
    for (int k = 0; k < 2; ++k)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[k][v] = 0.0f;
#pragma unroll
    for (int kc = 0; kc < UC; ++kc) {
      const rw_i8 b8 = {b[kc][0], b[kc][1], b[kc][2], b[kc][3], 0, 0, 0, 0};
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        const rw_i8 a8 = {a[k][kc][0], a[k][kc][1], a[k][kc][2], a[k][kc][3], 0, 0, 0, 0};
        // formats 4 = e2m1; scales 2^0
        acc[k] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a8, b8, acc[k], 4, 4, 0,
                                                                 0x7F7F7F7F, 0, 0x7F7F7F7F);
      }
    }
  };
  // any pair of the wave's that thr leaves open and the list may have room for (a
  // tile with more will be done by planes)
  float least = thr;
  auto open = [&](const rw_f16(&acc)[2]) {
    float mx = acc[0][0];
#pragma unroll
    for (int k = 0; k < 2; ++k)
#pragma unroll
      for (int v = 0; v < 16; ++v) mx = fmaxf(mx, acc[k][v]);
    return __any(mx >= least);
  };
  // Appends the wave's open pairs of column block cb: a bit per product
  // (element e = 16 k + v of the lane at bit 31 - e), then one pair per lane
  // and turn, with one LDS atomic per turn; `col`: what the list has for the
  // tile's first column.
  auto append = [&](const rw_f16(&acc)[2], int64_t m0, int64_t n0, int col, int cb) {
    uint32_t mask = 0;
#pragma unroll
    for (int k = 0; k < 2; ++k)
#pragma unroll
      for (int v = 0; v < 16; ++v) mask = mask + mask + (acc[k][v] >= thr ? 1u : 0u);
    const int nt = 32 * cb + (lane & 31);  // column in the tile
    int seen = 0;
    while (__any(mask != 0)) {
      const int e = mask ? __clz((int)mask) : 0;
      // product v: row 8 (v / 4) + 4 (lane / 32) + v % 4, column lane % 32
      const int mt = 64 * wid + 32 * (e >> 4) + 8 * ((e >> 2) & 3) + 4 * (lane >> 5) + (e & 3);
      const bool ok = mask != 0 && (uint32_t)m0 + mt < (uint32_t)n0 + nt && (uint32_t)n0 + nt < M;
      mask &= ~(0x80000000u >> e);
      const unsigned long long who = __ballot(ok);
      if (who == 0) continue;
      int at = 0;
      if (lane == 0) at = atomicAdd(&nlist, __popcll(who));
      seen = at = __builtin_amdgcn_readfirstlane(at);
      at += __popcll(who & ((1ull << lane) - 1));
      if (ok && at < kList) {
        if constexpr (kThree) {
          list_row[at] = (uint8_t)mt;
          list_col[at] = (uint16_t)(col + nt);
        } else {
          list[at] = (uint32_t)(mt << 16 | (col + nt));
        }
      }
    }
    if (seen > kList) least = INFINITY;
  };
  // code tiles from s on; returns the tile to go on with by planes (c1: none)
  auto by_code = [&](int s) {
    int rb, st, arow = -1, kept = 0;  // kept: pairs in the list
    if (!tile(s, rb, st)) return c1;
    for (;;) {
      const int64_t m0 = (int64_t)rb * kRwTile, n0 = (int64_t)st * kRwTile;
      if (rb != arow) {
        arow = rb;
#pragma unroll
        for (int k = 0; k < 2; ++k)
#pragma unroll
          for (int kc = 0; kc < UC; ++kc)
            a[k][kc] = *reinterpret_cast<const rw_i4*>(
                codes + (size_t)(2 * kc + (lane >> 5)) * Mpad + m0 + 64 * wid + 32 * k + (lane & 31));
      }
      fetch(st);  // the buffer's readers passed the last barrier
      // this wave's share of the tile's codes is in LDS; after the barrier all is
      __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0)
      __syncthreads();
      const int col = (int)(n0 - first_col(rb != p0)) + (rb != p0 ? kSecond : 0);
      least = thr;
      rw_i4 b0[UC], b1[UC];
      rw_f16 acc0[2], acc1[2];
      columns(b0, 0);
      for (int cb = 0; cb < kRwTile / 32; cb += 2) {
        columns(b1, cb + 1);
        products(b0, acc0);
        columns(b0, min(cb + 2, kRwTile / 32 - 1));
        products(b1, acc1);
        if (open(acc0)) append(acc0, m0, n0, col, cb);
        if (open(acc1)) append(acc1, m0, n0, col, cb + 1);
      }
      __syncthreads();  // the buffer's readers, the list
      const int now = nlist;
      if (now > kList) {
        // more open pairs than fit: this tile as a whole, and the rest of the run
        __syncthreads();  // every thread has read the count
        if (tid == 0) nlist = kept;
        return s;
      }
      kept = now;
      if (now > kList / 2 || s - base == kListTiles - 1) {
        __syncthreads();
        flush();
        kept = 0;
        base = s + 1;
      }
      if (!tile(++s, rb, st)) return c1;
    }
  };
  __syncthreads();
  int s = filter ? by_code(c0) : c0;
  by_planes(s);
  __syncthreads();
  flush();
}

// w = 1 / N and workgroup sums of it; k_meff_total adds them in order.
__global__ __launch_bounds__(256) void k_weights(const int32_t* __restrict__ n_sim, int64_t M,
                                                 double* __restrict__ w, double* __restrict__ part) {
  __shared__ double sh[16];
  double v = 0.0;
  for (int64_t m = (int64_t)blockIdx.x * 256 + threadIdx.x; m < M; m += (int64_t)gridDim.x * 256) {
    const double x = 1.0 / (double)n_sim[m];
    w[m] = x;
    v += x;
  }
  const double t = block_sum_f64(v, sh);
  if (threadIdx.x == 0) part[blockIdx.x] = t;
}

__global__ __launch_bounds__(256) void k_meff_total(const double* __restrict__ part, int n,
                                                    double* __restrict__ meff) {
  __shared__ double sh[16];
  const double t = block_sum_f64((int)threadIdx.x < n ? part[threadIdx.x] : 0.0, sh);
  if (threadIdx.x == 0) *meff = t;
}

template <int P, int W>
static void launch_count_pw(const ReweightPlan& plan, char* ws, int64_t M, int L, int T,
                            int32_t* n_sim, hipStream_t s) {
  const int64_t S = plan.Mpad / kRwTile;
  const int maxmis = L - T;  // similar iff mismatches <= L - T
  const int dims = rw_dims(W);
  const float thr = (float)(dims == 3 ? 3 * L - 4 * maxmis : L - 2 * maxmis);
  // where unrelated rows (about 3/4 of the positions differ) stay clear of the
  // bound: their d is about 3/8 L in one dimension, 9/16 L in three
  const int filter = maxmis * 20 <= (dims == 3 ? 9 : 6) * L ? 1 : 0;
  // runs of up to 16 tiles, shorter ones where that fills the device
  const int64_t tiles = (S + 1) / 2 * (S + 1);
  // (and longer ones where the grid would pass its limit of 2^32 threads)
  int64_t chunk = std::max<int64_t>(1, std::min<int64_t>(16, tiles / 2048));
  chunk = std::max(chunk, tiles >> 23);
  const int64_t items = (S + 1) / 2 * ceil_div(S + 1, chunk);
  hipLaunchKernelGGL((k_count_similar<P, W>), dim3((unsigned)items), dim3(kRwThreads), 0, s,
                     reinterpret_cast<const uint32_t*>(ws + plan.off_planes),
                     reinterpret_cast<const uint4*>(ws + plan.off_codes), plan.Mpad, M, maxmis, thr,
                     filter, (int)chunk, n_sim);
}

template <int W>
static void launch_count_w(const ReweightPlan& plan, char* ws, int64_t M, int L, int T,
                           int32_t* n_sim, hipStream_t s) {
  switch (plan.planes) {
    case 1: launch_count_pw<1, W>(plan, ws, M, L, T, n_sim, s); break;
    case 2: launch_count_pw<2, W>(plan, ws, M, L, T, n_sim, s); break;
    case 3: launch_count_pw<3, W>(plan, ws, M, L, T, n_sim, s); break;
    case 4: launch_count_pw<4, W>(plan, ws, M, L, T, n_sim, s); break;
    default: launch_count_pw<5, W>(plan, ws, M, L, T, n_sim, s); break;
  }
}

hipError_t launch_reweight(const int8_t* msa, int64_t M, int L, int q, int32_t T,
                           const ReweightPlan& plan, void* ws, int32_t* n_sim, double* w,
                           double* meff, int32_t* dev_err, hipStream_t s) {
  char* base = static_cast<char*>(ws);
  const int W = plan.words, P = plan.planes;
  // Unused planes (p >= P) are never read; padding bits are written as 0.
  hipLaunchKernelGGL(k_encode_rows, dim3((unsigned)ceil_div(plan.Mpad * W, 256)), dim3(256), 0, s,
                     msa, M, plan.Mpad, L, q, P, W,
                     reinterpret_cast<uint32_t*>(base + plan.off_planes),
                     reinterpret_cast<uint4*>(base + plan.off_codes), n_sim, dev_err);
  switch (W) {
#define BMDCA_RW_CASE(n) \
  case n:                \
    launch_count_w<n>(plan, base, M, L, T, n_sim, s); \
    break;
    BMDCA_RW_CASE(1) BMDCA_RW_CASE(2) BMDCA_RW_CASE(3) BMDCA_RW_CASE(4) BMDCA_RW_CASE(5)
    BMDCA_RW_CASE(6) BMDCA_RW_CASE(7) BMDCA_RW_CASE(8) BMDCA_RW_CASE(9) BMDCA_RW_CASE(10)
    BMDCA_RW_CASE(11) BMDCA_RW_CASE(12) BMDCA_RW_CASE(13) BMDCA_RW_CASE(14) BMDCA_RW_CASE(15)
    BMDCA_RW_CASE(16)
#undef BMDCA_RW_CASE
    default:
      return hipErrorInvalidValue;
  }
  double* red = reinterpret_cast<double*>(base + plan.off_red);
  const int nb = (int)std::min<int64_t>(kRwRed, ceil_div(M, 256));
  hipLaunchKernelGGL(k_weights, dim3((unsigned)nb), dim3(256), 0, s, n_sim, M, w, red);
  hipLaunchKernelGGL(k_meff_total, dim3(1), dim3(256), 0, s, red, nb, meff);
  return hipGetLastError();
}

}  // namespace bmdca
