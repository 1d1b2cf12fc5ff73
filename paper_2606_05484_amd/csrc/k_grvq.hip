// Grouped residual vector quantisation (Sec. 3.5, the coordinates
// decomposed into groups; App. E: group dimension 2, K = 256, R = 2): each
// token's r coordinates form r / 2 independent two-dimensional residuals,
// and group g is quantised round after round over the 2-D codewords
// C[l][j][2g : 2g + 2], the nearest by exact fp32 squared distance, the
// lowest index among equals.
//
// T r / 2 K L distances: at four operations plus a compare and two selects
// each, vector issue bounds a plain search (8192 tokens, r = 256, K = 256,
// L = 2: 101 us, which is that bound).  So the distances are screened on the
// matrix unit and only the winners' blocks are computed:
//   screen   s_j = ||C_j||^2 - 2 <R, C_j> = ||R - C_j||^2 - ||R||^2 as bf16
//            products of three-piece values (v = h + m + l): per coordinate
//            hh, hm, mh, mm, hl, lh, and the norm's pieces times one, 15 of
//            the 16 places of one v_mfma_f32_32x32x16_bf16 for 32 codewords
//            (rows) and 32 tokens (columns).  A lane sees one token's scores
//            of 16 codewords and keeps their minimum alone: half a vector
//            operation per score.
//   margin   fp32 rounding, u = 2^-24: the norm is off by 2u, the pieces left
//            out by u, the accumulation by 16u (each of its sums, of values
//            <= (|R| + |C_j|)^2), and the exact distance as it is computed
//            below by 4u of itself: less than 25u (|R| + |C_j|)^2 for each
//            side of a comparison.  The two sides are the codeword of the
//            smallest score, at distance d, and the nearest one, so |C_j| <=
//            |R| + d for both, and (2 |R| + d)^2 <= 5 (|R|^2 + d^2).  From
//            d^2 <= min + |R|^2 + 125u (|R|^2 + d^2): d^2 <= (1 + 2^-16) D,
//            D = min + |R|^2 + 2^-17 |R|^2.  The block of the nearest
//            codeword therefore has its minimum below
//              thr = min + 2^-15 (|R|^2 + D) + 1e-35   (2^-15 = 512u, twice
//            the 250u; the last term covers pieces and products below the
//            normal range).  Codewords far larger than the residual, as
//            outlier tokens leave them, do not widen it (with 2^-17 of the
//            largest |C_j|^2 in D, one codeword 3000 times the others: K =
//            256, L = 2, T = 32768, r = 256: 193.6 us a call, 147.6 so).
//            Codewords some thousand times smaller than the residual
//            do: their scores crowd inside 2^-14 |R|^2.
//   rescore  the blocks with a minimum below thr (one but for few searches; all
//            of them where a score or a norm is past the range of the pieces)
//            by the exact distances, eight codewords of a block to each of
//            the token's two lanes, the lowest index among equals.
// 38.9 us, bound by the vector unit (about 200 operations per 32 searches,
// half of them the rescoring).  The screen as fp32 products (two places, the
// norms as the C operand) took 58 us: those run on the vector unit's own
// adders, not beside it.
//
// Layout: a wave owns one group of 128 tokens (four column tiles, so that an
// operand row read from LDS serves four products and the chains of the
// rescoring overlap); a workgroup four neighbouring groups of 256 tokens, so
// two waves share a group's codebook round in LDS.  The next round's
// codewords are requested before the search.  Any L and K up to the limits
// below fit.
#include "common.hpp"
#include "kernels.hpp"

namespace mapl {

namespace {

constexpr int GQ_GROUPS = 4, GQ_BLOCKS = 2, GQ_WAVES = GQ_GROUPS * GQ_BLOCKS;  // groups and token blocks per workgroup
constexpr int GQ_NT = 4, GQ_TOK = 32 * GQ_NT * GQ_BLOCKS, GQ_KMAX = 256, GQ_LMAX = 8;

// v's three bf16 pieces (nearest rounding each time): their sum is v to
// 2^-27 |v|, and exact in most cases.
__device__ __forceinline__ void gq_split(float v, uint32_t& h, uint32_t& m, uint32_t& l) {
  h = f2bf(v);
  v -= bf2f(h);
  m = f2bf(v);
  l = f2bf(v - bf2f(m));
}
__device__ __forceinline__ uint32_t gq_pair(uint32_t lo, uint32_t hi) { return lo | hi << 16; }

// LDS place of a codeword: a tile's 256 bytes span the banks once, so tiles are
// 32 bytes apart for the lanes that read one block each of different tiles.
__device__ __forceinline__ int gq_slot(int j) { return j + (j >> 5 << 2); }

// KT: codeword tiles of 32 (K <= 32 KT; the rows past K are at infinity).
template <int KT>
__global__ __launch_bounds__(64 * GQ_WAVES, 4) void k_grvq(const float* __restrict__ Z0, const float* __restrict__ C,
                                                        int T, int r, int L, int K, uint8_t* __restrict__ codes) {
#if defined(__gfx950__)
  constexpr int KP = 32 * KT, CL = (KP + 127) / 128;  // codewords per lane when staged
  __shared__ __attribute__((aligned(16))) uint4 aw[GQ_GROUPS][KP][2];  // the product's operand rows
  __shared__ __attribute__((aligned(16))) float2 cw[GQ_GROUPS][KP + 4 * KT];
  __shared__ float cmax[GQ_GROUPS][GQ_BLOCKS];
  __shared__ __attribute__((aligned(4))) uint8_t out[GQ_TOK * GQ_LMAX][GQ_GROUPS];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, half = lane >> 5, col = lane & 31;
  const int grp = wave % GQ_GROUPS, blk = wave / GQ_GROUPS;
  const int G = r / 2, g0 = blockIdx.y * GQ_GROUPS, t0 = blockIdx.x * GQ_TOK;
  const float* cg = C + 2 * (g0 + grp);
  float2* cb = cw[grp];

  float2 cr[CL];  // the round being fetched: the group's two waves take 64 codewords in turn
  auto fetch = [&](int l) {
#pragma unroll
    for (int i = 0; i < CL; ++i) {
      const int j = lane + 64 * (blk + 2 * i);
      cr[i] = j < K ? *(const float2*)(cg + ((int64_t)l * K + j) * r) : make_float2(INFINITY, INFINITY);
    }
  };
  fetch(0);
  float2 R[GQ_NT];
#pragma unroll
  for (int n = 0; n < GQ_NT; ++n) {
    const int t = t0 + 32 * (GQ_NT * blk + n) + col;
    R[n] = t < T ? *(const float2*)(Z0 + (int64_t)t * r + 2 * (g0 + grp)) : make_float2(0.f, 0.f);
  }

  for (int l = 0; l < L; ++l) {
    if (l > 0) __syncthreads();  // the last round's codewords are done with
    float cm = 0.f;
#pragma unroll
    for (int i = 0; i < CL; ++i) {
      const int j = lane + 64 * (blk + 2 * i);
      const float n2 = fmaf(cr[i].y, cr[i].y, cr[i].x * cr[i].x);
      uint32_t h, m, lo, nh, nm, nl;
      gq_split(n2, nh, nm, nl);
      if (j < KP) {
        cb[gq_slot(j)] = cr[i];
        gq_split(cr[i].x, h, m, lo);
        aw[grp][j][0] = make_uint4(gq_pair(h, h), gq_pair(m, m), gq_pair(h, lo), gq_pair(nh, nm));
        gq_split(cr[i].y, h, m, lo);
        aw[grp][j][1] = make_uint4(gq_pair(h, h), gq_pair(m, m), gq_pair(h, lo), nl);
      }
      if (j < K) cm = fmaxf(cm, n2);
    }
    cm = wave_max(cm);
    if (lane == 0) cmax[grp][blk] = cm;
    __syncthreads();
    cm = fmaxf(cmax[grp][0], cmax[grp][1]);
    if (l + 1 < L) fetch(l + 1);

    float top = INFINITY;
    asm volatile("" : "+v"(top));  // a register: two scores then cost one v_min3 from the start
    float m[GQ_NT][KT], low[GQ_NT];
    uint4 b[GQ_NT];  // this half's coordinate of -2 R: (h, m), (h, m), (l, h), and ones for the norm's pieces
#pragma unroll
    for (int n = 0; n < GQ_NT; ++n) {
      uint32_t bh, bm, bl;
      gq_split(-2.f * (half ? R[n].y : R[n].x), bh, bm, bl);
      b[n] = make_uint4(gq_pair(bh, bm), gq_pair(bh, bm), gq_pair(bl, bh), half ? 0x3F80u : 0x3F803F80u);
      low[n] = INFINITY;
    }
#pragma unroll
    for (int kt = 0; kt < KT; ++kt) {
      const uint4 a = aw[grp][32 * kt + col][half];
#pragma unroll
      for (int n = 0; n < GQ_NT; ++n) {
        const f32x16_t s = mfma32x32x16(a, b[n], f32x16_t{});
        float v = fminf(fminf(top, s[0]), s[1]);
#pragma unroll
        for (int e = 2; e < 16; e += 2) v = fminf(fminf(v, s[e]), s[e + 1]);
        low[n] = fminf(low[n], v);
        asm volatile("" : "+v"(v));  // here: the products and folds would be sunk to their use,
        m[n][kt] = v;                // every score in a register until then
      }
    }

    // The four tiles' chains side by side: bounds and masks, the first block
    // of every token, the rare further ones, the merges of the lane pairs.
    uint32_t cand[GQ_NT];  // bit kt + KT (lane half): that block has to be computed
    float best[GQ_NT];
    int bj[GQ_NT];
    uint32_t rest = 0;
#pragma unroll
    for (int n = 0; n < GQ_NT; ++n) {
      const float v = fminf(low[n], __shfl_xor(low[n], 32, WAVE));
      const float rr = fmaf(R[n].y, R[n].y, R[n].x * R[n].x);
      const float thr = fmaf(0x1p-15f, rr + fmaxf(v + rr, 0.f) + 0x1p-17f * rr, v) + 1e-35f;
      uint32_t mine = 0;  // (thr - m is exact in sign; from the last tile down, bit kt ends in place)
#pragma unroll
      for (int kt = KT - 1; kt >= 0; --kt)
        mine = __builtin_amdgcn_alignbit(mine, __float_as_uint(m[n][kt] - thr), 31);
      const uint32_t other = __shfl_xor(mine, 32, WAVE);
      cand[n] = half ? other | mine << KT : mine | other << KT;
      if (!(fabsf(v) < INFINITY) | !(rr + cm < 1e37f) | (cand[n] == 0)) cand[n] = (1u << 2 * KT) - 1;
      best[n] = INFINITY;
      bj[n] = 0;
    }
    auto compute = [&](int n) {  // the lowest block left (cand[n] != 0)
      const int bit = __builtin_ctz(cand[n]);
      cand[n] &= cand[n] - 1;
      // the block's rows are 8 q + 4 (its half) + 0..3 of the tile: q = 2 half, 2 half + 1 here
      const int j0 = 32 * (bit & (KT - 1)) + (bit >= KT ? 4 : 0) + 16 * half;
      const float2* p = cb + gq_slot(j0);
      float bd = INFINITY;
      int bi = 0;
#pragma unroll
      for (int i = 0; i < 8; i += 2) {  // codewords 0..3 and 8..11 from j0
        const int o = i < 4 ? i : i + 4;
        const float4 c2 = *(const float4*)(p + o);
        float dx = R[n].x - c2.x, dy = R[n].y - c2.y;
        float dd = fmaf(dy, dy, dx * dx);
        if (dd < bd) { bd = dd; bi = o; }
        dx = R[n].x - c2.z;
        dy = R[n].y - c2.w;
        dd = fmaf(dy, dy, dx * dx);
        if (dd < bd) { bd = dd; bi = o + 1; }
      }
      bi += j0;
      if ((bd < best[n]) | ((bd == best[n]) & (bi < bj[n]))) { best[n] = bd; bj[n] = bi; }
    };
#pragma unroll
    for (int n = 0; n < GQ_NT; ++n) {
      compute(n);
      rest |= cand[n];
    }
    if (__any(rest)) {
#pragma unroll
      for (int n = 0; n < GQ_NT; ++n)
        while (cand[n]) compute(n);
    }
#pragma unroll
    for (int n = 0; n < GQ_NT; ++n) {
      const float od = __shfl_xor(best[n], 32, WAVE);
      const int oj = __shfl_xor(bj[n], 32, WAVE);
      if ((od < best[n]) | ((od == best[n]) & (oj < bj[n]))) bj[n] = oj;
    }
#pragma unroll
    for (int n = 0; n < GQ_NT; ++n) {
      const float2 w = cb[gq_slot(bj[n])];
      R[n].x -= w.x;
      R[n].y -= w.y;
      if (half == 0) out[(32 * (GQ_NT * blk + n) + col) * L + l][grp] = (uint8_t)bj[n];
    }
  }

  __syncthreads();
  const int rows = min(GQ_TOK, T - t0) * L;  // (token, round) rows of G codes
  for (int i = threadIdx.x; i < rows; i += 64 * GQ_WAVES)
    *(uint32_t*)(codes + ((int64_t)t0 * L + i) * G + g0) = *(const uint32_t*)out[i];
#endif
}

}  // namespace

bool grvq_supported(int r, int L, int K) { return r % (2 * GQ_GROUPS) == 0 && K <= GQ_KMAX && K % 2 == 0 && L >= 1 && L <= GQ_LMAX; }

hipError_t launch_grvq(const float* Z0, const float* C, int T, int r, int L, int K, uint8_t* codes, hipStream_t s) {
  if (T <= 0 || L <= 0) return hipSuccess;
  if (!grvq_supported(r, L, K)) return hipErrorInvalidValue;
  const dim3 grid((T + GQ_TOK - 1) / GQ_TOK, r / 2 / GQ_GROUPS), block(64 * GQ_WAVES);
  // as many tiles as K has, to the next power of two (K = 32 with two tiles,
  // T = 32768, r = 256, L = 2: the call 98.2 us, with one 80.6)
  if (K > 128) hipLaunchKernelGGL(k_grvq<8>, grid, block, 0, s, Z0, C, T, r, L, K, codes);
  else if (K > 64) hipLaunchKernelGGL(k_grvq<4>, grid, block, 0, s, Z0, C, T, r, L, K, codes);
  else if (K > 32) hipLaunchKernelGGL(k_grvq<2>, grid, block, 0, s, Z0, C, T, r, L, K, codes);
  else hipLaunchKernelGGL(k_grvq<1>, grid, block, 0, s, Z0, C, T, r, L, K, codes);
  return hipGetLastError();
}

}  // namespace mapl
