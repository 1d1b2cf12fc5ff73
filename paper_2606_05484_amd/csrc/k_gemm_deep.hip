// The token-major bf16 product of k_gemm_bf16.hip for launches that its
// 128-token tiles would spread over a fraction of the chip (any anchor width):
//
//   out[t, n] = sum_{c < Ka} A[t, c] W[n, c]  +  sum_{i < Kg} T[ids[t], i] W[n, Ka + i]
//
// Output tiles of BM x 64 (BM = 64 or 128); the four waves own 64 x 64 wave
// tiles, BM / 64 of them side by side, and share K: a wave multiplies KW-th
// of the 16-wide k-steps of every 64-wide stage (KW = 4 or 2), which halves
// the LDS bytes per product against splitting a small tile four ways.  Stages
// come by buffer_load ... lds into a ring of NS slots, NS - 1 ahead: at these
// sizes a workgroup's walk over K is bound by memory latency, and two
// workgroups per CU, each with a ring of 64 to 72 KB, cover it (rings twice
// as deep, one workgroup per CU: up to 50 % slower at 512 tiles, no faster at
// 16).  Stages past the last read zeros, so every step
// issues the same loads and waits on the same count.  LDS rows, swizzle and
// operand order are those of tn_gemm.hpp; the KW partial tiles are summed
// through LDS in a fixed order.
#include "tn_gemm.hpp"

namespace mapl {

namespace {

template <int BM, int NS>
__global__ __launch_bounds__(GTHREADS) void k_gemm_tn_deep(TnArgs g) {
#if defined(__HIP_DEVICE_COMPILE__)
  constexpr int BN = 64, WM = BM / 64, KW = 4 / WM, AB = BM / 32, WB = 2, LOADS = AB + WB;
  constexpr int SLOT = (BM + BN) * GK;                 // bf16 of a ring slot: token rows, then W rows
  constexpr int KPW = GK / 16 / KW;                    // k-steps per wave and stage
  static_assert(NS * SLOT * 2 >= 4 * 4 * 4096, "the partial tiles fit the ring");
  __shared__ __attribute__((aligned(1024))) bf16_t ring[NS * SLOT];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / KW, wk = wave % KW;
  // contiguous runs of (token tile, column tile) per XCD: the column tiles of
  // one token tile read its rows through one L2
  const int nt = g.N / BN, total = (g.M + BM - 1) / BM * nt;
  const int per = gridDim.x >> 3, v = (blockIdx.x & 7) * per + (blockIdx.x >> 3);
  if (v >= total) return;
  const int m0 = v / nt * BM, n0 = v % nt * BN;
  const int mrows = min(BM, g.M - m0);
  const __amdgpu_buffer_rsrc_t ra = rsrc(g.A + (int64_t)m0 * g.lda, (uint64_t)mrows * g.lda * 2);
  const __amdgpu_buffer_rsrc_t rt = rsrc(g.T, g.T ? (uint64_t)g.V * g.ldt * 2 : 0);
  const __amdgpu_buffer_rsrc_t rw = rsrc(g.W + (int64_t)n0 * g.ldw, (uint64_t)BN * g.ldw * 2);

  // DMA geometry as in tn_mainloop: lane i of 1 KiB block b fills row
  // 8 b + i / 8, physical chunk i % 8 = logical chunk (i % 8) ^ ((row >> 1) & 7)
  const int lrow = lane >> 3;
  const uint32_t lch[2] = {(uint32_t)((lane & 7) ^ (lane >> 4)), (uint32_t)((lane & 7) ^ (4 + (lane >> 4)))};
  int id[AB];
  uint32_t a_off[AB], w_off[WB];
#pragma unroll
  for (int j = 0; j < AB; ++j) {
    const int row = 8 * (wave * AB + j) + lrow;
    id[j] = g.Kg > 0 && row < mrows ? g.ids[m0 + row] : -1;
    a_off[j] = (uint32_t)row * (uint32_t)g.lda * 2u + 16u * lch[j & 1];
  }
#pragma unroll
  for (int j = 0; j < WB; ++j) {
    const int row = 8 * (wave * WB + j) + lrow;
    w_off[j] = (uint32_t)row * (uint32_t)g.ldw * 2u + 16u * lch[j & 1];
  }
  const int ka = g.Ka / GK, KS = ka + (g.Kg + GK - 1) / GK;
  auto issue = [&](int s, int slot) {
    bf16_t* sa = ring + slot * SLOT;
    bf16_t* sw = sa + BM * GK;
    const bool gath = s >= ka, live = s < KS;
    const int kc = gath ? (s - ka) * GK : s * GK;
    // columns of the stage that exist (the gathered width may end inside it)
    const int lim = !live ? 0 : gath ? g.Kg - kc : GK;
    const bool ok[2] = {8 * (int)lch[0] < lim, 8 * (int)lch[1] < lim};
#pragma unroll
    for (int j = 0; j < AB; ++j) {
      const lds_ptr dst = (lds_ptr)(sa + (wave * AB + j) * 512);
      if (gath) {
        const uint32_t o = (uint32_t)clamp_id(id[j], g.V) * (uint32_t)g.ldt * 2u + 16u * lch[j & 1];
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rt, dst, 16, ok[j & 1] ? o : OOB, kc * 2, 0, 0);
      } else {
        __builtin_amdgcn_raw_ptr_buffer_load_lds(ra, dst, 16, a_off[j], kc * 2, 0, 0);
      }
    }
    const int wc = (gath ? g.Ka + kc : kc) * 2;
#pragma unroll
    for (int j = 0; j < WB; ++j)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rw, (lds_ptr)(sw + (wave * WB + j) * 512), 16,
                                               ok[j & 1] ? w_off[j] : OOB, wc, 0, 0);
  };
  f32x16_t acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) acc[i][j] = f32x16_t{};
  uint32_t koff[KPW];
#pragma unroll
  for (int q = 0; q < KPW; ++q) koff[q] = tn_koff(wk * KPW + q, lane);
  const uint32_t rbase = lds_addr(ring);
#pragma unroll
  for (int s = 0; s < NS - 1; ++s) issue(s, s);
  int slot = 0;
  for (int s = 0; s < KS; ++s) {
    // stage s has landed (this wave's part, then everyone's), and every wave
    // has read stage s - 1, whose slot the next load takes
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(LOADS * (NS - 2)) : "memory");
    __builtin_amdgcn_s_barrier();
    const uint32_t ba = rbase + (uint32_t)slot * (SLOT * 2) + wm * 64 * (GK * 2);
    const uint32_t bw = rbase + (uint32_t)slot * (SLOT * 2) + BM * GK * 2;
    u32x4 f[KPW][4];
#pragma unroll
    for (int q = 0; q < KPW; ++q) {
      f[q][0] = lds_read_b128<0>(ba + koff[q]);
      f[q][1] = lds_read_b128<32 * GK * 2>(ba + koff[q]);
      f[q][2] = lds_read_b128<0>(bw + koff[q]);
      f[q][3] = lds_read_b128<32 * GK * 2>(bw + koff[q]);
    }
    issue(s + NS - 1, slot == 0 ? NS - 1 : slot - 1);
#pragma unroll
    for (int q = 0; q < KPW; ++q) lds_wait(f[q]);
#pragma unroll
    for (int q = 0; q < KPW; ++q)
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = mfma32x32x16(as_uint4(f[q][2 + j]), as_uint4(f[q][i]), acc[i][j]);
    slot = slot + 1 == NS ? 0 : slot + 1;
  }
  // The KW partial tiles: every wave leaves its blocks in LDS (block (i, j)
  // of wave w at 4 KiB slot 4 w + 2 i + j) and sums 4 / KW of its tile's
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the zero-filling loads past the last stage
  __syncthreads();
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int q = 0; q < 4; ++q)
        lds_write_b128(rbase + (uint32_t)(((wave * 4 + 2 * i + j) * 4 + q) * 1024 + lane * 16),
                       u32x4{__float_as_uint(acc[i][j][4 * q]), __float_as_uint(acc[i][j][4 * q + 1]),
                             __float_as_uint(acc[i][j][4 * q + 2]), __float_as_uint(acc[i][j][4 * q + 3])});
  lds_wait0();
  __syncthreads();
  const int half = lane >> 5;
  static_for<0, 4 / KW>([&](auto uc) {
    constexpr int U = decltype(uc)::value;
    const int blk = wk * (4 / KW) + U, i = blk >> 1, j = blk & 1;
    float c[16];
    u32x4 p[KW][4];
#pragma unroll
    for (int w = 0; w < KW; ++w)
#pragma unroll
      for (int q = 0; q < 4; ++q)
        p[w][q] = lds_read_b128(rbase + (uint32_t)((((wm * KW + w) * 4 + blk) * 4 + q) * 1024 + lane * 16));
#pragma unroll
    for (int w = 0; w < KW; ++w) lds_wait(p[w]);
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        float x = __uint_as_float(p[0][q][e]);
#pragma unroll
        for (int w = 1; w < KW; ++w) x += __uint_as_float(p[w][q][e]);
        c[4 * q + e] = x;
      }
    // lane: token lane % 32 of the block, columns 8 q + 4 half + 0..3
    const int t = m0 + wm * 64 + i * 32 + (lane & 31);
    if (g.out_f32) {
      float* o = (float*)g.out + (int64_t)t * g.ldo + n0 + j * 32 + 4 * half;
      if (t < g.M)
#pragma unroll
        for (int q = 0; q < 4; ++q) *(float4*)(o + 8 * q) = make_float4(c[4 * q], c[4 * q + 1], c[4 * q + 2], c[4 * q + 3]);
      return;
    }
    uint32_t h[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) h[e] = pack_bf2(c[2 * e], c[2 * e + 1]);
    // pair the lane halves: 16 B of columns 8 (2 q + half) .. +7
#pragma unroll
    for (int q = 0; q < 2; ++q)
#pragma unroll
      for (int w = 0; w < 2; ++w) {
        const auto sw2 = __builtin_amdgcn_permlane32_swap(h[4 * q + w], h[4 * q + 2 + w], false, false);
        h[4 * q + w] = sw2[0];
        h[4 * q + 2 + w] = sw2[1];
      }
    if (t < g.M)
#pragma unroll
      for (int q = 0; q < 2; ++q)
        *(uint4*)((bf16_t*)g.out + (int64_t)t * g.ldo + n0 + j * 32 + 8 * (2 * q + half)) =
            make_uint4(h[4 * q], h[4 * q + 1], h[4 * q + 2], h[4 * q + 3]);
  });
#endif
}

}  // namespace

hipError_t launch_gemm_tn_deep(const TnArgs& g, hipStream_t s) {
  if (g.Ka % GK || g.Kg % 16 || g.N % 64 || g.Ka + g.Kg > g.ldw) return hipErrorInvalidValue;
  const int64_t t64 = (int64_t)((g.M + 63) / 64) * (g.N / 64), t128 = (int64_t)((g.M + 127) / 128) * (g.N / 64);
  // 64-token tiles while two of their workgroups per CU hold them all
  // (M = 8192, N = 256, K = 1088: 10.2 us against 11.1 with 128), then 128
  // (M = 16384, K = 2112: 24.3 against 31.3)
  if (t64 <= 512)
    hipLaunchKernelGGL((k_gemm_tn_deep<64, 4>), dim3((unsigned)((t64 + 7) / 8 * 8)), dim3(GTHREADS), 0, s, g);
  else
    hipLaunchKernelGGL((k_gemm_tn_deep<128, 3>), dim3((unsigned)((t128 + 7) / 8 * 8)), dim3(GTHREADS), 0, s, g);
  return hipGetLastError();
}

}  // namespace mapl
