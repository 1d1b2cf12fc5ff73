// fp32 products with few output tiles: the fp32 codec path's calls (outputs
// of a few hundred rows) and the Stiefel step's Gram-shaped products of small
// projector sets.  Such launches are bound by one workgroup's chain of
// load - multiply steps over K, not by arithmetic: at T = 512, d = 256,
// r = 32 the 128 x 128 kernel runs 1 to 8 workgroups of K / 32 dependent
// stages of about 1 us each.  Here a workgroup owns one 32 x 32 output tile
// and its W waves (4 or 16) split K in 32-deep batches, dealt out round
// robin; every wave loads its operands straight into the matrix unit's
// layout (no LDS, no barrier), one batch ahead, and the W partial tiles are
// summed through LDS in wave order (bitwise reproducible).  A second segment
// adds another product to the same accumulators, its rows gathered by token
// id, so the anchor terms of Eqs. 1-2 need no gathered copy and no second
// pass over the output.  M = 512, N = 32, K = 256: 23.5 -> 6.1 us; M = N = 256,
// K = 1024, batch 3: 78 -> 11 us; the fp32 codec's four calls at T = 512,
// d = 256, r = 32: 17 launches, 271 us -> 11 launches, 65 us.
#include "common.hpp"
#include "kernels.hpp"

namespace mapl {

namespace {

constexpr int FS_T = 32, FS_KB = 32;  // output tile, K per batch
constexpr uint32_t FS_OOB = 0x80000000u;

// A buffer resource from `base` on, covering what is left of the operand.
// Offsets inside a batch stay far below 2^31 (the strides are a few thousand
// elements), so only the base needs 64 bits.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t fs_rsrc(const float* base, int64_t left) {
  const int64_t bytes = left * 4;
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(base), 0,
                                           (int)(bytes < 0 ? 0 : bytes > 0x7ffffff0ll ? 0x7ffffff0ll : bytes),
                                           0x00020000);
}

// One batch's operand values of a lane: element e = 4 u + i holds
// k = 8 u + 4 (lane / 32) + i of row (or column) lane % 32.
struct FsBatch {
  float a[16], b[16];
};

template <int W>
__global__ __launch_bounds__(64 * W) void k_gemm_f32s(GemmF32sArgs g) {
  __shared__ float part[W][16 * 64];
  const int tid = threadIdx.x, lane = tid & 63, half = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  int bm = blockIdx.x, bn = blockIdx.y;
  const int b = blockIdx.z;
  if (g.sym_upper) {  // tiles on and above the diagonal, row by row
    const int nt = (g.M + FS_T - 1) / FS_T;
    int t = blockIdx.x, row = 0;
    while (t >= nt - row) {
      t -= nt - row;
      ++row;
    }
    bm = row;
    bn = row + t;
  }
  const int m0 = bm * FS_T, n0 = bn * FS_T;
  const int m = m0 + (lane & 31), n = n0 + (lane & 31);
  const bool mok = m < g.M, nok = n < g.N;

  // this thread's output elements (slot tid / 64 + W q of the accumulators):
  // Cin is requested before the K loop
  constexpr int EPT = 16 / W > 0 ? 16 / W : 1;
  float cin[EPT];
#pragma unroll
  for (int q = 0; q < EPT; ++q) {
    const int om = m0 + acc_row(wave + W * q, lane);
    cin[q] = g.Cin && om < g.M && nok ? g.Cin[b * g.sCinb + om * g.sCinm + n * g.sCinn] : 0.f;
  }

  const int nb0 = (g.seg[0].K + FS_KB - 1) / FS_KB;
  const int nb = nb0 + (g.nseg > 1 ? (g.seg[1].K + FS_KB - 1) / FS_KB : 0);

  auto load = [&](int kb, FsBatch& x) {
    const bool second = kb >= nb0;
    const GemmF32Seg& s = g.seg[second ? 1 : 0];
    const int k0 = (second ? kb - nb0 : kb) * FS_KB;
    const int kl = s.K - k0;  // columns of K left
    const int64_t bA = second ? 0 : b * g.sAb, bB = second ? 0 : b * g.sBb;
    const int kc = 4 * half;
    // ---- A
    {
      // gathered rows: the lane's row offset in the table; the rest from the tile's first row
      const float* base;
      int64_t left;
      uint32_t row;
      if (s.gather == 1) {
        base = s.A + k0 * s.sAk;
        left = (int64_t)(s.V - 1) * s.sAm + (int64_t)(kl - 1) * s.sAk + 1;
        row = mok ? (uint32_t)clamp_id(s.ids[m], s.V) * (uint32_t)s.sAm * 4u : FS_OOB;
      } else {
        base = s.A + bA + (int64_t)m0 * s.sAm + (s.gather == 2 ? 0 : (int64_t)k0 * s.sAk);
        left = (int64_t)(g.M - m0 - 1) * s.sAm + (int64_t)((s.gather == 2 ? s.V : kl) - 1) * s.sAk + 1;
        row = mok ? (uint32_t)(lane & 31) * (uint32_t)s.sAm * 4u : FS_OOB;
      }
      const __amdgpu_buffer_rsrc_t r = fs_rsrc(base, left);
      if (s.gather == 2) {
        int id[16];
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          const int k = 8 * (e >> 2) + kc + (e & 3);
          id[e] = k < kl ? clamp_id(s.ids[k0 + k], s.V) : -1;
        }
#pragma unroll
        for (int e = 0; e < 16; ++e)
          x.a[e] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(
              r, id[e] >= 0 && mok ? row + (uint32_t)id[e] * (uint32_t)s.sAk * 4u : FS_OOB, 0, 0));
      } else if (s.sAk == 1 && s.sAm % 4 == 0 && s.K % 4 == 0 && ((uintptr_t)base & 15) == 0) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const bool ok = mok && 8 * u + kc < kl;
          const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(r, ok ? row + (8 * u + kc) * 4u : FS_OOB, 0, 0);
#pragma unroll
          for (int i = 0; i < 4; ++i) x.a[4 * u + i] = __uint_as_float(v[i]);
        }
      } else {
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          const int k = 8 * (e >> 2) + kc + (e & 3);
          x.a[e] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(
              r, mok && k < kl ? row + (uint32_t)k * (uint32_t)s.sAk * 4u : FS_OOB, 0, 0));
        }
      }
    }
    // ---- B
    {
      const float* base = s.B + bB + (int64_t)n0 * s.sBn + (int64_t)k0 * s.sBk;
      const int64_t left = (int64_t)(g.N - n0 - 1) * s.sBn + (int64_t)(kl - 1) * s.sBk + 1;
      const __amdgpu_buffer_rsrc_t r = fs_rsrc(base, left);
      const uint32_t col = nok ? (uint32_t)(lane & 31) * (uint32_t)s.sBn * 4u : FS_OOB;
      if (s.sBk == 1 && s.sBn % 4 == 0 && s.K % 4 == 0 && ((uintptr_t)base & 15) == 0) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const bool ok = nok && 8 * u + kc < kl;
          const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(r, ok ? col + (8 * u + kc) * 4u : FS_OOB, 0, 0);
#pragma unroll
          for (int i = 0; i < 4; ++i) x.b[4 * u + i] = __uint_as_float(v[i]);
        }
      } else {
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          const int k = 8 * (e >> 2) + kc + (e & 3);
          x.b[e] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(
              r, nok && k < kl ? col + (uint32_t)k * (uint32_t)s.sBk * 4u : FS_OOB, 0, 0));
        }
      }
    }
  };
  // A is scaled as it enters, B through the result: nothing leaves fp32's range
  // where the scaled operands do not
  const float pa = g.pre_a ? g.pre_a[b] : 1.f, alpha = g.alpha * (g.pre_b ? g.pre_b[b] : 1.f);
  f32x16_t acc = f32x16_t{};
  auto mul = [&](int kb, const FsBatch& x) {
    const float sg = g.seg[kb >= nb0 ? 1 : 0].sign * pa;
#pragma unroll
    for (int e = 0; e < 16; ++e) acc = mfma32x32x2f32(sg * x.a[e], x.b[e], acc);
  };
  FsBatch x0, x1;
  int kb = wave;
  if (kb < nb) load(kb, x0);
  for (; kb < nb; kb += 2 * W) {
    if (kb + W < nb) load(kb + W, x1);
    mul(kb, x0);
    if (kb + W >= nb) break;
    if (kb + 2 * W < nb) load(kb + 2 * W, x0);
    mul(kb + W, x1);
  }
#pragma unroll
  for (int e = 0; e < 16; ++e) part[wave][e * 64 + lane] = acc[e];
  __syncthreads();
  float* C = g.C + b * g.sCb;
#pragma unroll
  for (int q = 0; q < EPT; ++q) {
    const int e = wave + W * q;
    float v = part[0][e * 64 + lane];
#pragma unroll
    for (int w = 1; w < W; ++w) v += part[w][e * 64 + lane];
    const int om = m0 + acc_row(e, lane);
    v = alpha * v + g.beta * cin[q];
    if (om < g.M && nok) {
      C[om * g.sCm + n * g.sCn] = v;
      if (g.sym_upper && bm != bn) C[n * g.sCm + om * g.sCn] = v;
    }
  }
}

}  // namespace

// The 128 x 128 kernel takes the same time from one tile to 256 (a tile per
// CU), this one grows with the work: they meet at about 120 tiles whatever K
// is.  Measured (128-tile kernel / this one, us): 16 tiles K = 1024: 80 / 11,
// 64: 80 / 40, 128: 81 / 77; 96 tiles K = 2048: 152 / 103, 192: 153 / 203;
// 48 tiles K = 256: 25 / 10; 128 tiles K = 512: 44 / 45.
bool gemm_f32_small(int64_t M, int64_t N, int64_t batch) {
  return ((M + 127) / 128) * ((N + 127) / 128) * batch < 120;
}

hipError_t launch_gemm_f32s(const GemmF32sArgs& g, hipStream_t s) {
  if (g.M <= 0 || g.N <= 0 || g.batch <= 0) return hipSuccess;
  if (g.nseg < 1 || g.nseg > 2 || (g.nseg == 2 && g.batch != 1) || (g.sym_upper && g.M != g.N)) return hipErrorInvalidValue;
  int64_t nb = 0;
  for (int i = 0; i < g.nseg; ++i) {
    const GemmF32Seg& q = g.seg[i];
    // offsets inside a batch are 32-bit byte offsets (a gathered table is under 2 GiB)
    const int64_t lim = 1ll << 29, tab = q.gather == 1 ? q.V * q.sAm : q.gather == 2 ? q.V * q.sAk : 0;
    if (q.K < 0 || q.sAm < 0 || q.sAk < 0 || q.sBk < 0 || q.sBn < 0 || 32 * (q.sBk + q.sBn) > lim || tab > lim ||
        (q.gather != 1 ? 32 * q.sAm : 0) + (q.gather != 2 ? 32 * q.sAk : 0) + tab > lim + 1024 * 32)
      return hipErrorInvalidValue;
    nb += (q.K + FS_KB - 1) / FS_KB;
  }
  const int mt = (g.M + FS_T - 1) / FS_T, nt = (g.N + FS_T - 1) / FS_T;
  const dim3 grid = g.sym_upper ? dim3(mt * (mt + 1) / 2, 1, g.batch) : dim3(mt, nt, g.batch);
  // 16 waves where K has a batch for most of them, else 4
  if (nb > 8) hipLaunchKernelGGL((k_gemm_f32s<16>), grid, dim3(1024), 0, s, g);
  else hipLaunchKernelGGL((k_gemm_f32s<4>), grid, dim3(256), 0, s, g);
  return hipGetLastError();
}

}  // namespace mapl
