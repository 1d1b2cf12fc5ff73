// Products of commuting symmetric r x r matrices for the PolarExpress
// iteration (Eqs. 6 and 7 in the r x r space): C = alpha A B + beta Cin +
// diag I, every operand and result a polynomial of the same S, so all of
// them are symmetric and only the tiles on and above the diagonal are
// computed.
//
// A matrix travels between these launches as two fp16 planes of 2^8 x (hi =
// fp16(2^8 x), lo = fp16(2^8 x - hi)), in the order in which the matrix unit
// takes them: for each 32-row block and 16-column block, 1 KiB of 64 lanes x
// 16 bytes (lane l: row l % 32, columns 8 (l / 32) .. +7).  A product is
// hi.hi + hi.lo + lo.hi on v_mfma_f32_32x32x16_f16 with fp32 accumulation,
// scaled by 2^-16: the split of k_gemm_x3, made once where a value is
// produced instead of by every workgroup that reads it.  B enters as B^T, so
// both operands are read along their rows; for that every stored matrix is
// symmetric to the bit (tiles below the diagonal are copies, diagonal tiles
// are averaged with their transpose): with A B^T in place of A B the
// rounding's antisymmetric part would grow from step to step (tenfold error
// of the LMO's direction in a float32 emulation).  Ranks up to 64, where the
// products of a square projector are the worst conditioned for their size,
// keep A B and no mirroring: k_polar_small runs a whole segment of them in
// one launch.
//
// These launches are bound by latency and by what a CU can load, not by
// their 3 x 2 r^3 / 2 fp16 operations: so a workgroup's W waves split K,
// every wave reads whole 1 KiB fragments straight into registers (no LDS
// staging, no barriers in the loop; a 64 x 64 wave tile takes 8 KiB for
// twelve products), up to 2 D steps ahead, and the partial tiles are summed
// through LDS in wave order (bitwise reproducible).
#include "common.hpp"
#include "kernels.hpp"

namespace mapl {

namespace {

__device__ __forceinline__ __amdgpu_buffer_rsrc_t sy_rsrc(const void* base, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, (int)bytes, 0x00020000);
}

// hi and lo pieces of eight values v (already times 2^8)
__device__ __forceinline__ void sy_split8(const float (&v)[8], uint4& hi, uint4& lo) {
  uint32_t h[4], l[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    h[i] = pack_h2(v[2 * i], v[2 * i + 1]);
    l[i] = pack_h2(v[2 * i] - h2f(h[i] & 0xFFFFu), v[2 * i + 1] - h2f(h[i] >> 16));
  }
  hi = make_uint4(h[0], h[1], h[2], h[3]);
  lo = make_uint4(l[0], l[1], l[2], l[3]);
}

// Byte offset of lane l's 16 bytes of fragment (row block rb, column block cb)
__device__ __forceinline__ uint32_t sy_off(int rb, int cb, int lane, int r) {
  return (uint32_t)((rb * (r >> 4) + cb) * 64 + lane) * 16u;
}

// F: 32F x 32F output tile; W waves split the r / 16 column blocks; D blocks
// per register set, two sets.
template <int F, int W, int D>
__global__ __launch_bounds__(64 * W) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_sym(SymArgs g) {
  constexpr int T = 32 * F;
  constexpr int PARTF = F * F * 16 * 64;                        // floats of one wave's partial tile
  constexpr int LDF = W * PARTF > T * (T + 1) ? W * PARTF : T * (T + 1);
  __shared__ float sh[LDF];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // Tile t of matrix b.  Workgroups go to the 8 XCDs round robin by id, each
  // XCD with its own L2: XCD x takes a contiguous run of the (matrix, tile)
  // list, so that a matrix is read through one or two L2s only.
  const int nt = (g.r + T - 1) / T, ntile = nt * (nt + 1) / 2;
  const int per = gridDim.x >> 3, v = (blockIdx.x & 7) * per + (blockIdx.x >> 3);
  if (v >= ntile * g.batch) return;
  int b = v / ntile, t = v % ntile;
  int bm = 0;
  while (t >= nt - bm) {
    t -= nt - bm;
    ++bm;
  }
  const int bn = bm + t;
  const bool second = b >= g.P;  // the second product of a paired launch
  if (second) b -= g.P;
  const int64_t rr = (int64_t)g.r * g.r;
  const uint16_t* A = (second ? g.A2 : g.A) + 2 * rr * b;
  const uint16_t* B = g.B + 2 * rr * b;
  uint16_t* C = second ? g.C2 : g.C;
  const uint32_t plane = (uint32_t)rr * 2u;
  const __amdgpu_buffer_rsrc_t ra = sy_rsrc(A, 2 * plane), rb = sy_rsrc(B, 2 * plane);
  const int nrb = g.r >> 5, KB = g.r >> 4;
  constexpr uint32_t OOB = 0x80000000u;

  struct Set {
    u32x4 ah[D][F], al[D][F], bh[D][F], bl[D][F];
  };
  // blocks cb0, cb0 + W, ... (D of them); past the last block or row block: zeros
  auto load = [&](int cb0, Set& x) {
#pragma unroll
    for (int d = 0; d < D; ++d) {
      const int cb = cb0 + W * d;
#pragma unroll
      for (int i = 0; i < F; ++i) {
        const uint32_t oa = cb < KB && bm * F + i < nrb ? sy_off(bm * F + i, cb, lane, g.r) : OOB;
        const uint32_t ob = cb < KB && bn * F + i < nrb ? sy_off(bn * F + i, cb, lane, g.r) : OOB;
        x.ah[d][i] = __builtin_amdgcn_raw_buffer_load_b128(ra, oa, 0, 0);
        x.bh[d][i] = __builtin_amdgcn_raw_buffer_load_b128(rb, ob, 0, 0);
        x.al[d][i] = __builtin_amdgcn_raw_buffer_load_b128(ra, oa, plane, 0);
        x.bl[d][i] = __builtin_amdgcn_raw_buffer_load_b128(rb, ob, plane, 0);
      }
    }
  };
  f32x16_t acc[F][F];
#pragma unroll
  for (int i = 0; i < F; ++i)
#pragma unroll
    for (int j = 0; j < F; ++j) acc[i][j] = f32x16_t{};
  auto mul = [&](const Set& x) {
    auto mma = [](const u32x4& p, const u32x4& q, f32x16_t c) { return mfma32x32x16h(as_uint4(p), as_uint4(q), c); };
#pragma unroll
    for (int d = 0; d < D; ++d) {
#pragma unroll
      for (int i = 0; i < F; ++i)
#pragma unroll
        for (int j = 0; j < F; ++j) acc[i][j] = mma(x.al[d][i], x.bh[d][j], acc[i][j]);
#pragma unroll
      for (int i = 0; i < F; ++i)
#pragma unroll
        for (int j = 0; j < F; ++j) acc[i][j] = mma(x.ah[d][i], x.bl[d][j], acc[i][j]);
#pragma unroll
      for (int i = 0; i < F; ++i)
#pragma unroll
        for (int j = 0; j < F; ++j) acc[i][j] = mma(x.ah[d][i], x.bh[d][j], acc[i][j]);
    }
  };
  Set x0, x1;
  int cb = wave;
  load(cb, x0);
  if (cb + W * D < KB) load(cb + W * D, x1);

  // the thread's elements after the sum: slot (w EPW + q) of the tile's
  // F F 16 accumulator slots, w its wave
  constexpr int EPW = F * F * 16 / W;
  static_assert(EPW * W == F * F * 16, "slots split over the waves");
  auto pos = [&](int q, int& m, int& n) {
    const int s = wave * EPW + q, ij = s >> 4, e = s & 15;
    m = (ij / F) * 32 + acc_row(e, lane);
    n = (ij % F) * 32 + (lane & 31);
  };
  const float beta = g.beta * (g.beta_ptr ? g.beta_ptr[b] : 1.f);
  float cin[EPW];
#pragma unroll
  for (int q = 0; q < EPW; ++q) {
    int m, n;
    pos(q, m, n);
    m += bm * T;
    n += bn * T;
    cin[q] = g.Cin && m < g.r && n < g.r ? g.Cin[rr * b + (int64_t)m * g.r + n] : 0.f;
  }
  for (; cb < KB; cb += 2 * W * D) {
    mul(x0);
    if (cb + W * D >= KB) break;
    if (cb + 2 * W * D < KB) load(cb + 2 * W * D, x0);
    mul(x1);
    if (cb + 3 * W * D < KB) load(cb + 3 * W * D, x1);
  }
#pragma unroll
  for (int i = 0; i < F; ++i)
#pragma unroll
    for (int j = 0; j < F; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) sh[wave * PARTF + ((i * F + j) * 16 + e) * 64 + lane] = acc[i][j][e];
  __syncthreads();
  float sum[EPW];
  const float alpha = g.alpha * (1.f / 65536.f);
#pragma unroll
  for (int q = 0; q < EPW; ++q) {
    const int s = wave * EPW + q;
    float x = sh[s * 64 + lane];
#pragma unroll
    for (int w = 1; w < W; ++w) x += sh[w * PARTF + s * 64 + lane];
    int m, n;
    pos(q, m, n);
    x = alpha * x + beta * cin[q];
    sum[q] = bm * T + m == bn * T + n ? x + g.diag : x;
  }
  __syncthreads();
  // the tile, rows of T + 1 floats
#pragma unroll
  for (int q = 0; q < EPW; ++q) {
    int m, n;
    pos(q, m, n);
    sh[m * (T + 1) + n] = sum[q];
  }
  __syncthreads();
  // fragments of the tile and (off the diagonal) of its mirror: one fragment
  // row piece of 8 columns per thread and turn
  constexpr int PIECES = F * (2 * F) * 64;  // row blocks x column blocks x lanes
  float* Cf = g.Cf ? g.Cf + rr * b : nullptr;
#pragma unroll
  for (int mir = 0; mir < 2; ++mir) {
    if (mir && bm == bn) break;
    for (int p = tid; p < PIECES; p += 64 * W) {
      const int l = p & 63, blk = p >> 6, i = blk / (2 * F), c = blk % (2 * F);
      const int row = i * 32 + (l & 31), col = c * 16 + 8 * (l >> 5);  // in the tile (mirror: of its transpose)
      const int R0 = (mir ? bn : bm) * T, C0 = (mir ? bm : bn) * T;
      if (R0 + row >= g.r || C0 + col >= g.r) continue;
      float y[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const float up = sh[row * (T + 1) + col + e], lo = sh[(col + e) * (T + 1) + row];
        y[e] = bm == bn ? 0.5f * (up + lo) : mir ? lo : up;
      }
      if (Cf && !(mir && !g.cf_full)) {
        float4* o = (float4*)(Cf + (int64_t)(R0 + row) * g.r + C0 + col);
        o[0] = make_float4(y[0], y[1], y[2], y[3]);
        o[1] = make_float4(y[4], y[5], y[6], y[7]);
      }
      if (C) {
#pragma unroll
        for (int e = 0; e < 8; ++e) y[e] *= 256.f;
        uint4 hi, lo;
        sy_split8(y, hi, lo);
        char* o = (char*)(C + 2 * rr * b) + sy_off((R0 >> 5) + i, (C0 >> 4) + c, l, g.r);
        *(uint4*)o = hi;
        *(uint4*)(o + plane) = lo;
      }
    }
  }
}

// Planes of scale[b] S for fp32 S [P][r][r].  With part (the row-block
// maxima of launch_inf_norm_partial) the scale is 1 / nu^2, nu^2 their
// maximum, and 1 / nu, 1 / nu^2 are written out.
__global__ __launch_bounds__(256) void k_sym_split(const float* __restrict__ S, int r, const float* __restrict__ part,
                                                   int npart, uint16_t* __restrict__ C, float* __restrict__ inv_nu,
                                                   float* __restrict__ inv_nu2) {
  const int b = blockIdx.y;
  const int64_t rr = (int64_t)r * r;
  const int p = blockIdx.x * 256 + threadIdx.x;  // one piece of 8 columns
  const int l = p & 63, blk = p >> 6, KB = r >> 4, rb = blk / KB, cb = blk % KB;
  const bool ok = p < r * r / 8;
  float y[8];
  if (ok) {
    const int row = rb * 32 + (l & 31), col = cb * 16 + 8 * (l >> 5);
    const float* Sb = S + rr * b;
#pragma unroll
    for (int e = 0; e < 8; ++e)  // averaged with the transpose: symmetric to the bit
      y[e] = 0.5f * (Sb[(int64_t)row * r + col + e] + Sb[(int64_t)(col + e) * r + row]);
  }
  float sc = 256.f;
  if (part) {
    float nu2 = 0.f;
    for (int i = threadIdx.x & 63; i < npart; i += 64) nu2 = fmaxf(nu2, part[(int64_t)b * npart + i]);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) nu2 = fmaxf(nu2, __shfl_xor(nu2, o, WAVE));
    const float i2 = 1.f / nu2;
    sc *= i2;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
      inv_nu[b] = sqrtf(i2);
      inv_nu2[b] = i2;
    }
  }
  if (!ok) return;
#pragma unroll
  for (int e = 0; e < 8; ++e) y[e] *= sc;
  uint4 hi, lo;
  sy_split8(y, hi, lo);
  char* o = (char*)(C + 2 * rr * b) + (uint32_t)p * 16u;
  *(uint4*)o = hi;
  *(uint4*)(o + rr * 2) = lo;
}

// One segment of the iteration for r <= 64, a workgroup per projector with
// every matrix in LDS (fp32, rows of r + 1): S scaled, then per step Q~ =
// (a I + b S + c S S) / a, P~ <- P~ Q~, S <- a^2 Q~ (S Q~), the products as
// above (hi.hi + hi.lo + lo.hi of 2^8 x), each wave one 32 x 32 block.  The
// same steps as launches take 3 to 4 us each, of which 40 make a step.
template <int R>
__global__ __launch_bounds__(256) void k_polar_small(PolarSmallArgs g) {
  constexpr int LD = R + 1, NB = R / 32;
  __shared__ float S[R * LD], Q[R * LD], X[R * LD], Pm[R * LD];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, half = lane >> 5;
  const int b = blockIdx.x;
  float sc = 1.f;
  if (g.part) {
    float nu2 = 0.f;
    for (int i = 0; i < g.npart; ++i) nu2 = fmaxf(nu2, g.part[(int64_t)b * g.npart + i]);
    sc = 1.f / nu2;
    if (tid == 0) g.inv_nu[b] = sqrtf(sc);
  }
  float* Sg = g.S + (int64_t)b * R * R;
  for (int i = tid; i < R * R; i += 256) S[(i / R) * LD + i % R] = sc * Sg[i];
  __syncthreads();
  const bool on = wave < NB * NB;
  const int m0 = 32 * (wave / NB), n0 = 32 * (wave % NB);
  auto pieces = [&](const float (&v)[8], uint4& hi, uint4& lo) {
    float y[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) y[e] = 256.f * v[e];
    sy_split8(y, hi, lo);
  };
  // this wave's block of A B
  auto product = [&](const float* A, const float* B) {
    f32x16_t acc = f32x16_t{};
#pragma unroll
    for (int k0 = 0; k0 < R; k0 += 16) {
      float av[8], bv[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        av[e] = A[(m0 + (lane & 31)) * LD + k0 + 8 * half + e];
        bv[e] = B[(k0 + 8 * half + e) * LD + n0 + (lane & 31)];
      }
      uint4 ah, al, bh, bl;
      pieces(av, ah, al);
      pieces(bv, bh, bl);
      acc = mfma32x32x16h(al, bh, acc);
      acc = mfma32x32x16h(ah, bl, acc);
      acc = mfma32x32x16h(ah, bh, acc);
    }
    return acc;
  };
  auto store = [&](float* C, const f32x16_t& acc, float alpha) {
    if (on)
#pragma unroll
      for (int e = 0; e < 16; ++e) C[(m0 + acc_row(e, lane)) * LD + n0 + (lane & 31)] = alpha * (1.f / 65536.f) * acc[e];
    __syncthreads();
  };
  for (int k = 0; k < g.steps; ++k) {
    f32x16_t acc = f32x16_t{};
    if (on) {
      acc = product(S, S);
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const int m = m0 + acc_row(e, lane), n = n0 + (lane & 31);
        acc[e] = 65536.f * (g.c[k] * (acc[e] * (1.f / 65536.f)) + g.b[k] * S[m * LD + n] + (m == n ? 1.f : 0.f));
      }
    }
    store(Q, acc, 1.f);
    if (on) acc = k == 0 ? f32x16_t{} : product(Pm, Q);
    if (k == 0) {
      for (int i = tid; i < R * LD; i += 256) Pm[i] = Q[i];
      __syncthreads();
    } else {
      __syncthreads();  // every wave has read P~
      store(Pm, acc, 1.f);
    }
    if (k + 1 == g.steps) break;
    if (on) acc = product(S, Q);
    store(X, acc, 1.f);
    if (on) acc = product(Q, X);
    store(S, acc, g.a2[k]);  // S was last read before X's barrier
  }
  for (int i = tid; i < R * R; i += 256) Sg[i] = Pm[(i / R) * LD + i % R];
}

}  // namespace

hipError_t launch_polar_small(const PolarSmallArgs& g, hipStream_t s) {
  if (g.P <= 0) return hipSuccess;
  if (g.steps < 1 || g.steps > 16) return hipErrorInvalidValue;
  if (g.r == 32) hipLaunchKernelGGL(k_polar_small<32>, dim3(g.P), dim3(256), 0, s, g);
  else if (g.r == 64) hipLaunchKernelGGL(k_polar_small<64>, dim3(g.P), dim3(256), 0, s, g);
  else return hipErrorInvalidValue;
  return hipGetLastError();
}

hipError_t launch_sym(const SymArgs& g, hipStream_t s) {
  if (g.P <= 0) return hipSuccess;
  if (g.r < 32 || g.r % 32 || g.r > 1024 || (g.batch != g.P && !(g.batch == 2 * g.P && g.A2))) return hipErrorInvalidValue;
  const int n64 = (g.r + 63) / 64, t64 = n64 * (n64 + 1) / 2, n32 = g.r / 32, t32 = n32 * (n32 + 1) / 2;
  auto grid = [&](int tiles) { return dim3((unsigned)(((int64_t)tiles * g.batch + 7) / 8 * 8)); };
  // Tile and wave count, measured per launch (us; 32 x 32 with four waves, with
  // two, 64 x 64):
  //   r = 256, 3 matrices (108 / 30 tiles)      4.1    4.4    7.1
  //   r = 384, 8 matrices (624 / 168)           7.3    6.5    7.7
  //   r = 512, 11 matrices (1496 / 396)        14.8   15.3   12.7
  //   r = 512, 16 matrices (2176 / 576)        20.5   17.6   19.0
  //   r = 512, 32 matrices (4352 / 1152)       35.7   29.9   30.4
  // Small launches want K split four ways; 64 x 64 tiles load half the bytes
  // per product but only two of their workgroups fit a CU, so they win where
  // one round of 512 holds them and the chip is filled.  (The split k_gemm_x3
  // took 10.3, 23 and 36 us at 3 of 256, 16 and 32 of 512.)
  const int64_t w64 = (int64_t)t64 * g.batch, w32 = (int64_t)t32 * g.batch;
  if (g.r % 64 == 0 && w64 >= 256 && w64 <= 512)
    hipLaunchKernelGGL((k_sym<2, 4, 1>), grid(t64), dim3(256), 0, s, g);
  else if (w32 < 400)
    hipLaunchKernelGGL((k_sym<1, 4, 2>), grid(t32), dim3(256), 0, s, g);
  else
    hipLaunchKernelGGL((k_sym<1, 2, 4>), grid(t32), dim3(128), 0, s, g);
  return hipGetLastError();
}

hipError_t launch_sym_split(const float* S, int P, int r, const float* part, uint16_t* C, float* inv_nu,
                            float* inv_nu2, hipStream_t s) {
  if (P <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_sym_split, dim3((r * r / 8 + 255) / 256, P), dim3(256), 0, s, S, r, part, (r + 15) / 16, C,
                     inv_nu, inv_nu2);
  return hipGetLastError();
}

}  // namespace mapl
