// Gradient of the anchor table (Sec. 3.2: E_small is trainable, Eq. 3).
// Every token contributes a gradient row g[t] (from the GEMM kernels) to the
// table row of its id; the rows are summed per id in a fixed order, so the
// result is reproducible bit for bit (no floating-point atomics):
//   1. the (id, token) pairs ordered so that equal ids are adjacent and keep
//      their token order.  Up to 32768 tokens (anchor_sort_fits): a bin per 256 ids, one
//      workgroup per bin, beside the call's other preparation
//      (k_anchor_prep); longer lists by a stable LSD radix sort, 8-bit digits
//      (per-tile digit histograms, one exclusive scan, a stable scatter).
//      Ranks come from wave ballots in both;
//   2. a segmented sum over the sorted order in 64-position sub-chunks, one
//      wave each, walking its positions in order; a segment that crosses a
//      sub-chunk boundary leaves its pieces in per-sub-chunk slots;
//   3. a fix-up, one workgroup per segment that crosses sub-chunks, adding
//      its pieces in a fixed order (four interleaved wave sums, then the
//      waves in order).
// Zipf-distributed ids make a few rows very long (id 0 takes about a seventh
// of the tokens); the sub-chunk split keeps every wave's share at 64 rows.
#include "common.hpp"
#include "kernels.hpp"

namespace mapl {

namespace {

constexpr int RS_THREADS = 256, RS_TILE = 512, RS_ROUNDS = RS_TILE / RS_THREADS;
constexpr int SEG = 64;  // sorted positions per sub-chunk

// The preparation of one call as one launch of 1024-thread workgroups, by
// block: the sort (one per bin of ids), then the padded or projected
// companion W, then the zeroing of dA.  Each was a launch of its own of 3 to
// 6 us, and the radix sort six (T = 8192: 25 us).
constexpr int AP_THREADS = 1024, AP_WAVES = AP_THREADS / 64;

// Bin b of the sort: ids with id % nbins == b (nbins a power of two, at
// least V / 256, so id / nbins has 8 bits), or b == nbins for ids outside
// [0, V), which go last as 0x7fffffff.  The workgroup reads every id (they
// sit in the L2: 32 KB at T = 8192), so it knows its offset in the result
// and lists its own tokens in order without any exchange between workgroups;
// the list (all n tokens in the worst case) is then placed by its 8-bit
// digit: the waves' counts, their scan (digit-major), and each wave's
// positions 64 at a time, lanes of equal digit ranked by ballots.
template <int RPT>
__device__ __forceinline__ void sort_bin(const AnchorPrepArgs& a, int b, uint32_t* list, uint32_t (*cnt)[256], int* tot) {
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int base = wave * 64 * RPT + lane;
  const int sh = __builtin_ctz(a.nbins);
  int x[RPT];
#pragma unroll
  for (int j = 0; j < RPT; ++j) x[j] = base + 64 * j < a.n ? a.ids[base + 64 * j] : -1;
  auto bin = [&](int id) { return (unsigned)id < (unsigned)a.V ? id & (a.nbins - 1) : a.nbins; };
  int own = 0, lower = 0;
#pragma unroll
  for (int j = 0; j < RPT; ++j) {
    const bool ok = base + 64 * j < a.n;
    const int q = bin(x[j]);
    own += __popcll(__ballot(ok && q == b));
    lower += __popcll(__ballot(ok && q < b));
  }
  if (lane == 0) {
    tot[wave] = own;
    tot[AP_WAVES + wave] = lower;
  }
  for (int i = tid; i < AP_WAVES * 256; i += AP_THREADS) (&cnt[0][0])[i] = 0;
  __syncthreads();
  int at = 0, m = 0, off = 0;
#pragma unroll
  for (int w = 0; w < AP_WAVES; ++w) {
    at += w < wave ? tot[w] : 0;
    m += tot[w];
    off += tot[AP_WAVES + w];
  }
  if (m == 0) return;  // workgroup-uniform
  const uint64_t below = (1ull << lane) - 1ull;
#pragma unroll
  for (int j = 0; j < RPT; ++j) {
    const bool mine = base + 64 * j < a.n && bin(x[j]) == b;
    const uint64_t sel = __ballot(mine);
    const uint32_t dg = b < a.nbins ? (uint32_t)x[j] >> sh : 0u;
    if (mine) list[at + __popcll(sel & below)] = dg << 24 | (uint32_t)(base + 64 * j);
    at += __popcll(sel);
  }
  __syncthreads();
  const int per = (m + AP_THREADS - 1) / AP_THREADS * 64, i0 = wave * per, i1 = min(m, i0 + per);
  // lanes of lane 0's digit as one addition: additions to one word are done
  // one by one (nine tokens in ten of one id: T = 32768, V = 32000: the
  // call 96.5 us that way, 77.2 so)
  for (int i = i0 + lane; i < i1; i += 64) {
    const uint32_t dg = list[i] >> 24, d0 = __builtin_amdgcn_readfirstlane(dg);
    const uint64_t same = __ballot(dg == d0);
    if (lane == 0) atomicAdd(&cnt[wave][d0], (uint32_t)__popcll(same));
    else if (dg != d0) atomicAdd(&cnt[wave][dg], 1u);
  }
  __syncthreads();
  // exclusive offsets, digit-major: thread d < 256 its digit's total, a scan
  // over the digits by wave shuffles, then the waves in order
  uint32_t sum = 0;
  if (tid < 256) {
#pragma unroll
    for (int w = 0; w < AP_WAVES; ++w) sum += cnt[w][tid];
  }
  uint32_t inc = sum;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const uint32_t v = __shfl_up(inc, o, WAVE);
    if (lane >= o) inc += v;
  }
  if (tid < 256 && lane == 63) tot[wave] = (int)inc;
  __syncthreads();
  if (tid < 256) {
    uint32_t run = inc - sum;
    for (int w = 0; w < wave; ++w) run += (uint32_t)tot[w];
#pragma unroll
    for (int w = 0; w < AP_WAVES; ++w) {
      const uint32_t c = cnt[w][tid];
      cnt[w][tid] = run;
      run += c;
    }
  }
  __syncthreads();
  uint32_t* mine = cnt[wave];
  for (int i = i0; i < i1; i += 64) {  // wave-uniform
    const bool ok = i + lane < i1;
    const uint32_t e = ok ? list[i + lane] : 0u, dg = e >> 24;
    uint64_t peers = __ballot(ok);
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const bool bit = (dg >> k) & 1u;
      const uint64_t set = __ballot(bit);
      peers &= bit ? set : ~set;
    }
    const uint32_t pos = mine[dg];
    __builtin_amdgcn_wave_barrier();  // every lane has read its digit's position
    if (ok && (peers & below) == 0) mine[dg] = pos + (uint32_t)__popcll(peers);
    __builtin_amdgcn_wave_barrier();
    if (ok) {
      const int p = off + (int)pos + __popcll(peers & below);
      a.skey[p] = b < a.nbins ? (int32_t)(dg << sh | (uint32_t)b) : 0x7fffffff;
      a.sval[p] = (int32_t)(e & 0xFFFFFFu);
    }
  }
}

// W tile rows i0 .. i0+15, columns c0 .. c0+15 of bf16(B U~) (U~ = bf16(U)
// where it enters the matrix units), rows from k on zero: the sixteen waves
// take every sixteenth 32-wide k-step and their partial tiles are summed in
// wave order.
__device__ __forceinline__ void proj_tile(const AnchorPrepArgs& a, int i0, int c0, float* part) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, quad = lane >> 4;
  const int row = min(i0 + (lane & 15), a.k - 1), c = c0 + (lane & 15);
  f32x4_t acc = f32x4_t{};
  for (int kb = 32 * wave; kb < a.d; kb += 32 * AP_WAVES) {
    const uint4 p = *(const uint4*)(a.B + (int64_t)row * a.d + kb + 8 * quad);
    float q[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) q[e] = a.U[(int64_t)(kb + 8 * quad + e) * a.K + c];
    acc = mfma16x16x32(p, make_uint4(pack_bf2(q[0], q[1]), pack_bf2(q[2], q[3]), pack_bf2(q[4], q[5]), pack_bf2(q[6], q[7])),
                       acc);
  }
#pragma unroll
  for (int e = 0; e < 4; ++e) part[wave * 256 + (4 * quad + e) * 16 + (lane & 15)] = acc[e];
  __syncthreads();
  if (tid < 256) {
    float v = part[tid];
#pragma unroll
    for (int w = 1; w < AP_WAVES; ++w) v += part[w * 256 + tid];
    const int i = i0 + (tid >> 4);
    if (i < a.kp) a.W[(int64_t)i * a.K + c0 + (tid & 15)] = i < a.k ? (bf16_t)f2bf(v) : (bf16_t)0;
  }
}

template <int RPT>
__global__ __launch_bounds__(AP_THREADS) void k_anchor_prep(AnchorPrepArgs a) {
  __shared__ uint32_t xch[RPT > 4 ? RPT * AP_THREADS : 4 * AP_THREADS];  // also proj_tile's partial tiles
  __shared__ uint32_t cnt[AP_WAVES][256];
  __shared__ int tot[2 * AP_WAVES];
  int b = blockIdx.x;
  if constexpr (RPT > 0) {
    if (b <= a.nbins) {
      sort_bin<RPT>(a, b, xch, cnt, tot);
      return;
    }
    b -= a.nbins + 1;
  }
  if (b < a.wblocks) {
    if (a.U) {
      const int nc = a.K / 16;
      proj_tile(a, b / nc * 16, b % nc * 16, (float*)xch);
    } else {  // W[i][c] = B[i][c], rows from k on zero; 8 columns per thread
      const int64_t e = ((int64_t)b * AP_THREADS + threadIdx.x) * 8;
      if (e < (int64_t)a.kp * a.K)
        *(uint4*)(a.W + e) = e < (int64_t)a.k * a.K ? *(const uint4*)(a.B + e) : make_uint4(0u, 0u, 0u, 0u);
    }
    return;
  }
  b -= a.wblocks;
  const int64_t i = (int64_t)b * AP_THREADS + threadIdx.x;
  if (i < a.zero16) ((uint4*)a.dA)[i] = make_uint4(0u, 0u, 0u, 0u);
}

__global__ __launch_bounds__(RS_THREADS) void k_radix_hist(const int32_t* __restrict__ keys, int n, int shift,
                                                           int nb, int* __restrict__ hist) {
  __shared__ int h[256];
  h[threadIdx.x] = 0;
  __syncthreads();
  const int base = blockIdx.x * RS_TILE;
  for (int j = 0; j < RS_ROUNDS; ++j) {
    const int i = base + j * RS_THREADS + threadIdx.x;
    if (i < n) atomicAdd(&h[((uint32_t)keys[i] >> shift) & 255u], 1);
  }
  __syncthreads();
  hist[threadIdx.x * nb + blockIdx.x] = h[threadIdx.x];
}

// Exclusive scan, in place, of m counts (digit-major: all tiles of digit 0,
// then digit 1, ...), by one block: chunks of 8192 counts move through LDS
// with coalesced loads and stores, each thread scans 8 consecutive counts,
// the 1024 thread sums are scanned in LDS, and a carry links the chunks.
__global__ __launch_bounds__(1024) void k_radix_scan(int* __restrict__ hist, int m) {
  constexpr int PER = 8, CH = 1024 * PER;
  __shared__ int buf[CH];
  __shared__ int part[1024];
  const int tid = threadIdx.x;
  int carry = 0;
  for (int base = 0; base < m; base += CH) {
#pragma unroll
    for (int j = 0; j < PER; ++j) {
      const int i = base + j * 1024 + tid;
      buf[j * 1024 + tid] = i < m ? hist[i] : 0;
    }
    __syncthreads();
    int sum = 0;
#pragma unroll
    for (int j = 0; j < PER; ++j) sum += buf[tid * PER + j];
    part[tid] = sum;
    __syncthreads();
    for (int o = 1; o < 1024; o <<= 1) {
      const int v = tid >= o ? part[tid - o] : 0;
      __syncthreads();
      part[tid] += v;
      __syncthreads();
    }
    int run = carry + (tid ? part[tid - 1] : 0);
#pragma unroll
    for (int j = 0; j < PER; ++j) {
      const int c = buf[tid * PER + j];
      buf[tid * PER + j] = run;
      run += c;
    }
    const int total = part[1023];
    __syncthreads();
#pragma unroll
    for (int j = 0; j < PER; ++j) {
      const int i = base + j * 1024 + tid;
      if (i < m) hist[i] = buf[j * 1024 + tid];
    }
    carry += total;
    __syncthreads();  // buf and part are reused by the next chunk
  }
}

// Stable scatter of one tile: keys are taken in rounds of 256 in input
// order; within a round, lanes of a wave with the same digit are ranked by
// ballots, waves in order, and rounds in order, so equal digits keep their
// input order.  vals == null stands for vals[i] = i.
__global__ __launch_bounds__(RS_THREADS) void k_radix_scatter(const int32_t* __restrict__ keys,
                                                              const int32_t* __restrict__ vals, int n, int shift,
                                                              int nb, const int* __restrict__ offs,
                                                              int32_t* __restrict__ keys_out,
                                                              int32_t* __restrict__ vals_out) {
  __shared__ int base[256];
  __shared__ int wcnt[4][256];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  base[tid] = offs[tid * nb + blockIdx.x];
#pragma unroll
  for (int w = 0; w < 4; ++w) wcnt[w][tid] = 0;
  __syncthreads();
  const int b0 = blockIdx.x * RS_TILE;
  for (int j = 0; j < RS_ROUNDS; ++j) {
    const int i = b0 + j * RS_THREADS + tid;
    const bool ok = i < n;
    const int key = ok ? keys[i] : 0;
    const int val = ok ? (vals ? vals[i] : i) : 0;
    const int dg = (int)(((uint32_t)key >> shift) & 255u);
    uint64_t peers = __ballot(ok);
#pragma unroll
    for (int b = 0; b < 8; ++b) {
      const bool bit = (dg >> b) & 1;
      const uint64_t m = __ballot(bit);
      peers &= bit ? m : ~m;
    }
    const uint64_t lower = peers & ((1ull << lane) - 1ull);
    if (ok && lower == 0) wcnt[wave][dg] = __popcll(peers);
    __syncthreads();
    if (ok) {
      int pos = base[dg] + __popcll(lower);
      for (int w = 0; w < wave; ++w) pos += wcnt[w][dg];
      keys_out[pos] = key;
      vals_out[pos] = val;
    }
    __syncthreads();
    base[tid] += (wcnt[0][tid] + wcnt[1][tid]) + (wcnt[2][tid] + wcnt[3][tid]);
#pragma unroll
    for (int w = 0; w < 4; ++w) wcnt[w][tid] = 0;
    __syncthreads();
  }
}

// row[c] (+)= scale acc[q] for the lane's columns c = lane + 64 q < k
template <int NC>
__device__ __forceinline__ void seg_store(float* __restrict__ row, const float (&acc)[NC], int k, int lane,
                                          float scale, int add) {
#pragma unroll
  for (int q = 0; q < NC; ++q) {
    const int c = lane + 64 * q;
    if (c < k) row[c] = add ? row[c] + scale * acc[q] : scale * acc[q];
  }
}

// One wave per sub-chunk of 64 sorted positions: the rows of each segment
// (run of equal ids) are summed in sorted order; a segment wholly inside the
// sub-chunk is written to dA, a piece that continues from the previous
// sub-chunk goes to the head slot (flagged when it also continues into the
// next), a piece that starts here and continues goes to the tail slot.
// NC columns per lane (k <= 64 NC); 64 / NC rows are requested at a time.
template <int NC>
__global__ __launch_bounds__(256) void k_seg_partial(AnchorSegArgs a) {
  constexpr int BR = 64 / NC;
  __shared__ float stage[4][64 * 64];  // each wave its own part: no barrier
  const int lane = threadIdx.x & 63;
  // wave-uniform, and known to be: the walk below branches on scalars
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), s = blockIdx.x * 4 + wave;
  if (s >= a.nsub) return;
  const int p0 = s * SEG, np = min(a.n - p0, SEG);
  // lane u: position p0 + u, its id and token; a position ends a segment
  // where the next id differs (-1 and -2 mark "none"; ids are non-negative)
  const int idl = lane < np ? a.skey[p0 + lane] : -2;
  const int tl = lane < np ? a.sval[p0 + lane] : 0;
  const int prev_id = p0 > 0 ? __builtin_amdgcn_readfirstlane(a.skey[p0 - 1]) : -1;
  const int next_id = p0 + np < a.n ? __builtin_amdgcn_readfirstlane(a.skey[p0 + np]) : -1;
  int nid = __shfl_down(idl, 1, WAVE);
  if (lane == np - 1) nid = next_id;
  const uint64_t ends = __ballot(lane < np && (nid != idl || lane == np - 1));
  // the first segment continues the previous sub-chunk's (its sum goes to the
  // head slot), the last goes on in the next one's (tail slot)
  const int id0 = __builtin_amdgcn_readlane(idl, 0), idn = __builtin_amdgcn_readlane(idl, np - 1);
  const bool before = prev_id == id0, after = next_id == idn;
  const bool through = before && after && __builtin_ctzll(ends) == np - 1;  // one segment, from before to after
  if (lane == 0) {
    a.head_id[s] = before ? id0 : -1;
    a.head_thru[s] = through ? 1 : 0;
    a.tail_id[s] = after && !through ? idn : -1;
  }
  float* rows = stage[wave];
  float acc[NC];
#pragma unroll
  for (int q = 0; q < NC; ++q) acc[q] = 0.f;
  // Each segment's sum has one store, its place chosen by scalar selects: a
  // lone wave pays some 30 cycles per branch taken, and a walk with a branch
  // per row and place took 190 to 430 cycles per row (T = 8192, k = 64: 14 us
  // of the launch's 18; 11.5 in all now).
  auto walk = [&](auto addc) {
    constexpr bool ADD = decltype(addc)::value;
    bool first = before;  // the next sum is the head piece
    for (int pb = 0; pb < np; pb += BR) {
      // the batch's rows go to LDS straight from memory, all on their way
      // before the first is used: 16 bytes per lane and load
      static_assert(BR * NC == 64, "a batch is 4096 floats");
#pragma unroll 1
      for (int i = 0; i < 16; ++i) {
        const int f = i * 256 + lane * 4, u = f / (64 * NC), c = f % (64 * NC);
        const int t = __shfl(tl, min(pb + u, np - 1), WAVE);
        const float* src = a.g + (int64_t)t * a.ldg + min(c, (int)a.ldg - 4);  // columns past k are not stored
        __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)src,
                                         (__attribute__((address_space(3))) void*)(rows + i * 256), 16, 0, 0);
      }
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      const int pe = min(pb + BR, np);
      float cur[NC];
#pragma unroll
      for (int q = 0; q < NC; ++q) cur[q] = rows[q * 64 + lane];
      for (int p = pb; p < pe;) {
        const int end = p + __builtin_ctzll(ends >> p);  // the segment's last position
        const int stop = min(end, pe - 1);
        for (; p <= stop; ++p) {
          const float* nx = rows + min(p - pb + 1, BR - 1) * NC * 64;
#pragma unroll
          for (int q = 0; q < NC; ++q) {
            acc[q] += cur[q];
            cur[q] = nx[q * 64 + lane];
          }
        }
        if (end > stop) break;  // it goes on in the next batch
        const int id = __builtin_amdgcn_readlane(idl, end);
        const bool last = after && end == np - 1, piece = first || last;
        const bool ok = piece || (unsigned)id < (unsigned)a.V;  // an id outside [0, V) is a caller error: skipped
        float* row = piece ? (first ? a.headp : a.tailp) + (int64_t)s * a.k : a.dA + (int64_t)id * a.k;
        const float scale = piece ? 1.f : a.scale;
#pragma unroll
        for (int q = 0; q < NC; ++q) {
          const int c = lane + 64 * q;
          if (c < (ok ? a.k : 0)) {
            float x = scale * acc[q];
            if (ADD) x += piece ? 0.f : row[c];
            row[c] = x;
          }
          acc[q] = 0.f;
        }
        first = false;
      }
    }
  };
  if (a.accumulate) walk(std::true_type{});
  else walk(std::false_type{});
}

// Segments that cross sub-chunk boundaries, one workgroup per sub-chunk s
// whose tail piece starts one: its head pieces are those of sub-chunks
// s+1 .. e, e the first that does not continue further.  Wave w sums the
// pieces s+1+w, s+5+w, ... in order (eight requested at a time); the sum is
// tail + wave 0 + wave 1 + wave 2 + wave 3, a fixed order.
template <int NC>
__global__ __launch_bounds__(256) void k_seg_fixup(AnchorSegArgs a) {
  constexpr int FB = 8;
  __shared__ float part[4][64 * NC];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int s = blockIdx.x;
  const int id = a.tail_id[s];
  if (id < 0 || id >= a.V) return;  // workgroup-uniform
  // e: the first head piece after s that ends the segment (exists: a tail
  // piece continues into sub-chunk s + 1, and the last sub-chunk's head
  // piece never continues)
  int e = a.nsub - 1;
  for (int b = s + 1; b < a.nsub; b += 64) {
    const int i = b + lane;
    const uint64_t m = __ballot(i < a.nsub && a.head_thru[i] == 0);
    if (m) {
      e = b + __builtin_ctzll(m);
      break;
    }
  }
  float acc[NC];
#pragma unroll
  for (int q = 0; q < NC; ++q) acc[q] = 0.f;
  for (int b = s + 1 + wave; b <= e; b += 4 * FB) {
    float v[FB][NC];
#pragma unroll
    for (int u = 0; u < FB; ++u) {
      const int s2 = min(b + 4 * u, e);
#pragma unroll
      for (int q = 0; q < NC; ++q) {
        const int c = lane + 64 * q;
        v[u][q] = c < a.k ? a.headp[(int64_t)s2 * a.k + c] : 0.f;
      }
    }
#pragma unroll
    for (int u = 0; u < FB; ++u)
      if (b + 4 * u <= e) {
#pragma unroll
        for (int q = 0; q < NC; ++q) acc[q] += v[u][q];
      }
  }
#pragma unroll
  for (int q = 0; q < NC; ++q) part[wave][lane + 64 * q] = acc[q];
  __syncthreads();
  if (wave != 0) return;
  float tot[NC];
#pragma unroll
  for (int q = 0; q < NC; ++q) {
    const int c = lane + 64 * q;
    float x = c < a.k ? a.tailp[(int64_t)s * a.k + c] : 0.f;
    x += part[0][c];
    x += part[1][c];
    x += part[2][c];
    x += part[3][c];
    tot[q] = x;
  }
  seg_store<NC>(a.dA + (int64_t)id * a.k, tot, a.k, lane, a.scale, a.accumulate);
}

template <int NC>
void launch_segsum_nc(const AnchorSegArgs& a, hipStream_t s) {
  hipLaunchKernelGGL(k_seg_partial<NC>, dim3((a.nsub + 3) / 4), dim3(256), 0, s, a);
  hipLaunchKernelGGL(k_seg_fixup<NC>, dim3(a.nsub), dim3(256), 0, s, a);
}

}  // namespace

// A list of 32768 tokens fits the LDS beside the counts; 512 bins (V up to
// 131072) read the ids 512 times, 64 MB from the L2s at most.  A single bin
// (V <= 256) scatters every pair from one CU, where the radix sort needs one
// pass: the call (k = 32) with the bin / the radix sort, us: T = 8192: 27.5 /
// 32.7, 12000: 34.9 / 33.5, 16384: 38.5 / 34.2, 32768: 61.8 / 40.7; with two
// bins (V = 512) 32768: 45.9 / 57.4.
bool anchor_sort_fits(int64_t n, int64_t V) { return n <= (V <= 256 ? 10 : 32) * AP_THREADS && V <= 131072; }

hipError_t launch_anchor_prep(const AnchorPrepArgs& a, hipStream_t s) {
  AnchorPrepArgs g = a;
  const bool sort = a.skey != nullptr;
  if (sort && !anchor_sort_fits(a.n, a.V)) return hipErrorInvalidValue;
  if (a.W && (a.K % 16 || a.kp % 16 || a.d % 32)) return hipErrorInvalidValue;
  g.wblocks = !a.W ? 0 : a.U ? (a.kp / 16) * (a.K / 16) : (int)(((int64_t)a.kp * a.K / 8 + AP_THREADS - 1) / AP_THREADS);
  g.nbins = 1;
  while (g.nbins * 256 < g.V) g.nbins *= 2;
  const int64_t blocks = (sort ? g.nbins + 1 : 0) + g.wblocks + (a.zero16 + AP_THREADS - 1) / AP_THREADS;
  if (blocks <= 0) return hipSuccess;
  const dim3 grid((unsigned)blocks), thr(AP_THREADS);
  if (!sort) hipLaunchKernelGGL(k_anchor_prep<0>, grid, thr, 0, s, g);
  else if (a.n <= 2 * AP_THREADS) hipLaunchKernelGGL(k_anchor_prep<2>, grid, thr, 0, s, g);
  else if (a.n <= 8 * AP_THREADS) hipLaunchKernelGGL(k_anchor_prep<8>, grid, thr, 0, s, g);
  else if (a.n <= 16 * AP_THREADS) hipLaunchKernelGGL(k_anchor_prep<16>, grid, thr, 0, s, g);
  else hipLaunchKernelGGL(k_anchor_prep<32>, grid, thr, 0, s, g);
  return hipGetLastError();
}

int radix_tiles(int n) { return (n + RS_TILE - 1) / RS_TILE; }

hipError_t launch_sort_ids(const int32_t* ids, int n, int passes, int* hist, int32_t* k0, int32_t* v0, int32_t* k1,
                           int32_t* v1, const int32_t** skey, const int32_t** sval, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  const int nb = radix_tiles(n);
  const int32_t* kin = ids;
  const int32_t* vin = nullptr;
  int32_t* kb[2] = {k0, k1};
  int32_t* vb[2] = {v0, v1};
  for (int p = 0; p < passes; ++p) {
    hipLaunchKernelGGL(k_radix_hist, dim3(nb), dim3(RS_THREADS), 0, s, kin, n, 8 * p, nb, hist);
    hipLaunchKernelGGL(k_radix_scan, dim3(1), dim3(1024), 0, s, hist, 256 * nb);
    hipLaunchKernelGGL(k_radix_scatter, dim3(nb), dim3(RS_THREADS), 0, s, kin, vin, n, 8 * p, nb, hist, kb[p & 1],
                       vb[p & 1]);
    kin = kb[p & 1];
    vin = vb[p & 1];
  }
  *skey = kin;
  *sval = vin;
  return hipGetLastError();
}

hipError_t launch_anchor_segsum(const AnchorSegArgs& a, hipStream_t s) {
  if (a.n <= 0) return hipSuccess;
  if (a.k <= 64)
    launch_segsum_nc<1>(a, s);
  else if (a.k <= 128)
    launch_segsum_nc<2>(a, s);
  else if (a.k <= 256)
    launch_segsum_nc<4>(a, s);
  else if (a.k <= 512)
    launch_segsum_nc<8>(a, s);
  else
    return hipErrorInvalidValue;
  return hipGetLastError();
}

int anchor_sub_chunks(int n) { return (n + SEG - 1) / SEG; }

}  // namespace mapl
