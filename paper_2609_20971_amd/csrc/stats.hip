// Stage 1: per-key-block statistics (Sec. 3.1; Algorithm 1, statistics loops).
//
// stats_kernel: one workgroup per (KV head, key block) streams the block's
// B x 128 bf16 keys from HBM exactly once, coalesced (16 lanes cover one
// 256-byte row), keeps them in registers, and produces the centroid (mean over
// the block's actual key count) and the radius (max L2 distance to the
// centroid), plus the select-ready f16 copy of the centroid.
//
// quantile_kernel: one workgroup per KV head finds the head's 0.5 / 0.9 radius
// quantiles with an in-LDS histogram over its M radii and writes beta and
// the select-ready uplift of every block.  It is a separate launch because a
// device-wide "last workgroup" hand-off would need an agent-scope release per
// workgroup, which on a multi-XCD gfx950 writes back the whole L2 each time.
#include "rbs_device.hpp"
#include "rbs_launch.hpp"

namespace rbs {

constexpr int kStatsThreads = 256;

// Maximum of x over the 64 lanes, in every lane.
__device__ __forceinline__ uint32_t wave_max_u(uint32_t x) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    const uint32_t y = (uint32_t)__shfl_xor((int)x, off, kWave);
    x = y > x ? y : x;
  }
  return x;
}

// Block blockIdx.x of all the sequences' blocks (sequence s owns blocks
// t.blk[s] .. t.blk[s+1]-1 and tokens t.tok[s] .. t.tok[s+1]-1), KV head blockIdx.y.
template <int BS>
__global__ __launch_bounds__(kStatsThreads) void stats_kernel(const uint16_t* __restrict__ K, int64_t kv_head,
                                                             int64_t kv_tok, const SeqTable t,
                                                             float* __restrict__ centroids,
                                                             float* __restrict__ radii,
                                                             _Float16* __restrict__ cent16,
                                                             float* __restrict__ cnorm, float sel_scale) {
  constexpr int kRowsPerThread = BS / 16;
  __shared__ float red[4][kHeadDim];
  __shared__ float red_r[4];

  const int bg = blockIdx.x, g = blockIdx.y;
  const int sq = seq_of(t.blk, t.n, bg);
  const int b = bg - t.blk[sq];
  const int M = t.blk[t.n];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int chunk = tid & 15;  // 8 consecutive dims: 8*chunk .. 8*chunk+7
  const int rg = tid >> 4;     // row group: rows rg, rg+16, ...
  const int row0 = b * BS;
  const int nb = min(BS, t.tok[sq + 1] - t.tok[sq] - row0);
  const uint16_t* kb = K + g * kv_head + (int64_t)(t.tok[sq] + row0) * kv_tok + chunk * 8;

  uint4 raw[kRowsPerThread];
#pragma unroll
  for (int k = 0; k < kRowsPerThread; ++k) {
    const int r = rg + 16 * k;
    raw[k] = r < nb ? *reinterpret_cast<const uint4*>(kb + r * kv_tok) : make_uint4(0u, 0u, 0u, 0u);
  }

  // Column sums: own rows, then the four row groups of this wave, then waves.
  float s[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int k = 0; k < kRowsPerThread; ++k) {
    float f[8];
    unpack8(raw[k], f);
#pragma unroll
    for (int e = 0; e < 8; ++e) s[e] += f[e];
  }
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    s[e] += wave_xor_f(s[e], 16);
    s[e] += wave_xor_f(s[e], 32);
  }
  if (lane < 16) {
#pragma unroll
    for (int e = 0; e < 8; ++e) red[wave][chunk * 8 + e] = s[e];
  }
  __syncthreads();
  float c[8];
  const float count = (float)nb;
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const int x = chunk * 8 + e;
    c[e] = (((red[0][x] + red[1][x]) + red[2][x]) + red[3][x]) / count;
  }

  // Radius: squared distance per row (16 lanes share a row), max over rows.
  float best = 0.f;
#pragma unroll
  for (int k = 0; k < kRowsPerThread; ++k) {
    float f[8];
    unpack8(raw[k], f);
    float d2 = 0.f;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const float t = f[e] - c[e];
      d2 = fmaf(t, t, d2);
    }
    d2 += wave_xor_f(d2, 1);
    d2 += wave_xor_f(d2, 2);
    d2 += wave_xor_f(d2, 4);
    d2 += wave_xor_f(d2, 8);
    if (rg + 16 * k < nb) best = fmaxf(best, d2);
  }
  best = fmaxf(best, wave_xor_f(best, 16));
  best = fmaxf(best, wave_xor_f(best, 32));
  if (lane == 0) red_r[wave] = best;
  __syncthreads();

  const size_t blk = (size_t)g * M + bg;
  // Norm of the select-ready (scaled) centroid: the selector bounds its
  // logits with it (Cauchy-Schwarz).  Lanes 0-15 of wave 0 hold the 16 chunks.
  if (wave == 0) {
    float n2 = 0.f;
#pragma unroll
    for (int e = 0; e < 8; ++e) n2 = fmaf(c[e] * sel_scale, c[e] * sel_scale, n2);
    n2 += wave_xor_f(n2, 1);
    n2 += wave_xor_f(n2, 2);
    n2 += wave_xor_f(n2, 4);
    n2 += wave_xor_f(n2, 8);
    if (lane == 0) cnorm[blk] = sqrtf(n2);
  }
  if (tid < 16) {
    float4* dst = reinterpret_cast<float4*>(centroids + blk * kHeadDim + chunk * 8);
    dst[0] = make_float4(c[0], c[1], c[2], c[3]);
    dst[1] = make_float4(c[4], c[5], c[6], c[7]);
    f16x8 h;
#pragma unroll
    for (int e = 0; e < 8; ++e) h[e] = (_Float16)(c[e] * sel_scale);
    *reinterpret_cast<f16x8*>(cent16 + blk * kHeadDim + chunk * 8) = h;
  }
  if (tid == 0) radii[blk] = sqrtf(fmaxf(fmaxf(red_r[0], red_r[1]), fmaxf(red_r[2], red_r[3])));
}

// Coordinate-wise box of every key block for the Quest-style supporting
// selector (App. geometry, Eq. quest_box): per dimension the minimum a and
// maximum u over the block's keys, written as centre (u + a)/2 and half-width
// (u - a)/2 (both exact in fp32 for bf16 inputs), plus f16 copies scaled by
// log2(e)/sqrt(d) for the selector's MFMA.  Same layout and row mapping as
// stats_kernel: one workgroup per (KV head, key block), 16 lanes per row.
template <int BS>
__global__ __launch_bounds__(kStatsThreads) void box_kernel(const uint16_t* __restrict__ K, int64_t kv_head,
                                                           int64_t kv_tok, int N, int M,
                                                           float* __restrict__ center, float* __restrict__ half,
                                                           _Float16* __restrict__ center16,
                                                           _Float16* __restrict__ half16, float sel_scale) {
  constexpr int kRowsPerThread = BS / 16;
  __shared__ float red_lo[4][kHeadDim];
  __shared__ float red_hi[4][kHeadDim];
  const int b = blockIdx.x, g = blockIdx.y;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int chunk = tid & 15, rg = tid >> 4;
  const int row0 = b * BS;
  const int nb = min(BS, N - row0);
  const uint16_t* kb = K + g * kv_head + (int64_t)row0 * kv_tok + chunk * 8;
  float lo[8], hi[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    lo[e] = INFINITY;
    hi[e] = -INFINITY;
  }
#pragma unroll
  for (int k = 0; k < kRowsPerThread; ++k) {
    const int r = rg + 16 * k;
    if (r < nb) {
      float f[8];
      unpack8(*reinterpret_cast<const uint4*>(kb + r * kv_tok), f);
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        lo[e] = fminf(lo[e], f[e]);
        hi[e] = fmaxf(hi[e], f[e]);
      }
    }
  }
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    lo[e] = fminf(lo[e], wave_xor_f(lo[e], 16));
    lo[e] = fminf(lo[e], wave_xor_f(lo[e], 32));
    hi[e] = fmaxf(hi[e], wave_xor_f(hi[e], 16));
    hi[e] = fmaxf(hi[e], wave_xor_f(hi[e], 32));
  }
  if (lane < 16) {
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      red_lo[wave][chunk * 8 + e] = lo[e];
      red_hi[wave][chunk * 8 + e] = hi[e];
    }
  }
  __syncthreads();
  if (tid < 16) {
    const size_t base = ((size_t)g * M + b) * kHeadDim + chunk * 8;
    f16x8 c16, h16;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int x = chunk * 8 + e;
      const float a = fminf(fminf(red_lo[0][x], red_lo[1][x]), fminf(red_lo[2][x], red_lo[3][x]));
      const float u = fmaxf(fmaxf(red_hi[0][x], red_hi[1][x]), fmaxf(red_hi[2][x], red_hi[3][x]));
      const float c = (u + a) * 0.5f, hw = (u - a) * 0.5f;
      center[base + e] = c;
      half[base + e] = hw;
      c16[e] = (_Float16)(c * sel_scale);
      h16[e] = (_Float16)(hw * sel_scale);
    }
    *reinterpret_cast<f16x8*>(center16 + base) = c16;
    *reinterpret_cast<f16x8*>(half16 + base) = h16;
  }
}

// KV head blockIdx.x of sequence blockIdx.y: the quantiles of that sequence's
// radii (its own prompt's distribution), by T threads holding PER radii each.
//
// The four order statistics wanted (ranks ka, ka + 1, kb, kb + 1; 0-based, a rank
// past M - 1 taken as M - 1) are found from one histogram: non-negative IEEE
// floats order like their bit patterns, so (bits - min) >> shift is a monotone
// map onto kBins bins; the keys of each wanted rank's bin (a few) are listed by
// their offset in it, and one wave per rank finds the value among them by bitwise
// bisection with ballots (any number of keys, so any distribution).
// Latency-bound, one workgroup per head: a chain of six barriers (the 8-bit
// radix passes that it replaces took some twenty).  Kernel time at M = 32, 256,
// 1024, 2048, 4096: 5.6, 7.0, 8.8, 12.2, 20.4 -> 5.0, 6.1, 6.1, 7.0, 7.6 us.
constexpr int kBins = 1024;

template <int T, int PER>
__global__ __launch_bounds__(T) void quantile_kernel(const float* __restrict__ radii, const SeqTable t,
                                                     float* __restrict__ beta, float* __restrict__ quantiles,
                                                     float* __restrict__ uplift, float sel_scale) {
  constexpr int NW = T / kWave;
  constexpr int kBinsPer = kBins / T;  // bins of a thread's share of the scan
  __shared__ uint32_t hist[kBins];
  __shared__ uint32_t list[4][T * PER];  // keys of each wanted rank's bin
  __shared__ uint32_t red[2][NW];
  __shared__ uint32_t wave_sum[NW];
  __shared__ uint32_t bin_of[4], below[4], listed[4];  // per rank: its bin, keys below the bin, keys listed
  __shared__ float order[4];
  const int g = blockIdx.x, sq = blockIdx.y, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int M = t.blk[sq + 1] - t.blk[sq];
  const size_t base = (size_t)g * t.blk[t.n] + t.blk[sq];
  const float* rg_radii = radii + base;

  // Keys (the last one again past the end), their range.
  uint32_t key[PER];
  uint32_t hi = 0u, lo_inv = 0u;  // max of bits, max of ~bits
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    key[k] = __float_as_uint(rg_radii[min(tid + k * T, M - 1)]);
    hi = key[k] > hi ? key[k] : hi;
    lo_inv = ~key[k] > lo_inv ? ~key[k] : lo_inv;
  }
#pragma unroll
  for (int k = 0; k < kBinsPer; ++k) hist[tid + k * T] = 0u;
  if (tid < 4) listed[tid] = 0u;
  hi = wave_max_u(hi);
  lo_inv = wave_max_u(lo_inv);
  if (lane == 0) {
    red[0][wave] = hi;
    red[1][wave] = lo_inv;
  }
  __syncthreads();
#pragma unroll
  for (int w = 0; w < NW; ++w) {
    hi = red[0][w] > hi ? red[0][w] : hi;
    lo_inv = red[1][w] > lo_inv ? red[1][w] : lo_inv;
  }
  const uint32_t lo = ~lo_inv, range = hi - lo;
  const int shift = range < (uint32_t)kBins ? 0 : 22 - __clz((int)range);  // range >> shift < 1024

#pragma unroll
  for (int k = 0; k < PER; ++k)
    if (tid + k * T < M) atomicAdd(&hist[(key[k] - lo) >> shift], 1u);
  __syncthreads();

  // Exclusive scan over the bins (thread tid: bins kBinsPer tid ..) and, in the
  // bin that holds it, each wanted rank.  Linear interpolation between order
  // statistics: h = (M - 1) p, done in integers so the ranks are exact.
  const int n1 = M - 1;
  const int k50 = n1 / 2, k90 = (9 * n1) / 10;
  const uint32_t rank[4] = {(uint32_t)k50, (uint32_t)min(k50 + 1, n1), (uint32_t)k90, (uint32_t)min(k90 + 1, n1)};
  uint32_t c[kBinsPer], own = 0u;
#pragma unroll
  for (int k = 0; k < kBinsPer; ++k) {
    c[k] = hist[kBinsPer * tid + k];
    own += c[k];
  }
  uint32_t incl = own;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const uint32_t v = (uint32_t)__shfl_up((int)incl, off, kWave);
    if (lane >= off) incl += v;
  }
  if (lane == 63) wave_sum[wave] = incl;
  __syncthreads();
  uint32_t excl = incl - own;
#pragma unroll
  for (int w = 0; w < NW; ++w) excl += w < wave ? wave_sum[w] : 0u;
#pragma unroll
  for (int k = 0; k < kBinsPer; ++k) {
#pragma unroll
    for (int r = 0; r < 4; ++r)
      if (excl <= rank[r] && rank[r] < excl + c[k]) {
        bin_of[r] = (uint32_t)(kBinsPer * tid + k);
        below[r] = excl;
      }
    excl += c[k];
  }
  __syncthreads();

#pragma unroll
  for (int k = 0; k < PER; ++k) {
    const uint32_t bin = (key[k] - lo) >> shift;
#pragma unroll
    for (int r = 0; r < 4; ++r)
      if (tid + k * T < M && bin == bin_of[r])
        list[r][atomicAdd(&listed[r], 1u)] = key[k] - lo - (bin << shift);
  }
  __syncthreads();
  // Wave r: the value of rank (rank[r] - below[r]) among its list -- the largest v
  // such that no more keys than that lie below it.
  if (wave < 4) {
    const uint32_t n = listed[wave], want = rank[wave] - below[wave];
    const uint32_t mine = list[wave][(uint32_t)lane < n ? lane : 0];
    uint32_t v = 0u;
    for (int bit = shift - 1; bit >= 0; --bit) {
      const uint32_t probe = v | (1u << bit);
      uint32_t less = (uint32_t)__popcll(__ballot((uint32_t)lane < n && mine < probe));
      for (uint32_t e = kWave + lane; e - lane < n; e += kWave)
        less += (uint32_t)__popcll(__ballot(e < n && list[wave][e < n ? e : 0] < probe));
      if (less <= want) v = probe;
    }
    v += lo + (bin_of[wave] << shift);
    if (lane == 0) order[wave] = __uint_as_float(v);
  }
  __syncthreads();

  const float f50 = (n1 % 2) ? 0.5f : 0.0f;
  const float f90 = (float)((9 * n1) % 10) / 10.0f;
  const float r_low = order[0] + f50 * (order[1] - order[0]);
  const float r_high = order[2] + f90 * (order[3] - order[2]);
  const bool spread = r_high > r_low;
  const float span = r_high - r_low;
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    const int e = tid + k * T;
    if (e < M) {
      const float r = __uint_as_float(key[k]);
      float bt;
      if (spread) bt = fminf(fmaxf((r - r_low) / span, 0.0f), 1.0f);
      else bt = r > r_low ? 1.0f : 0.0f;
      beta[base + e] = bt;
      uplift[base + e] = r * bt * sel_scale;
    }
  }
  if (tid == 0) {
    const size_t q = (size_t)sq * gridDim.x + g;
    quantiles[2 * q + 0] = r_low;
    quantiles[2 * q + 1] = r_high;
  }
}

// The select-ready summary from statistics computed elsewhere: one wave per
// (KV head, block) converts the fp32 centroid (scaled by log2(e)/sqrt(d)) to
// f16, the norm of the scaled centroid, and the uplift r_b beta_b
// log2(e)/sqrt(d) -- the values stats_kernel and quantile_kernel write, from
// the same fp32 inputs and with the same arithmetic.
__global__ __launch_bounds__(256) void summarize_kernel(const float* __restrict__ centroids,
                                                        const float* __restrict__ radii,
                                                        const float* __restrict__ beta, int64_t n_rows,
                                                        _Float16* __restrict__ cent16, float* __restrict__ uplift,
                                                        float* __restrict__ cnorm, float sel_scale) {
  const int lane = threadIdx.x & 63;
  const int64_t row = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);  // (KV head, block), head-major
  if (row >= n_rows) return;
  // Lanes 0-15 each hold 8 consecutive dimensions, as in stats_kernel.
  float n2 = 0.f;
  if (lane < 16) {
    const float4* src = reinterpret_cast<const float4*>(centroids + row * kHeadDim + lane * 8);
    const float4 a = src[0], b = src[1];
    const float c[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
    f16x8 h;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      n2 = fmaf(c[e] * sel_scale, c[e] * sel_scale, n2);
      h[e] = (_Float16)(c[e] * sel_scale);
    }
    *reinterpret_cast<f16x8*>(cent16 + row * kHeadDim + lane * 8) = h;
  }
  n2 += wave_xor_f(n2, 1);
  n2 += wave_xor_f(n2, 2);
  n2 += wave_xor_f(n2, 4);
  n2 += wave_xor_f(n2, 8);
  if (lane == 0) {
    cnorm[row] = sqrtf(n2);
    uplift[row] = radii[row] * beta[row] * sel_scale;
  }
}

hipError_t launch_summarize(const float* centroids, const float* radii, const float* beta, int n_kv_heads,
                            int n_blocks, _Float16* cent16, float* uplift, float* cnorm, hipStream_t s) {
  const int64_t rows = (int64_t)n_kv_heads * n_blocks;
  const float sel_scale = kLog2e / sqrtf((float)kHeadDim);
  hipLaunchKernelGGL(summarize_kernel, dim3((unsigned)((rows + 3) / 4)), dim3(256), 0, s, centroids, radii, beta,
                     rows, cent16, uplift, cnorm, sel_scale);
  return hipGetLastError();
}

hipError_t launch_stats_varlen(const StatsArgs& a, const SeqTable& t, hipStream_t s) {
  const dim3 grid(t.blk[t.n], a.n_kv_heads);
  const float sel_scale = kLog2e / sqrtf((float)kHeadDim);
#define RBS_STATS_CASE(BSZ)                                                                                 \
  case BSZ:                                                                                                 \
    hipLaunchKernelGGL(stats_kernel<BSZ>, grid, dim3(kStatsThreads), 0, s, a.K, a.kv_head, a.kv_tok, t,     \
                       a.centroids, a.radii, a.cent16, a.cnorm, sel_scale);                                 \
    break;
  switch (a.block_size) {
    RBS_STATS_CASE(64)
    RBS_STATS_CASE(128)
    RBS_STATS_CASE(256)
    default: return hipErrorInvalidValue;
  }
#undef RBS_STATS_CASE
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  static_assert(1024 * 4 >= kMaxBlocks, "the largest quantile kernel holds every radius of a head");
  int m_max = 0;
  for (int q = 0; q < t.n; ++q) m_max = t.blk[q + 1] - t.blk[q] > m_max ? t.blk[q + 1] - t.blk[q] : m_max;
  const dim3 heads(a.n_kv_heads, t.n);
#define RBS_QUANTILE(T, PER)                                                                            \
  hipLaunchKernelGGL((quantile_kernel<T, PER>), heads, dim3(T), 0, s, a.radii, t, a.beta, a.quantiles, \
                     a.uplift, sel_scale)
  if (m_max <= 256) RBS_QUANTILE(256, 1);
  else if (m_max <= 1024) RBS_QUANTILE(1024, 1);
  else RBS_QUANTILE(1024, 4);
#undef RBS_QUANTILE
  return hipGetLastError();
}

hipError_t launch_stats(const StatsArgs& a, hipStream_t s) {
  return launch_stats_varlen(a, single_sequence(a.n_tokens, a.n_blocks), s);
}

hipError_t launch_box(const BoxArgs& a, hipStream_t s) {
  const dim3 grid(a.n_blocks, a.n_kv_heads);
  const float sel_scale = kLog2e / sqrtf((float)kHeadDim);
#define RBS_BOX_CASE(BSZ)                                                                                   \
  case BSZ:                                                                                                 \
    hipLaunchKernelGGL(box_kernel<BSZ>, grid, dim3(kStatsThreads), 0, s, a.K, a.kv_head, a.kv_tok,          \
                       a.n_tokens, a.n_blocks, a.center, a.half, a.center16, a.half16, sel_scale);          \
    break;
  switch (a.block_size) {
    RBS_BOX_CASE(64)
    RBS_BOX_CASE(128)
    RBS_BOX_CASE(256)
    default: return hipErrorInvalidValue;
  }
#undef RBS_BOX_CASE
  return hipGetLastError();
}

}  // namespace rbs
