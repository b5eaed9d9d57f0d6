// Device-wide exclusive scan and stable LSD radix sort (8-bit digits).
//
// Radix pass of the tiled sort: (1) each 256-thread block counts the digits of its 4096-item
// tile in LDS and writes a digit-major histogram; (2) one exclusive scan over
// all (digit, tile) counts gives every tile its output base per digit;
// (3) each block re-reads its tile in 16 rounds of 256 consecutive items and
// ranks each item among equal digits with 8 wave ballots (a wave-wide match),
// adding the counts of earlier waves and earlier rounds, which keeps the pass
// stable.
#include "internal.h"

namespace {

constexpr int SCAN_T = 256;
constexpr int SCAN_ITEMS = 8;
constexpr int SCAN_TILE = SCAN_T * SCAN_ITEMS;

__device__ __forceinline__ int64_t wave_incl_scan(int64_t v, int lane) {
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    int64_t t = __shfl_up(v, o, 64);
    if (lane >= o) v += t;
  }
  return v;
}

// Block-wide exclusive scan of one value per thread (256 threads); returns the
// exclusive prefix and writes the block total to *total.
__device__ __forceinline__ int64_t block_excl_scan(int64_t v, int64_t* total) {
  __shared__ int64_t wsum[SCAN_T / 64];
  int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  int64_t inc = wave_incl_scan(v, lane);
  if (lane == 63) wsum[w] = inc;
  __syncthreads();
  int64_t off = 0, tot = 0;
#pragma unroll
  for (int i = 0; i < SCAN_T / 64; ++i) {
    if (i < w) off += wsum[i];
    tot += wsum[i];
  }
  __syncthreads();
  *total = tot;
  return off + inc - v;
}

__global__ __launch_bounds__(SCAN_T) void k_scan_reduce(const int64_t* __restrict__ in,
                                                        int64_t n, int64_t* __restrict__ sums) {
  int64_t base = (int64_t)blockIdx.x * SCAN_TILE + (int64_t)threadIdx.x * SCAN_ITEMS;
  int64_t s = 0;
#pragma unroll
  for (int i = 0; i < SCAN_ITEMS; ++i)
    if (base + i < n) s += in[base + i];
  int64_t tot;
  (void)block_excl_scan(s, &tot);
  if (threadIdx.x == 0) sums[blockIdx.x] = tot;
}

// Exclusive scan of `m` tile sums by one block, in place.
__global__ __launch_bounds__(SCAN_T) void k_scan_tiles(int64_t* __restrict__ sums, int64_t m) {
  int64_t carry = 0;
  for (int64_t base = 0; base < m; base += SCAN_T) {
    int64_t i = base + threadIdx.x;
    int64_t v = i < m ? sums[i] : 0;
    int64_t tot;
    int64_t ex = block_excl_scan(v, &tot);
    if (i < m) sums[i] = carry + ex;
    carry += tot;
  }
}

__global__ __launch_bounds__(SCAN_T) void k_scan_down(const int64_t* __restrict__ in, int64_t n,
                                                      const int64_t* __restrict__ sums,
                                                      int64_t* __restrict__ out) {
  int64_t base = (int64_t)blockIdx.x * SCAN_TILE + (int64_t)threadIdx.x * SCAN_ITEMS;
  int64_t v[SCAN_ITEMS];
  int64_t s = 0;
#pragma unroll
  for (int i = 0; i < SCAN_ITEMS; ++i) {
    v[i] = base + i < n ? in[base + i] : 0;
    s += v[i];
  }
  int64_t tot;
  int64_t ex = block_excl_scan(s, &tot) + sums[blockIdx.x];
#pragma unroll
  for (int i = 0; i < SCAN_ITEMS; ++i) {
    if (base + i < n) out[base + i] = ex;
    ex += v[i];
  }
}

// Exclusive scan of up to SCAN_ONE values by one workgroup: one launch for the
// histograms and lists of small systems, where each of the three launches above
// costs more than the scan (the line lies where the one workgroup's rounds take
// as long as two launches).
constexpr int SCAN_ONE = 16384;
__global__ __launch_bounds__(1024) void k_scan_one(const int64_t* __restrict__ in, int n,
                                                   int64_t* __restrict__ out) {
  __shared__ int64_t wsum[16];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  int64_t carry = 0;
  for (int b = 0; b < n; b += 4096) {
    const int i0 = b + 4 * (int)threadIdx.x;
    int64_t v[4], s = 0;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      v[e] = i0 + e < n ? in[i0 + e] : 0;
      s += v[e];
    }
    const int64_t inc = wave_incl_scan(s, lane);
    if (lane == 63) wsum[w] = inc;
    __syncthreads();
    int64_t off = carry, tot = 0;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      if (i < w) off += wsum[i];
      tot += wsum[i];
    }
    int64_t ex = off + inc - s;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      if (i0 + e < n) out[i0 + e] = ex;
      ex += v[e];
    }
    carry += tot;
    __syncthreads();
  }
}

// Stable LSD radix sort of up to SS_N pairs by one workgroup, all passes in one
// launch: the pairs stay in registers, LDS holds them between passes. Up to here
// the 5 launches per pass of the tiled sort (40 for Morton keys) cost more than
// sorting on one compute unit: 35 us for 2,000 Morton keys and 72 us for 5,000,
// against 130 us of kernels and as much of launches.
constexpr int SS_T = 1024, SS_E = 8, SS_N = SS_T * SS_E;
__global__ __launch_bounds__(SS_T) void k_sort_small(uint64_t* __restrict__ keys,
                                                     uint32_t* __restrict__ vals, int n,
                                                     int passes) {
  __shared__ uint64_t sk[SS_N];
  __shared__ uint32_t sv[SS_N];
  __shared__ int base[256];
  __shared__ int wcnt[SS_T / 64][256];
  __shared__ int wtot[4];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const uint64_t lt = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
  uint64_t key[SS_E];
  uint32_t val[SS_E];
#pragma unroll
  for (int r = 0; r < SS_E; ++r) {
    const int i = r * SS_T + tid;
    key[r] = i < n ? keys[i] : 0;
    val[r] = i < n ? vals[i] : 0;
  }
  for (int i = tid; i < (SS_T / 64) * 256; i += SS_T) (&wcnt[0][0])[i] = 0;
  for (int p = 0; p < passes; ++p) {
    const int shift = 8 * p;
    if (tid < 256) base[tid] = 0;
    __syncthreads();
#pragma unroll
    for (int r = 0; r < SS_E; ++r)
      if (r * SS_T + tid < n) atomicAdd(&base[(key[r] >> shift) & 255], 1);
    __syncthreads();
    int c = 0, inc = 0;
    if (tid < 256) {
      c = base[tid];
      inc = (int)wave_incl_scan(c, lane);
      if (lane == 63) wtot[w] = inc;
    }
    __syncthreads();
    if (tid < 256) {
      int off = 0;
      for (int i = 0; i < w; ++i) off += wtot[i];
      base[tid] = off + inc - c;
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < SS_E; ++r) {
      if (r * SS_T >= n) break;   // uniform
      const bool valid = r * SS_T + tid < n;
      const int d = (int)((key[r] >> shift) & 255);
      const uint64_t vb = __ballot(valid);
      uint64_t m = valid ? vb : ~vb;
#pragma unroll
      for (int b = 0; b < 8; ++b) {
        const uint64_t bal = __ballot((d >> b) & 1);
        m &= ((d >> b) & 1) ? bal : ~bal;
      }
      const int rank = __popcll(m & lt);
      if (valid && rank == 0) wcnt[w][d] = __popcll(m);
      __syncthreads();
      if (valid) {
        int pos = base[d] + rank;
        for (int ww = 0; ww < w; ++ww) pos += wcnt[ww][d];
        sk[pos] = key[r];
        sv[pos] = val[r];
      }
      __syncthreads();
      if (tid < 256) {
        int add = 0;
        for (int ww = 0; ww < SS_T / 64; ++ww) {
          add += wcnt[ww][tid];
          wcnt[ww][tid] = 0;
        }
        base[tid] += add;
      }
      __syncthreads();
    }
#pragma unroll
    for (int r = 0; r < SS_E; ++r) {
      const int i = r * SS_T + tid;
      if (i < n) {
        key[r] = sk[i];
        val[r] = sv[i];
      }
    }
    __syncthreads();
  }
#pragma unroll
  for (int r = 0; r < SS_E; ++r) {
    const int i = r * SS_T + tid;
    if (i < n) {
      keys[i] = key[r];
      vals[i] = val[r];
    }
  }
}

constexpr int RS_T = 256;
constexpr int RS_ROUNDS = 16;
constexpr int RS_TILE = RS_T * RS_ROUNDS;

__global__ __launch_bounds__(RS_T) void k_radix_hist(const uint64_t* __restrict__ keys, int64_t n,
                                                     int shift, int64_t nblocks,
                                                     int64_t* __restrict__ hist) {
  __shared__ int cnt[256];
  cnt[threadIdx.x] = 0;
  __syncthreads();
  int64_t base = (int64_t)blockIdx.x * RS_TILE;
  for (int r = 0; r < RS_ROUNDS; ++r) {
    int64_t i = base + r * RS_T + threadIdx.x;
    if (i < n) atomicAdd(&cnt[(keys[i] >> shift) & 255], 1);
  }
  __syncthreads();
  hist[(int64_t)threadIdx.x * nblocks + blockIdx.x] = cnt[threadIdx.x];
}

__global__ __launch_bounds__(RS_T) void k_radix_scatter(
    const uint64_t* __restrict__ kin, const uint32_t* __restrict__ vin, uint64_t* __restrict__ kout,
    uint32_t* __restrict__ vout, int64_t n, int shift, int64_t nblocks,
    const int64_t* __restrict__ offs) {
  __shared__ int64_t base[256];
  __shared__ int run[256];
  __shared__ int wcnt[RS_T / 64][256];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  base[threadIdx.x] = offs[(int64_t)threadIdx.x * nblocks + blockIdx.x];
  run[threadIdx.x] = 0;
  for (int i = 0; i < RS_T / 64; ++i) wcnt[i][threadIdx.x] = 0;
  __syncthreads();
  const uint64_t lt = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
  int64_t tile = (int64_t)blockIdx.x * RS_TILE;
  for (int r = 0; r < RS_ROUNDS; ++r) {
    int64_t i = tile + r * RS_T + threadIdx.x;
    bool valid = i < n;
    uint64_t key = valid ? kin[i] : 0;
    uint32_t val = valid ? vin[i] : 0;
    int d = (int)((key >> shift) & 255);
    uint64_t vb = __ballot(valid);
    uint64_t m = valid ? vb : ~vb;
#pragma unroll
    for (int b = 0; b < 8; ++b) {
      uint64_t bal = __ballot((d >> b) & 1);
      m &= ((d >> b) & 1) ? bal : ~bal;
    }
    int rank = __popcll(m & lt);
    if (valid && rank == 0) wcnt[w][d] = __popcll(m);
    __syncthreads();
    if (valid) {
      int64_t pos = base[d] + run[d] + rank;
      for (int ww = 0; ww < w; ++ww) pos += wcnt[ww][d];
      kout[pos] = key;
      vout[pos] = val;
    }
    __syncthreads();
    int add = 0;
    for (int ww = 0; ww < RS_T / 64; ++ww) {
      add += wcnt[ww][threadIdx.x];
      wcnt[ww][threadIdx.x] = 0;
    }
    run[threadIdx.x] += add;
    __syncthreads();
  }
}

}  // namespace

void scan_exclusive_i64(hh_ctx ctx, const int64_t* in, int64_t* out, int64_t n) {
  if (n <= 0) return;
  if (n <= SCAN_ONE) {
    hipLaunchKernelGGL(k_scan_one, dim3(1), dim3(1024), 0, ctx->stream, in, (int)n, out);
    HIP_OK(hipGetLastError());
    return;
  }
  int64_t tiles = (n + SCAN_TILE - 1) / SCAN_TILE;
  DevBuf sums;
  sums.alloc(ctx, tiles * sizeof(int64_t));
  hipLaunchKernelGGL(k_scan_reduce, dim3(tiles), dim3(SCAN_T), 0, ctx->stream, in, n,
                     sums.as<int64_t>());
  hipLaunchKernelGGL(k_scan_tiles, dim3(1), dim3(SCAN_T), 0, ctx->stream, sums.as<int64_t>(),
                     tiles);
  hipLaunchKernelGGL(k_scan_down, dim3(tiles), dim3(SCAN_T), 0, ctx->stream, in, n,
                     sums.as<int64_t>(), out);
  HIP_OK(hipGetLastError());
}

void radix_sort_u64(hh_ctx ctx, uint64_t* keys, uint32_t* vals, int64_t n, int bits) {
  if (n <= 1) return;
  int passes = (bits + 7) / 8;
  if (n <= SS_N) {
    hipLaunchKernelGGL(k_sort_small, dim3(1), dim3(SS_T), 0, ctx->stream, keys, vals, (int)n,
                       passes);
    HIP_OK(hipGetLastError());
    return;
  }
  int64_t nblocks = (n + RS_TILE - 1) / RS_TILE;
  DevBuf k2, v2, hist;
  k2.alloc(ctx, n * sizeof(uint64_t));
  v2.alloc(ctx, n * sizeof(uint32_t));
  hist.alloc(ctx, 256 * nblocks * sizeof(int64_t));
  uint64_t *ka = keys, *kb = k2.as<uint64_t>();
  uint32_t *va = vals, *vb = v2.as<uint32_t>();
  for (int p = 0; p < passes; ++p) {
    int shift = 8 * p;
    hipLaunchKernelGGL(k_radix_hist, dim3(nblocks), dim3(RS_T), 0, ctx->stream, ka, n, shift,
                       nblocks, hist.as<int64_t>());
    scan_exclusive_i64(ctx, hist.as<int64_t>(), hist.as<int64_t>(), 256 * nblocks);
    hipLaunchKernelGGL(k_radix_scatter, dim3(nblocks), dim3(RS_T), 0, ctx->stream, ka, va, kb,
                       vb, n, shift, nblocks, hist.as<int64_t>());
    HIP_OK(hipGetLastError());
    std::swap(ka, kb);
    std::swap(va, vb);
  }
  if (ka != keys) {
    HIP_OK(hipMemcpyAsync(keys, ka, n * sizeof(uint64_t), hipMemcpyDeviceToDevice, ctx->stream));
    HIP_OK(hipMemcpyAsync(vals, va, n * sizeof(uint32_t), hipMemcpyDeviceToDevice, ctx->stream));
  }
}
