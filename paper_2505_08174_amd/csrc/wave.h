// Sums, maxima and row loads of one wave (64 lanes).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

// v of the source lane given by a DPP control; `old` where the source lane is
// outside the row or the row is masked off.
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ int dpp(int v, int old) {
  return __builtin_amdgcn_update_dpp(old, v, CTRL, ROW_MASK, 0xf, false);
}
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ double dpp(double v, double old) {
  return __hiloint2double(dpp<CTRL, ROW_MASK>(__double2hiint(v), __double2hiint(old)),
                          dpp<CTRL, ROW_MASK>(__double2loint(v), __double2loint(old)));
}
__device__ __forceinline__ double read_lane(double v, int l) {
  return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), l),
                          __builtin_amdgcn_readlane(__double2loint(v), l));
}

// (a of lanes 0-31 + a of lanes 32-63) in lanes 0-31, the same of b in lanes
// 32-63; and per pair of 16-lane rows: a's rows 0 + 1 (2 + 3) in row 0 (2), b's
// in row 1 (3). One swap of the two operands and one addition do what two
// shuffles, two selects and two additions would.
__device__ __forceinline__ double fold32(double a, double b) {
  const auto l = __builtin_amdgcn_permlane32_swap(__double2loint(a), __double2loint(b), false, false);
  const auto h = __builtin_amdgcn_permlane32_swap(__double2hiint(a), __double2hiint(b), false, false);
  return __hiloint2double((int)h[0], (int)l[0]) + __hiloint2double((int)h[1], (int)l[1]);
}
__device__ __forceinline__ double fold16(double a, double b) {
  const auto l = __builtin_amdgcn_permlane16_swap(__double2loint(a), __double2loint(b), false, false);
  const auto h = __builtin_amdgcn_permlane16_swap(__double2hiint(a), __double2hiint(b), false, false);
  return __hiloint2double((int)h[0], (int)l[0]) + __hiloint2double((int)h[1], (int)l[1]);
}

// Sums over the wave of N values, four to a register: value e ends in register
// e / 4, in lane 16 row + 15 with row = sum_row(e) (lane 15 of each 16-lane row
// holds the row's sum after the scans by row shifts 1, 2, 4, 8). No LDS
// traffic; 60 instructions for nine values, against 190 for nine separate
// scans over 64 lanes.
__host__ __device__ constexpr int sum_row(int e) { return ((e & 1) << 1) | ((e >> 1) & 1); }
template <int N>
struct WaveSums {
  double r[(N + 3) / 4];
};
template <int N>
__device__ __forceinline__ WaveSums<N> wave_sums(const double (&p)[N]) {
  WaveSums<N> w;
#pragma unroll
  for (int g = 0; g < (N + 3) / 4; ++g) {
    const double a = fold32(p[4 * g], 4 * g + 1 < N ? p[4 * g + 1] : 0.0);
    double v = 4 * g + 2 < N ? fold32(p[4 * g + 2], 4 * g + 3 < N ? p[4 * g + 3] : 0.0) : 0.0;
    v = fold16(a, v);
    v += dpp<0x111, 0xf>(v, 0.0);   // row_shr:1
    v += dpp<0x112, 0xf>(v, 0.0);   // row_shr:2
    v += dpp<0x114, 0xf>(v, 0.0);   // row_shr:4
    v += dpp<0x118, 0xf>(v, 0.0);   // row_shr:8
    w.r[g] = v;
  }
  return w;
}
// ... returned in every lane.
template <int N>
__device__ __forceinline__ void wave_sumv(double (&p)[N]) {
  const WaveSums<N> w = wave_sums(p);
#pragma unroll
  for (int e = 0; e < N; ++e) p[e] = read_lane(w.r[e / 4], 16 * sum_row(e) + 15);
}

// Largest value over the wave, in every lane.
__device__ __forceinline__ double wave_max(double v) {
  v = fmax(v, dpp<0x111, 0xf>(v, v));
  v = fmax(v, dpp<0x112, 0xf>(v, v));
  v = fmax(v, dpp<0x114, 0xf>(v, v));
  v = fmax(v, dpp<0x118, 0xf>(v, v));
  v = fmax(v, dpp<0x142, 0xa>(v, v));   // row_bcast:15 into rows 1, 3
  v = fmax(v, dpp<0x143, 0xc>(v, v));   // row_bcast:31 into rows 2, 3
  return read_lane(v, 63);
}
__device__ __forceinline__ int wave_min(int v) {
  v = min(v, dpp<0x111, 0xf>(v, v));
  v = min(v, dpp<0x112, 0xf>(v, v));
  v = min(v, dpp<0x114, 0xf>(v, v));
  v = min(v, dpp<0x118, 0xf>(v, v));
  v = min(v, dpp<0x142, 0xa>(v, v));
  v = min(v, dpp<0x143, 0xc>(v, v));
  return __builtin_amdgcn_readlane(v, 63);
}
// The largest v and the lowest i that comes with it, in every lane.
__device__ __forceinline__ void wave_best(double& v, int& i) {
  const double m = wave_max(v);
  i = wave_min(v == m ? i : 0x7fffffff);
  v = m;
}

// Rows of a factor (9 values each) through a buffer resource that ends with the
// factor: three 16-byte loads (FP32; five in FP64) at fixed offsets from a lane's
// first row, and rows past the end read as zeros without a test.
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
template <class T>
__device__ __forceinline__ __amdgpu_buffer_rsrc_t rows_rsrc(const T* f, int n) {
  return __builtin_amdgcn_make_buffer_rsrc((void*)f, 0, 9 * (int)sizeof(T) * n, 0x00027000);
}
__device__ __forceinline__ void load_row(__amdgpu_buffer_rsrc_t rs, int i, float (&v)[9]) {
  const int o = 36 * i;
  const u32x4 a = __builtin_amdgcn_raw_buffer_load_b128(rs, o, 0, 0);
  const u32x4 b = __builtin_amdgcn_raw_buffer_load_b128(rs, o + 16, 0, 0);
  const uint32_t c = __builtin_amdgcn_raw_buffer_load_b32(rs, o + 32, 0, 0);
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    v[e] = __uint_as_float(a[e]);
    v[4 + e] = __uint_as_float(b[e]);
  }
  v[8] = __uint_as_float(c);
}
__device__ __forceinline__ void load_row(__amdgpu_buffer_rsrc_t rs, int i, double (&v)[9]) {
  const int o = 72 * i;
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    const u32x4 a = __builtin_amdgcn_raw_buffer_load_b128(rs, o + 16 * t, 0, 0);
    v[2 * t] = __hiloint2double((int)a[1], (int)a[0]);
    v[2 * t + 1] = __hiloint2double((int)a[3], (int)a[2]);
  }
  const u32x2 b = __builtin_amdgcn_raw_buffer_load_b64(rs, o + 64, 0, 0);
  v[8] = __hiloint2double((int)b[1], (int)b[0]);
}
