// Near field with the seeded MLP kernel on MFMA tiles (the BF16 and the plain
// FP32 form, the latter on FP16 parts of FP32 values).
//
// A wave works on 64 consecutive targets (sorted rows, whichever leaves they
// are in), one per lane: in every step a lane takes the next source of its own
// leaf's near list and the wave evaluates its 64 pairs as two MFMA tiles. Each
// lane accumulates K(x_i - x_j) F_j for its own target in FP64 (owner
// computes, no atomics). The sources of a target are split over the four waves
// of a workgroup, whose rows are summed in LDS, and over `groups` workgroups,
// whose partial rows the combine adds in a fixed order, so that small systems
// still fill the chip.
//
// Bound: VALU issue in both forms (192 transcendentals per 64 pairs and lane; per
// 32 pairs about 330 other VALU instructions in BF16, 550 in FP32). Lanes with
// different sources cost a wave nothing, so targets need not be padded to whole
// waves per leaf (a leaf of 94 targets left a quarter of its last wave idle), and
// one lane per pair prepares and applies it (both halves of the wave did the same
// 32 pairs before). Measured, one wave per 32 targets and whole near list before,
// this split after: BF16, 500 particles 831 -> 25 us; BF16 hi + lo, 30,000
// particles 28.8 -> 12.5 ms; FP32, 5,000 particles 33.1 -> 4.3 ms, 100,000
// particles 244 -> 148 ms (76% of the FP32 MFMA rate), and with FP16 parts in
// place of FP32 MFMA 1.7 ms and 63 ms (1.27e10 pairs/s).
#include <algorithm>

#include "internal.h"
#include "mlp_mfma.h"
#include "near_walk.h"

#define T256_UNITS 256

namespace {


__global__ __launch_bounds__(T256_UNITS) void k_units_count(const int32_t* __restrict__ leaves,
                                                            int64_t nl,
                                                            const int4* __restrict__ nodes,
                                                            int64_t* __restrict__ cnt) {
  int64_t l = (int64_t)blockIdx.x * T256_UNITS + threadIdx.x;
  if (l > nl) return;
  if (l == nl) { cnt[nl] = 0; return; }
  int4 nd = nodes[leaves[l]];
  cnt[l] = (nd.y - nd.x + 31) / 32;
}

__global__ __launch_bounds__(T256_UNITS) void k_units_fill(const int64_t* __restrict__ cnt,
                                                           const int64_t* __restrict__ pos,
                                                           int64_t nl, int2* __restrict__ units) {
  int64_t l = (int64_t)blockIdx.x * T256_UNITS + threadIdx.x;
  if (l >= nl) return;
  for (int64_t c = 0; c < cnt[l]; ++c) units[pos[l] + c] = make_int2((int)l, (int)c);
}

struct NearB {
  NearTables t;
  const uint4* frags;
  const float* Fs;
  double* out;
  int groups;
  int input_mode;
};

template <bool ACC>
__global__ __launch_bounds__(NEAR_WG) void k_near_bf16(NearB a) {
  __shared__ bf16x8 fr[FR_TOTAL];
  stage_frags(fr, a.frags, NEAR_WG);
  __syncthreads();
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t s0 = 64 * ((int64_t)blockIdx.x / a.groups), s = s0 + lane;
  const int set = blockIdx.x % a.groups;
  const bool act = s < a.t.n;
  const int ss = (int)(act ? s : a.t.n - 1);
  const double xi0 = a.t.xs[3 * (int64_t)ss], xi1 = a.t.xs[3 * (int64_t)ss + 1],
               xi2 = a.t.xs[3 * (int64_t)ss + 2];
  const float c16 = (float)(1.0 / (16.0 * HH_PI));
  double u0 = 0, u1 = 0, u2 = 0;
  NearWalk wk;
  wk.start(a.t, ss, 4 * set + w, 4 * a.groups);
  const int steps = __builtin_amdgcn_readfirstlane(wave_max_i(wk.left));
  // source of the step, loaded while the step before is worked on
  double xj0 = a.t.xs[3 * (int64_t)wk.j], xj1 = a.t.xs[3 * (int64_t)wk.j + 1],
         xj2 = a.t.xs[3 * (int64_t)wk.j + 2];
  float g0 = a.Fs[3 * (int64_t)wk.j], g1 = a.Fs[3 * (int64_t)wk.j + 1],
        g2 = a.Fs[3 * (int64_t)wk.j + 2];
#pragma unroll 1
  for (int st = 0; st < steps; ++st) {
    float rx = (float)(xi0 - xj0), ry = (float)(xi1 - xj1), rz = (float)(xi2 - xj2);
    const bool none = wk.left <= 0;   // the lane's share has ended: not its last source again
    const float f0 = none ? 0.0f : g0, f1 = none ? 0.0f : g1, f2 = none ? 0.0f : g2;
    const bool skip = wk.j == ss || !act || none;
    if (wk.j == ss) { rx = 1.0f; ry = 0.0f; rz = 0.0f; }
    // which of two equally good remainders layer 1 gets (see pair_rest): fixed
    // by the list alone, whatever the split of the sources
    const bool exact = wk.unpaired();
    wk.next(a.t);
    xj0 = a.t.xs[3 * (int64_t)wk.j];
    xj1 = a.t.xs[3 * (int64_t)wk.j + 1];
    xj2 = a.t.xs[3 * (int64_t)wk.j + 2];
    g0 = a.Fs[3 * (int64_t)wk.j];
    g1 = a.Fs[3 * (int64_t)wk.j + 1];
    g2 = a.Fs[3 * (int64_t)wk.j + 2];
    const PairIn in = pair_in(a.input_mode, rx, ry, rz, exact);
    float q[9];
    mlp_pairs_bf16<ACC>(fr, in, q);
    pair_apply(q, skip ? 0.0f : in.rs * c16, f0, f1, f2, u0, u1, u2);
  }
  const double u[3] = {u0, u1, u2};
  write_rows(reinterpret_cast<double*>(fr), lane, w, u, s0, a.t.n, set, a.out);
}

// The plain FP32 form: the same walk, tiles of FP32 values in FP16 parts. F is
// FP32; each lane sums its target's terms in FP64.
template <class TO>
struct NearF {
  NearTables t;
  const uint4* frags;
  const float* Fs;
  TO* out;
  int groups;
  int input_mode;
  float sgn;   // +1: K(x_i - x_j); -1: K(x_j - x_i) (the transposed product)
};

template <class TO>
__global__ __launch_bounds__(NEAR_WG) void k_near_f32(NearF<TO> a) {
  __shared__ uint4 fr[X2_TOTAL];
  stage_frags_x2(fr, a.frags, NEAR_WG);
  __syncthreads();
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t s0 = 64 * ((int64_t)blockIdx.x / a.groups), s = s0 + lane;
  const int set = blockIdx.x % a.groups;
  const bool act = s < a.t.n;
  const int ss = (int)(act ? s : a.t.n - 1);
  const double xi0 = a.t.xs[3 * (int64_t)ss], xi1 = a.t.xs[3 * (int64_t)ss + 1],
               xi2 = a.t.xs[3 * (int64_t)ss + 2];
  const float c16 = (float)(1.0 / (16.0 * HH_PI));
  double u0 = 0, u1 = 0, u2 = 0;
  NearWalk wk;
  wk.start(a.t, ss, 4 * set + w, 4 * a.groups);
  const int steps = __builtin_amdgcn_readfirstlane(wave_max_i(wk.left));
#pragma unroll 1
  for (int st = 0; st < steps; ++st) {
    const int64_t j = wk.j;
    float rx = a.sgn * (float)(xi0 - a.t.xs[3 * j]);
    float ry = a.sgn * (float)(xi1 - a.t.xs[3 * j + 1]);
    float rz = a.sgn * (float)(xi2 - a.t.xs[3 * j + 2]);
    const bool none = wk.left <= 0;   // the lane's share has ended: not its last source again
    const float g0 = a.Fs[3 * j], g1 = a.Fs[3 * j + 1], g2 = a.Fs[3 * j + 2];
    const float f0 = none ? 0.0f : g0, f1 = none ? 0.0f : g1, f2 = none ? 0.0f : g2;
    const bool skip = wk.j == ss || !act || none;
    if (wk.j == ss) { rx = 1.0f; ry = 0.0f; rz = 0.0f; }
    const PairIn in = pair_in(a.input_mode, rx, ry, rz, false);
    float q[9];
    mlp_pairs_x2(fr, in.v0, in.v1, in.v2, q);
    pair_apply(q, skip ? 0.0f : in.rs * c16, f0, f1, f2, u0, u1, u2);
    wk.next(a.t);
  }
  const double u[3] = {u0, u1, u2};
  write_rows(reinterpret_cast<double*>(fr), lane, w, u, s0, a.t.n, set, a.out);
}

}  // namespace

// Work units of the FP32 backward (leaf rank, chunk of 32 targets): int2 units, their
// number is pos[n_leaves]. Made by each call for itself: a tree may be in use on other
// streams and in other threads.
void build_units(hh_ctx ctx, hh_tree t, DevBuf& units, DevBuf& pos) {
  hipStream_t st = ctx->stream;
  int64_t nl = t->n_leaves;
  DevBuf cnt;
  cnt.alloc(ctx, (nl + 1) * sizeof(int64_t));
  pos.alloc(ctx, (nl + 1) * sizeof(int64_t));
  units.alloc(ctx, (t->n / 32 + nl) * sizeof(int2));   // no leaf leaves more than one chunk unfilled
  unsigned g = (unsigned)((nl + 1 + T256_UNITS - 1) / T256_UNITS);
  hipLaunchKernelGGL(k_units_count, dim3(g), dim3(T256_UNITS), 0, st, t->leaves.as<int32_t>(), nl,
                     t->nodes.as<int4>(), cnt.as<int64_t>());
  scan_exclusive_i64(ctx, cnt.as<int64_t>(), pos.as<int64_t>(), nl + 1);
  hipLaunchKernelGGL(k_units_fill, dim3(g), dim3(T256_UNITS), 0, st, cnt.as<int64_t>(),
                     pos.as<int64_t>(), nl, units.as<int2>());
  HIP_OK(hipGetLastError());
}

// A share of 32 sources takes some 100 us, staging a workgroup's 48 KB of weights
// about 2. Below that, shares down to 4 sources as long as they fill idle compute
// units: at 500 particles, 32 sets of 4-source shares take 25 us, one set 160 us (a
// product 27.1 us; with shares of 2 sources 31.4, of 1 source 28.8).
int near_groups_mfma(hh_ctx ctx, hh_tree t, hh_part p) {
  return near_sets(ctx, t, p, 3, 32, 4);
}

void launch_near_bf16(hh_ctx ctx, hh_tree t, hh_part p, hh_kernel k, const void* Fs, void* out,
                      int groups, bool split) {
  HH_REQUIRE(k->kind == KIND_MLP, HH_ERR_INVALID_ARG, "the BF16 form needs the MLP kernel");
  NearB a;
  a.t = near_tables(t, p);
  a.frags = k->pbf.as<uint4>();
  a.Fs = (const float*)Fs;
  a.out = (double*)out;
  a.groups = groups;
  a.input_mode = k->input_mode;
  const unsigned grid = (unsigned)((t->n + 63) / 64 * groups);
  if (split)
    hipLaunchKernelGGL(k_near_bf16<true>, dim3(grid), dim3(NEAR_WG), 0, ctx->stream, a);
  else
    hipLaunchKernelGGL(k_near_bf16<false>, dim3(grid), dim3(NEAR_WG), 0, ctx->stream, a);
  HIP_OK(hipGetLastError());
}

template <class TO>
static void launch_near_f32_t(hh_ctx ctx, hh_tree t, hh_part p, hh_kernel k, const void* Fs,
                              void* out, int groups, float sgn) {
  NearF<TO> a;
  a.t = near_tables(t, p);
  a.frags = k->px2.as<uint4>();
  a.Fs = (const float*)Fs;
  a.out = (TO*)out;
  a.groups = groups;
  a.input_mode = k->input_mode;
  a.sgn = sgn;
  const unsigned grid = (unsigned)((t->n + 63) / 64 * groups);
  hipLaunchKernelGGL(k_near_f32<TO>, dim3(grid), dim3(NEAR_WG), 0, ctx->stream, a);
  HIP_OK(hipGetLastError());
}

void launch_near_f32(hh_ctx ctx, hh_tree t, hh_part p, hh_kernel k, const void* Fs, void* out,
                     int groups, float sgn) {
  HH_REQUIRE(k->kind == KIND_MLP, HH_ERR_INVALID_ARG, "the FP32 MFMA tile needs the MLP kernel");
  if (groups > 1)
    launch_near_f32_t<double>(ctx, t, p, k, Fs, out, groups, sgn);
  else
    launch_near_f32_t<float>(ctx, t, p, k, Fs, out, groups, sgn);
}
