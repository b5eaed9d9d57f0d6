// Near field: U_i += sum over inadmissible leaf blocks (tau, sigma) in P^H of
// sum_{j in sigma, j != i} K(x_i - x_j) F_j (Sec. 3.3.1), kernel evaluated on
// the fly and never stored: the forms on the VALU (the RPY kernels, and the MLP
// kernel in FP64).
//
// One lane per target and source share, as in the MFMA near field: a wave holds
// 64 consecutive targets, its lanes walk the near lists of their own leaves, and
// the sources are split over the four waves of a workgroup and over `groups`
// workgroups, whose partial rows the combine adds in a fixed order (owner
// computes, no atomics). Bound by VALU issue (square root and divisions of the
// RPY tensor). One workgroup per leaf, which staged the sources in LDS and left
// the rest of the chip idle at small sizes, took 800 us at 2,000 particles in
// FP64 (32 leaves) and 5.5 ms at 60,000 in FP32 (a quarter of its lanes past
// the leaf); this form takes 1.1 ms at 60,000, and the 6N kernel by particles
// 0.75 ms at 40,000 particles (5.05 ms row by row).
#include "devmath.h"
#include "internal.h"
#include "near_walk.h"

namespace {

template <class T, class TO>
struct NearArgs {
  NearTables t;
  const T* Fs;
  TO* out;
  int groups;
  KParams kp;
  T sgn;   // +1: K(x_i - x_j); -1: K(x_j - x_i) (transposed product)
};

template <class T, int KIND, class TO>
__global__ __launch_bounds__(NEAR_WG) void k_near_valu(NearArgs<T, TO> a) {
  __shared__ T wl[KIND == KIND_MLP ? MLP_NP : 1];
  __shared__ double red[4 * 64 * 3];
  if (KIND == KIND_MLP) {
    const T* w = (const T*)a.kp.w;
    for (int i = threadIdx.x; i < MLP_NP; i += NEAR_WG) wl[i] = w[i];
    __syncthreads();
  }
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t s0 = 64 * ((int64_t)blockIdx.x / a.groups), s = s0 + lane;
  const int set = blockIdx.x % a.groups;
  T u0 = 0, u1 = 0, u2 = 0;
  if (s < a.t.n) {
    const double* xs = a.t.xs;
    const double xi0 = xs[3 * s], xi1 = xs[3 * s + 1], xi2 = xs[3 * s + 2];
    NearWalk wk;
    wk.start(a.t, s, 4 * set + w, 4 * a.groups);
    // the next source is loaded while one is worked on
    double x0 = xs[3 * (int64_t)wk.j], x1 = xs[3 * (int64_t)wk.j + 1], x2 = xs[3 * (int64_t)wk.j + 2];
    T f0 = a.Fs[3 * (int64_t)wk.j], f1 = a.Fs[3 * (int64_t)wk.j + 1], f2 = a.Fs[3 * (int64_t)wk.j + 2];
    while (wk.left > 0) {
      const bool own = wk.j == s;
      const T rx = a.sgn * (T)(xi0 - x0), ry = a.sgn * (T)(xi1 - x1), rz = a.sgn * (T)(xi2 - x2);
      const T g0 = f0, g1 = f1, g2 = f2;
      wk.next(a.t);
      x0 = xs[3 * (int64_t)wk.j];
      x1 = xs[3 * (int64_t)wk.j + 1];
      x2 = xs[3 * (int64_t)wk.j + 2];
      f0 = a.Fs[3 * (int64_t)wk.j];
      f1 = a.Fs[3 * (int64_t)wk.j + 1];
      f2 = a.Fs[3 * (int64_t)wk.j + 2];
      if (own) continue;
      T K[9];
      kernel_entry<T>(a.kp, wl, rx, ry, rz, K);
      u0 += K[0] * g0 + K[1] * g1 + K[2] * g2;
      u1 += K[3] * g0 + K[4] * g1 + K[5] * g2;
      u2 += K[6] * g0 + K[7] * g1 + K[8] * g2;
    }
  }
  const double u[3] = {(double)u0, (double)u1, (double)u2};
  write_rows(red, lane, w, u, s0, a.t.n, set, a.out);
}

// The 6N kernel by particles: a lane owns the two rows of one particle and
// takes the two rows of one source particle per step, so the distance, its
// root and its reciprocals serve all four 3x3 entries (row by row, the two
// parities of a wave ran different entries in turn and every row pair took its
// own root and divisions).
template <class T, class TO>
__global__ __launch_bounds__(NEAR_WG) void k_near_rpy6(NearArgs<T, TO> a) {
  __shared__ double red[4 * 64 * 6];
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t np = a.t.n / 2;
  const int64_t s0 = 64 * ((int64_t)blockIdx.x / a.groups), s = s0 + lane;
  const int set = blockIdx.x % a.groups;
  T u[6] = {0, 0, 0, 0, 0, 0};
  if (s < np) {
    const double* xs = a.t.xs;
    const double xi0 = xs[6 * s], xi1 = xs[6 * s + 1], xi2 = xs[6 * s + 2];
    const T ra = (T)a.kp.a, c8 = (T)a.kp.c8, c6 = (T)a.kp.c6;
    NearWalk wk;
    wk.start<2>(a.t, s, 4 * set + w, 4 * a.groups);
    while (wk.left > 0) {
      const int64_t j = wk.j;
      const T rx = (T)(xi0 - xs[6 * j]), ry = (T)(xi1 - xs[6 * j + 1]), rz = (T)(xi2 - xs[6 * j + 2]);
      T f[6];
#pragma unroll
      for (int e = 0; e < 6; ++e) f[e] = a.Fs[6 * j + e];
      wk.next<2>(a.t);
      if (j == s) continue;
      T K[9], C[9], R[9];
      rpy_entry<T>(rx, ry, rz, ra, c8, c6, K);
      rpy6_entry<T>(1, 0, rx, ry, rz, ra, c8, c6, C);
      rpy6_entry<T>(1, 1, rx, ry, rz, ra, c8, c6, R);
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        u[d] += K[3 * d] * f[0] + K[3 * d + 1] * f[1] + K[3 * d + 2] * f[2];
        u[d] += C[3 * d] * f[3] + C[3 * d + 1] * f[4] + C[3 * d + 2] * f[5];
        u[3 + d] += C[3 * d] * f[0] + C[3 * d + 1] * f[1] + C[3 * d + 2] * f[2];
        u[3 + d] += R[3 * d] * f[3] + R[3 * d + 1] * f[4] + R[3 * d + 2] * f[5];
      }
    }
  }
  const double v[6] = {(double)u[0], (double)u[1], (double)u[2],
                       (double)u[3], (double)u[4], (double)u[5]};
  write_rows(red, lane, w, v, s0, np, set, a.out);
}

template <class T, class TO>
void launch_near_to(hh_ctx ctx, hh_tree t, hh_part p, hh_kernel k, const void* Fs, void* out,
                    int groups, double sgn) {
  NearArgs<T, TO> a;
  a.t = near_tables(t, p);
  a.Fs = (const T*)Fs;
  a.out = (TO*)out;
  a.groups = groups;
  a.kp = make_kparams(k, sizeof(T) == 8);
  a.sgn = (T)sgn;
  const int64_t rows = k->kind == KIND_RPY6 ? t->n / 2 : t->n;
  const dim3 grid((unsigned)((rows + 63) / 64 * groups));
  if (k->kind == KIND_MLP) {
    if constexpr (sizeof(T) == 8)   // in FP32 the MLP kernel runs on MFMA tiles
      hipLaunchKernelGGL((k_near_valu<T, KIND_MLP, TO>), grid, dim3(NEAR_WG), 0, ctx->stream, a);
  } else if (k->kind == KIND_RPY6)
    hipLaunchKernelGGL((k_near_rpy6<T, TO>), grid, dim3(NEAR_WG), 0, ctx->stream, a);
  else
    hipLaunchKernelGGL((k_near_valu<T, KIND_RPY, TO>), grid, dim3(NEAR_WG), 0, ctx->stream, a);
  HIP_OK(hipGetLastError());
}

template <class T>
void launch_near_t(hh_ctx ctx, hh_tree t, hh_part p, hh_kernel k, const void* Fs, void* out,
                   int groups, double sgn = 1.0) {
  if (groups > 1)
    launch_near_to<T, double>(ctx, t, p, k, Fs, out, groups, sgn);
  else
    launch_near_to<T, T>(ctx, t, p, k, Fs, out, groups, sgn);
}

}  // namespace

// The RPY kernels keep 4 workgroups and more on a compute unit, and a pair is cheap
// enough that a share below 16 sources costs more in its search for the first source
// and its partial row than it fills. The MLP kernel in FP64 (79 KB of LDS, two
// workgroups) takes the same split: a workgroup's 73 KB of weights are staged for 4,096
// pairs and more, some 3 ms of work. Products, one workgroup per leaf before and this
// split after: 700 particles 63.6 -> 1.8 ms, 2,000 194 -> 6.2, 12,000 919 -> 80 ms.
int near_groups(hh_ctx ctx, hh_tree t, hh_part p, hh_kernel k, int prec) {
  return k->kind == KIND_MLP && prec != HH_FP64 ? near_groups_mfma(ctx, t, p)
                                                : near_sets(ctx, t, p, 4, 32, 16);
}

// Near field with the displacement reversed: sum_j K(x_j - x_i) v_j, which is
// the transposed near product (K entries are symmetric 3x3 matrices).
void launch_near_neg(hh_ctx ctx, hh_tree t, hh_part p, hh_kernel k, int prec, const void* Vs,
                     void* out, int groups) {
  if (prec == HH_FP64)
    launch_near_t<double>(ctx, t, p, k, Vs, out, groups, -1.0);
  else if (k->kind == KIND_MLP)
    launch_near_f32(ctx, t, p, k, Vs, out, groups, -1.0f);
  else
    launch_near_t<float>(ctx, t, p, k, Vs, out, groups, -1.0);
}

void launch_near(hh_ctx ctx, hh_tree t, hh_part p, hh_kernel k, int prec, const void* Fs,
                 void* out, int groups) {
  if (prec == HH_FP64)
    launch_near_t<double>(ctx, t, p, k, Fs, out, groups);
  else if (prec == HH_FP32 && k->kind == KIND_MLP)
    launch_near_f32(ctx, t, p, k, Fs, out, groups);
  else if (prec == HH_FP32 || k->kind != KIND_MLP)
    launch_near_t<float>(ctx, t, p, k, Fs, out, groups);
  else
    launch_near_bf16(ctx, t, p, k, Fs, out, groups, prec == HH_BF16_SPLIT);
}
