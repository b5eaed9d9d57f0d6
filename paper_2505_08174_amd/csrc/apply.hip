// Far-field low-rank apply, self term, combine and unpermute; the matvec and
// ACA entry points.
//
// The low-rank product of an admissible block is applied right to left as in
// Sec. 3: t_k = sum_j q_k(j) F_j for every term (one workgroup per block),
// then u_i += sum_k c_k(i) t_k. The second half runs per target row: lanes walk
// from the row's leaf up to the root and add the terms of every admissible
// block whose target cluster contains it, in a fixed order, so the sum is
// deterministic without atomics. The same walk adds blocks that fell back to
// dense evaluation; the near-field rows and the self term alpha_1 F_i (Eq. (2))
// are added with it or after it, and U is written in the caller's order.
#include "api_guard.h"
#include "devmath.h"
#include "internal.h"
#include "near_walk.h"
#include "wave.h"

void plan_aca(hh_ctx ctx, hh_tree t, hh_part p, hh_lowrank lr, int force_streamed);
void run_aca_stored(hh_ctx ctx, hh_tree t, hh_part p, hh_kernel k, hh_lowrank lr);
void run_aca_batch(hh_ctx ctx, hh_tree t, hh_part p, hh_kernel k, hh_lowrank lr, size_t i,
                   const void* Fs, int64_t* counters);
void lowrank_stats(hh_ctx ctx, hh_tree t, hh_part p, hh_lowrank lr, bool toff);
hh_lowrank_s* build_lowrank_pivots(hh_ctx ctx, hh_tree t, hh_part p, hh_kernel k, int prec,
                                   const int32_t* rank, const int32_t* fallback,
                                   const int32_t* piv_i, const int32_t* piv_j);

namespace {

constexpr int T256 = 256;
inline unsigned nblk(int64_t n) { return (unsigned)((n + T256 - 1) / T256); }

template <class TI, class TO>
__global__ __launch_bounds__(T256) void k_gather_rows(const TI* __restrict__ F,
                                                      const int32_t* __restrict__ perm, int64_t n,
                                                      TO* __restrict__ Fs) {
  int64_t s = (int64_t)blockIdx.x * T256 + threadIdx.x;
  if (s >= n) return;
  int64_t o = perm[s];
  Fs[3 * s] = (TO)F[3 * o];
  Fs[3 * s + 1] = (TO)F[3 * o + 1];
  Fs[3 * s + 2] = (TO)F[3 * o + 2];
}

// t[toff[b] + k] = sum_j q_k(j) F_sigma(j) for every non-fallback block, blocks
// taken largest first (`order`; a replay has none and takes them as they come). One workgroup per block, its waves take the
// terms four at a time, lanes over the sources; the four terms' twelve sums
// share three registers in the wave sums. Bound by the one read of the factors'
// q halves. (One term at a time by the whole workgroup left most lanes of a
// block of 64-128 sources idle and took two barriers and three shuffled sums
// per term: 3.26 ms at 40,000 particles of the 6N form, now
// 2.55 ms, 5.5 TB/s of HBM traffic.)
template <class T>
__global__ __launch_bounds__(T256) void k_far_t(const int2* __restrict__ G, int64_t nG,
                                                const int32_t* __restrict__ order,
                                                const int4* __restrict__ nodes,
                                                const int32_t* __restrict__ rank,
                                                const int32_t* __restrict__ flag,
                                                const int64_t* __restrict__ fptr,
                                                const int64_t* __restrict__ toff,
                                                const T* __restrict__ pool,
                                                const T* __restrict__ Fs,
                                                double* __restrict__ tbuf) {
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  for (int64_t o = blockIdx.x; o < nG; o += gridDim.x) {
    const int64_t b = order ? order[o] : o;
    if (flag[b]) continue;
    const int2 g = G[b];
    const int4 nt = nodes[g.x], ns = nodes[g.y];
    const int c = nt.y - nt.x, q = ns.y - ns.x;
    const int l = rank[b];
    const T* F = Fs + 3 * (int64_t)ns.x;
    for (int k0 = 4 * w; k0 < l; k0 += 4 * (T256 / 64)) {
      const T* Q[4];
#pragma unroll
      for (int u = 0; u < 4; ++u)   // a term past the rank repeats the last one, unused
        Q[u] = pool + fptr[b * LMAX_CAP + min(k0 + u, l - 1)] + 9 * (int64_t)c;
      double v[12] = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
      for (int j = lane; j < q; j += 64) {
        T e[4][9];
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
          for (int d = 0; d < 9; ++d) e[u][d] = Q[u][9 * (int64_t)j + d];
        const double f0 = F[3 * j], f1 = F[3 * j + 1], f2 = F[3 * j + 2];
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
          for (int d = 0; d < 3; ++d)
            v[3 * u + d] += (double)e[u][3 * d] * f0 + (double)e[u][3 * d + 1] * f1 +
                            (double)e[u][3 * d + 2] * f2;
      }
      const WaveSums<12> s = wave_sums(v);
      if ((lane & 15) == 15) {
        const int row = lane >> 4, e0 = ((row & 1) << 1) | (row >> 1);
        double* t = tbuf + 3 * (toff[b] + k0);
#pragma unroll
        for (int r = 0; r < 3; ++r)
          if (k0 + (4 * r + e0) / 3 < l) t[4 * r + e0] = s.r[r];
      }
    }
  }
}

// Near-field row s: its partial rows in a fixed order.
template <class TU>
__device__ __forceinline__ void near_sum(const TU* __restrict__ Un, int groups, int64_t n,
                                         int64_t s, double& u0, double& u1, double& u2) {
#pragma unroll 4
  for (int g = 0; g < groups; ++g) {
    const TU* r = Un + 3 * ((int64_t)g * n + s);
    u0 += (double)r[0];
    u1 += (double)r[1];
    u2 += (double)r[2];
  }
}

template <class T>
struct FarArgs {
  const int32_t *leaf_of, *parent, *far_ptr;
  const int4* nodes;
  const int2* G;
  const int32_t *rank, *flag;
  const int64_t *fptr, *toff;
  const T* pool;
  const double* tbuf;
  const double* xs;
  const T* Fs;
  KParams kp;
  int64_t n;
  int sets;   // workgroups per 64 rows (sets of partial rows when > 1)
};

// Far field of 64 rows per workgroup, one lane per row and share: a lane walks
// from its row's leaf to the root and adds c_k(i) t_k of every admissible block
// whose target cluster holds the row, the blocks of a node dealt to the shares
// in turn (four waves, and `sets` workgroups). Every share adds in a fixed order.
// FB: blocks that fell back to dense evaluation exist. FINAL (one set): also adds
// the near-field rows and the self term and writes U in the caller's order;
// otherwise the rows of the set go to `part`. Bound by the one read of the
// factors' c halves (one lane per row walked alone, n/64 waves in all: 9.0 ms at
// 40,000 particles of the 6N form, now 3.2 ms; 2.9 to 0.39 ms at 30,000 BF16).
template <class T, class TU, class TO, int KIND, bool FB, bool FINAL>
__global__ __launch_bounds__(T256) void k_far_apply(FarArgs<T> a, const int32_t* __restrict__ perm,
                                                    const TU* __restrict__ Un, int groups,
                                                    TO* __restrict__ U, double* __restrict__ part) {
  __shared__ T wl[FB && KIND == KIND_MLP ? MLP_NP : 1];
  __shared__ double red[4 * 64 * 3];
  if (FB && KIND == KIND_MLP) {
    const T* w = (const T*)a.kp.w;
    for (int i = threadIdx.x; i < MLP_NP; i += T256) wl[i] = w[i];
    __syncthreads();
  }
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t s0 = 64 * ((int64_t)blockIdx.x / a.sets), s = s0 + lane;
  const int set = blockIdx.x % a.sets;
  const int share = 4 * set + w, shares = 4 * a.sets;
  double u[3] = {0, 0, 0};
  if (s < a.n) {
    // blocks are dealt round robin over the whole walk
    int turn = share;
    for (int tau = a.leaf_of[s]; tau >= 0; tau = a.parent[tau]) {
      const int p0 = a.far_ptr[tau], p1 = a.far_ptr[tau + 1];
      if (p0 + turn >= p1) {
        turn -= p1 - p0;
        continue;
      }
      const int il = (int)(s - a.nodes[tau].x);
      int p = p0 + turn;
      for (; p < p1; p += shares) {
        if (FB && a.flag[p]) {
          // dense fallback: evaluate the block row directly
          const int4 ns = a.nodes[a.G[p].y];
          const double x0 = a.xs[3 * s], x1 = a.xs[3 * s + 1], x2 = a.xs[3 * s + 2];
          T v0 = 0, v1 = 0, v2 = 0;
          for (int j = ns.x; j < ns.y; ++j) {
            T K[9];
            kernel_entry<T>(a.kp, wl, (T)(x0 - a.xs[3 * (int64_t)j]),
                            (T)(x1 - a.xs[3 * (int64_t)j + 1]), (T)(x2 - a.xs[3 * (int64_t)j + 2]),
                            K, (int)(s & 1), j & 1);
            T f0 = a.Fs[3 * (int64_t)j], f1 = a.Fs[3 * (int64_t)j + 1], f2 = a.Fs[3 * (int64_t)j + 2];
            v0 += K[0] * f0 + K[1] * f1 + K[2] * f2;
            v1 += K[3] * f0 + K[4] * f1 + K[5] * f2;
            v2 += K[6] * f0 + K[7] * f1 + K[8] * f2;
          }
          u[0] += v0; u[1] += v1; u[2] += v2;
          continue;
        }
        const int l = a.rank[p];
        const double* tb = a.tbuf + 3 * a.toff[p];
        const int64_t* fp = a.fptr + (int64_t)p * LMAX_CAP;
        const T* row = a.pool + 9 * (int64_t)il;
#pragma unroll 4
        for (int k = 0; k < l; ++k) {
          const T* e = row + fp[k];
          const double t0 = tb[3 * k], t1 = tb[3 * k + 1], t2 = tb[3 * k + 2];
          u[0] += (double)e[0] * t0 + (double)e[1] * t1 + (double)e[2] * t2;
          u[1] += (double)e[3] * t0 + (double)e[4] * t1 + (double)e[5] * t2;
          u[2] += (double)e[6] * t0 + (double)e[7] * t1 + (double)e[8] * t2;
        }
      }
      turn = p - p1;
    }
  }
  if (!FINAL) {
    write_rows(red, lane, w, u, s0, a.n, set, part);
    return;
  }
#pragma unroll
  for (int d = 0; d < 3; ++d) red[192 * w + 3 * lane + d] = u[d];
  __syncthreads();
  const int64_t r = s0 + threadIdx.x;
  if (threadIdx.x >= 64 || r >= a.n) return;
  double v[3] = {0, 0, 0};
  near_sum(Un, groups, a.n, r, v[0], v[1], v[2]);
  const double a1 = (r & 1) ? a.kp.alpha2 : a.kp.alpha1;
  const int64_t o = perm[r];
  const double* e = red + 3 * threadIdx.x;
#pragma unroll
  for (int d = 0; d < 3; ++d)
    U[3 * o + d] = (TO)((v[d] + (((e[d] + e[192 + d]) + e[384 + d]) + e[576 + d])) +
                        a1 * (double)a.Fs[3 * r + d]);
}

// Streamed mode: add the rows of the admissible blocks of launch r that
// contain particle s, walking from its leaf to the root (fixed order, no
// atomics). Block b's rows sit at uoff[pos[b]] - uoff[start of launch r].
__global__ __launch_bounds__(T256) void k_far_gather(
    int64_t n, const int32_t* __restrict__ leaf_of, const int32_t* __restrict__ parent,
    const int4* __restrict__ nodes, const int32_t* __restrict__ far_ptr, int32_t r,
    int64_t r0, const int32_t* __restrict__ lid, const int32_t* __restrict__ pos,
    const int64_t* __restrict__ uoff, const double* __restrict__ ublk, double* __restrict__ Uf) {
  int64_t s = (int64_t)blockIdx.x * T256 + threadIdx.x;
  if (s >= n) return;
  double u0 = 0, u1 = 0, u2 = 0;
  const int64_t base = uoff[r0];
  for (int tau = leaf_of[s]; tau >= 0; tau = parent[tau]) {
    const int p0 = far_ptr[tau], p1 = far_ptr[tau + 1];
    if (p0 >= p1) continue;
    const int64_t il = s - nodes[tau].x;
    for (int p = p0; p < p1; ++p) {
      if (lid[p] != r) continue;
      const double* u = ublk + 3 * (uoff[pos[p]] - base + il);
      u0 += u[0]; u1 += u[1]; u2 += u[2];
    }
  }
  Uf[3 * s] += u0;
  Uf[3 * s + 1] += u1;
  Uf[3 * s + 2] += u2;
}

template <class T, class TU, class TO>
__global__ __launch_bounds__(T256) void k_final(int64_t n, const int32_t* __restrict__ perm,
                                                const T* __restrict__ Fs, const TU* __restrict__ Un,
                                                int groups, const double* __restrict__ Uf,
                                                int far_sets, double alpha1, double alpha2,
                                                TO* __restrict__ U) {
  int64_t s = (int64_t)blockIdx.x * T256 + threadIdx.x;
  if (s >= n) return;
  const int64_t o = perm[s];
  const double a1 = (s & 1) ? alpha2 : alpha1;   // odd rows: rotational rows of a 6N kernel
  double u[3] = {0, 0, 0};
  near_sum(Un, groups, n, s, u[0], u[1], u[2]);
  double f[3] = {0, 0, 0};
  near_sum(Uf, far_sets, n, s, f[0], f[1], f[2]);
#pragma unroll
  for (int d = 0; d < 3; ++d) U[3 * o + d] = (TO)((u[d] + f[d]) + a1 * (double)Fs[3 * s + d]);
}

// Sets of partial rows of a product: near-field groups and far-field sets (1: the
// far field adds everything itself and needs no rows), and the bytes they take.
struct RowSets {
  int near = 1, far = 1;
};
int64_t near_bytes(hh_tree t, hh_kernel k, int prec, int groups) {
  return 3 * t->n * (int64_t)groups * (near_rows_f64(k, prec, groups) ? 8 : 4);
}
int64_t set_bytes(hh_tree t, hh_kernel k, int prec, RowSets r) {
  return (near_bytes(t, k, prec, r.near) + 255) / 256 * 256 +
         (r.far > 1 ? 3 * t->n * (int64_t)r.far * 8 : 0);
}
// Far-field sets: the walks of 64 rows by four waves, split further while that
// leaves compute units idle (8 resident workgroups each).
RowSets row_sets(hh_ctx ctx, hh_tree t, hh_part p, hh_kernel k, int prec) {
  RowSets r;
  r.near = near_groups(ctx, t, p, k, prec);
  const int64_t nw = (t->n + 63) / 64;
  if (p->nG > 0) r.far = (int)std::min<int64_t>(16, (8 * (int64_t)ctx->n_cu + nw - 1) / nw);
  return r;
}

// Stored mode. Fs_ws holds the sorted forces (3 n T), rows_ws the sets of partial
// rows; timed = false records no phase events.
template <class T, class TO>
void matvec_t(hh_ctx ctx, hh_tree t, hh_part p, hh_lowrank lr, hh_kernel k, const void* F,
              void* U, void* Fs_ws, void* rows_ws, RowSets r, bool timed) {
  hipStream_t st = ctx->stream;
  const int64_t n = t->n;
  T* Fs = (T*)Fs_ws;
  hipLaunchKernelGGL((k_gather_rows<T, T>), dim3(nblk(n)), dim3(T256), 0, st, (const T*)F,
                     t->perm.as<int32_t>(), n, Fs);
  {
    PhaseTimer timer(ctx, HH_PHASE_NEAR, timed);
    launch_near(ctx, t, p, k, lr->prec, Fs, rows_ws, r.near);
  }
  int64_t nG = p->nG;
  if (nG > 0) {
    PhaseTimer timer(ctx, HH_PHASE_FAR, timed);
    int grid = (int)std::min<int64_t>(nG, 8192);
    hipLaunchKernelGGL((k_far_t<T>), dim3(grid), dim3(T256), 0, st, p->G.as<int2>(), nG,
                       lr->order.as<int32_t>(), t->nodes.as<int4>(), lr->rank.as<int32_t>(),
                       lr->flag.as<int32_t>(), lr->fptr.as<int64_t>(), lr->toff.as<int64_t>(),
                       lr->pool.as<T>(), Fs, lr->tbuf.as<double>());
  }
  PhaseTimer timer(ctx, HH_PHASE_COMBINE, timed);
  double* part = (double*)((char*)rows_ws + (near_bytes(t, k, lr->prec, r.near) + 255) / 256 * 256);
  const bool f64 = near_rows_f64(k, lr->prec, r.near);
  if (nG > 0) {
    FarArgs<T> a;
    a.leaf_of = t->leaf_of.as<int32_t>();
    a.parent = t->parent.as<int32_t>();
    a.far_ptr = p->far_ptr.as<int32_t>();
    a.nodes = t->nodes.as<int4>();
    a.G = p->G.as<int2>();
    a.rank = lr->rank.as<int32_t>();
    a.flag = lr->flag.as<int32_t>();
    a.fptr = lr->fptr.as<int64_t>();
    a.toff = lr->toff.as<int64_t>();
    a.pool = lr->pool.as<T>();
    a.tbuf = lr->tbuf.as<double>();
    a.xs = t->xs.as<double>();
    a.Fs = Fs;
    a.kp = make_kparams(k, sizeof(T) == 8);
    a.n = n;
    a.sets = r.far;
    const dim3 grid((unsigned)((n + 63) / 64 * r.far));
    const int32_t* perm = t->perm.as<int32_t>();
    // <near-row type, kernel (read in fallbacks only), fallbacks, final>
#define FAR_APPLY(TU_, TO_, KIND_, FB_, FIN_)                                                  \
  hipLaunchKernelGGL((k_far_apply<T, TU_, TO_, KIND_, FB_, FIN_>), grid, dim3(T256), 0, st, a, \
                     perm, (const TU_*)rows_ws, r.near, (TO_*)U, part)
    const bool fb = lr->n_fallback > 0, mlp = k->kind == KIND_MLP;
    if (r.far > 1) {
      if (!fb) FAR_APPLY(double, double, KIND_RPY, false, false);
      else if (mlp) FAR_APPLY(double, double, KIND_MLP, true, false);
      else FAR_APPLY(double, double, KIND_RPY, true, false);
    } else if (f64) {
      if (!fb) FAR_APPLY(double, TO, KIND_RPY, false, true);
      else if (mlp) FAR_APPLY(double, TO, KIND_MLP, true, true);
      else FAR_APPLY(double, TO, KIND_RPY, true, true);
    } else {
      if (!fb) FAR_APPLY(T, TO, KIND_RPY, false, true);
      else if (mlp) FAR_APPLY(T, TO, KIND_MLP, true, true);
      else FAR_APPLY(T, TO, KIND_RPY, true, true);
    }
#undef FAR_APPLY
  }
  if (nG == 0 || r.far > 1) {
    const int far = nG == 0 ? 0 : r.far;
    if (f64)
      hipLaunchKernelGGL((k_final<T, double, TO>), dim3(nblk(n)), dim3(T256), 0, st, n,
                         t->perm.as<int32_t>(), Fs, (const double*)rows_ws, r.near, part, far,
                         k->alpha1, k->alpha2, (TO*)U);
    else
      hipLaunchKernelGGL((k_final<T, T, TO>), dim3(nblk(n)), dim3(T256), 0, st, n,
                         t->perm.as<int32_t>(), Fs, (const T*)rows_ws, r.near, part, far,
                         k->alpha1, k->alpha2, (TO*)U);
  }
  HIP_OK(hipGetLastError());
}

// Stored mode with the workspaces of the low-rank handle (sized on the first
// product, reused after).
template <class T, class TO>
void matvec_ws_t(hh_ctx ctx, hh_tree t, hh_part p, hh_lowrank lr, hh_kernel k, const void* F,
                 void* U) {
  const RowSets r = row_sets(ctx, t, p, k, lr->prec);
  lr->ws_f.ensure(ctx, 3 * t->n * sizeof(T));
  lr->ws_near.ensure(ctx, set_bytes(t, k, lr->prec, r));
  matvec_t<T, TO>(ctx, t, p, lr, k, F, U, lr->ws_f.p, lr->ws_near.p, r, true);
}

// Bytes of the sorted forces in the static scratch of the allocation-free
// product.
int64_t noalloc_forces(int64_t n, int prec) {
  return (3 * n * (prec == HH_FP64 ? 8 : 4) + 255) / 256 * 256;
}

// The allocation-free product: the same launches with the workspaces in the
// device's static scratch (base, HH_NOALLOC_SCRATCH_BYTES); the near-field
// sources and the far-field walks are split only if the partial rows fit.
template <class T, class TO>
void matvec_noalloc_t(hh_ctx ctx, hh_tree t, hh_part p, hh_lowrank lr, hh_kernel k,
                      const void* F, void* U, char* base) {
  const int64_t bf = noalloc_forces(t->n, lr->prec);
  RowSets r = row_sets(ctx, t, p, k, lr->prec);
  if (bf + set_bytes(t, k, lr->prec, r) > (int64_t)HH_NOALLOC_SCRATCH_BYTES) r.far = 1;
  if (bf + near_bytes(t, k, lr->prec, r.near) > (int64_t)HH_NOALLOC_SCRATCH_BYTES) r.near = 1;
  matvec_t<T, TO>(ctx, t, p, lr, k, F, U, base, base + bf, r, false);
}

template <class T, class TO>
void matvec_streamed_t(hh_ctx ctx, hh_tree t, hh_part p, hh_lowrank lr, hh_kernel k,
                       const void* F, void* U) {
  hipStream_t st = ctx->stream;
  const int64_t n = t->n;
  DevBuf& Fs = lr->ws_f;
  DevBuf& Un = lr->ws_near;
  DevBuf& Uf = lr->ws_far;
  DevBuf& counters = lr->ws_cnt;
  Fs.ensure(ctx, 3 * n * sizeof(T));
  const int groups = near_groups(ctx, t, p, k, lr->prec);
  Un.ensure(ctx, near_bytes(t, k, lr->prec, groups));
  Uf.ensure(ctx, 3 * n * sizeof(double));
  hipLaunchKernelGGL((k_gather_rows<T, T>), dim3(nblk(n)), dim3(T256), 0, st, (const T*)F,
                     t->perm.as<int32_t>(), n, Fs.as<T>());
  {
    PhaseTimer timer(ctx, HH_PHASE_NEAR);
    launch_near(ctx, t, p, k, lr->prec, Fs.p, Un.p, groups);
  }
  zero_words(ctx, Uf.p, 3 * n);
  const size_t nb = lr->bounds.size() - 1;
  counters.ensure(ctx, ACA_COUNTERS * nb * sizeof(int64_t));
  zero_words(ctx, counters.p, ACA_COUNTERS * (int64_t)nb);
  if (!lr->pool.p) lr->pool.alloc(ctx, lr->pool_elems * (lr->prec == HH_FP64 ? 8 : 4));
  if (!lr->ublk.p) lr->ublk.alloc(ctx, lr->ub_elems * 3 * sizeof(double));
  for (size_t i = 0; i < nb; ++i) {
    {
      PhaseTimer timer(ctx, HH_PHASE_ACA);
      run_aca_batch(ctx, t, p, k, lr, i, Fs.p, counters.as<int64_t>());
    }
    PhaseTimer timer(ctx, HH_PHASE_FAR);
    hipLaunchKernelGGL(k_far_gather, dim3(nblk(n)), dim3(T256), 0, st, n,
                       t->leaf_of.as<int32_t>(), t->parent.as<int32_t>(), t->nodes.as<int4>(),
                       p->far_ptr.as<int32_t>(), (int32_t)i, lr->bounds[i], lr->lid.as<int32_t>(),
                       lr->pos.as<int32_t>(), lr->uoff.as<int64_t>(), lr->ublk.as<double>(),
                       Uf.as<double>());
    HIP_OK(hipGetLastError());
  }
  {
    PhaseTimer timer(ctx, HH_PHASE_COMBINE);
    if (near_rows_f64(k, lr->prec, groups))
      hipLaunchKernelGGL((k_final<T, double, TO>), dim3(nblk(n)), dim3(T256), 0, st, n,
                         t->perm.as<int32_t>(), Fs.as<T>(), Un.as<double>(), groups,
                         Uf.as<double>(), 1, k->alpha1, k->alpha2, (TO*)U);
    else
      hipLaunchKernelGGL((k_final<T, T, TO>), dim3(nblk(n)), dim3(T256), 0, st, n,
                         t->perm.as<int32_t>(), Fs.as<T>(), Un.as<T>(), groups, Uf.as<double>(), 1,
                         k->alpha1, k->alpha2, (TO*)U);
  }
  HIP_OK(hipGetLastError());
  lr->stats_dirty = true;
}

}  // namespace

extern "C" {

hh_status hh_aca_build(hh_ctx ctx, hh_tree tree, hh_part part, hh_kernel kern,
                       hh_precision prec, double eps, int32_t l_max,
                       hh_lowrank freeze_pivots_from, hh_lowrank* out) {
  if (out) *out = nullptr;
  HH_API_BEGIN(ctx)
  HH_REQUIRE(out && tree && part && kern, HH_ERR_INVALID_ARG, "NULL argument");
  HH_REQUIRE(part->tree == tree, HH_ERR_INVALID_ARG, "partition was built on another tree");
  check_kernel_tree(tree, kern);
  HH_REQUIRE(kern->kind != KIND_RPY6 || prec == HH_FP64 || prec == HH_FP32, HH_ERR_INVALID_ARG,
             "the 6N kernel runs in HH_FP64 and HH_FP32");
  if (freeze_pivots_from) {
    // the recursion replayed with the pivots, ranks and fallbacks of an
    // earlier build on the same partition (eps and l_max unused)
    hh_lowrank src = freeze_pivots_from;
    HH_REQUIRE(src->part == part, HH_ERR_INVALID_ARG,
               "freeze_pivots_from was built on another partition");
    HH_REQUIRE(!src->streamed, HH_ERR_INVALID_ARG,
               "freeze_pivots_from must hold stored factors (streamed mode keeps none)");
    const int64_t nG = part->nG;
    std::vector<int32_t> rk(std::max<int64_t>(nG, 1)), fb(std::max<int64_t>(nG, 1));
    std::vector<int32_t> pv(std::max<int64_t>(nG, 1) * 2 * LMAX_CAP);
    std::vector<int32_t> pi(std::max<int64_t>(nG, 1) * LMAX_CAP),
        pj(std::max<int64_t>(nG, 1) * LMAX_CAP);
    if (nG > 0) {
      read_bytes(ctx, rk.data(), src->rank.p, nG * sizeof(int32_t));
      read_bytes(ctx, fb.data(), src->flag.p, nG * sizeof(int32_t));
      read_bytes(ctx, pv.data(), src->piv.p, nG * 2 * LMAX_CAP * sizeof(int32_t));
    }
    for (int64_t b = 0; b < nG; ++b)
      for (int m = 0; m < LMAX_CAP; ++m) {
        pi[b * LMAX_CAP + m] = pv[b * 2 * LMAX_CAP + m];
        pj[b * LMAX_CAP + m] = pv[b * 2 * LMAX_CAP + LMAX_CAP + m];
      }
    *out = build_lowrank_pivots(ctx, tree, part, kern, prec, rk.data(), fb.data(), pi.data(),
                                pj.data());
  } else {
    HH_REQUIRE(prec == HH_FP64 || prec == HH_FP32 || is_bf16(prec), HH_ERR_INVALID_ARG,
               "unknown precision");
    HH_REQUIRE(eps >= 0.0 && eps < INFINITY, HH_ERR_INVALID_ARG, "eps must be >= 0");
    HH_REQUIRE(l_max >= 1 && l_max <= LMAX_CAP, HH_ERR_INVALID_ARG, "l_max must be in [1, 64]");
    hh_lowrank_s* lr = new hh_lowrank_s();
    try {
      lr->ctx = ctx;
      lr->part = part;
      lr->prec = prec;
      lr->nG = part->nG;
      lr->l_max = l_max;
      lr->eps = eps;
      lr->kern = kern;
      plan_aca(ctx, tree, part, lr, 0);
      if (!lr->streamed) run_aca_stored(ctx, tree, part, kern, lr);
    } catch (...) {
      delete lr;
      throw;
    }
    *out = lr;
  }
  HH_API_END(ctx)
}

hh_status hh_matvec(hh_ctx ctx, hh_tree tree, hh_part part, hh_lowrank lr, hh_kernel kern,
                    hh_precision prec, const void* F, void* U) {
  HH_API_BEGIN(ctx)
  HH_REQUIRE(tree && part && lr && kern && F && U, HH_ERR_INVALID_ARG, "NULL argument");
  HH_REQUIRE(part->tree == tree && lr->part == part, HH_ERR_INVALID_ARG,
             "handles do not belong together");
  HH_REQUIRE(lr->prec == prec, HH_ERR_INVALID_ARG, "precision differs from the ACA build");
  HH_REQUIRE(lr->kern == kern, HH_ERR_INVALID_ARG, "kernel differs from the ACA build");
  // <storage, kernel and F type, U type>
  if (lr->streamed) {
    if (prec == HH_FP64)
      matvec_streamed_t<double, double>(ctx, tree, part, lr, kern, F, U);
    else if (prec == HH_FP32)
      matvec_streamed_t<float, float>(ctx, tree, part, lr, kern, F, U);
    else
      matvec_streamed_t<float, double>(ctx, tree, part, lr, kern, F, U);
  } else if (prec == HH_FP64) {
    matvec_ws_t<double, double>(ctx, tree, part, lr, kern, F, U);
  } else if (prec == HH_FP32) {
    matvec_ws_t<float, float>(ctx, tree, part, lr, kern, F, U);
  } else {
    matvec_ws_t<float, double>(ctx, tree, part, lr, kern, F, U);
  }
  HH_API_END(ctx)
}

hh_status hh_matvec_noalloc(hh_ctx ctx, hh_tree tree, hh_part part, hh_lowrank lr,
                            hh_kernel kern, hh_precision prec, const void* F, void* U) {
  HH_API_BEGIN(ctx)
  HH_REQUIRE(tree && part && lr && kern && F && U, HH_ERR_INVALID_ARG, "NULL argument");
  HH_REQUIRE(part->tree == tree && lr->part == part, HH_ERR_INVALID_ARG,
             "handles do not belong together");
  HH_REQUIRE(lr->prec == prec, HH_ERR_INVALID_ARG, "precision differs from the ACA build");
  HH_REQUIRE(lr->kern == kern, HH_ERR_INVALID_ARG, "kernel differs from the ACA build");
  HH_REQUIRE(ctx->noalloc_scratch, HH_ERR_HIP, "no scratch address on this device");
  char* base = (char*)ctx->noalloc_scratch;
  // the size limit first: it depends only on n, the kernel and the precision
  const int64_t n = tree->n;
  const int64_t need = noalloc_forces(n, prec) + near_bytes(tree, kern, prec, 1);
  HH_REQUIRE(need <= (int64_t)HH_NOALLOC_SCRATCH_BYTES, HH_ERR_CAPACITY,
             "hh_matvec_noalloc: " + std::to_string(n) + " particles need " +
                 std::to_string(need) + " bytes of scratch, more than the " +
                 std::to_string((int64_t)HH_NOALLOC_SCRATCH_BYTES) + " available");
  HH_REQUIRE(!lr->streamed, HH_ERR_INVALID_ARG,
             "hh_matvec_noalloc needs stored factors (streamed mode runs the ACA in the product)");
  if (prec == HH_FP64)
    matvec_noalloc_t<double, double>(ctx, tree, part, lr, kern, F, U, base);
  else if (prec == HH_FP32)
    matvec_noalloc_t<float, float>(ctx, tree, part, lr, kern, F, U, base);
  else
    matvec_noalloc_t<float, double>(ctx, tree, part, lr, kern, F, U, base);
  HH_API_END(ctx)
}

void hh_lowrank_free(hh_lowrank l) { delete l; }

hh_status hh_lowrank_info(hh_lowrank l, int64_t* n_blocks, int64_t* rank_sum,
                          int64_t* n_fallback, int64_t* samples, int64_t* bytes) {
  if (!l) return HH_ERR_INVALID_ARG;
  if (l->stats_dirty && (!l->streamed || l->pool.p)) {
    try {
      (void)hipSetDevice(l->ctx->device);
      lowrank_stats(l->ctx, l->part->tree, l->part, l, false);
    } catch (const hh_error& e) {
      l->ctx->last_error = e.msg;
      return e.st;
    }
  }
  if (n_blocks) *n_blocks = l->nG;
  if (rank_sum) *rank_sum = l->rank_sum;
  if (n_fallback) *n_fallback = l->n_fallback;
  if (samples) *samples = l->samples;
  if (bytes) *bytes = l->used_elems * (int64_t)(l->prec == HH_FP64 ? 8 : 4);
  return HH_OK;
}

hh_status hh_lowrank_export(hh_lowrank l, int32_t* rank, int32_t* fallback, int32_t* piv_i,
                            int32_t* piv_j) {
  if (!l) return HH_ERR_INVALID_ARG;
  hh_ctx ctx = l->ctx;
  HH_API_BEGIN(ctx)
  int64_t nG = l->nG;
  if (rank) read_bytes(ctx, rank, l->rank.p, nG * sizeof(int32_t));
  if (fallback) read_bytes(ctx, fallback, l->flag.p, nG * sizeof(int32_t));
  if (piv_i || piv_j) {
    std::vector<int32_t> pv(nG * 2 * LMAX_CAP);
    read_bytes(ctx, pv.data(), l->piv.p, pv.size() * sizeof(int32_t));
    for (int64_t b = 0; b < nG; ++b)
      for (int m = 0; m < LMAX_CAP; ++m) {
        if (piv_i) piv_i[b * LMAX_CAP + m] = pv[b * 2 * LMAX_CAP + m];
        if (piv_j) piv_j[b * LMAX_CAP + m] = pv[b * 2 * LMAX_CAP + LMAX_CAP + m];
      }
  }
  HH_API_END(ctx)
}

hh_status hh_lowrank_factor(hh_lowrank l, int64_t b, int32_t k, double* ck, double* qk) {
  if (!l) return HH_ERR_INVALID_ARG;
  hh_ctx ctx = l->ctx;
  HH_API_BEGIN(ctx)
  HH_REQUIRE(!l->streamed, HH_ERR_INVALID_ARG,
             "factors are not kept in streamed mode (they live only inside a batch)");
  HH_REQUIRE(b >= 0 && b < l->nG, HH_ERR_INVALID_ARG, "block index out of range");
  int32_t r;
  read_bytes(ctx, &r, l->rank.as<int32_t>() + b, sizeof(int32_t));
  HH_REQUIRE(k >= 0 && k < r, HH_ERR_INVALID_ARG, "term index out of range");
  hh_tree t = l->part->tree;
  int2 g;
  read_bytes(ctx, &g, l->part->G.as<int2>() + b, sizeof(int2));
  int4 nt, ns;
  read_bytes(ctx, &nt, t->nodes.as<int4>() + g.x, sizeof(int4));
  read_bytes(ctx, &ns, t->nodes.as<int4>() + g.y, sizeof(int4));
  int64_t off;
  read_bytes(ctx, &off, l->fptr.as<int64_t>() + b * LMAX_CAP + k, sizeof(int64_t));
  int64_t c = nt.y - nt.x, q = ns.y - ns.x;
  int64_t cnt = 9 * (c + q);
  std::vector<double> v(cnt);
  if (l->prec == HH_FP64) {
    read_bytes(ctx, v.data(), l->pool.as<double>() + off, cnt * sizeof(double));
  } else {
    std::vector<float> f(cnt);
    read_bytes(ctx, f.data(), l->pool.as<float>() + off, cnt * sizeof(float));
    for (int64_t i = 0; i < cnt; ++i) v[i] = f[i];
  }
  if (ck) for (int64_t i = 0; i < 9 * c; ++i) ck[i] = v[i];
  if (qk) for (int64_t i = 0; i < 9 * q; ++i) qk[i] = v[9 * c + i];
  HH_API_END(ctx)
}

}  // extern "C"
