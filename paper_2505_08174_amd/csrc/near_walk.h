// The near-field source walk of one target: every source of every near leaf
// of the target's leaf, in the order of the near list, or one share of it.
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>

#include "internal.h"

// Workgroups of the near field: four waves, 64 targets, four shares of their
// sources; `set` numbers the workgroups of the same targets.
constexpr int NEAR_WG = 256;

struct NearTables {
  const int32_t* leaf_of;    // leaf node of every sorted row
  const int32_t* leaf_id;    // leaf rank of a node
  const int32_t* near_ptr;   // near list of a leaf
  const int4* src;           // per list entry: source rows [x, y), z sources before it in the list
  const int32_t* near_q;     // sources of a leaf's whole list
  const double* xs;
  int64_t n;
};

inline NearTables near_tables(hh_tree t, hh_part p) {
  return NearTables{t->leaf_of.as<int32_t>(), t->leaf_id.as<int32_t>(), p->near_ptr.as<int32_t>(),
                    p->near_src.as<int4>(),   p->near_q.as<int32_t>(),  t->xs.as<double>(), t->n};
}

// Share `part` of `parts` of the sources of row s's near list (consecutive in
// the list, equal up to rounding). j is always a valid row; left <= 0 when the
// share is exhausted (or empty). R = 2: s, j and the counts are particles of a
// tree with two rows each.
struct NearWalk {
  int p, j, je, left;
  bool odd;   // the list entry holds an odd number of sources
  template <int R = 1>
  __device__ __forceinline__ void start(const NearTables& t, int64_t s, int part, int parts) {
    const int leaf = t.leaf_id[t.leaf_of[R * s]];
    const int q = t.near_q[leaf] / R;
    const int len = (q + parts - 1) / parts;
    const int64_t f0 = (int64_t)part * len;
    left = (int)min((int64_t)len, (int64_t)q - f0);
    int a = t.near_ptr[leaf], b = t.near_ptr[leaf + 1] - 1;
    while (a < b) {   // the last entry that starts at or before f0
      const int m = (a + b + 1) / 2;
      if (t.src[m].z / R <= f0) a = m; else b = m - 1;
    }
    p = a;
    const int4 e = t.src[p];
    j = e.x / R + (left > 0 ? (int)(f0 - e.z / R) : 0);
    je = e.y / R;
    odd = (e.y - e.x) & 1;
  }
  // j is the last source of an odd list entry
  __device__ __forceinline__ bool unpaired() const { return odd && j + 1 == je; }
  // to the next source (stays on the last one)
  template <int R = 1>
  __device__ __forceinline__ void next(const NearTables& t) {
    --left;
    if (left > 0 && ++j == je) {
      const int4 e = t.src[++p];
      j = e.x / R;
      je = e.y / R;
      odd = (e.y - e.x) & 1;
    }
  }
};

__device__ __forceinline__ int wave_max_i(int v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = max(v, __shfl_xor(v, o, 64));
  return v;
}

// Writes the sum of the workgroup's four waves' rows (fixed order) as partial
// row `set` of the 64 targets. red: 4 x 64 x N doubles of LDS that no wave
// still reads.
template <int N, class TO>
__device__ __forceinline__ void write_rows(double* __restrict__ red, int lane, int w,
                                           const double (&u)[N], int64_t s0, int64_t n, int set,
                                           TO* __restrict__ out) {
  __syncthreads();
#pragma unroll
  for (int d = 0; d < N; ++d) red[64 * N * w + N * lane + d] = u[d];
  __syncthreads();
  for (int e = threadIdx.x; e < 64 * N; e += NEAR_WG)
    if (N * s0 + e < N * n)
      out[N * ((int64_t)set * n + s0) + e] =
          (TO)(((red[e] + red[64 * N + e]) + red[128 * N + e]) + red[192 * N + e]);
}

// Sets of partial rows: workgroups per 64 targets. Twelve rounds of resident
// workgroups (`res` per compute unit) as long as a wave's share keeps `keep`
// sources (near lists differ by up to 2.5 times their mean, and with three rounds
// the last one ran half empty: near field of 21,504 beads 10.1 -> 8.9 ms, of
// 250,000 particles 102.6 -> 96.8 ms, of 60,000 with the RPY kernel 1.26 -> 1.10 ms;
// 6 and 24 rounds are within 3% of 12), and shares down to `least` sources while
// they fill idle compute units.
inline int near_sets(hh_ctx ctx, hh_tree t, hh_part p, int res, int keep, int least) {
  const int64_t nw = (t->n + 63) / 64;
  const int64_t q = std::max<int64_t>(1, p->near_pairs / t->n);   // sources per target
  const int64_t r = (int64_t)res * ctx->n_cu;
  const int64_t even = std::min((12 * r + nw - 1) / nw, q / (4 * keep));
  const int64_t fill = std::min((r + nw - 1) / nw, q / (4 * least));
  return (int)std::max<int64_t>(1, std::max(even, fill));
}
