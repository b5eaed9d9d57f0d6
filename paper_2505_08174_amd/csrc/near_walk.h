// The near-field source walk of one target: every source of every near leaf
// of the target's leaf, in the order of the near list, or one share of it.
#pragma once

#include <hip/hip_runtime.h>

#include "internal.h"

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
// share is exhausted (or empty).
struct NearWalk {
  int p, j, je, left;
  bool odd;   // the list entry holds an odd number of sources
  __device__ __forceinline__ void start(const NearTables& t, int64_t s, int part, int parts) {
    const int leaf = t.leaf_id[t.leaf_of[s]];
    const int q = t.near_q[leaf];
    const int len = (q + parts - 1) / parts;
    const int64_t f0 = (int64_t)part * len;
    left = (int)min((int64_t)len, (int64_t)q - f0);
    int a = t.near_ptr[leaf], b = t.near_ptr[leaf + 1] - 1;
    while (a < b) {   // the last entry that starts at or before f0
      const int m = (a + b + 1) / 2;
      if (t.src[m].z <= f0) a = m; else b = m - 1;
    }
    p = a;
    const int4 e = t.src[p];
    j = e.x + (left > 0 ? (int)(f0 - e.z) : 0);
    je = e.y;
    odd = (e.y - e.x) & 1;
  }
  // j is the last source of an odd list entry
  __device__ __forceinline__ bool unpaired() const { return odd && j + 1 == je; }
  // to the next source (stays on the last one)
  __device__ __forceinline__ void next(const NearTables& t) {
    --left;
    if (left > 0 && ++j == je) {
      const int4 e = t.src[++p];
      j = e.x;
      je = e.y;
      odd = (e.y - e.x) & 1;
    }
  }
};
