// Block partition, Algorithm 1, with the admissibility condition Eq. (7).
//
// The recursion of Algorithm 1 is run breadth-first: a frontier of candidate
// blocks (tau, sigma) starts at (root, root); each level is one launch that
// classifies every candidate (admissible -> P^G; both leaves -> P^H; else split
// the non-leaf side(s) into 2 or 4 sons) and appends it to the list it belongs
// to, one atomic per wave and list. The order of visits does not change the
// resulting sets, which are sorted by (tau, sigma) at the end. A level finds the
// size of its frontier on the device, so levels are launched eight at a time
// between readbacks. A level whose lists outgrow their buffers counts on, the levels
// after it do nothing, and that one level is run again with larger buffers.
// (Classification, three scans of three launches each, emission and a readback per
// level took 1.9 ms at 2,000 particles and 5.8 ms at 250,000; this walk and its sorts
// take 0.22 and 1.3 ms.)
//
// Eq. (7) on tight bounding boxes: diam^2 = (dx*dx + dy*dy) + dz*dz, the gap
// per axis g = max(0, lo_s - hi_t, lo_t - hi_s), dist^2 = (gx*gx + gy*gy) +
// gz*gz; admissible iff dist^2 > 0 and max(diam_t^2, diam_s^2) <= (eta*eta)
// dist^2. FP64, no contraction, fixed order (the result is exact-reproducible).
#include <algorithm>

#include "api_guard.h"
#include "internal.h"

#pragma clang fp contract(off)

namespace {

constexpr int T256 = 256;
inline unsigned nblk(int64_t n) { return (unsigned)((n + T256 - 1) / T256); }

__device__ __forceinline__ double diam2(const double* b) {
  double dx = b[3] - b[0], dy = b[4] - b[1], dz = b[5] - b[2];
  return (dx * dx + dy * dy) + dz * dz;
}

__device__ __forceinline__ double dist2(const double* t, const double* s) {
  double g[3];
#pragma unroll
  for (int d = 0; d < 3; ++d) g[d] = fmax(0.0, fmax(s[d] - t[d + 3], t[d] - s[d + 3]));
  return (g[0] * g[0] + g[1] * g[1]) + g[2] * g[2];
}

// Appends v of the lanes with on set to list behind its `base` entries (cap entries;
// counted past it).
__device__ __forceinline__ void append(bool on, int2 v, int2* __restrict__ list, int64_t base,
                                       unsigned long long* __restrict__ cnt, int64_t cap) {
  const uint64_t m = __ballot(on);
  if (m == 0) return;
  const int lane = threadIdx.x & 63, lead = __ffsll((unsigned long long)m) - 1;
  unsigned long long p0 = 0;
  if (lane == lead) p0 = atomicAdd(cnt, (unsigned long long)__popcll(m));
  p0 = __shfl(p0, lead, 64);
  const int64_t p = base + (int64_t)p0 + __popcll(m & (lane == 0 ? 0ull : (~0ull >> (64 - lane))));
  if (on && p < cap) list[p] = v;
}

// One level of the walk. The host knows the lists up to level0: their entries in
// P^G and P^H and the frontier of level0. cnt[3 l + 0, 1, 2]: what level l adds to P^G,
// P^H and the frontier of level l + 1, final for the levels before this one.
constexpr int BATCH = 8;   // levels between readbacks
struct Walk {
  const int4* nodes;
  const double* bbox;
  double eta2;
  int dense_mode, level0;
  int64_t nG, nH, nF;
  unsigned long long* cnt;
  int2 *G, *H, *fr[2];   // fr[l & 1]: the frontier of level l
  int64_t capG, capH, capF[2];
};

__global__ __launch_bounds__(T256) void k_level(Walk a, int level) {
  int64_t gb = a.nG, hb = a.nH, nf = a.nF;
  bool again = false;   // an earlier level outgrew its lists
#pragma unroll
  for (int k = 0; k < BATCH - 1; ++k) {   // loads of all counters in flight at once
    const int l = min(a.level0 + k, max(level - 1, 0));
    const int64_t g = a.cnt[3 * l], h = a.cnt[3 * l + 1], f = a.cnt[3 * l + 2];
    if (a.level0 + k < level) {
      gb += g;
      hb += h;
      nf = f;
      again |= gb > a.capG || hb > a.capH || nf > a.capF[(l + 1) & 1];
    }
  }
  if (again) return;
  const int2* __restrict__ fr = a.fr[level & 1];
  int2* __restrict__ next = a.fr[(level + 1) & 1];
  const int64_t capF = a.capF[(level + 1) & 1];
  unsigned long long* c = a.cnt + 3 * level;
  const int64_t step = (int64_t)gridDim.x * T256;
  for (int64_t i0 = (int64_t)blockIdx.x * T256; i0 < nf; i0 += step) {
    const int64_t i = i0 + threadIdx.x;
    const bool act = i < nf;
    int2 b = make_int2(0, 0);
    int4 nt = make_int4(0, 0, -1, -1), ns = nt;
    bool adm = false;
    if (act) {
      b = fr[i];
      nt = a.nodes[b.x];
      ns = a.nodes[b.y];
      if (!a.dense_mode) {
        const double* bt = a.bbox + 6 * (int64_t)b.x;
        const double* bs = a.bbox + 6 * (int64_t)b.y;
        const double d2 = dist2(bt, bs);
        adm = d2 > 0.0 && fmax(diam2(bt), diam2(bs)) <= a.eta2 * d2;
      }
    }
    const bool lt = nt.z < 0, ls = ns.z < 0;
    const bool split = act && !adm && !(lt && ls);
    append(act && adm, b, a.G, gb, c, a.capG);
    append(act && !adm && lt && ls, b, a.H, hb, c + 1, a.capH);
    append(split, make_int2(lt ? b.x : nt.z, ls ? b.y : ns.z), next, 0, c + 2, capF);
    append(split, make_int2(lt ? b.x : nt.w, ls ? b.y : ns.w), next, 0, c + 2, capF);
    append(split && !lt && !ls, make_int2(nt.z, ns.w), next, 0, c + 2, capF);
    append(split && !lt && !ls, make_int2(nt.w, ns.z), next, 0, c + 2, capF);
  }
}

__global__ __launch_bounds__(T256) void k_pack(const int2* __restrict__ L, int64_t m, int nb,
                                               uint64_t* __restrict__ key,
                                               uint32_t* __restrict__ val) {
  int64_t i = (int64_t)blockIdx.x * T256 + threadIdx.x;
  if (i >= m) return;
  int2 b = L[i];
  key[i] = ((uint64_t)b.x << nb) | (uint64_t)b.y;
  val[i] = (uint32_t)i;
}

__global__ __launch_bounds__(T256) void k_unpack(const uint64_t* __restrict__ key, int64_t m,
                                                 int nb, int2* __restrict__ L) {
  int64_t i = (int64_t)blockIdx.x * T256 + threadIdx.x;
  if (i >= m) return;
  uint64_t k = key[i];
  L[i] = make_int2((int)(k >> nb), (int)(k & ((1ull << nb) - 1)));
}

__global__ __launch_bounds__(T256) void k_near_ptr(const int2* __restrict__ H, int64_t nH,
                                                   const int32_t* __restrict__ leaf_id,
                                                   int64_t nl, int32_t* __restrict__ ptr) {
  int64_t p = (int64_t)blockIdx.x * T256 + threadIdx.x;
  if (p > nH) return;
  if (p == nH) { ptr[nl] = (int32_t)nH; return; }
  if (p == 0 || H[p - 1].x != H[p].x) ptr[leaf_id[H[p].x]] = (int32_t)p;
}

// Source rows of every near entry and, per leaf, the running and the total
// number of sources of its list: one wave per leaf, 64 entries at a time.
__global__ __launch_bounds__(T256) void k_near_src(const int2* __restrict__ H,
                                                   const int4* __restrict__ nodes,
                                                   const int32_t* __restrict__ ptr, int64_t nl,
                                                   int4* __restrict__ src,
                                                   int32_t* __restrict__ total) {
  const int64_t l = ((int64_t)blockIdx.x * T256 + threadIdx.x) >> 6;
  const int lane = threadIdx.x & 63;
  if (l >= nl) return;
  const int p0 = ptr[l], p1 = ptr[l + 1];
  int sum = 0;
  for (int b = p0; b < p1; b += 64) {
    const int p = b + lane;
    int4 ns = make_int4(0, 0, 0, 0);
    if (p < p1) ns = nodes[H[p].y];
    const int c = ns.y - ns.x;
    int v = c;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int u = __shfl_up(v, o, 64);
      if (lane >= o) v += u;
    }
    if (p < p1) src[p] = make_int4(ns.x, ns.y, sum + v - c, 0);
    sum += __shfl(v, 63, 64);
  }
  if (lane == 0) total[l] = sum;
}

__global__ __launch_bounds__(T256) void k_far_ptr(const int2* __restrict__ G, int64_t nG,
                                                  int64_t m, int32_t* __restrict__ ptr) {
  int64_t p = (int64_t)blockIdx.x * T256 + threadIdx.x;
  if (p > m) return;
  int64_t a = 0, b = nG;
  while (a < b) {
    int64_t mid = (a + b) / 2;
    if (G[mid].x < p) a = mid + 1; else b = mid;
  }
  ptr[p] = (int32_t)a;
}

__global__ __launch_bounds__(T256) void k_pair_sizes(const int2* __restrict__ L, int64_t m,
                                                     const int4* __restrict__ nodes,
                                                     unsigned long long* __restrict__ sum) {
  int64_t i = (int64_t)blockIdx.x * T256 + threadIdx.x;
  unsigned long long v = 0;
  if (i < m) {
    int2 b = L[i];
    int4 a = nodes[b.x], c = nodes[b.y];
    v = (unsigned long long)(a.y - a.x) * (unsigned long long)(c.y - c.x);
  }
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  if ((threadIdx.x & 63) == 0 && v) atomicAdd(sum, v);
}

// The frontier of level 0, and all counters of a walk.
__global__ void k_roots_frontier(const int32_t* __restrict__ roots, int nsys,
                                 int2* __restrict__ fr, unsigned long long* __restrict__ cnt,
                                 int ncnt) {
  int s = blockIdx.x * 256 + threadIdx.x;
  if (s < nsys) fr[s] = make_int2(roots[s], roots[s]);
  if (s < ncnt) cnt[s] = 0;
}

}  // namespace

// The m pairs of src, sorted, into dst.
static void sort_pairs(hh_ctx ctx, const int2* src, int64_t m, int nb, int2* dst) {
  if (m < 1) return;
  hipStream_t st = ctx->stream;
  DevBuf key, val;
  key.alloc(ctx, m * sizeof(uint64_t));
  val.alloc(ctx, m * sizeof(uint32_t));
  hipLaunchKernelGGL(k_pack, dim3(nblk(m)), dim3(T256), 0, st, src, m, nb, key.as<uint64_t>(),
                     val.as<uint32_t>());
  radix_sort_u64(ctx, key.as<uint64_t>(), val.as<uint32_t>(), m, 2 * nb);
  hipLaunchKernelGGL(k_unpack, dim3(nblk(m)), dim3(T256), 0, st, key.as<uint64_t>(), m, nb, dst);
  HIP_OK(hipGetLastError());
}

extern "C" {

hh_status hh_partition(hh_ctx ctx, hh_tree tree, double eta, int dense_mode, hh_part* out) {
  if (out) *out = nullptr;
  HH_API_BEGIN(ctx)
  HH_REQUIRE(out && tree, HH_ERR_INVALID_ARG, "NULL argument");
  HH_REQUIRE(eta > 0.0 && eta < INFINITY, HH_ERR_INVALID_ARG, "eta must be > 0 (Eq. (7))");
  HH_REQUIRE(tree->ctx == ctx, HH_ERR_INVALID_ARG, "tree belongs to another context");
  hipStream_t st = ctx->stream;
  PhaseTimer timer(ctx, HH_PHASE_PARTITION);
  hh_part_s* p = new hh_part_s();
  try {
    p->ctx = ctx;
    p->tree = tree;
    const int4* nodes = tree->nodes.as<int4>();
    const double* bbox = tree->bbox.as<double>();
    double eta2 = eta * eta;
    // Algorithm 1 starts at (I, I) for every independent system. Room for the
    // lists of the workloads (112 admissible and 41 inadmissible blocks per node
    // at 1M particles), more where a level needs it; in dense mode the lists of one
    // system are known (up to a GiB each here).
    constexpr int MAX_LEVELS = 200, NCNT = 3 * MAX_LEVELS;
    const int nsys = tree->n_sys;
    const int64_t m = tree->n_nodes, nl = tree->n_leaves;
    const int64_t all = dense_mode && nsys == 1 ? std::min<int64_t>(nl * nl, 1 << 27) : 0;
    DevBuf G, H, f[2], cnt;
    cnt.alloc(ctx, NCNT * sizeof(unsigned long long));
    std::vector<int64_t> c(NCNT);
    Walk w = {};
    w.nodes = nodes;
    w.bbox = bbox;
    w.eta2 = eta2;
    w.dense_mode = dense_mode;
    w.cnt = cnt.as<unsigned long long>();
    w.capG = all > 0 ? 1 : 160 * m + 1024;
    w.capH = std::max<int64_t>(all, 64 * m + 1024);
    w.capF[0] = w.capF[1] = std::max<int64_t>({160 * m + 1024, nsys, all});
    G.alloc(ctx, w.capG * sizeof(int2));
    H.alloc(ctx, w.capH * sizeof(int2));
    for (int i = 0; i < 2; ++i) {
      f[i].alloc(ctx, w.capF[i] * sizeof(int2));
      w.fr[i] = f[i].as<int2>();
    }
    hipLaunchKernelGGL(k_roots_frontier, dim3((std::max(nsys, NCNT) + 255) / 256), dim3(256), 0,
                       st, tree->roots.as<int32_t>(), nsys, w.fr[0], w.cnt, NCNT);
    // room for `need` entries of a list that holds `has`
    auto grow = [&](DevBuf& list, int64_t& cap, int64_t has, int64_t need) {
      if (need <= cap) return;
      cap = std::max(2 * cap, need + need / 4);
      DevBuf old;
      old.take(list);
      list.alloc(ctx, cap * sizeof(int2));
      if (has > 0)
        HIP_OK(hipMemcpyAsync(list.p, old.p, has * sizeof(int2), hipMemcpyDeviceToDevice, st));
    };
    for (w.nF = nsys; w.nF > 0;) {
      HH_REQUIRE(w.level0 < MAX_LEVELS, HH_ERR_CAPACITY, "partition deeper than 200 levels");
      w.G = G.as<int2>();
      w.H = H.as<int2>();
      for (int i = 0; i < 2; ++i) w.fr[i] = f[i].as<int2>();
      const unsigned grid = (unsigned)std::min<int64_t>(
          4 * (int64_t)ctx->n_cu, nblk(std::max(w.capF[0], w.capF[1])));
      const int end = std::min(w.level0 + BATCH, MAX_LEVELS);
      for (int l = w.level0; l < end; ++l)
        hipLaunchKernelGGL(k_level, dim3(grid), dim3(T256), 0, st, w, l);
      HIP_OK(hipGetLastError());
      const int l0 = w.level0;
      read_bytes(ctx, c.data() + 3 * l0, w.cnt + 3 * l0, 3 * (end - l0) * sizeof(int64_t));
      for (; w.level0 < end && w.nF > 0; ++w.level0) {
        const int l = w.level0, o = (l + 1) & 1;
        const int64_t ng = w.nG + c[3 * l], nh = w.nH + c[3 * l + 1], nf = c[3 * l + 2];
        HH_REQUIRE(ng < (1ll << 31) && nh < (1ll << 31) && nf < (1ll << 31), HH_ERR_CAPACITY,
                   "block lists exceed 2^31 entries");
        if (ng > w.capG || nh > w.capH || nf > w.capF[o]) {
          grow(G, w.capG, w.nG, ng);
          grow(H, w.capH, w.nH, nh);
          grow(f[o], w.capF[o], 0, nf);
          zero_words(ctx, w.cnt + 3 * l, 3);
          break;
        }
        w.nG = ng;
        w.nH = nh;
        w.nF = nf;
      }
    }
    p->nG = w.nG;
    p->nH = w.nH;
    p->G.alloc(ctx, std::max<int64_t>(1, p->nG) * sizeof(int2));
    p->H.alloc(ctx, std::max<int64_t>(1, p->nH) * sizeof(int2));
    int nb = 1;
    while ((1ll << nb) < tree->n_nodes) ++nb;
    sort_pairs(ctx, G.as<int2>(), p->nG, nb, p->G.as<int2>());
    sort_pairs(ctx, H.as<int2>(), p->nH, nb, p->H.as<int2>());
    p->near_ptr.alloc(ctx, (tree->n_leaves + 1) * sizeof(int32_t));
    p->far_ptr.alloc(ctx, (tree->n_nodes + 1) * sizeof(int32_t));
    hipLaunchKernelGGL(k_near_ptr, dim3(nblk(p->nH + 1)), dim3(T256), 0, st, p->H.as<int2>(),
                       p->nH, tree->leaf_id.as<int32_t>(), tree->n_leaves,
                       p->near_ptr.as<int32_t>());
    p->near_src.alloc(ctx, std::max<int64_t>(1, p->nH) * sizeof(int4));
    p->near_q.alloc(ctx, tree->n_leaves * sizeof(int32_t));
    hipLaunchKernelGGL(k_near_src, dim3(nblk(64 * tree->n_leaves)), dim3(T256), 0, st,
                       p->H.as<int2>(), nodes, p->near_ptr.as<int32_t>(), tree->n_leaves,
                       p->near_src.as<int4>(), p->near_q.as<int32_t>());
    hipLaunchKernelGGL(k_far_ptr, dim3(nblk(tree->n_nodes + 1)), dim3(T256), 0, st,
                       p->G.as<int2>(), p->nG, tree->n_nodes, p->far_ptr.as<int32_t>());
    unsigned long long* sums = (unsigned long long*)ctx->scratch_flag.p;
    HIP_OK(hipMemsetAsync(sums, 0, 2 * sizeof(unsigned long long), st));
    if (p->nH)
      hipLaunchKernelGGL(k_pair_sizes, dim3(nblk(p->nH)), dim3(T256), 0, st, p->H.as<int2>(),
                         p->nH, nodes, sums);
    if (p->nG)
      hipLaunchKernelGGL(k_pair_sizes, dim3(nblk(p->nG)), dim3(T256), 0, st, p->G.as<int2>(),
                         p->nG, nodes, sums + 1);
    HIP_OK(hipGetLastError());
    HIP_OK(hipMemcpyAsync(ctx->pinned, sums, 16, hipMemcpyDeviceToHost, st));
    ctx_sync(ctx);
    p->near_pairs = ctx->pinned[0];
    p->far_entries = ctx->pinned[1];
  } catch (...) {
    delete p;
    throw;
  }
  *out = p;
  HH_API_END(ctx)
}

void hh_part_free(hh_part p) { delete p; }

hh_status hh_part_info(hh_part p, int64_t* nG, int64_t* nH) {
  if (!p) return HH_ERR_INVALID_ARG;
  if (nG) *nG = p->nG;
  if (nH) *nH = p->nH;
  return HH_OK;
}

hh_status hh_part_stats(hh_part p, int64_t* near_pairs, int64_t* far_entries) {
  if (!p) return HH_ERR_INVALID_ARG;
  if (near_pairs) *near_pairs = p->near_pairs;
  if (far_entries) *far_entries = p->far_entries;
  return HH_OK;
}

hh_status hh_part_export(hh_part p, int32_t* G, int32_t* H) {
  if (!p) return HH_ERR_INVALID_ARG;
  hh_ctx ctx = p->ctx;
  HH_API_BEGIN(ctx)
  if (G) read_bytes(ctx, G, p->G.p, p->nG * sizeof(int2));
  if (H) read_bytes(ctx, H, p->H.p, p->nH * sizeof(int2));
  HH_API_END(ctx)
}

}  // extern "C"
