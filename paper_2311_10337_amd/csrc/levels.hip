// Alg. 5 by connected components: the discrete dendrogram's level l is the
// partition of the records into components of the line graph that keeps its
// edges with w <= threshold l. The paper computes it with one
// connected-components run per threshold. By Thm 3 (at every threshold) the
// components are those of the forest rows with w <= threshold, and the sorted
// forest rows of a level are a prefix of the rows, so each level adds its
// rows to the previous level's components, whose roots its labels name:
//   W = identity
//   level l: join the labels (level l-1) of the ends of the rows
//   [p_{l-1}, p_l) in W, then every record's label = the root in W of its
//   label at level l-1 (level -1: itself).
// A join hooks a larger root under a smaller node and halving moves a link to
// a grandparent, so a parent always has a smaller id than its child and every
// component's root is its smallest member: the labels are exactly the smallest
// member ids. Only roots of the level before are looked up in W, so W is never
// copied: it lies where the last level's labels go, and no workspace is
// needed. A level streams the labels once in and once out and reads W at the
// roots: 29 levels of 2e7 records in 3.5 ms (copying the labels, joining through
// the copy and compressing it in place took 4.2).
#include "ce_internal.h"

namespace ce {

namespace {

constexpr int B = 256;
// Records per thread of the label pass, their first reads in flight together: 4
// from LI_FROM records on (82 -> 76 us a level of 2e7 records; the joins lose by
// it, 59 -> 66), 1 below, where four would leave CUs idle.
constexpr int64_t LI_FROM = int64_t(1) << 21;

__device__ inline int32_t lc_ld(const int32_t *p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ inline int32_t lc_cached(const int32_t *p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
__device__ inline void lc_st(int32_t *p, int32_t v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// The root above x. Short walks halve the path that they follow. Rows of
// records at regular intervals hook each record to the one before, all at once,
// and a row that comes later walks that whole chain by itself, one read after
// another (1e6 links: 267 ms by halving; 141 when every row looked for its
// roots before it hooked, as the chain was then still being made). So a longer
// walk reads the links of LOOK neighbouring nodes at a time, through the caches
// (a stale link is an ancestor; a root is read again), follows them as far as
// they go, and leaves a link across STRIDE such windows behind it: 32 ms.
constexpr int FIND_STEPS = 16, LOOK = 16, STRIDE = 4;
__device__ inline int32_t lc_find(int32_t *par, int32_t x) {
  for (int steps = 0; steps < FIND_STEPS; steps++) {
    const int32_t p = lc_ld(&par[x]);
    if (p == x) return x;
    const int32_t g = lc_ld(&par[p]);
    if (g == p) return p;
    lc_st(&par[x], g);
    x = g;
  }
  while (true) {
    const int32_t from = x;
    for (int w = 0; w < STRIDE; w++) {
      int32_t link[LOOK];
#pragma unroll
      for (int k = 0; k < LOOK; k++) link[k] = lc_cached(&par[x > k ? x - k : 0]);
      const int32_t top = x;
#pragma unroll
      for (int k = 0; k < LOOK; k++)  // parents are smaller: the nodes of the window are met in this order
        if (x == top - k) x = link[k];
      const int32_t p = lc_ld(&par[x]);
      if (p == x) return x;
      x = p;
    }
    lc_st(&par[from], x);
  }
}

// flag |= 1: a row names a record >= n; |= 2: the rows are not in ascending w
__global__ __launch_bounds__(B) void k_lc_check(const uint32_t *tl, const uint32_t *hd, const int64_t *w, int64_t m,
                                                int64_t n, unsigned long long *flag) {
  uint32_t f = 0;
  for (int64_t j = (int64_t)blockIdx.x * B + threadIdx.x; j < m; j += (int64_t)gridDim.x * B) {
    if (tl[j] >= (uint64_t)n || hd[j] >= (uint64_t)n) f |= 1u;
    if (j + 1 < m && w[j] > w[j + 1]) f |= 2u;
  }
  if (__any(f != 0)) {
    const uint32_t all = (uint32_t)(__any(f & 1u) ? 1u : 0u) | (uint32_t)(__any(f & 2u) ? 2u : 0u);
    if (wave_lane() == 0) atomicOr(flag, (unsigned long long)all);
  }
}

// p[l] = number of rows with w <= thr[l] (rows ascending in w)
__global__ void k_lc_bounds(const int64_t *w, int64_t m, const int64_t *thr, int q, uint64_t *p) {
  for (int l = threadIdx.x; l < q; l += blockDim.x) {
    int64_t lo = 0, hi = m;
    while (lo < hi) {
      const int64_t mid = lo + (hi - lo) / 2;
      if (w[mid] <= thr[l]) lo = mid + 1;
      else hi = mid;
    }
    p[l] = (uint64_t)lo;
  }
}

__global__ void k_lc_zero(uint64_t *p, int64_t k) {
  for (int64_t i = threadIdx.x; i < k; i += blockDim.x) p[i] = 0;
}

// every record its own root, and its own label at a first level without rows
__global__ __launch_bounds__(B) void k_lc_iota(int32_t *W, int32_t *lab, int64_t n) {
  for (int64_t x = (int64_t)blockIdx.x * B + threadIdx.x; x < n; x += (int64_t)gridDim.x * B) {
    W[x] = (int32_t)x;
    if (lab) lab[x] = (int32_t)x;
  }
}

// Joins the components of the rows [a, b). The labels before this level are
// roots, so the first attempt needs no find: it fails only when the larger one
// was hooked in this level. The smaller may have been: linking to a node that
// is no root is as good, for its root is smaller still, so the two are never
// of one component. (Finding both roots first: 4.1 ms instead of 3.5 for 29
// levels of 2e7 records.)
__global__ __launch_bounds__(B) void k_lc_union(const uint32_t *tl, const uint32_t *hd, int64_t a, int64_t b,
                                                const int32_t *prev, int32_t *W) {
  for (int64_t j = a + (int64_t)blockIdx.x * B + threadIdx.x; j < b; j += (int64_t)gridDim.x * B) {
    int32_t u = (int32_t)tl[j], v = (int32_t)hd[j];
    if (prev) {
      u = prev[u];
      v = prev[v];
    }
    while (u != v) {
      const int32_t hi = u > v ? u : v, lo = u > v ? v : u;
      if (atomicCAS(&W[hi], hi, lo) == hi) break;
      u = lc_find(W, u);
      v = lc_find(W, v);
    }
  }
}

// Every record's label: the root of its label before. No hooks run now, and
// the roots go elsewhere, so walks may shorten W and read it through the caches
// (a stale link is an ancestor all the same). Only long walks do: the stores
// of short ones go to the few nodes above everything, one after another (4e5
// records at 8 levels: 0.52 ms with halving from the first or the eighth step,
// 0.19 without). A path of 1e6 rows in one level takes 0.28 ms this way, of 2e7
// 31.5.
constexpr int LONG_WALK = 64;
template <int LI>
__global__ __launch_bounds__(B) void k_lc_labels(const int32_t *prev, int32_t *W, int64_t n, int32_t *out) {
  const int64_t i0 = (int64_t)blockIdx.x * (B * LI) + threadIdx.x;
  int32_t x[LI], p[LI];
#pragma unroll
  for (int k = 0; k < LI; k++) {
    const int64_t i = i0 + (int64_t)k * B;
    x[k] = i < n ? (prev ? prev[i] : (int32_t)i) : 0;
  }
#pragma unroll
  for (int k = 0; k < LI; k++) p[k] = lc_cached(&W[x[k]]);
#pragma unroll
  for (int k = 0; k < LI; k++) {
    const int64_t i = i0 + (int64_t)k * B;
    if (i >= n) continue;
    const int32_t x0 = x[k];
    int steps = 0;
    for (; p[k] != x[k]; steps++) {
      if (steps >= LONG_WALK) {
        const int32_t g = lc_cached(&W[p[k]]);
        if (g != p[k]) lc_st(&W[x[k]], g);
        p[k] = g;
      }
      x[k] = p[k];
      p[k] = lc_cached(&W[x[k]]);
    }
    if (steps > LONG_WALK) lc_st(&W[x0], x[k]);
    out[i] = x[k];
  }
}

// The last level's labels take W's own place: only roots are stored, so every
// value a walk reads is an ancestor and the last store to each entry is its
// root. (A halving store, an intermediate ancestor, could land after another
// thread stored the root.) The roots shorten the walks behind them: workgroups
// start in the order of the records, parents are smaller, so a walk goes no
// further than the records in flight. A path of 1e6 rows takes 0.72 ms, of 2e7
// 10.6 (with shortening by atomicMin, which no stale store could undo, 3.1 at
// 1e6).
__global__ __launch_bounds__(B) void k_lc_labels_last(const int32_t *prev, int32_t *W, int64_t n) {
  for (int64_t i = (int64_t)blockIdx.x * B + threadIdx.x; i < n; i += (int64_t)gridDim.x * B) {
    int32_t x = prev ? prev[i] : (int32_t)i;
    for (int32_t p = lc_ld(&W[x]); p != x; p = lc_ld(&W[x])) x = p;
    lc_st(&W[i], x);
  }
}

}  // namespace

}  // namespace ce

using namespace ce;

extern "C" ce_status ce_level_components(const uint32_t *msf_tail, const uint32_t *msf_head, const int64_t *msf_w,
                                         int64_t m, int64_t n, const int64_t *thresholds, int64_t q,
                                         int32_t *labels, void *stream) {
  if (n < 0 || n > 0x7fffffffLL || m < 0 || m > 0x7fffffffLL) {
    set_error("n and m must be in [0, 2^31-1]");
    return CE_EINVAL;
  }
  if (q < 0 || q > CE_MAX_THRESHOLDS) {
    set_error("num_thresholds must be in [0, CE_MAX_THRESHOLDS]");
    return CE_EINVAL;
  }
  if (q > 0 && !thresholds) {
    set_error("thresholds is NULL");
    return CE_EINVAL;
  }
  for (int64_t l = 0; l < q; l++)
    if (thresholds[l] < 0 || (l > 0 && thresholds[l] <= thresholds[l - 1])) {
      set_error("thresholds must be >= 0 and strictly increasing");
      return CE_EINVAL;
    }
  if (q == 0 || n == 0) return CE_OK;
  if (!labels || (m > 0 && (!msf_tail || !msf_head || !msf_w))) {
    set_error("labels or a row array is NULL");
    return CE_EINVAL;
  }
  hipStream_t s = (hipStream_t)stream;
  uint64_t *h = pinned_scratch();
  if (!h) {
    set_error("hipHostMalloc of the readback buffer failed");
    return CE_EDEVICE;
  }
  // device words: [0] flags, [1..q] level bounds, then the thresholds
  const size_t words = 1 + (size_t)q + (size_t)q;
  void *dev = nullptr;
  CE_HIP(hipMallocAsync(&dev, sizeof(uint64_t) * words, s));
  struct Guard {
    void *p; hipStream_t s;
    ~Guard() { (void)hipFreeAsync(p, s); (void)hipStreamSynchronize(s); }
  } guard{dev, s};
  uint64_t *flag = (uint64_t *)dev, *p = flag + 1;
  int64_t *thr = (int64_t *)(p + q);
  CE_HIP(hipMemcpyAsync(thr, thresholds, sizeof(int64_t) * q, hipMemcpyHostToDevice, s));
  CE_LAUNCH(k_lc_zero, dim3(1), dim3(64), 0, s, flag, (int64_t)(1 + q));  // flags and bounds
  if (m > 0) {
    CE_LAUNCH(k_lc_check, dim3(grid_for(m, B)), dim3(B), 0, s, msf_tail, msf_head, msf_w, m, n,
              (unsigned long long *)flag);
    CE_LAUNCH(k_lc_bounds, dim3(1), dim3(64), 0, s, msf_w, m, thr, (int)q, p);
  }
  CE_HIP(hipGetLastError());
  uint64_t *hb = h + 128;  // bytes 1024 .. 1024 + 8 (q + 1) of the page
  CE_HIP(hipMemcpyAsync(hb, dev, sizeof(uint64_t) * (1 + q), hipMemcpyDeviceToHost, s));
  CE_HIP(hipStreamSynchronize(s));
  if (hb[0] & 1) {
    set_error("a row names a record >= n");
    return CE_ERANGE;
  }
  if (hb[0] & 2) {
    set_error("rows must be in ascending w (the order of the sorted forest)");
    return CE_EINVAL;
  }
  int32_t *W = labels + (q - 1) * n;
  CE_LAUNCH(k_lc_iota, dim3(grid_for(n, B)), dim3(B), 0, s, W, q > 1 && hb[1] == 0 ? labels : nullptr, n);
  int64_t prev = 0;
  for (int64_t l = 0; l < q; l++) {
    int32_t *lab = labels + l * n;
    const int32_t *before = l > 0 ? lab - n : nullptr;
    const int64_t end = (int64_t)hb[1 + l];
    if (end < prev || end > m) {
      set_error("internal: level bounds");
      return CE_EDEVICE;
    }
    if (end > prev)
      CE_LAUNCH(k_lc_union, dim3(grid_for(end - prev, B)), dim3(B), 0, s, msf_tail, msf_head, prev, end, before, W);
    if (l == q - 1) {
      if (end > prev || l > 0) CE_LAUNCH(k_lc_labels_last, dim3(grid_for(n, B)), dim3(B), 0, s, before, W, n);
    } else if (end > prev) {
      if (n >= LI_FROM)
        CE_LAUNCH(k_lc_labels<4>, dim3((unsigned)((n + B * 4 - 1) / (B * 4))), dim3(B), 0, s, before, W, n, lab);
      else
        CE_LAUNCH(k_lc_labels<1>, dim3((unsigned)((n + B - 1) / B)), dim3(B), 0, s, before, W, n, lab);
    } else if (before) {
      CE_HIP(hipMemcpyAsync(lab, before, sizeof(int32_t) * n, hipMemcpyDeviceToDevice, s));
    }
    CE_HIP(hipGetLastError());
    prev = end;
  }
  CE_HIP(hipStreamSynchronize(s));
  return CE_OK;
}
