// Stages A1-A6: validate, group-and-sort by (vertex, time), emit the path
// skeleton, Boruvka minimum spanning forest, sort the MSF by canonical key.
//
// Grouping (the per-vertex incidence lists of Alg. 3, time-sorted as in Alg. 2): the records
// are first sorted once by (t, id) with a stable radix sort on t - tmin; the
// position in that order is the record's rank. The 2n incidence entries
// (vertex, 2*rank+side) are then stably radix-sorted by vertex, so every
// vertex's list comes out in rank order, i.e. time order with ties by id,
// whatever its degree (hubs need no special splitting).
//
// Skeleton (Alg. 3 with the undirected node-local MST of Sec. 5.3): each list
// entry after the first links to its predecessor. The edge is stored at slot
// 2*head+side of its HEAD rank, so a record is the head of at most two skeleton
// edges. Its 64-bit key packs the canonical key (w, head id, 2^32-1-tail id):
//     key = w << (idbits+1) | head_id << 1 | bit
// where bit orders the (at most two) edges sharing a head by descending tail
// id. Edges with equal keys (a pair consecutive in both endpoint lists) are
// the same line-graph edge; one copy is dropped.
#include <algorithm>

#include "ce_internal.h"

namespace ce {

namespace {

constexpr int B = 256;

__device__ inline uint64_t t_to_ord(int64_t t) { return (uint64_t)t ^ (uint64_t(1) << 63); }

// hdr[0] |= 1 self loop, 2 id out of range; hdr[1] = min t (ordered), hdr[2] = max t (ordered).
// A record of graph g must name vertices in [0, voff[g+1] - voff[g]).
// At most 512 workgroups: each ends with two updates of one address, about 15
// ns apart (4 000 workgroups of 256 spent 92 us on 1e6 records).
__global__ __launch_bounds__(VB) void k_validate(const int32_t *src, const int32_t *dst, const int64_t *t, int64_t n,
                                                 const int64_t *eoff, const int64_t *voff, int64_t G,
                                                 uint64_t *hdr) {
  uint64_t mn = NONE64, mx = 0;
  uint32_t flag = 0;
  for (int64_t i = (int64_t)blockIdx.x * VB + threadIdx.x; i < n; i += (int64_t)gridDim.x * VB) {
    int32_t a = src[i], b = dst[i];
    const uint32_t g = G > 1 ? graph_of(eoff, G, i) : 0u;
    const int64_t V = voff[g + 1] - voff[g];
    if (a == b) flag |= 1u;
    if (a < 0 || b < 0 || (int64_t)a >= V || (int64_t)b >= V) flag |= 2u;
    uint64_t o = t_to_ord(t[i]);
    mn = o < mn ? o : mn;
    mx = o > mx ? o : mx;
  }
  put_validation(mn, mx, flag, hdr);
}

__global__ void k_init_hdr(uint64_t *hdr, OneGraph og) { init_hdr(hdr, og); }

// After validation: a time span wider than the plan's tbits bits is an error too (the keys would not fit).
__global__ void k_check_span(uint64_t *hdr, int64_t n, int tbits) {
  if (threadIdx.x != 0 || n == 0) return;
  const uint64_t span = hdr[H_TMAX] - hdr[H_TMIN];
  if (tbits < 64 && (span >> tbits) != 0) hdr[H_STATUS] |= 8;
}

__device__ inline int64_t tmin_of(const uint64_t *hdr) { return (int64_t)(hdr[H_TMIN] ^ (uint64_t(1) << 63)); }

// the time sort carries (id, src, dst) along, so grouping needs no gathers;
// vertex ids become global (graph offset + local id)
__global__ __launch_bounds__(B) void k_tkeys(const int64_t *t, const int32_t *src, const int32_t *dst, int64_t n,
                                             const int64_t *eoff, const int64_t *voff, int64_t G,
                                             const uint64_t *hdr, uint64_t *keys, uint4 *vals) {
  const int64_t tmin = tmin_of(hdr);
  for (int64_t i = (int64_t)blockIdx.x * B + threadIdx.x; i < n; i += (int64_t)gridDim.x * B) {
    const uint32_t g = G > 1 ? graph_of(eoff, G, i) : 0u;
    const uint32_t vb = (uint32_t)voff[g];
    keys[i] = (uint64_t)(t[i] - tmin);
    vals[i] = make_uint4((uint32_t)i, vb + (uint32_t)src[i], vb + (uint32_t)dst[i], 0u);
  }
}

// incidence entries in rank order: key = vertex, value (implicit) = 2r+side
// (times of up to 32 bits: the id joins them, as in the packed sort)
__global__ __launch_bounds__(B) void k_incidence(const uint4 *vals, int64_t n, bool pack, uint64_t *ts, uint32_t *perm,
                                                 uint32_t *ikey) {
  for (int64_t r = (int64_t)blockIdx.x * B + threadIdx.x; r < n; r += (int64_t)gridDim.x * B) {
    const uint4 v = vals[r];
    perm[r] = v.x;
    if (pack) ts[r] = (ts[r] << 32) | v.x;
    ikey[2 * r] = v.y;
    ikey[2 * r + 1] = v.z;
  }
}

// One graph whose time span fits 32 bits: the id rides in the key's low half,
// key = (t - tmin) << 32 | id, and the value is (src | dst << 32), so a radix
// pass over bits [32, 32 + bits(span)) moves 16 bytes per record instead of 24.
// Stability keeps ids in order within equal times either way.
__global__ __launch_bounds__(B) void k_tkeys_packed(const int64_t *t, const int32_t *src, const int32_t *dst,
                                                    int64_t n, const uint64_t *hdr, uint64_t *keys, uint64_t *vals) {
  const int64_t tmin = tmin_of(hdr);
  for (int64_t i = (int64_t)blockIdx.x * B + threadIdx.x; i < n; i += (int64_t)gridDim.x * B) {
    keys[i] = ((uint64_t)(t[i] - tmin) << 32) | (uint64_t)i;
    vals[i] = (uint64_t)(uint32_t)src[i] | ((uint64_t)(uint32_t)dst[i] << 32);
  }
}

// incidence entries from the packed sort; its keys stay as they are, in ts (keys may be ts itself)
__global__ __launch_bounds__(B) void k_incidence_packed(const uint64_t *keys, const uint64_t *vals, int64_t n,
                                                        uint64_t *ts, uint32_t *perm, uint32_t *ikey) {
  for (int64_t r = (int64_t)blockIdx.x * B + threadIdx.x; r < n; r += (int64_t)gridDim.x * B) {
    const uint64_t k = keys[r], v = vals[r];
    if (ts != keys) ts[r] = k;
    perm[r] = (uint32_t)k;
    ikey[2 * r] = (uint32_t)v;
    ikey[2 * r + 1] = (uint32_t)(v >> 32);
  }
}

// every incidence entry names its slot; the entry's neighbours in the same
// vertex list go there: before it the tail of its skeleton edge, after it the
// head of the edge whose tail it is (NONE at the list's ends). A scattered
// write costs a 32-byte transaction whatever its width.
// (an input that failed validation gets an empty skeleton, so everything after
// it runs on n isolated records and stays in bounds whatever the input held)
__global__ __launch_bounds__(B) void k_skel_links(const uint32_t *ikey, const uint32_t *ival, int64_t n2,
                                                  const uint64_t *hdr, uint2 *link) {
  const bool bad = hdr[H_STATUS] != 0;
  for (int64_t k = (int64_t)blockIdx.x * B + threadIdx.x; k < n2; k += (int64_t)gridDim.x * B) {
    const uint32_t v = ikey[k];
    uint2 l = make_uint2(NONE32, NONE32);
    if (!bad && k > 0 && ikey[k - 1] == v) l.x = ival[k - 1] >> 1;
    if (!bad && k + 1 < n2 && ikey[k + 1] == v) l.y = ival[k + 1] >> 1;
    link[ival[k]] = l;
  }
}

// Keys of a record's two skeleton edges as a head, and its first Boruvka
// minimum: every record starts as its own component, and its edges are the
// two it heads and the two it is the tail of.
// The low bit orders the two edges of a head by descending tail id; it only
// decides their order when they have the same weight (else w does), so the
// tails' ids are read only then. As a tail a record offers itself the key
// with that bit zero: no other edge of its has the same weight and head, so
// the choice is the same, and the first round compares without the bit.
// (Each head offering its keys to its tails instead, two atomics a record, took
// 3.84 ms at 5e7 records with burst-local tails, 15.8 at 2e8 and 88 at 2^30;
// reading the heads' times and ids takes 1.7, 9.2 and 77, and the wider links
// 1.0, 0.8 and 1.5 more.)
// PACKED: time and id of a rank in one word, time << 32 | id (times of up to 32
// bits), one random read a neighbour; with ids from perm it is 2.3, 14.2 and 112.
// Weight ranks (wraw set): the keys get their tie bits only, the weights go
// to wraw, and the minima wait for the ranks.
// The links lie where the keys go; a thread reads its own two first.
template <bool PACKED>
__global__ __launch_bounds__(B) void k_skel_keys(const uint64_t *ts, const uint32_t *perm, int64_t n, int idbits,
                                                 uint64_t *skel_key, uint2 *skel_tail, uint64_t *best,
                                                 uint64_t *wraw) {
  constexpr int TS = PACKED ? 32 : 0;
  for (int64_t h = (int64_t)blockIdx.x * B + threadIdx.x; h < n; h += (int64_t)gridDim.x * B) {
    const uint4 l = ((const uint4 *)skel_key)[h];
    const uint32_t t0 = l.x, t1 = l.z == l.x ? NONE32 : l.z;  // the same pair twice: one line-graph edge
    skel_tail[h] = make_uint2(t0, t1);
    const uint64_t xh = ts[h], th = xh >> TS, hid = PACKED ? (uint32_t)xh : perm[h];
    const uint64_t x0 = t0 != NONE32 ? ts[t0] : 0, x1 = t1 != NONE32 ? ts[t1] : 0;
    const uint64_t w0 = t0 != NONE32 ? th - (x0 >> TS) : 0, w1 = t1 != NONE32 ? th - (x1 >> TS) : 0;
    uint64_t b0 = 0, b1 = 0;
    if (t0 != NONE32 && t1 != NONE32 && w0 == w1) {
      const uint32_t i0 = PACKED ? (uint32_t)x0 : perm[t0], i1 = PACKED ? (uint32_t)x1 : perm[t1];
      b0 = i0 < i1 ? 1u : 0u;
      b1 = 1u - b0;
    }
    ulonglong2 k;
    if (wraw) {
      k.x = t0 != NONE32 ? (hid << 1) | b0 : NONE64;
      k.y = t1 != NONE32 ? (hid << 1) | b1 : NONE64;
      ((ulonglong2 *)skel_key)[h] = k;
      wraw[2 * h] = w0;
      wraw[2 * h + 1] = w1;
      best[h] = NONE64;
      continue;
    }
    k.x = t0 != NONE32 ? (w0 << (idbits + 1)) | (hid << 1) | b0 : NONE64;
    k.y = t1 != NONE32 ? (w1 << (idbits + 1)) | (hid << 1) | b1 : NONE64;
    ((ulonglong2 *)skel_key)[h] = k;
    uint64_t mine = k.x < k.y ? k.x : k.y;
#pragma unroll
    for (int side = 0; side < 2; side++) {
      const uint32_t x = side ? l.w : l.y;  // the head of an edge whose tail h is
      if (x == NONE32 || (side && l.w == l.y)) continue;
      const uint64_t y = ts[x];
      const uint64_t f = (((y >> TS) - th) << (idbits + 1)) | ((uint64_t)(PACKED ? (uint32_t)y : perm[x]) << 1);
      mine = f < mine ? f : mine;
    }
    best[h] = mine;
  }
}

// ---------------------------------------------------------------- Boruvka
// Every component that ever exists is a node: the records are nodes 0..n-1,
// and each round gives the components it forms the next free ids. best[x] is
// the minimum key leaving node x, bpar[x] the node of the component x merged
// into (x itself while it is a component of its own). Together they are the
// Boruvka tree: at most 2n nodes, parents after children, as deep as there
// were rounds.
//
// Round 1 runs on records (best[] was seeded while emitting the skeleton).
// Each later round runs on a contracted graph: live edges are records (key,
// endpoint nodes, slot), and the nodes of a round are a contiguous range
// [LO, HI), so its passes shrink with the components.
//
// One round is one slot of five kernels:
//   k_bv_min       minimum key per node over the live edges
//   k_bv_hook      every edge that is its endpoint's minimum hooks it
//   k_bv_compress  every node to the root of its hooks; roots get new ids
//                  (where nodes are many, after k_bv_links)
//   k_bv_link      bpar of every node = the new id of its root
//   k_contract     edges between different components, renamed
// preceded by k_bv_ctl, one workgroup that advances the state (live edges E,
// the node range, a filter split) from the counters of the slot before it.
// (With the state advanced by the last workgroup of the contraction, found by
// a ticket, and one counter update per 256-edge tile, 4096 workgroups queued
// at two addresses for about 15 ns each: a round of 1e6 edges took 145 us in
// its contraction alone, now 14. With that step alone a 1e6-record call went
// from 7.5 to 4.65 ms, a 2e5-record call from 2.74 to 2.04 ms, 5e7 records from
// 89.6 to 84.4 ms.) Every kernel reads the state when it starts; the host
// enqueues a number of slots that depends on sizes alone, and those after the
// forest is complete return at once.

// Boruvka state, words H_BV + k of the control block
enum : int {
  BV_ACT = 0,      // what this slot does: 0 nothing, 1 a round, 2 a filter split, 3 the heavy edges of the split
                   // (the listing of the forest's rows looks at it too)
  BV_E = 1,        // live edges of the current list
  BV_IN = 2,       // the list: edge buffer 0 or 1, or 2 = the skeleton rows themselves
  BV_OFF = 3,      // its first entry in that buffer
  BV_LO = 4,       // nodes of this round: [LO, HI)
  BV_HI = 5,
  BV_NB = 6,       // next free node id (a counter while a round runs)
  BV_MARK = 7,     // the range holds merged nodes too (rootc names another node for them)
  BV_LIGHT = 8,    // rounds run on the light edges of a split
  BV_SPLITDONE = 9,  // splits so far, MAX_SPLITS at most
  BV_PIVOT = 10,
  BV_SLO = 11,     // LO at the split
  BV_HB = 12,      // buffer holding the heavy edges at its back
  BV_EH = 13,      // heavy edges
  BV_CNT1 = 14, BV_CNT2 = 15,  // list counters
  BV_FIRST = 16,   // the first contraction splits its list at the pivot
  BV_WORDS = 24
};
enum : int { ACT_NONE = 0, ACT_ROUND = 1, ACT_SPLIT = 2, ACT_HEAVY = 3 };

struct EdgeLists {
  uint64_t *key[3];
  uint32_t *u[3], *v[3], *s[3];  // s[2] == nullptr: the slot of a skeleton row is its index
  int64_t cap;                   // entries of buffers 0 and 1
};

// the live list of the current round
struct Live {
  const uint64_t *key;
  const uint32_t *u, *v, *s;
  int64_t E;
};
__device__ inline Live live_list(const EdgeLists &L, const uint64_t *bv) {
  const int in = (int)bv[BV_IN];
  const int64_t off = (int64_t)bv[BV_OFF];
  return Live{L.key[in] + off, L.u[in] + off, L.v[in] + off, L.s[in] ? L.s[in] + off : nullptr, (int64_t)bv[BV_E]};
}
__device__ inline int out_buffer(const uint64_t *bv) {
  const int in = (int)bv[BV_IN];
  return in == 2 ? 0 : 1 - in;
}

// a round made the nodes up to nb: one more level of the tree
__device__ inline void bv_level(uint64_t *bv, uint64_t nb) {
  const uint64_t l = ++bv[H_BV_NLEV - H_BV];
  bv[H_LEV - H_BV + l] = nb;
}

// Before the first round: the state, every record a component of its own.
// Flat skeletons start as the live list (rows, counted on the device) of a
// round over the records, with no forest edge yet.
__global__ __launch_bounds__(B) void k_bv_start(int64_t n, int64_t slots, bool flat, const uint64_t *rows,
                                                uint8_t *msf_flag, uint32_t *bpar, uint64_t *bv) {
  const int64_t step = (int64_t)gridDim.x * B, i0 = (int64_t)blockIdx.x * B + threadIdx.x;
  for (int64_t r = i0; r < n; r += step) bpar[r] = (uint32_t)r;
  if (flat)  // the flags' region is a multiple of 256 bytes
    for (int64_t e = i0; e < (slots + 3) / 4; e += step) ((uint32_t *)msf_flag)[e] = 0u;
  if (blockIdx.x == 0 && threadIdx.x < BV_WORDS) {
    const int k = threadIdx.x;
    if (k == 0) {
      bv[H_LEV - H_BV] = (uint64_t)n;
      bv[H_BV_NLEV - H_BV] = 0;
    }
    bv[k] = k == BV_ACT ? ACT_ROUND : k == BV_E ? (flat ? *rows : 0) : k == BV_IN ? 2 : (k == BV_HI || k == BV_NB)
                                                                                          ? (uint64_t)n : 0;
  }
}

// First round, on records, per head: an edge that is the minimum of its head
// or its tail hooks that record onto the other (of a mutual pair the tail,
// the smaller one, stays) and joins the forest. Keys are unique, so one edge
// writes each record's hook. Streams the skeleton and reads the tails' minima;
// the flags say who chose the edge, so the dendrogram need not ask again. At
// 5e7 records 1.7 ms; finding each record's minimum edge from its key took 2.1
// and a rank for every input id 0.8 more.
__device__ inline uint8_t hook_first(uint64_t k, uint32_t t, uint32_t h, uint64_t bh, uint64_t bt, uint32_t *bpar) {
  if (k == NONE64) return 0;
  const bool ph = bh == k, pt = (bt ^ k) < 2;  // (a tail's minimum may lack the key's low bit)
  if (ph) bpar[h] = t;
  else if (pt) bpar[t] = h;
  else return 0;
  return (uint8_t)(MSF_EDGE | MSF_FIRST | (ph ? MSF_HEAD : 0) | (pt ? MSF_TAIL : 0));
}
__global__ __launch_bounds__(B) void k_bv_hook_first(int64_t n, const uint64_t *best, const ulonglong2 *skel_key,
                                                     const uint2 *skel_tail, uint32_t *bpar, uchar2 *msf_flag) {
  for (int64_t h = (int64_t)blockIdx.x * B + threadIdx.x; h < n; h += (int64_t)gridDim.x * B) {
    const ulonglong2 k = skel_key[h];
    const uint2 t = skel_tail[h];
    const uint64_t bh = best[h];
    const uint64_t b0 = k.x != NONE64 ? best[t.x] : 0, b1 = k.y != NONE64 ? best[t.y] : 0;
    uchar2 f;
    f.x = hook_first(k.x, t.x, (uint32_t)h, bh, b0, bpar);
    f.y = hook_first(k.y, t.y, (uint32_t)h, bh, b1, bpar);
    msf_flag[h] = f;
  }
}

// Later rounds, per edge: an edge that is its endpoint's minimum hooks it.
// Copies of one line-graph edge carry equal keys (hypergraphs): the
// compare-and-swap lets one of them in. On the skeleton's own rows (the first
// round of the flat modes) the flags say who chose the edge, as above: the
// dendrogram's gather takes 0.97 ms at 8e6 causal records without, 0.59 with.
__device__ inline uint8_t bv_hook_edge(uint64_t k, uint32_t u, uint32_t v, const uint64_t *best, uint32_t *bpar) {
  const bool pu = best[u] == k, pv = best[v] == k;
  bool won = false;
  if (pu && !(pv && u < v)) won |= atomicCAS(&bpar[u], u, v) == u;
  if (pv && !(pu && v < u)) won |= atomicCAS(&bpar[v], v, u) == v;
  return won ? (uint8_t)(MSF_EDGE | (pv ? MSF_HEAD : 0) | (pu ? MSF_TAIL : 0)) : (uint8_t)0;
}
__global__ __launch_bounds__(B) void k_bv_hook(EdgeLists L, const uint64_t *bv, const uint64_t *best, uint32_t *bpar,
                                               uint8_t *msf_flag) {
  if (bv[BV_ACT] != ACT_ROUND) return;
  const Live lv = live_list(L, bv);
  for (int64_t i = (int64_t)blockIdx.x * B + threadIdx.x; i < lv.E; i += (int64_t)gridDim.x * B) {
    const uint8_t f = bv_hook_edge(lv.key[i], lv.u[i], lv.v[i], best, bpar);
    if (!f) continue;
    if (lv.s) msf_flag[lv.s[i]] = MSF_EDGE;
    else msf_flag[i] = f | MSF_FIRST;  // the skeleton's rows: tail u, head v
  }
}

// The root of the hooks above node x. The walk halves the path it follows (each
// store moves a link to a grandparent), so long hook chains shrink as in
// pointer jumping; a stale link is still an ancestor, so every walk ends at the
// root (hooks form a forest: keys are unique, and of a mutual pair only one
// side hooks). The root goes to an array of its own, which no halving store
// touches. A walk longer than any forest allows marks the call failed.
constexpr uint32_t MAX_WALK = 1u << 26;
__device__ inline uint32_t link_ld(const uint32_t *p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ inline void link_st(uint32_t *p, uint32_t v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ inline uint32_t bv_root(uint32_t *bpar, uint32_t x, uint64_t *hdr) {
  for (uint32_t steps = 0;; steps++) {
    const uint32_t p = link_ld(&bpar[x]);
    if (p == x) return x;
    const uint32_t gp = link_ld(&bpar[p]);
    if (gp != p) link_st(&bpar[x], gp);
    x = gp;
    if (steps > MAX_WALK) {
      atomicOr((unsigned long long *)&hdr[H_STATUS], 16ull);
      return x;
    }
  }
}

// rootc[c - LO] = the root of node c, or for a root the new node's id; NONE for
// a node without edges and (after the heavy edges of a split, when the range
// holds nodes merged in earlier rounds) for a merged one. Before the heavy
// edges are contracted, every node's top: several heavy edges end in one node,
// so a climb per node and one read per end take 0.9 ms of a 5e7-record call
// where climbing from each end took 2.0 (and 6.7 ms less of a 2e8-record one).
//
// Records at regular intervals hook into one chain of neighbours, millions of
// links long. A tile first jumps along the links inside it, in LDS, so that a
// chain crosses a tile of up to 4096 nodes in one step: 2e6 such records of one
// vertex took 9.2 ms with walks alone, now 1.8. That holds while all tiles are
// in flight together; else a walk comes to tiles that have not been started
// (8e6 such records: 3.3 s, or 14.6 with hooks towards later ones). So past as
// many nodes as 512 tiles hold, which two workgroups a CU cover, the links of
// all tiles are shortened by a launch of its own before the walks: 4.6 and 7.1
// ms. Up to 2^18 nodes, one a thread, the walks do alone: a chain of all of them
// costs 0.05 ms, while the barriers took 2 % of any 7e4-record call. Other
// inputs take the same time either way.
constexpr int64_t BV_WALKS = (int64_t)LBK * 512;
// nodes whose tiles are in flight together (see list_items for the 512)
__host__ __device__ inline int64_t bv_flight(unsigned grid) {
  return grid < 512 ? (int64_t)LBK * grid : (int64_t)LBK * LCT * 512;
}
// jumps along the links inside [c0, c0 + len); a thread has the nodes
// threadIdx.x + k * LBK of it. Stores the links that have moved.
__device__ inline void tile_links(uint32_t c0, uint32_t len, const bool (&live)[LCT], uint32_t (&link)[LCT],
                                  uint32_t *s_link, uint32_t *bpar) {
#pragma unroll
  for (int k = 0; k < LCT; k++)
    if (threadIdx.x + k * LBK < len) s_link[threadIdx.x + k * LBK] = link[k];
  uint32_t changed = 0;
  bool moved = true;
  for (int round = 0; __syncthreads_or(moved) && round < 32; round++) {  // 12 rounds end any path of a tile
    moved = false;
#pragma unroll
    for (int k = 0; k < LCT; k++) {
      if (!live[k] || link[k] - c0 >= len) continue;
      const uint32_t up = s_link[link[k] - c0];
      if (up == link[k]) continue;
      s_link[threadIdx.x + k * LBK] = link[k] = up;
      changed |= 1u << k;
      moved = true;
    }
  }
#pragma unroll
  for (int k = 0; k < LCT; k++)
    if (changed >> k & 1u) link_st(&bpar[c0 + threadIdx.x + k * LBK], link[k]);
}
// (merged nodes of a marked range keep their parents; a node without an edge points to itself)
__global__ __launch_bounds__(LBK) void k_bv_links(const uint64_t *bv, uint32_t *bpar, const uint32_t *rootc) {
  const int64_t lo = (int64_t)bv[BV_LO], nc = (int64_t)bv[BV_HI] - lo;
  if (bv[BV_ACT] != ACT_ROUND || nc <= bv_flight(gridDim.x)) return;
  __shared__ uint32_t s_link[LBK * LCT];
  const bool marked = bv[BV_MARK] != 0;
  const int ct = list_items(nc);
  for (int64_t tile = blockIdx.x; tile * (LBK * ct) < nc; tile += gridDim.x) {
    bool live[LCT];
    uint32_t link[LCT];
    const int64_t t0 = tile * (LBK * ct), end = tile_end(nc, tile, LBK * ct);
#pragma unroll
    for (int k = 0; k < LCT; k++) {
      const int64_t i = t0 + threadIdx.x + (int64_t)k * LBK;
      const uint32_t c = (uint32_t)(lo + i);
      live[k] = i < end && !(marked && rootc[i] != c);
      link[k] = live[k] ? link_ld(&bpar[c]) : c;
    }
    tile_links((uint32_t)(lo + t0), (uint32_t)(end - t0), live, link, s_link, bpar);
    __syncthreads();  // (the links' LDS is used again)
  }
}
// (SMALL: at most BV_WALKS nodes in any round)
template <bool SMALL>
__global__ __launch_bounds__(LBK) void k_bv_compress(uint64_t *bv, const uint64_t *best, uint32_t *bpar,
                                                     uint32_t *rootc, uint64_t *hdr) {
  const uint64_t act = bv[BV_ACT];
  if (act == ACT_HEAVY) {  // the heavy edges' way up, which also marks the next round's range
    const int64_t lo = (int64_t)bv[BV_SLO], hi = (int64_t)bv[BV_NB];
    for (int64_t c = lo + (int64_t)blockIdx.x * LBK + threadIdx.x; c < hi; c += (int64_t)gridDim.x * LBK) {
      uint32_t x = (uint32_t)c;  // as many steps as light rounds at most
      for (uint32_t p = bpar[x]; p != x; p = bpar[x]) x = p;
      rootc[c - lo] = x;
    }
    return;
  }
  if (act != ACT_ROUND) return;
  const int64_t lo = (int64_t)bv[BV_LO], nc = (int64_t)bv[BV_HI] - lo;
  const bool marked = bv[BV_MARK] != 0, jump = !SMALL && nc > BV_WALKS && nc <= bv_flight(gridDim.x);
  const int ct = list_items(nc);
  __shared__ uint32_t s_link[SMALL ? 1 : LBK * LCT];
  for (int64_t tile = blockIdx.x; tile * (LBK * ct) < nc; tile += gridDim.x) {
    bool keep[LCT], live[LCT];
    uint32_t pos[LCT], link[LCT];
    const int64_t t0 = tile * (LBK * ct), end = tile_end(nc, tile, LBK * ct);
    auto root = [&](int k, int64_t i) {
      keep[k] = live[k] && link[k] == (uint32_t)(lo + i);
      if (!keep[k]) rootc[i] = live[k] ? bv_root(bpar, link[k], hdr) : NONE32;
    };
#pragma unroll
    for (int k = 0; k < LCT; k++) {
      const int64_t i = t0 + threadIdx.x + (int64_t)k * LBK;
      const uint32_t c = (uint32_t)(lo + i);
      keep[k] = live[k] = false;
      link[k] = c;
      if (i >= end) continue;
      live[k] = !(marked && rootc[i] != c) && best[c] != NONE64;  // (marked: some were merged before)
      if (live[k]) link[k] = link_ld(&bpar[c]);
      if (SMALL) root(k, i);
    }
    if (jump) tile_links((uint32_t)(lo + t0), (uint32_t)(end - t0), live, link, s_link, bpar);
#pragma unroll
    for (int k = 0; k < LCT; k++) {
      const int64_t i = t0 + threadIdx.x + (int64_t)k * LBK;
      if (!SMALL && i < end) root(k, i);
    }
    list_positions(keep, pos, (unsigned long long *)&bv[BV_NB]);
#pragma unroll
    for (int k = 0; k < LCT; k++)
      if (keep[k]) rootc[t0 + threadIdx.x + (int64_t)k * LBK] = pos[k];
  }
}

// node c -> the new node of its component; new nodes start without a minimum
__device__ inline void bv_link(uint32_t c, uint32_t rc, int64_t lo, const uint32_t *rootc, uint32_t *bpar) {
  if (rc == NONE32) return;
  bpar[c] = bpar[c] == c ? rc : rootc[rc - lo];
}
__global__ __launch_bounds__(B) void k_bv_link(const uint64_t *bv, const uint32_t *rootc, uint32_t *bpar,
                                               uint64_t *best) {
  if (bv[BV_ACT] != ACT_ROUND) return;
  const int64_t lo = (int64_t)bv[BV_LO], hi = (int64_t)bv[BV_HI], nb = (int64_t)bv[BV_NB];
  const int64_t step = (int64_t)gridDim.x * B, i0 = (int64_t)blockIdx.x * B + threadIdx.x;
  for (int64_t c = lo + i0; c < hi; c += step) bv_link((uint32_t)c, rootc[c - lo], lo, rootc, bpar);
  for (int64_t x = hi + i0; x < nb; x += step) {
    best[x] = NONE64;
    bpar[x] = (uint32_t)x;
  }
}

// first contraction: skeleton slots between different components, endpoints
// renamed to nodes; with a pivot, split as below
__global__ __launch_bounds__(LBK) void k_contract_first(int64_t n, const uint64_t *skel_key, const uint32_t *skel_tail,
                                                        const uint32_t *bpar, EdgeLists L, uint64_t *bv) {
  const int64_t n2 = 2 * n;
  const int ct = list_items(n2);
  const bool split = bv[BV_FIRST] != 0;
  const uint64_t pivot = split ? bv[BV_PIVOT] : NONE64;
  for (int64_t tile = blockIdx.x; tile * (LBK * ct) < n2; tile += gridDim.x) {
    bool keep[LCT], heavy[LCT];
    uint32_t pos[LCT], hpos[LCT], nu[LCT], nv[LCT];
    uint64_t kk[LCT];
    const int64_t base = tile * (LBK * ct) + threadIdx.x, end = tile_end(n2, tile, LBK * ct);
#pragma unroll
    for (int k = 0; k < LCT; k++) {
      const int64_t e = base + (int64_t)k * LBK;
      keep[k] = heavy[k] = false;
      kk[k] = e < end ? skel_key[e] : NONE64;
      nu[k] = nv[k] = 0;
      if (kk[k] == NONE64) continue;
      nu[k] = bpar[skel_tail[e]];
      nv[k] = bpar[e >> 1];
      keep[k] = nu[k] != nv[k] && kk[k] < pivot;
      heavy[k] = nu[k] != nv[k] && kk[k] >= pivot;
    }
    list_positions(keep, pos, (unsigned long long *)&bv[BV_CNT1]);
    if (split) list_positions(heavy, hpos, (unsigned long long *)&bv[BV_CNT2]);
#pragma unroll
    for (int k = 0; k < LCT; k++) {
      if (!keep[k] && !heavy[k]) continue;
      const int64_t p = keep[k] ? (int64_t)pos[k] : L.cap - 1 - (int64_t)hpos[k];
      L.key[0][p] = kk[k];
      L.u[0][p] = nu[k];
      L.v[0][p] = nv[k];
      L.s[0][p] = (uint32_t)(base + (int64_t)k * LBK);
    }
  }
}

// A round's contraction: edges between different components go to the front
// of the output buffer, renamed. The heavy edges of a split, parked since,
// go to the tops of their nodes. A split: the live edges with key below
// the pivot go to the front of the output buffer, the others to its back,
// counted down from cap (light and heavy together are E <= cap entries, so
// later contractions of the light part, which only shrink it, never reach the
// heavy part). The first contraction may split its list on the way.
__global__ __launch_bounds__(LBK) void k_contract(EdgeLists L, uint64_t *bv, const uint32_t *bpar,
                                                  const uint32_t *rootc) {
  const uint64_t act = bv[BV_ACT];
  if (act == ACT_NONE) return;
  const bool heavy = act == ACT_HEAVY;
  const int in = heavy ? (int)bv[BV_HB] : (int)bv[BV_IN], ob = heavy ? 1 - in : out_buffer(bv);
  const int64_t E = heavy ? (int64_t)bv[BV_EH] : (int64_t)bv[BV_E];
  const int64_t off = heavy ? L.cap - E : (int64_t)bv[BV_OFF];
  const uint64_t *key = L.key[in] + off;
  const uint32_t *eu = L.u[in] + off, *ev = L.v[in] + off;
  const uint32_t *es = L.s[in] ? L.s[in] + off : nullptr;
  unsigned long long *cnt = (unsigned long long *)&bv[BV_CNT1], *cnt2 = (unsigned long long *)&bv[BV_CNT2];
  const uint32_t *up = heavy ? rootc : bpar;  // node - ulo -> its component now
  const uint32_t ulo = heavy ? (uint32_t)bv[BV_SLO] : 0u;
  const int ct = list_items(E);
  if (act == ACT_SPLIT) {
    const uint64_t pivot = bv[BV_PIVOT];
    for (int64_t tile = blockIdx.x; tile * (LBK * ct) < E; tile += gridDim.x) {
      bool lt[LCT], ge[LCT];
      uint32_t pl[LCT], ph[LCT];
      uint64_t kk[LCT];
      const int64_t base = tile * (LBK * ct) + threadIdx.x, end = tile_end(E, tile, LBK * ct);
#pragma unroll
      for (int k = 0; k < LCT; k++) {
        const int64_t i = base + (int64_t)k * LBK;
        kk[k] = i < end ? key[i] : 0;
        lt[k] = i < end && kk[k] < pivot;
        ge[k] = i < end && kk[k] >= pivot;
      }
      list_positions(lt, pl, cnt);
      list_positions(ge, ph, cnt2);
#pragma unroll
      for (int k = 0; k < LCT; k++) {
        if (!lt[k] && !ge[k]) continue;
        const int64_t i = base + (int64_t)k * LBK;
        const int64_t p = lt[k] ? (int64_t)pl[k] : L.cap - 1 - (int64_t)ph[k];
        L.key[ob][p] = kk[k];
        L.u[ob][p] = eu[i];
        L.v[ob][p] = ev[i];
        L.s[ob][p] = es ? es[i] : (uint32_t)i;
      }
    }
    return;
  }
  const bool split = bv[BV_FIRST] != 0;
  const uint64_t pivot = split ? bv[BV_PIVOT] : NONE64;
  for (int64_t tile = blockIdx.x; tile * (LBK * ct) < E; tile += gridDim.x) {
    bool keep[LCT], hv[LCT];
    uint32_t pos[LCT], hpos[LCT], nu[LCT], nv[LCT];
    const int64_t base = tile * (LBK * ct) + threadIdx.x, end = tile_end(E, tile, LBK * ct);
#pragma unroll
    for (int k = 0; k < LCT; k++) {
      const int64_t i = base + (int64_t)k * LBK;
      keep[k] = hv[k] = false;
      nu[k] = nv[k] = 0;
      if (i >= end) continue;
      const uint32_t fu = up[eu[i] - ulo], fv = up[ev[i] - ulo];
      keep[k] = fu != fv;
      if (split && keep[k] && key[i] >= pivot) {
        hv[k] = true;
        keep[k] = false;
      }
      nu[k] = fu;
      nv[k] = fv;
    }
    list_positions(keep, pos, cnt);
    if (split) list_positions(hv, hpos, cnt2);
#pragma unroll
    for (int k = 0; k < LCT; k++) {
      if (!keep[k] && !hv[k]) continue;
      const int64_t i = base + (int64_t)k * LBK;
      const int64_t p = keep[k] ? (int64_t)pos[k] : L.cap - 1 - (int64_t)hpos[k];
      L.key[ob][p] = key[i];
      L.u[ob][p] = nu[k];
      L.v[ob][p] = nv[k];
      L.s[ob][p] = es ? es[i] : (uint32_t)i;
    }
  }
}

// Advances the state past the slot before this one and decides what this one
// does; one workgroup, so no other writes the words it reads.
//
// Filter split (Filter-Kruskal applied to Boruvka): a slot splits the list
// when live edges are at least `split_min` and more than twice the
// components; the pivot is the key of rank ~C*S/E among S evenly spaced
// samples of the list (sorted in LDS), so about one light edge per component.
// After a split, another where a plain round still left more than three
// quarters of the edges (parallel edges between few components), if enough
// slots are left for it: 4e6 hypergraph records 8.8 -> 8.4 ms, 1024 graphs 77.6
// -> 76; below split_min, or without the round in between, it lost at 1e6
// records (2.45 -> 2.52 ms) or 5e7 (49.0 -> 49.6).
constexpr int MAX_SPLITS = 3;
//
// Before the first contraction, k_bv_first decides the same from samples of
// the skeleton's slots alone (how many are live, and their keys), so that the
// contraction itself splits: a 5e7-record call 50.5 -> 49.0 ms, 4e6 hypergraph
// records 9.0 -> 8.7.
template <int S>
__device__ inline void sort_keys(uint64_t (&sk)[S], int i) {  // bitonic, ascending; S threads
  for (int k = 2; k <= S; k <<= 1) {
    for (int j = k >> 1; j > 0; j >>= 1) {
      const int p = i ^ j;
      if (p > i) {
        const uint64_t a = sk[i], b2 = sk[p];
        const bool up = (i & k) == 0;
        if ((a > b2) == up) { sk[i] = b2; sk[p] = a; }
      }
      __syncthreads();
    }
  }
}
constexpr int FIRST_SAMPLES = 1024;
__global__ __launch_bounds__(FIRST_SAMPLES) void k_bv_first(EdgeLists L, bool flat, int64_t slots, const uint32_t *bpar,
                                                            uint64_t *bv, int64_t split_min) {
  __shared__ uint64_t sk[FIRST_SAMPLES];
  const int64_t rows = flat ? (int64_t)bv[BV_E] : slots;
  if (rows <= 0) return;
  const int i = threadIdx.x;
  const int64_t e = (int64_t)((unsigned __int128)i * (uint64_t)rows / FIRST_SAMPLES);
  uint64_t k = L.key[2][e];
  if (k != NONE64 && bpar[L.u[2][e]] == bpar[flat ? L.v[2][e] : (uint32_t)(e >> 1)]) k = NONE64;
  sk[i] = k;
  const int live = __syncthreads_count(k != NONE64);
  sort_keys(sk, i);
  if (i != 0) return;
  const uint64_t C = bv[BV_NB] - bv[BV_HI];  // the nodes that the round made
  const uint64_t E = (uint64_t)((unsigned __int128)live * (uint64_t)rows / FIRST_SAMPLES);
  if ((int64_t)E < split_min || E <= 2 * C) return;
  bv[BV_PIVOT] = sk[(int64_t)((unsigned __int128)FIRST_SAMPLES * C / (uint64_t)rows)];  // below live / 2
  bv[BV_FIRST] = 1;
}
// whether the list that the last slot leaves is thinned (see k_bv_thin)
constexpr int64_t THIN_MIN = 16384;
__device__ inline bool bv_thins(const uint64_t *bv, int64_t n) {
  const uint64_t C = bv[BV_HI] - bv[BV_LO];
  return bv[BV_ACT] == ACT_ROUND && (int64_t)bv[BV_E] >= THIN_MIN && C * C <= (uint64_t)n / 2;
}
constexpr int SPLIT_SAMPLES = 256;
__global__ __launch_bounds__(SPLIT_SAMPLES) void k_bv_ctl(EdgeLists L, uint64_t *bv, int64_t split_min,
                                                          int left, int64_t n, uint64_t *pairs) {
  __shared__ uint64_t sk[SPLIT_SAMPLES];
  __shared__ int s_split;
  if (threadIdx.x == 0) {
    const uint64_t act = bv[BV_ACT], c1 = bv[BV_CNT1], c2 = bv[BV_CNT2], ob = (uint64_t)out_buffer(bv);
    uint64_t E = bv[BV_E], lo = bv[BV_LO], hi = bv[BV_HI], light = bv[BV_LIGHT];
    const uint64_t before = E;
    if (act == ACT_ROUND) {
      E = c1;
      bv[BV_IN] = ob;
      bv[BV_OFF] = 0;
      bv[BV_MARK] = 0;
      lo = hi;
      hi = bv[BV_NB];
      bv_level(bv, hi);
    }
    const bool first = bv[BV_FIRST] != 0;
    bv[BV_FIRST] = 0;
    if (act == ACT_SPLIT || first) {
      bv[BV_IN] = ob;
      bv[BV_SPLITDONE]++;
      if (c1 > 0) {  // light rounds first
        light = 1;
        E = c1;
        bv[BV_OFF] = 0;
        bv[BV_HB] = ob;
        bv[BV_EH] = c2;
        bv[BV_SLO] = lo;
      } else {  // no light edge: the heavy ones are the whole list
        E = c2;
        bv[BV_OFF] = (uint64_t)L.cap - c2;
      }
    } else if (act == ACT_HEAVY) {
      E = c1;
      bv[BV_IN] = 1 - bv[BV_HB];
      bv[BV_OFF] = 0;
      bv[BV_MARK] = 1;
      light = 0;
      lo = bv[BV_SLO];
      hi = bv[BV_NB];
    }
    uint64_t next = E > 0 ? ACT_ROUND : ACT_NONE;
    if (light && E == 0) next = ACT_HEAVY;  // light edges used up: the heavy ones are contracted next
    const uint64_t C = hi - lo;
    const bool again = bv[BV_SPLITDONE] > 0;
    const bool split = next == ACT_ROUND && !light && act == ACT_ROUND && (int64_t)E >= split_min && E > 2 * C &&
                       (!again || (bv[BV_SPLITDONE] < MAX_SPLITS && 4 * E > 3 * before &&
                                   left >= 2 * (64 - __clzll((long long)C)) + 4));
    bv[BV_ACT] = split ? (uint64_t)ACT_SPLIT : next;
    bv[BV_E] = E;
    bv[BV_LO] = lo;
    bv[BV_HI] = hi;
    bv[BV_LIGHT] = light;
    bv[BV_CNT1] = 0;
    bv[BV_CNT2] = 0;
    bv[H_M - H_BV] = 0;  // the forest's rows, counted after the last slot
    s_split = split;
  }
  __threadfence_block();
  __syncthreads();
  if (pairs && bv_thins(bv, n)) {
    const uint64_t C = bv[BV_HI] - bv[BV_LO];
    for (uint64_t p = threadIdx.x; p < C * C; p += SPLIT_SAMPLES) pairs[p] = NONE64;
  }
  if (!s_split) return;
  const Live lv = live_list(L, bv);
  const int i = threadIdx.x;
  sk[i] = lv.key[(int64_t)((unsigned __int128)i * (uint64_t)lv.E / SPLIT_SAMPLES)];
  __syncthreads();
  sort_keys(sk, i);
  if (i == 0) {
    const uint64_t C = bv[BV_HI] - bv[BV_LO];
    int64_t q = (int64_t)((unsigned __int128)SPLIT_SAMPLES * C / (uint64_t)lv.E);
    if (q > SPLIT_SAMPLES - 1) q = SPLIT_SAMPLES - 1;
    bv[BV_PIVOT] = sk[q];
  }
}

// Minima per index, of the keys that the threads of a workgroup offer: first in
// an LDS hash (late rounds send most edges to a few big components), then one
// atomicMin per index. For workgroups of LBK threads; call from all of them.
// min_flush ends a tile.
constexpr int MHS = 512;  // (1024, as many as the nodes of a small tile, cost 1e6-record calls 2 %)
struct MinHash {
  uint32_t k[MHS];
  unsigned long long v[MHS];
};
__device__ inline void min_clear(MinHash &h) {
  for (int i = threadIdx.x; i < MHS; i += LBK) { h.k[i] = NONE32; h.v[i] = NONE64; }
  __syncthreads();
}
__device__ inline void min_offer(MinHash &h, bool act, uint32_t c, unsigned long long kv, uint64_t *best) {
  unsigned long long kmin = kv;
  const bool upd = wave_combine_first(act, c, [&](bool mine, int leader) {
    const unsigned long long v = wave_min_u64(mine ? kv : NONE64);
    if ((int)wave_lane() == leader) kmin = v;
  });
  if (!upd) return;
  uint32_t sl = (c * 2654435761u) >> 23;  // 9 bits
  bool placed = false;
  for (int probe = 0; probe < HASH_PROBES && !placed; probe++) {
    uint32_t old = atomicCAS(&h.k[sl], NONE32, c);
    if (old == NONE32 || old == c) {
      if (kmin < h.v[sl]) atomicMin(&h.v[sl], kmin);
      placed = true;
    } else {
      sl = (sl + 1) & (MHS - 1);
    }
  }
  if (!placed && kmin < best[c]) atomicMin((unsigned long long *)&best[c], kmin);
}
__device__ inline void min_flush(MinHash &h, uint64_t *best) {
  __syncthreads();
  for (int i = threadIdx.x; i < MHS; i += LBK) {
    const uint32_t c = h.k[i];
    if (c == NONE32) continue;
    const unsigned long long v = h.v[i];
    if (v < best[c]) atomicMin((unsigned long long *)&best[c], v);
  }
  __syncthreads();
}

// per node, the minimum key over its live edges, in tiles of up to LBK * LCT edges
__global__ __launch_bounds__(LBK) void k_bv_min(EdgeLists L, const uint64_t *bv, uint64_t *best) {
  if (bv[BV_ACT] != ACT_ROUND) return;
  const Live lv = live_list(L, bv);
  __shared__ MinHash h;
  const int ct = list_items(lv.E);
  for (int64_t tile = blockIdx.x; tile * (LBK * ct) < lv.E; tile += gridDim.x) {
    min_clear(h);
    const int64_t tbase = tile * (LBK * ct);
    for (int k = 0; k < ct; k++) {
      const int64_t i = tbase + (int64_t)k * LBK + threadIdx.x;
      const bool act = i < lv.E;
      const unsigned long long kv = act ? lv.key[i] : NONE64;
      const uint32_t cu = act ? lv.u[i] : 0u, cv = act ? lv.v[i] : 0u;
      min_offer(h, act, cu, kv, best);
      min_offer(h, act, cv, kv, best);
    }
    min_flush(h, best);
  }
}

// One workgroup takes about 0.5 us per 1024 edges and step, and rounds that
// only halve the components keep their parallel edges: 4e5 records of a nested
// path with random second vertices left it 3e5 edges between 200 nodes, and
// the call took 6.2 ms. So a long list is thinned first, on the grid, to the
// smallest edge of each pair of nodes: 1.9 ms. The slots before leave at most
// 2^(ceil(bits(n) / 2) - 2) nodes (each round halves those with edges), so a
// table of all pairs fits where rootc lies; it is cleared by the last k_bv_ctl.
__device__ inline uint64_t pair_at(uint32_t u, uint32_t v, const uint64_t *bv) {
  const uint64_t lo = bv[BV_LO], C = bv[BV_HI] - lo;
  return ((u < v ? u : v) - lo) * C + ((u < v ? v : u) - lo);
}
__global__ __launch_bounds__(LBK) void k_bv_pairs(EdgeLists L, const uint64_t *bv, int64_t n, uint64_t *pairs) {
  if (!bv_thins(bv, n)) return;
  const Live lv = live_list(L, bv);
  __shared__ MinHash h;
  const int ct = list_items(lv.E);
  for (int64_t tile = blockIdx.x; tile * (LBK * ct) < lv.E; tile += gridDim.x) {
    min_clear(h);
    for (int k = 0; k < ct; k++) {
      const int64_t i = tile * (LBK * ct) + (int64_t)k * LBK + threadIdx.x;
      const bool act = i < lv.E;
      min_offer(h, act, act ? (uint32_t)pair_at(lv.u[i], lv.v[i], bv) : 0u, act ? lv.key[i] : NONE64, pairs);
    }
    min_flush(h, pairs);
  }
}
__global__ __launch_bounds__(LBK) void k_bv_thin(EdgeLists L, uint64_t *bv, int64_t n, const uint64_t *pairs) {
  if (!bv_thins(bv, n)) return;
  const Live lv = live_list(L, bv);
  const int ob = out_buffer(bv), ct = list_items(lv.E);
  for (int64_t tile = blockIdx.x; tile * (LBK * ct) < lv.E; tile += gridDim.x) {
    bool keep[LCT];
    uint32_t pos[LCT];
    const int64_t base = tile * (LBK * ct) + threadIdx.x, end = tile_end(lv.E, tile, LBK * ct);
#pragma unroll
    for (int k = 0; k < LCT; k++) {
      const int64_t i = base + (int64_t)k * LBK;
      keep[k] = i < end && pairs[pair_at(lv.u[i], lv.v[i], bv)] == lv.key[i];
    }
    list_positions(keep, pos, (unsigned long long *)&bv[BV_CNT1]);
#pragma unroll
    for (int k = 0; k < LCT; k++) {
      if (!keep[k]) continue;
      const int64_t i = base + (int64_t)k * LBK;
      L.key[ob][pos[k]] = lv.key[i];
      L.u[ob][pos[k]] = lv.u[i];
      L.v[ob][pos[k]] = lv.v[i];
      L.s[ob][pos[k]] = lv.s ? lv.s[i] : (uint32_t)i;
    }
  }
}

// What the enqueued slots of a small call leave (it does not split), in one
// workgroup: rounds of the same five steps with barriers between them.
// Components at least halve per round, so the tree's levels (H_LEV holds 96)
// end any call; past them the call fails.
constexpr int BTB = 1024;
__global__ __launch_bounds__(BTB) void k_bv_tail(EdgeLists L, uint64_t *bv, int64_t n, bool thin, uint64_t *best,
                                                 uint32_t *bpar, uint32_t *rootc, uint8_t *msf_flag, uint64_t *hdr) {
  if (bv[BV_ACT] == ACT_NONE) return;
  __shared__ uint32_t s_nb, s_cnt;
  Live lv = live_list(L, bv);
  int ob = out_buffer(bv);
  int64_t lo = (int64_t)bv[BV_LO], hi = (int64_t)bv[BV_HI];
  if (thin && bv_thins(bv, n)) {
    lv = Live{L.key[ob], L.u[ob], L.v[ob], L.s[ob], (int64_t)bv[BV_CNT1]};
    ob = 1 - ob;
  }
  int level = (int)bv[H_BV_NLEV - H_BV];
  const int tid = threadIdx.x;
  __syncthreads();  // (bv is written below)
  while (lv.E > 0 && level < H_LPOS - H_LEV - 1) {
    if (tid == 0) {
      s_nb = (uint32_t)hi;
      s_cnt = 0;
    }
    for (int64_t i = tid; i < lv.E; i += BTB) {
      const unsigned long long k = lv.key[i];
      const uint32_t u = lv.u[i], v = lv.v[i];
      if (k < best[u]) atomicMin((unsigned long long *)&best[u], k);
      if (k < best[v]) atomicMin((unsigned long long *)&best[v], k);
    }
    __syncthreads();
    for (int64_t i = tid; i < lv.E; i += BTB)
      if (bv_hook_edge(lv.key[i], lv.u[i], lv.v[i], best, bpar)) msf_flag[lv.s ? lv.s[i] : i] = MSF_EDGE;
    __syncthreads();
    for (int64_t c = lo + tid; c < hi; c += BTB) {
      uint32_t r = NONE32;
      if (best[c] != NONE64) {
        r = bv_root(bpar, (uint32_t)c, hdr);
        if (r == (uint32_t)c) r = atomicAdd(&s_nb, 1u);
      }
      rootc[c - lo] = r;
    }
    __syncthreads();
    const int64_t nb = s_nb;
    for (int64_t c = lo + tid; c < hi; c += BTB) bv_link((uint32_t)c, rootc[c - lo], lo, rootc, bpar);
    for (int64_t x = hi + tid; x < nb; x += BTB) {
      best[x] = NONE64;
      bpar[x] = (uint32_t)x;
    }
    __syncthreads();
    for (int64_t i = tid; i < lv.E; i += BTB) {
      const uint32_t fu = bpar[lv.u[i]], fv = bpar[lv.v[i]];
      if (fu == fv) continue;
      const uint32_t p = atomicAdd(&s_cnt, 1u);
      L.key[ob][p] = lv.key[i];
      L.u[ob][p] = fu;
      L.v[ob][p] = fv;
      L.s[ob][p] = lv.s ? lv.s[i] : (uint32_t)i;
    }
    __syncthreads();
    if (tid == 0) bv_level(bv, (uint64_t)nb);
    level++;
    lv = Live{L.key[ob], L.u[ob], L.v[ob], L.s[ob], (int64_t)s_cnt};
    ob = 1 - ob;
    lo = hi;
    hi = nb;
    __syncthreads();
  }
  if (tid == 0 && lv.E == 0) {
    bv[BV_E] = 0;
    bv[BV_ACT] = ACT_NONE;
    bv[BV_NB] = (uint64_t)hi;
  }
}

// rows with weight < limit (rows are sorted, so they are a prefix): one binary
// search; the prefix becomes the forest (the row count shrinks in place)
__global__ void k_prefix_below(const uint64_t *key, Cnt mc, uint64_t *m, uint64_t limit) {
  if (threadIdx.x != 0 || blockIdx.x != 0) return;
  int64_t lo = 0, hi = mc.get();
  while (lo < hi) {
    const int64_t mid = lo + (hi - lo) / 2;
    if (key[mid] < limit) lo = mid + 1;
    else hi = mid;
  }
  *m = (uint64_t)lo;
}

// ---------------------------------------------------------------- weight ranks
// When w << wshift does not fit the key word, the key's weight field holds the
// weight's rank among the distinct weights of the skeleton instead: ranks
// order exactly as the weights do, so every step that only compares keys is
// unchanged, and the weights themselves are read back from the times once the
// forest is known. Absent slots get the value 2^tbits, above every weight.
__global__ __launch_bounds__(B) void k_rank_absent(const uint64_t *skel_key, int64_t cnt, int tbits, uint64_t *wraw) {
  for (int64_t i = (int64_t)blockIdx.x * B + threadIdx.x; i < cnt; i += (int64_t)gridDim.x * B)
    if (skel_key[i] == NONE64) wraw[i] = uint64_t(1) << tbits;
}
// first position of every distinct present weight in sorted order
__global__ __launch_bounds__(B) void k_rank_flags(const uint64_t *w, int64_t cnt, int tbits, uint32_t *first) {
  const uint64_t absent = uint64_t(1) << tbits;
  for (int64_t i = (int64_t)blockIdx.x * B + threadIdx.x; i < cnt; i += (int64_t)gridDim.x * B)
    first[i] = w[i] != absent && (i == 0 || w[i] != w[i - 1]) ? 1u : 0u;
}
// rank = distinct weights before this one; the finished key is offered to both
// records' first Boruvka minimum (records start as their own components)
__global__ __launch_bounds__(B) void k_rank_apply(const uint64_t *w, const uint32_t *slot, const uint32_t *first,
                                                  const uint32_t *before, int64_t cnt, int tbits, int wshift, bool flat,
                                                  uint64_t *skel_key, const uint32_t *skel_tail,
                                                  const uint32_t *skel_tid, uint64_t *best) {
  const uint64_t absent = uint64_t(1) << tbits;
  for (int64_t i = (int64_t)blockIdx.x * B + threadIdx.x; i < cnt; i += (int64_t)gridDim.x * B) {
    if (w[i] == absent) continue;
    const uint32_t e = slot[i];
    const uint64_t rank = (uint64_t)(before[i] + first[i] - 1u);
    const uint64_t k = skel_key[e] | (rank << wshift);
    skel_key[e] = k;
    const uint32_t head = flat ? skel_tid[e] : e >> 1;
    atomicMin((unsigned long long *)&best[skel_tail[e]], (unsigned long long)k);
    atomicMin((unsigned long long *)&best[head], (unsigned long long)k);
  }
}
}  // namespace

uint64_t *pinned_scratch() {
  static thread_local uint64_t *p = nullptr;
  if (!p) {
    if (hipHostMalloc((void **)&p, 4096, hipHostMallocDefault) != hipSuccess) p = nullptr;
  }
  return p;
}

// Reads `count` (<= 32) u64 words through the first 256 bytes of the pinned page.
ce_status read_u64(const uint64_t *dev, uint64_t *host_out, int count, hipStream_t s) {
  if (count > 32) {
    set_error("internal: read_u64 count");
    return CE_EDEVICE;
  }
  uint64_t *h = pinned_scratch();
  if (!h) {
    set_error("hipHostMalloc of the readback buffer failed");
    return CE_EDEVICE;
  }
  CE_HIP(hipMemcpyAsync(h, dev, sizeof(uint64_t) * count, hipMemcpyDeviceToHost, s));
  CE_HIP(hipStreamSynchronize(s));
  for (int i = 0; i < count; i++) host_out[i] = h[i];
  return CE_OK;
}

// Enqueues validation: error bits, min and max time into the control block.
ce_status stage_validate(const int32_t *src, const int32_t *dst, const int64_t *t, const OneGraph &og, Bufs &b,
                         hipStream_t s) {
  CE_LAUNCH(k_init_hdr, dim3(1), dim3(256), 0, s, b.hdr, og);
  CE_HIP(hipGetLastError());
  if (b.n > 0) {
    CE_LAUNCH(k_validate, dim3(grid_for(b.n, VB, 512)), dim3(VB), 0, s, src, dst, t, b.n, b.eoff, b.voff, b.G,
              b.hdr);
    CE_HIP(hipGetLastError());
  }
  return CE_OK;
}

// After the plan's key width is known: a wider time span is an error as well.
ce_status stage_check_span(Bufs &b, hipStream_t s) {
  CE_LAUNCH(k_check_span, dim3(1), dim3(64), 0, s, b.hdr, b.n, b.tbits);
  CE_HIP(hipGetLastError());
  return CE_OK;
}

// The validation words (error bits, min t, max t) on the host: one read back.
ce_status read_validation(Bufs &b, hipStream_t s, uint64_t *flags, int64_t *tmin, int64_t *tmax) {
  uint64_t h[3];
  CE_TRY(read_u64(b.hdr, h, 3, s));
  *flags = h[0];
  *tmin = (int64_t)(h[1] ^ (uint64_t(1) << 63));
  *tmax = (int64_t)(h[2] ^ (uint64_t(1) << 63));
  return CE_OK;
}

bool choose_key_layout(Bufs &b, int64_t rows) {
  // CE_WEIGHT_RANKS=1 (read on every call) ranks the weights even when they fit
  const char *e = getenv("CE_WEIGHT_RANKS");
  const bool force = e && atoi(e) == 1;
  if (!force && b.tbits + b.wshift <= 63) {
    b.rank = false;
    b.keybits = b.tbits + b.wshift;
    return true;
  }
  const int rb = bits_for((uint64_t)(rows > 1 ? rows - 1 : 1));
  if (rb + b.wshift > 63) return false;
  b.rank = true;
  b.keybits = rb + b.wshift;
  return true;
}

// Ranks the raw weights of the first cnt skeleton slots (wraw, overwritten)
// and completes their keys and the first Boruvka minima; the keys' other bits
// are in place. Scratch from ws.
ce_status stage_rank_weights(Bufs &b, uint64_t *wraw, int64_t cnt, Ws &ws, hipStream_t s) {
  if (cnt <= 0) return CE_OK;
  size_t m0 = ws.mark();
  uint32_t *slot = ws.alloc<uint32_t>(cnt), *slot_alt = ws.alloc<uint32_t>(cnt);
  uint64_t *w_alt = ws.alloc<uint64_t>(cnt);
  uint32_t *first = ws.alloc<uint32_t>(cnt + 1), *before = ws.alloc<uint32_t>(cnt + 1);
  CE_WS_CHECK(ws);
  const unsigned g = grid_cap(cnt, B);
  CE_LAUNCH(k_rank_absent, dim3(g), dim3(B), 0, s, b.skel_key, cnt, b.tbits, wraw);
  CE_HIP(hipGetLastError());
  bool alt = false;
  CE_TRY((radix_sort_pairs<uint64_t, uint32_t>(wraw, slot, w_alt, slot_alt, Cnt(cnt), 0, b.tbits + 1, true, &alt, ws,
                                               s)));
  const uint64_t *w = alt ? w_alt : wraw;
  const uint32_t *sl = alt ? slot_alt : slot;
  CE_LAUNCH(k_rank_flags, dim3(g), dim3(B), 0, s, w, cnt, b.tbits, first);
  CE_HIP(hipGetLastError());
  CE_TRY(scan_exclusive_u32(first, before, Cnt(cnt), ws, s));
  CE_LAUNCH(k_rank_apply, dim3(g), dim3(B), 0, s, w, sl, first, before, cnt, b.tbits, b.wshift, b.flat, b.skel_key,
            b.skel_tail, b.skel_tid, b.best);
  CE_HIP(hipGetLastError());
  ws.release(m0);
  return CE_OK;
}

size_t stage_rank_weights_scratch(int64_t cnt) {
  Ws w;
  w.alloc<uint32_t>(cnt);
  w.alloc<uint32_t>(cnt);
  w.alloc<uint64_t>(cnt);
  w.alloc<uint32_t>(cnt + 1);
  w.alloc<uint32_t>(cnt + 1);
  const size_t a = radix_ws_bytes(cnt), c = scan_ws_bytes(cnt + 1);
  return w.off + (a > c ? a : c) + 4096;
}

size_t stage_sort_skeleton_scratch(int64_t n) {
  Ws w;
  w.alloc<uint64_t>(2 * n);  // raw weights, when the weights are ranked
  const size_t r0 = w.off;
  for (int k = 0; k < 4; k++) w.alloc<uint32_t>(2 * n);  // ikey, ival and their ping-pong copies
  size_t base = w.off;
  w.alloc<uint64_t>(n);  // tkey alt
  w.alloc<uint4>(n);     // (id, src, dst)
  w.alloc<uint4>(n);     // ... ping-pong
  size_t a = w.off + radix_ws_bytes(n);
  size_t b2 = base + radix_ws_bytes(2 * n);
  size_t c = r0 + stage_rank_weights_scratch(2 * n);
  if (b2 > a) a = b2;
  return (a > c ? a : c) + 1024;
}

// Records by (t, id): stable radix sort on t - tmin carrying (id, global src,
// global dst). b.ts receives the sorted times; *vals points at the
// sorted payload inside ws (the caller releases it).
ce_status sort_records_by_time(const int32_t *src, const int32_t *dst, const int64_t *t, Bufs &b, Ws &ws,
                               hipStream_t s, const uint4 **vals) {
  const int64_t n = b.n;
  uint64_t *tkey_alt = ws.alloc<uint64_t>(n);
  uint4 *tval = ws.alloc<uint4>(n);
  uint4 *tval_alt = ws.alloc<uint4>(n);
  CE_WS_CHECK(ws);
  CE_LAUNCH(k_tkeys, dim3(grid_for(n, B)), dim3(B), 0, s, t, src, dst, n, b.eoff, b.voff, b.G, b.hdr, b.ts, tval);
  CE_HIP(hipGetLastError());
  bool alt = false;
  CE_TRY((radix_sort_pairs<uint64_t, uint4>(b.ts, tval, tkey_alt, tval_alt, n, 0, b.tbits, false, &alt, ws, s)));
  if (alt) CE_HIP(hipMemcpyAsync(b.ts, tkey_alt, sizeof(uint64_t) * n, hipMemcpyDeviceToDevice, s));
  *vals = alt ? tval_alt : tval;
  return CE_OK;
}

ce_status stage_sort_skeleton(const int32_t *src, const int32_t *dst, const int64_t *t, Bufs &b, Ws &ws,
                              hipStream_t s) {
  const int64_t n = b.n, n2 = 2 * n;
  size_t m0 = ws.mark();
  uint64_t *wraw = b.rank ? ws.alloc<uint64_t>(n2) : nullptr;  // raw weights until they are ranked
  size_t m1 = ws.mark();
  uint32_t *ikey = ws.alloc<uint32_t>(n2);
  uint32_t *ival = ws.alloc<uint32_t>(n2);
  uint32_t *ikey_alt = ws.alloc<uint32_t>(n2);
  uint32_t *ival_alt = ws.alloc<uint32_t>(n2);
  CE_WS_CHECK(ws);
  const bool packed = b.tbits <= 32;  // b.ts ends up as time << 32 | id by rank, else as the time alone
  // 1. records by (t, id)
  // 2. incidence entries (vertex, 2*rank+side) in rank order, perm by rank
  {
    size_t m2 = ws.mark();
    if (b.G == 1 && packed) {
      uint64_t *kalt = ws.alloc<uint64_t>(n), *v0 = ws.alloc<uint64_t>(n), *v1 = ws.alloc<uint64_t>(n);
      CE_WS_CHECK(ws);
      CE_LAUNCH(k_tkeys_packed, dim3(grid_for(n, B)), dim3(B), 0, s, t, src, dst, n, b.hdr, b.ts, v0);
      CE_HIP(hipGetLastError());
      bool alt = false;
      CE_TRY((radix_sort_pairs<uint64_t, uint64_t>(b.ts, v0, kalt, v1, n, 32, 32 + b.tbits, false, &alt, ws, s)));
      CE_LAUNCH(k_incidence_packed, dim3(grid_for(n, B)), dim3(B), 0, s, alt ? kalt : b.ts, alt ? v1 : v0, n, b.ts,
                b.perm, ikey);
    } else {
      const uint4 *vals = nullptr;
      CE_TRY(sort_records_by_time(src, dst, t, b, ws, s, &vals));
      CE_LAUNCH(k_incidence, dim3(grid_for(n, B)), dim3(B), 0, s, vals, n, packed, b.ts, b.perm, ikey);
    }
    CE_HIP(hipGetLastError());
    ws.release(m2);
  }
  // stable sort by vertex keeps every list in rank order
  bool alt = false;
  CE_TRY((radix_sort_pairs<uint32_t, uint32_t>(ikey, ival, ikey_alt, ival_alt, n2, 0, b.vbits, true, &alt, ws, s)));
  const uint32_t *sk = alt ? ikey_alt : ikey;
  const uint32_t *sv = alt ? ival_alt : ival;
  // 3. skeleton: neighbours in the same vertex list, then packed keys and first minima
  CE_LAUNCH(k_skel_links, dim3(grid_for(n2, B)), dim3(B), 0, s, sk, sv, n2, b.hdr, (uint2 *)b.skel_key);
  CE_HIP(hipGetLastError());
  if (packed)
    CE_LAUNCH(k_skel_keys<true>, dim3(grid_for(n, B)), dim3(B), 0, s, b.ts, b.perm, n, b.idbits, b.skel_key,
              (uint2 *)b.skel_tail, b.best, wraw);
  else
    CE_LAUNCH(k_skel_keys<false>, dim3(grid_for(n, B)), dim3(B), 0, s, b.ts, b.perm, n, b.idbits, b.skel_key,
              (uint2 *)b.skel_tail, b.best, wraw);
  CE_HIP(hipGetLastError());
  ws.release(m1);
  if (b.rank) CE_TRY(stage_rank_weights(b, wraw, n2, ws, s));
  ws.release(m0);
  return CE_OK;
}

size_t stage_boruvka_scratch(int64_t n, int64_t slots) {
  Ws w;
  w.alloc<uint32_t>(n);          // roots of a round's nodes
  for (int k = 0; k < 2; k++) {  // edge lists (key, u, v, slot), ping-pong
    w.alloc<uint64_t>(slots);
    w.alloc<uint32_t>(slots);
    w.alloc<uint32_t>(slots);
    w.alloc<uint32_t>(slots);
  }
  return w.off + 1024;
}

// Slots the host enqueues after the first round: in every round the
// components that still have live edges at least halve, so bits(n) + 1 rounds
// end a run of plain rounds. With one split (a further one is made only where
// its slots are left), plain rounds before it and the light rounds together
// halve the components at least once per round, and so do the light rounds and the plain rounds after them:
// 2 (bits(n) + 1) + 1 rounds cover both, and two more slots split and
// contract the heavy edges.
static int boruvka_rounds(int64_t n, bool split_possible) {
  const int r = bits_for((uint64_t)n) + 1;
  return split_possible ? 2 * r + 3 : r;
}

// Lists are split from 2^20 live edges on, if they are more than twice the
// components; a call's tuning (ce_tuning.split_min_edges, CE_SPLIT_MIN_EDGES)
// overrides the 2^20 or turns the split off. A call may split if it has at least
// twice as many skeleton slots as that (of a call's slots about half are live
// after the first round), unless it is an asynchronous one of up to 2^22 slots under
// the built-in choice: that would enqueue all the slots of the bound, idle or
// not (1.1e6 and 2e6 records: 2.39 and 2.90 ms, without a split 1.96 and 2.73).
//
// A call of up to 2^22 slots that does not split enqueues half a round per bit
// of n and leaves the rest, if any, to one workgroup: an idle slot costs six
// launches of about 2 us and its level of the dendrogram one more. The rest is
// little: few components are left after so many rounds, and from 2^18 slots on
// (an idle pair of launches more) a long list is thinned before. Calls that
// split enqueue the full bound, as light rounds may leave any number of heavy
// edges between any number of components; with fewer slots, 1e6 records of two
// nested paths left 4e5 edges to the one workgroup and took 14.0 ms, now 2.3.
// (Synchronous calls with and without a split: 5e5 to 8e5 records 1.62 and 1.49
// ms, 1e6 2.02 and 1.83 or, of sparser graphs, 1.72 and 1.83, 2e6 2.48 and 2.60.)
BvPlan boruvka_plan(int64_t n, int64_t slots, bool sync) {
  constexpr int64_t SMALL = int64_t(1) << 22;
  const int64_t split_min = tuning().split_min_edges;
  BvPlan p;
  p.split_possible = slots / 2 >= split_min && (sync || slots > SMALL || split_min < Tuning().split_min_edges);
  p.tail = !p.split_possible && slots <= SMALL;
  p.thin = p.tail && slots > (int64_t(1) << 18);
  p.slots = boruvka_rounds(n, p.split_possible);
  if (p.tail) {
    const int few = slots <= 8192 ? 0 : bits_for((uint64_t)n) / 2 + 1;
    if (few < p.slots) p.slots = few;
  }
  return p;
}

// A synchronous call of the full bound looks whether the forest is complete, after
// LOOK_FROM slots and every LOOK_EVERY from there: a look is a round trip of
// about 25 us, an idle slot with its level of the dendrogram 15 to 30, and a
// call uses 12 to 17 slots of a bound of 49 to 61. 8e6 causal records 10.35 ->
// 9.89 ms, 4e6 hypergraph records 8.29 -> 7.94, 5e7 records 49.0 -> 48.4.
constexpr int LOOK_FROM = 12, LOOK_EVERY = 4;

ce_status stage_boruvka(Bufs &b, Ws &ws, hipStream_t s) {
  const int64_t n = b.n, n2 = b.slots;
  size_t m0 = ws.mark();
  uint32_t *rootc = ws.alloc<uint32_t>(n);
  EdgeLists L;
  for (int k = 0; k < 2; k++) {
    L.key[k] = ws.alloc<uint64_t>(n2);
    L.u[k] = ws.alloc<uint32_t>(n2);
    L.v[k] = ws.alloc<uint32_t>(n2);
    L.s[k] = ws.alloc<uint32_t>(n2);
  }
  CE_WS_CHECK(ws);
  L.key[2] = b.skel_key;
  L.u[2] = b.skel_tail;
  L.v[2] = b.skel_tid;
  L.s[2] = nullptr;
  L.cap = n2;
  uint64_t *bv = b.hdr + H_BV, *best = b.best;
  uint32_t *bpar = b.bpar;
  const unsigned gN = grid_cap(n, B), gE = grid_cap(n2, B), lN = list_blocks(n), lE = list_blocks(n2);
  CE_LAUNCH(k_bv_start, dim3(grid_cap(n, B)), dim3(B), 0, s, n, n2, b.flat, &b.hdr[H_C7], b.msf_flag, bpar, bv);
  // first round (its minima were seeded while the skeleton was emitted). Causal and hypergraph skeleton rows can
  // share a head, so theirs runs on the edge-list form, with the skeleton rows in place as the list (slot = row).
  if (b.flat)
    CE_LAUNCH(k_bv_hook, dim3(gE), dim3(B), 0, s, L, bv, best, bpar, b.msf_flag);
  else
    CE_LAUNCH(k_bv_hook_first, dim3(gN), dim3(B), 0, s, n, best, (const ulonglong2 *)b.skel_key,
              (const uint2 *)b.skel_tail, bpar, (uchar2 *)b.msf_flag);
  // (a round halves its nodes; after a split, up to half of all may be left in any slot, among the light rounds' own)
  const int64_t flight = bv_flight(lN);
  if (n > flight) CE_LAUNCH(k_bv_links, dim3(lN), dim3(LBK), 0, s, bv, bpar, rootc);
  const auto k_bv_compress_ = n <= BV_WALKS ? k_bv_compress<true> : k_bv_compress<false>;
  CE_LAUNCH(k_bv_compress_, dim3(lN), dim3(LBK), 0, s, bv, best, bpar, rootc, b.hdr);
  CE_LAUNCH(k_bv_link, dim3(gN), dim3(B), 0, s, bv, rootc, bpar, best);
  const BvPlan plan = boruvka_plan(n, n2, b.sync);
  const int64_t split_min = plan.split_possible ? tuning().split_min_edges : INT64_MAX;
  if (plan.split_possible)
    CE_LAUNCH(k_bv_first, dim3(1), dim3(FIRST_SAMPLES), 0, s, L, b.flat, n2, bpar, bv, split_min);
  if (b.flat)
    CE_LAUNCH(k_contract, dim3(lE), dim3(LBK), 0, s, L, bv, bpar, rootc);
  else
    CE_LAUNCH(k_contract_first, dim3(lE), dim3(LBK), 0, s, n, b.skel_key, b.skel_tail, bpar, L, bv);
  CE_HIP(hipGetLastError());
  // Filter split. When live edges far outnumber components, most of them run
  // between components that later rounds merge anyway, and every round would
  // scan them again. So the list is split at a pivot key: Boruvka runs on the
  // light edges (key below the pivot) alone until none is left, then the heavy
  // ones are contracted once and rounds go on with the survivors. Keys are
  // unique, so the forest is the same: a light edge outside the light forest
  // is the largest on a cycle of light edges, and contracting the light forest
  // keeps every heavy edge's cycles. The heavy edges wait, with the nodes they
  // had at the split, at the back of the buffer the split wrote.
  for (int r = 0; r < plan.slots; r++) {
    CE_LAUNCH(k_bv_ctl, dim3(1), dim3(SPLIT_SAMPLES), 0, s, L, bv, split_min, plan.slots - r, n, (uint64_t *)nullptr);
    if (b.sync && !plan.tail && r >= LOOK_FROM && r % LOOK_EVERY == 0) {
      uint64_t st[H_BV_NLEV - H_BV + 1];
      CE_TRY(read_u64(bv, st, H_BV_NLEV - H_BV + 1, s));
      if (st[BV_ACT] == ACT_NONE) {
        b.levels = (int)st[H_BV_NLEV - H_BV];
        break;
      }
    }
    CE_LAUNCH(k_bv_min, dim3(lE), dim3(LBK), 0, s, L, bv, best);
    CE_LAUNCH(k_bv_hook, dim3(gE), dim3(B), 0, s, L, bv, best, bpar, b.msf_flag);
    if (n >> (plan.split_possible ? 1 : r < 62 ? r + 1 : 63) > flight)
      CE_LAUNCH(k_bv_links, dim3(lN), dim3(LBK), 0, s, bv, bpar, rootc);
    CE_LAUNCH(k_bv_compress_, dim3(lN), dim3(LBK), 0, s, bv, best, bpar, rootc, b.hdr);
    CE_LAUNCH(k_bv_link, dim3(gN), dim3(B), 0, s, bv, rootc, bpar, best);
    CE_LAUNCH(k_contract, dim3(lE), dim3(LBK), 0, s, L, bv, bpar, rootc);
    CE_HIP(hipGetLastError());
  }
  uint64_t *pairs = plan.thin ? (uint64_t *)rootc : nullptr;
  CE_LAUNCH(k_bv_ctl, dim3(1), dim3(SPLIT_SAMPLES), 0, s, L, bv, split_min, 0, n, pairs);
  if (plan.thin) {
    CE_LAUNCH(k_bv_pairs, dim3(lE), dim3(LBK), 0, s, L, bv, n, pairs);
    CE_LAUNCH(k_bv_thin, dim3(lE), dim3(LBK), 0, s, L, bv, n, pairs);
  }
  if (plan.tail)
    CE_LAUNCH(k_bv_tail, dim3(1), dim3(BTB), 0, s, L, bv, n, plan.thin, best, bpar, rootc, b.msf_flag, b.hdr);
  CE_HIP(hipGetLastError());
  ws.release(m0);
  return CE_OK;
}

// Time-filtered line graph (Sec. 5.1): only edges with w <= max_dt. The
// filtered skeleton has the filtered line graph's components at every
// threshold up to max_dt (Thm 3), and Kruskal takes edges in key order, so
// its forest is the prefix of the sorted MSF with w <= max_dt.
ce_status stage_time_filter(Bufs &b, int64_t max_dt, hipStream_t s) {
  if (max_dt < 0) return CE_OK;
  // the sorted rows' weights ascend
  CE_LAUNCH(k_prefix_below, dim3(1), dim3(64), 0, s, b.msf_key, Cnt(&b.hdr[H_M], b.n > 1 ? b.n - 1 : 0), &b.hdr[H_M],
            (uint64_t)max_dt + 1);
  CE_HIP(hipGetLastError());
  return CE_OK;
}

}  // namespace ce
