// Stages A6-A7: the sorted MSF and its exact single-linkage dendrogram (Alg. 1
// steps 2 and 3).
//
// The paper builds the dendrogram with a union-find pass over the sorted MST
// edges and calls that pass an expensive serial operation (Sec. 3). Here it is
// read off the Boruvka tree, in the way of PANDORA (Sao, Prokopenko,
// Lebrun-Grandie: parallel dendrogram construction by tree contraction), with
// the contraction that Boruvka has made already.
//
// The parent of row e in the dendrogram is the smallest row on the boundary of
// C_e, the component that e completes. Let S be a node of the Boruvka tree (a
// set of records joined by rows chosen inside it) and best(S) the smallest row
// leaving it. Row e lies inside the node S0 where its two ends meet. While
// best(S) < e, C_e reaches past S; so e belongs to the chain of the first S at
// or above S0 with e < best(S). All rows of one chain contain its smallest
// row, the one that two components of the round that made S chose mutually
// (every other row chosen in that round leads down to it over smaller rows,
// and a row from below S is larger than a row chosen in that round). Hence, in
// each chain in row order:
//   - a row's parent is the next row, the last row's parent is best(S);
//   - a row e joins the rows before it to the component x that chose e (a
//     child of S0 with best(x) = e): its children are the previous row and
//     the last row of x's chain, or x itself when x is a record. The first
//     row was chosen from both sides and has two such children.
//   - sizes are prefix sums along the chain of the sizes joined.
// A row with e > best(S) for every S below the top ends in the top's chain.
//
// Steps: find every row's chain and chooser (two climbs of a few steps, for
// most rows one, made before the rows are sorted by key), sort the rows by
// chain (stable, rows are in order), add up
// chain sizes level by level (a chooser's chain is of an earlier round), one
// prefix sum over all rows, and write every row's node. All of it is gathers
// over the rows and a handful of streaming passes: 12.7 ms at 5e7 rows, the
// parents included, where interval halving with a union-find took 35.0 ms
// (768 dependent steps of two 20 us launches, a reset, an LDS stage, and a
// scatter for the parents); 0.2 ms against 0.55 at 7e4 rows.
#include "ce_internal.h"

namespace ce {

namespace {

constexpr int B = 256;

__global__ __launch_bounds__(B) void k_dn_init(uint32_t *kpar, int64_t n, uint32_t *up, int64_t mb) {
  const int64_t N = n > mb ? n : mb;
  for (int64_t i = (int64_t)blockIdx.x * B + threadIdx.x; i < N; i += (int64_t)gridDim.x * B) {
    if (i < n) kpar[i] = NONE32;
    if (i < mb) up[i] = NONE32;
  }
}

// The forest's slots. Every live edge must be gone by now (the bound on the
// enqueued slots guarantees it); if not, the call fails instead of returning a
// partial forest.
__global__ __launch_bounds__(LBK) void k_msf_list(const uint8_t *flag, int64_t n2, uint32_t *out, uint64_t *hdr) {
  if (blockIdx.x == 0 && threadIdx.x == 0 && hdr[H_BV] != 0) atomicOr((unsigned long long *)&hdr[H_STATUS], 32ull);
  unsigned long long *cnt = (unsigned long long *)&hdr[H_M];
  const int ct = list_items(n2);
  for (int64_t tile = blockIdx.x; tile * (LBK * ct) < n2; tile += gridDim.x) {
    bool keep[LCT];
    uint32_t pos[LCT];
    const int64_t base = tile * (LBK * ct) + threadIdx.x, end = tile_end(n2, tile, LBK * ct);
#pragma unroll
    for (int k = 0; k < LCT; k++) {
      const int64_t e = base + (int64_t)k * LBK;
      keep[k] = e < end && flag[e];
    }
    list_positions(keep, pos, cnt);
#pragma unroll
    for (int k = 0; k < LCT; k++)
      if (keep[k]) out[pos[k]] = (uint32_t)(base + (int64_t)k * LBK);
  }
}

// Per forest edge, in slot order: its key, and in one 16-byte record its ends'
// input ids, its chain (with bit 31 when both sides chose it) and who chose
// it (a record by its input id); mate[S] = the second chooser of a chain's
// first row. The climbs go from the two ends to the node where they meet and
// on to the chain; an edge of the first round, three in four, says who chose
// it, and its ends meet at the parent of its head, which is the next in line.
// Bound by the reads that are not: the tails' ids and the chains' minima.
// 3.2 ms at 5e7 rows (made after the sort, the climbs took 9.5).
constexpr uint32_t MUTUAL = 0x80000000u;
__global__ __launch_bounds__(B) void k_dn_gather(const uint32_t *list, Cnt mc, const uint8_t *flag,
                                                 const uint64_t *skel_key, const uint32_t *skel_tail,
                                                 const uint32_t *skel_head, bool flat, const uint32_t *perm,
                                                 const uint64_t *best, const uint32_t *bpar, int64_t n, uint64_t *okey,
                                                 uint4 *rec, uint32_t *mate, uint64_t *hdr) {
  const int64_t m = mc.get();
  // a forest has at most n - 1 rows; more means the call failed (row counts are clamped wherever they are read)
  if (blockIdx.x == 0 && threadIdx.x == 0 && (int64_t)hdr[H_M] > n - 1)
    atomicOr((unsigned long long *)&hdr[H_STATUS], 64ull);
  for (int64_t i = (int64_t)blockIdx.x * B + threadIdx.x; i < m; i += (int64_t)gridDim.x * B) {
    const uint32_t e = list[i], f = flag[e];
    const uint64_t key = skel_key[e];
    uint32_t x = skel_tail[e], y = flat ? skel_head[e] : e >> 1, cx = x, cy = y;
    const uint32_t tid = perm[x], hid = perm[y];
    okey[i] = key;
    bool px, py;
    if (f & MSF_FIRST) {
      px = (f & MSF_TAIL) != 0;
      py = (f & MSF_HEAD) != 0;
      x = y = bpar[y];
      cx = tid;
      cy = hid;
    } else {
      // parents have larger ids than their children, so the smaller end climbs
      for (int steps = 0; x != y && steps < 512; steps++) {
        if (x < y) { cx = x; x = bpar[x]; }
        else { cy = y; y = bpar[y]; }
      }
      px = best[cx] == key;
      py = best[cy] == key;
      cx = cx < (uint64_t)n ? perm[cx] : cx;
      cy = cy < (uint64_t)n ? perm[cy] : cy;
    }
    if (x != y || x < (uint64_t)n || (!px && !py)) {  // (cannot happen: the forest is a spanning one) stay in bounds
      atomicOr((unsigned long long *)&hdr[H_STATUS], 32ull);
      rec[i] = make_uint4(tid, hid, 0u, tid);
      continue;
    }
    uint32_t S = x;
    for (int k = 0; k < 512 && key > best[S]; k++) S = bpar[S];
    if (px && py) mate[S - n] = cy;
    rec[i] = make_uint4(tid, hid, (uint32_t)(S - n) | (px && py ? MUTUAL : 0u), px ? cx : cy);
  }
}

__device__ inline void set_parent(uint32_t x, uint32_t j, int64_t n, uint32_t *kpar, uint32_t *up) {
  if (x < (uint64_t)n) kpar[x] = (uint32_t)(n + j);
  else up[x - n] = j;
}

// Per sorted row: its ends, chain and chooser from the record of its edge, its
// weight in place of its key (the keys have done their work: the order).
// up[S] = the row best(S) of an inner node, kpar = that of a record. Bound by
// one random 16-byte read and one random 4-byte write a row: 3.9 ms at 5e7.
__global__ __launch_bounds__(B) void k_dn_rows(const uint32_t *idx, const uint4 *rec, Cnt mc, const int64_t *t,
                                               int wshift, bool rank, int64_t n, const uint32_t *mate,
                                               uint64_t *msf_key, uint64_t *msf_val, uint32_t *chain, uint64_t *pick,
                                               uint32_t *kpar, uint32_t *up) {
  const int64_t m = mc.get();
  for (int64_t j = (int64_t)blockIdx.x * B + threadIdx.x; j < m; j += (int64_t)gridDim.x * B) {
    const uint4 r = rec[idx[j]];
    msf_val[j] = (uint64_t)r.x | ((uint64_t)r.y << 32);
    msf_key[j] = rank ? (uint64_t)(t[r.y] - t[r.x]) : msf_key[j] >> wshift;
    const uint32_t S = r.z & ~MUTUAL;
    chain[j] = S;
    pick[j] = (uint64_t)j | ((uint64_t)r.w << 32);
    set_parent(r.w, (uint32_t)j, n, kpar, up);
    if (r.z & MUTUAL)  // two records chose each other, or two inner nodes
      set_parent(r.w < (uint64_t)n ? r.x ^ r.y ^ r.w : mate[S], (uint32_t)j, n, kpar, up);
  }
}

// first position and last row of every chain; sums start empty. Block 0 also
// finds where each level's chains start (a level: the nodes of one round).
__global__ __launch_bounds__(B) void k_dn_chains(const uint32_t *sc, const uint64_t *sp, Cnt mc, int64_t n,
                                                 uint32_t *cstart, uint32_t *top, uint32_t *T, uint64_t *hdr) {
  const int64_t m = mc.get();
  for (int64_t p = (int64_t)blockIdx.x * B + threadIdx.x; p < m; p += (int64_t)gridDim.x * B) {
    const uint32_t S = sc[p];
    if (p == 0 || sc[p - 1] != S) {
      cstart[S] = (uint32_t)p;
      T[S] = 0;
    }
    if (p + 1 == m || sc[p + 1] != S) top[S] = (uint32_t)sp[p];
  }
  if (blockIdx.x == 0 && threadIdx.x <= (uint32_t)hdr[H_BV_NLEV]) {
    const uint32_t S = (uint32_t)(hdr[H_LEV + threadIdx.x] - (uint64_t)n);
    int64_t lo = 0, hi = m;
    while (lo < hi) {
      const int64_t mid = lo + (hi - lo) / 2;
      if (sc[mid] < S) lo = mid + 1;
      else hi = mid;
    }
    hdr[H_LPOS + threadIdx.x] = (uint64_t)lo;
  }
}

// records joined at a row by chooser z: one, or the whole chain of z
__device__ inline uint32_t dn_size(uint32_t z, int64_t n, const uint32_t *T) {
  return z < (uint64_t)n ? 1u : __hip_atomic_load(&T[z - n], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// One level: the records joined at each of its rows, summed per chain. Rows
// of a chain are neighbours, so a wave sums its stretch of up to 1024 rows in
// registers (segmented by chain, the open segment carried along) and adds once
// per chain: a chain of 2e7 rows makes 2e4 atomics.
__device__ inline void dn_level(const uint32_t *sc, const uint64_t *sp, const uint32_t *mate, int64_t n, int64_t a,
                                int64_t b, int64_t gw, int64_t W, uint32_t *side, uint32_t *T) {
  const int lane = (int)wave_lane();
  const int64_t span = b - a;
  int64_t it = (span + 64 * W - 1) / (64 * W);
  it = it < 1 ? 1 : (it > 16 ? 16 : it);
  for (int64_t w0 = gw; w0 * 64 * it < span; w0 += W) {
    uint32_t ckey = NONE32, carry = 0;
    for (int64_t k = 0; k < it; k++) {
      const int64_t p = a + (w0 * it + k) * 64 + lane;
      const bool act = p < b;
      const uint32_t S = act ? sc[p] : NONE32;
      uint32_t before = __shfl_up(S, 1, 64);
      if (lane == 0) before = act && p > 0 ? sc[p - 1] : NONE32;
      uint32_t v = 0;
      if (act) {
        v = dn_size((uint32_t)(sp[p] >> 32), n, T);
        if (before != S) v += dn_size(mate[S], n, T);
        side[p] = v;
      }
#pragma unroll
      for (int d = 1; d < 64; d <<= 1) {
        const uint32_t kk = __shfl_up(S, d, 64), vv = __shfl_up(v, d, 64);
        if (lane >= d && kk == S) v += vv;
      }
      const uint32_t S0 = __shfl(S, 0, 64);
      if (S0 == ckey) {
        if (S == ckey) v += carry;
      } else if (ckey != NONE32 && lane == 0) {
        atomicAdd(&T[ckey], carry);
      }
      const uint32_t after = __shfl_down(S, 1, 64);
      if (act && lane < 63 && after != S) atomicAdd(&T[S], v);
      ckey = __shfl(S, 63, 64);
      carry = __shfl(v, 63, 64);
    }
    if (ckey != NONE32 && lane == 0) atomicAdd(&T[ckey], carry);
  }
}

__global__ __launch_bounds__(B) void k_dn_level(const uint32_t *sc, const uint64_t *sp, const uint32_t *mate, int64_t n,
                                                int level, const uint64_t *hdr, uint32_t *side, uint32_t *T) {
  if ((uint64_t)level > hdr[H_BV_NLEV]) return;
  dn_level(sc, sp, mate, n, (int64_t)hdr[H_LPOS + level - 1], (int64_t)hdr[H_LPOS + level],
           (int64_t)blockIdx.x * (B / 64) + (threadIdx.x >> 6), (int64_t)gridDim.x * (B / 64), side, T);
}

// the levels after the enqueued ones of a small call, in one workgroup
constexpr int TB = 1024;
__global__ __launch_bounds__(TB) void k_dn_level_tail(const uint32_t *sc, const uint64_t *sp, const uint32_t *mate,
                                                      int64_t n, int from, const uint64_t *hdr, uint32_t *side,
                                                      uint32_t *T) {
  const int L = (int)hdr[H_BV_NLEV];
  for (int l = from; l <= L; l++) {
    dn_level(sc, sp, mate, n, (int64_t)hdr[H_LPOS + l - 1], (int64_t)hdr[H_LPOS + l], threadIdx.x >> 6, TB / 64, side,
             T);
    __syncthreads();  // (the sums are read and added to past the workgroup's caches)
  }
}

// one 16-byte node per row (a scattered write costs a transaction whatever its
// width): children, size, parent. P = exclusive prefix sums of side.
__global__ __launch_bounds__(B) void k_dn_emit(const uint32_t *sc, const uint64_t *sp, const uint32_t *P,
                                               const uint32_t *cstart, const uint32_t *top, const uint32_t *mate,
                                               const uint32_t *up, int64_t n, Cnt mc, uint4 *node) {
  const int64_t m = mc.get();
  for (int64_t p = (int64_t)blockIdx.x * B + threadIdx.x; p < m; p += (int64_t)gridDim.x * B) {
    const uint32_t S = sc[p];
    const uint64_t v = sp[p];
    const uint32_t x = (uint32_t)(v >> 32);
    const uint32_t c0 = cstart[S];
    uint32_t a, par;
    if ((uint32_t)p == c0) {
      const uint32_t y = mate[S];
      a = y < (uint64_t)n ? y : (uint32_t)(n + top[y - n]);
    } else {
      a = (uint32_t)(n + (uint32_t)sp[p - 1]);
    }
    if (p + 1 < m && sc[p + 1] == S) {
      par = (uint32_t)(n + (uint32_t)sp[p + 1]);
    } else {
      const uint32_t u = up[S];  // rows past a cutoff are not there
      par = (int64_t)u < m ? (uint32_t)(n + u) : NONE32;
    }
    node[(uint32_t)v] = make_uint4(a, x < (uint64_t)n ? x : (uint32_t)(n + top[x - n]), P[p + 1] - P[c0], par);
  }
}

__global__ __launch_bounds__(B) void k_dn_unpack(const uint4 *node, int64_t n, Cnt mc, uint32_t *kc_u, uint32_t *kc_v,
                                                 uint32_t *ksize, uint32_t *kpar) {
  const int64_t m = mc.get();
  for (int64_t j = (int64_t)blockIdx.x * B + threadIdx.x; j < m; j += (int64_t)gridDim.x * B) {
    const uint4 v = node[j];
    kc_u[j] = v.x;
    kc_v[j] = v.y;
    ksize[j] = v.z;
    kpar[n + j] = v.w;
  }
}

// with a cutoff: records whose row was cut off have no parent
__global__ __launch_bounds__(B) void k_dn_trim(uint32_t *kpar, int64_t n, Cnt mc) {
  const int64_t m = mc.get();
  for (int64_t r = (int64_t)blockIdx.x * B + threadIdx.x; r < n; r += (int64_t)gridDim.x * B)
    if ((int64_t)kpar[r] >= n + m) kpar[r] = NONE32;
}

// Buffers of the two steps below, at the same places in both; a forest has at
// most mb rows and mb inner nodes. Three lie where the skeleton arrays were
// (dead once the edges are gathered), the edges' records in the second half
// of kpar and the three arrays behind it (written last), the others in scratch.
struct Chains {
  uint32_t *up, *key, *key_alt;     // skeleton arrays
  uint32_t *mate, *idx, *idx_alt;   // idx and idx_alt are pick_alt's bytes
  uint64_t *pick, *pick_alt, *mkey_alt;  // mkey_alt is pick's
  uint4 *rec;
};
int64_t row_bound(int64_t n, int64_t slots) { return slots < n ? slots : n; }
ce_status carve(const Bufs &b, Ws &ws, Chains &c) {
  const int64_t mb = row_bound(b.n, b.slots);
  Ws x;
  x.base = (char *)b.skel_key;
  x.cap = (size_t)((char *)b.best - (char *)b.skel_key);
  c.up = x.alloc<uint32_t>(mb);
  c.key = x.alloc<uint32_t>(mb);
  c.key_alt = x.alloc<uint32_t>(mb);
  c.mate = ws.alloc<uint32_t>(mb);
  c.pick_alt = ws.alloc<uint64_t>(mb);
  c.idx = (uint32_t *)c.pick_alt;
  c.idx_alt = c.idx + mb;
  c.pick = c.mkey_alt = ws.alloc<uint64_t>(mb);
  // 16 bytes for each of at most n - 1 rows from the next 16-byte boundary: kpar's half and three arrays of n words
  c.rec = (uint4 *)(((uintptr_t)(b.kpar + b.n) + 15) & ~(uintptr_t)15);
  CE_WS_CHECK(x);
  CE_WS_CHECK(ws);
  return CE_OK;
}

}  // namespace

size_t stage_dendrogram_scratch(int64_t n, int64_t slots) {
  const int64_t mb = row_bound(n, slots);
  Ws w;
  w.alloc<uint32_t>(mb);
  w.alloc<uint64_t>(mb);
  w.alloc<uint64_t>(mb);
  const size_t sort = radix_ws_bytes(mb), scan = scan_ws_bytes(mb + 1);
  return w.off + (sort > scan ? sort : scan) + 1024;
}

// The forest's rows (m on the device, at most n - 1) sorted by key: weights in
// msf_key, ends in msf_val, and every row's chain.
ce_status stage_rows(Bufs &b, Ws &ws, hipStream_t s) {
  const int64_t n = b.n, n2 = b.slots, mb = row_bound(n, n2);
  size_t m0 = ws.mark();
  Chains c;
  CE_TRY(carve(b, ws, c));
  uint32_t *list = (uint32_t *)b.msf_val;  // written after the list is read
  CE_LAUNCH(k_msf_list, dim3(list_blocks(n2)), dim3(LBK), 0, s, b.msf_flag, n2, list, b.hdr);
  const Cnt m(&b.hdr[H_M], mb < n - 1 ? mb : n - 1);
  // gather into the key buffer from which an odd or even number of radix
  // passes ends in msf_key, so no copy follows the sort
  const int passes = b.keybits > 8 ? (b.keybits + 7) / 8 : 1;
  uint64_t *gk = (passes & 1) ? c.mkey_alt : b.msf_key, *ok = (passes & 1) ? b.msf_key : c.mkey_alt;
  const unsigned g = grid_cap(mb, B);
  CE_LAUNCH(k_dn_gather, dim3(g), dim3(B), 0, s, list, m, b.msf_flag, b.skel_key, b.skel_tail, b.skel_tid, b.flat,
            b.perm, b.best, b.bpar, n, gk, c.rec, c.mate, b.hdr);
  CE_HIP(hipGetLastError());
  bool alt = false;
  CE_TRY((radix_sort_pairs<uint64_t, uint32_t>(gk, c.idx, ok, c.idx_alt, m, 0, b.keybits, true, &alt, ws, s)));
  if ((alt ? ok : gk) != b.msf_key) {  // (not reached: the pass count is as computed)
    set_error("internal: sorted forest is not in place");
    return CE_EDEVICE;
  }
  CE_LAUNCH(k_dn_init, dim3(grid_cap(n, B)), dim3(B), 0, s, b.kpar, n, c.up, mb);
  CE_LAUNCH(k_dn_rows, dim3(g), dim3(B), 0, s, alt ? c.idx_alt : c.idx, c.rec, m, b.t, b.wshift, b.rank, n, c.mate,
            b.msf_key, b.msf_val, c.key, c.pick, b.kpar, c.up);
  CE_HIP(hipGetLastError());
  ws.release(m0);
  return CE_OK;
}

// The dendrogram of the rows that are left (a cutoff drops the largest).
ce_status stage_dendrogram(Bufs &b, bool cut, Ws &ws, hipStream_t s) {
  const int64_t n = b.n, mb = row_bound(n, b.slots);
  if (n <= 1) return CE_OK;
  const Cnt m(&b.hdr[H_M], mb < n - 1 ? mb : n - 1);
  size_t m0 = ws.mark();
  Chains c;
  CE_TRY(carve(b, ws, c));
  bool alt = false;
  CE_TRY((radix_sort_pairs<uint32_t, uint64_t>(c.key, c.pick, c.key_alt, c.pick_alt, m, 0,
                                               bits_for((uint64_t)(mb - 1)), false, &alt, ws, s)));
  const uint32_t *sc = alt ? c.key_alt : c.key;
  const uint64_t *sp = alt ? c.pick_alt : c.pick;
  uint32_t *cstart = alt ? c.key : c.key_alt;
  uint32_t *top = (uint32_t *)(alt ? c.pick : c.pick_alt), *T = top + mb;
  // the Boruvka tree is done with since the chains are known: its parents (2n words) hold the sizes joined, its
  // minima (2n words of 8 bytes) the nodes
  uint32_t *side = b.bpar;
  uint4 *node = (uint4 *)b.best;
  const unsigned g = grid_cap(mb, B);
  CE_LAUNCH(k_dn_chains, dim3(g), dim3(B), 0, s, sc, sp, m, n, cstart, top, T, b.hdr);
  CE_HIP(hipGetLastError());
  const BvPlan plan = boruvka_plan(n, b.slots, b.sync);
  const unsigned gl = grid_for(mb, B, 2048);
  const int levels = b.levels > 0 ? b.levels : plan.slots + 1;  // the first round and the enqueued ones
  for (int l = 1; l <= levels && !(plan.tail && plan.slots == 0); l++)
    CE_LAUNCH(k_dn_level, dim3(gl), dim3(B), 0, s, sc, sp, c.mate, n, l, b.hdr, side, T);
  if (plan.tail)
    CE_LAUNCH(k_dn_level_tail, dim3(1), dim3(TB), 0, s, sc, sp, c.mate, n, plan.slots == 0 ? 1 : levels + 1, b.hdr,
              side, T);
  CE_HIP(hipGetLastError());
  CE_TRY(scan_exclusive_u32(side, side, m, ws, s));
  CE_LAUNCH(k_dn_emit, dim3(g), dim3(B), 0, s, sc, sp, side, cstart, top, c.mate, c.up, n, m, node);
  if (b.G == 1) b.node = node;  // unpacked where the rows are written
  else CE_LAUNCH(k_dn_unpack, dim3(g), dim3(B), 0, s, node, n, m, b.kc_u, b.kc_v, b.ksize, b.kpar);
  if (cut) CE_LAUNCH(k_dn_trim, dim3(grid_cap(n, B)), dim3(B), 0, s, b.kpar, n, m);
  CE_HIP(hipGetLastError());
  ws.release(m0);
  return CE_OK;
}

}  // namespace ce
