// Device-wide primitives: exclusive scan and a stable LSD radix sort.
//
// The radix sort is a reduce-then-scan design tiled for 64-wide waves:
// each block owns a tile of 1024 to 4096 keys; the scatter pass ranks keys
// stably inside the tile with 8 ballots per 64-key chunk (lanes with equal
// digits form a peer mask), stages the tile in LDS in digit order, keys
// first and then values in the same space, and writes it out in runs of
// consecutive addresses. Up to 4096 pairs are sorted
// by one workgroup in one launch; up to 96 tiles a pass is two launches
// (counts, scatter), beyond three.
#include "ce_internal.h"

namespace ce {

namespace {

constexpr int SB = 256;          // scan block
constexpr int SIPT = 8;          // scan items per thread
constexpr int STILE = SB * SIPT; // 2048

__device__ inline uint32_t wave_incl_scan(uint32_t x, int lane) {
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    uint32_t y = __shfl_up(x, d, 64);
    if (lane >= d) x += y;
  }
  return x;
}

// exclusive scan of one value per thread across a 256-thread block
__device__ inline uint32_t block_excl_scan(uint32_t x, uint32_t *lds_w /*[4]*/, uint32_t *total) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  uint32_t inc = wave_incl_scan(x, lane);
  if (lane == 63) lds_w[w] = inc;
  __syncthreads();
  uint32_t before = 0, tot = 0;
#pragma unroll
  for (int i = 0; i < SB / 64; i++) {
    uint32_t v = lds_w[i];
    if (i < w) before += v;
    tot += v;
  }
  __syncthreads();
  if (total) *total = tot;
  return before + inc - x;
}

// SIPT consecutive elements from position base (a multiple of SIPT; the arrays
// start at 16-byte boundaries), zero past n
__device__ inline void scan_load(const uint32_t *in, int64_t base, int64_t n, uint32_t (&v)[SIPT]) {
  static_assert(SIPT == 8, "two 16-byte loads");
  if (base + SIPT <= n) {
    const uint4 a = *(const uint4 *)(in + base), b = *(const uint4 *)(in + base + 4);
    v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w;
    v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
  } else {
#pragma unroll
    for (int k = 0; k < SIPT; k++) v[k] = base + k < n ? in[base + k] : 0u;
  }
}
__device__ inline void scan_load(const uint8_t *in, int64_t base, int64_t n, uint32_t (&v)[SIPT]) {
  if (base + SIPT <= n) {
    const uint2 a = *(const uint2 *)(in + base);
#pragma unroll
    for (int k = 0; k < SIPT; k++) v[k] = ((k < 4 ? a.x : a.y) >> (8 * (k & 3))) & 255u;
  } else {
#pragma unroll
    for (int k = 0; k < SIPT; k++) v[k] = base + k < n ? in[base + k] : 0u;
  }
}

// Tiles of STILE elements; a block takes tiles blockIdx.x, + gridDim.x, ...
// up to the live count's tiles (the grid is capped, so a small or empty live
// count costs little).
template <class T>
__global__ __launch_bounds__(SB) void k_scan_reduce(const T *in, Cnt nc, uint32_t *sums) {
  __shared__ uint32_t lw[SB / 64];
  const int64_t n = nc.get();
  const int64_t tiles = (n + STILE - 1) / STILE;
  for (int64_t tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
    uint32_t v[SIPT], acc = 0;
    scan_load(in, tile * STILE + (int64_t)threadIdx.x * SIPT, n, v);
#pragma unroll
    for (int k = 0; k < SIPT; k++) acc += v[k];
    uint32_t tot;
    block_excl_scan(acc, lw, &tot);
    if (threadIdx.x == 0) sums[tile] = tot;
  }
}

// Up to SDIRECT tiles (scanned false) a block adds up the sums before its
// tile itself: at most SDIRECT / 256 reads a thread against one more launch.
constexpr int64_t SDIRECT = 2048;
template <class T>
__global__ __launch_bounds__(SB) void k_scan_apply(const T *in, uint32_t *out, Cnt nc, const uint32_t *sums,
                                                   bool scanned) {
  __shared__ uint32_t lw[SB / 64];
  const int64_t n = nc.get();
  const int64_t tiles = (n + STILE - 1) / STILE;
  for (int64_t tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
    const int64_t base = tile * STILE + (int64_t)threadIdx.x * SIPT;
    uint32_t v[SIPT], acc = 0, before;
    if (scanned) {
      before = sums[tile];
    } else {
      uint32_t part = 0;
      for (int64_t q = threadIdx.x; q < tile; q += SB) part += sums[q];
      block_excl_scan(part, lw, &before);
    }
    scan_load(in, base, n, v);
#pragma unroll
    for (int k = 0; k < SIPT; k++) acc += v[k];
    uint32_t run = block_excl_scan(acc, lw, nullptr) + before;
    uint32_t o[SIPT];
#pragma unroll
    for (int k = 0; k < SIPT; k++) {
      o[k] = run;
      run += v[k];
    }
    if (base + SIPT <= n) {
      *(uint4 *)(out + base) = make_uint4(o[0], o[1], o[2], o[3]);
      *(uint4 *)(out + base + 4) = make_uint4(o[4], o[5], o[6], o[7]);
    } else {
#pragma unroll
      for (int k = 0; k < SIPT; k++)
        if (base + k < n) out[base + k] = o[k];
    }
    if (base < n && base + SIPT >= n) out[n] = run;  // the thread of the last element
  }
  if (tiles == 0 && blockIdx.x == 0 && threadIdx.x == 0) out[0] = 0;
}

// single-block exclusive scan for up to STILE elements; out[n] = total
template <class T>
__global__ __launch_bounds__(SB) void k_scan_small(const T *in, uint32_t *out, Cnt nc) {
  __shared__ uint32_t lw[SB / 64];
  const int64_t n = nc.get();
  int64_t base = (int64_t)threadIdx.x * SIPT;
  uint32_t v[SIPT];
  uint32_t acc = 0;
  scan_load(in, base, n, v);
#pragma unroll
  for (int k = 0; k < SIPT; k++) acc += v[k];
  uint32_t tot;
  uint32_t run = block_excl_scan(acc, lw, &tot);
#pragma unroll
  for (int k = 0; k < SIPT; k++) {
    if (base + k < n) out[base + k] = run;
    run += v[k];
  }
  if (threadIdx.x == 0) out[n] = tot;
}

}  // namespace

size_t scan_ws_bytes(int64_t n) {
  size_t b = 0;
  while (n > STILE) {
    int64_t nb = (n + STILE - 1) / STILE;
    b += 2 * (((size_t)(nb + 1) * 4 + 255) & ~size_t(255));
    n = nb;
  }
  return b + 512;
}

template <class T>
ce_status scan_exclusive(const T *in, uint32_t *out, Cnt n, Ws &ws, hipStream_t s) {
  if (n.v <= STILE) {
    CE_LAUNCH(k_scan_small<T>, dim3(1), dim3(SB), 0, s, in, out, n);
    CE_HIP(hipGetLastError());
    return CE_OK;
  }
  // one sum per tile of the live count; the sums are scanned with the tile count as their count
  int64_t nb = (n.v + STILE - 1) / STILE;
  size_t m = ws.mark();
  uint32_t *sums = ws.alloc<uint32_t>(nb + 1);
  uint32_t *sums_sc = ws.alloc<uint32_t>(nb + 1);
  CE_WS_CHECK(ws);
  const bool direct = nb <= SDIRECT;
  const unsigned g = grid_for(nb, 1, 2048);
  CE_LAUNCH(k_scan_reduce<T>, dim3(g), dim3(SB), 0, s, in, n, sums);
  CE_HIP(hipGetLastError());
  if (!direct) CE_TRY(scan_exclusive<uint32_t>(sums, sums_sc, n.p ? Cnt(n.p, nb, n.sh + 11) : Cnt(nb), ws, s));
  CE_LAUNCH(k_scan_apply<T>, dim3(g), dim3(SB), 0, s, in, out, n, direct ? sums : sums_sc, !direct);
  CE_HIP(hipGetLastError());
  ws.release(m);
  return CE_OK;
}
template ce_status scan_exclusive<uint8_t>(const uint8_t *, uint32_t *, Cnt, Ws &, hipStream_t);
ce_status scan_exclusive_u32(const uint32_t *in, uint32_t *out, Cnt n, Ws &ws, hipStream_t s) {
  return scan_exclusive<uint32_t>(in, out, n, ws, s);
}

// ------------------------------------------------------------ segment bounds
namespace {

// off[g] = first position p with key[p] >= g, for g in [0, G]; each of the
// n+1 gaps between neighbouring keys writes the offsets that fall in it
__global__ __launch_bounds__(256) void k_seg_bounds(const uint32_t *key, Cnt nc, Cnt gc, uint32_t *off) {
  const int64_t n = nc.get(), G = gc.get();
  for (int64_t p = (int64_t)blockIdx.x * 256 + threadIdx.x; p <= n; p += (int64_t)gridDim.x * 256) {
    const int64_t lo = p == 0 ? 0 : (int64_t)key[p - 1] + 1;
    const int64_t hi = p == n ? G : (int64_t)key[p];
    for (int64_t g = lo; g <= hi; g++) off[g] = (uint32_t)p;
  }
}

}  // namespace

ce_status segment_bounds_u32(const uint32_t *sorted_keys, Cnt n, Cnt G, uint32_t *off, hipStream_t s) {
  CE_LAUNCH(k_seg_bounds, dim3(grid_cap(n.v + 1, 256)), dim3(256), 0, s, sorted_keys, n, G, off);
  CE_HIP(hipGetLastError());
  return CE_OK;
}

// ------------------------------------------------------------ radix sort
namespace {

constexpr int RB = 256;              // block, but for the widest tiles
// keys per thread (IPT): 4, 8 or 16 (a tuning choice); a tile is RB * IPT keys

// Digit counts per tile. Up to RS_FEW tiles, tile-major: a scatter workgroup
// adds up the rows before its own itself, 256 digits at a time. Beyond,
// digit-major, and k_rs_digits turns each digit's row into tile offsets.
constexpr int RS_FEW = 96;
constexpr int RS_ROWS = 32;  // rows of counts in flight
template <class K, int IPT, int RB>
__global__ __launch_bounds__(RB) void k_rs_hist(const K *keys, Cnt nc, int shift, uint32_t *hist,
                                                int nblocks) {
  constexpr int TILE = RB * IPT, RW = RB / 64;
  __shared__ uint32_t cnt[RW][256];
  const int64_t n = nc.get();  // tiles past a device count write zero counts
  const int w = threadIdx.x >> 6;
  for (int i = threadIdx.x; i < RW * 256; i += RB) (&cnt[0][0])[i] = 0;
  __syncthreads();
  const int64_t base = (int64_t)blockIdx.x * TILE;
  constexpr int VK = 16 / sizeof(K);  // keys per 16-byte load
  if (base + TILE <= n && ((uintptr_t)keys & 15) == 0) {
    struct alignas(16) Vec { K k[VK]; };
    const Vec *p = (const Vec *)(keys + base);
    Vec v[IPT / VK];
#pragma unroll
    for (int k = 0; k < IPT / VK; k++) v[k] = p[k * RB + threadIdx.x];
#pragma unroll
    for (int k = 0; k < IPT / VK; k++)
#pragma unroll
      for (int q = 0; q < VK; q++) atomicAdd(&cnt[w][(uint32_t)(v[k].k[q] >> shift) & 255u], 1u);
  } else {
#pragma unroll
    for (int k = 0; k < IPT; k++) {
      int64_t i = base + k * RB + threadIdx.x;
      if (i < n) atomicAdd(&cnt[w][(uint32_t)(keys[i] >> shift) & 255u], 1u);
    }
  }
  __syncthreads();
  for (int d = threadIdx.x; d < 256; d += RB) {
    uint32_t c = 0;
#pragma unroll
    for (int q = 0; q < RW; q++) c += cnt[q][d];
    hist[nblocks <= RS_FEW ? (int64_t)blockIdx.x * 256 + d : (int64_t)d * nblocks + blockIdx.x] = c;
  }
}

// one workgroup per digit: its counts become offsets inside the digit, their sum goes to total[digit]
constexpr int DB = 1024;
__global__ __launch_bounds__(DB) void k_rs_digits(uint32_t *hist, int nblocks, uint32_t *total) {
  __shared__ uint32_t lw[DB / 64];
  uint32_t *row = hist + (int64_t)blockIdx.x * nblocks;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  uint32_t run = 0;
  for (int64_t b0 = 0; b0 < nblocks; b0 += DB * 4) {
    uint32_t v[4], acc = 0;
    const int64_t i0 = b0 + threadIdx.x * 4;
#pragma unroll
    for (int k = 0; k < 4; k++) {
      v[k] = i0 + k < nblocks ? row[i0 + k] : 0u;
      acc += v[k];
    }
    const uint32_t inc = wave_incl_scan(acc, lane);
    if (lane == 63) lw[w] = inc;
    __syncthreads();
    uint32_t before = 0, tot = 0;
#pragma unroll
    for (int q = 0; q < DB / 64; q++) {
      if (q < w) before += lw[q];
      tot += lw[q];
    }
    __syncthreads();
    uint32_t at = run + before + inc - acc;
#pragma unroll
    for (int k = 0; k < 4; k++) {
      if (i0 + k < nblocks) row[i0 + k] = at;
      at += v[k];
    }
    run += tot;
  }
  if (threadIdx.x == 0) total[blockIdx.x] = run;
}

template <class V>
__device__ inline V iota_value(int64_t i) { return V(i); }
template <>
__device__ inline uint4 iota_value<uint4>(int64_t i) { return make_uint4((uint32_t)i, 0u, 0u, 0u); }

// exclusive scan over the 256 digits, one a thread of the first four waves; call from all threads
__device__ inline uint32_t digit_excl_scan(uint32_t x, uint32_t *lds_w /*[4]*/) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const uint32_t inc = wave_incl_scan(x, lane);
  if (lane == 63 && w < 4) lds_w[w] = inc;
  __syncthreads();
  uint32_t before = 0;
#pragma unroll
  for (int i = 0; i < 4; i++)
    if (i < w) before += lds_w[i];
  __syncthreads();
  return before + inc - x;
}

template <class K, class V, int IPT, int RB>
__global__ __launch_bounds__(RB) void k_rs_scatter(const K *kin, const V *vin, K *kout, V *vout, Cnt nc,
                                                   int shift, const uint32_t *hist, const uint32_t *total,
                                                   int nblocks, int iota) {
  constexpr int TILE = RB * IPT, RW = RB / 64, WT = TILE / RW;  // keys per tile, per wave (IPT chunks of 64)
  const int64_t n = nc.get();
  if ((int64_t)blockIdx.x * TILE >= n) return;
  __shared__ uint32_t wcnt[RW][256];
  __shared__ uint32_t dbase[256], gbase[256];
  __shared__ uint32_t lw[4];
  // keys, then values, pass through the same LDS on their way out
  __shared__ alignas(16) char stage[TILE * (sizeof(K) > sizeof(V) ? sizeof(K) : sizeof(V))];
  K *skey = (K *)stage;
  V *sval = (V *)stage;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  for (int i = tid; i < RW * 256; i += RB) (&wcnt[0][0])[i] = 0;
  // where this tile's keys of digit `tid` go: after all smaller digits and the same digit in earlier tiles
  uint32_t all = 0, mine = 0;
  if (tid < 256) {
    if (nblocks <= RS_FEW) {
      for (int q0 = 0; q0 < nblocks; q0 += RS_ROWS) {
        uint32_t c[RS_ROWS];
#pragma unroll
        for (int k = 0; k < RS_ROWS; k++) c[k] = q0 + k < nblocks ? hist[(q0 + k) * 256 + tid] : 0u;
#pragma unroll
        for (int k = 0; k < RS_ROWS; k++) {
          all += c[k];
          if (q0 + k < (int)blockIdx.x) mine += c[k];
        }
      }
    } else {
      all = total[tid];
      mine = hist[(int64_t)tid * nblocks + blockIdx.x];
    }
  }
  all = digit_excl_scan(all, lw);
  if (tid < 256) gbase[tid] = all + mine;
  __syncthreads();
  const int64_t tbase = (int64_t)blockIdx.x * TILE;
  const uint64_t below = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
  K key[IPT];
  V val[IPT];
  uint32_t off[IPT];
  uint32_t dig[IPT];
#pragma unroll
  for (int c = 0; c < IPT; c++) {
    const int64_t i = tbase + (int64_t)w * WT + c * 64 + lane;
    const bool valid = i < n;
    K k = valid ? kin[i] : K(0);
    V v = valid ? (iota ? iota_value<V>(i) : vin[i]) : V{};
    uint32_t d = (uint32_t)(k >> shift) & 255u;
    uint64_t peers = __ballot(valid);
#pragma unroll
    for (int b = 0; b < 8; b++) {
      const bool bit = (d >> b) & 1u;
      const uint64_t bb = __ballot(bit);
      peers &= bit ? bb : ~bb;
    }
    const int leader = valid ? (__ffsll((unsigned long long)peers) - 1) : lane;
    uint32_t old = 0;
    if (valid && lane == leader) old = atomicAdd(&wcnt[w][d], (uint32_t)__popcll(peers));
    old = __shfl(old, leader, 64);
    key[c] = k;
    val[c] = v;
    dig[c] = valid ? d : 256u;
    off[c] = old + (uint32_t)__popcll(peers & below);
  }
  __syncthreads();
  // per digit: exclusive prefix over waves, then exclusive scan over digits
  uint32_t tot = 0;
  if (tid < 256) {
    const int d = tid;
    uint32_t run = 0;
#pragma unroll
    for (int q = 0; q < RW; q++) {
      uint32_t t = wcnt[q][d];
      wcnt[q][d] = run;
      run += t;
    }
    tot = run;
  }
  __syncthreads();
  const uint32_t ex = digit_excl_scan(tot, lw);
  if (tid < 256) dbase[tid] = ex;
  __syncthreads();
#pragma unroll
  for (int c = 0; c < IPT; c++) {
    if (dig[c] < 256u) {
      off[c] += dbase[dig[c]] + wcnt[w][dig[c]];
      skey[off[c]] = key[c];
    }
  }
  __syncthreads();
  const int64_t rem = n - tbase;
  const int valid_n = rem < TILE ? (int)rem : TILE;
  uint32_t to[IPT];
#pragma unroll
  for (int c = 0; c < IPT; c++) {
    const int i = c * RB + tid;
    if (i < valid_n) {
      const K k = skey[i];
      const uint32_t d = (uint32_t)(k >> shift) & 255u;
      to[c] = gbase[d] + ((uint32_t)i - dbase[d]);
      kout[to[c]] = k;
    }
  }
  __syncthreads();
#pragma unroll
  for (int c = 0; c < IPT; c++)
    if (dig[c] < 256u) sval[off[c]] = val[c];
  __syncthreads();
#pragma unroll
  for (int c = 0; c < IPT; c++) {
    const int i = c * RB + tid;
    if (i < valid_n) vout[to[c]] = sval[i];
  }
}

// A sort of up to RS_SMALL pairs in one workgroup, all passes in LDS: a wave
// ranks 256 neighbouring keys, and the pairs move through LDS between passes.
// (SMI chunks of 64 keys a wave: one chunk spreads up to 1024 keys over all waves)
constexpr int RS_SMALL = 4096, SMB = 1024, SMW = SMB / 64;
template <class K, class V, int SMI>
__global__ __launch_bounds__(SMB) void k_rs_small(const K *kin, const V *vin, K *kout, V *vout, Cnt nc, int begin_bit,
                                                  int end_bit, int iota) {
  __shared__ uint32_t wcnt[SMW][256];
  __shared__ uint32_t dbase[256];
  __shared__ uint32_t lw[4];
  __shared__ K skey[SMB * SMI];
  __shared__ V sval[SMB * SMI];
  const int n = (int)nc.get();
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const uint64_t below = lanes_below((uint32_t)lane);
  K key[SMI];
  V val[SMI];
#pragma unroll
  for (int c = 0; c < SMI; c++) {
    const int i = w * (64 * SMI) + c * 64 + lane;
    key[c] = i < n ? kin[i] : K(0);
    val[c] = i < n ? (iota ? iota_value<V>(i) : vin[i]) : V{};
  }
  for (int shift = begin_bit; shift < end_bit; shift += 8) {
    for (int i = tid; i < SMW * 256; i += SMB) (&wcnt[0][0])[i] = 0;
    __syncthreads();
    uint32_t off[SMI], dig[SMI];
#pragma unroll
    for (int c = 0; c < SMI; c++) {
      const bool valid = w * (64 * SMI) + c * 64 + lane < n;
      const uint32_t d = (uint32_t)(key[c] >> shift) & 255u;
      uint64_t peers = __ballot(valid);
#pragma unroll
      for (int b = 0; b < 8; b++) {
        const bool bit = (d >> b) & 1u;
        const uint64_t bb = __ballot(bit);
        peers &= bit ? bb : ~bb;
      }
      const int leader = valid ? (__ffsll((unsigned long long)peers) - 1) : lane;
      uint32_t old = 0;
      if (valid && lane == leader) old = atomicAdd(&wcnt[w][d], (uint32_t)__popcll(peers));
      old = __shfl(old, leader, 64);
      dig[c] = valid ? d : 256u;
      off[c] = old + (uint32_t)__popcll(peers & below);
    }
    __syncthreads();
    uint32_t tot = 0, inc = 0;
    if (tid < 256) {  // per digit: offsets of the waves; then the digits' own
#pragma unroll
      for (int q = 0; q < SMW; q++) {
        const uint32_t t = wcnt[q][tid];
        wcnt[q][tid] = tot;
        tot += t;
      }
      inc = wave_incl_scan(tot, lane);
      if (lane == 63) lw[w] = inc;
    }
    __syncthreads();
    if (tid < 256) {
      uint32_t before = 0;
#pragma unroll
      for (int q = 0; q < 4; q++)
        if (q < w) before += lw[q];
      dbase[tid] = before + inc - tot;
    }
    __syncthreads();
#pragma unroll
    for (int c = 0; c < SMI; c++) {
      if (dig[c] < 256u) {
        const uint32_t p = dbase[dig[c]] + wcnt[w][dig[c]] + off[c];
        skey[p] = key[c];
        sval[p] = val[c];
      }
    }
    __syncthreads();
#pragma unroll
    for (int c = 0; c < SMI; c++) {
      const int i = w * (64 * SMI) + c * 64 + lane;
      if (i < n) {
        key[c] = skey[i];
        val[c] = sval[i];
      }
    }
  }
#pragma unroll
  for (int c = 0; c < SMI; c++) {
    const int i = w * (64 * SMI) + c * 64 + lane;
    if (i < n) {
      kout[i] = key[c];
      vout[i] = val[c];
    }
  }
}

// Up to 2^24 keys a sort may take 4 keys per thread (its histogram is sized
// for that); larger sorts take at least 8. A tile of 4096 keys stages up to
// 16 bytes of each in LDS: 64 KiB of the 160 KiB a gfx950 workgroup may use.
//
// Eight keys a thread (the default) means 2048-key tiles of 256 threads up to
// RS_WIDE keys and 4096-key tiles of 512 threads beyond: runs of 16 keys a
// digit instead of 8, and half the digit counts, whose columns are strided. At
// 5e7 records the sorts take 1.8 ms less so (2.5e8 incidences and more: 8.3 of
// 226), at 1e6 records 0.03 of 2.84, and lines at 6e6 or 1.2e7 keys lost 0.3 to
// 0.4 ms of 1e7-record calls. Tiles of 8192 keys leave one workgroup on a CU
// (53.1 ms against 50.3), 16 keys a thread at 256 threads too few waves (51.6).
constexpr int64_t RS_WIDE = int64_t(1) << 19;
int radix_ipt(int64_t n) {
  int ipt = tuning().radix_ipt;
  if (ipt != 4 && ipt != 8 && ipt != 16) ipt = 8;
  if (ipt == 4 && n > (int64_t(1) << 24)) ipt = 8;
  if (ipt == 8 && n <= (int64_t)RB * 4 * RS_FEW) ipt = 4;  // twice the workgroups where few tiles leave CUs idle
  return ipt;
}

template <class K, class V, int IPT, int RB>
ce_status radix_passes(K *k0, V *v0, K *k1, V *v1, Cnt n, int begin_bit, int end_bit, bool iota_values,
                       bool *result_in_alt, Ws &ws, hipStream_t s) {
  constexpr int TILE = RB * IPT;
  const int64_t nb64 = (n.v + TILE - 1) / TILE;
  if (nb64 > 0x7fffffff) return CE_EINVAL;
  const int nb = (int)nb64;
  size_t m = ws.mark();
  uint32_t *hist = ws.alloc<uint32_t>((size_t)nb * 256);
  uint32_t *total = ws.alloc<uint32_t>(256);
  CE_WS_CHECK(ws);
  K *ki = k0, *ko = k1;
  V *vi = v0, *vo = v1;
  bool alt = false;
  bool first = true;
  if (end_bit <= begin_bit) end_bit = begin_bit + 1;  // one stable pass still materialises identity values
  for (int shift = begin_bit; shift < end_bit; shift += 8) {
    CE_LAUNCH((k_rs_hist<K, IPT, RB>), dim3((unsigned)nb), dim3(RB), 0, s, ki, n, shift, hist, nb);
    CE_HIP(hipGetLastError());
    if (nb > RS_FEW) CE_LAUNCH(k_rs_digits, dim3(256), dim3(DB), 0, s, hist, nb, total);
    CE_LAUNCH((k_rs_scatter<K, V, IPT, RB>), dim3((unsigned)nb), dim3(RB), 0, s, ki, (const V *)vi, ko, vo, n,
                       shift, hist, total, nb, (first && iota_values) ? 1 : 0);
    CE_HIP(hipGetLastError());
    first = false;
    K *tk = ki; ki = ko; ko = tk;
    V *tv = vi; vi = vo; vo = tv;
    alt = !alt;
  }
  *result_in_alt = alt;
  ws.release(m);
  return CE_OK;
}

}  // namespace

size_t radix_ws_bytes(int64_t n) {
  const int64_t tile = RB * (n > (int64_t(1) << 24) ? 8 : 4);  // the smallest tile a sort of n keys takes
  const int64_t nb = (n + tile - 1) / tile;
  return (size_t)nb * 1024 + 1024 + 512;
}

template <class K, class V>
ce_status radix_sort_pairs(K *k0, V *v0, K *k1, V *v1, Cnt n, int begin_bit, int end_bit, bool iota_values,
                           bool *result_in_alt, Ws &ws, hipStream_t s) {
  *result_in_alt = false;
  if (n.v <= 0) return CE_OK;
  if (n.v <= RS_SMALL) {  // the output goes where that many passes would have left it
    if (end_bit <= begin_bit) end_bit = begin_bit + 1;
    const bool alt = ((end_bit - begin_bit + 7) / 8) & 1;
    K *ko = alt ? k1 : k0;
    V *vo = alt ? v1 : v0;
    if (n.v <= SMB)
      CE_LAUNCH((k_rs_small<K, V, 1>), dim3(1), dim3(SMB), 0, s, k0, (const V *)v0, ko, vo, n, begin_bit, end_bit,
                iota_values ? 1 : 0);
    else
      CE_LAUNCH((k_rs_small<K, V, RS_SMALL / SMB>), dim3(1), dim3(SMB), 0, s, k0, (const V *)v0, ko, vo, n, begin_bit,
                end_bit, iota_values ? 1 : 0);
    CE_HIP(hipGetLastError());
    *result_in_alt = alt;
    return CE_OK;
  }
  switch (radix_ipt(n.v)) {
    case 4:
      return radix_passes<K, V, 4, RB>(k0, v0, k1, v1, n, begin_bit, end_bit, iota_values, result_in_alt, ws, s);
    case 16:
      return radix_passes<K, V, 16, RB>(k0, v0, k1, v1, n, begin_bit, end_bit, iota_values, result_in_alt, ws, s);
    default:
      if (n.v > RS_WIDE)
        return radix_passes<K, V, 8, 2 * RB>(k0, v0, k1, v1, n, begin_bit, end_bit, iota_values, result_in_alt, ws, s);
      return radix_passes<K, V, 8, RB>(k0, v0, k1, v1, n, begin_bit, end_bit, iota_values, result_in_alt, ws, s);
  }
}

template ce_status radix_sort_pairs<uint64_t, uint32_t>(uint64_t *, uint32_t *, uint64_t *, uint32_t *, Cnt, int,
                                                        int, bool, bool *, Ws &, hipStream_t);
template ce_status radix_sort_pairs<uint32_t, uint32_t>(uint32_t *, uint32_t *, uint32_t *, uint32_t *, Cnt, int,
                                                        int, bool, bool *, Ws &, hipStream_t);
template ce_status radix_sort_pairs<uint32_t, uint64_t>(uint32_t *, uint64_t *, uint32_t *, uint64_t *, Cnt, int,
                                                        int, bool, bool *, Ws &, hipStream_t);
template ce_status radix_sort_pairs<uint64_t, uint4>(uint64_t *, uint4 *, uint64_t *, uint4 *, Cnt, int, int,
                                                     bool, bool *, Ws &, hipStream_t);
template ce_status radix_sort_pairs<uint64_t, uint64_t>(uint64_t *, uint64_t *, uint64_t *, uint64_t *, Cnt, int,
                                                        int, bool, bool *, Ws &, hipStream_t);

}  // namespace ce
