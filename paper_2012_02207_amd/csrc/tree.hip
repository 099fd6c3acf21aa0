// Tree construction on gfx950: root box, 63-bit Morton keys, stable LSD radix
// sort, sorted SoA gather, breadth-first cells, masses, centres and radii.
//
// The paper builds an octree over the bodies (section 2.1, flowchart caption)
// and reuses the tree of its base code without describing it; the reading
// implemented here: cubic root box over the bodies' extent, 21 bits per axis,
// x most significant within each octal digit, a stable sort (ties keep the
// caller's order), cells = maximal runs of keys sharing a prefix, a cell with
// more than n_leaf bodies split into its non-empty octants (unless at level 21),
// ids breadth first (by level, then key order).  Expansion centre = centre of
// mass; size = largest distance of a body from it (section 2.3, "sizes").
#include <hip/hip_runtime.h>

#include <algorithm>
#include <climits>
#include <cmath>

#include "fmm_device.h"

namespace fmm {

// ===================================================================== scan
constexpr int SCAN_T = 256, SCAN_I = 8, SCAN_TILE = SCAN_T * SCAN_I;

__device__ inline int block_excl_scan(int v, int* sh, int& total) {
  // sh: SCAN_T ints; returns exclusive prefix of v over the block
  int t = threadIdx.x;
  sh[t] = v;
  __syncthreads();
  for (int o = 1; o < SCAN_T; o <<= 1) {
    int a = t >= o ? sh[t - o] : 0;
    __syncthreads();
    sh[t] += a;
    __syncthreads();
  }
  total = sh[SCAN_T - 1];
  int ex = sh[t] - v;
  __syncthreads();
  return ex;
}

__global__ void __launch_bounds__(SCAN_T) k_scan_reduce(const int* in, int64_t n, int* bsum) {
  __shared__ int sh[SCAN_T];
  int64_t base = (int64_t)blockIdx.x * SCAN_TILE;
  int s = 0;
  for (int i = 0; i < SCAN_I; i++) {
    int64_t j = base + (int64_t)i * SCAN_T + threadIdx.x;
    if (j < n) s += in[j];
  }
  int tot;
  block_excl_scan(s, sh, tot);
  if (threadIdx.x == 0) bsum[blockIdx.x] = tot;
}

// exclusive scan of one tile per block, plus a per-block offset
__global__ void __launch_bounds__(SCAN_T) k_scan_apply(const int* in, int* out, int64_t n,
                                                      const int* boff, long long* total,
                                                      int64_t nblocks) {
  __shared__ int sh[SCAN_T];
  int64_t base = (int64_t)blockIdx.x * SCAN_TILE + (int64_t)threadIdx.x * SCAN_I;
  int v[SCAN_I];
  int s = 0;
  for (int i = 0; i < SCAN_I; i++) {
    int64_t j = base + i;
    v[i] = j < n ? in[j] : 0;
    s += v[i];
  }
  int tot;
  int ex = block_excl_scan(s, sh, tot);
  int off = (boff ? boff[blockIdx.x] : 0) + ex;
  for (int i = 0; i < SCAN_I; i++) {
    int64_t j = base + i;
    if (j < n) out[j] = off;
    off += v[i];
  }
  if (total && blockIdx.x == nblocks - 1 && threadIdx.x == SCAN_T - 1)
    *total = (long long)(boff ? boff[blockIdx.x] : 0) + (long long)tot;
}

void exclusive_scan(Ctx& c, const int* in, int* out, int64_t n, long long* total_dev) {
  // recursive three-phase scan; scratch from c.scan_tmp
  int64_t sizes[16];  // block counts of the recursion levels (SCAN_TILE^16 exceeds any n)
  int nlev = 0;
  int64_t m = n;
  while (m > SCAN_TILE) {
    m = ceil_div(m, SCAN_TILE);
    sizes[nlev++] = m;
  }
  size_t need = 0;
  for (int l = 0; l < nlev; l++) need += 2 * (size_t)sizes[l] + 64;
  ensure(c.ws, c.scan_tmp, need + 64);
  if (n == 0) {
    if (total_dev) HIPCHK(hipMemsetAsync(total_dev, 0, sizeof(long long), c.stream));
    return;
  }
  if (nlev == 0) {
    hipLaunchKernelGGL(k_scan_apply, dim3(1), dim3(SCAN_T), 0, c.stream, in, out, n, nullptr,
                       total_dev, (int64_t)1);
    HIPCHK(hipGetLastError());
    return;
  }
  // level 0
  int* bsum = c.scan_tmp.p;
  int* boff = bsum + sizes[0] + 32;
  int64_t nb = sizes[0];
  hipLaunchKernelGGL(k_scan_reduce, dim3(nb), dim3(SCAN_T), 0, c.stream, in, n, bsum);
  HIPCHK(hipGetLastError());
  // scan of block sums (recursive via a nested context-free call)
  {
    // temporarily carve the remaining scratch for the recursion
    dbuf<int> saved = c.scan_tmp;
    c.scan_tmp.p = boff + nb + 32;
    c.scan_tmp.cap = saved.cap - (size_t)(c.scan_tmp.p - saved.p);
    exclusive_scan(c, bsum, boff, nb, nullptr);
    c.scan_tmp = saved;
  }
  hipLaunchKernelGGL(k_scan_apply, dim3(nb), dim3(SCAN_T), 0, c.stream, in, out, n, boff,
                     total_dev, nb);
  HIPCHK(hipGetLastError());
}

// ===================================================================== root box
constexpr int BB_T = 256;

__global__ void __launch_bounds__(BB_T) k_bbox_partial(const double* pos, int64_t n, double* part) {
  __shared__ double sh[6][BB_T];
  double lo[3], hi[3];
  int64_t i0 = (int64_t)blockIdx.x * BB_T + threadIdx.x;
  int64_t first = i0 < n ? i0 : 0;
  for (int d = 0; d < 3; d++) lo[d] = hi[d] = pos[3 * first + d];
  for (int64_t i = i0; i < n; i += (int64_t)gridDim.x * BB_T)
    for (int d = 0; d < 3; d++) {
      double v = pos[3 * i + d];
      if (v < lo[d]) lo[d] = v;
      if (v > hi[d]) hi[d] = v;
    }
  for (int d = 0; d < 3; d++) {
    sh[d][threadIdx.x] = lo[d];
    sh[3 + d][threadIdx.x] = hi[d];
  }
  __syncthreads();
  for (int o = BB_T / 2; o > 0; o >>= 1) {
    if (threadIdx.x < o)
      for (int d = 0; d < 3; d++) {
        double a = sh[d][threadIdx.x + o], b = sh[3 + d][threadIdx.x + o];
        if (a < sh[d][threadIdx.x]) sh[d][threadIdx.x] = a;
        if (b > sh[3 + d][threadIdx.x]) sh[3 + d][threadIdx.x] = b;
      }
    __syncthreads();
  }
  if (threadIdx.x < 6) part[blockIdx.x * 6 + threadIdx.x] = sh[threadIdx.x][0];
}

// lo = min, L = largest extent (1 if zero), s = 2^21 / L  (rootbox = lo[3], L, s)
__global__ void __launch_bounds__(BB_T) k_bbox_final(const double* part, int nb, double* rootbox) {
  __shared__ double sh[6][BB_T];
  int t = threadIdx.x;
  double lo[3], hi[3];
  for (int d = 0; d < 3; d++) {
    lo[d] = part[d];
    hi[d] = part[3 + d];
  }
  for (int b = t; b < nb; b += BB_T)
    for (int d = 0; d < 3; d++) {
      if (part[6 * b + d] < lo[d]) lo[d] = part[6 * b + d];
      if (part[6 * b + 3 + d] > hi[d]) hi[d] = part[6 * b + 3 + d];
    }
  for (int d = 0; d < 3; d++) {
    sh[d][t] = lo[d];
    sh[3 + d][t] = hi[d];
  }
  __syncthreads();
  for (int o = BB_T / 2; o > 0; o >>= 1) {
    if (t < o)
      for (int d = 0; d < 3; d++) {
        if (sh[d][t + o] < sh[d][t]) sh[d][t] = sh[d][t + o];
        if (sh[3 + d][t + o] > sh[3 + d][t]) sh[3 + d][t] = sh[3 + d][t + o];
      }
    __syncthreads();
  }
  if (t != 0) return;
  double L = sh[3][0] - sh[0][0];
  if (sh[4][0] - sh[1][0] > L) L = sh[4][0] - sh[1][0];
  if (sh[5][0] - sh[2][0] > L) L = sh[5][0] - sh[2][0];
  if (L == 0.0) L = 1.0;
  rootbox[0] = sh[0][0];
  rootbox[1] = sh[1][0];
  rootbox[2] = sh[2][0];
  rootbox[3] = L;
  rootbox[4] = 2097152.0 / L;
}

// one workgroup per system (the systems of a batch): the same box over the
// bodies [off[s], off[s+1]) (min and max are exact in any order)
__global__ void __launch_bounds__(BB_T) k_bbox_sys(const double* pos, const int* off, double* rootbox) {
  __shared__ double sh[6][BB_T];
  int sys = blockIdx.x, t = threadIdx.x;
  int64_t b = off[sys], e = off[sys + 1];
  double lo[3], hi[3];
  for (int d = 0; d < 3; d++) lo[d] = hi[d] = pos[3 * b + d];
  for (int64_t i = b + t; i < e; i += BB_T)
    for (int d = 0; d < 3; d++) {
      double v = pos[3 * i + d];
      if (v < lo[d]) lo[d] = v;
      if (v > hi[d]) hi[d] = v;
    }
  for (int d = 0; d < 3; d++) {
    sh[d][t] = lo[d];
    sh[3 + d][t] = hi[d];
  }
  __syncthreads();
  for (int o = BB_T / 2; o > 0; o >>= 1) {
    if (t < o)
      for (int d = 0; d < 3; d++) {
        if (sh[d][t + o] < sh[d][t]) sh[d][t] = sh[d][t + o];
        if (sh[3 + d][t + o] > sh[3 + d][t]) sh[3 + d][t] = sh[3 + d][t + o];
      }
    __syncthreads();
  }
  if (t != 0) return;
  double L = sh[3][0] - sh[0][0];
  if (sh[4][0] - sh[1][0] > L) L = sh[4][0] - sh[1][0];
  if (sh[5][0] - sh[2][0] > L) L = sh[5][0] - sh[2][0];
  if (L == 0.0) L = 1.0;
  double* rb = rootbox + 8 * sys;
  rb[0] = sh[0][0];
  rb[1] = sh[1][0];
  rb[2] = sh[2][0];
  rb[3] = L;
  rb[4] = 2097152.0 / L;
}

// ===================================================================== keys
__device__ __forceinline__ uint64_t spread3(uint64_t x) {
  x &= 0x1fffffull;
  x = (x | (x << 32)) & 0x1f00000000ffffull;
  x = (x | (x << 16)) & 0x1f0000ff0000ffull;
  x = (x | (x << 8)) & 0x100f00f00f00f00full;
  x = (x | (x << 4)) & 0x10c30c30c30c30c3ull;
  x = (x | (x << 2)) & 0x1249249249249249ull;
  return x;
}

__device__ __forceinline__ uint64_t compact3(uint64_t x) {
  x &= 0x1249249249249249ull;
  x = (x ^ (x >> 2)) & 0x10c30c30c30c30c3ull;
  x = (x ^ (x >> 4)) & 0x100f00f00f00f00full;
  x = (x ^ (x >> 8)) & 0x1f0000ff0000ffull;
  x = (x ^ (x >> 16)) & 0x1f00000000ffffull;
  x = (x ^ (x >> 32)) & 0x1fffffull;
  return x;
}

// key of a body in the box (lo, L, 2^21 / L)
__device__ __forceinline__ uint64_t morton_key(const double* x, const double* rootbox) {
  double s = rootbox[4];
  uint64_t q[3];
  for (int d = 0; d < 3; d++) {
    double t = floor((x[d] - rootbox[d]) * s);
    uint64_t v = (uint64_t)t;
    q[d] = v > 2097151ull ? 2097151ull : v;
  }
  return (spread3(q[0]) << 2) | (spread3(q[1]) << 1) | spread3(q[2]);
}

__global__ void k_keys(const double* pos, int64_t n, const double* rootbox_all, const int* sys_off,
                       int nsys, uint64_t* key, int* idx) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const double* rootbox = rootbox_all + (nsys > 1 ? 8 * system_of(sys_off, nsys, i) : 0);
  key[i] = morton_key(pos + 3 * i, rootbox);
  idx[i] = (int)i;
}

// ===================================================================== radix sort
// Stable LSD sort of (63-bit key, int payload), 8-bit digits.  Each block ranks a
// tile of I x RS_T keys: waves walk their sub-tile in 64-key chunks, computing
// for every key its rank among equal digits with 8 ballots, so the rank order
// equals the input order (stability).  Global digit offsets come from a
// per-digit scan of the digit-major block histograms (k_rs_rowscan).
// 16 keys per thread, or 4 up to RS_SMALL keys, whose few large tiles would leave
// most of the chip idle (30011 bodies: 16 us per scatter of 8 tiles, 6.5 of 30).
constexpr int RS_T = 256, RS_W = RS_T / 64, RS_I = 16, RS_I_SMALL = 4;
constexpr int64_t RS_SMALL = 1 << 19;

template <int RS_I, class K>
__global__ void __launch_bounds__(RS_T) k_rs_hist(const K* key, int64_t n, int shift, int* hist,
                                                  int nblocks) {
  __shared__ int cnt[256];
  cnt[threadIdx.x] = 0;
  __syncthreads();
  int64_t base = (int64_t)blockIdx.x * RS_T * RS_I;
  for (int i = 0; i < RS_I; i++) {
    int64_t j = base + (int64_t)i * RS_T + threadIdx.x;
    if (j < n) atomicAdd(&cnt[(key[j] >> shift) & 255], 1);
  }
  __syncthreads();
  hist[(int64_t)threadIdx.x * nblocks + blockIdx.x] = cnt[threadIdx.x];
}

// Per digit, the exclusive prefix of its tile counts over the tiles (one
// workgroup per digit, the row in runs of 8 x RS_T counts, each thread taking
// 8 consecutive ones), and the digit's total.  The scatter adds the totals of
// the smaller digits itself.
__global__ void __launch_bounds__(RS_T) k_rs_rowscan(const int* __restrict__ hist, int nblocks, int* offs,
                                                     int* rowtot) {
  __shared__ int wsum[2][RS_W];
  int d = blockIdx.x, lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int* row = hist + (int64_t)d * nblocks;
  int* orow = offs + (int64_t)d * nblocks;
  int carry = 0;
  for (int base = 0, it = 0; base < nblocks; base += 8 * RS_T, it ^= 1) {
    int t0 = base + (int)threadIdx.x * 8;
    int v[8], sum = 0;
#pragma unroll
    for (int k = 0; k < 8; k++) {
      v[k] = t0 + k < nblocks ? row[t0 + k] : 0;
      sum += v[k];
    }
    int incl = sum;
    for (int o = 1; o < 64; o <<= 1) {
      int y = __shfl_up(incl, o, 64);
      if (lane >= o) incl += y;
    }
    if (lane == 63) wsum[it][w] = incl;  // alternate buffers: no second barrier per run
    __syncthreads();
    int before = 0, total = 0;
    for (int ww = 0; ww < RS_W; ww++) {
      if (ww < w) before += wsum[it][ww];
      total += wsum[it][ww];
    }
    int run = carry + before + incl - sum;
#pragma unroll
    for (int k = 0; k < 8; k++) {
      if (t0 + k < nblocks) orow[t0 + k] = run;
      run += v[k];
    }
    carry += total;
  }
  if (threadIdx.x == 0) rowtot[d] = carry;
}

// Exclusive prefix of x over the workgroup's RS_T threads (sum: the total).
__device__ __forceinline__ int rs_block_excl(int x, int* wsum, int& sum) {
  int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  int incl = x;
  for (int o = 1; o < 64; o <<= 1) {
    int y = __shfl_up(incl, o, 64);
    if (lane >= o) incl += y;
  }
  if (lane == 63) wsum[w] = incl;
  __syncthreads();
  int before = 0;
  sum = 0;
  for (int ww = 0; ww < RS_W; ww++) {
    if (ww < w) before += wsum[ww];
    sum += wsum[ww];
  }
  __syncthreads();
  return before + incl - x;
}

template <int RS_I, bool VAL, class K>
struct RadixTile {
  int wcnt[RS_W][256];
  int goff[256], lofs[256], wsum[RS_W];
  K sk[RS_T * RS_I];
  int sv[VAL ? RS_T * RS_I : 1];
};

// Ranks as above, then the tile [tile0, tile0 + tcount) is reordered by digit in
// LDS and written out with consecutive lanes on consecutive destinations (each
// digit's run of the tile is contiguous in the output, from goff on), so the
// global writes coalesce.
template <int RS_I, bool VAL, class KI, class KO>
__device__ __forceinline__ void radix_tile(RadixTile<RS_I, VAL, KI>& s, const KI* kin, const int* vin, KO* kout,
                                           int* vout, int64_t n, int64_t tile0, int tcount, int shift, int dmask = 255) {
  int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  for (int t = threadIdx.x; t < RS_W * 256; t += RS_T) (&s.wcnt[0][0])[t] = 0;
  __syncthreads();
  int base = w * (64 * RS_I);
  KI k[RS_I];
  int v[RS_I], rank[RS_I];
  uint64_t lt = lanemask_lt();
  for (int c = 0; c < RS_I; c++) {
    int j = base + c * 64 + lane;
    bool valid = j < tcount;
    k[c] = valid ? kin[tile0 + j] : 0;
    if (VAL) v[c] = valid ? vin[tile0 + j] : 0;
    int d = (int)((k[c] >> shift) & dmask);
    uint64_t peers = ballot(valid);
    for (int b = 0; b < 8; b++) {
      bool bit = (d >> b) & 1;
      uint64_t bb = ballot(bit);
      peers &= bit ? bb : ~bb;
    }
    int before = __popcll(peers & lt);
    int cnt = s.wcnt[w][d];
    rank[c] = cnt + before;
    // the highest peer publishes the new running count for this digit
    if (valid && (peers >> lane) == 1ull) s.wcnt[w][d] = cnt + __popcll(peers);
    __builtin_amdgcn_wave_barrier();
  }
  __syncthreads();
  // per digit: offsets of the waves within the tile's run, and the run length
  int d0 = threadIdx.x, tot = 0;
  for (int ww = 0; ww < RS_W; ww++) {
    int t = s.wcnt[ww][d0];
    s.wcnt[ww][d0] = tot;
    tot += t;
  }
  int all;
  s.lofs[d0] = rs_block_excl(tot, s.wsum, all);
  __syncthreads();
  for (int c = 0; c < RS_I; c++) {
    if (base + c * 64 + lane >= tcount) continue;
    int d = (int)((k[c] >> shift) & dmask);
    int lp = s.lofs[d] + s.wcnt[w][d] + rank[c];
    s.sk[lp] = k[c];
    if (VAL) s.sv[lp] = v[c];
  }
  __syncthreads();
  for (int t = threadIdx.x; t < tcount; t += RS_T) {
    KI key = s.sk[t];
    int d = (int)((key >> shift) & dmask);
    int64_t dst = (int64_t)s.goff[d] + (t - s.lofs[d]);
    if (dst < n) {  // always true when the ranks are consistent with the histogram
      kout[dst] = (KO)key;
      if (VAL) vout[dst] = s.sv[t];
    }
  }
}

template <int RS_I, bool VAL, class KI, class KO>
__global__ void __launch_bounds__(RS_T) k_rs_scatter(const KI* kin, const int* vin, KO* kout, int* vout,
                                                     int64_t n, int shift, const int* offs, const int* rowtot,
                                                     int nblocks) {
  __shared__ RadixTile<RS_I, VAL, KI> s;
  // start of this digit in the output: the totals of the smaller digits
  // plus the counts of the earlier tiles
  int all, excl = rs_block_excl(rowtot[threadIdx.x], s.wsum, all);
  s.goff[threadIdx.x] = excl + offs[(int64_t)threadIdx.x * nblocks + blockIdx.x];
  int64_t tile0 = (int64_t)blockIdx.x * (RS_T * RS_I);
  radix_tile<RS_I, VAL, KI, KO>(s, kin, vin, kout, vout, n, tile0,
                                (int)min((int64_t)(RS_T * RS_I), n - tile0), shift);
}

// ---- second split of a list already split into 256 parts ----------------------
// The parts' sizes are rowtot; a tile belongs to one part (at most one partial
// tile per part), and a part's tiles are split by the next 8 bits on their own.
struct SplitTile {
  int part, first, count;  // part, first entry and entries of this tile (part -1: no such tile)
  int tile, tiles;         // first tile of the part, its tiles
  int start;               // first entry of the part
};
// tile blk, or (part >= 0) the tiles of that part
template <int TILE>
__device__ __forceinline__ SplitTile split_tile(const int* rowtot, int blk, int part, int* wsum, SplitTile* sh) {
  int d = threadIdx.x, all;
  int sz = rowtot[d], nt = (sz + TILE - 1) / TILE;
  int start = rs_block_excl(sz, wsum, all);
  int tile = rs_block_excl(nt, wsum, all);
  if (d == 0) sh->part = -1;
  __syncthreads();
  if (part >= 0 ? d == part : (blk >= tile && blk < tile + nt)) {
    int o = part >= 0 ? 0 : (blk - tile) * TILE;
    *sh = SplitTile{d, start + o, min(TILE, sz - o), tile, nt, start};
  }
  __syncthreads();
  return *sh;
}

template <int RS_I>
__global__ void __launch_bounds__(RS_T) k_split_hist(const uint32_t* __restrict__ key, int shift, int dmask,
                                                     const int* __restrict__ rowtot, int* __restrict__ hist) {
  __shared__ int cnt[256], wsum[RS_W];
  __shared__ SplitTile sh;
  cnt[threadIdx.x] = 0;
  SplitTile t = split_tile<RS_T * RS_I>(rowtot, blockIdx.x, -1, wsum, &sh);
  if (t.part < 0) return;
  for (int j = threadIdx.x; j < t.count; j += RS_T) atomicAdd(&cnt[(key[t.first + j] >> shift) & dmask], 1);
  __syncthreads();
  hist[(int64_t)blockIdx.x * 256 + threadIdx.x] = cnt[threadIdx.x];
}

// a workgroup per part: the counts become the destinations of the tiles' runs
// (a thread per digit down the tiles), and the starts of the part's sub-parts
template <int RS_I>
__global__ void __launch_bounds__(RS_T) k_split_scan(const int* __restrict__ rowtot, int* hist, int sub, int* fstart) {
  __shared__ int wsum[RS_W];
  __shared__ SplitTile sh;
  SplitTile t = split_tile<RS_T * RS_I>(rowtot, 0, blockIdx.x, wsum, &sh);
  int d = threadIdx.x;
  int* h = hist + (int64_t)t.tile * 256 + d;
  int tot = 0;
#pragma unroll 8
  for (int i = 0; i < t.tiles; i++) tot += h[i * 256];
  int all, run = t.start + rs_block_excl(tot, wsum, all);
  if (d < sub) fstart[blockIdx.x * sub + d] = run;
  if (blockIdx.x == 255 && d == 0) fstart[256 * sub] = t.start + all;
  for (int i0 = 0; i0 < t.tiles; i0 += 8) {
    int v[8];
#pragma unroll
    for (int k = 0; k < 8; k++) v[k] = h[min(i0 + k, t.tiles - 1) * 256];
#pragma unroll
    for (int k = 0; k < 8; k++) {
      if (i0 + k < t.tiles) h[(i0 + k) * 256] = run;
      run += v[k];
    }
  }
}

template <int RS_I>
__global__ void __launch_bounds__(RS_T) k_split_scatter(const uint32_t* __restrict__ kin, uint32_t* __restrict__ kout,
                                                        int64_t n, int shift, int dmask, const int* __restrict__ rowtot,
                                                        const int* __restrict__ dest) {
  __shared__ RadixTile<RS_I, false, uint32_t> s;
  __shared__ SplitTile sh;
  SplitTile t = split_tile<RS_T * RS_I>(rowtot, blockIdx.x, -1, s.wsum, &sh);
  if (t.part < 0) return;
  s.goff[threadIdx.x] = dest[(int64_t)blockIdx.x * 256 + threadIdx.x];
  radix_tile<RS_I, false, uint32_t, uint32_t>(s, kin, nullptr, kout, nullptr, n, t.first, t.count, shift, dmask);
}

// One 8-bit pass from kin (and vin) to kout (vout).
template <bool VAL, class KI, class KO>
static void radix_pass(Ctx& c, const KI* kin, const int* vin, KO* kout, int* vout, int64_t n, int shift) {
  bool small = n <= RS_SMALL;
  int nb = (int)ceil_div(n, RS_T * (small ? RS_I_SMALL : RS_I));
  ensure(c.ws, c.sort_hist, (size_t)256 * nb * 2 + 256 + 64);
  int* hist = c.sort_hist.p;
  int* offs = hist + (size_t)256 * nb;
  int* rowtot = offs + (size_t)256 * nb;
  auto kh = small ? k_rs_hist<RS_I_SMALL, KI> : k_rs_hist<RS_I, KI>;
  auto ks = small ? k_rs_scatter<RS_I_SMALL, VAL, KI, KO> : k_rs_scatter<RS_I, VAL, KI, KO>;
  hipLaunchKernelGGL(kh, dim3(nb), dim3(RS_T), 0, c.stream, kin, n, shift, hist, nb);
  hipLaunchKernelGGL(k_rs_rowscan, dim3(256), dim3(RS_T), 0, c.stream, hist, nb, offs, rowtot);
  hipLaunchKernelGGL(ks, dim3(nb), dim3(RS_T), 0, c.stream, kin, vin, kout, vout, n, shift, offs, rowtot, nb);
  HIPCHK(hipGetLastError());
}

// Stable LSD sort of n keys over bits [0, nbits) (8 bits per pass), with an
// optional int payload.  Data ping-pongs between (k0, v0) and (k1, v1); the
// return value tells which buffer holds the result (0 or 1).
int radix_sort(Ctx& c, uint64_t* k0, int* v0, uint64_t* k1, int* v1, int64_t n, int nbits) {
  if (n <= 0) return 0;
  int src = 0;
  uint64_t* kk[2] = {k0, k1};
  int* vv[2] = {v0, v1};
  for (int shift = 0; shift < nbits; shift += 8) {
    if (v0)
      radix_pass<true>(c, kk[src], vv[src], kk[1 - src], vv[1 - src], n, shift);
    else
      radix_pass<false>(c, kk[src], (const int*)nullptr, kk[1 - src], (int*)nullptr, n, shift);
    src = 1 - src;
  }
  return src;
}

// Splits n 64-bit keys by the 8 bits from bit `shift` on; the low 32 bits of the
// keys go to out.  Returns the 256 parts' sizes (device).
const int* radix_split(Ctx& c, const uint64_t* in, uint32_t* out, int64_t n, int shift) {
  radix_pass<false>(c, in, (const int*)nullptr, out, (int*)nullptr, n, shift);
  int nb = (int)ceil_div(n, RS_T * (n <= RS_SMALL ? RS_I_SMALL : RS_I));
  return c.sort_hist.p + (size_t)512 * nb;
}

// scratch of radix_split2 behind radix_split's
size_t radix_split2_ints(int64_t n, int sub) {
  int64_t nb = ceil_div(n, RS_T * (n <= RS_SMALL ? RS_I_SMALL : RS_I));
  int64_t nt = ceil_div(n, RS_T * RS_I) + 256;
  return (size_t)(512 * nb + 256 + 256 * nt + 256 * sub + 64);
}

// Splits each of the 256 parts again, by the log2(sub) bits from bit `shift` on
// (sub <= 256; c.sort_hist holds radix_split2_ints).  Returns the first
// entries of the 256 sub sub-parts, and n (device).
const int* radix_split2(Ctx& c, const uint32_t* in, uint32_t* out, int64_t n, int shift, int sub, const int* rowtot) {
  int nt = (int)(ceil_div(n, RS_T * RS_I) + 256);
  int* hist = const_cast<int*>(rowtot) + 256;
  int* fstart = hist + (size_t)256 * nt;
  hipLaunchKernelGGL(k_split_hist<RS_I>, dim3(nt), dim3(RS_T), 0, c.stream, in, shift, sub - 1, rowtot, hist);
  hipLaunchKernelGGL(k_split_scan<RS_I>, dim3(256), dim3(RS_T), 0, c.stream, rowtot, hist, sub, fstart);
  hipLaunchKernelGGL(k_split_scatter<RS_I>, dim3(nt), dim3(RS_T), 0, c.stream, in, out, n, shift, sub - 1, rowtot, hist);
  HIPCHK(hipGetLastError());
  return fstart;
}

// sorts c.key[0]/c.idx[0] (n entries) over bits [0, nbits); result in key[0]/idx[0]
void radix_sort_keys(Ctx& c, int64_t n, int nbits) {
  int r = radix_sort(c, c.key[0].p, c.idx[0].p, c.key[1].p, c.idx[1].p, n, nbits);
  if (r != 0) {
    std::swap(c.key[0], c.key[1]);
    std::swap(c.idx[0], c.idx[1]);
  }
}

// second key of a batch: the system of each body of the key-sorted order
// (from its caller index), payload = its position in that order
__global__ void k_sys_keys(const int* idx, int64_t n, const int* sys_off, int nsys, uint64_t* skey,
                           int* spos) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  skey[i] = (uint64_t)system_of(sys_off, nsys, idx[i]);
  spos[i] = (int)i;
}

__global__ void k_apply_pos(const int* spos, int64_t n, const uint64_t* kin, const int* vin,
                            uint64_t* kout, int* vout) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  int j = spos[i];
  kout[i] = kin[j];
  vout[i] = vin[j];
}

__global__ void k_gather(const double* pos, const double* mass, const int* idx, int64_t n, double* sx,
                         double* sy, double* sz, double4* pm) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  int o = idx[i];
  double x = pos[3 * (int64_t)o], y = pos[3 * (int64_t)o + 1], z = pos[3 * (int64_t)o + 2], m = mass[o];
  sx[i] = x;
  sy[i] = y;
  sz[i] = z;
  pm[i] = make_double4(x, y, z, m);
}

// ===================================================================== small systems
// Box, keys, sort and gather of one system of up to TS_MAX bodies by one
// workgroup: one launch instead of 28 (8 passes of three, two for the box, keys
// and gather), each of which costs some 5 us whatever its size (with the
// lists below, 1000 bodies 860 -> 600 us, 4096 1.22 -> 0.99 ms).
constexpr int TS_I = 8;
constexpr int TS_MAX = BS_T * TS_I;

// The box as k_bbox_final forms it, the keys, their stable sort in LDS, and the
// bodies gathered into that order.  Bound by latency: 27 us at 1000 bodies, 54 at 4096.
__global__ void __launch_bounds__(BS_T) k_tree_small(const double* __restrict__ pos, const double* __restrict__ mass,
                                                     int n, double* __restrict__ rootbox, uint64_t* __restrict__ key,
                                                     int* __restrict__ idx, double* __restrict__ sx,
                                                     double* __restrict__ sy, double* __restrict__ sz,
                                                     double4* __restrict__ pm) {
  __shared__ BlockSort<uint64_t, TS_I, true> bs;
  __shared__ double ext[6][(BS_T / 64)];
  __shared__ double box[5];
  int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  double lo[3], hi[3];
  for (int d = 0; d < 3; d++) lo[d] = hi[d] = pos[3 * min(tid, n - 1) + d];
  for (int i = tid; i < n; i += BS_T)
    for (int d = 0; d < 3; d++) {
      double v = pos[3 * i + d];
      if (v < lo[d]) lo[d] = v;
      if (v > hi[d]) hi[d] = v;
    }
  for (int d = 0; d < 3; d++) {
    for (int o = 32; o > 0; o >>= 1) {
      double a = __shfl_xor(lo[d], o, 64), b = __shfl_xor(hi[d], o, 64);
      if (a < lo[d]) lo[d] = a;
      if (b > hi[d]) hi[d] = b;
    }
    if (lane == 0) {
      ext[d][w] = lo[d];
      ext[3 + d][w] = hi[d];
    }
  }
  __syncthreads();
  if (tid == 0) {
    double L = 0.0;
    for (int d = 0; d < 3; d++) {
      double a = ext[d][0], b = ext[3 + d][0];
      for (int ww = 1; ww < (BS_T / 64); ww++) {
        if (ext[d][ww] < a) a = ext[d][ww];
        if (ext[3 + d][ww] > b) b = ext[3 + d][ww];
      }
      box[d] = a;
      if (d == 0 || b - a > L) L = b - a;
    }
    if (L == 0.0) L = 1.0;
    box[3] = L;
    box[4] = 2097152.0 / L;
    for (int k = 0; k < 5; k++) rootbox[k] = box[k];
  }
  __syncthreads();
  int C = (n + BS_T - 1) / BS_T;
  uint64_t k[TS_I];
  int v[TS_I];
#pragma unroll
  for (int c = 0; c < TS_I; c++) {
    int i = (w * C + c) * 64 + lane;
    bool ok = c < C && i < n;
    k[c] = ok ? morton_key(pos + 3 * i, box) : ~0ull;
    v[c] = i;
  }
  block_sort(bs, k, v, C, 64);
#pragma unroll
  for (int c = 0; c < TS_I; c++) {
    int i = (w * C + c) * 64 + lane;
    if (c < C && i < n) {
      int o = v[c];
      key[i] = k[c];
      idx[i] = o;
      double x = pos[3 * o], y = pos[3 * o + 1], z = pos[3 * o + 2], m = mass[o];
      sx[i] = x;
      sy[i] = y;
      sz[i] = z;
      pm[i] = make_double4(x, y, z, m);
    }
  }
}

// ===================================================================== cells
// The cells straight from the sorted keys, all levels at once.  With lcp the
// number of leading octal digits that two keys share (-1 across systems) and
// D(i) the deepest level on which body i is in a cell of more than n_leaf
// bodies (the largest lcp(key[k], key[k + n_leaf]) over the windows k .. k +
// n_leaf that hold i), body i's leaf is on level Lf(i) = min(D(i) + 1, 21),
// the cells that start at i are those of the levels lcp(key[i-1], key[i]) + 1
// .. Lf(i), and the cells that end with it those of lcp(key[i], key[i+1]) + 1
// .. Lf(i).  Ids are breadth first, so a cell's id is its level's first id plus
// the number of that level's cells that start before it: k_cell_levels counts
// the starts per level and tile, k_rs_rowscan sums them over the tiles, and
// k_cell_emit writes the cells, the leaf list and every body's leaf.  Three
// launches (35 us in all at N = 2^20, 25 us at N = 1000) instead of three per
// level for 12 to 22 levels and four for the leaf lists (290 and 150 us).
constexpr int CT_T = 256, CT_TILE = 1024, CT_NLEAF_MAX = 1024;
constexpr int CT_LEVELS = FMM_MAX_LEVEL + 1;  // levels 0..21
constexpr int CT_ROWS = 2 * CT_LEVELS;        // counts per tile: cells of each level, leaves of each level

// leading octal digits shared by two 63-bit keys
__device__ __forceinline__ int key_lcp(uint64_t a, uint64_t b) {
  return a == b ? FMM_MAX_LEVEL : (__builtin_clzll(a ^ b) - 1) / 3;
}

// lev[i]: (lcp(key[i-1], key[i]) + 1) << 8 | Lf(i); cnt[row * nblocks + block]:
// the tile's counts; also clears nchild[0 .. cap), which the emit counts up
__global__ void __launch_bounds__(CT_T) k_cell_levels(int n, int n_leaf, const uint64_t* __restrict__ key,
                                                      const int* __restrict__ sys_off, int nsys,
                                                      unsigned short* __restrict__ lev, int* __restrict__ cnt,
                                                      int nblocks, int* __restrict__ nchild, int cap) {
  __shared__ signed char win[2][CT_TILE + CT_NLEAF_MAX];
  __shared__ int rows[CT_ROWS];
  for (int i = blockIdx.x * CT_T + threadIdx.x; i < cap; i += gridDim.x * CT_T) nchild[i] = 0;
  if (threadIdx.x < CT_ROWS) rows[threadIdx.x] = 0;
  int t0 = blockIdx.x * CT_TILE;
  int w0 = t0 - n_leaf;        // first window of the tile's bodies
  int nw = CT_TILE + n_leaf;   // windows w0 .. t0 + CT_TILE - 1
  for (int u = threadIdx.x; u < nw; u += CT_T) {
    int k = w0 + u, c = -1;
    if (k >= 0 && k + n_leaf < n) {
      bool same = nsys == 1 || sys_off[system_of(sys_off, nsys, k) + 1] > k + n_leaf;
      if (same) c = min(key_lcp(key[k], key[k + n_leaf]), FMM_MAX_LEVEL - 1);
    }
    win[0][u] = (signed char)c;
  }
  __syncthreads();
  // largest over 2^j windows from each on, up to the last j with 2^j <= n_leaf + 1
  int cur = 0, len = 1;
  while (2 * len <= n_leaf + 1) {
    for (int u = threadIdx.x; u < nw; u += CT_T) {
      signed char x = win[cur][u];
      if (u + len < nw) x = max(x, win[cur][u + len]);
      win[cur ^ 1][u] = x;
    }
    cur ^= 1;
    len *= 2;
    __syncthreads();
  }
  for (int u = threadIdx.x; u < CT_TILE; u += CT_T) {
    int i = t0 + u;
    if (i >= n) continue;
    int D = max(win[cur][u], win[cur][u + n_leaf + 1 - len]);  // windows i - n_leaf .. i
    int Lf = D + 1;
    int a = -1;
    if (i > 0) {
      bool same = nsys == 1 || sys_off[system_of(sys_off, nsys, i)] != i;
      if (same) a = key_lcp(key[i - 1], key[i]);
    }
    lev[i] = (unsigned short)((a + 1) << 8 | Lf);
    for (int l = a + 1; l <= Lf; l++) atomicAdd(&rows[l], 1);
    if (a < Lf) atomicAdd(&rows[CT_LEVELS + Lf], 1);
  }
  __syncthreads();
  if (threadIdx.x < CT_ROWS) cnt[(size_t)threadIdx.x * nblocks + blockIdx.x] = rows[threadIdx.x];
}

// Bodies per wavefront of a tile are taken 64 at a time; the ranks of the
// starts within 64 bodies come from ballots.  Ids of cap and more are not
// written (the host enlarges the arrays and emits again).
__global__ void __launch_bounds__(CT_T) k_cell_emit(int n, const unsigned short* __restrict__ lev,
                                                    const int* __restrict__ offs, const int* __restrict__ rowtot,
                                                    int nblocks, int cap, int* __restrict__ c_level,
                                                    int* __restrict__ c_begin, int* __restrict__ c_end,
                                                    int* __restrict__ c_parent, int* __restrict__ c_child0,
                                                    int* __restrict__ c_nchild, int* __restrict__ leaf_of,
                                                    int* __restrict__ leaves) {
  constexpr int W = CT_T / 64, STEPS = CT_TILE / CT_T;
  __shared__ int base[W][CT_ROWS];  // first id (or leaf rank) of each wavefront's part, by row
  int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  int i0 = blockIdx.x * CT_TILE + w * 64 * STEPS;
  int top = 0;  // deepest level that has cells
  for (int l = 0; l < CT_LEVELS; l++)
    if (rowtot[l] > 0) top = l;
  // counts of this wavefront's part
  int mine = 0;  // lane r: count of row r
  for (int k = 0; k < STEPS; k++) {
    int i = i0 + 64 * k + lane;
    int v = i < n ? lev[i] : 0xff00;
    int a1 = v >> 8, Lf = v & 255;
    for (int l = 0; l <= top; l++) {
      uint64_t st = ballot(a1 <= l && l <= Lf), lf = ballot(a1 <= l && l == Lf);
      if (lane == l) mine += (int)__popcll(st);
      if (lane == CT_LEVELS + l) mine += (int)__popcll(lf);
    }
  }
  if (lane < CT_ROWS) base[w][lane] = mine;
  __syncthreads();
  if (threadIdx.x < CT_ROWS) {
    int r = threadIdx.x;
    // the row's start: totals of the rows before it (of its kind), then the tiles before this one
    int run = offs[(size_t)r * nblocks + blockIdx.x];
    for (int q = r < CT_LEVELS ? 0 : CT_LEVELS; q < r; q++) run += rowtot[q];
    for (int ww = 0; ww < W; ww++) {
      int c = base[ww][r];
      base[ww][r] = run;
      run += c;
    }
  }
  __syncthreads();
  uint64_t lt = lanemask_lt();
  int next = lane < CT_ROWS ? base[w][lane] : 0;  // lane r: next id (or leaf rank) of row r
  for (int k = 0; k < STEPS; k++) {
    int i = i0 + 64 * k + lane;
    bool ok = i < n;
    int v = ok ? lev[i] : 0xff00;
    int a1 = v >> 8, Lf = v & 255;
    int next1 = ok && i + 1 < n ? lev[i + 1] >> 8 : 0;  // levels above this one's go on past body i
    int prev = -1;       // the cell that holds body i, one level up
    bool prev_st = false;
    for (int l = 0; l <= top; l++) {
      bool st = a1 <= l && l <= Lf, in = ok && l <= Lf;
      uint64_t sm = ballot(st), lm = ballot(st && l == Lf);
      int id0 = __builtin_amdgcn_readlane(next, l), lf0 = __builtin_amdgcn_readlane(next, CT_LEVELS + l);
      int id = id0 + (int)__popcll(sm & lt) + (st ? 1 : 0) - 1;  // the level's last cell that starts at or before i
      if (st && id < cap) {
        c_level[id] = l;
        c_begin[id] = i;
        c_parent[id] = prev;
        if (l == Lf) {
          c_child0[id] = -1;
          leaves[lf0 + (int)__popcll(lm & lt)] = id;
        }
        if (prev >= 0) {
          atomicAdd(&c_nchild[prev], 1);
          if (prev_st) c_child0[prev] = id;
        }
      }
      if (in && id < cap) {
        if (next1 <= l) c_end[id] = i + 1;
        if (l == Lf) leaf_of[i] = id;
      }
      prev = id;
      prev_st = st;
      if (lane == l) next += (int)__popcll(sm);
      if (lane == CT_LEVELS + l) next += (int)__popcll(lm);
    }
  }
}

// Mass, first moments and centre of mass; leaves sum their bodies in sorted order,
// internal cells their children in octant order.  The leaves of all levels in one
// launch, then the internal cells from the deepest level up: every run of
// consecutive levels of up to MC_TOP cells each by one workgroup, level by level,
// a larger level by a launch of its own.  (Levels do not only shrink towards the
// root: a tight clump leaves a few cells on each of many levels below the widest
// one.)  A launch per level for leaves and cells alike took 87 us at 16384 bodies
// and 150 us at 2^20; this takes 20 and 48 us.
struct MomentView {
  const int *cb, *c0, *nch, *level;
  const uint64_t* key;
  const double* rootbox;
  const int* sys_off;
  int nsys;
  double *m, *sx, *sy, *sz, *cx, *cy, *cz;
};

__device__ __forceinline__ void store_moments(const MomentView& v, int c, double M, double X, double Y, double Z) {
  v.m[c] = M;
  v.sx[c] = X;
  v.sy[c] = Y;
  v.sz[c] = Z;
  if (M != 0.0) {
    v.cx[c] = X / M;
    v.cy[c] = Y / M;
    v.cz[c] = Z / M;
  } else {  // massless cell: centre of its cubic box
    int level = v.level[c];
    const double* rootbox = v.rootbox + (v.nsys > 1 ? 8 * system_of(v.sys_off, v.nsys, v.cb[c]) : 0);
    uint64_t k0 = v.key[v.cb[c]];
    int sh = FMM_MAX_LEVEL - level;
    double h = ldexp(rootbox[3], -level);
    double q0 = (double)(compact3(k0 >> 2) >> sh), q1 = (double)(compact3(k0 >> 1) >> sh),
           q2 = (double)(compact3(k0) >> sh);
    v.cx[c] = rootbox[0] + (q0 + 0.5) * h;
    v.cy[c] = rootbox[1] + (q1 + 0.5) * h;
    v.cz[c] = rootbox[2] + (q2 + 0.5) * h;
  }
}

// (bodies are read eight ahead of their sums)
__global__ void k_leaf_moments(int nleaf, const int* __restrict__ leaves, const int* __restrict__ ce, MomentView v,
                               const double4* __restrict__ pm) {
  int li = blockIdx.x * blockDim.x + threadIdx.x;
  if (li >= nleaf) return;
  int c = leaves[li];
  double M = 0.0, X = 0.0, Y = 0.0, Z = 0.0;
  int i = v.cb[c], e = ce[c];
  auto add = [&](const double4& b) {
    M = M + b.w;
    X = X + b.w * b.x;
    Y = Y + b.w * b.y;
    Z = Z + b.w * b.z;
  };
  for (; i + 8 <= e; i += 8) {
    double4 b[8];
#pragma unroll
    for (int u = 0; u < 8; u++) b[u] = pm[i + u];
#pragma unroll
    for (int u = 0; u < 8; u++) add(b[u]);
  }
  for (; i < e; i++) add(pm[i]);
  store_moments(v, c, M, X, Y, Z);
}

__device__ __forceinline__ void cell_sums(const MomentView& v, int c) {
  int k0 = v.c0[c], kn = v.nch[c];
  if (kn == 0) return;
  double M = 0.0, X = 0.0, Y = 0.0, Z = 0.0;
  double m[8], x[8], y[8], z[8];
#pragma unroll
  for (int j = 0; j < 8; j++) {
    int k = k0 + (j < kn ? j : 0);
    m[j] = v.m[k];
    x[j] = v.sx[k];
    y[j] = v.sy[k];
    z[j] = v.sz[k];
  }
#pragma unroll
  for (int j = 0; j < 8; j++) {
    if (j < kn) {
      M = M + m[j];
      X = X + x[j];
      Y = Y + y[j];
      Z = Z + z[j];
    }
  }
  store_moments(v, c, M, X, Y, Z);
}

__global__ void k_cell_sums(int first, int count, MomentView v) {
  int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t < count) cell_sums(v, first + t);
}

// the levels from `from` up to `to`, one workgroup; lvl: first ids (by level)
struct LevelIds {
  int first[FMM_MAX_LEVEL + 2];
};
__global__ void __launch_bounds__(1024) k_cell_sums_run(int from, int to, LevelIds lvl, MomentView v) {
  for (int l = from; l >= to; l--) {
    for (int c = lvl.first[l] + threadIdx.x; c < lvl.first[l + 1]; c += 1024) cell_sums(v, c);
    __syncthreads();  // (global writes of the level are visible to the workgroup)
  }
}

// radius: exact max over each cell's bodies of the squared distance to its
// centre (order independent), in chunks of RAD_CH bodies
constexpr int RAD_T = 256, RAD_CH = CELL_CHUNK;

__global__ void k_rad_chunks(const int* cb, const int* ce, int ncell, int* nchunk) {
  int c = blockIdx.x * blockDim.x + threadIdx.x;
  if (c >= ncell) return;
  nchunk[c] = (int)ceil_div(ce[c] - cb[c], RAD_CH);
}

// one wavefront per chunk (the count stays on the device, so the launch needs
// no host round trip; the grid covers an upper bound of it)
__global__ void __launch_bounds__(RAD_T) k_radius(const int* cb, const int* ce, const int* choff,
                                                 const long long* nchunks, int ncell, const double* sx,
                                                 const double* sy, const double* sz, const double* cx,
                                                 const double* cy, const double* cz,
                                                 unsigned long long* r2bits) {
  int blk = blockIdx.x * (RAD_T / 64) + (threadIdx.x >> 6);
  int lane = threadIdx.x & 63;
  if (blk >= (int)*nchunks) return;
  // cell owning this chunk: last c with choff[c] <= blk
  int lo = 0, hi = ncell - 1;
  while (lo < hi) {
    int mid = (lo + hi + 1) >> 1;
    if (choff[mid] <= blk)
      lo = mid;
    else
      hi = mid - 1;
  }
  int c = lo;
  int64_t b = cb[c] + (int64_t)(blk - choff[c]) * RAD_CH;
  int64_t e = b + RAD_CH < ce[c] ? b + RAD_CH : ce[c];
  double x0 = cx[c], y0 = cy[c], z0 = cz[c];
  double best = 0.0;
  for (int64_t i = b + lane; i < e; i += 64) {
    double dx = sx[i] - x0, dy = sy[i] - y0, dz = sz[i] - z0;
    double d2 = (dx * dx + dy * dy) + dz * dz;
    if (d2 > best) best = d2;
  }
  for (int o = 32; o > 0; o >>= 1) {
    double other = __shfl_xor(best, o, 64);
    if (other > best) best = other;
  }
  if (lane == 0) atomicMax(&r2bits[c], (unsigned long long)__double_as_longlong(best));
}

// radius from the squared maximum; also the packed (centre, radius) record
// the walks read
__global__ void k_radius_final(const unsigned long long* r2bits, int ncell, const double* cx, const double* cy,
                               const double* cz, double* rad, double4* geo) {
  int c = blockIdx.x * blockDim.x + threadIdx.x;
  if (c >= ncell) return;
  double r = sqrt(__longlong_as_double((long long)r2bits[c]));
  rad[c] = r;
  geo[c] = make_double4(cx[c], cy[c], cz[c], r);
}

static inline dim3 grid1(int64_t n, int t = 256) { return dim3((unsigned)ceil_div(n, t)); }

// every body is in one cell per level: at most (depth + 1) n / CELL_CHUNK + ncell chunks
unsigned cell_chunk_blocks(const Ctx& c, int waves_per_block) {
  int64_t max_chunks = (int64_t)(c.depth + 1) * ceil_div(c.n, CELL_CHUNK) + c.ncell;
  return (unsigned)ceil_div(max_chunks, waves_per_block);
}

constexpr int MC_TOP = 2048;  // cells of a level, up to which one workgroup takes it

// mass, centre of mass and radius of every cell from the sorted bodies
void cell_moments(Ctx& c, bool with_radius) {
  hipStream_t s = c.stream;
  int nc = (int)c.ncell, nsys = c.nsys;
  long long* tot = (long long*)c.counters.p;
  ensure(c.ws, c.c_mass, nc);
  ensure(c.ws, c.c_sx, nc);
  ensure(c.ws, c.c_sy, nc);
  ensure(c.ws, c.c_sz, nc);
  ensure(c.ws, c.c_cx, nc);
  ensure(c.ws, c.c_cy, nc);
  ensure(c.ws, c.c_cz, nc);
  ensure(c.ws, c.c_rad, nc);
  ensure(c.ws, c.c_rad2bits, nc);
  MomentView v{c.c_begin.p, c.c_child0.p, c.c_nchild.p, c.c_level.p, c.key[0].p, c.rootbox.p, c.sys_off.p, nsys,
               c.c_mass.p, c.c_sx.p, c.c_sy.p, c.c_sz.p, c.c_cx.p, c.c_cy.p, c.c_cz.p};
  hipLaunchKernelGGL(k_leaf_moments, grid1(c.nleaf, 64), dim3(64), 0, s, (int)c.nleaf, c.leaves.p, c.c_end.p, v,
                     c.pm.p);
  LevelIds ids{};
  for (int l = 0; l <= c.depth; l++) ids.first[l] = c.lvl_first[l];
  for (int level = c.depth - 1; level >= 0;) {
    int to = level;
    if (c.lvl_count[level] <= MC_TOP) {
      while (to > 0 && c.lvl_count[to - 1] <= MC_TOP) to--;
      hipLaunchKernelGGL(k_cell_sums_run, dim3(1), dim3(1024), 0, s, level, to, ids, v);
    } else {
      hipLaunchKernelGGL(k_cell_sums, grid1(c.lvl_count[level], 64), dim3(64), 0, s, c.lvl_first[level],
                         c.lvl_count[level], v);
    }
    level = to - 1;
  }
  HIPCHK(hipGetLastError());
  if (!with_radius) return;
  // radii
  ensure(c.ws, c.c_split, (size_t)nc + 64);
  ensure(c.ws, c.cell_choff, (size_t)nc + 64);
  int* nchunk = c.c_split.p;
  int* choff = c.cell_choff.p;
  long long* nchunks = (long long*)(c.counters.p + 4);
  hipLaunchKernelGGL(k_rad_chunks, grid1(nc), dim3(256), 0, s, c.c_begin.p, c.c_end.p, nc, nchunk);
  exclusive_scan(c, nchunk, choff, nc, nchunks);
  zero_fill(c, c.c_rad2bits.p, sizeof(unsigned long long) * nc);
  hipLaunchKernelGGL(k_radius, dim3(cell_chunk_blocks(c, RAD_T / 64)), dim3(RAD_T), 0, s, c.c_begin.p,
                     c.c_end.p, choff, nchunks, nc, c.sx.p, c.sy.p, c.sz.p, c.c_cx.p, c.c_cy.p, c.c_cz.p,
                     c.c_rad2bits.p);
  ensure(c.ws, c.c_geo, (size_t)nc);
  hipLaunchKernelGGL(k_radius_final, grid1(nc), dim3(256), 0, s, c.c_rad2bits.p, nc, c.c_cx.p, c.c_cy.p,
                     c.c_cz.p, c.c_rad.p, c.c_geo.p);
}

// Positions and masses changed, tree topology, order and lists kept: the
// sorted bodies, cell masses and centres are recomputed from the stored
// order.  The radii are not (they serve the acceptance test, which is not
// rerun, and the FP32 scaling, for which any positive size works), so the
// sequence needs no host round trip.
void refresh_frozen(Ctx& c, const double* pos, const double* mass) {
  hipLaunchKernelGGL(k_gather, grid1(c.n), dim3(256), 0, c.stream, pos, mass, c.idx[0].p, c.n, c.sx.p,
                     c.sy.p, c.sz.p, c.pm.p);
  HIPCHK(hipGetLastError());
  cell_moments(c, false);
}

void build_tree(Ctx& c, int64_t n, const double* pos, const double* mass) {
  hipStream_t s = c.stream;
  c.n = n;
  int nsys = c.nsys;
  for (int k = 0; k < 2; k++) {
    ensure(c.ws, c.key[k], n);
    ensure(c.ws, c.idx[k], n);
  }
  ensure(c.ws, c.sx, n);
  ensure(c.ws, c.sy, n);
  ensure(c.ws, c.sz, n);
  ensure(c.ws, c.leaf_of, n);
  ensure(c.ws, c.rootbox, (size_t)8 * nsys);
  {
    int* before = c.sys_off.p;
    ensure(c.ws, c.sys_off, (size_t)nsys + 1);
    if (c.sys_off.p != before) c.sys_off_uploaded.clear();
  }
  {
    // the device copy is reused while the split is unchanged (no host
    // allocation while it is: the comparison runs over the stored vectors)
    if (c.h_sys_off.empty()) c.h_sys_off.assign({0, n});
    bool same = c.sys_off_uploaded.size() == c.h_sys_off.size();
    for (size_t k = 0; same && k < c.h_sys_off.size(); k++) same = c.sys_off_uploaded[k] == (int)c.h_sys_off[k];
    if (!same) {
      c.sys_off_uploaded.assign(c.h_sys_off.begin(), c.h_sys_off.end());
      HIPCHK(hipMemcpyAsync(c.sys_off.p, c.sys_off_uploaded.data(), c.sys_off_uploaded.size() * sizeof(int),
                            hipMemcpyHostToDevice, s));
      HIPCHK(hipStreamSynchronize(s));
    }
  }
  ensure(c.ws, c.pm, n);
  if (nsys == 1 && n <= TS_MAX) {
    if (c.have_events) HIPCHK(hipEventRecord(c.ev[15], s));
    hipLaunchKernelGGL(k_tree_small, dim3(1), dim3(BS_T), 0, s, pos, mass, (int)n, c.rootbox.p, c.key[0].p,
                       c.idx[0].p, c.sx.p, c.sy.p, c.sz.p, c.pm.p);
    HIPCHK(hipGetLastError());
    if (c.have_events) {
      HIPCHK(hipEventRecord(c.ev[16], s));
      HIPCHK(hipEventRecord(c.ev[17], s));
    }
  } else {
    if (nsys == 1) {
      int nbb = (int)std::min<int64_t>(1024, ceil_div(n, BB_T));
      ensure(c.ws, c.bbox_part, (size_t)6 * nbb);
      hipLaunchKernelGGL(k_bbox_partial, dim3(nbb), dim3(BB_T), 0, s, pos, n, c.bbox_part.p);
      hipLaunchKernelGGL(k_bbox_final, dim3(1), dim3(BB_T), 0, s, c.bbox_part.p, nbb, c.rootbox.p);
    } else {
      hipLaunchKernelGGL(k_bbox_sys, dim3(nsys), dim3(BB_T), 0, s, pos, c.sys_off.p, c.rootbox.p);
    }
    hipLaunchKernelGGL(k_keys, grid1(n), dim3(256), 0, s, pos, n, c.rootbox.p, c.sys_off.p, nsys,
                       c.key[0].p, c.idx[0].p);
    HIPCHK(hipGetLastError());
    if (c.have_events) HIPCHK(hipEventRecord(c.ev[15], s));
    radix_sort_keys(c, n, 64);
    if (nsys > 1) {
      // stable pass over the system id: (system, key, caller index) order
      for (int k = 0; k < 2; k++) {
        ensure(c.ws, c.skey[k], n);
        ensure(c.ws, c.spos[k], n);
      }
      hipLaunchKernelGGL(k_sys_keys, grid1(n), dim3(256), 0, s, c.idx[0].p, n, c.sys_off.p, nsys,
                         c.skey[0].p, c.spos[0].p);
      int bits = 1;
      while ((1 << bits) < nsys) bits++;
      int r = radix_sort(c, c.skey[0].p, c.spos[0].p, c.skey[1].p, c.spos[1].p, n, bits);
      hipLaunchKernelGGL(k_apply_pos, grid1(n), dim3(256), 0, s, c.spos[r].p, n, c.key[0].p, c.idx[0].p,
                         c.key[1].p, c.idx[1].p);
      HIPCHK(hipGetLastError());
      std::swap(c.key[0], c.key[1]);
      std::swap(c.idx[0], c.idx[1]);
    }
    if (c.have_events) HIPCHK(hipEventRecord(c.ev[16], s));
    hipLaunchKernelGGL(k_gather, grid1(n), dim3(256), 0, s, pos, mass, c.idx[0].p, n, c.sx.p, c.sy.p,
                       c.sz.p, c.pm.p);
    HIPCHK(hipGetLastError());
    if (c.have_events) HIPCHK(hipEventRecord(c.ev[17], s));
  }

  // the cells (see k_cell_levels); more of them than the arrays hold: larger
  // arrays, and the cells written again
  size_t cap = (size_t)std::max<int64_t>(1024, 4 * n / std::max(1, c.prm.n_leaf) + 64 + 2 * nsys);
  if (c.c_level.epoch == c.ws.epoch) cap = std::max(cap, c.c_level.cap);
  ensure(c.ws, c.counters, COUNTERS);  // the full size at once: counters[4..5] must outlive this call
  int nb = (int)ceil_div(n, CT_TILE);
  ensure(c.ws, c.sort_hist, (size_t)CT_ROWS * nb * 2 + CT_ROWS + 64);
  int* cnt = c.sort_hist.p;
  int* offs = cnt + (size_t)CT_ROWS * nb;
  int* rowtot = offs + (size_t)CT_ROWS * nb;
  ensure(c.ws, c.lev, (size_t)n);
  int* h = (int*)c.hbuf;  // read-back: cells of each level, then leaves of each level
  int64_t ncell = 0, nleaf = 0;
  for (int attempt = 0;; attempt++) {
    for (auto* b : {&c.c_level, &c.c_begin, &c.c_end, &c.c_parent, &c.c_child0, &c.c_nchild, &c.leaves})
      ensure(c.ws, *b, cap);
    int icap = (int)std::min(cap, (size_t)INT_MAX / 16);
    hipLaunchKernelGGL(k_cell_levels, dim3(nb), dim3(CT_T), 0, s, (int)n, c.prm.n_leaf, c.key[0].p, c.sys_off.p,
                       nsys, c.lev.p, cnt, nb, c.c_nchild.p, icap);
    hipLaunchKernelGGL(k_rs_rowscan, dim3(CT_ROWS), dim3(RS_T), 0, s, cnt, nb, offs, rowtot);
    hipLaunchKernelGGL(k_cell_emit, dim3(nb), dim3(CT_T), 0, s, (int)n, c.lev.p, offs, rowtot, nb, icap,
                       c.c_level.p, c.c_begin.p, c.c_end.p, c.c_parent.p, c.c_child0.p, c.c_nchild.p, c.leaf_of.p,
                       c.leaves.p);
    HIPCHK(hipGetLastError());
    HIPCHK(hipMemcpyAsync(h, rowtot, CT_ROWS * sizeof(int), hipMemcpyDeviceToHost, s));
    HIPCHK(hipStreamSynchronize(s));
    ncell = nleaf = 0;
    for (int l = 0; l < CT_LEVELS; l++) {
      ncell += h[l];
      nleaf += h[CT_LEVELS + l];
    }
    if (ncell <= icap) break;
    if (attempt > 0 || ncell > INT_MAX / 16) throw hip_error{hipErrorUnknown, "too many cells"};
    cap = (size_t)ncell;
  }
  c.lvl_first.clear();
  c.lvl_count.clear();
  int first = 0;
  for (int l = 0; l < CT_LEVELS && h[l] > 0; l++) {
    c.lvl_first.push_back(first);
    c.lvl_count.push_back(h[l]);
    first += h[l];
  }
  c.ncell = ncell;
  c.depth = (int)c.lvl_first.size() - 1;
  c.nleaf = nleaf;
  cell_moments(c, true);
  HIPCHK(hipGetLastError());
}

}  // namespace fmm
