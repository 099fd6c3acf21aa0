// Dual-tree walks on gfx950 (section 2.1 "Dual-tree Walk", section 2.3).
//
// Both walks expand a frontier of cell pairs level-synchronously from
// (root, root).  A pair (A, A) with A a leaf is a near-field self pair; an
// internal A yields its child pairs (c_i, c_j), i <= j.  A pair A != B is
// accepted (both directed pairs recorded), or, if both are leaves, recorded as
// a near-field leaf pair in both directions, or split: B when A is a leaf or
// when B is larger and not a leaf, A otherwise (ties split A).
//   * estimate walk: accept iff (r_A + r_B) < theta_est r (the "theta < 1"
//     estimate of the scalar force, section 2.3);
//   * main walk: the error-controlled mutual criterion
//     theta < 1 and E_{A->B} M_A / r^2 < eps f_B and E_{B->A} M_B / r^2 < eps f_A
//     (section 2.3), with E from the per-order norms P_k.
// Emission order inside a step is not fixed (wave-aggregated atomics); the
// recorded pair SETS are, and every list is afterwards grouped by sink and
// sorted by source, so all consumers see a deterministic order.
#include <hip/hip_runtime.h>

#include <functional>

#include <algorithm>
#include <climits>

#include "fmm_device.h"
#include "fmm_tables.h"

namespace fmm {


struct CellView {
  const int *nch, *c0;
  const double4* geo;  // (centre x, y, z, radius) per cell, one 32-byte record
  const double *mass, *pkb, *fmin;
  int p;
  double theta, err_tol;
  int geometric;
};

__device__ __forceinline__ double com_r2(const double4& a, const double4& b) {
  double dx = b.x - a.x;
  double dy = b.y - a.y;
  double dz = b.z - a.z;
  return (dx * dx + dy * dy) + dz * dz;
}

// E_{A->B} M_A / r^2 with M_A cancelled; sums in the order the definition
// lists (k ascending), each term (C(p,k) P_{k,A}) r_B^{p-k}, with C(p,k) P_{k,A}
// formed once per cell by the upward pass.  P = 0: the order is the run-time
// v.p (orders without an unrolled instance), with the same operations in the
// same order.
template <int P>
__device__ double mac_lhs(const CellView& v, int A, double rA, double rB, double r, double r2) {
  constexpr int PM = P > 0 ? P : FMM_TABLE_PMAX;
  const int p = P > 0 ? P : v.p;
  double rp = r;
#pragma unroll
  for (int i = 2; i <= PM; i++)
    if (i <= p) rp = rp * r;
  double mx = rA > rB ? rA : rB;
  double pref = (8.0 * mx) / (rA + rB);
  double pw[PM + 1];
  pw[0] = 1.0;
  double powB = 1.0;
#pragma unroll
  for (int j = 1; j <= PM; j++) {
    powB = powB * rB;
    pw[j] = powB;
  }
  const double* PA = v.pkb + (size_t)A * (p + 1);
  double SA = 0.0;
#pragma unroll
  for (int k = 0; k <= PM; k++)
    if (k <= p) SA = SA + PA[k] * pw[p - k];
  return (pref * (SA / rp)) / r2;
}

template <int KIND, int P>
__device__ bool accept(const CellView& v, int A, int B, const double4& gA, const double4& gB) {
  double r2 = com_r2(gA, gB);
  double r = sqrt(r2);
  double rA = gA.w, rB = gB.w;
  if constexpr (KIND == 0) {
    return (rA + rB) < v.theta * r;
  } else {
    if (!((rA + rB) < v.theta * r)) return false;
    if (v.geometric) return true;
    if (rA + rB == 0.0) return true;
    double lab = mac_lhs<P>(v, A, rA, rB, r, r2);
    double lba = mac_lhs<P>(v, B, rB, rA, r, r2);
    return (lab < v.err_tol * v.fmin[B]) && (lba < v.err_tol * v.fmin[A]);
  }
}

__device__ __forceinline__ int wave_incl_scan(int x) {
  int lane = lane_id();
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    int y = __shfl_up(x, o, 64);
    if (lane >= o) x += y;
  }
  return x;
}

constexpr int WALK_T = 512;  // threads per workgroup of the walk kernels

// One workgroup-aggregated allocation of `cnt` slots from the 64-bit counter
// *ctr: a wave scan, the wave totals combined through LDS, one atomic per
// workgroup.
__device__ __forceinline__ long long block_alloc(int cnt, unsigned long long* ctr, int& excl, int* sh,
                                                 long long* shb) {
  int incl = wave_incl_scan(cnt);
  int wv = threadIdx.x >> 6;
  if (lane_id() == 63) sh[wv] = incl;
  __syncthreads();
  if (threadIdx.x == 0) {
    int run = 0;
    for (int w = 0; w < WALK_T / 64; w++) {
      int t = sh[w];
      sh[w] = run;
      run += t;
    }
    *shb = run > 0 ? (long long)atomicAdd(ctr, (unsigned long long)run) : 0;
  }
  __syncthreads();
  excl = incl - cnt + sh[wv];
  long long base = *shb;
  __syncthreads();
  return base;
}

// Device counters of a walk (64-bit, each on its own cache line, at the int
// offsets below): three rotating frontier sizes, the totals of accepted and
// near-field entries, and the largest frontier seen.  Step k reads its
// frontier size from slot k % 3, appends to slot (k+1) % 3 and clears slot
// (k+2) % 3 for the step after, so consecutive steps need no host round trip.
// 64-bit totals cannot wrap; the host rejects lists longer than the int32
// CSR arrays can index (walk_list_fits).
constexpr int WC_FRONT = 0, WC_ACC = 96, WC_NEAR = 128, WC_MAXF = 160, WC_INTS = 192;
constexpr int WALK_BLOCKS = 1024;  // persistent grid; blocks stride over the frontier

__device__ __forceinline__ unsigned long long* wc64(int* ctr, int off) {
  return reinterpret_cast<unsigned long long*>(ctr + off);
}

template <int KIND, int P>
__global__ void __launch_bounds__(WALK_T) k_walk(CellView v, int step, const int2* fin, int fin_cap,
                                              int2* fout, long long fcap, int* ctr, uint64_t* acc_list,
                                              long long acap, uint64_t* near_list, long long ncap,
                                              int bits) {
  long long nin_all = (long long)*wc64(ctr, WC_FRONT + 32 * (step % 3));
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    *wc64(ctr, WC_FRONT + 32 * ((step + 2) % 3)) = 0ull;
    atomicMax(wc64(ctr, WC_MAXF), (unsigned long long)nin_all);
  }
  int nin = (int)min(nin_all, (long long)fin_cap);  // an overflowed frontier is redone by the host
  unsigned long long* fctr = wc64(ctr, WC_FRONT + 32 * ((step + 1) % 3));
  __shared__ int sh[WALK_T / 64];
  __shared__ long long shb;
  for (int base = blockIdx.x * WALK_T; base < nin; base += gridDim.x * WALK_T) {
    int t = base + threadIdx.x;
    bool live = t < nin;
    int A = 0, B = 0, nkids = 0, nacc = 0, nnear = 0, mode = 0;
    // mode: 0 none, 1 self children, 2 split A, 3 split B
    if (live) {
      int2 pr = fin[t];
      A = pr.x;
      B = pr.y;
      int kA = v.nch[A], kB = v.nch[B];
      if (A == B) {
        if (kA == 0) {
          nnear = 1;
        } else {
          mode = 1;
          nkids = kA * (kA + 1) / 2;
        }
      } else {
        double4 gA = v.geo[A], gB = v.geo[B];
        if (accept<KIND, P>(v, A, B, gA, gB)) {
          nacc = 2;
        } else if (kA == 0 && kB == 0) {
          nnear = 2;
        } else {
          bool splitB = (kA == 0) || (gB.w > gA.w && kB != 0);
          mode = splitB ? 3 : 2;
          nkids = splitB ? kB : kA;
        }
      }
    }
    int ek, ea, en;
    long long bk = block_alloc(nkids, fctr, ek, sh, &shb);
    long long ba = block_alloc(nacc, wc64(ctr, WC_ACC), ea, sh, &shb);
    long long bn = block_alloc(nnear, wc64(ctr, WC_NEAR), en, sh, &shb);
    if (!live) continue;
    long long o = bk + ek;
    if (mode == 1) {
      int c0 = v.c0[A], k = v.nch[A];
      for (int i = 0; i < k; i++)
        for (int j = i; j < k; j++, o++)
          if (o < fcap) fout[o] = make_int2(c0 + i, c0 + j);
    } else if (mode == 2) {
      int c0 = v.c0[A];
      for (int i = 0; i < nkids; i++, o++)
        if (o < fcap) fout[o] = make_int2(c0 + i, B);
    } else if (mode == 3) {
      int c0 = v.c0[B];
      for (int j = 0; j < nkids; j++, o++)
        if (o < fcap) fout[o] = make_int2(A, c0 + j);
    }
    // list entries: (sink << bits) | source
    uint64_t kab = ((uint64_t)B << bits) | (uint64_t)A, kba = ((uint64_t)A << bits) | (uint64_t)B;
    if (nacc) {
      long long q = ba + ea;
      if (q + 1 < acap) {
        acc_list[q] = kab;
        acc_list[q + 1] = kba;
      }
    }
    if (nnear) {
      long long q = bn + en;
      if (nnear == 1) {
        if (q < ncap) near_list[q] = kab;
      } else if (q + 1 < ncap) {
        near_list[q] = kab;
        near_list[q + 1] = kba;
      }
    }
  }
}

// the walks start from (root, root) of every system; counters cleared
__global__ void k_seed(int2* f, int nsys, int* ctr) {
  int s = blockIdx.x * blockDim.x + threadIdx.x;
  if (s < nsys) f[s] = make_int2(s, s);
  if (s < WC_INTS) ctr[s] = s == WC_FRONT ? nsys : 0;  // low half of the 64-bit frontier size
}

// ---- grouping by sink, sorted by source ----------------------------------
// The keys (sink << bits | source) are all different, so their order is given
// by their values and any sort will do.  In general they are radix-sorted; CSR
// offsets then come from a lower bound per sink and the sources are the low bits.
__global__ void k_csr_off(const uint64_t* keys, int64_t cnt, int nseg, int bits, int* off) {
  int s = blockIdx.x * blockDim.x + threadIdx.x;
  if (s > nseg) return;
  uint64_t t = (uint64_t)s << bits;
  int64_t lo = 0, hi = cnt;
  while (lo < hi) {
    int64_t mid = (lo + hi) >> 1;
    if (keys[mid] < t)
      lo = mid + 1;
    else
      hi = mid;
  }
  off[s] = (int)lo;
}

__global__ void k_extract_src(const uint64_t* keys, int64_t cnt, uint64_t mask, int* src) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < cnt) src[i] = (int)(keys[i] & mask);
}

// off[from .. to] = at of each valid lane, whole wavefronts: the sinks without
// entries between two of a list.  Long runs (a batch of many small systems has
// lists of few entries for 65536 sinks, and a lane alone takes 1.7 ms for
// those) are written by all lanes.
__device__ __forceinline__ void fill_offsets(bool valid, int from, int to, int at, int* __restrict__ off, int lane) {
  bool apart = valid && to - from >= WAVE;
  if (valid && !apart)
    for (int t = from; t <= to; t++) off[t] = at;
  for (uint64_t todo = ballot(apart); todo; todo &= todo - 1) {
    int l = __builtin_ctzll(todo);
    int f = __builtin_amdgcn_readlane(from, l), e = __builtin_amdgcn_readlane(to, l);
    int v = __builtin_amdgcn_readlane(at, l);
    for (int t = f + lane; t <= e; t += WAVE) off[t] = v;
  }
}

// A list of up to GS_MAX entries of 32-bit keys by one workgroup: sort, sources
// and offsets in one launch instead of three per pass and two (a launch costs
// some 5 us whatever its size).
constexpr int GS_I = 20;
constexpr int GS_MAX = BS_T * GS_I;

__global__ void __launch_bounds__(BS_T) k_group_small(const uint64_t* __restrict__ raw, int cnt, int nseg, int bits,
                                                      int* __restrict__ src, int* __restrict__ off) {
  __shared__ BlockSort<uint32_t, GS_I, false> bs;
  int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  int C = (cnt + BS_T - 1) / BS_T;
  uint32_t k[GS_I];
  int v[GS_I];
#pragma unroll
  for (int c = 0; c < GS_I; c++) {
    int i = (w * C + c) * 64 + lane;
    k[c] = c < C && i < cnt ? (uint32_t)raw[i] : 0xffffffffu;
  }
  block_sort(bs, k, v, C, 2 * bits);
  // (bs.sk holds the sorted keys) entry i starts the lists of the sinks after
  // the one before it, up to its own; the sinks after the last start at the end
  uint32_t mask = (1u << bits) - 1u;
  for (int base = 0; base <= cnt; base += BS_T) {
    int i = base + tid;
    int from = i > 0 && i <= cnt ? (int)(bs.sk[i - 1] >> bits) + 1 : 0;
    int to = nseg;
    if (i < cnt) {
      uint32_t q = bs.sk[i];
      src[i] = (int)(q & mask);
      to = (int)(q >> bits);
    }
    fill_offsets(i <= cnt, from, to, i, off, lane);
  }
}

// The entries of part f = blockIdx.x of a list split by its keys' top bits (the
// sinks [f << sb, (f + 1) << sb) of the ncell), sorted in LDS: sources and offsets.
// The starts of the parts are fstart, or the prefix of the 256 sizes rowtot.  A
// part that does not fit (T I entries) is sorted by the same workgroup in global
// memory, between x and y.
template <int T, int I>
__global__ void __launch_bounds__(T) k_group_parts(uint32_t* x, uint32_t* y, const int* __restrict__ rowtot,
                                                   const int* __restrict__ fstart, int ncell, int sb, int bits,
                                                   int* __restrict__ src, int* __restrict__ off) {
  __shared__ BlockSort<uint32_t, I, false, T> bs;
  int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, f = blockIdx.x;
  int s0, s1;
  if (fstart) {
    s0 = fstart[f];
    s1 = fstart[f + 1];
  } else {  // (one size per thread: the sum of those before f)
    int sz = tid < 256 ? rowtot[tid] : 0;
    int before = tid < f ? sz : 0;
    if (tid < 256) {
      for (int o = 32; o > 0; o >>= 1) before += __shfl_xor(before, o, 64);
      if (lane == 0) bs.wsum[w] = before;
      if (tid == f) bs.dstart[0] = sz;
    }
    __syncthreads();
    s0 = bs.wsum[0] + bs.wsum[1] + bs.wsum[2] + bs.wsum[3];
    s1 = s0 + bs.dstart[0];
    __syncthreads();
  }
  int n = s1 - s0;
  int lo = f << sb, hi = min((f + 1) << sb, ncell);  // this part's sinks
  if (f == (int)gridDim.x - 1 && tid == 0) off[ncell] = s1;
  int nbits = sb + bits;  // the rest of the key
  uint32_t mask = (1u << bits) - 1u;
  // entry i starts the lists of the sinks after the one before it, up to its
  // own; the sinks after the last start at the end
  auto emit = [&](const uint32_t* keys) {
    for (int base = 0; base <= n; base += T) {
      int i = base + tid;
      int from = i > 0 && i <= n ? (int)(keys[i - 1] >> bits) + 1 : 0;
      int to = hi - lo - 1;
      if (i < n) {
        uint32_t q = keys[i];
        src[s0 + i] = (int)(q & mask);
        to = (int)(q >> bits);
      }
      fill_offsets(i <= n, from, to, s0 + i, off + lo, lane);
    }
  };
  uint32_t low = nbits < 32 ? (1u << nbits) - 1u : ~0u;
  if (n <= T * I) {
    int C = (n + T - 1) / T;
    uint32_t k[I];
    int v[I];
#pragma unroll
    for (int c = 0; c < I; c++) {
      int i = (w * C + c) * 64 + lane;
      k[c] = c < C && i < n ? x[s0 + i] & low : low;
    }
    block_sort(bs, k, v, C, nbits);
    emit(bs.sk);
  } else {
    uint32_t *in = x + s0, *out = y + s0;
    uint64_t lt = lanemask_lt();
    for (int shift = 0; shift < nbits; shift += 8) {
      if (tid < 256) bs.dstart[tid] = 0;
      __syncthreads();
      for (int i = tid; i < n; i += T) atomicAdd(&bs.dstart[(in[i] & low) >> shift & 255], 1);
      __syncthreads();
      int tot = tid < 256 ? bs.dstart[tid] : 0, incl = tot;
      if (tid < 256) {
        for (int o = 1; o < 64; o <<= 1) {
          int up = __shfl_up(incl, o, 64);
          if (lane >= o) incl += up;
        }
        if (lane == 63) bs.wsum[w] = incl;
      }
      __syncthreads();
      if (tid < 256) {
        for (int ww = 0; ww < w; ww++) incl += bs.wsum[ww];
        bs.dstart[tid] = incl - tot;  // the digit's next place
      }
      for (int base = 0; base < n; base += T) {
        for (int t = tid; t < T / 64 * 256; t += T) (&bs.wcnt[0][0])[t] = 0;
        __syncthreads();
        bool valid = base + tid < n;
        uint32_t key = valid ? in[base + tid] & low : 0u;
        int d = (int)(key >> shift & 255);
        uint64_t peers = ballot(valid);
        for (int b = 0; b < 8; b++) {
          bool bit = (d >> b) & 1;
          uint64_t bb = ballot(bit);
          peers &= bit ? bb : ~bb;
        }
        if (valid && (peers >> lane) == 1ull) bs.wcnt[w][d] = __popcll(peers);
        __syncthreads();
        if (tid < 256) {
          int run = bs.dstart[tid];
          for (int ww = 0; ww < T / 64; ww++) {
            int t = bs.wcnt[ww][tid];
            bs.wcnt[ww][tid] = run;
            run += t;
          }
          bs.dstart[tid] = run;
        }
        __syncthreads();
        if (valid) out[bs.wcnt[w][d] + __popcll(peers & lt)] = key;
        __syncthreads();
      }
      uint32_t* t = in;
      in = out;
      out = t;
    }
    emit(in);
  }
}

static int list_bits(int64_t ncell) {
  int b = 1;
  while (((int64_t)1 << b) < ncell) b++;
  return b;
}

// One workgroup sorts a short list.  Otherwise the list is split by the sink's
// top bits, moved once or twice (the first time as 32-bit keys), and the parts are
// sorted in LDS: 3 + 3 + 1 launches and 40 bytes per entry at the most, in place of
// an LSD sort's 3 per 8 bits of the key and two, and 24 bytes per 8 bits.  Once
// where the 256 parts hold up to GP_ONCE entries on average; else up to 256 times 256
// parts of up to GP_TWICE.
// More than 2^20 cells (keys over 40 bits): the LSD sort.  Against it everywhere:
// 256 systems of 1032 to 65006 bodies (mean 15512) 41.4 -> 38.3 ms (the sorts
// 7.0 -> 3.9), 2^22 bodies 31.4 -> 29.4, 30011 1.37 -> 1.27.  GP_ONCE 4096 and 16384 time alike; GP_TWICE 640
// costs 2^20 bodies 0.1 ms, 3000 2^18 in FP64 0.05.
constexpr int64_t GP_ONCE = 8192, GP_TWICE = 1536;

static void group_by_sink(Ctx& c, CellList& L) {
  hipStream_t s = c.stream;
  int nc = (int)c.ncell;
  int bits = list_bits(c.ncell);
  ensure(c.ws, L.off, (size_t)nc + 1);
  ensure(c.ws, L.src, (size_t)std::max<int64_t>(L.count, 1));
  if (L.count == 0) {  // (a batch of systems of one cell each, say)
    zero_fill(c, L.off.p, ((size_t)nc + 1) * sizeof(int));
  } else if (2 * bits <= 32 && L.count <= GS_MAX) {
    hipLaunchKernelGGL(k_group_small, dim3(1), dim3(BS_T), 0, s, L.raw.p, (int)L.count, nc, bits, L.src.p, L.off.p);
  } else if (bits <= 20) {
    int fb = std::min(8, bits);
    // entries per part on average with the top b bits (parts past the cells are empty)
    auto mean = [&](int b) { return L.count / std::max<int64_t>(1, (int64_t)nc >> (bits - b)); };
    bool twice = mean(fb) > GP_ONCE && bits > 8;
    int sub = 1;
    if (twice)
      while (fb < std::min(16, bits) && (fb == 8 || mean(fb) > GP_TWICE)) {
        fb++;
        sub *= 2;
      }
    int sb = bits - fb;
    ensure(c.ws, L.tmp, (size_t)(L.count / 2 + 1));
    if (twice) ensure(c.ws, c.sort_hist, radix_split2_ints(L.count, sub));
    uint32_t *x = (uint32_t*)L.tmp.p, *y = (uint32_t*)L.raw.p;
    const int* fstart = nullptr;
    const int* rowtot = radix_split(c, L.raw.p, x, L.count, 2 * bits - std::min(8, bits));
    unsigned grid = (unsigned)ceil_div(nc, (int64_t)1 << sb);
    if (twice) {
      fstart = radix_split2(c, x, y, L.count, 2 * bits - fb, sub, rowtot);
      hipLaunchKernelGGL((k_group_parts<256, 16>), dim3(grid), dim3(256), 0, s, y, x, rowtot, fstart, nc, sb, bits,
                         L.src.p, L.off.p);
    } else {
      hipLaunchKernelGGL((k_group_parts<BS_T, GS_I>), dim3(grid), dim3(BS_T), 0, s, x, y, rowtot, fstart, nc, sb, bits,
                         L.src.p, L.off.p);
    }
  } else {
    ensure(c.ws, L.tmp, (size_t)L.count);
    int r = radix_sort(c, L.raw.p, nullptr, L.tmp.p, nullptr, L.count, 2 * bits);
    const uint64_t* sorted = r == 0 ? L.raw.p : L.tmp.p;
    hipLaunchKernelGGL(k_extract_src, dim3((unsigned)ceil_div(L.count, 256)), dim3(256), 0, s, sorted, L.count,
                       ((uint64_t)1 << bits) - 1, L.src.p);
    hipLaunchKernelGGL(k_csr_off, dim3((unsigned)ceil_div(nc + 1, 256)), dim3(256), 0, s, sorted, L.count, nc, bits,
                       L.off.p);
  }
  HIPCHK(hipGetLastError());
}

// beside: host work (launches on other streams) done once, right after the
// first batch of walk steps is enqueued and before the host waits for them
template <int KIND, int P>
static void run_walk(Ctx& c, CellList& acc, CellList& nearl, bool group,
                     const std::function<void()>& beside = {}) {
  hipStream_t s = c.stream;
  CellView v{};
  v.nch = c.c_nchild.p;
  v.c0 = c.c_child0.p;
  v.geo = c.c_geo.p;
  v.mass = c.c_mass.p;
  v.pkb = c.pkb.p;
  v.fmin = c.fmin.p;
  v.p = c.p;
  v.theta = KIND == 0 ? c.prm.theta_est : c.prm.theta;
  v.err_tol = c.err_tol;
  v.geometric = c.prm.mac == FMM_MAC_GEOMETRIC;
  size_t fcap0 = std::max<size_t>(4096, (size_t)c.ncell * 4);
  ensure(c.ws, c.front[0], fcap0);
  ensure(c.ws, c.front[1], fcap0);
  ensure(c.ws, acc.raw, (size_t)c.ncell * 8 + 64);  // (kept as large as earlier calls left it)
  ensure(c.ws, nearl.raw, (size_t)c.ncell * 8 + 64);
  ensure(c.ws, c.counters, COUNTERS);
  int* ctr = c.counters.p + 256;
  int bits = list_bits(c.ncell);
  long long* h = c.hbuf;  // the counters, read back as 64-bit values
  auto H = [&](int off) { return h[off / 2]; };
  // A pair's step count is at most the sum of its cells' levels plus one, so
  // 2 depth + 2 steps drain the frontier; the host checks once at the end.
  int steps = 2 * c.depth + 2;
  long long nacc = 0, nnear = 0;
  auto fcap_of = [&](const dbuf<int2>& f) { return (int)std::min<size_t>(f.cap, (size_t)INT_MAX); };
  for (int attempt = 0;; attempt++) {
    int sblocks = (int)ceil_div(std::max(c.nsys, WC_INTS), 256);
    hipLaunchKernelGGL(k_seed, dim3((unsigned)sblocks), dim3(256), 0, s, c.front[0].p, c.nsys, ctr);
    int step = 0;
    bool done = false;
    while (!done) {
      for (int e = 0; e < steps; e++, step++)
        hipLaunchKernelGGL((k_walk<KIND, P>), dim3(WALK_BLOCKS), dim3(WALK_T), 0, s, v, step,
                           c.front[step & 1].p, fcap_of(c.front[step & 1]), c.front[1 - (step & 1)].p,
                           (long long)fcap_of(c.front[1 - (step & 1)]), ctr, acc.raw.p,
                           (long long)acc.raw.cap, nearl.raw.p, (long long)nearl.raw.cap, bits);
      HIPCHK(hipGetLastError());
      if (beside && attempt == 0 && step == steps) beside();
      HIPCHK(hipMemcpyAsync(h, ctr, WC_INTS * sizeof(int), hipMemcpyDeviceToHost, s));
      HIPCHK(hipStreamSynchronize(s));
      done = H(WC_FRONT + 32 * (step % 3)) == 0;  // frontier of the next step is empty
      if (H(WC_MAXF) > std::min(fcap_of(c.front[0]), fcap_of(c.front[1]))) break;  // overflowed: redo
    }
    nacc = H(WC_ACC);
    nnear = H(WC_NEAR);
    long long need_f = H(WC_MAXF);
    if (!walk_list_fits(nacc) || !walk_list_fits(nnear) || !walk_list_fits(need_f))
      throw unsupported_error{"interaction list or walk frontier longer than 2^31 - 64 entries"};
    bool again = false;
    int64_t slack = c.ws.arena ? 1 : 2;  // twice the need, except in the fixed scratch
    if (need_f > std::min(fcap_of(c.front[0]), fcap_of(c.front[1]))) {
      ensure(c.ws, c.front[0], (size_t)need_f * 2);
      ensure(c.ws, c.front[1], (size_t)need_f * 2);
      again = true;
    }
    if ((size_t)nacc + 2 > acc.raw.cap) {
      ensure(c.ws, acc.raw, (size_t)(nacc * slack) + 64);
      again = true;
    }
    if ((size_t)nnear + 2 > nearl.raw.cap) {
      ensure(c.ws, nearl.raw, (size_t)(nnear * slack) + 64);
      again = true;
    }
    if (!again) break;
    if (attempt > 8) throw hip_error{hipErrorUnknown, "walk buffers did not converge"};
  }
  acc.count = nacc;
  nearl.count = nnear;
  if (group) {
    group_by_sink(c, acc);
    group_by_sink(c, nearl);
  }
}

// ---- scalar-force estimate -----------------------------------------------
// F_B = sum over accepted sources A (ascending) of M_A / r^2
__global__ void k_fcell(int ncell, const int* off, const int* src, const double* mass,
                        const double* cx, const double* cy, const double* cz, double* F) {
  int B = blockIdx.x * blockDim.x + threadIdx.x;
  if (B >= ncell) return;
  double f = 0.0;
  for (int k = off[B]; k < off[B + 1]; k++) {
    int A = src[k];
    double dx = cx[B] - cx[A], dy = cy[B] - cy[A], dz = cz[B] - cz[A];
    double r2 = (dx * dx + dy * dy) + dz * dz;
    f = f + mass[A] / r2;
  }
  F[B] = f;
}

// near_i = sum_{j near, j != i} m_j / d^2, partners in ascending id, bodies in
// sorted order, one running sum per body (k_fleaf adds the far part).  The sum
// of a body is one chain of additions in a fixed order, but its terms are
// independent, and the FP64 division is most of the work.  A body's own term
// has d2 = 0 and counts as +0.  The partners are read as 64-body chunks
// (BodyStream), the next one fetched while the current one is summed.

__device__ __forceinline__ double near_term(const double4& s, const double4& me, bool use) {
  double dx = s.x - me.x, dy = s.y - me.y, dz = s.z - me.z;
  double d2 = (dx * dx + dy * dy) + dz * dz;
  return use && d2 > 0.0 ? s.w / d2 : 0.0;
}

// Where the leaves fill the chip: one wavefront per sink leaf, the chunk in
// LDS, the n_B sink bodies replicated over G = 64 / n_B lane groups.  With
// G > 1 the groups form the terms of G partners side by side and pass them
// through LDS to the adds.  Bound by FP64 issue of the divisions; with one
// lane per sink body (45 of 64 lanes idle in a 19-body leaf) the kernel took
// 887 us at N = 2^20, p = 10 (635 us now) and 4.3 ms at N = 2^22 (2.6 ms).
constexpr int NF_WAVES = 4;
constexpr int NF_STEPS = 4;  // terms per lane formed before they are added

__global__ void __launch_bounds__(64 * NF_WAVES) k_near_f(int nleaves, const int* __restrict__ leaves,
                                                          const int* __restrict__ cb,
                                                          const int* __restrict__ ce,
                                                          const int* __restrict__ off,
                                                          const int* __restrict__ src,
                                                          const double4* __restrict__ pm, double* f) {
  __shared__ double4 sbuf[NF_WAVES][64];
  __shared__ double tbuf[NF_WAVES][64 * NF_STEPS];
  int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  int nblk = (nleaves + NF_WAVES - 1) / NF_WAVES;
  int blk = xcd_block();
  int li = blk * NF_WAVES + wv;
  if (blk >= nblk || li >= nleaves) return;
  int B = leaves[li];
  int b = cb[B], e = ce[B];
  int qb = off[B], qe = off[B + 1];
  for (int i0 = b; i0 < e; i0 += 64) {
    int nB = min(64, e - i0);
    int G = 64 / nB;
    int g = lane / nB, sl = lane - g * nB;
    bool act = g < G;
    double4 me = pm[i0 + sl];
    double near = 0.0;
    BodyStream st;
    st.start(src, cb, ce, qb, qe, lane);
    int j, na = st.next(lane, b, j);
    double4 cur = pm[j];
    while (na > 0) {
      __builtin_amdgcn_wave_barrier();
      sbuf[wv][lane] = cur;
      __builtin_amdgcn_wave_barrier();
      int nn = st.next(lane, b, j);
      cur = pm[j];
      __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0): the staged chunk is visible to the wave
      if (G == 1) {  // a lane per body: term and add side by side
        int tmax = act ? na : 0;
        for (int t = 0; t < tmax; t++) near = near + near_term(sbuf[wv][t], me, true);
      } else {
        for (int base = 0; base < na; base += NF_STEPS * G) {
          __builtin_amdgcn_wave_barrier();
#pragma unroll
          for (int u = 0; u < NF_STEPS; u++) {
            int t = base + u * G + g;
            if (act && base + u * G < na) tbuf[wv][u * G * nB + lane] = near_term(sbuf[wv][t & 63], me, t < na);
          }
          __builtin_amdgcn_wave_barrier();
          __builtin_amdgcn_s_waitcnt(0xc07f);  // the terms are visible to the wave
          int cnt = min(NF_STEPS * G, na - base);
          const double* tb = &tbuf[wv][sl];
          int k = 0;
          for (; k + 4 <= cnt; k += 4) {
            double t0 = tb[k * nB], t1 = tb[(k + 1) * nB], t2 = tb[(k + 2) * nB], t3 = tb[(k + 3) * nB];
            near = near + t0;
            near = near + t1;
            near = near + t2;
            near = near + t3;
          }
          for (; k < cnt; k++) near = near + tb[k * nB];
        }
      }
      na = nn;
    }
    if (g == 0) f[i0 + sl] = near;
    __builtin_amdgcn_wave_barrier();
  }
}

// Up to NF_FEW leaves the longest list is the kernel's length (in a 4096-body
// model a 64-body leaf of the outskirts has all 4096 bodies as partners): a
// workgroup of 16 wavefronts per leaf, each with four of its bodies at a time.
// A lane holds one partner of the chunk and forms its terms for the four
// bodies (wave-uniform); the terms go through LDS to a lane per body, which
// adds its 64 in order.  At 4096 bodies, p = 6 the near sums took 659 us with a
// wavefront per leaf and take 181 this way, at 1000 bodies 170 and 39, at 2737
// leaves (50021 bodies) 243 and 91; at 5358 leaves the two are equal (240), and
// where the leaves fill the chip the chains of adds lose (320 against 243 us at
// 14391 leaves).  So they do with large leaves (n_leaf = 400 and more at 2^20
// bodies of a cube, 4096 leaves: 10.1 against 7.1 ms): where the leaves have more
// than NF_LANES blocks of 64 bodies in all, a leaf of 64 and more takes a wavefront
// per block, a lane per body, as in k_near_f, unless its list is more than twice the
// mean (an outskirts leaf of a 2^20-body model has all bodies as partners, and is
// the kernel's length).
constexpr int NF_FEW = 4096;
constexpr int64_t NF_LANES = 8192;

// The terms of the lane's body (v; no body: mass 0) for sinks k .. k+3 of pm,
// written to t[0], t[65], t[130], t[195].  masses_safe: every mass of the chunk
// is 0 or div_safe; with the distances safe too the quotients come from
// div_scaled, the same bits as the operator's.
__device__ __forceinline__ void near_terms(const double4& v, const double4* __restrict__ sink, int last,
                                           bool masses_safe, double* t) {
  double d[4], m[4];
  bool safe = masses_safe;
#pragma unroll
  for (int u = 0; u < 4; u++) {
    double4 me = sink[min(u, last)];
    double dx = v.x - me.x, dy = v.y - me.y, dz = v.z - me.z;
    double d2 = (dx * dx + dy * dy) + dz * dz;
    bool ok = d2 > 0.0;  // (operands selected, not the quotient: no branch per term)
    m[u] = ok ? v.w : 0.0;
    d[u] = ok ? d2 : 1.0;
    safe = safe && div_safe(d[u]);
  }
  if (ballot(!safe) == 0) {
#pragma unroll
    for (int u = 0; u < 4; u++) t[65 * u] = div_scaled(m[u], d[u]);
  } else {
#pragma unroll
    for (int u = 0; u < 4; u++) t[65 * u] = m[u] / d[u];
  }
}

// adds the terms t[0 .. cnt) in order, cnt a multiple of 8; the next eight are
// read while eight are added
__device__ __forceinline__ double add_terms(double near, const double* t, int cnt) {
  double a[8];
#pragma unroll
  for (int u = 0; u < 8; u++) a[u] = t[u];
  for (int k = 8; k < cnt; k += 8) {
    double c[8];
#pragma unroll
    for (int u = 0; u < 8; u++) c[u] = t[k + u];
#pragma unroll
    for (int u = 0; u < 8; u++) near = near + a[u];
#pragma unroll
    for (int u = 0; u < 8; u++) a[u] = c[u];
  }
#pragma unroll
  for (int u = 0; u < 8; u++) near = near + a[u];
  return near;
}

__global__ void __launch_bounds__(1024) k_near_f_few(int nleaves, const int* __restrict__ leaves,
                                                     const int* __restrict__ cb, const int* __restrict__ ce,
                                                     const int* __restrict__ off, const int* __restrict__ src,
                                                     const double4* __restrict__ pm, int lane_entries,
                                                     double* __restrict__ f) {
  __shared__ __align__(32) double tbuf[16][4 * 65 + 4];
  int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  int li = xcd_block();
  if (li >= nleaves) return;
  int B = leaves[li];
  int b = cb[B], e = ce[B];
  int qb = off[B], qe = off[B + 1];
  double* tw = tbuf[wv];
  if (e - b >= 64 && qe - qb <= lane_entries) {
    double4* sb = (double4*)tw;  // the staged chunk
    for (int i0 = b + wv * 64; i0 < e; i0 += 1024) {
      double4 me = pm[min(i0 + lane, e - 1)];
      double near = 0.0;
      BodyStream st;
      st.start(src, cb, ce, qb, qe, lane);
      int j, na = st.next(lane, b, j);
      double4 cur = pm[j];
      while (na > 0) {
        __builtin_amdgcn_wave_barrier();
        sb[lane] = cur;
        __builtin_amdgcn_wave_barrier();
        int nn = st.next(lane, b, j);
        cur = pm[j];
        __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0): the staged chunk is visible to the wave
        for (int t = 0; t < na; t++) near = near + near_term(sb[t], me, true);
        na = nn;
      }
      if (i0 + lane < e) f[i0 + lane] = near;
      __builtin_amdgcn_wave_barrier();
    }
    return;
  }
  int mine = min(lane, 3) * 65;
  for (int i0 = b + wv * 4; i0 < e; i0 += 64) {
    int nB = min(4, e - i0);
    double near = 0.0;
    BodyStream st;
    st.start(src, cb, ce, qb, qe, lane);
    int j, na = st.next(lane, -1, j);
    double4 cur = make_double4(0.0, 0.0, 0.0, 0.0);  // no body: mass 0
    if (j >= 0) cur = pm[j];
    while (na > 0) {
      double4 v = cur;
      int nn = st.next(lane, -1, j);
      cur = make_double4(0.0, 0.0, 0.0, 0.0);
      if (j >= 0) cur = pm[j];
      bool msafe = ballot(!(v.w == 0.0 || div_safe(v.w))) == 0;
      near_terms(v, pm + i0, nB - 1, msafe, tw + lane);
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0): the terms are visible to the wave
      near = add_terms(near, tw + mine, (na + 7) & ~7);
      __builtin_amdgcn_wave_barrier();
      na = nn;
    }
    if (lane < nB) f[i0 + lane] = near;
  }
}

// f_i = (F summed from the root down to the leaf) + near_i, in that order, for
// the bodies of every leaf (f holds near_i on entry); one thread per leaf
__global__ void k_fleaf(int nleaves, const int* leaves, const int* cb, const int* ce, const int* parent,
                        const double* F, double* f) {
  int li = blockIdx.x * blockDim.x + threadIdx.x;
  if (li >= nleaves) return;
  int c = leaves[li];
  int path[FMM_MAX_LEVEL + 2];
  int len = 0;
  for (int q = c; q >= 0; q = parent[q]) path[len++] = q;
  double far = 0.0;
  for (int k = len - 1; k >= 0; k--) far = far + F[path[k]];
  for (int i = cb[c]; i < ce[c]; i++) f[i] = far + f[i];
}

// fmin_c = min of f over the cell's bodies (the same as the minimum over its
// children), a wavefront per chunk of CELL_CHUNK bodies; f >= 0, so the bit
// patterns order as the values and the chunks combine by an integer atomicMin
// (fmin starts at +inf)
constexpr int FM_T = 256;
__global__ void __launch_bounds__(FM_T) k_cell_min(const int* cb, const int* ce, const int* choff,
                                                   const long long* nchunks, int ncell, const double* f,
                                                   unsigned long long* fmin_bits) {
  int blk = blockIdx.x * (FM_T / 64) + (threadIdx.x >> 6);
  int lane = threadIdx.x & 63;
  if (blk >= (int)*nchunks) return;
  int lo = 0, hi = ncell - 1;  // cell owning this chunk: last c with choff[c] <= blk
  while (lo < hi) {
    int mid = (lo + hi + 1) >> 1;
    if (choff[mid] <= blk)
      lo = mid;
    else
      hi = mid - 1;
  }
  int c = lo;
  int64_t b = cb[c] + (int64_t)(blk - choff[c]) * CELL_CHUNK;
  int64_t e = b + CELL_CHUNK < ce[c] ? b + CELL_CHUNK : ce[c];
  double m = INFINITY;
  for (int64_t i = b + lane; i < e; i += 64) m = f[i] < m ? f[i] : m;
  for (int o = 32; o > 0; o >>= 1) {
    double other = __shfl_xor(m, o, 64);
    m = other < m ? other : m;
  }
  if (lane == 0) atomicMin(&fmin_bits[c], (unsigned long long)__double_as_longlong(m));
}

__global__ void k_fill_inf(unsigned long long* p, int n) {
  int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = 0x7ff0000000000000ull;
}

// The far sums F_B (list grouped on the second side stream, with the third
// set of sort scratch) run beside the near sums on the caller's stream; after
// the join the leaves add the two, then the cell minima are taken.
void estimate_walk(Ctx& c, const std::function<void()>& beside) {
  hipStream_t s = c.stream;
  int nc = (int)c.ncell;
  ensure(c.ws, c.fcell, nc);
  ensure(c.ws, c.fmin, nc);
  ensure(c.ws, c.fpart, (size_t)c.n);
  run_walk<0, 0>(c, c.est_far, c.est_near, false, beside);
  stream_wait(c.fork[6], s, c.side2);
  {
    OnStream on(c, c.side2);
    SideScratch alt(c, 3);
    group_by_sink(c, c.est_far);
    hipLaunchKernelGGL(k_fcell, dim3((nc + 255) / 256), dim3(256), 0, c.side2, nc, c.est_far.off.p,
                       c.est_far.src.p, c.c_mass.p, c.c_cx.p, c.c_cy.p, c.c_cz.p, c.fcell.p);
  }
  group_by_sink(c, c.est_near);
  if (c.nleaf <= NF_FEW)
    hipLaunchKernelGGL(k_near_f_few, dim3(xcd_grid(c.nleaf)), dim3(1024), 0, s, (int)c.nleaf, c.leaves.p,
                       c.c_begin.p, c.c_end.p, c.est_near.off.p, c.est_near.src.p, c.pm.p,
                       c.n > 64 * NF_LANES ? (int)(2 * c.est_near.count / c.nleaf) : 0, c.fpart.p);
  else
    hipLaunchKernelGGL(k_near_f, dim3(xcd_grid(ceil_div(c.nleaf, NF_WAVES))), dim3(64 * NF_WAVES), 0, s,
                       (int)c.nleaf, c.leaves.p, c.c_begin.p, c.c_end.p, c.est_near.off.p, c.est_near.src.p,
                       c.pm.p, c.fpart.p);
  stream_wait(c.fork[7], c.side2, s);
  hipLaunchKernelGGL(k_fleaf, dim3((unsigned)ceil_div(c.nleaf, 128)), dim3(128), 0, s, (int)c.nleaf, c.leaves.p,
                     c.c_begin.p, c.c_end.p, c.c_parent.p, c.fcell.p, c.fpart.p);
  unsigned long long* fmin_bits = (unsigned long long*)c.fmin.p;
  hipLaunchKernelGGL(k_fill_inf, dim3((nc + 255) / 256), dim3(256), 0, s, fmin_bits, nc);
  hipLaunchKernelGGL(k_cell_min, dim3(cell_chunk_blocks(c, FM_T / 64)), dim3(FM_T), 0, s, c.c_begin.p, c.c_end.p,
                     c.cell_choff.p, (const long long*)(c.counters.p + 4), nc, c.fpart.p, fmin_bits);
  HIPCHK(hipGetLastError());
}

template <int P>
static bool mac_dispatch(Ctx& c) {
  if constexpr (P > FMM_GPU_PMAX) {
    if (c.p > FMM_TABLE_PMAX) return false;
    run_walk<1, 0>(c, c.m2l, c.p2p, false);  // higher orders: run-time p
    return true;
  } else {
    if (c.p == P) {
      run_walk<1, P>(c, c.m2l, c.p2p, false);  // grouped by the caller (group_list)
      return true;
    }
    return mac_dispatch<P + 1>(c);
  }
}

// the acceptance walk's list grouped by sink (CSR, sources ascending)
void group_list(Ctx& c, CellList& L) { group_by_sink(c, L); }

void mac_walk(Ctx& c) {
  if (!mac_dispatch<1>(c)) throw hip_error{hipErrorInvalidValue, "walk order not compiled"};
}

}  // namespace fmm
