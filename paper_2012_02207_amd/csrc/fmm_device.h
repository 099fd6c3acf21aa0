// Device helpers shared by the gfx950 kernels of this library.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <type_traits>

#include "fmm_internal.h"

namespace fmm {

constexpr int WAVE = 64;

__device__ __forceinline__ int lane_id() { return __lane_id(); }

__device__ __forceinline__ uint64_t ballot(bool p) { return __ballot(p); }

__device__ __forceinline__ uint64_t lanemask_lt() {
  int l = lane_id();
  return l == 0 ? 0ull : (~0ull >> (64 - l));
}

// Workgroup i runs on XCD i mod 8.  Per-sink kernels take their sinks in
// chunks of XCD_CHUNK consecutive workgroups, the chunks dealt to the XCDs in
// turn: each XCD gets an even share of the work (sinks in one range of the
// list differ in cost) while neighbouring sinks, which share sources, still
// run on the same XCD.  The grid is a whole number of rounds (xcd_grid).
constexpr int XCD_CHUNK = 8;  // measured: 1, 4 and 8 within 0.7%; 32 and 128 slower (2.9%, 1.4%)
__device__ __forceinline__ int xcd_block() {
  int j = blockIdx.x >> 3, x = blockIdx.x & 7;
  return ((j / XCD_CHUNK) * 8 + x) * XCD_CHUNK + j % XCD_CHUNK;
}

// wave-wide broadcast of a double from lane `src`
__device__ __forceinline__ double shfl_d(double v, int src) { return __shfl(v, src, WAVE); }

// full-wave sum (every lane receives the total); butterfly over xor partners
__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o, WAVE);
  return v;
}

__device__ __forceinline__ float wave_sum_f(float v) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o, WAVE);
  return v;
}

__device__ __forceinline__ double wave_max(double v) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) v = fmax(v, __shfl_xor(v, o, WAVE));
  return v;
}

__host__ __device__ inline int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

// grid for xcd_block(): nblk blocks rounded up to whole rounds of 8 chunks
inline unsigned xcd_grid(int64_t nblk) {
  int64_t r = 8 * (int64_t)XCD_CHUNK;
  return (unsigned)(r * ceil_div(nblk, r));
}

// n! in FP64 by repeated multiplication (evaluation-side normalisations only)
__device__ __forceinline__ double fmm_fact_dev(int n) {
  double r = 1.0;
  for (int i = 2; i <= n; i++) r *= (double)i;
  return r;
}


// reciprocal square root to full FP64 accuracy: the hardware estimate y (about
// 2^-27 relative) and one third-order step, y (1 + e/2 + 3 e^2/8) with
// e = 1 - x y^2
__device__ __forceinline__ double rsqrt_d(double x) {
  double y = __builtin_amdgcn_rsq(x);
  double e = fma(-(x * y), y, 1.0);
  return fma(y * e, fma(e, 0.375, 0.5), y);
}

// ---- division without the operator's scaling --------------------------------
// a / d rounded correctly, as the operator does, for operands well inside the
// exponent range (div_safe): two Newton steps on the hardware reciprocal, then
// the quotient corrected by its exact remainder (Markstein's division by fused
// multiply-adds).  Nine FP64 instructions; the operator's scaling and fix-up
// instructions about double that time.
__device__ __forceinline__ double div_scaled(double a, double d) {
  double y = __builtin_amdgcn_rcp(d);
  y = fma(y, fma(-d, y, 1.0), y);
  y = fma(y, fma(-d, y, 1.0), y);
  double q = a * y;
  return fma(fma(-d, q, a), y, q);
}

// 2^-500 <= |x| < 2^500 (false for 0, infinities and NaN)
__device__ __forceinline__ bool div_safe(double x) {
  unsigned e = ((unsigned)(__double_as_longlong(x) >> 52)) & 0x7ffu;
  return e - 523u < 1000u;
}

// Segment and tile of an extra near-field item (NfPlan) in one int: a leaf of
// segments has at most 64 bodies, so 8 tiles (code >= 0); a larger one has none.
__device__ __forceinline__ int nf_code(int seg, int tile) { return tile < 8 ? seg * 8 + tile : -tile; }
__device__ __forceinline__ void nf_decode(int code, int& seg, int& tile) {
  seg = code < 0 ? 0 : code >> 3;
  tile = code < 0 ? -code : code & 7;
}

// segment seg of the nseg of sink B's list [b, e) (M2lSeg)
__device__ __forceinline__ void m2l_segment(const M2lSeg& sg, int B, int nseg, int seg, int& b, int& e) {
  if (nseg <= 1) return;
  int K = sg.seglen ? sg.seglen[B] : sg.K;
  b += seg * K;
  e = min(e, b + K);
}
// first source of [b, e) whose id is >= first_lo (ids are breadth first, so the
// sources above the root levels form a prefix of the ascending list)
__device__ __forceinline__ int split_point(const int* src, int b, int e, int first_lo) {
  int lo = b, hi = e;
  while (lo < hi) {
    int mid = (lo + hi) >> 1;
    if (src[mid] < first_lo)
      lo = mid + 1;
    else
      hi = mid;
  }
  return lo;
}

// work item `it` of the plan: leaf index, segment and tile; false if there is none
__device__ __forceinline__ bool nf_item(const NfPlan& plan, int it, int& li, int& seg, int& tile) {
  li = it;
  seg = tile = 0;
  if (it >= plan.nleaf) {
    int x = it - plan.nleaf, front = plan.nextra[0];
    if (it >= plan.max_items || x >= front + plan.nextra[1]) return false;
    int2 v = plan.extra[x < front ? x : plan.max_items - 1 - (it - front)];
    li = v.x;
    nf_decode(v.y, seg, tile);
  }
  return true;
}

// sinks [s0, s0 + count) of tile `tile` of a leaf of nB bodies
__device__ __forceinline__ int nf_tile_count(int nB) { return (nB + NF_TILE - 1) / NF_TILE; }
__device__ __forceinline__ void nf_tile(int nB, int tile, int& s0, int& count) {
  int64_t n = nB;
  int tiles = nf_tile_count(nB);
  s0 = (int)(n * tile / tiles);
  count = (int)(n * (tile + 1) / tiles) - s0;
}

// a / d rounded correctly for an integer d of a recurrence (1 <= d < 2^20), from
// y = rcp_newton(d), which does not depend on a: three dependent instructions
// instead of the operator's eleven.  Numerators outside div_safe (the
// harmonics of offsets that underflow) take the operator.  For every d up to 4096 y
// itself is 1 / d rounded correctly; the recurrences' largest is 900.
__device__ __forceinline__ double rcp_newton(double d) {
  double y = __builtin_amdgcn_rcp(d);
  y = fma(y, fma(-d, y, 1.0), y);
  return fma(y, fma(-d, y, 1.0), y);
}
__device__ __forceinline__ double div_by(double a, double d, double y) {
  double q = a * y;
  q = fma(fma(-d, q, a), y, q);
  q = a == 0.0 ? a : q;  // (the sign of a zero)
  bool far = a != 0.0 && !div_safe(a);
  if (ballot(far)) q = far ? a / d : q;
  return q;
}

// (n, m) of coefficient index t = n (n + 1) / 2 + m, and n of entry
// t = n (n + 1) + m of a both-sign layout
__device__ __forceinline__ void coef_nm(int t, int& n, int& m) {
  n = (int)((__builtin_sqrtf(8.0f * (float)t + 1.0f) - 1.0f) * 0.5f);  // exact or one off
  if (cidx(n + 1, 0) <= t) n++;
  if (cidx(n, 0) > t) n--;
  m = t - cidx(n, 0);
}
// Task u of the (child, coefficient) tasks of kn children in order of n, so that
// the lanes of a wavefront share the length of their sums.
__device__ __forceinline__ void child_task(int u, int kn, int& j, int& n, int& m) {
  coef_nm(u / kn, n, m);
  int r = u - kn * cidx(n, 0);
  j = r / (n + 1);
  m = r - j * (n + 1);
}
__device__ __forceinline__ int both_sign_n(int t) {
  int n = (int)__builtin_sqrtf((float)t);
  if ((n + 1) * (n + 1) <= t) n++;
  if (n * n > t) n--;
  return n;
}

// entries of segment seg of a list [qb, qe) cut into nseg segments (NfPlan)
__device__ __forceinline__ void segment_bounds(int nseg, int seg, int& qb, int& qe) {
  int64_t len = qe - qb;
  int b = qb;
  qb = b + (int)(len * seg / nseg);
  qe = b + (int)(len * (seg + 1) / nseg);
}

// system of body i: the last s with off[s] <= i
__device__ __forceinline__ int system_of(const int* off, int nsys, int64_t i) {
  int lo = 0, hi = nsys - 1;
  while (lo < hi) {
    int mid = (lo + hi + 1) >> 1;
    if (off[mid] <= i)
      lo = mid;
    else
      hi = mid - 1;
  }
  return lo;
}

// ---- stable LSD radix sort within one workgroup of T threads (1024 or 256) ------
// Up to I keys per thread (and payloads, with VAL), in registers: wavefront w
// holds positions (w C + c) 64 + lane, c < C, of the T C keys (pad with all
// ones: they stay last).  Per 8-bit pass a key's rank among equal digits comes
// from ballots, as in the tiled sort of tree.hip, and the keys move through LDS.
constexpr int BS_T = 1024;
template <class K, int I, bool VAL, int T = BS_T>
struct BlockSort {
  K sk[T * I];
  int sv[VAL ? T * I : 1];
  int wcnt[T / 64][256];
  int dstart[256], wsum[4];
};

template <class K, int I, bool VAL, int T>
__device__ inline void block_sort(BlockSort<K, I, VAL, T>& s, K (&k)[I], int (&v)[I], int C, int nbits) {
  constexpr int BS_T = T, BS_W = T / 64;
  int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  uint64_t lt = lanemask_lt();
  for (int shift = 0; shift < nbits; shift += 8) {
    for (int t = tid; t < BS_W * 256; t += BS_T) (&s.wcnt[0][0])[t] = 0;
    __syncthreads();
    int rank[I];
#pragma unroll
    for (int c = 0; c < I; c++) {
      if (c < C) {
        int d = (int)((k[c] >> shift) & 255);
        uint64_t peers = ~0ull;
#pragma unroll
        for (int b = 0; b < 8; b++) {
          bool bit = (d >> b) & 1;
          uint64_t bb = ballot(bit);
          peers &= bit ? bb : ~bb;
        }
        int cnt = s.wcnt[w][d];
        rank[c] = cnt + __popcll(peers & lt);
        __builtin_amdgcn_wave_barrier();
        if ((peers >> lane) == 1ull) s.wcnt[w][d] = cnt + __popcll(peers);  // the highest peer
        __builtin_amdgcn_wave_barrier();
      }
    }
    __syncthreads();
    if (tid < 256) {  // per digit: starts of the wavefronts' runs, and of the digit
      int tot = 0;
      for (int ww = 0; ww < BS_W; ww++) {
        int t = s.wcnt[ww][tid];
        s.wcnt[ww][tid] = tot;
        tot += t;
      }
      int incl = tot;
      for (int o = 1; o < 64; o <<= 1) {
        int y = __shfl_up(incl, o, 64);
        if (lane >= o) incl += y;
      }
      if (lane == 63) s.wsum[w] = incl;
      s.dstart[tid] = incl - tot;
    }
    __syncthreads();
    if (tid < 256) {
      int before = 0;
      for (int ww = 0; ww < w; ww++) before += s.wsum[ww];
      s.dstart[tid] += before;
    }
    __syncthreads();
#pragma unroll
    for (int c = 0; c < I; c++) {
      if (c < C) {
        int d = (int)((k[c] >> shift) & 255);
        int lp = s.dstart[d] + s.wcnt[w][d] + rank[c];
        s.sk[lp] = k[c];
        if (VAL) s.sv[lp] = v[c];
      }
    }
    __syncthreads();
#pragma unroll
    for (int c = 0; c < I; c++) {
      if (c < C) {
        int at = (w * C + c) * 64 + lane;
        k[c] = s.sk[at];
        if (VAL) v[c] = s.sv[at];
      }
    }
    // (the next pass writes sk only after further barriers)
  }
}

// ---- the bodies of a list of leaves as a stream of 64-body chunks ----------
// One wavefront reads the bodies of the list src[q .. qe) (cells, bodies
// [cb, ce) each) in list order, 64 at a time whatever the leaves' sizes: short
// leaves share a chunk.  The lanes hold a window of 64 list entries (first body
// and count), loaded side by side and the next window one window ahead, so that
// no chunk waits for the chain list entry -> cell bounds -> bodies.
struct BodyStream {
  const int *src, *cb, *ce;
  int q, qe;         // list entries not in a window yet
  int wb, wn;        // this lane's entry of the window: first body, count
  int pb, pe, pcnt;  // the next window (first body, end; not waited for), its entries
  int e, nwin, used; // current entry, entries of the window, bodies used of the current one

  __device__ __forceinline__ void fetch(int lane) {
    pcnt = min(64, qe - q);
    if (pcnt > 0) {
      int A = src[q + min(lane, pcnt - 1)];
      pb = cb[A];
      pe = ce[A];
    }
    q += pcnt;
  }
  __device__ __forceinline__ void start(const int* src_, const int* cb_, const int* ce_, int q0, int q1, int lane) {
    src = src_;
    cb = cb_;
    ce = ce_;
    q = q0;
    qe = q1;
    e = nwin = used = 0;
    fetch(lane);
  }
  // This lane's body of the next chunk (`none` past the end of the chunk);
  // returns the chunk's size, 0 at the end of the list.
  __device__ __forceinline__ int next(int lane, int none, int& body) {
    int cnt = 0;
    body = none;
    while (cnt < 64) {
      if (e == nwin) {
        if (pcnt == 0) break;
        wb = pb;
        wn = pe - pb;
        nwin = pcnt;
        e = 0;
        fetch(lane);
      }
      int b = __builtin_amdgcn_readlane(wb, e) + used, n = __builtin_amdgcn_readlane(wn, e) - used;
      int take = min(n, 64 - cnt);
      if ((unsigned)(lane - cnt) < (unsigned)take) body = b + lane - cnt;
      cnt += take;
      if (take == n) {
        e++;
        used = 0;
      } else {
        used += take;
      }
    }
    return cnt;
  }
};

// ---- cross-lane transpose-reduce (the M2L kernels) ------------------------
// D values per lane summed over the 64 lanes in six halving steps with
// partner distances 32, 16, 8, 4, 2, 1.  With L values left, a lane keeps the
// first ceil(L/2) of them or the rest, by that bit of its lane id, and adds its
// partner's copy of the kept part; once a single value is left the steps are
// plain butterflies.  A lane on the upper side of an odd L keeps one slot more
// than there are values: that pad slot holds an unused sum, and pads only ever
// meet pads (partners share every earlier bit), so they need no clearing.
// The total of value j ends in lane reduce_owner(D, j).
constexpr int reduce_len(int D, int t) {
  int L = D;
  for (int k = 0; k < t; k++) L = (L + 1) / 2;
  return L;
}
constexpr int reduce_owner(int D, int j) {
  int lane = 0, L = D;
  for (int t = 0; t < 6; t++) {
    if (L >= 2) {
      int h = (L + 1) / 2;
      if (j >= h) {
        lane |= 32 >> t;
        j -= h;
      }
      L = h;
    }
  }
  return lane;
}

// reduce_owner inverted: the value j whose total this lane ends with, and
// whether that is a real value (not a pad)
template <int D>
__device__ __forceinline__ void reduce_slot(int lane, int& j, int& real) {
  j = 0;
  int left = D;  // real values in this lane's part
  bool ok = true;
#pragma unroll
  for (int t = 0; t < 6; t++) {
    int L = reduce_len(D, t);
    bool bit = (lane & (32 >> t)) != 0;
    if (L >= 2) {
      int H = (L + 1) / 2;
      j += bit ? H : 0;
      left = bit ? left - H : (left < H ? left : H);
    } else {
      ok = ok && !bit;
    }
  }
  real = ok && left >= 1;
}

// DPP control of the steps at distances 8, 4, 2, 1 (t = 2..5): row mirror,
// half-row mirror, quad_perm [2,3,0,1], quad_perm [1,0,3,2]; each pairs lanes
// that differ in that bit
constexpr int reduce_dpp_ctrl(int t) { return t == 2 ? 0x140 : t == 3 ? 0x141 : t == 4 ? 0x4E : 0xB1; }

// lanes 32..63 of a <-> lanes 0..31 of b (T = 0), or the odd 16-lane rows of a
// <-> the even rows of b (T = 1)
template <int T>
__device__ __forceinline__ void lane_swap(uint32_t& a, uint32_t& b) {
  if constexpr (T == 0) {
    auto r = __builtin_amdgcn_permlane32_swap(a, b, false, false);
    a = (uint32_t)r[0];
    b = (uint32_t)r[1];
  } else {
    auto r = __builtin_amdgcn_permlane16_swap(a, b, false, false);
    a = (uint32_t)r[0];
    b = (uint32_t)r[1];
  }
}
template <int T>
__device__ __forceinline__ void lane_swap(float& a, float& b) {
  uint32_t ua = __builtin_bit_cast(uint32_t, a), ub = __builtin_bit_cast(uint32_t, b);
  lane_swap<T>(ua, ub);
  a = __builtin_bit_cast(float, ua);
  b = __builtin_bit_cast(float, ub);
}
template <int T>
__device__ __forceinline__ void lane_swap(double& a, double& b) {
  uint64_t ua = __builtin_bit_cast(uint64_t, a), ub = __builtin_bit_cast(uint64_t, b);
  uint32_t alo = (uint32_t)ua, ahi = (uint32_t)(ua >> 32), blo = (uint32_t)ub, bhi = (uint32_t)(ub >> 32);
  lane_swap<T>(alo, blo);
  lane_swap<T>(ahi, bhi);
  a = __builtin_bit_cast(double, ((uint64_t)ahi << 32) | alo);
  b = __builtin_bit_cast(double, ((uint64_t)bhi << 32) | blo);
}

// the value of v in the lane that DPP control CTRL selects
template <int CTRL>
__device__ __forceinline__ float dpp_read(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xF, 0xF, false));
}
template <int CTRL>
__device__ __forceinline__ double dpp_read(double v) {
  uint64_t u = __builtin_bit_cast(uint64_t, v);
  int lo = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)u, CTRL, 0xF, 0xF, false);
  int hi = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)(u >> 32), CTRL, 0xF, 0xF, false);
  return __builtin_bit_cast(double, ((uint64_t)(uint32_t)hi << 32) | (uint32_t)lo);
}

// compile-time loop: f(std::integral_constant<int, i>) for i in [I, E)
template <int I, int E, class F>
__device__ __forceinline__ void unroll_for(F&& f) {
  if constexpr (I < E) {
    f(std::integral_constant<int, I>{});
    unroll_for<I + 1, E>(f);
  }
}

// x[0..D) of every lane -> the cross-lane totals (in place, see above); each
// lane adds its last value to *acc_slot, meaningful in the owner lanes only
template <int D, class T>
__device__ __forceinline__ void reduce_lanes(T* x, double* acc_slot, int lane) {
  unroll_for<0, 6>([&](auto tc) {
    constexpr int t = tc;
    constexpr int L = reduce_len(D, t);
    constexpr int H = (L + 1) / 2;
    if constexpr (t < 2) {
      unroll_for<0, H>([&](auto ic) {
        constexpr int i = ic;
        T a = x[i], b = x[i];  // L == 1 (or the pad of an odd L): a butterfly
        if constexpr (i + H < L) b = x[i + H];
        lane_swap<t>(a, b);
        x[i] = a + b;
      });
    } else {
      constexpr int CTRL = reduce_dpp_ctrl(t);
      bool hi = (lane & (32 >> t)) != 0;
      unroll_for<0, H>([&](auto ic) {
        constexpr int i = ic;
        T r = x[i] + dpp_read<CTRL>(x[i]);
        if constexpr (i + H < L) {
          T q = x[i + H] + dpp_read<CTRL>(x[i + H]);
          r = hi ? q : r;
        }
        x[i] = r;
      });
    }
  });
  *acc_slot += (double)x[0];
}

}  // namespace fmm
