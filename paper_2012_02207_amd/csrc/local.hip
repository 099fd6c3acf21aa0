// Downward pass and near field on gfx950 (section 2.1): L2L shifts each cell's
// local expansion to its children, L2P evaluates the leaf expansion at every
// body (potential and force), P2P adds the direct sum over the near-field leaf
// pairs, and the results are written in the caller's body order.  Also the
// plain O(N^2) direct sum used for checks.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "fmm_device.h"

namespace fmm {

// L2L, one workgroup per parent: L_child(j, i) += sum_{k <= p-j} sum_{l=-k..k}
// L_parent(j+k, i+l) conj(Y_k^l(z_child - z_parent)).  The parent expansion
// and the conjugated harmonics of every child are laid out in LDS for both
// signs of the order (entry n(n+1) + m, m = -n..n), which makes every sum a
// branch-free loop; lanes evaluate harmonic columns, then (child,
// coefficient) sums, a thread for (almost) every one: a launch is bound by the
// chain of its longest sum (24 us for a level of any size with 256 threads
// at p = 10, 11 us now; at N = 2^20 all levels 425 and 262 us).
constexpr int L2L_T_MAX = 1024;

// G: children per pass (their harmonics share LDS with the parent's expansion;
// 8 = all at once, fewer at the orders where eight do not fit)
__global__ void __launch_bounds__(L2L_T_MAX) k_l2l(int p, int first, int count, const int* __restrict__ c0,
                                                    const int* __restrict__ nch, const double* __restrict__ cx,
                                                    const double* __restrict__ cy, const double* __restrict__ cz,
                                                    double* loc, int G) {
  extern __shared__ double lds[];
  const int L2L_T = blockDim.x;
  int P = first + blockIdx.x;
  if (blockIdx.x >= count || nch[P] == 0) return;
  int nc = ncoef(p), S = (p + 1) * (p + 1);
  int k0 = c0[P], kn = nch[P];
  double2* Lx = (double2*)lds;  // [S]
  double2* Yc = Lx + S;         // [child of the pass][S]
  int t = threadIdx.x;
  const double* Lp = loc + (size_t)P * nc * 2;
  for (int u = t; u < S; u += L2L_T) {
    int n = both_sign_n(u);
    int m = u - n * n - n, am = m < 0 ? -m : m;
    double a = Lp[2 * cidx(n, am)], b = Lp[2 * cidx(n, am) + 1];
    if (m < 0) {
      double sg = (am & 1) ? -1.0 : 1.0;
      a = sg * a;
      b = -sg * b;
    }
    Lx[u] = make_double2(a, b);
  }
  for (int j0 = 0; j0 < kn; j0 += G) {
    int gn = min(G, kn - j0);
    if (j0 > 0) __syncthreads();  // the previous pass has read its harmonics
    for (int u = t; u < gn * (p + 1); u += L2L_T) {  // column m of child j's harmonics
      int j = u / (p + 1), m = u - j * (p + 1);
      int ch = k0 + j0 + j;
      double x = cx[ch] - cx[P], y = cy[ch] - cy[P], z = cz[ch] - cz[P];
      double r2 = fma(x, x, fma(y, y, z * z));
      double pr = 1.0, pi = 0.0;
      for (int n = 1; n <= m; n++) {
        double inv = -rcp_newton((double)(2 * n));
        double tr = fma(x, pr, -y * pi), ti = fma(x, pi, y * pr);
        pr = tr * inv;
        pi = ti * inv;
      }
      double2* Y = Yc + j * S;
      double sg = (m & 1) ? -1.0 : 1.0;
      // conj(Y_n^m) at +m; conj(Y_n^-m) = (-1)^m Y_n^m at -m
      Y[m * m + m + m] = make_double2(pr, -pi);
      if (m > 0) Y[m * m] = make_double2(sg * pr, sg * pi);
      double ar2 = 0.0, ai2 = 0.0, ar1 = pr, ai1 = pi;
      for (int n = m + 1; n <= p; n++) {
        double k = (double)(2 * n - 1) * z, inv = rcp_newton((double)((n + m) * (n - m)));
        double vr = fma(k, ar1, -r2 * ar2) * inv, vi = fma(k, ai1, -r2 * ai2) * inv;
        Y[n * n + n + m] = make_double2(vr, -vi);
        if (m > 0) Y[n * n + n - m] = make_double2(sg * vr, sg * vi);
        ar2 = ar1;
        ai2 = ai1;
        ar1 = vr;
        ai1 = vi;
      }
    }
    __syncthreads();
    for (int u = t; u < gn * nc; u += L2L_T) {
      int j, jn, i;
      child_task(u, gn, j, jn, i);
      int q = cidx(jn, i);
      const double2* Y = Yc + j * S;
      double sr = 0.0, si = 0.0;
      for (int k = 0; k <= p - jn; k++) {
        int n = jn + k;
        const double2* Ln = Lx + n * n + n + i - k;
        const double2* Yk = Y + k * k;
#pragma unroll 4
        for (int r = 0; r <= 2 * k; r++) {  // l = r - k
          double2 a = Ln[r], b = Yk[r];
          sr = fma(a.x, b.x, fma(-a.y, b.y, sr));
          si = fma(a.x, b.y, fma(a.y, b.x, si));
        }
      }
      double* Lc = loc + (size_t)(k0 + j0 + j) * nc * 2;
      Lc[2 * q] += sr;
      Lc[2 * q + 1] += si;
    }
  }
}

// L2P: the local expansion L shifted to offset (X, Y, Z) from its centre;
// harmonics built column by column and each used once.
__device__ __forceinline__ void l2p_eval(int p, const double* __restrict__ L, double X, double Y,
                                         double Z, double& ax, double& ay, double& az, double& ph) {
  double r2 = fma(X, X, fma(Y, Y, Z * Z));
  double s00 = 0.0, s10 = 0.0, s11r = 0.0, s11i = 0.0;
  double dr = 1.0, di = 0.0;  // Y_m^m
  for (int m = 0; m <= p; m++) {
    if (m > 0) {
      double inv = -1.0 / (double)(2 * m);
      double tr = fma(X, dr, -Y * di), ti = fma(X, di, Y * dr);
      dr = tr * inv;
      di = ti * inv;
    }
    double yr = dr, yi2 = di, pr2 = 0.0, pi2 = 0.0;
    for (int k = m; k <= p; k++) {
      if (k > m) {
        double kk = (double)(2 * k - 1) * Z, inv = 1.0 / (double)((k + m) * (k - m));
        double vr = fma(kk, yr, -r2 * pr2) * inv, vi = fma(kk, yi2, -r2 * pi2) * inv;
        pr2 = yr;
        pi2 = yi2;
        yr = vr;
        yi2 = vi;
      }
      // Y_k^m = (yr, yi2); contributions of the +m and -m terms
      double w = m == 0 ? 1.0 : 2.0;
      double Lr = L[2 * cidx(k, m)], Li = L[2 * cidx(k, m) + 1];
      s00 = fma(w, fma(Lr, yr, Li * yi2), s00);
      if (k + 1 <= p) {
        double Ur = L[2 * cidx(k + 1, m)], Ui = L[2 * cidx(k + 1, m) + 1];
        s10 = fma(w, fma(Ur, yr, Ui * yi2), s10);
        // + L_{k+1}^{m+1} conj(Y_k^m)
        double Vr = L[2 * cidx(k + 1, m + 1)], Vi = L[2 * cidx(k + 1, m + 1) + 1];
        s11r = fma(Vr, yr, fma(Vi, yi2, s11r));
        s11i = fma(Vi, yr, fma(-Vr, yi2, s11i));
        if (m >= 2) {  // the -m term: -conj(L_{k+1}^{m-1}) Y_k^m
          double Wr = L[2 * cidx(k + 1, m - 1)], Wi = L[2 * cidx(k + 1, m - 1) + 1];
          s11r = fma(-Wr, yr, fma(-Wi, yi2, s11r));
          s11i = fma(-Wr, yi2, fma(Wi, yr, s11i));
        } else if (m == 1) {  // the -1 term: -L_{k+1}^0 Y_k^1
          double Wr = L[2 * cidx(k + 1, 0)], Wi = L[2 * cidx(k + 1, 0) + 1];
          s11r = fma(-Wr, yr, fma(Wi, yi2, s11r));
          s11i = fma(-Wr, yi2, fma(-Wi, yr, s11i));
        }
      }
    }
  }
  ax = -s11r;
  ay = -s11i;
  az = s10;
  ph = -s00;
}

// P2P.  One wavefront per work item (NfPlan); the sums of each body are the
// near-field (acc, pot) of nearbuf, sorted order, or a later segment's partial
// sums.  Bound by vector ALU issue in both precisions.
//
// FP64: a lane per source body, taken 64 at a time from the list whatever the
// leaves' sizes (BodyStream; the next chunk fetched while this one is summed),
// against a tile of up to 8 sink bodies, whose positions are wave-uniform, so
// a pair costs no LDS read and every lane works.  Past the end of the list a lane
// holds the tile's first sink, without mass: a body of the item's own, so that
// nothing of another system is read.  Each lane keeps the tile's
// partial sums in registers; they are added across the lanes at the end of the
// list (reduce_lanes).  With a lane
// per (sink, source group) pair and the sources in LDS the pair loop took 2190 us
// alone at N = 2^18, p = 10 (9.8e8 pairs); this way it took 1843 us with a
// wavefront per leaf, which left the chip to the few longest leaves (1.5
// wavefronts per SIMD on average), and 1124 us with the sinks in tiles.
// Wavefronts (items) per workgroup of the near-field kernels.  A workgroup keeps
// its place until its longest item ends, so with four, 2.6 of the 4 wavefronts
// per SIMD that fit were in flight in FP64, 3.7 of 6 in mixed precision: 2^18
// bodies in FP64 4.40 ms (4.34 with one), 2^20 mixed 8.24 (8.04), 256 systems
// of 1032 to 65006 bodies (mean 15512) 37.7 (36.6).
constexpr int LG_WAVES = 1;

// the pairs of an item added to the sum of its workgroup's slot (NF_PAIRS)
__device__ __forceinline__ void count_pairs(unsigned long long* npairs, long long pairs) {
  atomicAdd(npairs + (blockIdx.x & (NF_PAIR_SLOTS - 1)) * (NF_PAIR_STRIDE / 2), (unsigned long long)pairs);
}

// the sinks i0 .. i0 + TS over the list src[qb .. qe), their sums to out or (add)
// onto what is there; returns the body pairs (a body with itself is none)
template <int TS>
__device__ __forceinline__ long long near_tile64(int i0, int qb, int qe, int lane, const int* __restrict__ src,
                                                 const int* __restrict__ cb, const int* __restrict__ ce,
                                                 const double4* __restrict__ pm, double eps2,
                                                 double* __restrict__ out, bool add) {
  double acc[4 * TS];
#pragma unroll
  for (int k = 0; k < 4 * TS; k++) acc[k] = 0.0;
  const double4* sink = pm + i0;
  BodyStream st;
  st.start(src, cb, ce, qb, qe, lane);
  int j, na = st.next(lane, i0, j);
  double4 cur = pm[j];
  long long pairs = 0;
  while (na > 0) {
    double4 v = cur;
    bool live = lane < na;
    if (!live) v.w = 0.0;  // past the end of the list: no mass
    int self = j - i0;     // the sink that this lane's body is, if any
    pairs += (long long)na * TS - __popcll(ballot(live && (unsigned)self < (unsigned)TS));
    int nn = st.next(lane, i0, j);
    cur = pm[j];
#pragma unroll
    for (int k = 0; k < TS; k++) {
      double dx = v.x - sink[k].x, dy = v.y - sink[k].y, dz = v.z - sink[k].z;
      double d2 = fma(dx, dx, fma(dy, dy, fma(dz, dz, eps2)));
      double rinv = rsqrt_d(d2);
      rinv = d2 > 0.0 && self != k ? rinv : 0.0;
      double mr = v.w * rinv, mr3 = mr * rinv * rinv;
      acc[4 * k] = fma(mr3, dx, acc[4 * k]);
      acc[4 * k + 1] = fma(mr3, dy, acc[4 * k + 1]);
      acc[4 * k + 2] = fma(mr3, dz, acc[4 * k + 2]);
      acc[4 * k + 3] -= mr;
    }
    na = nn;
  }
  double tot = 0.0;
  reduce_lanes<4 * TS>(acc, &tot, lane);
  int c, real;
  reduce_slot<4 * TS>(lane, c, real);
  if (real) out[c] = add ? out[c] + tot : tot;
  return pairs;
}

__global__ void __launch_bounds__(64 * LG_WAVES) __attribute__((amdgpu_waves_per_eu(4))) k_near_fp64(
    const int* __restrict__ leaves, NfPlan plan, const int* __restrict__ cb, const int* __restrict__ ce,
    const int* __restrict__ off, const int* __restrict__ srcl, const double4* __restrict__ pm, double eps2,
    double4* __restrict__ nearbuf, double4* __restrict__ part, unsigned long long* npairs) {
  int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  int li, seg, tile;
  if (!nf_item(plan, xcd_block() * LG_WAVES + wv, li, seg, tile)) return;
  int B = leaves[li];
  int nseg = plan.cell_nseg[B], send = seg + 1;
  int b = cb[B], e = ce[B];
  double4* out = nearbuf + b;
  if (nseg > 1) {
    int pbase = plan.cell_pbase[B];
    if (pbase < 0) send = nseg;
    if (seg > 0) out = part + (int64_t)pbase + (int64_t)(seg - 1) * (e - b);
  }
  int s0, ts;
  nf_tile(e - b, tile, s0, ts);
  double* o = (double*)(out + s0);
  long long pairs = 0;
  for (bool add = false; seg < send; seg++, add = true) {
    int qb = off[B], qe = off[B + 1];
    if (nseg > 1) segment_bounds(nseg, seg, qb, qe);
    switch (ts) {
#define FMM_NEAR_TILE(T) \
  case T: pairs += near_tile64<T>(b + s0, qb, qe, lane, srcl, cb, ce, pm, eps2, o, add); break;
      FMM_NEAR_TILE(1)
      FMM_NEAR_TILE(2)
      FMM_NEAR_TILE(3)
      FMM_NEAR_TILE(4)
      FMM_NEAR_TILE(5)
      FMM_NEAR_TILE(6)
      FMM_NEAR_TILE(7)
      FMM_NEAR_TILE(8)
#undef FMM_NEAR_TILE
    }
  }
  if (lane == 0 && pairs > 0) count_pairs(npairs, pairs);
}

// Mixed precision: the n_B sink bodies are replicated over
// G = 64 / n_B lane groups, and group g takes every G-th body of each source
// leaf, so nearly every lane works even though leaves hold ~20 bodies.  Each
// source leaf is staged once in LDS with one coalesced load and read by the
// groups as broadcasts.  The G partial sums are combined in group order
// (deterministic) into the body's near-field (acc, pot), sorted order.
// Pair arithmetic in FP32 on the separation formed in FP64 and rounded
// once; FP32 partial sums are carried into FP64 after every source leaf
// (blocked compensation: the FP32 error grows with the leaf, not the list).
// one source body s (mass ms) acting on the sink me; CHECK: a pair at d2 = 0
// (or NaN) counts as rinv = 0, without it as rinv = inf (NaN)
template <bool CHECK>
__device__ __forceinline__ void pair32(const double4& s, float ms, const double4& me, float eps2f, float& fx,
                                       float& fy, float& fz, float& fp) {
  float dx = (float)(s.x - me.x), dy = (float)(s.y - me.y), dz = (float)(s.z - me.z);
  float d2 = fmaf(dx, dx, fmaf(dy, dy, fmaf(dz, dz, eps2f)));
  float rinv = __builtin_amdgcn_rsqf(d2);
  if (CHECK) rinv = d2 > 0.f ? rinv : 0.f;
  float mr = ms * rinv;
  float mr3 = mr * rinv * rinv;
  fx = fmaf(mr3, dx, fx);
  fy = fmaf(mr3, dy, fy);
  fz = fmaf(mr3, dz, fz);
  fp -= mr;
}

// staged source record: FP64 position, the mass rounded to FP32 once here and
// kept in the low word of .w (the high word is not read)
struct Staged {
  double2 xy;
  uint4 zm;
};
// body min(j0 + lane, je - 1) (lane32: 32 times the lane; the address is a scalar
// base plus a 32-bit offset)
__device__ __forceinline__ Staged load_staged(const double4* pm, int j0, int je, unsigned lane32) {
  const char* base = (const char*)(pm + min(j0, je - 1));
  unsigned o = min(lane32, (unsigned)max(je - j0 - 1, 0) * 32u);
  Staged r;
  r.xy = *(const double2*)(base + o);
  r.zm = *(const uint4*)(base + o + 16u);
  return r;
}
__device__ __forceinline__ void put_staged(double4* d, Staged r) {
  double m = __hiloint2double((int)r.zm.w, (int)r.zm.z);
  r.zm.z = __float_as_uint((float)m);
  *(double2*)d = r.xy;
  *(uint4*)&d->z = r.zm;
}

__device__ __forceinline__ float mass32(const double4& v) {
  return __uint_as_float((unsigned)__double_as_longlong(v.w));
}

// Bound by VALU issue: 18 instructions of 4 cycles per pair (rsq 8), 20 of all
// the kernel's, and 77% of the lanes used (counted from the lists: 21% are left
// over by leaves that do not divide 64, the rest by last rounds).  So what is not
// a pair's own arithmetic is kept off the vector unit (N = 2^20, 3.16e9 pairs: 25.5
// to 20 instructions per round of the groups, 2.85 to 2.34 ms):
//  - The records of a group's bodies are adjacent in LDS (slot g S + t / G for
//    body t of group t mod G), so a round of four pairs takes one address.
//  - The trip count na / G is the same for every lane and stays in SGPRs; only the
//    last, partial round is masked.  Lanes past G n_B repeat the last group and
//    are not read.
//  - The fast rounds take no d2 > 0 test.  A coincident pair (d2 = 0) or a NaN
//    turns fp into inf or NaN for good, so one test of fp per chunk finds it, and the
//    chunk is summed again, in the same order, with the test per pair.
// S is odd for up to 16 groups (stride 8 S banks: no two of 8 groups on the same
// ones); G S <= 127.
// Occupancy: 6 waves per SIMD (<= 80 VGPRs, measured best), with the sink
// leaf's data wave-uniform (SGPRs).
constexpr int LG_SLOTS = 128;
__global__ void __launch_bounds__(64 * LG_WAVES) __attribute__((amdgpu_waves_per_eu(6))) k_leaf_group(const int* __restrict__ leaves,
                                                              NfPlan plan, const int* __restrict__ cb,
                                                              const int* __restrict__ ce,
                                                              const int* __restrict__ off,
                                                              const int* __restrict__ srcl,
                                                              const double4* __restrict__ pm,
                                                              double eps2, double4* nearbuf,
                                                              double4* __restrict__ part,
                                                              unsigned long long* npairs, int gmax) {
  // the staged chunk; at the end of a segment the groups' sums (4 x 64 doubles)
  __shared__ double4 sbuf[LG_WAVES][LG_SLOTS];
  // totals of an unsplit list's segments, one body per lane (in LDS: the registers
  // would cost all lists a wavefront per SIMD)
  __shared__ double2 tbuf[LG_WAVES][2][64];
  int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  int li, seg, tile;  // (one tile in mixed precision)
  if (!nf_item(plan, xcd_block() * LG_WAVES + wv, li, seg, tile)) return;
  float eps2f = (float)eps2;
  long long pairs = 0;  // body pairs of this leaf (self pairs excluded), wave-uniform
  const double4* sb = sbuf[wv];
  unsigned lane32 = 32u * (unsigned)lane;
  double2(*rb)[64] = (double2(*)[64])sbuf[wv];  // the groups' sums, (x, y) and (z, potential)
  double2(*tb)[64] = tbuf[wv];
  int B = leaves[li];
  int nseg = plan.cell_nseg[B];
  int b = cb[B], e = ce[B];
  int qb = off[B], qe = off[B + 1];
  // output: the near field itself, or the partial sums of a later segment
  double4* out = nearbuf;
  int folds = 1;  // segments taken, one after the other
  if (nseg > 1) {  // (the leaf's bodies fit one wavefront)
    int pbase = plan.cell_pbase[B];
    if (pbase < 0)
      folds = nseg;
    else
      segment_bounds(nseg, seg, qb, qe);
    if (seg > 0) out = part + ((int64_t)pbase + (int64_t)(seg - 1) * (e - b) - b);
  }
  for (int i0 = b; i0 < e; i0 += 64) {
    int nB = min(64, e - i0);
    int G = 64 / nB;
    if (gmax > 0 && G > gmax) G = gmax;  // fewer groups: longer runs per lane, fewer partial sums
    int S = (64 + G - 1) / G;
    if (G <= 16) S |= 1;
    int invG = (65536 + G - 1) / G;  // x / G = (x invG) >> 16 for x <= 64
    int g = lane / nB, s = lane - g * nB;
    g = min(g, G - 1);
    double4* put = sbuf[wv] + (lane % G) * S + lane / G;
    int i = i0 + s;
    double4 me = pm[i];
    double nx = 0.0, ny = 0.0, nz = 0.0, np = 0.0;
    float fx = 0.f, fy = 0.f, fz = 0.f, fp = 0.f;
    // the groups' sums in LDS, to be combined in order
    auto put_groups = [&]() {
      __builtin_amdgcn_wave_barrier();
      rb[0][lane] = make_double2(nx, ny);
      rb[1][lane] = make_double2(nz, np);
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_s_waitcnt(0xc07f);
    };
    int fold = 0, qfold = qe;  // segments added up so far, end of the present one
    if (folds > 1) {
      int q0 = qb;
      qfold = qe;
      segment_bounds(folds, 0, q0, qfold);
    }
    // source chunks (<= 64 bodies of one source leaf) in list order; the
    // next chunk is fetched into registers while the current one is summed
    int q = qb, j0 = 0, je = 0;
    Staged cur{};
    if (q < qe) {
      int A = srcl[q];
      j0 = cb[A];
      je = ce[A];
      cur = load_staged(pm, j0, je, lane32);
    }
    while (q < qe) {
      int na = min(64, je - j0);
      pairs += (long long)nB * na - max(0, min(i0 + nB, j0 + na) - max(i0, j0));
      int nq = q, nj0 = j0 + 64, nje = je;
      if (nj0 >= je) {
        nq = q + 1;
        if (nq < qe) {
          int A = srcl[nq];
          nj0 = cb[A];
          nje = ce[A];
        }
      }
      __builtin_amdgcn_wave_barrier();
      put_staged(put, cur);
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0): the staged chunk is visible to the wave
      cur = load_staged(pm, nj0, nje, lane32);  // (after the last chunk: its last body again)
      int nr = (na * invG) >> 16, rem = na - nr * G;  // full rounds, bodies of the partial one
      // the sink's own leaf: its pair with itself gets mass 0 (with eps = 0
      // the d2 > 0 test also removes it); other chunks hold no sink body
      bool slow = j0 < i0 + nB && i0 < j0 + na;
      const double4* t = sb + g * S;
      if (!slow) {
        float sx = fx, sy = fy, sz = fz, sp = fp;  // (not 0 in the later chunks of a leaf)
        const double4* u = t;
        for (int r = nr >> 2; r > 0; r--, u += 4) {
          double4 s0 = u[0], s1 = u[1], s2 = u[2], s3 = u[3];
          pair32<false>(s0, mass32(s0), me, eps2f, fx, fy, fz, fp);
          pair32<false>(s1, mass32(s1), me, eps2f, fx, fy, fz, fp);
          pair32<false>(s2, mass32(s2), me, eps2f, fx, fy, fz, fp);
          pair32<false>(s3, mass32(s3), me, eps2f, fx, fy, fz, fp);
        }
        if (nr & 2) {
          double4 s0 = u[0], s1 = u[1];
          pair32<false>(s0, mass32(s0), me, eps2f, fx, fy, fz, fp);
          pair32<false>(s1, mass32(s1), me, eps2f, fx, fy, fz, fp);
          u += 2;
        }
        if (nr & 1) {
          double4 s0 = u[0];
          pair32<false>(s0, mass32(s0), me, eps2f, fx, fy, fz, fp);
          u++;
        }
        if (g < rem) {
          double4 s0 = u[0];
          pair32<false>(s0, mass32(s0), me, eps2f, fx, fy, fz, fp);
        }
        slow = ballot(!__builtin_isfinite(fp)) != 0;
        if (slow) {
          fx = sx;
          fy = sy;
          fz = sz;
          fp = sp;
        }
      }
      if (slow) {
        int ti = i - j0;
        for (int r = 0; r < nr; r++) {
          double4 s0 = t[r];
          pair32<true>(s0, g + r * G != ti ? mass32(s0) : 0.f, me, eps2f, fx, fy, fz, fp);
        }
        if (g < rem) {
          double4 s0 = t[nr];
          pair32<true>(s0, g + nr * G != ti ? mass32(s0) : 0.f, me, eps2f, fx, fy, fz, fp);
        }
      }
      if (nq != q) {  // end of a source leaf: carry the FP32 block into FP64
        nx += (double)fx;
        ny += (double)fy;
        nz += (double)fz;
        np += (double)fp;
        fx = fy = fz = fp = 0.f;
        if (nq == qfold && nq < qe) {  // end of a segment
          put_groups();
          if (lane < nB)
#pragma unroll 1
            for (int k = 0; k < 2; k++) {  // (one after the other: registers)
              double2 t = make_double2(0.0, 0.0);
              for (int gg = 0; gg < G; gg++) {
                double2 v = rb[k][gg * nB + s];
                t.x += v.x;
                t.y += v.y;
              }
              if (fold > 0) {
                double2 v = tb[k][lane];
                t.x = v.x + t.x;
                t.y = v.y + t.y;
              }
              tb[k][lane] = t;
            }
          nx = ny = nz = np = 0.0;
          fold++;
          int q0 = qb;
          qfold = qe;
          segment_bounds(folds, fold, q0, qfold);
        }
      }
      q = nq;
      j0 = nj0;
      je = nje;
    }
    put_groups();
    if (lane < nB) {
      double tx = 0.0, ty = 0.0, tz = 0.0, tp = 0.0;
      for (int gg = 0; gg < G; gg++) {
        double2 u = rb[0][gg * nB + s], v = rb[1][gg * nB + s];
        tx += u.x;
        ty += u.y;
        tz += v.x;
        tp += v.y;
      }
      if (fold > 0) {
        double2 u = tb[0][lane], v = tb[1][lane];
        tx = u.x + tx;
        ty = u.y + ty;
        tz = v.x + tz;
        tp = v.y + tp;
      }
      out[i] = make_double4(tx, ty, tz, tp);
    }
    __builtin_amdgcn_wave_barrier();
  }
  if (lane == 0 && pairs > 0) count_pairs(npairs, pairs);
}

// Which of the two kernels the near field of a context takes: in every precision
// but mixed the FP64 one (a frozen evaluation may run under FMM_DIRECT), whose
// plan has tiles.
static bool nf_tiled(const Ctx& c) { return c.prm.precision != FMM_MIXED; }

// Near-field work items (NfPlan), one thread per leaf; ctr: counters[NF_COUNTERS ..].
// List entries per segment, at least: a 1024th of the system's bodies (four times
// that in FP64, whose items hold at most 8 sinks), from NF_SEG_MIN or
// NF_SEG_MIN_TILED to NF_SEG_MAX, for leaves of up to 64 bodies, and in proportion
// more of smaller leaves; and a 32nd of the list (NF_SEG_PER).  A small system has
// few leaves with long lists (4096 bodies: 303 leaves of 226 entries), and only
// short segments spread them over the chip; a large one has enough leaves, and
// only the outliers are cut (at N = 2^18 one leaf holds 2776 entries, 42 times the
// mean work).  The bound is the system's and the list's own, so that a system of a
// batch sums in the same order as alone.
// Mixed: with 256 entries or more whatever the size the near field of 30011 bodies
// took 678 us (319 now).  At least 8, 16, 24 and 32: 8192 bodies 1.08, 0.98, 0.93 and
// 0.93 ms, frozen 16384 524, 509, 458 and 455 us, near field of 1000 43, 45, 49 and 52 us.
// FP64, at least 32, 64 and 96: 4096 bodies 0.90, 0.86 and 0.84 ms, jerk of 2000
// 1.02, 1.02 and 1.05.  No bound on the segments of a list: 30000 bodies at p = 4,
// err_tol = 1e-9 (lists of 1600) 3.8 ms, 2.2 with 32: the slots run out otherwise.
constexpr int NF_SEG_MIN = 24, NF_SEG_MIN_TILED = 64, NF_SEG_MAX = 512;
constexpr int NF_SEG_DIV = 1024, NF_SEG_TILED = 4;
constexpr int NF_SEG_PER = 32;
// What is split (whatever is, the sums are the same): lists longer than a 65536th
// of all entries (NF_ITEMS), or where the leaves alone fill the chip some times over
// (NF_FULL wavefronts) lists of more than twice the mean length.  NF_SLOTS, NF_SPLIT:
// slots for partial sums (32 B each) and later segments' items, at the most; the
// grid covers that many items, and a wavefront that finds none costs 0.8 ns.  Later
// segments come first among the extra items, then the later tiles in the order of
// the leaves, whose lists are the longer the shallower the leaf: the longest items
// have to start early.  (The atomics for slots delay the wavefronts that have long
// lists, so the tiles are claimed before them; after them all items of those
// wavefronts came last: the near field of 2^18 bodies alone 1.18 -> 1.14 ms in FP64,
// the gradient's 2.47 -> 2.36.)
constexpr int64_t NF_ITEMS = 65536, NF_FULL = 24576, NF_SLOTS = 1 << 20, NF_SPLIT = 65536;

// len: entries of the list (0: the least of any list)
__host__ __device__ inline int nf_segment(int64_t bodies, int max_nb, int tiled, int len) {
  int64_t k = bodies / NF_SEG_DIV * (tiled ? NF_SEG_TILED : 1), least = tiled ? NF_SEG_MIN_TILED : NF_SEG_MIN;
  k = k < least ? least : k;
  k = k > NF_SEG_MAX ? NF_SEG_MAX : k;
  k = k * 64 / max_nb;
  int part = (len + NF_SEG_PER - 1) / NF_SEG_PER;
  return k < part ? part : (int)k;
}

__global__ void k_nf_plan(const int* __restrict__ leaves, int nleaf, const int* __restrict__ cb,
                          const int* __restrict__ ce, const int* __restrict__ off, const int* __restrict__ sys_off,
                          int nsys, int max_nb, int tiled, int long_len, int max_slots, int max_split, int extra_max,
                          int* cell_nseg, int* cell_pbase, int2* extra, int* ctr) {
  int li = blockIdx.x * blockDim.x + threadIdx.x;
  if (li >= nleaf) return;
  int B = leaves[li];
  int len = off[B + 1] - off[B], nB = ce[B] - cb[B];
  int sys = nsys > 1 ? system_of(sys_off, nsys, cb[B]) : 0;
  int K = nf_segment(sys_off[sys + 1] - sys_off[sys], max_nb, tiled, len);
  int ns = (nB <= 64 && len > K) ? (len + K - 1) / K : 1;
  int nt = tiled ? nf_tile_count(nB) : 1;
  if (nt > 1) {  // (claimed before any slots: see above)
    int x = extra_max - 1 - atomicAdd(ctr + 9, nt - 1);
    for (int t = 1; t < nt; t++) extra[x--] = make_int2(li, nf_code(0, t));
  }
  int pbase = -1;
  if (ns > 1 && len > long_len) {  // split, if there are slots and items left
    unsigned long long need = (unsigned long long)(ns - 1) * nB, more = (unsigned long long)(ns - 1) * nt;
    unsigned long long at = atomicAdd((unsigned long long*)(ctr + 4), need);
    if (at + need <= (unsigned long long)max_slots &&
        atomicAdd((unsigned long long*)(ctr + 6), more) + more <= (unsigned long long)max_split)
      pbase = (int)at;
  }
  cell_nseg[B] = ns;
  cell_pbase[B] = pbase;
  if (pbase >= 0) {
    int x = atomicAdd(ctr + 8, (ns - 1) * nt);
    for (int k = 1; k < ns; k++)
      for (int t = 0; t < nt; t++) extra[x++] = make_int2(li, nf_code(k, t));
    atomicAdd(ctr + 2, ns - 1);
  }
}

// the partial sums of segments 1..ns-1 of split leaves added, in segment
// order, to the first segment's sums
__global__ void k_nf_combine(int64_t n, const int* __restrict__ leaf_of, const int* __restrict__ cb,
                             const int* __restrict__ ce, const int* __restrict__ cell_nseg,
                             const int* __restrict__ cell_pbase, const double4* __restrict__ part,
                             double4* nearbuf) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  int B = leaf_of[i];
  int ns = cell_nseg[B];
  if (ns <= 1 || cell_pbase[B] < 0) return;
  int nB = ce[B] - cb[B];
  const double4* pp = part + cell_pbase[B] + (i - cb[B]);
  double4 t = nearbuf[i];
#pragma unroll 4
  for (int k = 1; k < ns; k++) {
    double4 v = pp[(size_t)(k - 1) * nB];
    t.x += v.x;
    t.y += v.y;
    t.z += v.z;
    t.w += v.w;
  }
  nearbuf[i] = t;
}

// Builds c.nf for the current leaves and near-field list (on c.stream; the
// counters at c.counters[44..45] are cleared by the caller).
void plan_near_field(Ctx& c) {
  int nleaf = (int)c.nleaf;
  int64_t cnt = c.p2p.count;
  int max_nb = std::min(64, c.prm.n_leaf);
  int tiled = nf_tiled(c);
  ensure(c.ws, c.nf_cell_nseg, (size_t)c.ncell);
  ensure(c.ws, c.nf_cell_pbase, (size_t)c.ncell);
  // a list of len > K entries has ceil(len / K) segments, so the later segments
  // number fewer than cnt / K, with the smallest K of any system
  int64_t segs = cnt / nf_segment(c.nsys > 1 ? 1 : c.n, max_nb, tiled, 0);
  int64_t slots = std::min(NF_SLOTS, segs * 64);
  if (c.ws.limit || c.ws.arena) {
    // Where memory is limited: as many slots as fit beside the buffers still to come,
    // those of the M2L (up to a segment per 512 pairs) and, in a context's own
    // workspace, of the gradient; none, if need be.
    int64_t expansion = ncoef(c.p) * 16, segments = c.m2l.count / 512 + 1;
    int64_t later = 12 * c.ncell + segments * (8 + (c.p <= FMM_GPU_PMAX ? expansion : 0)) + c.n + 65536;
    int64_t fit;
    if (c.ws.arena) {
      fit = ((int64_t)(c.ws.arena_cap - c.ws.arena_used) - later) / 40;  // (8 bytes of extra items per slot)
    } else {
      later += 2 * c.ncell * expansion + 128 * c.n;
      fit = std::min(ceil_div(cnt, 4), ((int64_t)c.ws.limit - (int64_t)c.ws.bytes - later - later / 4) / 130);
      if ((int64_t)c.nf_part.cap > c.nf.max_slots) fit = std::max<int64_t>(fit, c.nf.max_slots);  // (held already)
    }
    slots = std::min(slots, std::max<int64_t>(fit, 0));
  }
  // (a split list has no more extra items than slots)
  int64_t split = std::min({NF_SPLIT, slots, segs * (tiled ? 64 / NF_TILE : 1)});
  int64_t extra_max = split + (tiled ? c.n / NF_TILE : 0);  // with tiles n_B / 8 of every leaf besides
  ensure(c.ws, c.nf_extra, (size_t)extra_max + 1);
  ensure(c.ws, c.nf_part, (size_t)slots + 1);
  int64_t waves = nleaf + (tiled ? c.n / NF_TILE : 0);
  int long_len = (int)(waves < NF_FULL ? cnt / NF_ITEMS : 2 * cnt / nleaf);
  int* ctr = c.counters.p + NF_COUNTERS;
  hipLaunchKernelGGL(k_nf_plan, dim3((unsigned)ceil_div(nleaf, 256)), dim3(256), 0, c.stream, c.leaves.p, nleaf,
                     c.c_begin.p, c.c_end.p, c.p2p.off.p, c.sys_off.p, c.nsys, max_nb, tiled, long_len,
                     (int)slots, (int)split, (int)extra_max, c.nf_cell_nseg.p, c.nf_cell_pbase.p, c.nf_extra.p, ctr);
  HIPCHK(hipGetLastError());
  c.nf = NfPlan{c.nf_cell_nseg.p, c.nf_cell_pbase.p, c.nf_extra.p, ctr + 8, nleaf,
                (int)(nleaf + extra_max), (int)slots};
}

void launch_near_field(Ctx& c) {
  if (c.nleaf <= 0) return;
  ensure(c.ws, c.nearbuf, (size_t)c.n);
  const int* leaves = c.leaves.p;
  // the plan's counters and the body-pair counts, read by fmm_stats
  unsigned long long* npairs = (unsigned long long*)(c.counters.p + NF_PAIRS);
  zero_fill(c, c.counters.p + NF_COUNTERS, (COUNTERS - NF_COUNTERS) * sizeof(int));
  plan_near_field(c);
  int nblk = (c.nf.max_items + LG_WAVES - 1) / LG_WAVES;
  unsigned grid = xcd_grid(nblk);
  double e2 = c.eps_soft * c.eps_soft;
  int gmax = c.prm.p2p_groups;
  if (!nf_tiled(c))
    hipLaunchKernelGGL(k_leaf_group, dim3(grid), dim3(64 * LG_WAVES), 0, c.stream, leaves, c.nf,
                       c.c_begin.p, c.c_end.p, c.p2p.off.p, c.p2p.src.p, c.pm.p, e2, c.nearbuf.p,
                       c.nf_part.p, npairs, gmax);
  else
    hipLaunchKernelGGL(k_near_fp64, dim3(grid), dim3(64 * LG_WAVES), 0, c.stream, leaves, c.nf, c.c_begin.p,
                       c.c_end.p, c.p2p.off.p, c.p2p.src.p, c.pm.p, e2, c.nearbuf.p, c.nf_part.p, npairs);
  HIPCHK(hipGetLastError());
  if (c.nf.max_slots > 0) {
    hipLaunchKernelGGL(k_nf_combine, dim3((unsigned)ceil_div(c.n, 256)), dim3(256), 0, c.stream, c.n,
                       c.leaf_of.p, c.c_begin.p, c.c_end.p, c.nf_cell_nseg.p, c.nf_cell_pbase.p, c.nf_part.p,
                       c.nearbuf.p);
    HIPCHK(hipGetLastError());
  }
}

// Far field by L2P (the leaf's local expansion shifted to the body:
// Phi = -Re L'_0^0, a = (-Re L'_1^1, -Im L'_1^1, Re L'_1^0)) plus the near
// field, summed in FP64 and written in the caller's order; one thread per body.
__global__ void __launch_bounds__(256) k_far_final(int p, int64_t n, const int* __restrict__ leaf_of,
                                                   const double* __restrict__ cx, const double* __restrict__ cy,
                                                   const double* __restrict__ cz, const double* __restrict__ loc,
                                                   const double4* __restrict__ pm,
                                                   const double4* __restrict__ nearbuf,
                                                   const int* __restrict__ perm, double* acc, double* pot) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  int B = leaf_of[i];
  double4 me = pm[i], nf = nearbuf[i];
  double ax, ay, az, ph;
  l2p_eval(p, loc + (size_t)B * ncoef(p) * 2, me.x - cx[B], me.y - cy[B], me.z - cz[B], ax, ay, az, ph);
  int64_t o = perm[i];
  acc[3 * o] = ax + nf.x;
  acc[3 * o + 1] = ay + nf.y;
  acc[3 * o + 2] = az + nf.z;
  pot[o] = ph + nf.w;
}

void launch_far_final(Ctx& c, double* acc, double* pot) {
  hipLaunchKernelGGL(k_far_final, dim3((unsigned)ceil_div(c.n, 256)), dim3(256), 0, c.stream, c.p, c.n,
                     c.leaf_of.p, c.c_cx.p, c.c_cy.p, c.c_cz.p, c.loc.p, c.pm.p, c.nearbuf.p, c.idx[0].p,
                     acc, pot);
  HIPCHK(hipGetLastError());
}

void launch_l2l(Ctx& c) { launch_l2l_buf(c, c.loc.p); }

void launch_l2l_buf(Ctx& c, double* loc) {
  size_t S = (size_t)(c.p + 1) * (c.p + 1);
  int G = sizeof(double2) * 9 * S <= 128 * 1024 ? 8 : 1;  // children per pass within 128 KB of LDS
  size_t lds = sizeof(double2) * (1 + G) * S;
  int tasks = G * ncoef(c.p), rounds = (int)ceil_div(tasks, L2L_T_MAX);
  int threads = (int)ceil_div(tasks, 64 * rounds) * 64;
  for (int level = 0; level < c.depth; level++) {  // parents at this level, children one below
    int first = c.lvl_first[level], count = c.lvl_count[level];
    hipLaunchKernelGGL(k_l2l, dim3(count), dim3(threads), lds, c.stream, c.p, first, count, c.c_child0.p,
                       c.c_nchild.p, c.c_cx.p, c.c_cy.p, c.c_cz.p, loc, G);
  }
  HIPCHK(hipGetLastError());
}

// ---- plain direct sum (FP64, compensated accumulation)
__device__ __forceinline__ void two_sum_acc(double& s, double& c, double v) {
  double t = s + v;
  double bp = t - s;
  c += (s - (t - bp)) + (v - bp);
  s = t;
}

// One workgroup of T threads per S sinks: the threads share the sources (a
// coalesced stride over the bodies), every source loaded serves the S sinks,
// whose positions are wave-uniform, and the threads' compensated sums are
// merged by two-sums at the end (wave, then workgroup; a fixed order).
// Bound by FP64 issue (about 60 instructions per pair).  A thread per sink
// left the chip idle where an error check has few sinks: 4096 sinks were 16
// workgroups, 275 ms over 2^20 sources (7.3 ms this way).
template <int S, int T>
__global__ void __launch_bounds__(T) k_direct(int64_t n, const double* __restrict__ pos,
                                              const double* __restrict__ mass, double eps2, int64_t nsink,
                                              const int32_t* __restrict__ sinks, double* __restrict__ acc,
                                              double* __restrict__ pot) {
  constexpr int W = T / 64;
  __shared__ double2 part[W][4 * S];
  int64_t s0 = (int64_t)blockIdx.x * S;
  int64_t id[S];
  double x[S], y[S], z[S];
#pragma unroll
  for (int k = 0; k < S; k++) {
    int64_t s = s0 + k < nsink ? s0 + k : nsink - 1;  // past the end: the last sink again, not written
    id[k] = sinks ? sinks[s] : s;
    x[k] = pos[3 * id[k]];
    y[k] = pos[3 * id[k] + 1];
    z[k] = pos[3 * id[k] + 2];
  }
  double sum[4 * S], cor[4 * S];
#pragma unroll
  for (int k = 0; k < 4 * S; k++) sum[k] = cor[k] = 0.0;
  for (int64_t j = threadIdx.x; j < n; j += T) {
    double jx = pos[3 * j], jy = pos[3 * j + 1], jz = pos[3 * j + 2], m = mass[j];
#pragma unroll
    for (int k = 0; k < S; k++) {
      double dx = jx - x[k], dy = jy - y[k], dz = jz - z[k];
      double d2 = fma(dx, dx, fma(dy, dy, fma(dz, dz, eps2)));
      bool ok = j != id[k] && d2 > 0.0 && d2 < INFINITY;
      double rinv = ok ? rsqrt_d(d2) : 0.0;
      double mr = m * rinv, mr3 = mr * rinv * rinv;
      two_sum_acc(sum[4 * k], cor[4 * k], mr3 * dx);
      two_sum_acc(sum[4 * k + 1], cor[4 * k + 1], mr3 * dy);
      two_sum_acc(sum[4 * k + 2], cor[4 * k + 2], mr3 * dz);
      two_sum_acc(sum[4 * k + 3], cor[4 * k + 3], -mr);
    }
  }
  int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
#pragma unroll
  for (int k = 0; k < 4 * S; k++) {
    for (int o = 32; o >= 1; o >>= 1) {
      double os = __shfl_xor(sum[k], o, 64), oc = __shfl_xor(cor[k], o, 64);
      two_sum_acc(sum[k], cor[k], os);
      cor[k] += oc;
    }
    if (lane == 0) part[wv][k] = make_double2(sum[k], cor[k]);
  }
  __syncthreads();
  int k = threadIdx.x;
  if (k < 4 * S && s0 + k / 4 < nsink) {
    double s = part[0][k].x, c = part[0][k].y;
    for (int w = 1; w < W; w++) {
      two_sum_acc(s, c, part[w][k].x);
      c += part[w][k].y;
    }
    int64_t o = s0 + k / 4;
    if ((k & 3) == 3)
      pot[o] = s + c;
    else
      acc[3 * o + (k & 3)] = s + c;
  }
}

// Up to DS_FEW sinks: one per workgroup of 1024 threads, so that 64 sinks
// still give 1024 wavefronts; more: four per workgroup of 256, a quarter of
// the source traffic per pair.
constexpr int64_t DS_FEW = 1024;

void direct_sum(int64_t n, const double* pos, const double* mass, double eps2, int64_t nsink,
                const int32_t* sinks, double* acc, double* pot, hipStream_t s) {
  if (nsink <= DS_FEW)
    hipLaunchKernelGGL((k_direct<1, 1024>), dim3((unsigned)nsink), dim3(1024), 0, s, n, pos, mass, eps2, nsink,
                       sinks, acc, pot);
  else
    hipLaunchKernelGGL((k_direct<4, 256>), dim3((unsigned)ceil_div(nsink, 4)), dim3(256), 0, s, n, pos, mass,
                       eps2, nsink, sinks, acc, pot);
  HIPCHK(hipGetLastError());
}

// ---- input validation (optional): non-finite positions, negative / NaN masses
__global__ void k_check(const double* pos, const double* mass, int64_t n, int* bad) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  bool ok = isfinite(pos[3 * i]) && isfinite(pos[3 * i + 1]) && isfinite(pos[3 * i + 2]) &&
            isfinite(mass[i]) && mass[i] >= 0.0;
  if (!ok) atomicOr(bad, 1);
}

bool check_inputs_dev(Ctx& c, const double* pos, const double* mass, int64_t n) {
  ensure(c.ws, c.counters, 64);
  int* bad = c.counters.p + 32;
  HIPCHK(hipMemsetAsync(bad, 0, sizeof(int), c.stream));
  hipLaunchKernelGGL(k_check, dim3((unsigned)ceil_div(n, 256)), dim3(256), 0, c.stream, pos, mass, n, bad);
  HIPCHK(hipGetLastError());
  HIPCHK(hipMemcpyAsync(c.hbuf, bad, sizeof(int), hipMemcpyDeviceToHost, c.stream));
  HIPCHK(hipStreamSynchronize(c.stream));
  return ((int*)c.hbuf)[0] == 0;
}

}  // namespace fmm
