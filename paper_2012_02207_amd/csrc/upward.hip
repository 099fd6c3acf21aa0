// Upward pass on gfx950: P2M at the leaves, M2M towards the root and the
// per-order norms P_k of every cell's multipole.
//
// P2M: M_n^m = sum_i m_i Y_n^m(x_i - z) over the cell's bodies (section 2.2,
// multipole-moment equation).  M2M shifts each child's moments to the parent
// centre with the regular addition theorem (section 2.1).  P_k^2 =
// sum_{m=-k..k} (k-m)!(k+m)! |M_k^m|^2 (section 2.3).  These values enter the
// acceptance test, so every sum runs sequentially in a fixed order with
// separately rounded products: bodies in sorted order, children in octant
// order, terms in (k, l) order.  A wavefront owns one cell: lanes evaluate the
// harmonics of different bodies (or children) into LDS, then lanes owning
// different coefficients accumulate over the bodies in order.
#include <hip/hip_runtime.h>

#include <climits>

#include "fmm_device.h"
#include "fmm_tables.h"

namespace fmm {

static __constant__ double c_fact[2 * FMM_TABLE_PMAX + 2];
static __constant__ double c_binom[FMM_TABLE_PMAX + 1][FMM_TABLE_PMAX + 1];
static bool g_up_tables[64] = {};  // per device

// Column m of the regular harmonics of (x, y, z), rounded as the defining
// two-term recurrences are written (no contraction),
//   Y_0^0 = 1, Y_n^n = -(x + i y) Y_{n-1}^{n-1} / (2n),
//   Y_n^m = ((2n-1) z Y_{n-1}^m - r^2 Y_{n-2}^m) / ((n+m)(n-m)):
// the diagonal Y_1^1 .. Y_m^m, then Y_n^m for n = m+1..p.  Lanes evaluate
// different columns (and bodies) in parallel.  The chain of a column is bound by
// latency, most of it the divisions', whose reciprocals leave the chain (div_by).
template <class Store>
__device__ inline void regular_column_exact(int p, int m, double x, double y, double z, Store store) {
  double r2 = (x * x + y * y) + z * z;
  double pr = 1.0, pi = 0.0;
  for (int n = 1; n <= m; n++) {
    double den = (double)(2 * n), rcp = rcp_newton(den);
    double tr = x * pr - y * pi;
    double ti = x * pi + y * pr;
    pr = div_by(-tr, den, rcp);
    pi = div_by(-ti, den, rcp);
  }
  store(m, pr, pi);
  double ar2 = 0.0, ai2 = 0.0, ar1 = pr, ai1 = pi;
  for (int n = m + 1; n <= p; n++) {
    double den = (double)((n + m) * (n - m)), rcp = rcp_newton(den);
    double k = (double)(2 * n - 1) * z;
    double nr = k * ar1, ni = k * ai1;
    if (n - 2 >= m) {
      double br = r2 * ar2, bi = r2 * ai2;
      nr = nr - br;
      ni = ni - bi;
    }
    double vr = div_by(nr, den, rcp), vi = div_by(ni, den, rcp);
    store(n, vr, vi);
    ar2 = ar1;
    ai2 = ai1;
    ar1 = vr;
    ai1 = vi;
  }
}

// P2M, a wavefront per leaf.  Bodies in batches of 64 / (p+1): a lane evaluates
// one column of one body's harmonics into LDS, as the real values of the order's
// coefficients (entry n^2: Re Y_n^0, n^2 + 2m - 1 and n^2 + 2m: Re, Im Y_n^m);
// then each lane adds up to V of the (p+1)^2 values over the batch in sorted body
// order (Im M_n^0 is 0).  Bound by FP64 issue.  A workgroup of 256 threads per
// leaf, whose lanes ran the two loops of unequal columns one after the other and
// mostly idled in the sums, took 471 us at N = 2^20, p = 10, this one 350.
constexpr int P2M_WAVES = 4;

__host__ __device__ inline int p2m_batch(int p) { return 64 / (p + 1); }

// Column m of the harmonics of (x, y, z), as regular_column_exact, its diagonal
// and its vertical steps in one loop, so that lanes of different columns keep
// step.
template <class Store>
__device__ inline void regular_column_lockstep(int p, int m, double x, double y, double z, Store store) {
  double r2 = (x * x + y * y) + z * z;
  double ar1 = 1.0, ai1 = 0.0, ar2 = 0.0, ai2 = 0.0;  // the last value, and the one before it in the column
  if (m == 0) store(0, 1.0, 0.0);
  for (int n = 1; n <= p; n++) {
    bool diag = n <= m;
    double den = diag ? (double)(2 * n) : (double)((n + m) * (n - m)), rcp = rcp_newton(den);
    double k = diag ? x : (double)(2 * n - 1) * z;
    double br = (diag ? y : r2) * (diag ? ai1 : ar2), bi = (diag ? y : r2) * (diag ? ar1 : ai2);
    double nr = k * ar1, ni = k * ai1;
    if (diag) {
      nr = -(nr - br);
      ni = -(ni + bi);
    } else if (n - 2 >= m) {
      nr = nr - br;
      ni = ni - bi;
    }
    ar2 = diag ? 0.0 : ar1;
    ai2 = diag ? 0.0 : ai1;
    ar1 = div_by(nr, den, rcp);
    ai1 = div_by(ni, den, rcp);
    if (n >= m) store(n, ar1, ai1);
  }
}

// (leaves of up to `most` bodies)
template <int V>
__global__ void __launch_bounds__(64 * P2M_WAVES) k_p2m(int p, const int* __restrict__ leaves, int nleaves, int most,
                                                        const int* __restrict__ cb, const int* __restrict__ ce,
                                                        const double4* __restrict__ pm, const double* __restrict__ cx,
                                                        const double* __restrict__ cy, const double* __restrict__ cz,
                                                        double* __restrict__ mult) {
  extern __shared__ double lds[];
  int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  int li = blockIdx.x * P2M_WAVES + wv;
  if (li >= nleaves) return;
  int c = leaves[li];
  int S = (p + 1) * (p + 1), batch = p2m_batch(p);
  double* val = lds + (size_t)wv * S * batch;  // [body][value]
  double x0 = cx[c], y0 = cy[c], z0 = cz[c];
  int b = cb[c], e = ce[c];
  if (e - b > most) return;
  int hb = lane / (p + 1), hm = lane - hb * (p + 1);  // harmonic lane: body hb, column hm
  double sum[V];
#pragma unroll
  for (int v = 0; v < V; v++) sum[v] = 0.0;
  for (int i0 = b; i0 < e; i0 += batch) {
    int cnt = min(batch, e - i0);
    bool act = hb < cnt;
    double4 q = pm[act ? i0 + hb : i0];
    __builtin_amdgcn_wave_barrier();
    if (act)
      regular_column_lockstep(p, hm, q.x - x0, q.y - y0, q.z - z0, [&](int n, double vr, double vi) {
        double* w = val + hb * S + n * n + 2 * hm;
        if (hm > 0) {
          w[-1] = vr;
          w[0] = vi;
        } else {
          w[0] = vr;
        }
      });
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0): the batch is visible to the wave
    for (int j = 0; j < cnt; j++) {
      double m = __shfl(q.w, j * (p + 1), 64);
#pragma unroll
      for (int v = 0; v < V; v++) {
        double t = m * val[j * S + min(lane + 64 * v, S - 1)];
        sum[v] = sum[v] + t;
      }
    }
    __builtin_amdgcn_wave_barrier();
  }
  double* out = mult + (size_t)c * ncoef(p) * 2;
#pragma unroll
  for (int v = 0; v < V; v++) {
    int k = lane + 64 * v;
    if (k < S) {
      int n = both_sign_n(k), j = k - n * n, m = (j + 1) >> 1;
      out[2 * cidx(n, m) + (j > 0 && !(j & 1) ? 1 : 0)] = sum[v];
      if (j == 0) out[2 * cidx(n, 0) + 1] = 0.0;
    }
  }
}

// P2M of the leaves of more than `most` bodies, a workgroup per leaf: the wavefronts
// share the harmonics of a batch and then the values, each summed over the batch in
// sorted body order as above.  One wavefront takes 4 ms for a leaf of 1000 bodies
// at p = 30, long after all others have ended.
constexpr int P2M_WIDE = 8;
constexpr int64_t P2M_FULL = 2048;  // leaves that fill the chip with a wavefront each

__global__ void __launch_bounds__(64 * P2M_WIDE) k_p2m_wide(int p, const int* __restrict__ leaves, int most,
                                                            const int* __restrict__ cb, const int* __restrict__ ce,
                                                            const double4* __restrict__ pm,
                                                            const double* __restrict__ cx,
                                                            const double* __restrict__ cy,
                                                            const double* __restrict__ cz, double* __restrict__ mult) {
  extern __shared__ double lds[];
  int c = leaves[blockIdx.x];
  int b = cb[c], e = ce[c];
  if (e - b <= most) return;
  constexpr int T = 64 * P2M_WIDE;
  int tid = threadIdx.x, wv = tid >> 6, lane = tid & 63;
  int S = (p + 1) * (p + 1), per = p2m_batch(p), batch = per * P2M_WIDE;
  double* val = lds;                   // [body][value]
  double* mass = lds + (size_t)S * batch;
  double x0 = cx[c], y0 = cy[c], z0 = cz[c];
  int hl = lane / (p + 1), hm = lane - hl * (p + 1), hb = wv * per + hl;  // body hb of the batch, column hm
  constexpr int V = ((FMM_TABLE_PMAX + 1) * (FMM_TABLE_PMAX + 1) + T - 1) / T;
  double sum[V];
#pragma unroll
  for (int v = 0; v < V; v++) sum[v] = 0.0;
  for (int i0 = b; i0 < e; i0 += batch) {
    int cnt = min(batch, e - i0);
    if (hl < per && hb < cnt) {
      double4 q = pm[i0 + hb];
      if (hm == 0) mass[hb] = q.w;
      regular_column_lockstep(p, hm, q.x - x0, q.y - y0, q.z - z0, [&](int n, double vr, double vi) {
        double* w = val + hb * S + n * n + 2 * hm;
        if (hm > 0) {
          w[-1] = vr;
          w[0] = vi;
        } else {
          w[0] = vr;
        }
      });
    }
    __syncthreads();
#pragma unroll
    for (int v = 0; v < V; v++) {
      int k = tid + T * v;
      if (k < S)
#pragma unroll 4
        for (int j = 0; j < cnt; j++) {
          double t = mass[j] * val[j * S + k];
          sum[v] = sum[v] + t;
        }
    }
    __syncthreads();
  }
  double* out = mult + (size_t)c * ncoef(p) * 2;
#pragma unroll
  for (int v = 0; v < V; v++) {
    int k = tid + T * v;
    if (k < S) {
      int n = both_sign_n(k), j = k - n * n, m = (j + 1) >> 1;
      out[2 * cidx(n, m) + (j > 0 && !(j & 1) ? 1 : 0)] = sum[v];
      if (j == 0) out[2 * cidx(n, 0) + 1] = 0.0;
    }
  }
}

// M2M, one workgroup per parent.  The children's harmonics Y_k^l(z_c - z_P)
// and moments M_j^q are laid out in LDS for both signs of their order
// (entry n(n+1) + m, m = -n..n, the negative orders from the stored ones by
// the conjugate symmetry, exact), so that every sum is a branch-free loop in
// the defining order.  Each (child, coefficient) pair is a task: the child's
// shifted moment summed over k, then l ascending, products rounded
// separately; the parent's coefficient then adds its children's sums in
// octant order.  A sum is at most p + 1 terms of one child long, not eight
// children long, and the workgroup has a thread for (almost) every task, so a
// level's launch, bound by the chain of its longest sum, is short: with 128
// threads and five tasks each a launch took 47 us at p = 10 whatever the
// level of up to a thousand parents (16 us now), and at p = 20, a child at a
// time, 334 us (60).
constexpr int M2M_T = 128;                 // threads of k_m2m_stream
constexpr int M2M_ALL_CHILDREN_PMAX = 22;  // the eight-children layout up to this order (135 KB of LDS)
constexpr int M2M_T_MAX = 1024;
constexpr int M2M_TASKS = (8 * ncoef(M2M_ALL_CHILDREN_PMAX) + M2M_T_MAX - 1) / M2M_T_MAX;

__global__ void __launch_bounds__(M2M_T_MAX) k_m2m(int p, int first, int count, const int* __restrict__ c0,
                                                    const int* __restrict__ nch, const double* __restrict__ cx,
                                                    const double* __restrict__ cy, const double* __restrict__ cz,
                                                    double* mult) {
  extern __shared__ double lds[];
  const int M2M_T = blockDim.x;
  int c = first + blockIdx.x;
  if (blockIdx.x >= count || nch[c] == 0) return;
  int nc = ncoef(p);
  int S = (p + 1) * (p + 1);
  int k0 = c0[c], kn = nch[c];
  double2* Yx = (double2*)lds;  // [child][S]
  double2* Mx = Yx + 8 * S;     // [child][S]
  int t = threadIdx.x;
  for (int u = t; u < kn * (p + 1); u += M2M_T) {  // harmonics, both signs of l
    int j = u / (p + 1), m = u - j * (p + 1);
    int ch = k0 + j;
    double2* Y = Yx + j * S;
    double sg = (m & 1) ? -1.0 : 1.0;
    regular_column_exact(p, m, cx[ch] - cx[c], cy[ch] - cy[c], cz[ch] - cz[c],
                         [&](int n, double vr, double vi) {
                           Y[n * n + n + m] = make_double2(vr, vi);
                           if (m > 0) Y[n * n + n - m] = make_double2(sg * vr, -sg * vi);
                         });
  }
  const double* src = mult + (size_t)k0 * nc * 2;
  for (int u = t; u < kn * S; u += M2M_T) {  // moments, both signs of q
    int j = u / S, r = u - j * S;
    int n = both_sign_n(r);
    int q = r - n * n - n;
    const double* cm = src + (size_t)j * nc * 2;
    int aq = q < 0 ? -q : q;
    double a = cm[2 * cidx(n, aq)], bb = cm[2 * cidx(n, aq) + 1];
    if (q < 0) {
      double sg = (aq & 1) ? -1.0 : 1.0;
      a = sg * a;
      bb = -sg * bb;
    }
    Mx[u] = make_double2(a, bb);
  }
  __syncthreads();
  // per-child sums, held in registers until every task has read the tables
  double pr[M2M_TASKS], pi[M2M_TASKS];
#pragma unroll
  for (int w = 0; w < M2M_TASKS; w++) {
    pr[w] = pi[w] = 0.0;
    int u = t + M2M_T * w;
    if (u < kn * nc) {
      int j, n, m;
      child_task(u, kn, j, n, m);
      const double2* Y = Yx + j * S;
      const double2* M = Mx + j * S;
      double sr = 0.0, si = 0.0;
      for (int k = 0; k <= n; k++) {
        int jj = n - k;
        int lo = max(-k, m - jj), hi = min(k, m + jj);
        const double2* Yk = Y + k * k + k + lo;
        const double2* Mj = M + jj * jj + jj + m - lo;
        int cnt = hi - lo + 1;
#pragma unroll 4
        for (int r = 0; r < cnt; r++) {  // l = lo + r
          double2 a = Yk[r], bq = Mj[-r];
          double tr = a.x * bq.x - a.y * bq.y;
          double ti = a.x * bq.y + a.y * bq.x;
          sr = sr + tr;
          si = si + ti;
        }
      }
      pr[w] = sr;
      pi[w] = si;
    }
  }
  __syncthreads();
  double2* part = Yx;  // [child][coefficient], over the harmonics
#pragma unroll
  for (int w = 0; w < M2M_TASKS; w++) {
    int u = t + M2M_T * w;
    if (u < kn * nc) {
      int j, n, m;
      child_task(u, kn, j, n, m);
      part[j * nc + cidx(n, m)] = make_double2(pr[w], pi[w]);
    }
  }
  __syncthreads();
  double* out = mult + (size_t)c * nc * 2;
  for (int q = t; q < nc; q += M2M_T) {
    double sr = 0.0, si = 0.0;
    for (int j = 0; j < kn; j++) {
      double2 v = part[j * nc + q];
      sr = sr + v.x;
      si = si + v.y;
    }
    out[2 * q] = sr;
    out[2 * q + 1] = si;
  }
}

// threads for the 8 ncoef(p) tasks of eight children in the fewest rounds
static int m2m_threads(int p) {
  int tasks = 8 * ncoef(p), rounds = (int)ceil_div(tasks, M2M_T_MAX);
  return (int)ceil_div(tasks, 64 * rounds) * 64;
}

size_t m2m_lds_bytes(int p) { return sizeof(double2) * 2 * 8 * (size_t)(p + 1) * (p + 1); }

// The same M2M with one child at a time in LDS (harmonics and moments of that
// child only), for the orders whose eight children do not fit: each lane sums
// a child's shifted moment (k, then l) and adds it to its running coefficient
// child by child in octant order, so it rounds exactly as k_m2m.
constexpr int M2M_SMAXK = (ncoef(FMM_TABLE_PMAX) + M2M_T - 1) / M2M_T;

__global__ void __launch_bounds__(M2M_T) k_m2m_stream(int p, int first, int count, const int* c0,
                                                       const int* nch, const double* cx, const double* cy,
                                                       const double* cz, double* mult) {
  extern __shared__ double lds[];
  int c = first + blockIdx.x;
  if (blockIdx.x >= count || nch[c] == 0) return;
  int nc = ncoef(p);
  int S = (p + 1) * (p + 1);
  int k0 = c0[c], kn = nch[c];
  double2* Y = (double2*)lds;  // [S] harmonics of the current child
  double2* Mx = Y + S;         // [S] its moments, both signs of q
  int t = threadIdx.x;
  double sr[M2M_SMAXK], si[M2M_SMAXK];
  for (int q = 0; q < M2M_SMAXK; q++) sr[q] = si[q] = 0.0;
  for (int j = 0; j < kn; j++) {
    int ch = k0 + j;
    for (int m = t; m <= p; m += M2M_T) {
      double sg = (m & 1) ? -1.0 : 1.0;
      regular_column_exact(p, m, cx[ch] - cx[c], cy[ch] - cy[c], cz[ch] - cz[c],
                           [&](int n, double vr, double vi) {
                             Y[n * n + n + m] = make_double2(vr, vi);
                             if (m > 0) Y[n * n + n - m] = make_double2(sg * vr, -sg * vi);
                           });
    }
    const double* cm = mult + (size_t)ch * nc * 2;
    for (int r = t; r < S; r += M2M_T) {
      int n = both_sign_n(r);
      int q = r - n * n - n;
      int aq = q < 0 ? -q : q;
      double a = cm[2 * cidx(n, aq)], bb = cm[2 * cidx(n, aq) + 1];
      if (q < 0) {
        double sg = (aq & 1) ? -1.0 : 1.0;
        a = sg * a;
        bb = -sg * bb;
      }
      Mx[r] = make_double2(a, bb);
    }
    __syncthreads();
    for (int q = 0; q < M2M_SMAXK; q++) {
      int u = t + M2M_T * q;
      if (u >= nc) break;
      int n, m;
      coef_nm(u, n, m);
      double ar = 0.0, ai = 0.0;  // this child's sum, added to the parent's below
      for (int k = 0; k <= n; k++) {
        int jj = n - k;
        int lo = max(-k, m - jj), hi = min(k, m + jj);
        const double2* Yk = Y + k * k + k + lo;
        const double2* Mj = Mx + jj * jj + jj + m - lo;
        int cnt = hi - lo + 1;
        for (int r = 0; r < cnt; r++) {  // l = lo + r
          double2 a = Yk[r], bq = Mj[-r];
          double tr = a.x * bq.x - a.y * bq.y;
          double ti = a.x * bq.y + a.y * bq.x;
          ar = ar + tr;
          ai = ai + ti;
        }
      }
      sr[q] = sr[q] + ar;
      si[q] = si[q] + ai;
    }
    __syncthreads();
  }
  double* out = mult + (size_t)c * nc * 2;
  for (int q = 0; q < M2M_SMAXK; q++) {
    int u = t + M2M_T * q;
    if (u < nc) {
      out[2 * u] = sr[q];
      out[2 * u + 1] = si[q];
    }
  }
}


// P_k = sqrt( (k!)^2 |M_k^0|^2 + sum_{m=1..k} 2 (k-m)!(k+m)! |M_k^m|^2 ), and the
// product C(p, k) P_k used by the acceptance test
__global__ void k_pk(int p, int ncell, const double* mult, double* pk, double* pkb) {
  int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= (int64_t)ncell * (p + 1)) return;
  int c = (int)(t / (p + 1)), k = (int)(t % (p + 1));
  const double* M = mult + (size_t)c * ncoef(p) * 2;
  double acc = 0.0;
  for (int m = 0; m <= k; m++) {
    double re = M[2 * cidx(k, m)], im = M[2 * cidx(k, m) + 1];
    double w = (m == 0) ? (c_fact[k] * c_fact[k]) : (2.0 * (c_fact[k - m] * c_fact[k + m]));
    acc = acc + w * (re * re + im * im);
  }
  double P = sqrt(acc);
  pk[t] = P;
  pkb[t] = c_binom[p][k] * P;
}

// M2M from the deepest parents to the roots over the multipole buffer `mult`
void m2m_levels(Ctx& c, double* mult) {
  for (int level = c.depth - 1; level >= 0; level--) {
    int first = c.lvl_first[level], count = c.lvl_count[level];
    if (c.p <= M2M_ALL_CHILDREN_PMAX)
      hipLaunchKernelGGL(k_m2m, dim3(count), dim3(m2m_threads(c.p)), m2m_lds_bytes(c.p), c.stream, c.p, first, count,
                         c.c_child0.p, c.c_nchild.p, c.c_cx.p, c.c_cy.p, c.c_cz.p, mult);
    else
      hipLaunchKernelGGL(k_m2m_stream, dim3(count), dim3(M2M_T), m2m_lds_bytes(c.p) / 8, c.stream, c.p, first,
                         count, c.c_child0.p, c.c_nchild.p, c.c_cx.p, c.c_cy.p, c.c_cz.p, mult);
    HIPCHK(hipGetLastError());
  }
}

void upload_up_tables() {
  int dev = 0;
  HIPCHK(hipGetDevice(&dev));
  if (g_up_tables[dev & 63]) return;
  HIPCHK(hipMemcpyToSymbol(HIP_SYMBOL(c_fact), fmm_fact_table, sizeof(fmm_fact_table)));
  HIPCHK(hipMemcpyToSymbol(HIP_SYMBOL(c_binom), fmm_binom_table, sizeof(fmm_binom_table)));
  g_up_tables[dev & 63] = true;
}

void upward_pass(Ctx& c) {
  upload_up_tables();
  int p = c.p, nc = (int)c.ncell;
  ensure(c.ws, c.mult, (size_t)nc * ncoef(p) * 2);
  ensure(c.ws, c.pk, (size_t)nc * (p + 1));
  // the leaf list and count come from the tree build, so nothing here waits
  // for the device
  expansions_up(c);
}

// P2M at the leaves (the list from the tree build), M2M to the roots, P_k
void expansions_up(Ctx& c) {
  hipStream_t s = c.stream;
  int p = c.p, nc = (int)c.ncell;
  int S = (p + 1) * (p + 1);
  // Leaves of more than 64 bodies where the leaves are few, of more than 512 where
  // they fill the chip, take a workgroup each; there are none unless n_leaf is
  // larger, or bodies coincide to the last level.
  int most = c.nleaf < P2M_FULL ? 64 : 512;
  bool wide = c.prm.n_leaf > most || c.depth == FMM_MAX_LEVEL;
  auto p2m = S <= 2 * 64 ? k_p2m<2> : S <= 4 * 64 ? k_p2m<4> : S <= 9 * 64 ? k_p2m<9> : k_p2m<16>;
  hipLaunchKernelGGL(p2m, dim3((unsigned)ceil_div(c.nleaf, P2M_WAVES)), dim3(64 * P2M_WAVES),
                     sizeof(double) * S * p2m_batch(p) * P2M_WAVES, s, p, c.leaves.p, (int)c.nleaf,
                     wide ? most : INT_MAX, c.c_begin.p, c.c_end.p, c.pm.p, c.c_cx.p, c.c_cy.p, c.c_cz.p, c.mult.p);
  if (wide)
    hipLaunchKernelGGL(k_p2m_wide, dim3((unsigned)c.nleaf), dim3(64 * P2M_WIDE),
                       sizeof(double) * (S + 1) * p2m_batch(p) * P2M_WIDE, s, p, c.leaves.p, most, c.c_begin.p,
                       c.c_end.p, c.pm.p, c.c_cx.p, c.c_cy.p, c.c_cz.p, c.mult.p);
  HIPCHK(hipGetLastError());
  m2m_levels(c, c.mult.p);
  int64_t npk = (int64_t)nc * (p + 1);
  ensure(c.ws, c.pkb, (size_t)npk);
  hipLaunchKernelGGL(k_pk, dim3((unsigned)ceil_div(npk, 256)), dim3(256), 0, s, p, nc, c.mult.p, c.pk.p,
                     c.pkb.p);
  HIPCHK(hipGetLastError());
  if (c.prm.precision == FMM_MIXED && mixed_supported(p)) launch_normalize32(c);
}

}  // namespace fmm
