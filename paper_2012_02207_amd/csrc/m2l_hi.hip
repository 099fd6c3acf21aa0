// Rotation-accelerated M2L for any order up to 30 (section 2.4), FP64, on the
// matrix cores.
//
// The same operator as k_m2l_fp64 (m2l.hip): for a directed pair A -> B the
// source moments are rotated about z by alpha = pi/2 - phi, their x and z
// swapped, rotated about z by -theta and swapped again, so that R = z_B - z_A
// lies along +z; translated along z, where only T_j^0(r z) = j!/r^{j+1} is
// non-zero; then rotated back with the transposed sequence in the scaled basis
// Lhat_n^m = L_n^m / ((n-m)!(n+m)!).  W_n, the swap of order n, couples Re^m with
// Re^m' only when m + m' + n is even and Im^m with Im^m' when it is odd, so it is
// four blocks: the Re or the Im parts, input orders m of one parity.
//
// The register-resident kernel holds a whole expansion per lane, which stops
// fitting beyond p = 16 (441 values at p = 20).  Here a workgroup of eight
// wavefronts takes 16 NT pairs of one sink at a time, and each wavefront owns
// four orders, n = w, 15 - w, 16 + w, 31 - w, whose swap matrices stay in its
// registers.  A swap is a product of a constant block (up to 16 x 16) with the
// coefficients of 16 pairs: v_mfma_f64_16x16x4f64, the pairs as columns.  Its
// result, row 4r + lane/16 of column lane%16 in register r, is the operand layout
// of the next product, and the Re and the Im block of a parity have the same
// rows, so rotation, swap, rotation and swap of an order run in registers, from
// the moments' loads on; only the translation, which couples the orders, goes
// through LDS.
// Measured at N = 10^5, p = 20, err_tol = 1e-7 (9.1e5 pairs): 4.34 ms alone; a
// wavefront per pair with its coefficients shared by the lanes, two loads per
// multiply-add, took 28.2 ms.
#include <hip/hip_runtime.h>

#include <vector>

#include "fmm_device.h"
#include "fmm_tables.h"

namespace fmm {

namespace hi {

constexpr int PMAX = FMM_TABLE_PMAX;  // orders with swap tables (section 2.4: p <= 30)
constexpr int WAVES = 8;
constexpr int SLOTS = 4;  // orders per wavefront; slot s: 8s <= n < 8s + 8, up to s + 1 K-steps of four orders m

typedef double v4d __attribute__((ext_vector_type(4)));

// order of slot s of wavefront w
__host__ __device__ constexpr int slot_order(int s, int w) { return (s & 1) ? 8 * s + 7 - w : 8 * s + w; }

// swap block of (n, part, parity of the input order) in operand layout: K-step
// ks, lane l: output row l % 16, input order m = parity + 2 (4 ks + l / 16)
__host__ __device__ constexpr int frag_index(int n, int part, int par, int ks) {
  return ((n * 2 + part) * 2 + par) * 4 + ks;
}

}  // namespace hi

static __device__ double g_swap_frag[hi::frag_index(hi::PMAX + 1, 0, 0, 0) * 64];
static __constant__ double c_fact_hi[2 * hi::PMAX + 2];
static bool g_hi_tables[64] = {};  // per device

// One order of one wavefront: its swap blocks, and the coefficients of 16 NT
// pairs as operands.  c[part][b][t][ks]: parity slot b of tile t; the orders m of
// slot b have parity b before the first swap and after the second, b ^ (n & 1)
// between them.
template <int SLOT, int NT>
struct HiOrder {
  static constexpr int KS = SLOT + 1;
  double w[2][2][KS];

  __device__ __forceinline__ void load_swap(int n, int lane) {
#pragma unroll
    for (int part = 0; part < 2; part++)
#pragma unroll
      for (int b = 0; b < 2; b++)
#pragma unroll
        for (int ks = 0; ks < KS; ks++)
          w[part][b][ks] = g_swap_frag[hi::frag_index(n, part, b, ks) * 64 + lane];
  }

  // c <- W c; odd: the input of slot b has parity 1 - b.  The Im parts change
  // slots, so that a slot's Re and Im rows stay the same orders m.
  template <bool ODD>
  __device__ __forceinline__ void swap(double (&c)[2][2][NT][KS]) const {
#pragma unroll
    for (int part = 0; part < 2; part++)
#pragma unroll
      for (int t = 0; t < NT; t++) {
        hi::v4d d[2];
#pragma unroll
        for (int b = 0; b < 2; b++) {
          d[b] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
          for (int ks = 0; ks < KS; ks++)
            d[b] = __builtin_amdgcn_mfma_f64_16x16x4f64(w[part][ODD ? 1 - b : b][ks], c[part][b][t][ks], d[b], 0, 0, 0);
        }
#pragma unroll
        for (int b = 0; b < 2; b++)
#pragma unroll
          for (int ks = 0; ks < KS; ks++) c[part][b ^ part][t][ks] = d[b][ks];
      }
  }

  // rotation about z, (C, S)_m <- (C cos ma - S sin ma, C sin ma + S cos ma), with
  // (cos ma, sin ma) of pair col at tab[m * 16 NT + col]; flip: slot b holds
  // parity 1 - b; sgn = -1 rotates by -a
  __device__ __forceinline__ static void rotate(double (&c)[2][2][NT][KS], const double2* tab, int p, int flip,
                                                double sgn, int lane) {
#pragma unroll
    for (int b = 0; b < 2; b++)
#pragma unroll
      for (int ks = 0; ks < KS; ks++) {
        int m = min((b ^ flip) + 2 * (4 * ks + (lane >> 4)), p);  // (rows past the order are zero)
#pragma unroll
        for (int t = 0; t < NT; t++) {
          double2 cs = tab[m * 16 * NT + 16 * t + (lane & 15)];
          double sn = sgn * cs.y, C = c[0][b][t][ks], S = c[1][b][t][ks];
          c[0][b][t][ks] = fma(C, cs.x, -S * sn);
          c[1][b][t][ks] = fma(C, sn, S * cs.x);
        }
      }
  }

  // rotation, swap, rotation, swap: forward (by a, then b) or back (by -b after
  // the first swap, by -a after the second)
  template <bool BACK>
  __device__ __forceinline__ void turn(double (&c)[2][2][NT][KS], int n, int p, const double2* ta, const double2* tb,
                                       int lane) const {
    int odd = n & 1;
    if (!BACK) rotate(c, ta, p, 0, 1.0, lane);
    swap<false>(c);
    rotate(c, tb, p, odd, BACK ? -1.0 : 1.0, lane);
    if (odd)
      swap<true>(c);
    else
      swap<false>(c);
    if (BACK) rotate(c, ta, p, 0, -1.0, lane);
  }

  // the moments of the pairs' sources, turned, to v (row n^2 + real-basis entry,
  // rs values apart)
  __device__ __forceinline__ void forward(int n, int p, const double2* const (&M)[NT], const double2* ta,
                                          const double2* tb, double* v, int rs, int lane) const {
    double c[2][2][NT][KS];
#pragma unroll
    for (int b = 0; b < 2; b++)
#pragma unroll
      for (int ks = 0; ks < KS; ks++) {
        int m = b + 2 * (4 * ks + (lane >> 4));
#pragma unroll
        for (int t = 0; t < NT; t++) {
          double2 x = M[t][cidx(n, min(m, n))];
          c[0][b][t][ks] = m <= n ? x.x : 0.0;
          c[1][b][t][ks] = m <= n && m > 0 ? x.y : 0.0;
        }
      }
    turn<false>(c, n, p, ta, tb, lane);
#pragma unroll
    for (int b = 0; b < 2; b++)
#pragma unroll
      for (int ks = 0; ks < KS; ks++) {
        int m = b + 2 * (4 * ks + (lane >> 4));
        if (m <= n) {
#pragma unroll
          for (int t = 0; t < NT; t++) {
            double* o = v + (n * n + 2 * m) * rs + 16 * t + (lane & 15);
            if (m > 0) {
              o[-rs] = c[0][b][t][ks];
              o[0] = c[1][b][t][ks];
            } else {
              o[0] = c[0][b][t][ks];
            }
          }
        }
      }
  }

  // the translated coefficients from v, turned back and added over the pairs to
  // acc (real basis)
  __device__ __forceinline__ void back(int n, int p, const double2* ta, const double2* tb, const double* v, int rs,
                                       double* acc, int lane) const {
    double c[2][2][NT][KS];
#pragma unroll
    for (int b = 0; b < 2; b++)
#pragma unroll
      for (int ks = 0; ks < KS; ks++) {
        int m = b + 2 * (4 * ks + (lane >> 4));
        bool ok = m <= n && m + n <= p;  // (the translation reaches no others)
#pragma unroll
        for (int t = 0; t < NT; t++) {
          const double* o = v + (n * n + 2 * min(m, n)) * rs + 16 * t + (lane & 15);
          c[0][b][t][ks] = ok ? o[m > 0 ? -rs : 0] : 0.0;
          c[1][b][t][ks] = ok && m > 0 ? o[0] : 0.0;
        }
      }
    turn<true>(c, n, p, ta, tb, lane);
#pragma unroll
    for (int b = 0; b < 2; b++)
#pragma unroll
      for (int ks = 0; ks < KS; ks++) {
        int m = b + 2 * (4 * ks + (lane >> 4));
#pragma unroll
        for (int part = 0; part < 2; part++) {
          double s = c[part][b][0][ks];
#pragma unroll
          for (int t = 1; t < NT; t++) s += c[part][b][t][ks];
          s += dpp_read<0x140>(s);  // over the 16 lanes of the row
          s += dpp_read<0x141>(s);
          s += dpp_read<0x4E>(s);
          s += dpp_read<0xB1>(s);
          if ((lane & 15) == 0 && m <= n && m >= part) acc[n * n + (part ? 2 * m : m > 0 ? 2 * m - 1 : 0)] += s;
        }
      }
  }
};

// M2L of the list of each sink (a workgroup per sink, or per segment of a long
// list, see M2lSeg), or of the listed sinks; with B >= first_lo only the sources
// below first_lo are taken (the FP64 part of mixed precision).
// NT tiles of 16 pairs at a time, orders up to PM.  WHOLE: the plan has no extra
// items, and a workgroup adds up the segments of a long list itself.
template <int NT, int PM, bool WHOLE>
__global__ void __launch_bounds__(64 * hi::WAVES) k_m2l_hi(int p, int ncell, int first_lo,
                                                           const int* __restrict__ sinks,
                                                           const int* __restrict__ nsinks,
                                                           const int* __restrict__ off, const int* __restrict__ src,
                                                           const double* __restrict__ cx, const double* __restrict__ cy,
                                                           const double* __restrict__ cz,
                                                           const double* __restrict__ mult, double* __restrict__ loc,
                                                           M2lSeg sg) {
  extern __shared__ double lds[];
  constexpr int PT = 16 * NT, RS = PT + 1;  // pairs at a time; row stride in V
  constexpr int T_MAX = PM + 1;
  const int S = (p + 1) * (p + 1), NC = ncoef(p);
  double* V = lds;
  double2* ta = (double2*)(lds + ((S * RS + 1) & ~1));  // (cos m alpha, sin m alpha) [m][pair]
  double2* tb = ta + (p + 1) * PT;                      // of -theta
  double* rin = (double*)(tb + (p + 1) * PT);           // 1 / r of each pair, 0 past the end of the list
  double* acc = rin + PT;                               // [S] the sink's expansion
  int* ids = (int*)(acc + S);                           // sources of the pairs
  const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  HiOrder<0, NT> o0;
  HiOrder<1, NT> o1;
  HiOrder<2, NT> o2;
  HiOrder<3, NT> o3;
  const int n0 = hi::slot_order(0, wv), n1 = hi::slot_order(1, wv), n2 = hi::slot_order(2, wv),
            n3 = hi::slot_order(3, wv);
  if (n0 <= p) o0.load_swap(n0, lane);
  if (n1 <= p) o1.load_swap(n1, lane);
  if (n2 <= p) o2.load_swap(n2, lane);
  if (PM >= 24 && n3 <= p) o3.load_swap(n3, lane);
  int count = sinks ? *nsinks : sg.nseg ? ncell + *sg.nextra : ncell;
  for (int it = blockIdx.x; it < count; it += gridDim.x) {
    int B = sinks ? sinks[it] : it, seg = 0;
    if (!sinks && it >= ncell) {
      int2 x = sg.extra[it - ncell];
      B = x.x;
      seg = x.y;
    }
    int b0 = off[B], e0 = off[B + 1];
    if (B >= first_lo) e0 = split_point(src, b0, e0, first_lo);
    double* out = loc + (size_t)B * NC * 2;
    if (b0 == e0) {
      for (int k = tid; k < NC * 2; k += 64 * hi::WAVES) out[k] = 0.0;
      continue;
    }
    double bx = cx[B], by = cy[B], bz = cz[B];
    int b = b0, e = e0, K = 0;
    if (sg.nseg && sg.nseg[B] > 1) {
      K = sg.seglen ? sg.seglen[B] : sg.K;
      b += seg * K;
      e = min(e0, b + K);
      if (seg > 0) out = sg.part + (size_t)(sg.pbase[B] + seg - 1) * NC * 2;
    }
    while (true) {
      __syncthreads();  // the previous sums have been read
      for (int k = tid; k < S; k += 64 * hi::WAVES) acc[k] = 0.0;
      for (int base = b; base < e; base += PT) {
        __syncthreads();  // the previous pairs' tables have been read
        if (tid < 2 * PT) {  // angle multiples by the angle-addition recurrence, alpha and -theta
          int pr = tid % PT, k = base + pr;
          bool act = k < e;
          int A = src[act ? k : b];
          double Rx = bx - cx[A], Ry = by - cy[A], Rz = bz - cz[A];
          double rho2 = fma(Rx, Rx, Ry * Ry);
          double r2 = fma(Rz, Rz, rho2);
          double rinv = 1.0 / sqrt(r2), rho = sqrt(rho2);
          double c1, s1;
          double2* t;
          if (tid < PT) {
            c1 = rho > 0.0 ? Ry / rho : 0.0;
            s1 = rho > 0.0 ? Rx / rho : 1.0;
            t = ta;
            ids[pr] = A;
            rin[pr] = act ? rinv : 0.0;
          } else {
            c1 = Rz * rinv;
            s1 = -rho * rinv;
            t = tb;
          }
          double cm = 1.0, sm = 0.0;
          for (int m = 0; m <= p; m++) {
            t[m * PT + pr] = make_double2(cm, sm);
            double c2 = fma(cm, c1, -sm * s1);
            sm = fma(sm, c1, cm * s1);
            cm = c2;
          }
        }
        __syncthreads();
        {
          const double2* M[NT];
#pragma unroll
          for (int t = 0; t < NT; t++) M[t] = (const double2*)mult + (size_t)ids[16 * t + (lane & 15)] * NC;
          if (n0 <= p) o0.forward(n0, p, M, ta, tb, V, RS, lane);
          if (n1 <= p) o1.forward(n1, p, M, ta, tb, V, RS, lane);
          if (n2 <= p) o2.forward(n2, p, M, ta, tb, V, RS, lane);
          if (PM >= 24 && n3 <= p) o3.forward(n3, p, M, ta, tb, V, RS, lane);
        }
        __syncthreads();
        // Translation along z, Lhat_n^m = (-1)^{n+m} / ((n-m)!(n+m)!)
        // sum_{k=m}^{p-n} M'_k^m j!/r^{j+1}, j = n + k: a wavefront per order m, a
        // lane per pair and part, in place (the lane reads its column, then writes)
        for (int h = 0; h < 2; h++) {
          int m = h ? 15 - wv : wv, part = lane / PT, col = lane % PT, K = p - 2 * m;
          if (K < 0) continue;
          double g[T_MAX], s[T_MAX];
          double ri = rin[col], rp = ri;
          for (int j = 0; j < 2 * m; j++) rp *= ri;
#pragma unroll
          for (int j = 0; j < T_MAX; j++) {
            s[j] = 0.0;
            if (j <= K) {
              g[j] = c_fact_hi[2 * m + j] * rp;
              rp *= ri;
            } else {
              g[j] = 0.0;
            }
          }
          if (part < 2 && !(m == 0 && part == 1)) {
            int row = part ? 2 * m : m > 0 ? 2 * m - 1 : 0;
#pragma unroll
            for (int kk = 0; kk < T_MAX; kk++) {
              if (kk <= K) {
                int k = m + kk;
                double x = V[(k * k + row) * RS + col];
#pragma unroll
                for (int nn = 0; nn < T_MAX - kk; nn++)
                  if (nn + kk <= K) s[nn] = fma(x, g[nn + kk], s[nn]);
              }
            }
#pragma unroll
            for (int nn = 0; nn < T_MAX; nn++) {
              if (nn <= K) {
                int n = m + nn;
                double f = ((nn & 1) ? -1.0 : 1.0) / (c_fact_hi[nn] * c_fact_hi[n + m]);
                V[(n * n + row) * RS + col] = s[nn] * f;
              }
            }
          }
        }
        __syncthreads();
        if (n0 <= p) o0.back(n0, p, ta, tb, V, RS, acc, lane);
        if (n1 <= p) o1.back(n1, p, ta, tb, V, RS, acc, lane);
        if (n2 <= p) o2.back(n2, p, ta, tb, V, RS, acc, lane);
        if (PM >= 24 && n3 <= p) o3.back(n3, p, ta, tb, V, RS, acc, lane);
      }
      __syncthreads();
      // back to the unscaled basis: L_n^m = (n-m)!(n+m)! Lhat_n^m
      for (int u = tid; u < S; u += 64 * hi::WAVES) {
        int n = both_sign_n(u), j = u - n * n, m = (j + 1) >> 1;
        bool im = j > 0 && !(j & 1);
        double* o = out + 2 * cidx(n, m) + (im ? 1 : 0);
        double v = acc[u] * (c_fact_hi[n - m] * c_fact_hi[n + m]);
        *o = WHOLE && b > b0 ? *o + v : v;
        if (j == 0) out[2 * cidx(n, 0) + 1] = 0.0;
      }
      if (!WHOLE || e == e0) break;
      b = e;
      e = min(e0, b + K);
    }
  }
}

void upload_hi_tables() {
  int dev = 0;
  HIPCHK(hipGetDevice(&dev));
  if (g_hi_tables[dev & 63]) return;
  std::vector<double> fr((size_t)hi::frag_index(hi::PMAX + 1, 0, 0, 0) * 64, 0.0);
  for (int n = 0; n <= hi::PMAX; n++) {
    int D = 2 * n + 1, sw = n * (4 * n * n - 1) / 3;  // dense table offset of order n
    for (int part = 0; part < 2; part++)
      for (int par = 0; par < 2; par++)
        for (int ks = 0; ks < 4; ks++)
          for (int l = 0; l < 64; l++) {
            int mo = (par ^ (n & 1) ^ part) + 2 * (l & 15), mi = par + 2 * (4 * ks + (l >> 4));
            if (mo > n || mi > n || (part && (mo == 0 || mi == 0))) continue;
            int i = part ? 2 * mo : mo > 0 ? 2 * mo - 1 : 0, j = part ? 2 * mi : mi > 0 ? 2 * mi - 1 : 0;
            fr[(size_t)hi::frag_index(n, part, par, ks) * 64 + l] = fmm_swap_table[sw + i * D + j];
          }
  }
  HIPCHK(hipMemcpyToSymbol(HIP_SYMBOL(g_swap_frag), fr.data(), sizeof(double) * fr.size()));
  HIPCHK(hipMemcpyToSymbol(HIP_SYMBOL(c_fact_hi), fmm_fact_table, sizeof(double) * (2 * hi::PMAX + 2)));
  g_hi_tables[dev & 63] = true;
}

static size_t m2l_hi_lds_bytes(int p, int nt) {
  size_t S = (size_t)(p + 1) * (p + 1), pt = 16 * (size_t)nt;
  return sizeof(double) * (((S * (pt + 1) + 1) & ~(size_t)1) + 4 * (p + 1) * pt + pt + S) + sizeof(int) * pt;
}

// any order up to 30; sinks == nullptr: every sink cell (its long lists in
// segments, whole lists only), else the listed ones
void launch_m2l_hi(Ctx& c, int first_lo, const double* mult, double* loc, const int* sinks,
                   const int* nsinks) {
  if (c.p > hi::PMAX) throw unsupported_error{"expansion order above 30"};
  upload_hi_tables();
  int nc = (int)c.ncell;
  M2lSeg sg{};
  // (where memory is limited no list is split: its partial expansions take up to 8 KB each)
  bool whole = c.ws.arena || c.ws.limit;
  if (!sinks && first_lo >= nc) sg = plan_m2l(c, 0, !whole);
  unsigned grid = sinks ? 2048u : (unsigned)std::max(sg.nseg ? sg.max_items : nc, 1);
  // 32 pairs at a time where their coefficients fit the 160 KB of LDS (p <= 20)
  constexpr int P_TWO = 20;
  auto kern = c.p <= P_TWO ? (whole ? k_m2l_hi<2, P_TWO, true> : k_m2l_hi<2, P_TWO, false>)
                           : (whole ? k_m2l_hi<1, hi::PMAX, true> : k_m2l_hi<1, hi::PMAX, false>);
  hipLaunchKernelGGL(kern, dim3(grid), dim3(64 * hi::WAVES), m2l_hi_lds_bytes(c.p, c.p <= P_TWO ? 2 : 1), c.stream,
                     c.p, nc, first_lo, sinks, nsinks, c.m2l.off.p, c.m2l.src.p, c.c_cx.p, c.c_cy.p, c.c_cz.p, mult,
                     loc, sg);
  HIPCHK(hipGetLastError());
  if (sg.nseg) combine_m2l(c, sg, 0, loc);
}

}  // namespace fmm
