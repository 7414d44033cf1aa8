// Eigendecomposition of the reduced operator and prediction coefficients.
//
// Sec. 2.3: A~ = V Lambda V^-1 and Phi = U V (the projected DMD modes), and
// the prediction u(t) = Phi Lambda^(t/dt) Phi^+ u(0).
//
// k_eig (one workgroup, FP64), on demand for the eigenpairs:
//   1. Householder reduction of A~ to upper Hessenberg form H = Q^T A~ Q;
//   2. Francis double-shift QR iteration to the real Schur form T = Z^T A~ Z
//      (1x1 and standardised 2x2 diagonal blocks), accumulating Z;
//   3. eigenvectors of T by back-substitution (complex arithmetic), eight
//      lanes per eigenvalue, then V = Z X, unit 2-norm, largest entry real > 0;
//   4. order by |lambda| descending, then Im descending.
// k_power_coef: the prediction's coefficients for a chunk of steps, as
// powers of A~ applied to U^T x_a (equal to the eigenvector form at integer
// steps, see below), folded with the basis coefficients (U = S[:, :m] Q,
// so U c = S (Q c)).
#include <hip/hip_runtime.h>
#include <math.h>

#include <type_traits>

#include "odmd_internal.h"
#include "pass.h"
#include "xlane.h"

namespace odmd {

constexpr int LDH = RMAX + 1;
constexpr double EPS = 2.220446049250313e-16;

struct cplx {
  double re, im;
};
__device__ __forceinline__ cplx cmul(cplx a, cplx b) {
  return {a.re * b.re - a.im * b.im, a.re * b.im + a.im * b.re};
}
__device__ __forceinline__ cplx csub(cplx a, cplx b) { return {a.re - b.re, a.im - b.im}; }
__device__ __forceinline__ cplx cadd(cplx a, cplx b) { return {a.re + b.re, a.im + b.im}; }
// Smith's algorithm for a / b
__device__ __forceinline__ cplx cdiv(cplx a, cplx b) {
  if (fabs(b.re) >= fabs(b.im)) {
    const double t = b.im / b.re, den = b.re + b.im * t;
    return {(a.re + a.im * t) / den, (a.im - a.re * t) / den};
  }
  const double t = b.re / b.im, den = b.re * t + b.im;
  return {(a.re * t + a.im) / den, (a.im * t - a.re) / den};
}
__device__ __forceinline__ double cabs2(cplx a) { return hypot(a.re, a.im); }

#define Hm(i, j) H[(j) * LDH + (i)]
#define Zm(i, j) Z[(j) * LDH + (i)]

// The value of v in the given lane (a wave-uniform index), in every lane.
__device__ __forceinline__ double readlane_d(double v, int lane) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_readlane((int)b, lane);
  const int hi = __builtin_amdgcn_readlane((int)(b >> 32), lane);
  return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

// Scaling by powers of two (exact), compiled in for SMALL only: the exponent
// that brings m to [0.5, 1), zero for m = 0, and v 2^e.
template <bool SMALL>
__device__ __forceinline__ int exponent_of(double m) { return SMALL ? __builtin_amdgcn_frexp_exp(m) : 0; }
template <bool SMALL>
__device__ __forceinline__ double times_2(double v, int e) { return SMALL ? ldexp(v, e) : v; }

// Householder reflector P = I - beta w w^T mapping (x, y, z) to (alpha, 0, 0),
// w = (w0, y, z): with nrm = ||(x, y, z)|| and alpha = -sign(x) nrm,
// w0 = x - alpha and beta = 2 / w.w = 1 / (nrm (nrm + |x|)).  Its dependent
// chain is the bulge chase's: nrm by one Goldschmidt step from the hardware
// estimate (2^-24 relative, then 2^-47) and a residual correction, beta by a
// third-order step from the reciprocal estimate of the uncorrected
// denominator, which runs beside the correction; the products with w run
// beside beta.  No branch: the matrix is scaled to entries of order one, so
// nothing overflows, and a vector whose square underflows to below 2^-900 is
// zero for it (the identity, y and z dropped).  SMALL (see eig_body): the
// vector is brought to order one first; P is the same for any multiple of it.
struct Reflector {
  double w0, w1, w2, beta, alpha;
};
template <bool SMALL>
__device__ __forceinline__ Reflector make_reflector(double x, double y, double z) {
  constexpr double TINY = 0x1p-900;
  const int ex = exponent_of<SMALL>(fmax(fabs(x), fmax(fabs(y), fabs(z))));
  x = times_2<SMALL>(x, -ex);
  y = times_2<SMALL>(y, -ex);
  z = times_2<SMALL>(z, -ex);
  const double s0 = __builtin_fma(z, z, __builtin_fma(y, y, x * x));
  const bool ok = s0 > TINY;
  const double ss = fmax(s0, TINY);
  const double rn = __builtin_amdgcn_rsq(ss);
  double g = ss * rn, h = 0.5 * rn;            // nrm, 1 / (2 nrm)
  const double rd = __builtin_amdgcn_rcp(__builtin_fma(g, fabs(x), ss));
  const double e = __builtin_fma(-g, h, 0.5);
  g = __builtin_fma(g, e, g);
  h = __builtin_fma(h, e, h);
  g = __builtin_fma(__builtin_fma(-g, g, ss), h, g);
  const double den = __builtin_fma(g, fabs(x), ss);
  const double f = __builtin_fma(-den, rd, 1.0);
  const double al = x >= 0.0 ? -g : g;
  Reflector R;
  R.w0 = x - al;
  R.w1 = y;
  R.w2 = z;
  R.beta = ok ? __builtin_fma(rd, __builtin_fma(f, f, f), rd) : 0.0;
  R.alpha = times_2<SMALL>(ok ? al : x, ex);
  return R;
}

// k_eig's workgroup: wavefronts 0 .. EIG_K-1 carry one bulge each, with
// vectors as many more apply the reflectors to Z; the reduction and the
// eigenvectors use all of them.
constexpr int EIG_K = 4;
constexpr int EIG_GAP = 3;               // rows between neighbouring bulges
constexpr int EIG_MIN = 5;               // active rows per bulge, at least
template <bool VECS>
constexpr int eig_threads() { return (VECS ? 2 : 1) * EIG_K * 64; }

// Steps 1 and 2: H (LDS, scaled, zero past n x n) to its real Schur form, with
// vectors Z.  True if an eigenvalue was not found.  (SMALL: see eig_body.  The
// thread's indexes are handed in: formed again here, the same code took 1 %
// longer at rank 64 with vectors.)
template <bool VECS, bool SMALL>
__device__ __forceinline__ bool schur(double* H, double* Z, double* wr, double* wi, double (*red)[RMAX],
                                      double (*redb)[RMAX], Reflector (*rf)[2], const int n, const double hn,
                                      const int tid, const int t, const int wave) {
  // 1. Hessenberg reduction.  Both sides of a reflector I - beta v v^T in one
  //    update from the old H, with a = beta H^T v, b = beta H v and
  //    c = b - beta (v.b) v:  H <- H - v a^T - c v^T; and Z <- Z - (beta Z v) v^T.
  //    The first EIG_K wavefronts take H: thread (t, part) keeps the entries
  //    H(part + EIG_K e, t) in registers (the column sums and the update need
  //    no LDS reads, which bounded this phase) and writes them to LDS, where
  //    the row sums read them; with vectors the others take Z, thread
  //    (t, part) the entries Z(t, part + EIG_K e).  v_i and c_i come from
  //    lane i's register.
  const int part = wave & (EIG_K - 1);
  const bool onH = !VECS || wave < EIG_K;
  constexpr int NE1 = RMAX / EIG_K;
  double own[NE1];
#pragma unroll
  for (int e = 0; e < NE1; ++e)
    own[e] = onH ? Hm(part + EIG_K * e, t) : (t == part + EIG_K * e ? 1.0 : 0.0);
  for (int k = 0; k + 2 < n; ++k) {
    double hk = Hm(t, k);
    int ex = 0;
    double top = 0.0;                    // SMALL: the largest entry to annihilate
    if (SMALL) {
      top = wave_max(t > k + 1 ? fabs(hk) : 0.0);
      ex = exponent_of<SMALL>(wave_max(t > k ? fabs(hk) : 0.0));
      hk = times_2<SMALL>(hk, -ex);
    }
    double x2 = t > k + 1 ? hk * hk : 0.0;
    x2 = add_half_pair(add_row_pair(row_sum(x2)));
    const double x0 = readlane_d(hk, k + 1);
    const bool none = SMALL ? top == 0.0 : x2 <= 0x1p-900;    // uniform: nothing to annihilate
    const double nrm = none ? fabs(x0) : sqrt(__builtin_fma(x0, x0, x2));
    const double al = none ? x0 : (x0 >= 0.0 ? -nrm : nrm);
    const double beta = none ? 0.0 : 1.0 / (nrm * (nrm + fabs(x0)));
    const double vt = none ? 0.0 : (t == k + 1 ? x0 - al : (t > k + 1 ? hk : 0.0));
    double a = 0.0, a2 = 0.0, b = 0.0, b2 = 0.0;
    if (onH) {
      double m[NE1];                     // row t
#pragma unroll
      for (int e = 0; e < NE1; ++e) m[e] = Hm(t, part + EIG_K * e);
#pragma unroll
      for (int e = 0; e < NE1; e += 2) {
        const double v0 = readlane_d(vt, part + EIG_K * e), v1 = readlane_d(vt, part + EIG_K * (e + 1));
        a = __builtin_fma(v0, own[e], a);
        a2 = __builtin_fma(v1, own[e + 1], a2);
        b = __builtin_fma(v0, m[e], b);
        b2 = __builtin_fma(v1, m[e + 1], b2);
      }
      red[part][t] = a + a2;
    } else {
#pragma unroll
      for (int e = 0; e < NE1; e += 2) {
        b = __builtin_fma(readlane_d(vt, part + EIG_K * e), own[e], b);
        b2 = __builtin_fma(readlane_d(vt, part + EIG_K * (e + 1)), own[e + 1], b2);
      }
    }
    redb[wave][t] = b + b2;
    __syncthreads();
    a = b = 0.0;
#pragma unroll
    for (int p = 0; p < EIG_K; ++p) {
      a += red[p][t];
      b += redb[(wave & ~(EIG_K - 1)) + p][t];
    }
    a *= beta;
    b *= beta;
    if (onH) {
      const double vb = add_half_pair(add_row_pair(row_sum(vt * b)));
      const double ct = __builtin_fma(-beta * vb, vt, b);
      const bool colk = t == k;          // its entries are al and zeros by construction
#pragma unroll
      for (int e = 0; e < NE1; ++e) {
        const int i = part + EIG_K * e;
        const double g = __builtin_fma(-readlane_d(ct, i), vt, __builtin_fma(-readlane_d(vt, i), a, own[e]));
        own[e] = colk && i > k ? (i == k + 1 ? times_2<SMALL>(al, ex) : 0.0) : g;
        Hm(i, t) = own[e];
      }
    } else {
#pragma unroll
      for (int e = 0; e < NE1; ++e) own[e] = __builtin_fma(-b, readlane_d(vt, part + EIG_K * e), own[e]);
    }
    __syncthreads();
  }
  if (VECS && !onH) {
#pragma unroll
    for (int e = 0; e < NE1; ++e) Zm(t, part + EIG_K * e) = own[e];
  }

  // 2. Francis double-shift QR to real Schur form.  Every wavefront takes
  //    the same decisions from the same H.
  int hi = n - 1, its = 0, total = 0;
  bool fail = false;
  while (hi >= 0) {
    // l = the largest index in [1, hi] whose subdiagonal entry is
    // negligible, else 0: every lane tests one entry, one ballot
    bool neg = false;
    if (t >= 1 && t <= hi) {
      double s = fabs(Hm(t - 1, t - 1)) + fabs(Hm(t, t));
      if (s == 0.0) s = hn;
      neg = fabs(Hm(t, t - 1)) <= EPS * s;
    }
    const unsigned long long mask = __ballot(neg);
    const int l = mask ? 63 - __builtin_clzll(mask) : 0;
    __syncthreads();
    if (l > 0 && tid == 0) Hm(l, l - 1) = 0.0;
    if (l == hi) {
      if (tid == 0) {
        wr[hi] = Hm(hi, hi);
        wi[hi] = 0.0;
      }
      --hi;
      its = 0;
      continue;                          // (the entry just cleared is not read below hi)
    }
    if (l == hi - 1) {
      const int p = hi - 1, q = hi;
      const double a = Hm(p, p), b = Hm(p, q), c = Hm(q, p), d = Hm(q, q);
      const double pp = 0.5 * (a - d);
      const int ex = exponent_of<SMALL>(fmax(fabs(pp), fmax(fabs(b), fabs(c))));
      const double ps = times_2<SMALL>(pp, -ex);
      const double disc = ps * ps + times_2<SMALL>(b, -ex) * times_2<SMALL>(c, -ex);
      __syncthreads();
      if (disc >= 0.0) {
        const double sq = times_2<SMALL>(sqrt(disc), ex);
        const double zz = pp + (pp >= 0.0 ? sq : -sq);
        double la = d + zz, lb = (zz != 0.0) ? d - b * c / zz : d;
        // rotation whose first column is the eigenvector (zz, c) of la
        const double h = hypot(zz, c);
        if (h > 0.0) {
          const double cs = zz / h, sn = c / h;
          if (wave == 0 && t >= p && t < n) {      // rows p, q from the left (G^T)
            const double u = Hm(p, t), v = Hm(q, t);
            Hm(p, t) = cs * u + sn * v;
            Hm(q, t) = -sn * u + cs * v;
          }
          __syncthreads();
          if (wave == 0 && t <= q) {               // columns p, q from the right
            const double u = Hm(t, p), v = Hm(t, q);
            Hm(t, p) = cs * u + sn * v;
            Hm(t, q) = -sn * u + cs * v;
          }
          if (VECS && wave == EIG_K && t < n) {
            const double u = Zm(t, p), v = Zm(t, q);
            Zm(t, p) = cs * u + sn * v;
            Zm(t, q) = -sn * u + cs * v;
          }
          __syncthreads();
          if (tid == 0) Hm(q, p) = 0.0;
          la = Hm(p, p);
          lb = Hm(q, q);
        }
        if (tid == 0) {
          wr[p] = la;
          wi[p] = 0.0;
          wr[q] = lb;
          wi[q] = 0.0;
        }
      } else if (tid == 0) {
        wr[p] = wr[q] = a - pp;          // (a + d) / 2
        wi[p] = times_2<SMALL>(sqrt(-disc), ex);
        wi[q] = -times_2<SMALL>(sqrt(-disc), ex);
      }
      hi -= 2;
      its = 0;
      continue;
    }
    if (total >= 30 * n) {
      fail = true;
      break;
    }
    ++its;
    ++total;
    const int N = hi - l + 1;            // at least 3
    int K = min(EIG_K, max(1, N / EIG_MIN));
    double s, tt;                        // the shifts' sum and product, times 2^-es and 2^-2 es
    int es;
    if (its == 10 || its == 20) {        // exceptional shift
      const double w = fabs(Hm(hi, hi - 1)) + fabs(Hm(hi - 1, hi - 2));
      es = exponent_of<SMALL>(w);
      const double ws = times_2<SMALL>(w, -es);
      s = 1.5 * ws;
      tt = ws * ws;
      K = 1;
    } else {
      double a = Hm(hi - 1, hi - 1), b = Hm(hi - 1, hi), c = Hm(hi, hi - 1), d = Hm(hi, hi);
      es = exponent_of<SMALL>(fmax(fmax(fabs(a), fabs(b)), fmax(fabs(c), fabs(d))));
      a = times_2<SMALL>(a, -es);
      b = times_2<SMALL>(b, -es);
      c = times_2<SMALL>(c, -es);
      d = times_2<SMALL>(d, -es);
      s = a + d;
      tt = a * d - b * c;
    }
    __syncthreads();                     // the shifts (and H(l, l-1) = 0) before the first rows change
    // Bulge chase.  Bulge b starts EIG_GAP b steps after the first; its
    // reflector acts on rows, then columns, k .. k+2 (k .. k+1 in its last
    // step, where w2 = 0).  Rows of different bulges are disjoint, and so are
    // their columns; row and column hi + 1 <= RMAX exist.  A step is two
    // barriers, also for a wavefront that waits for its start or for the
    // others' end, so every wavefront meets 2 (N - 1 + EIG_GAP (K - 1)).
    const int b = wave & (EIG_K - 1);
    auto idle = [](int steps) {
      for (int i = 0; i < 2 * steps; ++i) __syncthreads();
    };
    if (b >= K) {
      idle(N - 1 + EIG_GAP * (K - 1));
    } else if (onH) {
      idle(EIG_GAP * b);
      // the first column of the shifted square (up to a power of two)
      double h00 = Hm(l, l), h10 = Hm(l + 1, l), h01 = Hm(l, l + 1), h11 = Hm(l + 1, l + 1), h21 = Hm(l + 2, l + 1);
      if (SMALL) {
        const int eb = max(es, exponent_of<SMALL>(fmax(fmax(fmax(fabs(h00), fabs(h10)), fmax(fabs(h01), fabs(h11))), fabs(h21))));
        s = times_2<SMALL>(s, es - eb);
        tt = times_2<SMALL>(tt, 2 * (es - eb));
        h00 = times_2<SMALL>(h00, -eb);
        h10 = times_2<SMALL>(h10, -eb);
        h01 = times_2<SMALL>(h01, -eb);
        h11 = times_2<SMALL>(h11, -eb);
        h21 = times_2<SMALL>(h21, -eb);
      }
      double x = h00 * h00 + h01 * h10 - s * h00 + tt;
      double y = h10 * (h00 + h11 - s);
      double z = h10 * h21;
      double* pc = H + t * LDH + l;                    // column t, rows k ..
      double* pr = H + l * LDH + t;                    // row t, columns k ..
      int bc = -1;                                     // bulge column: none in the first step
      for (int k = l; k < hi; ++k) {
        double c0 = pc[0], c1 = pc[1], c2 = pc[2];
        const Reflector R = make_reflector<SMALL>(x, y, z);
        if (VECS && t == 0) rf[b][(k - l) & 1] = R;
        double d = -R.beta * __builtin_fma(R.w2, c2, __builtin_fma(R.w1, c1, R.w0 * c0));
        const bool bulge = t == bc;                    // it becomes (alpha, 0, 0)
        pc[0] = bulge ? R.alpha : __builtin_fma(d, R.w0, c0);
        pc[1] = bulge ? 0.0 : __builtin_fma(d, R.w1, c1);
        pc[2] = bulge ? 0.0 : __builtin_fma(d, R.w2, c2);
        __syncthreads();
        c0 = pr[0], c1 = pr[LDH], c2 = pr[2 * LDH];
        d = -R.beta * __builtin_fma(R.w2, c2, __builtin_fma(R.w1, c1, R.w0 * c0));
        c0 = __builtin_fma(d, R.w0, c0);
        pr[0] = c0;
        pr[LDH] = __builtin_fma(d, R.w1, c1);
        pr[2 * LDH] = __builtin_fma(d, R.w2, c2);
        // the next step's (x, y, z): the new H(k+1 .. k+3, k), zero past hi
        x = readlane_d(c0, k + 1);
        y = readlane_d(c0, (k + 2) & 63);
        const long long zm = k + 3 <= hi ? -1ll : 0ll;
        z = __longlong_as_double(__double_as_longlong(readlane_d(c0, (k + 3) & 63)) & zm);
        bc = k;
        ++pc;
        pr += LDH;
        __syncthreads();
      }
      idle(EIG_GAP * (K - 1 - b));
    } else if (VECS) {
      // Z's columns: the reflector is read after its step's first barrier
      // and applied while the bulges go on (two slots per bulge: the one
      // read here is written again two steps on, behind this wavefront's
      // next arrival)
      idle(EIG_GAP * b);
      double* pz = Z + l * LDH + t;
      for (int k = l; k < hi; ++k) {
        __syncthreads();
        const Reflector R = rf[b][(k - l) & 1];
        const double c0 = pz[0], c1 = pz[LDH], c2 = pz[2 * LDH];
        __syncthreads();
        const double d = -R.beta * __builtin_fma(R.w2, c2, __builtin_fma(R.w1, c1, R.w0 * c0));
        pz[0] = __builtin_fma(d, R.w0, c0);
        pz[LDH] = __builtin_fma(d, R.w1, c1);
        pz[2 * LDH] = __builtin_fma(d, R.w2, c2);
        pz += LDH;
      }
      idle(EIG_GAP * (K - 1 - b));
    }
  }
  return fail;
}

// VECS false: eigenvalues only (no Z, eigenvectors or V); the cache level
// eig_valid is 1 after such a call and 2 after a call with vectors.  Both
// run the same operations on H, so the eigenvalues are the same bit for bit.
//
// Latency bounds it: one workgroup, a serial chain of reflectors.  The chain
// is cut in three ways.  (1) EIG_K bulges are chased at once, EIG_GAP rows
// apart, one wavefront each, all with the shifts of the trailing 2 x 2 block:
// a group of K sweeps over N rows takes N - 1 + 3 (K - 1) steps instead of
// K (N - 1), for about 1.4 times the sweeps (the K sweeps share their
// shifts, so a group converges with order K + 1 instead of 2^K).  (2) A step
// has two phases, a barrier after each: every bulge applies its reflector
// to its three rows (lane t is column t), then to its three columns (lane t
// is row t).  H is zero below the bulges and padded with zero rows and
// columns, so no lane is masked and no entry of the 3 x 3 block is formed
// twice.  (3) Z's columns are left to wavefronts of their own, and the
// reduction and eigenvector sums are split over the workgroup.
// Squares and products of two entries of a block far below the rest of the
// matrix vanish (an exactly decoupled block of 1e-67 of the largest entry
// never converged).  A matrix that holds such an entry, above zero and below
// SMALL_ENTRY of the largest, takes a form of the solver that forms them from
// entries scaled by powers of two.  The others come below that only by
// convergence, where dropping an entry is harmless, and take the form without
// (a test for small vectors in every step cost 46 of 1250 us, rank 64 with
// vectors).
// A~ of rank 40 (n = 160,000 wake): 415 us (854 with one wavefront and one
// bulge); with vectors at rank 64: 1137 us (2388).  A step takes about 840
// cycles (1160 before; one bulge alone 630), with vectors 1030.
constexpr double SMALL_ENTRY = 0x1p-200;
template <bool VECS>
__device__ __forceinline__ void eig_body(DevState* st) {
  if (st->eig_valid >= (VECS ? 2 : 1)) return;
  constexpr int NTH = eig_threads<VECS>();
  __shared__ double H[(RMAX + 2) * LDH];         // zero past n x n
  __shared__ double Z[VECS ? (RMAX + 2) * LDH : 1];
  __shared__ double Xr[VECS ? (RMAX + 1) * LDH : 1];
  __shared__ double Xi[VECS ? (RMAX + 1) * LDH : 1];
  __shared__ double wr[RMAX], wi[RMAX], red[EIG_K][RMAX];
  __shared__ double redb[NTH / 64][RMAX];
  __shared__ Reflector rf[EIG_K][2];
  __shared__ int pos[RMAX], below[NTH / 64];
  const int tid = threadIdx.x, t = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n = st->r;
  if (n == 0) {
    if (tid == 0) {
      st->eig_valid = 2;
      st->eig_status = 0;
    }
    return;
  }
  // A~ scaled by a power of two to entries of order one (exact), zero past n
  double hn = 0.0;
  constexpr int NL = RMAX * RMAX / NTH;
  double av[NL];                         // every load in flight at once
#pragma unroll
  for (int u = 0; u < NL; ++u) {
    const int i = t, j = wave + u * (NTH / 64);
    const bool in = i < n && j < n;
    const double v = st->At[in ? j * RMAX + i : 0];
    av[u] = in ? v : 0.0;
  }
#pragma unroll
  for (int u = 0; u < NL; ++u) hn = fmax(hn, fabs(av[u]));
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) hn = fmax(hn, __shfl_xor(hn, o, 64));
  if (t == 0) red[0][wave] = hn;
  __syncthreads();
#pragma unroll
  for (int w = 0; w < NTH / 64; ++w) hn = fmax(hn, red[0][w]);
  const int ex = hn > 0.0 && hn < INFINITY ? ilogb(hn) : 0;
  bool low = false;
#pragma unroll
  for (int u = 0; u < NL; ++u) low = low || (av[u] != 0.0 && fabs(av[u]) < SMALL_ENTRY * hn);
  const bool wave_low = __ballot(low) != 0;
  if (t == 0) below[wave] = wave_low;
  // row RMAX and the columns past RMAX are zero too
  for (int idx = tid; idx < 2 * LDH; idx += NTH) H[RMAX * LDH + idx] = 0.0;
  if (tid < RMAX) H[tid * LDH + RMAX] = 0.0;
#pragma unroll
  for (int u = 0; u < NL; ++u) H[(wave + u * (NTH / 64)) * LDH + t] = ldexp(av[u], -ex);
  if (VECS) {                            // Z's columns past RMAX (their values are not used)
    for (int idx = tid; idx < 2 * LDH; idx += NTH) Z[RMAX * LDH + idx] = 0.0;
  }
  hn = hn > 0.0 && hn < INFINITY ? ldexp(hn, -ex) : 1.0;
  __syncthreads();
  bool small_entries = false;
#pragma unroll
  for (int w = 0; w < NTH / 64; ++w) small_entries = small_entries || below[w] != 0;

  const bool fail = small_entries ? schur<VECS, true>(H, Z, wr, wi, red, redb, rf, n, hn, tid, t, wave)
                                  : schur<VECS, false>(H, Z, wr, wi, red, redb, rf, n, hn, tid, t, wave);
  __syncthreads();

  // 3. eigenvectors of the quasi-triangular T by back-substitution (complex
  //    arithmetic), eight lanes per eigenvalue: the sums over the known
  //    entries are split over the lanes, which then all form the new ones
  const double smin = fmax(EPS * hn, 1e-300);
  const int ev = tid >> 3, el = tid & 7;
  if (VECS && ev < n && !fail) {
    double* xr = Xr + ev * LDH;
    double* xi = Xi + ev * LDH;
    const cplx lam = {wr[ev], wi[ev]};
    for (int i = el; i < n; i += 8) xr[i] = xi[i] = 0.0;
    wave_lds_fence();
    int start;
    double mx;                            // running bound of the entries, for the rescaling test
    if (wi[ev] == 0.0) {
      if (el == 0) xr[ev] = 1.0;
      start = ev - 1;
      mx = 1.0;
    } else {
      const int p = (wi[ev] > 0.0) ? ev : ev - 1;  // block (p, p+1)
      const int q = p + 1;
      const cplx a = {Hm(p, p), 0.0}, b = {Hm(p, q), 0.0};
      const cplx c = {Hm(q, p), 0.0}, d = {Hm(q, q), 0.0};
      cplx u1 = b, u2 = csub(lam, a);            // from row 1
      cplx w1 = csub(lam, d), w2 = c;            // from row 2
      if (cabs2(u1) + cabs2(u2) < cabs2(w1) + cabs2(w2)) {
        u1 = w1;
        u2 = w2;
      }
      if (small_entries) {
        // (of order one, so that the squares of a small block's vector do not vanish)
        const int eu = exponent_of<true>(fmax(fmax(fabs(u1.re), fabs(u1.im)), fmax(fabs(u2.re), fabs(u2.im))));
        u1 = {times_2<true>(u1.re, -eu), times_2<true>(u1.im, -eu)};
        u2 = {times_2<true>(u2.re, -eu), times_2<true>(u2.im, -eu)};
      }
      if (el == 0) {
        xr[p] = u1.re;
        xi[p] = u1.im;
        xr[q] = u2.re;
        xi[q] = u2.im;
      }
      start = p - 1;
      mx = fmax(fabs(u1.re) + fabs(u1.im), fabs(u2.re) + fabs(u2.im));
    }
    wave_lds_fence();
    int i = start;
    while (i >= 0) {
      const bool blk = i > 0 && Hm(i, i - 1) != 0.0;
      // s = sum_{j > i} H(row, j) x_j for the one or two rows of this block
      // (H real: two real sums per row)
      const int i0 = blk ? i - 1 : i;
      double sr = 0.0, si = 0.0;         // row i0
      double ur = 0.0, ui = 0.0;         // row i (a 1 x 1 block reads the same row)
#pragma unroll 2
      for (int j = i + 1 + el; j < n; j += 8) {
        const double vr = xr[j], vi = xi[j], h = Hm(i0, j), g = Hm(i, j);
        sr = __builtin_fma(h, vr, sr);
        si = __builtin_fma(h, vi, si);
        ur = __builtin_fma(g, vr, ur);
        ui = __builtin_fma(g, vi, ui);
      }
      sr = oct_sum(sr);
      si = oct_sum(si);
      ur = oct_sum(ur);
      ui = oct_sum(ui);
      if (!blk) {
        cplx den = csub({Hm(i, i), 0.0}, lam);
        if (cabs2(den) < smin) den = {smin, 0.0};
        const cplx v = cdiv({-sr, -si}, den);
        if (el == 0) {
          xr[i] = v.re;
          xi[i] = v.im;
        }
        mx = fmax(mx, fabs(v.re) + fabs(v.im));
        i -= 1;
      } else {
        const cplx m00 = csub({Hm(i0, i0), 0.0}, lam), m01 = {Hm(i0, i), 0.0};
        const cplx m10 = {Hm(i, i0), 0.0}, m11 = csub({Hm(i, i), 0.0}, lam);
        cplx det = csub(cmul(m00, m11), cmul(m01, m10));
        if (cabs2(det) < smin * smin) det = {smin * smin, 0.0};
        const cplx r0 = {-sr, -si}, r1 = {-ur, -ui};
        const cplx x0 = cdiv(csub(cmul(r0, m11), cmul(m01, r1)), det);
        const cplx x1 = cdiv(csub(cmul(m00, r1), cmul(m10, r0)), det);
        if (el == 0) {
          xr[i0] = x0.re;
          xi[i0] = x0.im;
          xr[i] = x1.re;
          xi[i] = x1.im;
        }
        mx = fmax(mx, fmax(fabs(x0.re) + fabs(x0.im), fabs(x1.re) + fabs(x1.im)));
        i -= 2;
      }
      wave_lds_fence();
      // rescale to keep the entries bounded
      if (mx > 1e100) {
        const double f = 1.0 / mx;
        for (int jj = el; jj < n; jj += 8) {
          xr[jj] *= f;
          xi[jj] *= f;
        }
        mx = 1.0;
        wave_lds_fence();
      }
    }
  }

  // the eigenvalues at their rank in the output order; with vectors,
  // V = Z X normalised, at the same rank
  if (tid < n) redb[0][tid] = hypot(wr[tid], wi[tid]);    // |lambda| (redb is free after the reduction)
  __syncthreads();
  if (tid < n && !fail) {
    const double ml = redb[0][tid];
    int rank = 0;
    for (int j = 0; j < n; ++j) {
      const double mj = redb[0][j];
      rank += (mj > ml) || (mj == ml && (wi[j] > wi[tid] || (wi[j] == wi[tid] && j < tid)));
    }
    st->lam_re[rank] = ldexp(wr[tid], ex);
    st->lam_im[rank] = ldexp(wi[tid], ex);
    if (VECS) pos[tid] = rank;
  }
  if (VECS) {
    __syncthreads();
    if (ev < n && !fail) {
      // lane el of an eigenvalue's eight holds the entries el, el + 8, ...
      // of Z X[:, ev] (Z is zero past n rows)
      constexpr int NE = RMAX / 8;
      double ar[NE], ai[NE];
#pragma unroll
      for (int u = 0; u < NE; ++u) ar[u] = ai[u] = 0.0;
      for (int j = 0; j < n; ++j) {
        const double vr = Xr[ev * LDH + j], vi = Xi[ev * LDH + j];
#pragma unroll
        for (int u = 0; u < NE; ++u) {
          const double z = Zm(el + 8 * u, j);
          ar[u] = __builtin_fma(z, vr, ar[u]);
          ai[u] = __builtin_fma(z, vi, ai[u]);
        }
      }
      // unit norm, largest-modulus entry (the first of equal ones) real and
      // positive: multiply by conj(v_ib) / (|v_ib| ||v||)
      double nrm2 = 0.0, best = -1.0, vbr = 0.0, vbi = 0.0;
      int ib = 0;
#pragma unroll
      for (int u = 0; u < NE; ++u) {
        const double m2 = ar[u] * ar[u] + ai[u] * ai[u];
        if (el + 8 * u < n) {
          nrm2 += m2;
          if (m2 > best) {
            best = m2;
            ib = el + 8 * u;
            vbr = ar[u];
            vbi = ai[u];
          }
        }
      }
      nrm2 = oct_sum(nrm2);
#pragma unroll
      for (int o = 4; o > 0; o >>= 1) {
        const double ob = __shfl_xor(best, o, 8), orr = __shfl_xor(vbr, o, 8), oi = __shfl_xor(vbi, o, 8);
        const int oib = __shfl_xor(ib, o, 8);
        const bool take = ob > best || (ob == best && oib < ib);
        best = take ? ob : best;
        vbr = take ? orr : vbr;
        vbi = take ? oi : vbi;
        ib = take ? oib : ib;
      }
      const double m = sqrt(best), f = 1.0 / sqrt(nrm2);
      const double pr = vbr / m * f, pi = -vbi / m * f;
      double* __restrict__ vr = st->V_re + pos[ev] * RMAX;
      double* __restrict__ vi = st->V_im + pos[ev] * RMAX;
#pragma unroll
      for (int u = 0; u < NE; ++u) {
        const int i = el + 8 * u;
        if (i < n) {
          vr[i] = ar[u] * pr - ai[u] * pi;
          vi[i] = i == ib ? 0.0 : ar[u] * pi + ai[u] * pr;
        }
      }
    }
  }
  __threadfence();
  __syncthreads();

  if (tid == 0) {
    st->eig_status = fail;
    if (fail) latch_status(st, ST_NOCONV);
    st->eig_valid = VECS ? 2 : 1;
  }
}

// Prediction coefficients by powers of A~ (Sec. 2.3).  With U orthonormal,
// Phi = U V and the anchor x_a (Phi^+ x_a = V^-1 U^T x_a = V^-1 p_y), the
// state k steps ahead Phi Lambda^k Phi^+ x_a = U V Lambda^k V^-1 p_y equals
// U A~^k p_y: the same states without the eigendecomposition (and defined
// also where A~ has no full set of eigenvectors).  One workgroup forms
// c_k = A~^k p_y for one chunk of steps k0+1 .. k0+K by doubling: c_{k0+1}
// = A~ c_{k0}; with columns 1 .. w known and P = A~^w, columns w+1 .. 2w
// are P times columns 1 .. w, then P <- P^2.  The columns stay in LDS
// (leading dimension r | 1; the host sizes chunks by coef_chunk(r_max)),
// and are written out as Q c_k, the coefficients of the stored columns
// (U = S[:, :m] Q).  c_{k0+K} is kept in cfwd, where the next chunk starts.
// Products are 16 x 16 FP64 matrix-core tiles (16x16x4 operand layout:
// lane l supplies row or column l % 16 at k-step offset l / 16; element v
// of lane l's result is row 4 v + l / 16, column l % 16), spread over the
// workgroup's 16 wavefronts: a doubling's products and its squaring are
// one list of tiles.
typedef double d4_t __attribute__((ext_vector_type(4)));
constexpr int LP = RMAX + 1;            // leading dimension of the LDS matrices
constexpr int PC_THREADS = 1024;
constexpr int PC_NWV = PC_THREADS / 64;
constexpr int PC_NA = RMAX * RMAX / PC_THREADS;                    // A~ entries per thread
constexpr int PC_NQ = (CMAX * LP + PC_THREADS - 1) / PC_THREADS;   // Q entries per thread

struct PowerLds {
  double M[2 * RMAX * LP];              // A~^w and its square; then Q
  double col[PC_LCOL];                  // c_k of this chunk, column kk at kk * ldc
  double sv[RMAX];
};
static_assert(CMAX * LP <= 2 * RMAX * LP, "Q fits the power buffers");

// One 16 x 16 tile: sum over the k-steps s < 4 NT of A(s) B(s), where a(s)
// and b(s) give this lane's operands; two accumulators over alternate
// k-steps.  NT 16-row tiles cover the rank (entries past it are zero).
// The operands of a half of the k-steps (all of them for one or two
// tiles) are loaded before its products (the scheduling barrier keeps the
// compiler from spreading the loads between the products, where each pair
// of products waited for the next loads); halves keep a 1024-thread
// workgroup within 128 registers.
template <int NT, class FA, class FB>
__device__ __forceinline__ d4_t tile_sum(FA a, FB b) {
  constexpr int NH = NT > 2 ? 2 : 1;        // halves of the k-steps (fewer live operands)
  constexpr int KH = 4 * NT / NH;
  d4_t d0 = {0.0, 0.0, 0.0, 0.0}, d1 = d0;
#pragma unroll
  for (int hf = 0; hf < NH; ++hf) {
    double av[KH], bv[KH];
#pragma unroll
    for (int s = 0; s < KH; ++s) {
      av[s] = a(hf * KH + s);
      bv[s] = b(hf * KH + s);
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int s = 0; s < KH; s += 2) {
      d0 = __builtin_amdgcn_mfma_f64_16x16x4f64(av[s], bv[s], d0, 0, 0, 0);
      d1 = __builtin_amdgcn_mfma_f64_16x16x4f64(av[s + 1], bv[s + 1], d1, 0, 0, 0);
    }
  }
  return d0 + d1;
}

template <int NT>
__device__ __forceinline__ void power_body(DevState* st, PowerLds& S, int k0, int K, int koff, int n, int m) {
  const int t = threadIdx.x, l = t & 63, wv = t >> 6;
  const int lr = l & 15, lk = l >> 4;                // operand row/column, k-step offset
  const int ldc = n | 1;
  double* const out = st->coefA + koff * CMAX;       // column kk at out + kk * CMAX
  // every load of A~, Q and the start vector in flight at once
  double ra[PC_NA], rq[PC_NQ];
#pragma unroll
  for (int u = 0; u < PC_NA; ++u) {
    const int idx = t + u * PC_THREADS, i = idx % RMAX, j = idx / RMAX;
    const bool ok = i < n && j < n;
    const double x = st->At[ok ? j * RMAX + i : 0];
    ra[u] = ok ? x : 0.0;
  }
#pragma unroll
  for (int u = 0; u < PC_NQ; ++u) {
    const int idx = t + u * PC_THREADS, k = idx % LP, c = idx / LP;
    const bool ok = c < m && k < n;
    const double x = st->Q[ok ? c * RMAX + k : 0];
    rq[u] = ok ? x : 0.0;
  }
  const double s0 = t < n ? (k0 == 0 ? st->py[t] : st->cfwd[t]) : 0.0;
  double* P = S.M;
  double* P2 = S.M + RMAX * LP;
#pragma unroll
  for (int u = 0; u < PC_NA; ++u) {
    const int idx = t + u * PC_THREADS;
    P[(idx / RMAX) * LP + idx % RMAX] = ra[u];
  }
  if (t < RMAX) S.sv[t] = s0;
  __syncthreads();
  if (t < n) {                                       // c_{k0+1} = A~ c_{k0}
    double a[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int j = 0; j < 16 * NT; ++j) a[j & 3] = __builtin_fma(P[j * LP + t], S.sv[j], a[j & 3]);
    S.col[t] = (a[0] + a[1]) + (a[2] + a[3]);
  }
  __syncthreads();
  for (int w = 1; w < K; w *= 2) {
    // jobs: columns w .. w+cnt-1 = P (= A~^w) times columns 0 .. cnt-1, as
    // (16 columns, 16 rows) tiles; then, unless this is the last doubling,
    // the tiles of P2 = P P (= A~^2w)
    const int cnt = min(w, K - w);
    const int jp = (cnt + 15) / 16 * NT;
    const int js = 2 * w < K ? NT * NT : 0;
    for (int j = wv; j < jp + js; j += PC_NWV) {
      if (j < jp) {
        const int ct = j / NT, it = j % NT;
        const int c = ct * 16 + lr;
        const bool cv = c < cnt;
        const d4_t d = tile_sum<NT>(
            [&](int s) {
              const int k = 4 * s + lk;
              const bool ok = cv && k < n;
              const double x = S.col[ok ? c * ldc + k : 0];
              return ok ? x : 0.0;
            },
            [&](int s) { return P[(4 * s + lk) * LP + it * 16 + lr]; });
        const int i = it * 16 + lr;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int cc = ct * 16 + 4 * v + lk;
          if (cc < cnt && i < n) S.col[(w + cc) * ldc + i] = d[v];
        }
      } else {
        const int it = (j - jp) % NT, jt = (j - jp) / NT;
        const d4_t d = tile_sum<NT>([&](int s) { return P[(4 * s + lk) * LP + it * 16 + lr]; },
                                    [&](int s) { return P[(jt * 16 + lr) * LP + 4 * s + lk]; });
#pragma unroll
        for (int v = 0; v < 4; ++v) P2[(jt * 16 + lr) * LP + it * 16 + 4 * v + lk] = d[v];
      }
    }
    if (js) {
      double* const tmp = P;
      P = P2;
      P2 = tmp;
    }
    __syncthreads();
  }
  if (t < n) st->cfwd[t] = S.col[(K - 1) * ldc + t];
  double* const sQ = S.M;                            // the powers are done
#pragma unroll
  for (int u = 0; u < PC_NQ; ++u) {
    const int idx = t + u * PC_THREADS;
    if (idx < CMAX * LP) sQ[idx] = rq[u];
  }
  __syncthreads();
  // out column kk = Q c_kk, as (16 columns, 16 rows c) tiles over the rows
  // c < m (rounded up to 16); the rows above are zero
  const int CT = (m + 15) / 16;
  const int jf = (K + 15) / 16 * CT;
  for (int j = wv; j < jf; j += PC_NWV) {
    const int ct = j / CT, jt = j % CT;
    const int kk = ct * 16 + lr;
    const bool kv = kk < K;
    const int cq = jt * 16 + lr;
    const bool qv = cq < CMAX;
    const d4_t d = tile_sum<NT>(
        [&](int s) {
          const int k = 4 * s + lk;
          const bool ok = kv && k < n;
          const double x = S.col[ok ? kk * ldc + k : 0];
          return ok ? x : 0.0;
        },
        [&](int s) {
          const double q = sQ[(qv ? cq : 0) * LP + 4 * s + lk];
          return qv ? q : 0.0;
        });
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int kc = ct * 16 + 4 * v + lk;
      if (kc < K && qv) out[kc * CMAX + cq] = d[v];
    }
  }
  const int c0 = 16 * CT;
  if (c0 < CMAX)
    for (int idx = t; idx < K * (CMAX - c0); idx += PC_THREADS)
      out[(idx / (CMAX - c0)) * CMAX + c0 + idx % (CMAX - c0)] = 0.0;
}

__device__ __forceinline__ void power_entry(DevState* st, int k0, int K, int koff) {
  __shared__ PowerLds S;
  const int n = st->r, m = st->m;
  if (n == 0 || K > coef_chunk(n) || koff + K > COEF_CHUNK) {   // (the host sends neither)
    for (int idx = threadIdx.x; idx < K * CMAX && koff + idx / CMAX < COEF_CHUNK; idx += PC_THREADS)
      st->coefA[koff * CMAX + idx] = 0.0;
    if (threadIdx.x == 0) latch_status(st, n == 0 ? ST_EMPTY : ST_NOCONV);
    return;
  }
  switch ((n + 15) / 16) {
    case 1: power_body<1>(st, S, k0, K, koff, n, m); break;
    case 2: power_body<2>(st, S, k0, K, koff, n, m); break;
    case 3: power_body<3>(st, S, k0, K, koff, n, m); break;
    default: power_body<4>(st, S, k0, K, koff, n, m); break;
  }
}

__global__ __launch_bounds__(PC_THREADS) void k_power_coef(DevState* st, int k0, int K, int koff) {
  power_entry(st, k0, K, koff);
}

// The first chunk (k0 = 0) of several streams: one workgroup per entry of a
// device-resident table of states and step counts.
__global__ __launch_bounds__(PC_THREADS) void k_power_coef_batch(DevState* const* __restrict__ sts,
                                                                 const int* __restrict__ Ks) {
  power_entry(sts[blockIdx.x], 0, Ks[blockIdx.x], 0);
}

// Coefficients that materialise the basis: column k of U is S[:, :m] Q[:, k].
__global__ __launch_bounds__(256) void k_basis_coef(DevState* st) {
  const int m = st->m, r = st->r;
  for (int idx = threadIdx.x; idx < CMAX * RMAX; idx += 256) {
    const int c = idx % CMAX, k = idx / CMAX;
    st->coefA[k * CMAX + c] = (c < m && k < r) ? st->Q[c * RMAX + k] : 0.0;
  }
}

template <bool VECS>
__global__ __launch_bounds__(eig_threads<VECS>()) void k_eig(DevState* st) { eig_body<VECS>(st); }

hipError_t launch_eig(DevState* st, bool vectors, hipStream_t s) {
  if (vectors) hipLaunchKernelGGL(k_eig<true>, dim3(1), dim3(eig_threads<true>()), 0, s, st);
  else hipLaunchKernelGGL(k_eig<false>, dim3(1), dim3(eig_threads<false>()), 0, s, st);
  return hipGetLastError();
}

hipError_t launch_power_coef(DevState* st, int k0, int steps, int koff, hipStream_t s) {
  hipLaunchKernelGGL(k_power_coef, dim3(1), dim3(PC_THREADS), 0, s, st, k0, steps, koff);
  return hipGetLastError();
}

hipError_t launch_power_coef_batch(DevState* const* sts, const int* steps, int count, hipStream_t s) {
  hipLaunchKernelGGL(k_power_coef_batch, dim3(count), dim3(PC_THREADS), 0, s, sts, steps);
  return hipGetLastError();
}

hipError_t launch_basis_coef(DevState* st, hipStream_t s) {
  hipLaunchKernelGGL(k_basis_coef, dim3(1), dim3(256), 0, s, st);
  return hipGetLastError();
}

}  // namespace odmd
