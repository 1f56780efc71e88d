// epilogues.hpp -- per-row epilogues fused into the Q / A / A^T products of
// one HPR-QP iteration (Algorithm 4 with the closed forms of Section 3.1).
//
// Names follow the paper: xh = xhat, wh = wbar_{Q}^{t+1/2}, yb/wb/xb/zb =
// ybar/wbar_Q/xbar/zbar, *_a = anchor u^{r,0}.  Linearity caches (GPU only):
// ATy = A^T y and Qw = Q w_Q are carried through the Halpern step instead of
// being recomputed (they are reset from exact products at every restart).
#pragma once
#include "common.hpp"

// The formulas of an iteration that more than one kernel evaluates (one launch
// per product, one workgroup per segment).  The fused multiply-adds are written
// out: left to the compiler they differ from kernel to kernel, and so would the
// last bit of an iterate.
__device__ __forceinline__ double halpern(double rho, double a, double r) {   // rho a + (1 - rho) r
  return __builtin_fma(rho, a, (1.0 - rho) * r);
}
__device__ __forceinline__ double reflect(double bar, double u) { return __builtin_fma(2.0, bar, -u); }   // 2 bar - u
__device__ __forceinline__ double y_arg(double av, double sA, double y) { return __builtin_fma(-sA, y, av); }   // r_y
__device__ __forceinline__ double w_bar(double sQ, double w, double xh, double inv, double kappa, double d) {
  return __builtin_fma(kappa, d, __builtin_fma(sQ, w, xh) * inv);   // (sQ w + xh) / (1 + sQ) + kappa d
}
__device__ __forceinline__ double z_arg(double x, double sigma, double Qw, double ATy, double c) {
  return __builtin_fma(sigma, ATy - Qw - c, x);   // r_z
}

// out_i = q_i
struct EpiStore {
  double* out;
  static constexpr int NR = 0;
  static constexpr unsigned MAXMASK = 0u;
  __device__ void setup(const DevParams*, int) {}
  __device__ __forceinline__ void operator()(int i, double q, double*) const { out[i] = q; }
};

// Q-apply #1:  q1 = Q xhat;  v = xhat + sigma (Qw - Q w_half)
//   with Q w_half = (sigma lamQ Qw + q1)/(1 + sigma lamQ)  ("update-w", first line)
//   which simplifies to v = xhat + kappa (Qw - q1), kappa = sigma/(1+sigma lamQ).
// v is the argument of A in r_y ("update-y").
struct EpiQ1 {
  const double* xh; const double* Qw; double* v; double* q1;
  double kappa;
  static constexpr int NR = 0;
  // panel-ordered product: prefetched chunks, four row blocks per workgroup
  // (random QP, n = 1e6: 45.9 against 46.4 us; A v and A^T ybar lose with it)
  static constexpr bool PANEL_PREFETCH = true;
  static constexpr unsigned MAXMASK = 0u;
  __device__ void setup(const DevParams* p, int j) { IterScalars s; s.load(p, j); kappa = s.kappa; }
  struct Ops { double xh, Qw; };
  __device__ __forceinline__ Ops load(int i) const { return Ops{xh[i], ld_stream(Qw + i)}; }
  __device__ __forceinline__ void operator()(int i, double q, double*, const Ops& o) const {
    st_stream(q1 + i, q);                                   // read once, by Q-apply #2
    v[i] = __builtin_fma(kappa, o.Qw - q, o.xh);            // v is gathered next: keep it cached
  }
  __device__ __forceinline__ void operator()(int i, double q, double* acc) const { (*this)(i, q, acc, load(i)); }
};

// A-product:  r_y = A v - sigma lamA y;  ybar = (Pi_K(r_y) - r_y)/(sigma lamA)  ("update-y");
// Halpern:    y+ = rho y_a + (1 - rho)(2 ybar - y).
// acc[0] += ||y - ybar||^2   (merit R~ of this iteration)
// acc[1] += ||ybar - y_a||^2 (theta~_1 of Algorithm 5)
struct EpiY {
  const double *l, *u, *ya; double *y, *ybar;
  int want_r, want_th;
  double sA, rho;
  static constexpr int NR = 2;
  static constexpr unsigned MAXMASK = 0u;
  __device__ void setup(const DevParams* p, int j) { IterScalars s; s.load(p, j); sA = s.sA; rho = s.rho; }
  struct Ops { double y, ya, l, u; };
  __device__ __forceinline__ Ops load(int i) const {
    return Ops{ld_stream(y + i), ld_stream(ya + i), ld_stream(l + i), ld_stream(u + i)};
  }
  __device__ __forceinline__ void operator()(int i, double q, double* acc) const { (*this)(i, q, acc, load(i)); }
  __device__ __forceinline__ void operator()(int i, double q, double* acc, const Ops& o) const {
    const double yi = o.y, yai = o.ya;
    const double r = y_arg(q, sA, yi);
    const double yb = (clampd(r, o.l, o.u) - r) / sA;
    ybar[i] = yb;                                            // gathered next by A^T
    st_stream(y + i, halpern(rho, yai, reflect(yb, yi)));
    if (want_r) { const double t = yi - yb; acc[0] += t * t; }
    if (want_th) { const double t = yb - yai; acc[1] += t * t; }
  }
};

// A^T-product:  g = A^T ybar;  d = g - A^T y = A^T (ybar - y);
// cache Halpern:  A^T y+ = rho A^T y_a + (1 - rho)(2 g - A^T y).
// At checks also g and e = g - A^T y_a (for theta~ and eta_d).
struct EpiAT {
  double *ATy; const double* ATya; double *d, *g, *e;
  int check;
  double rho;
  static constexpr int NR = 0;
  static constexpr unsigned MAXMASK = 0u;
  __device__ void setup(const DevParams* p, int j) { IterScalars s; s.load(p, j); rho = s.rho; }
  struct Ops { double aty, atya; };
  __device__ __forceinline__ Ops load(int i) const { return Ops{ld_stream(ATy + i), ld_stream(ATya + i)}; }
  __device__ __forceinline__ void operator()(int i, double q, double* acc) const { (*this)(i, q, acc, load(i)); }
  __device__ __forceinline__ void operator()(int i, double q, double*, const Ops& o) const {
    const double aty = o.aty, atya = o.atya;
    d[i] = q - aty;                                          // gathered next by Q-apply #2
    st_stream(ATy + i, halpern(rho, atya, reflect(q, aty)));
    if (check) { g[i] = q; e[i] = q - atya; }
  }
};

// Q-apply #2 with the Halpern epilogue and the next iteration's z/x step.
//   q2 = Q d = Q A^T (ybar - y)
//   w_half = (sigma lamQ w + xh)/(1+sigma lamQ);  wbar = w_half + kappa d        ("update-w")
//   Q wbar = (sigma lamQ Qw + q1)/(1+sigma lamQ) + kappa q2
//   Halpern: x+ = rho x_a + (1-rho) xh  (since 2 xbar - x = xh),
//            w+ = rho w_a + (1-rho)(2 wbar - w),  Qw+ likewise.
//   Next z/x step ("update-z", "update-x") with A^T y+ already written by EpiAT:
//            r_z = x+ + sigma(-Qw+ + A^T y+ - c), xbar' = Pi_C(r_z), zbar' = (xbar' - r_z)/sigma,
//            xh' = 2 xbar' - x+.
// Reductions (u - ubar differences, du = u - ubar):
//   acc[0..5] = <dw,Q dw>, <Q dw, A^T dy>, |dx|^2, <A^T dy, Q A^T dy>, <A^T dy, dx>, <Q dw, dx>
//     with A^T dy = -d, Q A^T dy = -q2, dx = xbar - xh;
//   acc[6..8] (checks) with D = ubar - u_a: <Dw, Q Dw>, <Q Dw, e>, |Dx|^2.
// The panel-ordered product loads the Halpern anchors (wa, Qwa, xa) of the
// epilogue below at the start of its last panel (Pre, preload; random QP,
// n = 1e6: 58.1 against 58.6 us; preloading more operands gains nothing more
// and takes registers).  The other products load them in the epilogue.
struct EpiQ2 {
  double *xh, *w, *Qw, *XB, *ZB;
  const double *q1, *d, *wa, *Qwa, *xa, *ATy, *c, *L, *U, *e;
  double *wbar, *qwbar, *x, *xbar_out;
  int want_r, check, xb_next, trace;
  double l1;                      // lambda of phi (0: the box projection)
  double sigma, sQ, inv, kappa, rho;
  static constexpr int NR = 9;
  static constexpr bool PANEL_PREFETCH = true;   // panel-ordered product: prefetch the next chunk
  static constexpr unsigned MAXMASK = 0u;
  __device__ void setup(const DevParams* p, int j) {
    IterScalars s; s.load(p, j);
    sigma = s.sigma; sQ = s.sQ; inv = s.inv; kappa = s.kappa; rho = s.rho;
  }
  // operands loaded early by the panel-ordered product (before its last panel)
  struct Pre { double wa, Qwa, xa; };
  __device__ __forceinline__ Pre preload(int i) const {
    return Pre{ld_stream(wa + i), ld_stream(Qwa + i), ld_stream(xa + i)};
  }
  struct Ops { double xh, w, Qw, d, q1, wa, Qwa, xa, ATy, c, L, U; };
  __device__ __forceinline__ Ops load(int i, const Pre& p) const {
    return Ops{ld_stream(xh + i), ld_stream(w + i), ld_stream(Qw + i), d[i], ld_stream(q1 + i), p.wa, p.Qwa, p.xa,
               ld_stream(ATy + i), ld_stream(c + i), ld_stream(L + i), ld_stream(U + i)};
  }
  __device__ __forceinline__ Ops load(int i) const { return load(i, preload(i)); }
  __device__ __forceinline__ void operator()(int i, double q2, double* acc, const Pre& pf) const {
    (*this)(i, q2, acc, load(i, pf));
  }
  __device__ __forceinline__ void operator()(int i, double q2, double* acc) const { (*this)(i, q2, acc, load(i)); }
  __device__ __forceinline__ void operator()(int i, double q2, double* acc, const Ops& o) const {
    const double xhi = o.xh, wi = o.w, Qwi = o.Qw, di = o.d, wai = o.wa, Qwai = o.Qwa, xai = o.xa;
    const double wb = w_bar(sQ, wi, xhi, inv, kappa, di);
    const double Qwb = w_bar(sQ, Qwi, o.q1, inv, kappa, q2);
    if (want_r || check || trace) {
      const double xb = XB[i];
      if (want_r) {
        const double dw = wi - wb, Qdw = Qwi - Qwb, ATdy = -di, QATdy = -q2, dx = xb - xhi;
        acc[0] += dw * Qdw; acc[1] += Qdw * ATdy; acc[2] += dx * dx;
        acc[3] += ATdy * QATdy; acc[4] += ATdy * dx; acc[5] += Qdw * dx;
      }
      if (check) {
        wbar[i] = wb; qwbar[i] = Qwb;
        const double Dw = wb - wai, QDw = Qwb - Qwai, Dx = xb - xai;
        acc[6] += Dw * QDw; acc[7] += QDw * e[i]; acc[8] += Dx * Dx;
      }
      if (trace) { wbar[i] = wb; xbar_out[i] = xb; }
    }
    const double xn = halpern(rho, xai, xhi);
    const double wn = halpern(rho, wai, reflect(wb, wi));
    const double Qwn = halpern(rho, Qwai, reflect(Qwb, Qwi));
    st_stream(w + i, wn); st_stream(Qw + i, Qwn);
    if (trace) x[i] = xn;
    const double rz = z_arg(xn, sigma, Qwn, o.ATy, o.c);
    const double xbn = prox_phi(rz, sigma * l1, o.L, o.U);
    xh[i] = reflect(xbn, xn);                                // gathered next by Q-apply #1
    if (xb_next) { XB[i] = xbn; ZB[i] = (xbn - rz) / sigma; }
  }
};

// Without rows (m = 0) d = 0 and Q d = 0, so the Q xhat product carries the whole
// iteration: wbar = w_half and EpiQ2 directly on q1 = Q xhat.  For products whose
// last step gathers neither xh nor any other vector written here (the Gram Q: it
// gathers Ahat xhat).
struct EpiQ0 {
  EpiQ2 e;
  static constexpr int NR = EpiQ2::NR;
  static constexpr unsigned MAXMASK = EpiQ2::MAXMASK;
  __device__ void setup(const DevParams* p, int j) { e.setup(p, j); }
  using Ops = EpiQ2::Ops;
  __device__ __forceinline__ Ops load(int i) const {
    return Ops{ld_stream(e.xh + i), ld_stream(e.w + i), ld_stream(e.Qw + i), 0.0, 0.0, ld_stream(e.wa + i),
               ld_stream(e.Qwa + i), ld_stream(e.xa + i), ld_stream(e.ATy + i), ld_stream(e.c + i), ld_stream(e.L + i),
               ld_stream(e.U + i)};
  }
  __device__ __forceinline__ void operator()(int i, double q, double* acc) const { (*this)(i, q, acc, load(i)); }
  __device__ __forceinline__ void operator()(int i, double q, double* acc, Ops o) const {
    o.q1 = q;
    e(i, 0.0, acc, o);
  }
};

// Stand-alone z/x step (start of a solve and after a restart):
//   r_z = x + sigma(-Qw + A^T y - c); xbar = Pi_C(r_z); zbar = (xbar - r_z)/sigma; xh = 2 xbar - x.
struct EpiStage1 {
  const double *x, *Qw, *ATy, *c, *L, *U; double *xh, *XB, *ZB;
  double l1;
  double sigma;
  static constexpr int NR = 0;
  static constexpr unsigned MAXMASK = 0u;
  __device__ void setup(const DevParams* p, int) { sigma = p->sigma; }
  __device__ __forceinline__ void operator()(int i, double, double*) const {
    const double xi = x[i];
    const double rz = xi + sigma * (-Qw[i] + ATy[i] - c[i]);
    const double xb = prox_phi(rz, sigma * l1, L[i], U[i]);
    xh[i] = 2.0 * xb - xi; XB[i] = xb; ZB[i] = (xb - rz) / sigma;
  }
};

// Primal residual and the y-part of the dual objective at (x, y) from A x:
//   acc[0] = max |Ax - Pi_K(Ax)|, acc[1] = max |Ax|,
//   acc[2] = sum_i (l_i y_i^+ + u_i y_i^-), acc[3] = #(nonzero y_i against an infinite bound)
// With diagonal preconditioning, ie = 1/E turns the scaled row (A~ x~)_i into
// the given problem's (A x)_i; the objective terms are invariant.
struct EpiResA {
  const double *l, *u, *y;
  const double* ie;   // NULL: no preconditioning
  static constexpr int NR = 4;
  static constexpr unsigned MAXMASK = 0x3u;
  __device__ void setup(const DevParams*, int) {}
  __device__ __forceinline__ void operator()(int i, double ax, double* acc) const {
    const double li = l[i], ui = u[i], yi = y[i];
    const double s = ie ? ie[i] : 1.0;
    acc[0] = fmax(acc[0], fabs(ax - clampd(ax, li, ui)) * s);
    acc[1] = fmax(acc[1], fabs(ax) * s);
    if (yi > 0.0) { if (isinf(li)) acc[3] += 1.0; else acc[2] += li * yi; }
    else if (yi < 0.0) { if (isinf(ui)) acc[3] += 1.0; else acc[2] += ui * yi; }
  }
};

// Dual residual and the rest of the objectives at (x, z) from Q x and g = A^T y:
//   acc[0] = max |-Qx + g + z - c|, acc[1] = max |g|, acc[2] = max |Qx|,
//   acc[3] = <x, Qx>, acc[4] = <c, x> + lambda ||x||_1, acc[5] = -phi^*(-z) (for
//   lambda = 0: sum_j (L_j z_j^+ + U_j z_j^-)), acc[6] = #(z_j making phi^*(-z) infinite).
// Optionally copies x, z to the output buffers.  With diagonal
// preconditioning, id = 1/D maps the scaled dual quantities back (the dual
// residual, A^T y and Q x of the given problem are 1/D times the scaled ones).
struct EpiResQ {
  const double *x, *z, *g, *c, *L, *U; double *xo, *zo;
  const double* id;   // NULL: no preconditioning
  double l1;          // lambda of phi: acc[4] also holds lambda ||x||_1
  static constexpr int NR = 7;
  static constexpr unsigned MAXMASK = 0x7u;
  __device__ void setup(const DevParams*, int) {}
  __device__ __forceinline__ void operator()(int i, double qx, double* acc) const {
    const double xi = x[i], zi = z[i], gi = g ? g[i] : 0.0, ci = c[i];
    const double s = id ? id[i] : 1.0;
    acc[0] = fmax(acc[0], fabs(-qx + gi + zi - ci) * s);
    acc[1] = fmax(acc[1], fabs(gi) * s);
    acc[2] = fmax(acc[2], fabs(qx) * s);
    acc[3] += xi * qx;
    acc[4] += ci * xi + l1 * fabs(xi);
    bool inf = false;
    acc[5] += neg_conj_phi(zi, l1, L[i], U[i], &inf);
    if (inf) acc[6] += 1.0;
    if (xo) { xo[i] = xi; zo[i] = zi; }
  }
};

// acc[0] = max |q_i| s_i (s NULL: 1): the inf-norm of a product, optionally
// rescaled row by row
struct EpiMaxAbs {
  const double* s;
  static constexpr int NR = 1;
  static constexpr unsigned MAXMASK = 0x1u;
  __device__ void setup(const DevParams*, int) {}
  __device__ __forceinline__ void operator()(int i, double q, double* acc) const {
    acc[0] = fmax(acc[0], fabs(q) * (s ? s[i] : 1.0));
  }
};

// theta~_3 = <e, Q e>, e = A^T (ybar - y_a)
struct EpiTheta3 {
  const double* e;
  static constexpr int NR = 1;
  static constexpr unsigned MAXMASK = 0u;
  __device__ void setup(const DevParams*, int) {}
  __device__ __forceinline__ void operator()(int i, double q, double* acc) const { acc[0] += e[i] * q; }
};

// restart: Qw = Qw_a = Q wbar (exact product)
struct EpiStore2 {
  double *a, *b;
  static constexpr int NR = 0;
  static constexpr unsigned MAXMASK = 0u;
  __device__ void setup(const DevParams*, int) {}
  __device__ __forceinline__ void operator()(int i, double q, double*) const { a[i] = q; b[i] = q; }
};

// power method: w = s M v stored; acc[0] += v_i w_i (Rayleigh quotient), acc[1] += w_i^2
struct EpiPow {
  const double* v; double* w;
  double s;
  static constexpr int NR = 2;
  static constexpr unsigned MAXMASK = 0u;
  __device__ void setup(const DevParams*, int) {}
  struct Ops { double v; };
  __device__ __forceinline__ Ops load(int i) const { return Ops{v[i]}; }
  __device__ __forceinline__ void operator()(int i, double q, double* acc) const { (*this)(i, q, acc, load(i)); }
  __device__ __forceinline__ void operator()(int i, double q, double* acc, const Ops& o) const {
    const double wi = q * s;
    w[i] = wi; acc[0] += o.v * wi; acc[1] += wi * wi;
  }
};
