// Host-side quadrature tables of the library: Gauss-Legendre rules, the
// per-triangle regular rules and the Sauter-Schwab region rules.  Built once
// per (rule, order) and uploaded to the device by the context.
#include <array>
#include <cmath>
#include <stdexcept>

#include "bem_internal.h"

namespace bem {

// Gauss-Legendre nodes on [-1,1] are the zeros of the Legendre polynomial
// P_q; each is found by Newton's method from the classical estimate
// cos(pi (4k + 3) / (4q + 2)), with P_q and its derivative evaluated by the
// three-term recurrence (n+1) P_{n+1} = (2n+1) x P_n - n P_{n-1} and
// P_q' = q (x P_q - P_{q-1}) / (x^2 - 1).  Weights 2 / ((1 - x^2) P_q'^2).
static void legendre_and_derivative(int q, double x, double *p, double *dp) {
  double pm1 = 1.0, pq = x;
  for (int n = 1; n < q; ++n) {
    const double pn1 = ((2 * n + 1) * x * pq - n * pm1) / (n + 1);
    pm1 = pq;
    pq = pn1;
  }
  if (q == 0) pq = 1.0, pm1 = 0.0;
  *p = pq;
  *dp = q * (x * pq - pm1) / (x * x - 1.0);
}

void gauss_legendre01(int q, double *x, double *w) {
  if (q < 1) throw std::invalid_argument("gauss order");
  for (int k = 0; k < q; ++k) {
    double z = std::cos(M_PI * (4.0 * k + 3.0) / (4.0 * q + 2.0));
    double p, dp;
    for (int it = 0; it < 200; ++it) {
      legendre_and_derivative(q, z, &p, &dp);
      const double step = p / dp;
      z -= step;
      if (std::fabs(step) <= 1e-17) break;
    }
    legendre_and_derivative(q, z, &p, &dp);
    // z decreases with k: fill from the back so nodes on [0,1] increase
    x[q - 1 - k] = 0.5 * (1.0 + z);
    w[q - 1 - k] = 1.0 / ((1.0 - z * z) * dp * dp);  // = (2 / (...)) / 2
  }
}

TriRule triangle_rule(int rule, int q) {
  TriRule r;
  if (rule == BEM_RULE_TRI7) {
    // Radon's seven-point degree-5 rule: centroid plus two orbits of three
    // points (barycentric (a, a, 1 - 2a)), weights summing to one.
    const double rt = std::sqrt(15.0);
    const double a[2] = {(6.0 - rt) / 21.0, (6.0 + rt) / 21.0};
    const double wo[2] = {(155.0 - rt) / 1200.0, (155.0 + rt) / 1200.0};
    std::vector<std::array<double, 4>> pts;  // l0, l1, l2, weight
    pts.push_back({1.0 / 3.0, 1.0 / 3.0, 1.0 / 3.0, 9.0 / 40.0});
    for (int o = 0; o < 2; ++o) {
      const double b = 1.0 - 2.0 * a[o];
      pts.push_back({a[o], a[o], b, wo[o]});
      pts.push_back({a[o], b, a[o], wo[o]});
      pts.push_back({b, a[o], a[o], wo[o]});
    }
    // x = l0 v0 + l1 v1 + l2 v2 = Phi(l1 + l2, l2); int_tau f = (sqrt(g)/2) sum w f
    for (auto &p : pts) {
      r.s.push_back(p[1] + p[2]);
      r.t.push_back(p[2]);
      r.w.push_back(0.5 * p[3]);
    }
    return r;
  }
  if (q < 1 || q > BEM_MAX_ORDER) throw std::invalid_argument("order");
  // Duffy: (s, t) = (x1, x1 x2) on [0,1]^2, Jacobian x1 (Sec. 2.2)
  std::vector<double> gx(q), gw(q);
  gauss_legendre01(q, gx.data(), gw.data());
  for (int a = 0; a < q; ++a)
    for (int b = 0; b < q; ++b) {
      r.s.push_back(gx[a]);
      r.t.push_back(gx[a] * gx[b]);
      r.w.push_back(gw[a] * gw[b] * gx[a]);
    }
  return r;
}

std::vector<double> duffy_table(int q) {
  std::vector<double> x(q), w(q), t;
  gauss_legendre01(q, x.data(), w.data());
  const int H = q / 2, HC = (q + 1) / 2;
  // eta pairs 1/2 +- delta from the outermost, then the centre
  auto delta = [&](int k) { return 0.5 * (x[q - 1 - k] - x[k]); };
  for (int j = 0; j < q; ++j)
    t.insert(t.end(), {x[j], x[j] * x[j], w[j] * x[j], w[j] * x[j] * x[j]});
  for (int k = 0; k < H; ++k) t.push_back(delta(k));
  for (int k = 0; k < H; ++k) t.push_back(delta(k) * delta(k));
  for (int k = 0; k < HC; ++k) t.push_back(w[k]);
  for (int k = 0; k < H; ++k) t.push_back(w[k] * delta(k));
  for (int j = 0; j < q; ++j)
    for (int k = 0; k < H; ++k) t.push_back(x[j] * delta(k));
  for (int j = 0; j < q; ++j)
    for (int k = 0; k < HC; ++k) t.push_back(w[j] * x[j] * w[k]);
  for (int j = 0; j < q; ++j) {
    const double c = x[j] - 2.0 / 3.0;
    t.insert(t.end(), {c, c * c});
  }
  return t;
}

std::vector<double> general_table(const TriRule &r) {
  const size_t n = r.s.size();
  std::vector<double> t(9 * n);
  for (size_t k = 0; k < n; ++k) {
    const double s = r.s[k], e = r.t[k] - 0.5 * s, c = s - 2.0 / 3.0, d = r.t[k] - 1.0 / 3.0;
    const double row[9] = {s, r.t[k], r.w[k], e, c, d, c * c, c * e, e * e};
    for (int f = 0; f < 9; ++f) t[f * n + k] = row[f];
  }
  return t;
}

// Weights rounded to FP32 one by one have a sum that is off by up to 4e-8 (the
// seven-point rule by 3e-8, order 3 in products of two weights by 3.7e-8), a bias
// of every entry as large as the rounding of its sum.  The rounding error of one
// weight is carried to the next instead: mult(k) times weight k enters the sum.
template <class At, class Mult>
static void carry_weights(std::vector<float> &t, const std::vector<double> &exact, int n, At &&at, Mult &&mult) {
  double carry = 0.0;
  for (int k = 0; k < n; ++k) {
    const double w = exact[at(k)], m = mult(k);
    t[at(k)] = (float)(w + carry / m);
    carry += m * (w - (double)t[at(k)]);
  }
}

std::vector<float> duffy_table32(int q) {
  const std::vector<double> d = duffy_table(q);
  std::vector<float> t(d.begin(), d.end());
  const int H = q / 2, HC = (q + 1) / 2;
  const int W = 4 * q + 2 * H, WF = W + HC + H + q * H;  // DuffyAt
  auto pair = [&](int k) { return k < H ? 2.0 : 1.0; };  // an eta pair's weight enters twice
  carry_weights(t, d, q, [](int j) { return 4 * j + 2; }, [](int) { return 1.0; });
  carry_weights(t, d, HC, [&](int k) { return W + k; }, pair);
  carry_weights(t, d, q * HC, [&](int k) { return WF + k; }, [&](int k) { return pair(k % HC); });
  return t;
}

std::vector<float> general_table32(const TriRule &r) {
  const std::vector<double> d = general_table(r);
  std::vector<float> t(d.begin(), d.end());
  const int n = (int)r.s.size();
  carry_weights(t, d, n, [&](int k) { return 2 * n + k; }, [](int) { return 1.0; });
  return t;
}

// One point of a Sauter-Schwab region: returns (x^1, x^2, y^1, y^2) and the
// Jacobian of the region map at (xi, h1, h2, h3) in [0,1]^4.  The maps send
// [0,1]^4 onto a piece of {0 <= x2 <= x1 <= 1}^2 such that the pieces of one
// class tile it; the singular set (x^ = y^, resp. the common edge x^2 = y^2
// = 0 with x^1 = y^1, resp. the common vertex 0) is pulled back to xi = 0,
// where the Jacobian's factor xi^3 cancels the kernel's singularity.
static void ss_point(int cls, int reg, double xi, double h1, double h2, double h3,
                     double out[4], double *jac) {
  switch (cls) {
    case CLS_IDENTICAL: {
      double p[4];
      const int piece = reg >> 1;
      if (piece == 0) {
        p[0] = xi;
        p[1] = xi * (1.0 - h1 + h1 * h2);
        p[2] = xi * (1.0 - h1 * h2 * h3);
        p[3] = xi * (1.0 - h1);
      } else if (piece == 1) {
        p[0] = xi;
        p[1] = xi * h1 * (1.0 - h2 + h2 * h3);
        p[2] = xi * (1.0 - h1 * h2);
        p[3] = xi * h1 * (1.0 - h2);
      } else {
        p[0] = xi * (1.0 - h1 * h2 * h3);
        p[1] = xi * h1 * (1.0 - h2 * h3);
        p[2] = xi;
        p[3] = xi * h1 * (1.0 - h2);
      }
      // odd pieces: the mirror image with x^ and y^ exchanged
      const int sw = (reg & 1) ? 2 : 0;
      out[0] = p[sw];
      out[1] = p[sw + 1];
      out[2] = p[2 - sw];
      out[3] = p[3 - sw];
      *jac = xi * xi * xi * h1 * h1 * h2;
      return;
    }
    case CLS_EDGE: {
      const double x3 = xi * xi * xi;
      switch (reg) {
        case 0:
          out[0] = xi;                     out[1] = xi * h1 * h3;
          out[2] = xi * (1.0 - h1 * h2);    out[3] = xi * h1 * (1.0 - h2);
          *jac = x3 * h1 * h1;
          return;
        case 1:
          out[0] = xi;                     out[1] = xi * h1;
          out[2] = xi * (1.0 - h1 * h2 * h3); out[3] = xi * h1 * h2 * (1.0 - h3);
          break;
        case 2:
          out[0] = xi * (1.0 - h1 * h2);    out[1] = xi * h1 * (1.0 - h2);
          out[2] = xi;                     out[3] = xi * h1 * h2 * h3;
          break;
        case 3:
          out[0] = xi * (1.0 - h1 * h2 * h3); out[1] = xi * h1 * h2 * (1.0 - h3);
          out[2] = xi;                     out[3] = xi * h1;
          break;
        default:
          out[0] = xi * (1.0 - h1 * h2 * h3); out[1] = xi * h1 * (1.0 - h2 * h3);
          out[2] = xi;                     out[3] = xi * h1 * h2;
          break;
      }
      *jac = x3 * h1 * h1 * h2;
      return;
    }
    default: {  // CLS_VERTEX
      const double a0 = xi, a1 = xi * h1, b0 = xi * h2, b1 = xi * h2 * h3;
      if (reg == 0) {
        out[0] = a0; out[1] = a1; out[2] = b0; out[3] = b1;
      } else {
        out[0] = b0; out[1] = b1; out[2] = a0; out[3] = a1;
      }
      *jac = xi * xi * xi * h2;
      return;
    }
  }
}

// Every region map above is linear in xi and every Jacobian carries the
// factor xi^3, so a rule point factors into its xi part and its eta part:
//   (x^, y^) = xi * g(eta),   weight = (w_a xi_a^3) * (w_b w_c w_d J(eta) / xi^3).
// The table stores g (the map at xi = 1) and the eta weight for every region
// and (eta1, eta2, eta3) Gauss triple; the xi nodes and weights are separate.
SSRule ss_rule(int cls, int q) {
  if (q < 1 || q > BEM_MAX_ORDER) throw std::invalid_argument("order");
  const int nreg = cls == CLS_IDENTICAL ? 6 : cls == CLS_EDGE ? 5 : cls == CLS_VERTEX ? 2 : 0;
  if (!nreg) throw std::invalid_argument("class");
  std::vector<double> gx(q), gw(q);
  gauss_legendre01(q, gx.data(), gw.data());
  SSRule r;
  for (int reg = 0; reg < nreg; ++reg)
    for (int b = 0; b < q; ++b)
      for (int c = 0; c < q; ++c)
        for (int d = 0; d < q; ++d) {
          double p[4], jac;
          ss_point(cls, reg, 1.0, gx[b], gx[c], gx[d], p, &jac);  // xi = 1: J = eta part
          r.xs.push_back(p[0]);
          r.xt.push_back(p[1]);
          r.ys.push_back(p[2]);
          r.yt.push_back(p[3]);
          r.w.push_back(gw[b] * gw[c] * gw[d] * jac);
        }
  return r;
}

// Singular rule of the piecewise-constant entries.  On a common edge or
// triangle the difference of the two points is proportional to xi h1 (edge)
// or xi h1 h2 (identical) as well: with p that product,
//   x - y = p (g1 E1_i + g2 E2_i - g3 E1_j - g4 E2_j) = p d,
// so that 1/|x - y| and <x - y, n> / |x - y|^3 factor into a power of p and a
// function of d alone.  The q^4 points per region then split into few
// directions d (2 q^3 for a vertex, 5 q^2 for an edge, 3 q for an identical
// pair) and one set of radial nodes p for all of them -- the same rule, summed
// in another order.  Differences are written without cancellation: with a
// common edge or triangle E1_j = E1_i and g1 is the coefficient of their
// difference.  Identical pairs serve the single layer only (the double layer
// vanishes): the regions with x^ and y^ exchanged add the same sums again, so
// three regions carry twice their weight.
SingularRule singular_rule(int cls, int q) {
  if (q < 1 || q > BEM_MAX_ORDER) throw std::invalid_argument("order");
  std::vector<double> x(q), w(q);
  gauss_legendre01(q, x.data(), w.data());
  SingularRule r;
  auto dir = [&](double g1, double g2, double g3, double g4, double wt) {
    const double g[4] = {g1, g2, g3, g4};
    for (int k = 0; k < 4; ++k) r.g[k].push_back(g[k]);
    r.w.push_back(wt);
  };
  // the radial weights: Jacobian times |x - y|^-1 (single layer) resp. times
  // <x - y, n> / |x - y|^3 ~ p^-2 (double layer), in powers of p's factors
  auto radial = [&](double p, double ws, double wd) {
    r.p.push_back(p);
    r.ws.push_back(ws);
    r.wd.push_back(wd);
  };
  switch (cls) {
    case CLS_VERTEX:  // J = xi^3 h2
      for (int a = 0; a < q; ++a)
        for (int b = 0; b < q; ++b)
          for (int c = 0; c < q; ++c) dir(1.0, x[a], x[b], x[b] * x[c], w[a] * w[b] * w[c] * x[b]);
      for (int a = 0; a < q; ++a)
        for (int b = 0; b < q; ++b)
          for (int c = 0; c < q; ++c) dir(x[b], x[b] * x[c], 1.0, x[a], w[a] * w[b] * w[c] * x[b]);
      for (int a = 0; a < q; ++a) radial(x[a], w[a] * x[a] * x[a], w[a] * x[a]);
      break;
    case CLS_EDGE:  // J = xi^3 h1^2 in the first region, xi^3 h1^2 h2 in the others; p = xi h1
      for (int reg = 0; reg < 5; ++reg)
        for (int b = 0; b < q; ++b)
          for (int c = 0; c < q; ++c) {
            const double u = x[b], v = x[c], wt = w[b] * w[c];
            switch (reg) {
              case 0: dir(u, v, 0.0, 1.0 - u, wt); break;
              case 1: dir(u * v, 1.0, 0.0, u * (1.0 - v), wt * u); break;
              case 2: dir(-u, 1.0 - u, 0.0, u * v, wt * u); break;
              case 3: dir(-u * v, u * (1.0 - v), 0.0, 1.0, wt * u); break;
              default: dir(-u * v, 1.0 - u * v, 0.0, u, wt * u); break;
            }
          }
      // xi_a h_b = xi_b h_a: one node for both
      for (int a = 0; a < q; ++a)
        for (int b = a; b < q; ++b) {
          double ws = w[a] * w[b] * x[a] * x[a] * x[b], wd = w[a] * w[b] * x[a];
          if (b != a) ws += w[a] * w[b] * x[b] * x[b] * x[a], wd += w[a] * w[b] * x[b];
          radial(x[a] * x[b], ws, wd);
        }
      break;
    case CLS_IDENTICAL:  // J = xi^3 h1^2 h2; p = xi h1 h2
      for (int a = 0; a < q; ++a) dir(x[a], 1.0, 0.0, 0.0, 2.0 * w[a]);
      for (int a = 0; a < q; ++a) dir(1.0, x[a], 0.0, 0.0, 2.0 * w[a]);
      for (int a = 0; a < q; ++a) dir(-x[a], 1.0 - x[a], 0.0, 0.0, 2.0 * w[a]);
      for (int a = 0; a < q; ++a)
        for (int b = a; b < q; ++b)
          for (int c = b; c < q; ++c) {
            // xi^2 h1 of every distinct order of the three nodes
            const double t[3] = {x[a], x[b], x[c]};
            double ws = 0.0;
            int orders = 0;
            for (int i = 0; i < 3; ++i)
              for (int j = 0; j < 3; ++j)
                if (i != j) ws += t[i] * t[i] * t[j], ++orders;
            const int distinct = a == b && b == c ? 1 : a == b || b == c ? 3 : 6;
            radial(t[0] * t[1] * t[2], ws * distinct / orders * w[a] * w[b] * w[c], 0.0);
          }
      break;
    default: throw std::invalid_argument("class");
  }
  // Helmholtz: sum_p ws e^{i p t} and sum_p wd (1 - i p t) e^{i p t} as power
  // series in t = kappa |d|, split into even and odd powers of t (the
  // coefficient of (i t)^k is mu_k / k!, resp. nu_k (1 - k) / k!); the first
  // even coefficients are the Laplace moments
  double fact = 1.0;
  for (int k = 0; k < 2 * kSeries; ++k) {
    if (k) fact *= k;
    double mu = 0.0, nu = 0.0;
    for (size_t i = 0; i < r.p.size(); ++i) {
      const double pk = std::pow(r.p[i], k);
      mu += r.ws[i] * pk;
      nu += r.wd[i] * pk;
    }
    const double sgn = (k / 2) % 2 ? -1.0 : 1.0;
    r.series[k % 2][k / 2] = sgn * mu / fact;
    r.series[2 + k % 2][k / 2] = sgn * nu * (1 - k) / fact;
  }
  return r;
}

XiRule xi_rule(int q) {
  if (q < 1 || q > BEM_MAX_ORDER) throw std::invalid_argument("order");
  std::vector<double> gx(q), gw(q);
  gauss_legendre01(q, gx.data(), gw.data());
  XiRule r;
  for (int a = 0; a < q; ++a) {
    r.x.push_back(gx[a]);
    r.w3.push_back(gw[a] * gx[a] * gx[a] * gx[a]);
  }
  return r;
}

}  // namespace bem
