// Host side of the C ABI: descriptor checks, grid tables, device uploads and
// the exported entry points.  Tables follow the paper's grid design (Sec. 3.1),
// the refinement matrices R = A_s A^-1 (Eqs. 12-19) and the implicit z
// diffusion of the scalar step (Eqs. 2, 5-7).
#include <math.h>
#include <string.h>

#include <algorithm>
#include <cstdlib>
#include <new>
#include <vector>

#include <rocprofiler-sdk-roctx/roctx.h>

#include "mr_internal.h"

namespace {

using std::vector;

struct Axis {
  int n = 0, m = 1, nc = 0;
  bool periodic = true;
  vector<double> f, h, c, dc;  // faces, widths, centres, centre distances across faces
};

int build_axis(const double* faces, int n, int m, bool periodic, Axis& ax) {
  if (!faces || n < 1 || m < 1 || n % m) return MR_EINVAL;
  ax.n = n;
  ax.m = m;
  ax.nc = n / m;
  ax.periodic = periodic;
  ax.f.assign(faces, faces + n + 1);
  for (int i = 0; i <= n; ++i)
    if (!std::isfinite(ax.f[i])) return MR_EINVAL;
  for (int i = 0; i < n; ++i)
    if (!(ax.f[i + 1] > ax.f[i])) return MR_EINVAL;
  ax.h.resize(n);
  ax.c.resize(n);
  for (int i = 0; i < n; ++i) {
    ax.h[i] = ax.f[i + 1] - ax.f[i];
    ax.c[i] = 0.5 * (ax.f[i] + ax.f[i + 1]);
  }
  if (periodic) {
    const double len = ax.f[n] - ax.f[0];
    ax.dc.resize(n);
    for (int i = 0; i < n; ++i) ax.dc[i] = ax.c[i] - (i ? ax.c[i - 1] : ax.c[n - 1] - len);
  } else {
    ax.dc.resize(n + 1);
    ax.dc[0] = 0.5 * ax.h[0];
    ax.dc[n] = 0.5 * ax.h[n - 1];
    for (int i = 1; i < n; ++i) ax.dc[i] = ax.c[i] - ax.c[i - 1];
  }
  return MR_OK;
}

// True when the widths of the axis are equal to within 1e-13 relative.
bool uniform_axis(const Axis& ax) {
  const double h0 = ax.h[0];
  for (double h : ax.h)
    if (fabs(h - h0) > 1e-13 * h0) return false;
  return true;
}

// Fourth-order face weights of an axis (Sec. 2.2): the stencil of face f is
// the two cells on each side of it, cells f-2..f+1.  On a walled axis only the
// cells that exist take part (three next to a wall cell, two when the axis has
// two cells) and the wall faces get zero rows; on a periodic axis the stencil
// wraps around, the cells beyond an end taking the period added to (or
// subtracted from) their coordinates, and face n repeats face 0.  The face
// value of the polynomial whose cell means equal the cell values is the
// derivative at the face of the polynomial that interpolates the primitive
// P(e_j) = sum_{s<j} h_s theta_s at the stencil's edges e_0..e_m, so cell s
// gets h_s * sum_{j>s} L_j'(x_f), L_j the Lagrange basis on the edges.
// Returns (n+1)*4 weights, face f's for the cells f-2..f+1 in that order.
vector<double> face_weights4(const Axis& ax) {
  const int n = ax.n;
  const double len = ax.f[n] - ax.f[0];
  // left edge of stencil cell c (beyond the ends of a periodic axis: the
  // edge of the cell it wraps to, shifted by whole periods)
  auto edge = [&](int c) {
    if (c >= 0 && c <= n) return ax.f[c];
    const int r = ((c % n) + n) % n;
    return ax.f[r] + (double)((c - r) / n) * len;
  };
  vector<double> w((size_t)(n + 1) * 4, 0.0);
  for (int f = ax.periodic ? 0 : 1; f < n; ++f) {
    int lo = f - 2, hi = f + 1;
    if (!ax.periodic) lo = std::max(lo, 0), hi = std::min(hi, n - 1);
    const int m = hi - lo + 1;
    const double xf = ax.f[f], sc = ax.h[f];
    double e[5];
    for (int q = 0; q <= m; ++q) e[q] = (edge(lo + q) - xf) / sc;
    double dl[5];   // L_j'(0)
    for (int jj = 0; jj <= m; ++jj) {
      double sum = 0.0;
      for (int l = 0; l <= m; ++l) {
        if (l == jj) continue;
        double prod = 1.0 / (e[jj] - e[l]);
        for (int r = 0; r <= m; ++r)
          if (r != jj && r != l) prod *= (0.0 - e[r]) / (e[jj] - e[r]);
        sum += prod;
      }
      dl[jj] = sum;
    }
    for (int q = 0; q < m; ++q) {
      double acc = 0.0;
      for (int jj = q + 1; jj <= m; ++jj) acc += dl[jj];
      w[(size_t)f * 4 + (lo + q - (f - 2))] = (e[q + 1] - e[q]) * acc;
    }
  }
  if (ax.periodic)
    for (int q = 0; q < 4; ++q) w[(size_t)n * 4 + q] = w[q];
  return w;
}

// Means of 1, x, x^2 over [a, b]: a row of A (Eq. 15) or A_s (Eq. 18).
void interval_means(double a, double b, double* row) {
  row[0] = 1.0;
  row[1] = 0.5 * (a + b);
  row[2] = (a * a + a * b + b * b) / 3.0;
}

// Solve the 3x3 system M y = rhs by Gaussian elimination with partial pivoting.
bool solve3(double M[3][3], double rhs[3], double y[3]) {
  int p[3] = {0, 1, 2};
  double A[3][4];
  for (int r = 0; r < 3; ++r) {
    for (int c = 0; c < 3; ++c) A[r][c] = M[r][c];
    A[r][3] = rhs[r];
  }
  for (int col = 0; col < 3; ++col) {
    int piv = col;
    for (int r = col + 1; r < 3; ++r)
      if (fabs(A[r][col]) > fabs(A[piv][col])) piv = r;
    if (A[piv][col] == 0.0) return false;
    if (piv != col)
      for (int c = 0; c < 4; ++c) std::swap(A[piv][c], A[col][c]);
    for (int r = col + 1; r < 3; ++r) {
      const double f = A[r][col] / A[col][col];
      for (int c = col; c < 4; ++c) A[r][c] -= f * A[col][c];
    }
  }
  (void)p;
  for (int r = 2; r >= 0; --r) {
    double s = A[r][3];
    for (int c = r + 1; c < 3; ++c) s -= A[r][c] * y[c];
    y[r] = s / A[r][r];
  }
  return true;
}

int stencil_start(const Axis& ax, int I) {
  if (ax.periodic) return I - 1;
  return std::min(std::max(I - 1, 0), ax.nc - 3);
}

// R_I = A_s A^-1 for every coarse cell (local coordinate (x - centre)/H), and
// the wrapped stencil cell indices.  m = 1 gives R = [0 1 0] on the cell itself.
int refinement_table(const Axis& ax, vector<double>& R, vector<int>& idx, vector<int>& start) {
  const int nc = ax.nc, m = ax.m;
  R.assign((size_t)nc * m * 3, 0.0);
  idx.assign((size_t)nc * 3, 0);
  start.assign(nc, 0);
  if (m == 1) {
    for (int I = 0; I < nc; ++I) {
      R[(size_t)I * 3 + 1] = 1.0;
      for (int r = 0; r < 3; ++r) idx[I * 3 + r] = ((I - 1 + r) % nc + nc) % nc;
      start[I] = I - 1;
    }
    return MR_OK;
  }
  if (nc < 3) return MR_EINVAL;
  const double len = ax.f[ax.n] - ax.f[0];
  for (int I = 0; I < nc; ++I) {
    const double X0 = ax.f[(size_t)I * m], X1 = ax.f[(size_t)(I + 1) * m];
    const double centre = 0.5 * (X0 + X1), H = X1 - X0;
    const int s = stencil_start(ax, I);
    start[I] = s;
    double A[3][3];
    for (int r = 0; r < 3; ++r) {
      int cell = s + r;
      double shift = 0.0;
      if (ax.periodic) {
        if (cell < 0) { cell += nc; shift = -len; }
        if (cell >= nc) { cell -= nc; shift = len; }
      }
      idx[I * 3 + r] = cell;
      const double a = (ax.f[(size_t)cell * m] + shift - centre) / H;
      const double b = (ax.f[(size_t)(cell + 1) * m] + shift - centre) / H;
      interval_means(a, b, A[r]);
    }
    // R A = A_s  <=>  A^T R^T = A_s^T : one 3x3 solve per sub-interval row
    double At[3][3];
    for (int r = 0; r < 3; ++r)
      for (int c = 0; c < 3; ++c) At[r][c] = A[c][r];
    for (int q = 0; q < m; ++q) {
      const double a = (ax.f[(size_t)I * m + q] - centre) / H;
      const double b = (ax.f[(size_t)I * m + q + 1] - centre) / H;
      double row[3], y[3];
      interval_means(a, b, row);
      double Mt[3][3];
      memcpy(Mt, At, sizeof(Mt));
      if (!solve3(Mt, row, y)) return MR_EINVAL;
      for (int r = 0; r < 3; ++r) R[((size_t)I * m + q) * 3 + r] = y[r];
    }
  }
  return MR_OK;
}

struct Problem {
  Axis x, y, z;
  double kappa = 0.0;
  bool sweep_ok = false;   // the column-sweep step applies
};

int check_desc(const mr_desc* d, Problem& P) {
  if (!d) return MR_EINVAL;
  if (d->ncx < 1 || d->ncy < 1 || d->ncz < 1 || d->mx < 1 || d->my < 1 || d->mz < 1) return MR_EINVAL;
  const int64_t nx = (int64_t)d->ncx * d->mx, ny = (int64_t)d->ncy * d->my, nz = (int64_t)d->ncz * d->mz;
  if (nx > (1 << 20) || ny > (1 << 20) || nz > (1 << 20)) return MR_ESHAPE;
  if (nx * ny * (nz + 1) > (int64_t)INT32_MAX) return MR_ESHAPE;   // kernels index with int32
  if ((d->mx > 1 && d->ncx < 3) || (d->my > 1 && d->ncy < 3) || (d->mz > 1 && d->ncz < 3)) return MR_EINVAL;
  if (d->bc_bot != MR_DIRICHLET && d->bc_bot != MR_ADIABATIC) return MR_EINVAL;
  if (d->bc_top != MR_DIRICHLET && d->bc_top != MR_ADIABATIC) return MR_EINVAL;
  if (d->precision != MR_FP64 && d->precision != MR_FP32) return MR_EINVAL;
  // the step kernels address a z level with 32-bit byte offsets
  if (nx * ny * (d->precision == MR_FP64 ? 8 : 4) > (int64_t)UINT32_MAX) return MR_ESHAPE;
  if (!(d->dt > 0.0) || !std::isfinite(d->dt)) return MR_EINVAL;
  if (!(d->ra > 0.0) || !(d->pr > 0.0) || !std::isfinite(d->ra * d->pr)) return MR_EINVAL;
  if (d->n_avg < 0) return MR_EINVAL;
  if (!std::isfinite(d->t_bot) || !std::isfinite(d->t_top)) return MR_EINVAL;
  if ((d->side_x != MR_PERIODIC && d->side_x != MR_WALLS) || (d->side_y != MR_PERIODIC && d->side_y != MR_WALLS))
    return MR_EINVAL;
  // explicit z share: up to 1/2 the z part stays unconditionally stable
  if (!(d->z_explicit >= 0.0 && d->z_explicit <= 0.5)) return MR_EINVAL;
  if (d->face_order != 0 && d->face_order != 2 && d->face_order != 4) return MR_EINVAL;
  if (d->step_method < 0 || d->step_method > 2) return MR_EINVAL;
  if (d->sweep_tile < 0 || d->sweep_tile > mr::kSweepShapes) return MR_EINVAL;
  if (d->sweep_tile == 1 && d->precision != MR_FP64) return MR_EINVAL;   // 256 x 4 is FP64 only
  int st;
  if ((st = build_axis(d->xf, (int)nx, d->mx, d->side_x == MR_PERIODIC, P.x)) != MR_OK) return st;
  if ((st = build_axis(d->yf, (int)ny, d->my, d->side_y == MR_PERIODIC, P.y)) != MR_OK) return st;
  if ((st = build_axis(d->zf, (int)nz, d->mz, false, P.z)) != MR_OK) return st;
  P.kappa = 1.0 / sqrt(d->ra * d->pr);
  // explicit x/y diffusion: the leapfrog step is forward Euler over 2 dt
  const double hxm = *std::min_element(P.x.h.begin(), P.x.h.end());
  const double hym = *std::min_element(P.y.h.begin(), P.y.h.end());
  const double num = 2.0 * d->dt * P.kappa * (4.0 / (hxm * hxm) + 4.0 / (hym * hym));
  if (!(num <= 1.0)) return MR_EINVAL;
  // column sweeps: x and y periodic with uniform widths, the plain method
  P.sweep_ok = d->side_x == MR_PERIODIC && d->side_y == MR_PERIODIC && uniform_axis(P.x) &&
               uniform_axis(P.y) && d->z_explicit == 0.0 && d->face_order != 4;
  if (d->step_method == 2 && !P.sweep_ok) return MR_EINVAL;
  // columns beyond the line solver's chunks need the sweeps
  if (nz > (int64_t)mr::kMaxChunks * mr::kMaxChunkLen && (!P.sweep_ok || d->step_method == 1))
    return MR_ESHAPE;
  return MR_OK;
}

double kind_tau(int kind, double dt) {
  return kind == mr::KIND_STARTUP ? dt : (kind == mr::KIND_AVERAGE ? 1.5 * dt : 2.0 * dt);
}

// Tridiagonal I - tk Lz (rows k: sub couples k-1, sup couples k+1) and the
// Dirichlet wall source b_z with Lz theta = Lz0 theta + b_z.
void z_system(const Axis& z, const mr_desc* d, double tk, double* sub, double* diag, double* sup,
              double* bz) {
  const int nz = z.n;
  for (int k = 0; k < nz; ++k) {
    const double lo = k > 0 ? -tk / (z.h[k] * z.dc[k]) : 0.0;
    const double hi = k < nz - 1 ? -tk / (z.h[k] * z.dc[k + 1]) : 0.0;
    if (sub) sub[k] = lo;
    if (sup) sup[k] = hi;
    double dg = 1.0 - lo - hi;
    double b = 0.0;
    if (k == 0 && d->bc_bot == MR_DIRICHLET) {
      dg += tk / (z.h[0] * z.dc[0]);
      b += d->t_bot / (z.h[0] * z.dc[0]);
    }
    if (k == nz - 1 && d->bc_top == MR_DIRICHLET) {
      dg += tk / (z.h[nz - 1] * z.dc[nz]);
      b += d->t_top / (z.h[nz - 1] * z.dc[nz]);
    }
    if (diag) diag[k] = dg;
    if (bz) bz[k] = b;
  }
}

// Host image of one ZSys.
struct ZHost {
  vector<double> m, a, cp, G, B, Fe, Gs, Bs, tkb;
};

// Thomas factors and chunk coupling vectors of the system (sub, diag, sup),
// for chunks [c L, (c+1) L).  The tables are padded to nch*L rows: rows k >= nz
// are identity rows decoupled from the system (m = 1, a = cp = 0), so every
// chunk has exactly L rows.  With the forward sweep d_k = m_k r_k + a_k d_{k-1}
// and back substitution x_k = d_k - cp_k x_{k+1}, a chunk that starts its
// sweeps from zero gets x_hat; the true solution is x_k = x_hat_k + D G_k + X B_k
// with D = d at the level below the chunk and X = x at the level above it.
bool z_factors(int nz, int L, const double* sub, const double* diag, const double* sup, ZHost& z) {
  const int nch = (nz + L - 1) / L;
  const int np = nch * L;
  z.m.assign(np, 1.0); z.a.assign(np, 0.0); z.cp.assign(np, 0.0); z.G.assign(np, 0.0); z.B.assign(np, 0.0);
  z.Fe.resize(nch); z.Gs.resize(nch); z.Bs.resize(nch);
  double cprev = 0.0;
  for (int k = 0; k < nz; ++k) {
    const double den = diag[k] - (k ? sub[k] * cprev : 0.0);
    if (den == 0.0 || !std::isfinite(den)) return false;
    z.m[k] = 1.0 / den;
    z.a[k] = k ? -sub[k] * z.m[k] : 0.0;
    z.cp[k] = k < nz - 1 ? sup[k] * z.m[k] : 0.0;
    cprev = z.cp[k];
  }
  vector<double> F(np);
  for (int c = 0; c < nch; ++c) {
    const int k0 = c * L, k1 = k0 + L;
    double f = 1.0;
    for (int k = k0; k < k1; ++k) { f *= z.a[k]; F[k] = f; }
    double g = 0.0, b = 1.0;
    for (int k = k1 - 1; k >= k0; --k) {
      g = F[k] - z.cp[k] * g;
      z.G[k] = g;
      b *= -z.cp[k];
      z.B[k] = b;
    }
    z.Fe[c] = F[k1 - 1];
    z.Gs[c] = z.G[k0];
    z.Bs[c] = z.B[k0];
  }
  return true;
}

// Factors of the column-sweep steps for the system (sub, diag, sup), both
// elimination directions: upward (the Thomas factors above, back substitution
// downward) and downward (the mirrored recurrences, back substitution upward).
struct SweepHost {
  vector<double> up_m, up_a, up_cb, dn_m, dn_a, dn_cb, tkb;
};

bool sweep_factors(int nz, const double* sub, const double* diag, const double* sup, SweepHost& z) {
  z.up_m.assign(nz, 0.0); z.up_a.assign(nz, 0.0); z.up_cb.assign(nz, 0.0);
  z.dn_m.assign(nz, 0.0); z.dn_a.assign(nz, 0.0); z.dn_cb.assign(nz, 0.0);
  double c = 0.0;
  for (int k = 0; k < nz; ++k) {
    const double den = diag[k] - (k ? sub[k] * c : 0.0);
    if (den == 0.0 || !std::isfinite(den)) return false;
    z.up_m[k] = 1.0 / den;
    z.up_a[k] = k ? -sub[k] * z.up_m[k] : 0.0;
    z.up_cb[k] = k < nz - 1 ? sup[k] * z.up_m[k] : 0.0;
    c = z.up_cb[k];
  }
  c = 0.0;
  for (int k = nz - 1; k >= 0; --k) {
    const double den = diag[k] - (k < nz - 1 ? sup[k] * c : 0.0);
    if (den == 0.0 || !std::isfinite(den)) return false;
    z.dn_m[k] = 1.0 / den;
    z.dn_a[k] = k < nz - 1 ? -sup[k] * z.dn_m[k] : 0.0;
    z.dn_cb[k] = k > 0 ? sub[k] * z.dn_m[k] : 0.0;
    c = z.dn_cb[k];
  }
  return true;
}

// Number of walk positions after (cb) or before (a) each position whose values
// still matter to its solution or elimination value: the shortest distance over
// which the product of the recurrence's factors falls to eps.  `out` takes the
// larger of itself and that; one product moves along with both ends.
template <typename At, typename Out>
void reach(int n, At factor, double eps, Out out) {
  double p = 1.0;
  int e = 0;   // p: the product of the factors s .. e-1
  for (int s = 0; s < n; ++s) {
    if (e < s) e = s, p = 1.0;
    while (e < n && p > eps) p *= fabs(factor(e++));
    out(s) = std::max(out(s), e - s);
    const double f = fabs(factor(s));
    if (f > 0.0 && p > 0.0) p /= f;
    else e = s + 1, p = 1.0;   // (a zero factor ends every reach; start anew)
  }
}
// Lz0 rows (a Dirichlet wall adds to the diagonal; its wall value is the
// separate source b_z), padded with zeros to n.
struct LzRows {
  vector<double> lo, di, hi;
};
LzRows lz0_rows(const Axis& z, const mr_desc* d, int n) {
  const int nz = z.n;
  const vector<double>&h = z.h, &dc = z.dc;
  LzRows r{vector<double>(n, 0.0), vector<double>(n, 0.0), vector<double>(n, 0.0)};
  for (int k = 0; k < nz; ++k) {
    r.lo[k] = k > 0 ? 1.0 / (h[k] * dc[k]) : 0.0;
    r.hi[k] = k < nz - 1 ? 1.0 / (h[k] * dc[k + 1]) : 0.0;
    double dg = -(r.lo[k] + r.hi[k]);
    if (k == 0 && d->bc_bot == MR_DIRICHLET) dg -= 1.0 / (h[0] * dc[0]);
    if (k == nz - 1 && d->bc_top == MR_DIRICHLET) dg -= 1.0 / (h[nz - 1] * dc[nz]);
    r.di[k] = dg;
  }
  return r;
}

// One system's streaming tables in one walk direction, by walk position.
struct StreamHost {
  vector<double> m, a, cb;
};
StreamHost stream_walk(const SweepHost& h, bool down) {
  StreamHost w;
  w.m = down ? h.dn_m : h.up_m;
  w.a = down ? h.dn_a : h.up_a;
  w.cb = down ? h.dn_cb : h.up_cb;
  // the downward factors pair with an upward back substitution: theta_k = e_k - dn_cb_k theta_{k-1}
  if (down)
    for (vector<double>* v : {&w.m, &w.a, &w.cb}) std::reverse(v->begin(), v->end());
  return w;
}

template <typename T>
vector<mr::StreamRow<T>> stream_rows(const vector<double>& ihz, const SweepHost& h, const StreamHost& walk, bool rev,
                                     bool down) {
  const int nz = (int)ihz.size();
  vector<mr::StreamRow<T>> r((size_t)nz + 2 * mr::kStreamRowPad);
  memset((void*)r.data(), 0, r.size() * sizeof(r[0]));
  for (int s = 0; s < nz; ++s) {
    const int k = down ? nz - 1 - s : s;
    mr::StreamRow<T>& o = r[(size_t)s + mr::kStreamRowPad];
    o.em = walk.m[s];
    o.ea = walk.a[s];
    o.tkb = h.tkb[k];
    // 1/hz of this level, of the one below and of the one above (0: a wall)
    const double ih = ihz[k], ihl = k > 0 ? ihz[k - 1] : 0.0, ihh = k < nz - 1 ? ihz[k + 1] : 0.0;
    const double lo = k > 0 ? ih : 0.0, hi = k < nz - 1 ? ih : 0.0;
    if (rev) {
      o.c0 = (T)(down ? -ihl : ihh);
      o.c1 = (T)(down ? -lo : hi);
      o.c2 = (T)(down ? -hi : lo);
      o.c3 = (T)(down ? -ihh : ihl);
    } else {
      if (sizeof(T) == 8) {
        o.c0 = (T)(down ? -lo : hi);
        o.c2 = (T)(down ? hi : -lo);
      } else {
        o.c0 = (T)((down ? lo : hi) != 0.0);
        o.c1 = (T)ih;
        o.c2 = (T)((down ? hi : lo) != 0.0);
      }
    }
  }
  return r;
}

// The variants' streaming rows of one step kind (tau), by walk position.
template <typename T>
vector<mr::VarRow<T>> variant_rows(const Problem& P, const mr_desc* d, const SweepHost& h, double tau) {
  const Axis& z = P.z;
  const int nz = z.n;
  vector<mr::VarRow<T>> r((size_t)nz + 2 * mr::kStreamRowPad);
  memset((void*)r.data(), 0, r.size() * sizeof(r[0]));
  const vector<double> w4 = face_weights4(z);
  const LzRows lz = lz0_rows(z, d, nz);
  const double tkw = tau * P.kappa * d->z_explicit;
  for (int k = 0; k < nz; ++k) {
    mr::VarRow<T>& c = r[(size_t)k + 2 + mr::kStreamRowPad];   // closes level k
    c.em = h.up_m[k];
    c.ea = h.up_a[k];
    c.tkb = h.tkb[k];
    c.tz = (T)(tau / z.h[k]);
    mr::VarRow<T>& o = r[(size_t)k + 1 + mr::kStreamRowPad];   // face k and level k's explicit share
    for (int q = 0; q < 4 && k > 0; ++q)
      o.cz[q] = (T)(d->face_order == 4 ? w4[(size_t)k * 4 + q] : (q == 1 || q == 2 ? 0.5 : 0.0));
    o.lz[0] = (T)(tkw * lz.lo[k]);
    o.lz[1] = (T)(tkw * lz.di[k]);
    o.lz[2] = (T)(tkw * lz.hi[k]);
  }
  return r;
}

vector<double> stream_cb(const StreamHost& w) {
  vector<double> cb(w.cb.size() + 2 * mr::kStreamPad, 0.0);
  std::copy(w.cb.begin(), w.cb.end(), cb.begin() + mr::kStreamPad);
  return cb;
}

// Chunk length and count of the line solver for `tiles` column tiles (one
// workgroup each) of nz levels.  A chunk is one wavefront's serial walk, so
// short chunks shorten the step until the registers of a CU run out (about 8
// wavefronts).  One round of tiles: the shortest chunks that make at most 8.
// Several rounds: at most 4, so that two workgroups share a CU; columns too
// tall for that, chunks of 24 if they make at most 8 (with 32 a workgroup of 5
// or 6 wavefronts leaves the rest of its CU idle).  Taller ones: the shortest
// of 32, 36 and 40 that makes at most 16.  The plain FP64 step in several rounds
// takes chunks of 24 from 161 levels on only (150^3 61 us with 32, 63 with 24;
// 300 x 280 x 90 108 and 123).  One step in us, against chunks of 32:
// 64^3 13.3 to 28.0 (FP64), 9.3 to 17.6 (FP32); 128^3 26 to 35, 15.8 to 19.5;
// 160 x 160 x 64 24.4 to 35.4, 15.2 to 20.5; 251 x 251 x 192 168 to 204, 86 to
// 106; side walls, fourth-order faces and an explicit z share at 186^3 134 to
// 160, 78 to 101; the same at 251 x 251 x 128 with chunks of 16 (8 of them)
// instead of 32 (4): 133 to 122.
// FP64 with 3 to 4 tiles a CU: two chunks for 33 to 64 levels (the tiles are all
// resident and the CU has its 8 wavefronts): 256 x 256 x 64 48.8 us with chunks of
// 16, 42.9 with 32; 224 x 224 x 64 44.9 and 39.5; 256 x 256 x 48 36.6 and 33.6 with
// 24; at 3 tiles and fewer a CU 16 is the faster or level (192 x 256 x 64 in fourth
// order 36 and 41).  There, 65 to 96 levels in second order: 32, not 24, whose reverse
// step takes 82 us against 69 with walls at 256 x 256 x 96 (forward 70 and 68).
int choose_chunks(int nz, int64_t tiles, int cus, bool f64, bool plain, bool ord4, int& L, int& nch) {
  const bool plain64 = f64 && plain, resident = f64 && tiles > 3 * (int64_t)cus && tiles <= 4 * (int64_t)cus;
  const int most = tiles <= cus ? 8 : resident && nz > 32 && nz <= 64 ? 2 : 4;
  const bool no24 = most == 4 && (plain64 || (resident && !ord4));
  L = 0;
  for (int l : mr::kChunkLens)
    if (!L && l <= 32 && l * most >= nz && (l != 24 || !no24)) L = l;
  if (!L && 24 * 8 >= nz && (!plain64 || nz > 160)) L = 24;
  for (int l : mr::kChunkLens)
    if (!L && l >= 32 && l * mr::kMaxChunks >= nz) L = l;
  if (!L) return MR_ESHAPE;
  nch = (nz + L - 1) / L;
  return MR_OK;
}

// One step of the line solver in us, estimated: the longest of
//   - one chunk's walk (a level 1.1 us in FP64, 0.58 in FP32), longer where more
//     than 8 wavefronts share a CU's registers;
//   - the levels that the fullest CU walks, at what a wavefront's level takes of a
//     busy CU (0.175 us, 0.092), five more a tile for its start and end;
//   - the six values of every cell (4.6 TB/s as long as they fit the Infinity Cache,
//     then 3.8 in FP64 and 4.3 in FP32);
// a tenth more where rows are not whole 64-byte lines (not the FP32 variants), and
// more for the variants (kl, kw).
// In us, estimated and timed: FP64 64 x 64 x 256 38 and 37, 128^3 22 and 25, 186^3 108
// and 102, 200^3 120 and 114, 320 x 320 x 64 85 and 77, 96 x 96 x 300 57 and 58, 256^3
// 212 and 199; FP32 128^3 12 and 14, 150^3 33 and 35, 200^3 84 and 77, 64 x 64 x 512 37
// and 35, 256^3 96 and 96; walls, fourth order and explicit z at 150 x 150 x 300 FP64
// 149 and 145, FP32 72 and 85; walls at 186 x 186 x 100 FP32 37 and 34.
double line_us(const Problem& P, const mr_desc* d, int64_t tiles, int cus, int L, int nch) {
  const bool f64 = d->precision == MR_FP64, ord4 = d->face_order == 4, expz = d->z_explicit > 0.0;
  const double kl = 1.0 + (ord4 ? 0.15 : 0.0) + (expz ? (f64 ? 0.1 : 0.4) : 0.0);
  const double kw = 1.0 + (ord4 && f64 ? 0.15 : 0.0) + (expz ? (f64 ? 0.15 : 0.1) : 0.0);
  const double levels = kw * nch * L;
  const double fill = std::min(1.0, (double)tiles / cus), rounds = (double)((tiles + cus - 1) / cus);
  double chunk = f64 ? 3.0 + 1.1 * L * kl : std::max(11.0, 3.0 + 0.58 * L * kl);
  if (nch > 8) {
    chunk *= 1.0 + (f64 ? 0.1 * (nch - 8) : P.sweep_ok ? 0.07 * (nch - 8) : 0.18 * std::min(nch - 8, 2));
    chunk *= 1.0 + 0.45 * std::min(fill, 0.6);
    if ((ord4 || expz) && nch > 12) chunk *= f64 ? 1.3 : 1.2;   // (128 registers a lane: these kernels spill)
  }
  const double walked = tiles > cus ? (f64 ? 0.175 : 0.092) * rounds * (levels + 5.0 * kw)
                                    : levels * (f64 ? 0.115 + 0.06 * fill : 0.055 + 0.037 * fill);
  const double bytes = (f64 ? 48.0 : 24.0) * P.x.n * P.y.n * P.z.n;
  const double mem = bytes / (bytes < 2.4e8 ? 4.6e6 : f64 ? 3.8e6 : 4.3e6);
  return std::max({chunk, walked, mem}) * (P.x.n * (f64 ? 8 : 4) % 64 && (f64 || P.sweep_ok) ? 1.1 : 1.0);
}

// Byte buffer that hands out 256-byte aligned slots.
struct Packer {
  vector<char> buf;
  size_t put(const void* p, size_t bytes) {
    size_t off = (buf.size() + 255) & ~(size_t)255;
    buf.resize(off + bytes);
    if (bytes) memcpy(buf.data() + off, p, bytes);
    return off;
  }
  template <typename T>
  size_t put(const vector<T>& v) { return put(v.data(), v.size() * sizeof(T)); }
};

template <typename T>
vector<T> cast(const vector<double>& v) { return vector<T>(v.begin(), v.end()); }

vector<double> inv(const vector<double>& v) {
  vector<double> o(v.size());
  for (size_t i = 0; i < v.size(); ++i) o[i] = 1.0 / v[i];
  return o;
}

struct GeomOffsets {
  size_t hx, ihx, idxc, hy, ihy, idyc, hz, ihz, iHX, iHY, Rx, Ry, Rz, sx, sy, sz, zlo, zhi;
  size_t lzl, lzd, lzh, lztl, lzth, c4z, c4zt, c4x, c4y;
};

template <typename T>
GeomOffsets pack_geom(Packer& pk, const Problem& P, const mr_desc* d, const vector<double>* R,
                      const vector<int>* idx, int npad) {
  GeomOffsets o;
  o.hx = pk.put(cast<T>(P.x.h));
  o.ihx = pk.put(cast<T>(inv(P.x.h)));
  o.idxc = pk.put(cast<T>(inv(P.x.dc)));
  o.hy = pk.put(cast<T>(P.y.h));
  o.ihy = pk.put(cast<T>(inv(P.y.h)));
  o.idyc = pk.put(cast<T>(inv(P.y.dc)));
  o.hz = pk.put(cast<T>(P.z.h));
  o.ihz = pk.put(cast<T>(inv(P.z.h)));
  vector<double> HX(P.x.nc), HY(P.y.nc);
  for (int I = 0; I < P.x.nc; ++I) HX[I] = 1.0 / (P.x.f[(size_t)(I + 1) * P.x.m] - P.x.f[(size_t)I * P.x.m]);
  for (int J = 0; J < P.y.nc; ++J) HY[J] = 1.0 / (P.y.f[(size_t)(J + 1) * P.y.m] - P.y.f[(size_t)J * P.y.m]);
  o.iHX = pk.put(cast<T>(HX));
  o.iHY = pk.put(cast<T>(HY));
  o.Rx = pk.put(cast<T>(R[0]));
  o.Ry = pk.put(cast<T>(R[1]));
  o.Rz = pk.put(cast<T>(R[2]));
  o.sx = pk.put(idx[0]);
  o.sy = pk.put(idx[1]);
  o.sz = pk.put(idx[2]);
  // interior-face masks of the z levels (the walls carry no advective flux),
  // zero on the padding rows of the line solver
  vector<double> lo(npad, 0.0), hi(npad, 0.0);
  for (int k = 0; k < P.z.n; ++k) {
    lo[k] = k > 0 ? 1.0 : 0.0;
    hi[k] = k < P.z.n - 1 ? 1.0 : 0.0;
  }
  o.zlo = pk.put(cast<T>(lo));
  o.zhi = pk.put(cast<T>(hi));
  const int nz = P.z.n;
  const LzRows lz = lz0_rows(P.z, d, npad);
  const vector<double>&zl = lz.lo, &zd = lz.di, &zh = lz.hi;
  vector<double> ztl(npad, 0.0), zth(npad, 0.0);   // the transpose
  for (int k = 0; k < nz; ++k) {
    ztl[k] = k > 0 ? zh[k - 1] : 0.0;
    zth[k] = k < nz - 1 ? zl[k + 1] : 0.0;
  }
  o.lzl = pk.put(cast<T>(zl));
  o.lzd = pk.put(cast<T>(zd));
  o.lzh = pk.put(cast<T>(zh));
  o.lztl = pk.put(cast<T>(ztl));
  o.lzth = pk.put(cast<T>(zth));
  // fourth-order z faces, padded: faces 0..npad, cells per level 0..npad-1
  const vector<double> w4 = face_weights4(P.z);
  vector<double> c4((size_t)(npad + 1) * 4, 0.0), c4t((size_t)npad * 4, 0.0);
  for (int f = 0; f <= nz; ++f)
    for (int q = 0; q < 4; ++q) c4[(size_t)f * 4 + q] = w4[(size_t)f * 4 + q];
  for (int k = 0; k < nz; ++k)
    for (int q = 0; q < 4; ++q) {
      const int f = k - 1 + q;   // cell k is slot 3 - q of face k - 1 + q
      if (f >= 0 && f <= nz) c4t[(size_t)k * 4 + q] = w4[(size_t)f * 4 + (3 - q)];
    }
  o.c4z = pk.put(cast<T>(c4));
  o.c4zt = pk.put(cast<T>(c4t));
  o.c4x = pk.put(cast<T>(face_weights4(P.x)));
  o.c4y = pk.put(cast<T>(face_weights4(P.y)));
  return o;
}

template <typename T>
mr::Geom<T> geom_ptrs(char* base, const GeomOffsets& o) {
  mr::Geom<T> g;
  g.hx = (const T*)(base + o.hx); g.ihx = (const T*)(base + o.ihx); g.idxc = (const T*)(base + o.idxc);
  g.hy = (const T*)(base + o.hy); g.ihy = (const T*)(base + o.ihy); g.idyc = (const T*)(base + o.idyc);
  g.hz = (const T*)(base + o.hz); g.ihz = (const T*)(base + o.ihz);
  g.iHX = (const T*)(base + o.iHX); g.iHY = (const T*)(base + o.iHY);
  g.Rx = (const T*)(base + o.Rx); g.Ry = (const T*)(base + o.Ry); g.Rz = (const T*)(base + o.Rz);
  g.sx = (const int*)(base + o.sx); g.sy = (const int*)(base + o.sy); g.sz = (const int*)(base + o.sz);
  g.zlo = (const T*)(base + o.zlo); g.zhi = (const T*)(base + o.zhi);
  g.lzl = (const T*)(base + o.lzl); g.lzd = (const T*)(base + o.lzd); g.lzh = (const T*)(base + o.lzh);
  g.lztl = (const T*)(base + o.lztl); g.lzth = (const T*)(base + o.lzth);
  g.c4z = (const T*)(base + o.c4z); g.c4zt = (const T*)(base + o.c4zt);
  g.c4x = (const T*)(base + o.c4x); g.c4y = (const T*)(base + o.c4y);
  return g;
}

struct ZOffsets {
  size_t m, a, cp, G, B, Fe, Gs, Bs, tkb;
};

ZOffsets pack_z(Packer& pk, const ZHost& z) {
  ZOffsets o;
  o.m = pk.put(z.m); o.a = pk.put(z.a); o.cp = pk.put(z.cp); o.G = pk.put(z.G); o.B = pk.put(z.B);
  o.Fe = pk.put(z.Fe); o.Gs = pk.put(z.Gs); o.Bs = pk.put(z.Bs); o.tkb = pk.put(z.tkb);
  return o;
}

struct SweepOffsets {
  size_t up_m, up_a, up_cb, dn_m, dn_a, dn_cb, tkb;
};

SweepOffsets pack_sweep(Packer& pk, const SweepHost& z) {
  SweepOffsets o;
  o.up_m = pk.put(z.up_m); o.up_a = pk.put(z.up_a); o.up_cb = pk.put(z.up_cb);
  o.dn_m = pk.put(z.dn_m); o.dn_a = pk.put(z.dn_a); o.dn_cb = pk.put(z.dn_cb);
  o.tkb = pk.put(z.tkb);
  return o;
}

mr::SweepSys sweep_ptrs(char* base, const SweepOffsets& o) {
  mr::SweepSys z;
  z.up_m = (const double*)(base + o.up_m); z.up_a = (const double*)(base + o.up_a);
  z.up_cb = (const double*)(base + o.up_cb); z.dn_m = (const double*)(base + o.dn_m);
  z.dn_a = (const double*)(base + o.dn_a); z.dn_cb = (const double*)(base + o.dn_cb);
  z.tkb = (const double*)(base + o.tkb);
  return z;
}

mr::ZSys z_ptrs(char* base, const ZOffsets& o) {
  mr::ZSys z;
  z.m = (const double*)(base + o.m); z.a = (const double*)(base + o.a); z.cp = (const double*)(base + o.cp);
  z.G = (const double*)(base + o.G); z.B = (const double*)(base + o.B);
  z.Fe = (const double*)(base + o.Fe); z.Gs = (const double*)(base + o.Gs); z.Bs = (const double*)(base + o.Bs);
  z.tkb = (const double*)(base + o.tkb);
  return z;
}

int hip_fail(mr_ctx* c, hipError_t e) {
  if (c) c->last_err = (int)e;
  (void)hipGetLastError();
  return MR_EHIP;
}

inline hipStream_t as_stream(void* s) { return (hipStream_t)s; }

size_t elem_size(const mr_ctx* c) { return c->precision == MR_FP64 ? 8 : 4; }

// A roctx range named after an entry point, around its host work and its
// launches, so that a marker trace (rocprofv3 --marker-trace) shows each call
// beside the kernels it enqueued.
struct CallRange {
  explicit CallRange(const char* name) { roctxRangePushA(name); }
  ~CallRange() { roctxRangePop(); }
  CallRange(const CallRange&) = delete;
  CallRange& operator=(const CallRange&) = delete;
};

}  // namespace

#define MR_CALL_RANGE() CallRange mr_call_range_(__func__)

// ===================================================================== C ABI
extern "C" {

const char* mr_status_string(int status) {
  switch (status) {
    case MR_OK: return "ok";
    case MR_EINVAL: return "invalid argument";
    case MR_ESHAPE: return "unsupported size";
    case MR_EHIP: return "HIP runtime error";
    case MR_ENOMEM: return "out of device memory";
    case MR_ENONFINITE: return "non-finite value in reduction";
    default: return "unknown status";
  }
}

int mr_last_hip_error(const mr_ctx* ctx) { return ctx ? ctx->last_err : 0; }

int mr_get_step_method(const mr_ctx* ctx, int32_t* method) {
  if (!ctx || !method) return MR_EINVAL;
  *method = ctx->sweep_pref ? 2 : 1;
  return MR_OK;
}

int mr_get_step_form(const mr_ctx* ctx, int32_t call, int32_t* form) {
  if (!ctx || !form || call < 0 || call > 3) return MR_EINVAL;
  const bool back = call >= 2, sequence = call & 1;
  if (sequence && ctx->sweep_flat) *form = 2;
  else if (ctx->stream_d || (!back && ctx->stream_v)) *form = 3;
  else if (sequence ? ctx->sweep_pref : back ? ctx->nch == 0 : ctx->sweep_single) *form = 2;
  else *form = 1;
  return MR_OK;
}

int mr_get_dims(const mr_ctx* ctx, int32_t* nx, int32_t* ny, int32_t* nz, int32_t* precision) {
  if (!ctx) return MR_EINVAL;
  if (nx) *nx = ctx->nx;
  if (ny) *ny = ctx->ny;
  if (nz) *nz = ctx->nz;
  if (precision) *precision = ctx->precision;
  return MR_OK;
}

int mr_host_refinement_table(const mr_desc* desc, int32_t axis, double* R_out, int32_t* start_out) {
  Problem P;
  int st = check_desc(desc, P);
  if (st != MR_OK) return st;
  if (axis < 0 || axis > 2) return MR_EINVAL;
  const Axis& ax = axis == 0 ? P.x : (axis == 1 ? P.y : P.z);
  vector<double> R;
  vector<int> idx, start;
  if ((st = refinement_table(ax, R, idx, start)) != MR_OK) return st;
  if (R_out) memcpy(R_out, R.data(), R.size() * sizeof(double));
  if (start_out)
    for (int I = 0; I < ax.nc; ++I) start_out[I] = start[I];
  return MR_OK;
}

int mr_host_z_system(const mr_desc* desc, int64_t n, double* sub, double* diag, double* sup,
                     double* bz, double* tau_out) {
  Problem P;
  int st = check_desc(desc, P);
  if (st != MR_OK) return st;
  if (n < 0) return MR_EINVAL;
  const double tau = kind_tau(mr::step_kind(n, desc->n_avg), desc->dt);
  z_system(P.z, desc, tau * P.kappa * (1.0 - desc->z_explicit), sub, diag, sup, bz);
  if (tau_out) *tau_out = tau;
  return MR_OK;
}

int mr_host_z_face_weights(const mr_desc* desc, double* w_out) {
  Problem P;
  int st = check_desc(desc, P);
  if (st != MR_OK) return st;
  if (!w_out) return MR_EINVAL;
  const vector<double> w = face_weights4(P.z);
  memcpy(w_out, w.data(), w.size() * sizeof(double));
  return MR_OK;
}

int mr_host_face_weights(const mr_desc* desc, int32_t axis, double* w_out) {
  Problem P;
  int st = check_desc(desc, P);
  if (st != MR_OK) return st;
  if (!w_out || axis < 0 || axis > 2) return MR_EINVAL;
  const vector<double> w = face_weights4(axis == 0 ? P.x : (axis == 1 ? P.y : P.z));
  memcpy(w_out, w.data(), w.size() * sizeof(double));
  return MR_OK;
}

int mr_init(const mr_desc* desc, mr_ctx** out) {
  MR_CALL_RANGE();
  if (!out) return MR_EINVAL;
  Problem P;
  int st = check_desc(desc, P);
  if (st != MR_OK) return st;
  int L = 0, nch = 0;
  // columns taller than the line solver's chunks: only the column-sweep step
  // (check_desc has made sure that it applies)
  int cus = 0, dev = 0;
  if (hipGetDevice(&dev) != hipSuccess ||
      hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus < 1)
    cus = 256;
  const int lrows = desc->precision == MR_FP64 ? 2 : 1, lcols = mr::kWave / lrows;   // patch of a line workgroup
  const int64_t ltiles = (int64_t)((P.x.n + lcols - 1) / lcols) * ((P.y.n + lrows - 1) / lrows);
  if (choose_chunks(P.z.n, ltiles, cus, desc->precision == MR_FP64, P.sweep_ok, desc->face_order == 4, L, nch) != MR_OK)
    L = nch = 0;
  const int npad = std::max(nch * L, P.z.n);

  vector<double> R[3];
  vector<int> idx[3], start[3];
  const Axis* axes[3] = {&P.x, &P.y, &P.z};
  for (int a = 0; a < 3; ++a)
    if ((st = refinement_table(*axes[a], R[a], idx[a], start[a])) != MR_OK) return st;

  Packer pk;
  GeomOffsets o64 = pack_geom<double>(pk, P, desc, R, idx, npad);
  GeomOffsets o32 = pack_geom<float>(pk, P, desc, R, idx, npad);
  ZOffsets zfo[mr::NKINDS], zto[mr::NKINDS];
  SweepOffsets swo[mr::NKINDS], swto[mr::NKINDS];
  double taus[mr::NKINDS];
  const int nz = P.z.n;
  const bool f64 = desc->precision == MR_FP64;
  // the implicit z systems of the step kinds and their factors
  struct Kind {
    vector<double> sub, diag, sup, bz, tsub, tsup;
    SweepHost sh, sht;
  };
  vector<Kind> kinds(mr::NKINDS);
  for (int kind = 0; kind < mr::NKINDS; ++kind) {
    Kind& q = kinds[kind];
    const double tau = kind_tau(kind, desc->dt);
    taus[kind] = tau;
    const double tk = tau * P.kappa;
    for (vector<double>* v : {&q.sub, &q.diag, &q.sup, &q.bz, &q.tsub, &q.tsup}) v->assign(nz, 0.0);
    // the implicit share (1 - w) of the z diffusion; the wall source stays whole
    z_system(P.z, desc, tk * (1.0 - desc->z_explicit), q.sub.data(), q.diag.data(), q.sup.data(), q.bz.data());
    if (!sweep_factors(nz, q.sub.data(), q.diag.data(), q.sup.data(), q.sh)) return MR_EINVAL;
    q.sh.tkb.assign(nz, 0.0);
    for (int k = 0; k < nz; ++k) q.sh.tkb[k] = tk * q.bz[k];
    // transpose: sub^T_k = sup_{k-1}, sup^T_k = sub_{k+1}
    for (int k = 0; k < nz; ++k) {
      q.tsub[k] = k > 0 ? q.sup[k - 1] : 0.0;
      q.tsup[k] = k < nz - 1 ? q.sub[k + 1] : 0.0;
    }
    // (the reverse steps' systems: no wall source)
    if (!sweep_factors(nz, q.tsub.data(), q.diag.data(), q.tsup.data(), q.sht)) return MR_EINVAL;
    q.sht.tkb.assign(nz, 0.0);
  }

  // the streaming step runs where it applies but on small grids where the line solver
  // is faster; the lines lie where the two are level at short look-aheads (longer ones:
  // below).  One step in us, streaming against line solver, 13 levels ahead:
  //   FP64 with copies into LDS of 4 bytes (odd N_x), 4.5e6 cells: 187 x 187 x 100 60 and
  //     65, 255 x 255 x 64 52 and 54, 127^3 48 and 28; 255^3 194 and 278;
  //   FP64 else, one round of tiles, 64 levels: 64^3 18 and 12, 128 x 128 x 64 25 and 15;
  //     64 x 64 x 96 18 and 20, 64 x 64 x 128 19 and 21;
  //   FP32, one round, 128 levels: 64 x 64 x 128 14 and 12, 128^3 22 and 14; 64 x 64 x 256
  //     18 and 20, 64 x 64 x 512 26 and 35;
  //   FP32, several rounds, 2.5e6 cells: 160 x 160 x 96 24 and 18, 192 x 192 x 64 24 and
  //     18, 200 x 200 x 60 (2.4e6) 24 and 25; 300 x 280 x 30 (2.52e6) 19 and 21, 186 x 186
  //     x 100 32 and 37
  const bool one_round = ltiles <= cus;
  const int64_t cells = (int64_t)P.x.n * P.y.n * nz;
  bool streams = P.sweep_ok && desc->step_method == 0 &&
                 (nch == 0 || cells >= 4500000 ||
                  (f64 ? P.x.n % 2 == 0 && !(one_round && nz <= 64) : (one_round ? nz > 128 : cells >= 2500000)));
  // the variants' forward step streams (x and y of uniform widths) on grids of 2.5e6
  // cells and more (FP64 with 4-byte copies 4.5e6) and on tall columns in one round of
  // tiles.  Streaming against line solver, with walls, fourth order and explicit z / with
  // walls alone: FP64 186^3 75 and 126 / 78 and 100, 256^3 184 and 232 / 180 and 200, 300 x
  // 280 x 30 29 and 39 / 28 and 36, 64 x 64 x 256 27 and 52 / 29 and 38; 160 x 160 x 64 33
  // and 27 / 33 and 23, 64^3 22 and 15 / 27 and 12; odd 255^3 183 and 298 / 167 and 267;
  // FP32 186^3 45 and 76 / 47 and 50, 300 x 280 x 30 20 and 20 / 19 and 19, 64 x 64 x 256 21
  // and 34 / 20 and 22; 160 x 160 x 64 22 and 18 / 22 and 14
  const bool copies4 = f64 && P.x.n % 2 != 0;
  bool streamv = !P.sweep_ok && desc->step_method == 0 && nch > 0 && uniform_axis(P.x) && uniform_axis(P.y) &&
                 (cells >= (copies4 ? 4500000 : 2500000) || (one_round && nz > 128 && !copies4));
  size_t vro[mr::NKINDS], vcbo[mr::NKINDS];
  const vector<double> ihz = inv(P.z.h);
  size_t sro[2][2][mr::NKINDS], scbo[2][2][mr::NKINDS];   // streaming tables: [transposed][down][kind]
  const double eps = f64 ? mr::kTruncate64 : mr::kTruncate32;
  int ahead = 0;                                      // the streaming step's look-ahead
  vector<int> after[2], before[2];                    // its reach after / before each walk position
  for (int d = 0; d < 2; ++d) after[d].assign(nz, 0), before[d].assign(nz, 0);
  auto add_reach = [&](const SweepHost& h, int d) {
    const StreamHost w = stream_walk(h, d);
    reach(nz, [&](int k) { return w.cb[k]; }, eps, [&](int k) -> int& { return after[d][k]; });
    reach(nz, [&](int k) { return w.a[nz - 1 - k]; }, eps, [&](int k) -> int& { return before[d][nz - 1 - k]; });
    ahead = std::max(ahead, *std::max_element(after[d].begin(), after[d].end()));
  };
  // the streaming step's look-ahead, tiles and z segments
  int stream_d = 0;
  mr::StreamPlan plan;
  if (streams || streamv) {
    for (const Kind& q : kinds) {
      add_reach(q.sh, 0);
      for (int d = 0; d < 2 && streams; ++d) add_reach(q.sht, d);
      if (streams) add_reach(q.sh, 1);
    }
    for (int d = mr::kStreamDepths; d > 0; --d)
      if (ahead <= mr::kStreamDepth[d - 1]) stream_d = d;
    if (stream_d) plan = mr::stream_plan(P.x.n, P.y.n, nz, f64, streamv, cus, stream_d - 1, before, after);
    // the bounds above were set at short look-aheads; a longer one is walked by every
    // segment of a column and takes a CU's registers: the estimates decide (up to 16
    // levels ahead with a twentieth in favour of streaming, where both err least that
    // way).  One step in us, line solver and streaming, by the look-ahead: FP64 128^3
    // 25 and 36 (16 levels), 46 (28), 44 (44), 57 (60), 192^3 96 and 87, 93, 97, 110, 64
    // x 64 x 256 37 and 23, 30, 38, 48; FP32 186^3 55 and 48, 65, 67, 78, 160 x 160 x 200
    // 38 and 34, 44, 52, 61; with walls, FP64 96 x 96 x 160 30 and 52 (28).  Of 2246 steps
    // timed in both forms over 73 grids and 7 look-aheads, 88 take 5% longer in the form
    // so chosen (the worst 1.5 times)
    const double favour = mr::kStreamDepth[std::max(stream_d - 1, 0)] <= 16 ? 1.05 : 1.0;
    if (stream_d == 0 || (nch > 0 && plan.us > favour * line_us(P, desc, ltiles, cus, L, nch))) {
      streams = streamv = false;
      stream_d = 0;
      plan = mr::StreamPlan();
    }
  }
  // (one allocation for the streaming tables: 13 sets of rows and back factors)
  if (streams) pk.buf.reserve(pk.buf.size() + 16 * (size_t)(nz + 2 * mr::kStreamPad) * (sizeof(mr::StreamRow<double>) + 64));
  auto pack_stream = [&](const SweepHost& h, int kind, bool rev) {
    if (!streams) return;
    for (int d = 0; d < 2; ++d) {
      const StreamHost w = stream_walk(h, d);
      sro[rev][d][kind] = f64 ? pk.put(stream_rows<double>(ihz, h, w, rev, d)) : pk.put(stream_rows<float>(ihz, h, w, rev, d));
      scbo[rev][d][kind] = pk.put(stream_cb(w));
    }
  };
  for (int kind = 0; kind < mr::NKINDS; ++kind) {
    const Kind& q = kinds[kind];
    swo[kind] = pack_sweep(pk, q.sh);
    pack_stream(q.sh, kind, false);
    if (streamv) {
      const double tau = taus[kind];
      vro[kind] = f64 ? pk.put(variant_rows<double>(P, desc, q.sh, tau)) : pk.put(variant_rows<float>(P, desc, q.sh, tau));
      vcbo[kind] = pk.put(stream_cb(stream_walk(q.sh, false)));
    }
    swto[kind] = pack_sweep(pk, q.sht);
    pack_stream(q.sht, kind, true);
    if (nch == 0) continue;
    ZHost zh, th;
    if (!z_factors(nz, L, q.sub.data(), q.diag.data(), q.sup.data(), zh)) return MR_EINVAL;
    zh.tkb.assign((size_t)nch * L, 0.0);
    std::copy(q.sh.tkb.begin(), q.sh.tkb.end(), zh.tkb.begin());
    if (!z_factors(nz, L, q.tsub.data(), q.diag.data(), q.tsup.data(), th)) return MR_EINVAL;
    th.tkb.assign((size_t)nch * L, 0.0);
    zfo[kind] = pack_z(pk, zh);
    zto[kind] = pack_z(pk, th);
  }
  // identity factors for the start-up step's reverse sweep (no solve)
  SweepHost shid;
  shid.up_m.assign(nz, 1.0); shid.dn_m.assign(nz, 1.0);
  shid.up_a.assign(nz, 0.0); shid.dn_a.assign(nz, 0.0);
  shid.up_cb.assign(nz, 0.0); shid.dn_cb.assign(nz, 0.0);
  shid.tkb.assign(nz, 0.0);
  const SweepOffsets swido = pack_sweep(pk, shid);
  size_t o_sid = 0, o_sidcb = 0;
  if (streams) {
    const StreamHost w = stream_walk(shid, false);
    o_sid = f64 ? pk.put(stream_rows<double>(ihz, shid, w, true, false)) : pk.put(stream_rows<float>(ihz, shid, w, true, false));
    o_sidcb = pk.put(stream_cb(w));
  }
  const size_t o_seg[2] = {pk.put(plan.seg[0]), pk.put(plan.seg[1])};
  vector<double> dcz(P.z.dc);
  size_t o_hx64 = pk.put(P.x.h), o_hy64 = pk.put(P.y.h), o_dcz = pk.put(dcz), o_idcz = pk.put(inv(dcz)), o_hz64 = pk.put(P.z.h);

  mr_ctx* c = new (std::nothrow) mr_ctx();
  if (!c) return MR_ENOMEM;
  memset((void*)c, 0, sizeof(mr_ctx));
  c->nx = P.x.n; c->ny = P.y.n; c->nz = P.z.n;
  c->ncx = P.x.nc; c->ncy = P.y.nc; c->ncz = P.z.nc;
  c->mx = desc->mx; c->my = desc->my; c->mz = desc->mz;
  c->precision = desc->precision;
  c->kappa = P.kappa; c->dt = desc->dt; c->ra = desc->ra; c->pr = desc->pr;
  c->t_bot = desc->t_bot; c->t_top = desc->t_top;
  c->bc_bot = desc->bc_bot; c->bc_top = desc->bc_top; c->n_avg = desc->n_avg;
  c->wx = desc->side_x == MR_WALLS;
  c->wy = desc->side_y == MR_WALLS;
  c->z_explicit = desc->z_explicit;
  c->face_order = desc->face_order == 4 ? 4 : 2;
  c->uniform_xy = !c->wx && !c->wy && uniform_axis(P.x) && uniform_axis(P.y);
  c->uhx = P.x.n / (P.x.f[P.x.n] - P.x.f[0]);
  c->uhy = P.y.n / (P.y.f[P.y.n] - P.y.f[0]);
  c->L = L; c->nch = nch;
  for (int k = 0; k < mr::NKINDS; ++k) c->tau[k] = taus[k];
  {
    // total horizontal area, compensated
    double s = 0.0, comp = 0.0;
    for (int j = 0; j < P.y.n; ++j)
      for (int i = 0; i < P.x.n; ++i) {
        const double v = P.x.h[i] * P.y.h[j];
        const double t = s + v;
        comp += fabs(s) >= fabs(v) ? (s - t) + v : (v - t) + s;
        s = t;
      }
    c->atot = s + comp;
    c->atot_lo = (s - c->atot) + comp;
    c->vtot = c->atot * (P.z.f[P.z.n] - P.z.f[0]);
  }
  hipError_t e = hipGetDevice(&c->device);
  if (e != hipSuccess) { int r = hip_fail(c, e); delete c; return r; }
  // the allocation-free entry point's fixed memory on this device
  e = mr::scratch_init(c->device);
  if (e != hipSuccess) { int r = hip_fail(c, e); delete c; return r; }
  e = hipMalloc(&c->tables, pk.buf.size());
  if (e != hipSuccess) { delete c; (void)hipGetLastError(); return MR_ENOMEM; }
  e = hipMemcpy(c->tables, pk.buf.data(), pk.buf.size(), hipMemcpyHostToDevice);
  if (e != hipSuccess) { (void)hipFree(c->tables); int r = hip_fail(c, e); delete c; return r; }
  char* base = (char*)c->tables;
  c->g64 = geom_ptrs<double>(base, o64);
  c->g32 = geom_ptrs<float>(base, o32);
  for (int k = 0; k < mr::NKINDS; ++k) {
    if (nch > 0) {
      c->zf[k] = z_ptrs(base, zfo[k]);
      c->zt[k] = z_ptrs(base, zto[k]);
    }
    c->sw[k] = sweep_ptrs(base, swo[k]);
    c->swt[k] = sweep_ptrs(base, swto[k]);
  }
  c->swid = sweep_ptrs(base, swido);
  // where nothing streams, step sequences run as column sweeps where the line solver cannot take the
  // columns, and where the sweep's tiles keep the GPU full: at least 16
  // wavefronts per CU in all, and either one round of tiles (one workgroup
  // per CU: the sweep kernels run 4 wavefronts per SIMD) or rounds at least
  // 3/4 full.  Measured in one run: at 256^3 (64 tiles of 256 x 4 columns)
  // the line solver is 2.7x (FP64) and 2.5x (FP32) faster; at 576^3 (432
  // tiles of 192 x 4) the sweeps are 10% and 20% faster; at 1024 x 1024 x 512
  // (1024 tiles) 27% and 25% faster.
  c->sweep_shape = desc->sweep_tile > 0 ? desc->sweep_tile - 1 : mr::sweep_pick_shape(c->nx, f64);
  const mr::SweepShape sh = mr::kSweepShape[c->sweep_shape];
  const int tw = 64 * sh.segs;
  const int64_t tiles = (int64_t)((c->nx + tw - 1) / tw) * ((c->ny + sh.rows - 1) / sh.rows);
  const int64_t slots = cus, rounds = (tiles + slots - 1) / slots;
  const bool fills = tiles * sh.segs * sh.rows >= 16 * (int64_t)cus && (rounds == 1 || 4 * tiles >= 3 * rounds * slots);
  c->sweep_pref = desc->step_method == 2 || (desc->step_method == 0 && P.sweep_ok && (nch == 0 || fills));
  c->sweep_single = nch == 0 || desc->step_method == 2;
  c->stream_d = streams ? stream_d : 0;
  c->stream_v = streamv ? stream_d : 0;
  // a streaming step walks 8 levels at least and one behind: sequences on flat grids
  // whose sweep tiles keep the GPU full run as sweeps, us a step FP64 / FP32: 1024 x
  // 1024 columns of 2 levels 35.6 / 23.8 and 47.9 / 38.5 streaming, of 3 levels 46.9 / 30.8
  // and 54.3 / 40.9, of 4 57.7 / 38.8 and 58.5 / 41.8; 768 x 512 of 4 27.1 and 22.7 / 16.6 and 17.0
  c->sweep_flat = c->stream_d && c->sweep_pref && nz <= (f64 ? 3 : 4);
  c->stream_shape = plan.shape;
  c->stream_nseg = plan.nseg;
  for (int d = 0; d < 2; ++d) c->stream_seg[d] = (const int*)(base + o_seg[d]);
  if (c->stream_d) {
    const double* cb = (const double*)(base + o_sidcb) + mr::kStreamPad;
    c->sid64 = {(const mr::StreamRow<double>*)(base + o_sid) + mr::kStreamRowPad, cb};
    c->sid32 = {(const mr::StreamRow<float>*)(base + o_sid) + mr::kStreamRowPad, cb};
  }
  for (int k = 0; k < mr::NKINDS && c->stream_v; ++k) {
    const size_t row = f64 ? sizeof(mr::VarRow<double>) : sizeof(mr::VarRow<float>);
    c->vrow[k] = base + vro[k] + mr::kStreamRowPad * row;
    c->vcb[k] = (const double*)(base + vcbo[k]) + mr::kStreamPad;
  }
  for (int k = 0; k < mr::NKINDS && c->stream_d; ++k)
    for (int r = 0; r < 2; ++r)
      for (int d = 0; d < 2; ++d) {
        const double* cb = (const double*)(base + scbo[r][d][k]) + mr::kStreamPad;
        c->sr64[r][d][k] = {(const mr::StreamRow<double>*)(base + sro[r][d][k]) + mr::kStreamRowPad, cb};
        c->sr32[r][d][k] = {(const mr::StreamRow<float>*)(base + sro[r][d][k]) + mr::kStreamRowPad, cb};
      }
  c->hx64 = (const double*)(base + o_hx64);
  c->areaw = (const double*)(base + o_hy64);
  c->dcz = (const double*)(base + o_dcz);
  c->idcz = (const double*)(base + o_idcz);
  c->hz64 = (const double*)(base + o_hz64);
  *out = c;
  return MR_OK;
}

int mr_destroy(mr_ctx* ctx) {
  if (!ctx) return MR_OK;
  if (ctx->tables) (void)hipFree(ctx->tables);
  if (ctx->interp_tmp) (void)hipFree(ctx->interp_tmp);
  if (ctx->interp_bwd_tmp) (void)hipFree(ctx->interp_bwd_tmp);
  if (ctx->red) (void)hipFree(ctx->red);
  for (void* p : ctx->sweep_e)
    if (p) (void)hipFree(p);
  delete ctx;
  return MR_OK;
}

#define MR_LAUNCH(call)                              \
  do {                                               \
    hipError_t e_ = (call);                          \
    if (e_ != hipSuccess) return hip_fail(ctx, e_);  \
  } while (0)

int mr_interpolate_velocity(mr_ctx* ctx, const void* U, const void* V, const void* W, void* u,
                            void* v, void* w, void* stream) {
  MR_CALL_RANGE();
  if (!ctx || !U || !V || !W || !u || !v || !w) return MR_EINVAL;
  MR_LAUNCH(mr::launch_refine(ctx, U, V, W, u, v, w, as_stream(stream)));
  return MR_OK;
}

int mr_interpolate_velocity_backward(mr_ctx* ctx, const void* gu, const void* gv, const void* gw,
                                     void* gU, void* gV, void* gW, void* stream) {
  MR_CALL_RANGE();
  if (!ctx || !gu || !gv || !gw || !gU || !gV || !gW) return MR_EINVAL;
  MR_LAUNCH(mr::launch_refine_transpose(ctx, gu, gv, gw, gU, gV, gW, as_stream(stream)));
  return MR_OK;
}

int mr_divergence(mr_ctx* ctx, const void* u, const void* v, const void* w, double* dev_out,
                  void* stream) {
  MR_CALL_RANGE();
  if (!ctx || !u || !v || !w || !dev_out) return MR_EINVAL;
  MR_LAUNCH(mr::launch_divergence(ctx, u, v, w, dev_out, as_stream(stream)));
  return MR_OK;
}

// Whether a sequence on a flat grid can run as sweeps: their fields are allocated
// on first use, which a capture forbids (it streams then).
static bool flat_sweeps(mr_ctx* ctx, hipStream_t s) {
  if (!ctx->sweep_flat) return false;
  if (ctx->sweep_e[0] && ctx->sweep_e[1]) return true;
  hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(s, &st) != hipSuccess || st != hipStreamCaptureStatusNone) return false;
  if (mr::ensure_sweep_buffers(ctx) == hipSuccess) return true;
  (void)hipGetLastError();
  return false;
}

int mr_scalar_step(mr_ctx* ctx, int64_t n, const void* th_prev, const void* th_cur, void* th_next,
                   const void* u, const void* v, const void* w, void* stream) {
  MR_CALL_RANGE();
  if (!ctx || n < 0 || !th_cur || !th_next || !u || !v || !w) return MR_EINVAL;
  if (n > 0 && !th_prev) return MR_EINVAL;
  if (th_next == th_cur || th_next == th_prev) return MR_EINVAL;
  const void* thp = n > 0 ? th_prev : th_cur;
  if (ctx->stream_d) {
    MR_LAUNCH(mr::launch_stream_step(ctx, n, ctx->sweep_single ? 0 : -1, thp, th_cur, th_next, u, v, w,
                                     as_stream(stream)));
    return MR_OK;
  }
  if (ctx->stream_v) {
    MR_LAUNCH(mr::launch_stream_step_var(ctx, n, thp, th_cur, th_next, u, v, w, as_stream(stream)));
    return MR_OK;
  }
  if (ctx->sweep_single) {
    // one column sweep and its back substitution
    void* outs[1] = {th_next};
    MR_LAUNCH(mr::launch_sweep_steps(ctx, n, 1, thp, th_cur, outs, u, v, w, as_stream(stream)));
    return MR_OK;
  }
  MR_LAUNCH(mr::launch_step(ctx, n, thp, th_cur, th_next, u, v, w, as_stream(stream)));
  return MR_OK;
}

int mr_scalar_steps(mr_ctx* ctx, int64_t n0, int32_t count, const void* th_prev, const void* th_cur,
                    void* const* outs, const void* u, const void* v, const void* w, void* stream) {
  MR_CALL_RANGE();
  if (!ctx || n0 < 0 || count < 1 || !th_cur || !outs || !u || !v || !w) return MR_EINVAL;
  if (n0 > 0 && !th_prev) return MR_EINVAL;
  const void* thp = n0 > 0 ? th_prev : th_cur;
  // every output differs from the two levels before it
  for (int32_t q = 0; q < count; ++q) {
    const void* l1 = q >= 1 ? outs[q - 1] : th_cur;
    const void* l2 = q >= 2 ? outs[q - 2] : (q == 1 ? th_cur : thp);
    if (!outs[q] || outs[q] == l1 || outs[q] == l2) return MR_EINVAL;
  }
  hipStream_t s = as_stream(stream);
  const bool flat = flat_sweeps(ctx, s);
  if (ctx->stream_d && !flat) {
    for (int32_t q = 0; q < count; ++q) {
      const void* a = q >= 2 ? outs[q - 2] : (q == 1 ? th_cur : thp);
      const void* b = q >= 1 ? outs[q - 1] : th_cur;
      MR_LAUNCH(mr::launch_stream_step(ctx, n0 + q, ctx->sweep_pref ? q : -1, a, b, outs[q], u, v, w, s));
    }
    return MR_OK;
  }
  if (ctx->stream_v) {
    for (int32_t q = 0; q < count; ++q) {
      const void* a = q >= 2 ? outs[q - 2] : (q == 1 ? th_cur : thp);
      const void* b = q >= 1 ? outs[q - 1] : th_cur;
      MR_LAUNCH(mr::launch_stream_step_var(ctx, n0 + q, a, b, outs[q], u, v, w, s));
    }
    return MR_OK;
  }
  if (ctx->sweep_pref) {
    MR_LAUNCH(mr::launch_sweep_steps(ctx, n0, count, thp, th_cur, outs, u, v, w, s));
    return MR_OK;
  }
  for (int32_t q = 0; q < count; ++q) {
    const void* a = q >= 2 ? outs[q - 2] : (q == 1 ? th_cur : thp);
    const void* b = q >= 1 ? outs[q - 1] : th_cur;
    MR_LAUNCH(mr::launch_step(ctx, n0 + q, a, b, outs[q], u, v, w, s));
  }
  return MR_OK;
}

int mr_adjoint_seed(mr_ctx* ctx, int64_t n, const void* lam, void* mu_out, void* stream) {
  MR_CALL_RANGE();
  if (!ctx || n < 0 || !lam || !mu_out || lam == mu_out) return MR_EINVAL;
  if (ctx->nch == 0) {
    // columns beyond the line solver: a column-by-column solve
    MR_LAUNCH(mr::launch_sweep_seed(ctx, n, lam, mu_out, as_stream(stream)));
    return MR_OK;
  }
  MR_LAUNCH(mr::launch_seed(ctx, n, lam, mu_out, as_stream(stream)));
  return MR_OK;
}

int mr_scalar_step_backward(mr_ctx* ctx, int64_t n, const void* mu_next, const void* mu_cur,
                            const void* lam_add, void* out, const void* u, const void* v,
                            const void* w, void* stream) {
  MR_CALL_RANGE();
  if (!ctx || n < 0 || !mu_cur || !out || !u || !v || !w) return MR_EINVAL;
  if (out == mu_cur || (mu_next && out == mu_next) || (lam_add && out == lam_add)) return MR_EINVAL;
  if (ctx->stream_d && !lam_add) {
    MR_LAUNCH(mr::launch_stream_step_backward(ctx, n, mu_next, mu_cur, out, u, v, w, as_stream(stream)));
    return MR_OK;
  }
  if (ctx->nch == 0) {
    // columns beyond the line solver: the reverse step as a column sweep
    // and its back substitution (no lam_add there)
    if (lam_add) return MR_ESHAPE;
    hipStream_t s = as_stream(stream);
    if (n == 0) {
      MR_LAUNCH(mr::launch_sweep_bwd0(ctx, mu_next, mu_cur, out, u, v, w, s));
    } else {
      void* outs[1] = {out};
      MR_LAUNCH(mr::launch_sweep_bwd_steps(ctx, n, 1, mu_next, mu_cur, outs, u, v, w, s));
    }
    return MR_OK;
  }
  MR_LAUNCH(mr::launch_step_backward(ctx, n, mu_next, mu_cur, lam_add, out, u, v, w,
                                     as_stream(stream)));
  return MR_OK;
}

int mr_scalar_steps_backward(mr_ctx* ctx, int64_t n0, int32_t count, const void* mu_next, const void* mu_cur,
                             void* const* outs, const void* u, const void* v, const void* w, void* stream) {
  MR_CALL_RANGE();
  if (!ctx || count < 1 || n0 - count + 1 < 1 || !mu_cur || !outs || !u || !v || !w) return MR_EINVAL;
  // every output differs from the two levels before it
  for (int32_t q = 0; q < count; ++q) {
    const void* l1 = q >= 1 ? outs[q - 1] : mu_cur;
    const void* l2 = q >= 2 ? outs[q - 2] : (q == 1 ? mu_cur : mu_next);
    if (!outs[q] || outs[q] == l1 || outs[q] == l2) return MR_EINVAL;
  }
  hipStream_t s = as_stream(stream);
  const bool flat = flat_sweeps(ctx, s);
  if (ctx->stream_d && !flat) {
    for (int32_t q = 0; q < count; ++q) {
      const void* nxt = q >= 2 ? outs[q - 2] : (q == 1 ? mu_cur : mu_next);
      const void* cur = q >= 1 ? outs[q - 1] : mu_cur;
      MR_LAUNCH(mr::launch_stream_step_backward(ctx, n0 - q, nxt, cur, outs[q], u, v, w, s));
    }
    return MR_OK;
  }
  if (ctx->sweep_pref) {
    MR_LAUNCH(mr::launch_sweep_bwd_steps(ctx, n0, count, mu_next, mu_cur, outs, u, v, w, s));
    return MR_OK;
  }
  if (ctx->nch == 0) return MR_ESHAPE;
  for (int32_t q = 0; q < count; ++q) {
    const void* nxt = q >= 2 ? outs[q - 2] : (q == 1 ? mu_cur : mu_next);
    const void* cur = q >= 1 ? outs[q - 1] : mu_cur;
    MR_LAUNCH(mr::launch_step_backward(ctx, n0 - q, nxt, cur, nullptr, outs[q], u, v, w, s));
  }
  return MR_OK;
}

int mr_velocity_grad(mr_ctx* ctx, int32_t count, const int64_t* steps, const void* const* thetas,
                     const void* const* mus, void* gu, void* gv, void* gw, void* stream) {
  MR_CALL_RANGE();
  if (!ctx || count < 1 || count > 16 || !steps || !thetas || !mus || !gu || !gv || !gw)
    return MR_EINVAL;
  for (int s = 0; s < count; ++s)
    if (steps[s] < 0 || !thetas[s] || !mus[s]) return MR_EINVAL;
  MR_LAUNCH(mr::launch_velocity_grad(ctx, count, steps, thetas, mus, gu, gv, gw, as_stream(stream)));
  return MR_OK;
}

int mr_nusselt(mr_ctx* ctx, const void* theta, const void* w, double* dev_profile, mr_nu* host_out,
               void* stream) {
  MR_CALL_RANGE();
  if (!ctx || !theta || !w || !dev_profile) return MR_EINVAL;
  hipStream_t s = as_stream(stream);
  MR_LAUNCH(mr::launch_nusselt(ctx, theta, w, dev_profile, s));
  if (host_out) {
    double tmp[5];
    MR_LAUNCH(hipMemcpyAsync(tmp, dev_profile + ctx->nz + 1, sizeof(tmp), hipMemcpyDeviceToHost, s));
    MR_LAUNCH(hipStreamSynchronize(s));
    host_out->nu_bot = tmp[0];
    host_out->nu_top = tmp[1];
    host_out->nu_vol = tmp[2];
    host_out->nu_paper = tmp[3];
    host_out->mean_theta = tmp[4];
    for (double t : tmp)
      if (!std::isfinite(t)) return MR_ENONFINITE;
  }
  return MR_OK;
}

int mr_nusselt_noalloc(mr_ctx* ctx, const void* theta, const void* w, double* dev_profile,
                       void* stream) {
  MR_CALL_RANGE();
  if (!ctx || !theta || !w || !dev_profile) return MR_EINVAL;
  return mr::nusselt_fixed(ctx, theta, w, dev_profile, as_stream(stream));
}

int mr_thermal_dissipation(mr_ctx* ctx, const void* theta, double* dev_out, double* host_out,
                           void* stream) {
  MR_CALL_RANGE();
  if (!ctx || !theta || !dev_out) return MR_EINVAL;
  hipStream_t s = as_stream(stream);
  MR_LAUNCH(mr::launch_dissipation(ctx, theta, dev_out, s));
  if (host_out) {
    MR_LAUNCH(hipMemcpyAsync(host_out, dev_out, 4 * sizeof(double), hipMemcpyDeviceToHost, s));
    MR_LAUNCH(hipStreamSynchronize(s));
    for (int q = 0; q < 4; ++q)
      if (!std::isfinite(host_out[q])) return MR_ENONFINITE;
  }
  return MR_OK;
}

int mr_interpolate_velocity_time(mr_ctx* ctx, const void* U0, const void* V0, const void* W0,
                                 const void* U1, const void* V1, const void* W1, int64_t i,
                                 int64_t mt, void* u, void* v, void* w, void* stream) {
  MR_CALL_RANGE();
  if (!ctx || !U0 || !V0 || !W0 || !U1 || !V1 || !W1 || !u || !v || !w) return MR_EINVAL;
  if (mt < 1 || i < 0 || i > mt) return MR_EINVAL;
  MR_LAUNCH(mr::launch_refine_time(ctx, U0, V0, W0, U1, V1, W1, (double)i / (double)mt, u, v, w,
                                   as_stream(stream)));
  return MR_OK;
}

int mr_integrate_scalar(mr_ctx* ctx, const void* theta, void* theta_c, void* stream) {
  MR_CALL_RANGE();
  if (!ctx || !theta || !theta_c || theta == theta_c) return MR_EINVAL;
  MR_LAUNCH(mr::launch_integrate(ctx, theta, theta_c, as_stream(stream)));
  return MR_OK;
}

int mr_coarse_step(mr_ctx* ctx, int64_t n0, int32_t mt, const void* U0, const void* V0,
                   const void* W0, const void* U1, const void* V1, const void* W1, void* u, void* v,
                   void* w, void* const* ring, int32_t* prev, int32_t* cur, void* theta_c,
                   void* stream) {
  MR_CALL_RANGE();
  if (!ctx || n0 < 0 || mt < 1 || !U0 || !V0 || !W0 || !U1 || !V1 || !W1 || !u || !v || !w)
    return MR_EINVAL;
  if (!ring || !prev || !cur) return MR_EINVAL;
  int p = *prev, c = *cur;
  if (c < 0 || c > 2 || (n0 > 0 && (p < 0 || p > 2 || p == c))) return MR_EINVAL;
  if (!ring[0] || !ring[1] || !ring[2] || ring[0] == ring[1] || ring[0] == ring[2] ||
      ring[1] == ring[2])
    return MR_EINVAL;
  if (n0 == 0) p = c;
  hipStream_t s = as_stream(stream);
  if (ctx->sweep_pref && (!ctx->stream_d || flat_sweeps(ctx, s))) {
    // column sweeps: the kernel of sub-step i finishes theta^{n0+i-1} and
    // starts sub-step i on the velocity refined just before it (the velocity
    // at the start of the sub-step, fraction (i-1)/mt)
    const int c0 = c;
    for (int32_t i = 1; i <= mt; ++i) {
      MR_LAUNCH(mr::launch_refine_time(ctx, U0, V0, W0, U1, V1, W1, (double)(i - 1) / (double)mt, u, v, w, s));
      const int q = i - 1;
      int o = 0;
      while (o == c || o == p) ++o;
      // q = 0 reads theta^{n0} itself; q > 0 writes theta^{n0+q} into the free buffer
      MR_LAUNCH(mr::launch_sweep_step(ctx, n0, q, q == 0 ? ring[p] : ring[c], ring[c0],
                                      q == 0 ? nullptr : ring[o], u, v, w, s));
      if (q > 0) {
        p = c;
        c = o;
      }
    }
    int o = 0;
    while (o == c || o == p) ++o;
    MR_LAUNCH(mr::launch_sweep_finish(ctx, n0, mt, ring[o], s));
    p = c;
    c = o;
  } else {
    for (int32_t i = 1; i <= mt; ++i) {
      MR_LAUNCH(mr::launch_refine_time(ctx, U0, V0, W0, U1, V1, W1, (double)(i - 1) / (double)mt, u, v, w, s));
      const int64_t n = n0 + i - 1;
      int o = 0;
      while (o == c || o == p) ++o;   // the buffer holding neither level
      MR_LAUNCH(ctx->stream_d ? mr::launch_stream_step(ctx, n, ctx->sweep_pref ? i - 1 : -1, ring[p], ring[c], ring[o], u,
                                                       v, w, s)
                : ctx->stream_v ? mr::launch_stream_step_var(ctx, n, ring[p], ring[c], ring[o], u, v, w, s)
                                : mr::launch_step(ctx, n, ring[p], ring[c], ring[o], u, v, w, s));
      p = c;
      c = o;
    }
  }
  if (theta_c) MR_LAUNCH(mr::launch_integrate(ctx, ring[c], theta_c, s));
  *prev = p;
  *cur = c;
  return MR_OK;
}

int mr_copy_probe(const void* src, void* dst, int64_t nbytes, void* stream) {
  if (!src || !dst || nbytes < 0 || (nbytes & 15) || ((uintptr_t)src & 15) || ((uintptr_t)dst & 15))
    return MR_EINVAL;
  hipError_t e = mr::launch_copy(src, dst, nbytes, as_stream(stream));
  if (e != hipSuccess) { (void)hipGetLastError(); return MR_EHIP; }
  return MR_OK;
}

}  // extern "C"
