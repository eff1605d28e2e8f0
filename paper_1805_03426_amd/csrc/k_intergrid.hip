// Inter-grid kernels around the dense scalar step: the upscale integration of
// the scalar to the coarse grid (Sec. 3.3, Eq. 20, as the volume-weighted mean
// over the sub-cells) and the dissipation Nusselt number Nu_T = eps_T (Ra Pr)^(1/2)
// with eps_T = kappa <|grad theta|^2>_V (Sec. 4.1, Eq. 23).
//
// Integration: one lane per coarse cell, 256 consecutive ones (x fastest) a
// workgroup.  A lane reads its mx values of each of the my x mz dense rows at
// once (mx <= 4; larger factors: integrate_columns), all of them independent, and
// sums in double: the columns over the rows first, then across x.  The dense
// field is read once.
//
// Dissipation: every dense cell owns its low x face, low y face and low z face
// (and the top plate for the last level); each face adds its squared
// difference quotient times its dual volume.  Two-pass, fixed partition
// (tiles of columns x level ranges) and fixed combining order with double-double
// partial sums, so the result is compensated and bitwise reproducible.
#include <algorithm>

#include "mr_internal.h"

namespace mr {
namespace {

constexpr int kIntBlock = 256;

// MX <= 4, MY, MZ: the refinement factors, MY and MZ 0 for any (then from the arguments).
template <typename T, int MX, int MY, int MZ>
__global__ void __launch_bounds__(kIntBlock) integrate_kernel(const T* th, T* tc, const double* hx,
                                                              const double* hy, const double* hz,
                                                              int nx, int ny, int my_, int mz_,
                                                              int ncx, int ncy, int cells) {
  const int c = xcd_remap(blockIdx.x, gridDim.x) * kIntBlock + threadIdx.x;
  if (c >= cells) return;
  const int my = MY ? MY : my_, mz = MZ ? MZ : mz_;
  const int KJ = c / ncx, I = c - KJ * ncx, K = KJ / ncy, J = KJ - K * ncy;
  const size_t nxy = (size_t)nx * ny;
  double acc[MX], vyz = 0.0;
#pragma unroll
  for (int q = 0; q < MX; ++q) acc[q] = 0.0;
  for (int kk = 0; kk < mz; ++kk) {
    for (int jj = 0; jj < my; ++jj) {
      T v[MX];
      load_vec<T, MX>(th + (size_t)(K * mz + kk) * nxy + (size_t)(J * my + jj) * nx + I * MX, v);
      const double wyz = hy[J * my + jj] * hz[K * mz + kk];
#pragma unroll
      for (int q = 0; q < MX; ++q) acc[q] += (double)v[q] * wyz;
      vyz += wyz;
    }
  }
  double num = 0.0, hxs = 0.0;
#pragma unroll
  for (int q = 0; q < MX; ++q) {
    const double w = hx[I * MX + q];
    num += acc[q] * w;
    hxs += w;
  }
  tc[c] = (T)(num / (hxs * vyz));
}

// M_x = 1 with several dense rows a coarse cell, on rows of coarse cells that
// fill wavefronts: as above, but a wavefront stays in one coarse row, so that the
// y and z widths are scalar loads (as vector loads they are as many again as the
// field's).  FP64, 512 x 512 x 128, M = 1, 2, 2: 69 us, 80 without it; 256^3 26.5
// and 29.2.
template <typename T>
__global__ void __launch_bounds__(kIntBlock) integrate_rows(const T* th, T* tc, const double* hx, const double* hy,
                                                            const double* hz, int nx, int ny, int my, int mz, int ncy,
                                                            int ntx, int tiles) {
  const int tile = blockIdx.x * (kIntBlock / kWave) + __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int row = tile / ntx, K = row / ncy, J = row - K * ncy;
  const int I = (tile - row * ntx) * kWave + threadIdx.x % kWave;
  if (tile >= tiles || I >= nx) return;
  const size_t nxy = (size_t)nx * ny;
  const T* const p = th + (size_t)K * mz * nxy + (size_t)J * my * nx + I;
  const double *const py = hy + J * my, *const pz = hz + K * mz;
  double acc = 0.0, vyz = 0.0;
  for (int kk = 0; kk < mz; ++kk)
    for (int jj = 0; jj < my; ++jj) {
      const double wyz = py[jj] * pz[kk];
      acc += (double)p[(size_t)kk * nxy + (size_t)jj * nx] * wyz;
      vyz += wyz;
    }
  const double w = hx[I];
  tc[(size_t)row * nx + I] = (T)(acc * w / (w * vyz));
}

// M_x from 5 to kIntBlock: a lane per dense column of a coarse cell,
// floor(kIntBlock / mx) consecutive coarse cells (x fastest) a workgroup.  A lane
// sums its column over the cell's dense rows, so that the lanes read rows of the
// field side by side (a lane per coarse cell reads every line mx times: 256^3
// FP64, M = 16, 2, 2 317 us, here 29; M = 5, 2, 2 89 and 28); the cell's first
// lane adds the columns up in order.  U: dense rows whose loads go out together
// (4 from M_y = 4 on: M = 8, 8, 8 22 us, 30 with 1; M = 5, 2, 2 30 with 4).
template <typename T, int U>
__global__ void __launch_bounds__(kIntBlock) integrate_columns(const T* th, T* tc, const double* hx,
                                                               const double* hy, const double* hz, int nx, int ny,
                                                               int mx, int my, int mz, int ncx, int ncy, int cells) {
  __shared__ double s_acc[kIntBlock];
  __shared__ double s_hx[kIntBlock];
  const int t = threadIdx.x, cell = t / mx, sub = t - cell * mx, per = kIntBlock / mx;
  const int c = xcd_remap(blockIdx.x, gridDim.x) * per + cell;
  const bool on = cell < per && c < cells;
  double acc = 0.0, vyz = 0.0, wx = 0.0;
  if (on) {
    const int KJ = c / ncx, I = c - KJ * ncx, K = KJ / ncy, J = KJ - K * ncy;
    const T* p = th + ((size_t)K * mz * ny + (size_t)J * my) * nx + I * mx + sub;
    const size_t nxy = (size_t)nx * ny;
    wx = hx[I * mx + sub];
    for (int kk = 0; kk < mz; ++kk)
#pragma unroll U
      for (int jj = 0; jj < my; ++jj) {
        const double wyz = hy[J * my + jj] * hz[K * mz + kk];
        acc += (double)p[kk * nxy + (size_t)jj * nx] * wyz;
        vyz += wyz;
      }
  }
  s_acc[t] = acc * wx;
  s_hx[t] = wx;
  __syncthreads();
  if (on && sub == 0) {
    double num = 0.0, hxs = 0.0;
    for (int q = 0; q < mx; ++q) {
      num += s_acc[t + q];
      hxs += s_hx[t + q];
    }
    tc[c] = (T)(num / (hxs * vyz));
  }
}

template <typename T>
hipError_t launch_integrate_t(mr_ctx* c, const T* th, T* tc, hipStream_t s) {
  const int cells = c->ncx * c->ncy * c->ncz;
  const dim3 block(kIntBlock);
  if (c->mx > 4) {
    const int per = kIntBlock / c->mx;
    if (per < 1) return hipErrorInvalidValue;
    auto k = c->my >= 4 ? integrate_columns<T, 4> : integrate_columns<T, 1>;
    hipLaunchKernelGGL(k, dim3((unsigned)((cells + per - 1) / per)), block, 0, s, th, tc, c->hx64, c->areaw, c->hz64,
                       c->nx, c->ny, c->mx, c->my, c->mz, c->ncx, c->ncy, cells);
    return hipGetLastError();
  }
  const int ntx = (c->ncx + kWave - 1) / kWave;
  if (c->mx == 1 && c->my * c->mz > 1 && 5 * c->ncx >= 4 * ntx * kWave) {   // (at least 4/5 of the lanes in use)
    const int tiles = ntx * c->ncy * c->ncz, waves = kIntBlock / kWave;
    hipLaunchKernelGGL(integrate_rows<T>, dim3((unsigned)((tiles + waves - 1) / waves)), block, 0, s, th, tc, c->hx64,
                       c->areaw, c->hz64, c->nx, c->ny, c->my, c->mz, c->ncy, ntx, tiles);
    return hipGetLastError();
  }
  const dim3 grid((unsigned)((cells + kIntBlock - 1) / kIntBlock));
  // the equal factors 2 and 3 unrolled whole (their loads go out together)
  auto k = integrate_kernel<T, 1, 0, 0>;
  if (c->mx == 2 && c->my == 2 && c->mz == 2) k = integrate_kernel<T, 2, 2, 2>;
  else if (c->mx == 3 && c->my == 3 && c->mz == 3) k = integrate_kernel<T, 3, 3, 3>;
  else if (c->mx == 2) k = integrate_kernel<T, 2, 0, 0>;
  else if (c->mx == 3) k = integrate_kernel<T, 3, 0, 0>;
  else if (c->mx == 4) k = integrate_kernel<T, 4, 0, 0>;
  hipLaunchKernelGGL(k, grid, block, 0, s, th, tc, c->hx64, c->areaw, c->hz64, c->nx, c->ny, c->my, c->mz, c->ncx,
                     c->ncy, cells);
  return hipGetLastError();
}

// Nu_T partials: a workgroup of kDissRows wavefronts covers kDissRows rows of
// 64 V columns and a range of kb levels; a lane walks up V consecutive columns
// carrying theta(k-1), reads its own values, the one to their left and the row
// below (both mostly from the cache) and accumulates the faces on the low side
// of its cells (plus the top plate for the last level).  At a ragged row end the
// last lanes move back to the row's last V cells; those counted by the lane
// before weigh nothing.  kDissAhead levels are loaded together; each column's
// faces of those levels are summed in double (a term is a difference, its square
// and a product with the width, each rounded once, then kDissAhead - 1 positive
// sums and the column's weight: relative error at most kDissAhead + 5 eps) and
// enter the double-double sums column by column.  Fixed partition: part[b] holds
// the three double-double sums of the workgroup of logical index b; consecutive
// tiles run on one XCD.
constexpr int kDissMaxParts = 2048;
constexpr int kDissAhead = 4;
constexpr int kDissRows = 4;
constexpr int kDissWaves = 8192;   // wavefronts to aim for (32 per CU)

__device__ __forceinline__ double ztab(const double* p, int k) {
  return ((const __attribute__((address_space(4))) double*)(p))[k];
}

template <typename T, int V>
__global__ void __launch_bounds__(64 * kDissRows) diss_partial(const T* th, const double* hx, const double* hy,
                                                               const double* hz, const double* idxc,
                                                               const double* idyc, const double* idcz, int nx,
                                                               int ny, int nz, int nbx, int nby, int kb, int walx,
                                                               int waly, int dir_bot, int dir_top, double t_bot,
                                                               double t_top, double* part) {
  __shared__ DD sh[3][kDissRows];
  const int b = xcd_remap(blockIdx.x, gridDim.x);
  const int bx = b % nbx, by = (b / nbx) % nby, kc = b / (nbx * nby);
  const int lane = threadIdx.x, r = __builtin_amdgcn_readfirstlane(threadIdx.y);
  const int i_raw = (bx * kWave + lane) * V, j_raw = by * kDissRows + r;
  const int i = min(i_raw, nx - V), j = min(j_raw, ny - 1);
  // across a side wall the neighbour is the cell itself: the wall face adds nothing
  const int im = i == 0 ? (walx ? 0 : nx - 1) : i - 1;
  const int jm = j == 0 ? (waly ? 0 : ny - 1) : j - 1;
  const size_t nxy = (size_t)nx * ny;
  const int k0 = kc * kb, k1 = min(nz, k0 + kb);
  const T* cc = th + (size_t)j * nx + i;
  const T* cx = th + (size_t)j * nx + im;
  const T* ch = th + (size_t)jm * nx + i;
  double wx[V], wy[V], area[V];
#pragma unroll
  for (int q = 0; q < V; ++q) {
    const bool on = j_raw < ny && i + q >= i_raw;
    wx[q] = on ? idxc[i + q] * hy[j] : 0.0;
    wy[q] = on ? idyc[j] * hx[i + q] : 0.0;
    area[q] = on ? hx[i + q] * hy[j] : 0.0;
  }
  DD sx{0.0, 0.0}, sy{0.0, 0.0}, sz{0.0, 0.0};
  double below[V];
  {
    T t[V];
    load_vec<T, V>(cc + (size_t)max(k0 - 1, 0) * nxy, t);
#pragma unroll
    for (int q = 0; q < V; ++q) below[q] = t[q];
  }
  for (int kk = k0; kk < k1; kk += kDissAhead) {
    T c[kDissAhead][V], h[kDissAhead][V], x[kDissAhead];
#pragma unroll
    for (int l = 0; l < kDissAhead; ++l) {
      const size_t lv = (size_t)min(kk + l, k1 - 1) * nxy;
      load_vec<T, V>(cc + lv, c[l]);
      load_vec<T, V>(ch + lv, h[l]);
      x[l] = cx[lv];
    }
    double ax[V], ay[V], az[V];
#pragma unroll
    for (int q = 0; q < V; ++q) ax[q] = ay[q] = az[q] = 0.0;
#pragma unroll
    for (int l = 0; l < kDissAhead; ++l) {
      const int k = kk + l;
      if (k >= k1) break;
      const double hzk = ztab(hz, k), idz = ztab(idcz, k);
#pragma unroll
      for (int q = 0; q < V; ++q) {
        const double v = c[l][q];
        const double dx = v - (double)(q ? c[l][q ? q - 1 : 0] : x[l]);
        const double dy = v - (double)h[l][q];
        ax[q] += dx * dx * hzk;
        ay[q] += dy * dy * hzk;
        if (k > 0) {
          const double dz = v - below[q];
          az[q] += dz * dz * idz;
        } else if (dir_bot) {
          const double dz = v - t_bot;
          az[q] += dz * dz * idz;
        }
        if (k == nz - 1 && dir_top) {
          const double dz = t_top - v;
          az[q] += dz * dz * ztab(idcz, nz);
        }
        below[q] = v;
      }
    }
#pragma unroll
    for (int q = 0; q < V; ++q) {
      sx = dd_add(sx, ax[q] * wx[q]);
      sy = dd_add(sy, ay[q] * wy[q]);
      sz = dd_add(sz, az[q] * area[q]);
    }
  }
  sx = wave_sum(sx);
  sy = wave_sum(sy);
  sz = wave_sum(sz);
  if (lane == 0) {
    sh[0][r] = sx;
    sh[1][r] = sy;
    sh[2][r] = sz;
  }
  __syncthreads();
  if (lane == 0 && r == 0) {
    for (int q = 1; q < kDissRows; ++q) {
      sx = dd_merge(sx, sh[0][q]);
      sy = dd_merge(sy, sh[1][q]);
      sz = dd_merge(sz, sh[2][q]);
    }
    double* o = part + (size_t)b * 6;
    o[0] = sx.s; o[1] = sx.c;
    o[2] = sy.s; o[3] = sy.c;
    o[4] = sz.s; o[5] = sz.c;
  }
}

// One workgroup: strided double-double merge of the partials, the shuffle
// tree in each wavefront, then the four wavefronts in order;
// out = {Nu_T, <theta_x^2>, <theta_y^2>, <theta_z^2>}.
constexpr int kDissFinal = 1024;

__global__ void __launch_bounds__(kDissFinal) diss_final(const double* part, int nb, double vtot,
                                                         double nufac, double* out) {
  __shared__ DD sh[3][kDissFinal / kWave];
  DD sx{0.0, 0.0}, sy{0.0, 0.0}, sz{0.0, 0.0};
  for (int p = threadIdx.x; p < nb; p += kDissFinal) {
    const double* o = part + (size_t)p * 6;
    sx = dd_merge(sx, DD{o[0], o[1]});
    sy = dd_merge(sy, DD{o[2], o[3]});
    sz = dd_merge(sz, DD{o[4], o[5]});
  }
  sx = wave_sum(sx);
  sy = wave_sum(sy);
  sz = wave_sum(sz);
  const int wv = threadIdx.x / kWave, lane = threadIdx.x % kWave;
  if (lane == 0) {
    sh[0][wv] = sx;
    sh[1][wv] = sy;
    sh[2][wv] = sz;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int q = 1; q < kDissFinal / kWave; ++q) {
      sx = dd_merge(sx, sh[0][q]);
      sy = dd_merge(sy, sh[1][q]);
      sz = dd_merge(sz, sh[2][q]);
    }
    const double gx = (sx.s + sx.c) / vtot, gy = (sy.s + sy.c) / vtot, gz = (sz.s + sz.c) / vtot;
    out[0] = nufac * (gx + gy + gz);
    out[1] = gx;
    out[2] = gy;
    out[3] = gz;
  }
}

}  // namespace

hipError_t launch_integrate(mr_ctx* c, const void* th, void* tc, hipStream_t s) {
  return c->precision == MR_FP64 ? launch_integrate_t<double>(c, (const double*)th, (double*)tc, s)
                                 : launch_integrate_t<float>(c, (const float*)th, (float*)tc, s);
}

namespace {

struct DissGrid {
  int V, nbx, nby, kb;
  int64_t nb;
};
DissGrid diss_grid(const mr_ctx* c) {
  DissGrid g;
  // cells a lane: two in FP64; one in FP32, four on large grids whose rows fill the
  // wider tiles; one on rows of one cell.  In us, 8e6 cells: FP32 with one, two and four
  // 450 x 177 x 100 22.5, 23.3, 25.4; 256 x 312 x 100 22.0, 21.3, 22.6; 40 x 2000 x 100
  // 25.6, 35.1, 55.4 (four leave most lanes of a short row idle); 8 x 10000 x 100 72, 108,
  // 205; FP64 with one and two 450 x 177 x 100 26.2, 25.1; 256 x 312 x 100 26.1, 23.5; 40 x
  // 2000 x 100 31.5, 36.3.  FP32, one and four, 2e7 cells and more: 1000 x 100 x 200 33.0,
  // 34.6; 450 x 300 x 200 47.9, 42.5; 1024 x 1024 x 64 76.7, 69.2; 640 x 640 x 256 (rows
  // of 2 1/2 tiles) 127, 130
  const int wide = (c->nx + 4 * kWave - 1) / (4 * kWave) * 4 * kWave;
  const bool four = (int64_t)c->nx * c->ny * c->nz >= 25000000 && 8 * (int64_t)c->nx >= 7 * (int64_t)wide;
  g.V = c->precision != MR_FP64 ? (four ? 4 : 1) : c->nx >= 2 ? 2 : 1;
  g.nbx = (c->nx + kWave * g.V - 1) / (kWave * g.V);
  g.nby = (c->ny + kDissRows - 1) / kDissRows;
  const int64_t tiles = (int64_t)g.nbx * g.nby;
  // level ranges: about kDissWaves wavefronts in all (ranges as long as that
  // allows: each workgroup ends with a reduction), at most kDissMaxParts partials
  const int64_t want = (kDissWaves / kDissRows + tiles - 1) / tiles;
  const int nkb = (int)std::max<int64_t>(1, std::min<int64_t>({(int64_t)c->nz, want, kDissMaxParts / tiles}));
  g.kb = (c->nz + nkb - 1) / nkb;
  g.nb = tiles * ((c->nz + g.kb - 1) / g.kb);
  return g;
}

}  // namespace

size_t diss_bytes(const mr_ctx* c) { return sizeof(double) * 6 * (size_t)diss_grid(c).nb; }

hipError_t launch_dissipation(mr_ctx* c, const void* th, double* out, hipStream_t s) {
  const bool f64 = c->precision == MR_FP64;
  const DissGrid d = diss_grid(c);
  if (d.nb > INT32_MAX) return hipErrorInvalidValue;
  const int nbx = d.nbx, nby = d.nby, kb = d.kb;
  const int64_t nb = d.nb;
  const hipError_t e = ensure_red(c);
  if (e != hipSuccess) return e;
  const int db = c->bc_bot == MR_DIRICHLET, dtp = c->bc_top == MR_DIRICHLET;
  const Geom<double>& g = c->g64;
  const dim3 block(kWave, kDissRows);
  if (f64) {
    auto k = d.V == 2 ? diss_partial<double, 2> : diss_partial<double, 1>;
    hipLaunchKernelGGL(k, dim3((unsigned)nb), block, 0, s, (const double*)th, c->hx64, c->areaw, c->hz64, g.idxc,
                       g.idyc, c->idcz, c->nx, c->ny, c->nz, nbx, nby, kb, c->wx, c->wy, db, dtp, c->t_bot, c->t_top,
                       c->red);
  } else {
    auto k = d.V == 4 ? diss_partial<float, 4> : diss_partial<float, 1>;
    hipLaunchKernelGGL(k, dim3((unsigned)nb), block, 0, s, (const float*)th, c->hx64, c->areaw, c->hz64, g.idxc,
                       g.idyc, c->idcz, c->nx, c->ny, c->nz, nbx, nby, kb, c->wx, c->wy, db, dtp, c->t_bot, c->t_top,
                       c->red);
  }
  hipLaunchKernelGGL(diss_final, dim3(1), dim3(kDissFinal), 0, s, (const double*)c->red, (int)nb, c->vtot,
                     c->kappa * sqrt(c->ra * c->pr), out);
  return hipGetLastError();
}

}  // namespace mr
