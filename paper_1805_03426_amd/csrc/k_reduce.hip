// Reductions: the discrete divergence check of the refined velocity
// (Sec. 3.2), the heat-flux Nusselt profile and mean scalar (Eq. 22), and a
// plain streaming copy used as the bandwidth reference.
//
// Every reduction is two-pass with a fixed partition and a fixed combining
// order (wavefront shuffles, then LDS, then a single final block), so results
// are bitwise reproducible.  Nusselt sums are double-double (error-free
// two-sum), i.e. compensated.
#include <algorithm>
#include <mutex>

#include "mr_internal.h"

namespace mr {

// Fixed device memory for the Nusselt partials of the allocation-free entry
// point: nz faces x at most kNuMaxParts horizontal parts x 4 doubles, for nz up
// to kNuMaxFaces (2.1 MB per GPU, held until the process ends).
// In host code the array's name is only a stand-in: its device address comes
// from hipGetSymbolAddress, once per device, with that device current.
constexpr int kNuMaxParts = 64;
constexpr size_t kNuScratchDoubles = (size_t)1024 * kNuMaxParts * 4;
static __device__ __align__(256) double scratch[kNuScratchDoubles];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
double* g_scratch[kMaxDevices] = {};
}  // namespace

hipError_t scratch_init(int device) {
  if (device < 0 || device >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (g_scratch[device]) return hipSuccess;
  int cur = -1;
  hipError_t e = hipGetDevice(&cur);
  if (e != hipSuccess) return e;
  if (cur != device) return hipErrorInvalidDevice;
  void* ptr = nullptr;
  e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
  if (e != hipSuccess) return e;
  g_scratch[device] = (double*)ptr;
  return hipSuccess;
}

namespace {

__device__ __forceinline__ double shfl_down_d(double v, int off) {
  return __shfl_down(v, off, kWave);
}

// ------------------------------------------------------------- divergence
// A workgroup of kDivRows wavefronts covers kDivRows rows of 64 V columns and
// walks up a range of levels; a lane owns V consecutive cells of a row (16-byte
// loads that need the element's alignment only) and carries w of the face
// below, so u and w are read once and v twice, the second time mostly from the
// cache.  At a ragged row end the last lanes move back to the row's last V
// cells: cells counted twice do not change a maximum.  The largest relative
// divergence is kept as a fraction (|div|, sum |flux|) compared by
// cross-multiplication, so that a cell costs no division.
// Bound by the bytes of u, v and w.  Timed: see launch_divergence.
constexpr int kDivRows = 4;
constexpr int kDivWaves = 8192;   // wavefronts to aim for (32 a CU)

__device__ __forceinline__ double rtab(const double* p, int k) {
  return ((const __attribute__((address_space(4))) double*)(p))[k];
}

template <typename T, int V>
__global__ void __launch_bounds__(64 * kDivRows) div_kernel(const T* u, const T* v, const T* w, const double* hx,
                                                            const double* hy, const double* hz, int nx, int ny,
                                                            int nz, int nbx, int nby, int kb, int wx, int wy,
                                                            double* part) {
  __shared__ double sh[2][kDivRows];
  const int b = xcd_remap(blockIdx.x, gridDim.x);
  const int bx = b % nbx, by = (b / nbx) % nby, kc = b / (nbx * nby);
  const size_t nxy = (size_t)nx * ny;
  const int i0 = min((bx * kWave + (int)threadIdx.x) * V, nx - V);
  const int j = min(by * kDivRows + __builtin_amdgcn_readfirstlane(threadIdx.y), ny - 1);
  const int jp = j == ny - 1 ? 0 : j + 1, in = i0 + V == nx ? 0 : i0 + V;
  const bool vl0 = wy && j == 0, vr0 = wy && j == ny - 1;
  const bool ul0 = wx && i0 == 0, ur0 = wx && i0 + V == nx;   // the low wall face (stored) and the high one carry nothing
  const double hyj = rtab(hy, j);
  double hxi[V];
#pragma unroll
  for (int q = 0; q < V; ++q) hxi[q] = hx[i0 + q];
  const int k0 = kc * kb, k1 = min(nz, k0 + kb);
  const size_t cc = (size_t)j * nx + i0, cp = (size_t)jp * nx + i0, cn = (size_t)j * nx + in;
  T wl[V];
  load_vec<T, V>(w + (size_t)k0 * nxy + cc, wl);
  double mabs = 0.0, rnum = 0.0, rden = 1.0;   // largest |div| and largest |div| / sum |flux|
#pragma unroll 2
  for (int k = k0; k < k1; ++k) {
    const size_t base = (size_t)k * nxy;
    T uu[V + 1], vl_[V], vr_[V], wr[V];
    load_vec<T, V>(u + base + cc, uu);
    uu[V] = u[base + cn];
    load_vec<T, V>(v + base + cc, vl_);
    load_vec<T, V>(v + base + cp, vr_);
    load_vec<T, V>(w + base + nxy + cc, wr);
    const double hzk = rtab(hz, k), ax = hyj * hzk;
#pragma unroll
    for (int q = 0; q < V; ++q) {
      const double ay = hxi[q] * hzk, az = hxi[q] * hyj;
      const double ul = q == 0 && ul0 ? 0.0 : (double)uu[q];
      const double ur = q == V - 1 && ur0 ? 0.0 : (double)uu[q + 1];
      const double vl = vl0 ? 0.0 : (double)vl_[q];
      const double vr = vr0 ? 0.0 : (double)vr_[q];
      const double wlq = wl[q], wrq = wr[q];
      const double dv = fabs((ur - ul) * ax + (vr - vl) * ay + (wrq - wlq) * az);
      const double tot = (fabs(ul) + fabs(ur)) * ax + (fabs(vl) + fabs(vr)) * ay + (fabs(wlq) + fabs(wrq)) * az;
      mabs = fmax(mabs, dv);
      if (tot > 0.0 && dv * rden > rnum * tot) {
        rnum = dv;
        rden = tot;
      }
      wl[q] = wr[q];
    }
  }
  double mrel = rnum / rden;
  for (int off = kWave / 2; off > 0; off >>= 1) {
    mabs = fmax(mabs, shfl_down_d(mabs, off));
    mrel = fmax(mrel, shfl_down_d(mrel, off));
  }
  const int wv = threadIdx.y;
  if (threadIdx.x == 0) {
    sh[0][wv] = mabs;
    sh[1][wv] = mrel;
  }
  __syncthreads();
  if (threadIdx.x == 0 && wv == 0) {
    for (int q = 1; q < kDivRows; ++q) {
      mabs = fmax(mabs, sh[0][q]);
      mrel = fmax(mrel, sh[1][q]);
    }
    part[2 * b] = mabs;
    part[2 * b + 1] = mrel;
  }
}

constexpr int kMaxFinal = 1024;

__global__ void __launch_bounds__(kMaxFinal) max_final(const double* part, int n, double* out) {
  __shared__ double sh[2][kMaxFinal / kWave];
  double a = 0.0, b = 0.0;
  for (int q = threadIdx.x; q < n; q += kMaxFinal) {
    a = fmax(a, part[2 * q]);
    b = fmax(b, part[2 * q + 1]);
  }
  for (int off = kWave / 2; off > 0; off >>= 1) {
    a = fmax(a, shfl_down_d(a, off));
    b = fmax(b, shfl_down_d(b, off));
  }
  if (threadIdx.x % kWave == 0) {
    sh[0][threadIdx.x / kWave] = a;
    sh[1][threadIdx.x / kWave] = b;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int q = 1; q < kMaxFinal / kWave; ++q) {
      a = fmax(a, sh[0][q]);
      b = fmax(b, sh[1][q]);
    }
    out[0] = a;
    out[1] = b;
  }
}

// ---------------------------------------------------------------- Nusselt
// partials[(k*P + p)*4 + {conv s,c, mean s,c}]: the convective flux sum of face
// k and the scalar sum of level k (gradients are differences of level sums, so
// both keep the rounding errors of their products too).  Block (p, q) covers
// the horizontal range p of faces and levels kNuFaces*q .. kNuFaces*(q + 1) - 1,
// V consecutive cells of the level a lane (16-byte loads that need the
// element's alignment only; the row index is one division per V cells, and
// cells past the range's end weigh nothing).  Each lane walks the group's faces
// for its cells carrying theta of the level below, so a level is read once per
// group of faces instead of once per face.
constexpr int kNuFaces = 2;   // timed: 2 faces per group beat 1, 3, 4, 8 and 16

// a + b * c with the product's rounding error kept (no contraction: a product
// fused into the sums would count its error twice).
__device__ __forceinline__ DD dd_fma(DD a, double b, double c) {
#pragma clang fp contract(off)
  const double p = b * c;
  const double t = a.s + p;
  const double bp = t - a.s;
  const double e = (a.s - (t - bp)) + (p - bp);
  return {t, a.c + (e + __builtin_fma(b, c, -p))};
}

template <typename T, int V>
__global__ void __launch_bounds__(256) nu_partial(const T* th, const T* w, const double* hx,
                                                  const double* hy, int nx, int ny, int nz, int P, double* part) {
  __shared__ DD sh[2][256 / kWave];
  const int kf0 = blockIdx.y * kNuFaces;   // first face of the group
  const int p = blockIdx.x;
  const int nxy = nx * ny;
  const int per = ((nxy + P - 1) / P + V - 1) / V * V;
  const int lo = min(nxy, p * per), hi = min(nxy, lo + per);
  DD conv[kNuFaces], mean[kNuFaces];
#pragma unroll
  for (int f = 0; f < kNuFaces; ++f) conv[f] = mean[f] = DD{0.0, 0.0};
  for (int r0 = lo + threadIdx.x * V; r0 < hi; r0 += blockDim.x * V) {
    // the level's last lane moves back to its last V cells; those that belong
    // to the lane before weigh nothing
    const int e0 = min(r0, nxy - V);
    // the level below the group (for face 0 level 0: that face carries no flux), the group's levels, w on its faces
    T t[kNuFaces + 1][V], wt[kNuFaces][V];
    load_vec<T, V>(th + (size_t)max(kf0 - 1, 0) * nxy + e0, t[0]);
#pragma unroll
    for (int f = 0; f < kNuFaces; ++f) {
      const size_t lv = (size_t)min(kf0 + f, nz - 1) * nxy;
      load_vec<T, V>(th + lv + e0, t[f + 1]);
      load_vec<T, V>(w + lv + e0, wt[f]);
    }
    const int j = e0 / nx, i0 = e0 - j * nx;
    double area[V];
    if (i0 + V <= nx) {
      const double hyj = hy[j];
      double hxi[V];
      load_vec<double, V>(hx + i0, hxi);
#pragma unroll
      for (int q = 0; q < V; ++q) area[q] = hxi[q] * hyj;
    } else {   // across the end of a row (V <= nx)
#pragma unroll
      for (int q = 0; q < V; ++q) area[q] = i0 + q < nx ? hx[i0 + q] * hy[j] : hx[i0 + q - nx] * hy[j + 1];
    }
#pragma unroll
    for (int q = 0; q < V; ++q) {
      if (e0 + q < r0) area[q] = 0.0;
#pragma unroll
      for (int f = 0; f < kNuFaces; ++f) {
        mean[f] = dd_fma(mean[f], (double)t[f + 1][q], area[q]);
        const double mid = 0.5 * ((double)t[f][q] + (double)t[f + 1][q]);
        conv[f] = dd_add(conv[f], (double)wt[f][q] * mid * area[q]);
      }
    }
  }
  const int wv = threadIdx.x / kWave, lane = threadIdx.x % kWave;
#pragma unroll
  for (int f = 0; f < kNuFaces; ++f) {
    const int k = kf0 + f;
    if (k >= nz) break;
    DD c = wave_sum(conv[f]), m = wave_sum(mean[f]);
    __syncthreads();   // the previous face's merge has read sh
    if (lane == 0) {
      sh[0][wv] = c;
      sh[1][wv] = m;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
      for (int q = 1; q < (int)blockDim.x / kWave; ++q) {
        c = dd_merge(c, sh[0][q]);
        m = dd_merge(m, sh[1][q]);
      }
      double* o = part + ((size_t)k * P + p) * 4;
      o[0] = c.s; o[1] = c.c;
      o[2] = m.s; o[3] = m.c;
    }
  }
}

// One workgroup: Nu_k of every face from the partials, LANES lanes a face (each
// merges every LANES-th partial, then a shuffle tree), then the summary sums as a
// fixed tree (per-thread strided double-double sums, wave shuffles, then the
// wavefronts in order).  Per-face values stay in LDS.  Up to 1024 threads, four
// lanes a face: with one thread a face (256 in all) it took 16-17 us for 200 to 256
// levels, waiting on 33 to 64 partials one after the other.  With less than four
// partials a face, one lane and up to 256 threads: the Nusselt profile of 32 x 32 x
// 300 15.3 us with 1024, 11.0 with 256.
constexpr int kNuMaxFaces = 1024;
constexpr int kNuFinal = 1024;
constexpr int kNuLanes = 4;

template <int LANES>
__global__ void __launch_bounds__(LANES * (kNuFinal / kNuLanes)) nu_final(const double* part, int P, int nz,
                                                     const double* dcz, const double* hz, double atot,
                                                     double atot_lo, double sq, int dir_bot, int dir_top, double t_bot,
                                                     double t_top, double* prof) {
  __shared__ double s_nu[kNuMaxFaces + 1];   // the convective flux sums, then Nu_k
  __shared__ DD s_mean[kNuMaxFaces];
  __shared__ DD scratch[4][LANES * (kNuFinal / kNuLanes) / kWave];
  __shared__ double total[4];
  const int sub = threadIdx.x % LANES;
  for (int k0 = 0; k0 < nz; k0 += (int)blockDim.x / LANES) {
    const int k = k0 + (int)threadIdx.x / LANES;
    const int kc = min(k, nz - 1);
    DD conv{0.0, 0.0}, mean{0.0, 0.0};
#pragma unroll 4
    for (int p = sub; p < P; p += LANES) {
      const double* o = part + ((size_t)kc * P + p) * 4;
      conv = dd_merge(conv, DD{o[0], o[1]});
      mean = dd_merge(mean, DD{o[2], o[3]});
    }
#pragma unroll
    for (int off = LANES / 2; off > 0; off >>= 1) {
      conv = dd_merge(conv, DD{__shfl_down(conv.s, off, LANES), __shfl_down(conv.c, off, LANES)});
      mean = dd_merge(mean, DD{__shfl_down(mean.s, off, LANES), __shfl_down(mean.c, off, LANES)});
    }
    if (sub == 0 && k < nz) {
      s_nu[k] = conv.s + conv.c;
      s_mean[k] = mean;
    }
  }
  __syncthreads();
  for (int k = threadIdx.x; k <= nz; k += blockDim.x) {
    // area times the mean difference across face k; a plate's wall value at half a cell
    double cs = 0.0, gs = 0.0;
    if (k > 0 && k < nz) {
      const DD a = s_mean[k], b = s_mean[k - 1];
      const DD g = dd_merge(a, DD{-b.s, -b.c});
      cs = s_nu[k];
      gs = g.s + g.c;
    } else if (k == 0 ? dir_bot : dir_top) {
      const DD a = s_mean[k == 0 ? 0 : nz - 1];
      const DD g = k == 0 ? dd_fma(dd_fma(a, -t_bot, atot), -t_bot, atot_lo)
                          : dd_fma(dd_fma(DD{-a.s, -a.c}, t_top, atot), t_top, atot_lo);
      gs = g.s + g.c;
    }
    const double nu = sq * (cs / atot) - (gs / dcz[k]) / atot;
    prof[k] = nu;
    s_nu[k] = nu;   // (face k's own thread: nobody else reads its sum)
  }
  __syncthreads();
  DD sum[4] = {{0.0, 0.0}, {0.0, 0.0}, {0.0, 0.0}, {0.0, 0.0}};   // vol, paper, mean theta, height
  for (int k = threadIdx.x; k <= nz; k += blockDim.x) {
    sum[0] = dd_add(sum[0], dcz[k] * s_nu[k]);
    if (k > 0 && k < nz) sum[1] = dd_add(sum[1], s_nu[k]);
    if (k < nz) {
      sum[2] = dd_add(sum[2], (s_mean[k].s + s_mean[k].c) * hz[k]);
      sum[3] = dd_add(sum[3], hz[k]);
    }
  }
  const int wv = threadIdx.x / kWave, lane = threadIdx.x % kWave;
  // the four trees side by side
#pragma unroll 1
  for (int off = kWave / 2; off > 0; off >>= 1)
#pragma unroll
    for (int q = 0; q < 4; ++q)
      sum[q] = dd_merge(sum[q], DD{__shfl_down(sum[q].s, off, kWave), __shfl_down(sum[q].c, off, kWave)});
#pragma unroll
  for (int q = 0; q < 4; ++q)
    if (lane == 0) scratch[q][wv] = sum[q];
  __syncthreads();
  if (threadIdx.x < 4) {
    DD t = scratch[threadIdx.x][0];
#pragma unroll 1
    for (int v = 1; v < (int)blockDim.x / kWave; ++v) t = dd_merge(t, scratch[threadIdx.x][v]);
    total[threadIdx.x] = t.s + t.c;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    prof[nz + 1] = s_nu[0];
    prof[nz + 2] = s_nu[nz];
    prof[nz + 3] = total[0];
    prof[nz + 4] = nz > 1 ? total[1] / (nz - 1) : 0.0;
    prof[nz + 5] = total[2] / (atot * total[3]);
  }
}

// ------------------------------------------------------------------- copy
__global__ void __launch_bounds__(256) copy_kernel(const int4* __restrict__ src, int4* __restrict__ dst,
                                                   int64_t n) {
  for (int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; t < n; t += (int64_t)gridDim.x * blockDim.x)
    dst[t] = src[t];
}

// Cells a lane takes: 16 bytes of them, one where a row is shorter than that.
// The number of horizontal parts of the Nusselt partials: about 4096 cells
// each, at most kNuMaxParts.
bool wide_rows(const mr_ctx* c) { return c->nx >= (c->precision == MR_FP64 ? 2 : 4); }

int nu_parts(const mr_ctx* c) {
  const int64_t nxy = (int64_t)c->nx * c->ny;
  int64_t P = (nxy + 256 * 16 - 1) / (256 * 16);
  return (int)std::max<int64_t>(1, std::min<int64_t>(P, kNuMaxParts));
}

// The two Nusselt kernels with the partials in `part`.
void nusselt_kernels(mr_ctx* c, const void* th, const void* w, double* prof, double* part, int P,
                     hipStream_t s) {
  const dim3 grid(P, (c->nz + kNuFaces - 1) / kNuFaces), block(256);
  const bool vec = wide_rows(c);
  if (c->precision == MR_FP64) {
    auto k = vec ? nu_partial<double, 2> : nu_partial<double, 1>;
    hipLaunchKernelGGL(k, grid, block, 0, s, (const double*)th, (const double*)w, c->hx64, c->areaw, c->nx, c->ny,
                       c->nz, P, part);
  } else {
    auto k = vec ? nu_partial<float, 4> : nu_partial<float, 1>;
    hipLaunchKernelGGL(k, grid, block, 0, s, (const float*)th, (const float*)w, c->hx64, c->areaw, c->nx, c->ny,
                       c->nz, P, part);
  }
  const int lanes = P < kNuLanes ? 1 : kNuLanes;
  const int nf = std::min(kNuFinal / kNuLanes * lanes, (c->nz * lanes + kWave - 1) / kWave * kWave);
  auto fin = lanes == 1 ? nu_final<1> : nu_final<kNuLanes>;
  hipLaunchKernelGGL(fin, dim3(1), dim3(nf), 0, s, (const double*)part, P, c->nz, c->dcz, c->hz64, c->atot,
                     c->atot_lo, sqrt(c->ra * c->pr), c->bc_bot == MR_DIRICHLET, c->bc_top == MR_DIRICHLET, c->t_bot, c->t_top,
                     prof);
}

}  // namespace

namespace {

// The divergence's launch: level ranges for about kDivWaves wavefronts in all, 8 levels at least.
struct DivGrid {
  int V, nbx, nby, kb;
  int64_t nb;
};
DivGrid div_grid(const mr_ctx* c) {
  DivGrid g;
  g.V = wide_rows(c) ? (c->precision == MR_FP64 ? 2 : 4) : 1;
  g.nbx = (c->nx + kWave * g.V - 1) / (kWave * g.V);
  g.nby = (c->ny + kDivRows - 1) / kDivRows;
  const int64_t tiles = (int64_t)g.nbx * g.nby;
  const int nkb = (int)std::max<int64_t>(1, std::min<int64_t>((kDivWaves / kDivRows + tiles - 1) / tiles, c->nz / 8));
  g.kb = (c->nz + nkb - 1) / nkb;
  g.nb = tiles * ((c->nz + g.kb - 1) / g.kb);
  return g;
}

size_t nu_bytes(const mr_ctx* c) {
  return c->nz > kNuMaxFaces ? 0 : sizeof(double) * 4 * (size_t)c->nz * nu_parts(c);
}

}  // namespace

// One buffer for the partials of all three reductions, as large as the largest
// needs: whichever is called first allocates it, and it is neither moved nor
// freed before the context is, so a captured call keeps a valid address whatever
// is called after it.
hipError_t ensure_red(mr_ctx* c) {
  if (c->red) return hipSuccess;
  const size_t bytes = std::max({sizeof(double) * 2 * (size_t)div_grid(c).nb, nu_bytes(c), diss_bytes(c)});
  const hipError_t e = hipMalloc((void**)&c->red, bytes);
  if (e != hipSuccess) c->red = nullptr;
  return e;
}

hipError_t launch_divergence(mr_ctx* c, const void* u, const void* v, const void* w, double* out,
                             hipStream_t s) {
  const bool f64 = c->precision == MR_FP64, vec = wide_rows(c);
  const DivGrid g = div_grid(c);
  if (g.nb > INT32_MAX) return hipErrorInvalidValue;
  const int nbx = g.nbx, nby = g.nby, kb = g.kb;
  const int64_t nb = g.nb;
  const hipError_t e = ensure_red(c);
  if (e != hipSuccess) return e;
  const dim3 grid((unsigned)nb), block(kWave, kDivRows);
  if (f64) {
    auto k = vec ? div_kernel<double, 2> : div_kernel<double, 1>;
    hipLaunchKernelGGL(k, grid, block, 0, s, (const double*)u, (const double*)v, (const double*)w, c->hx64, c->areaw,
                       c->hz64, c->nx, c->ny, c->nz, nbx, nby, kb, c->wx, c->wy, c->red);
  } else {
    auto k = vec ? div_kernel<float, 4> : div_kernel<float, 1>;
    hipLaunchKernelGGL(k, grid, block, 0, s, (const float*)u, (const float*)v, (const float*)w, c->hx64, c->areaw,
                       c->hz64, c->nx, c->ny, c->nz, nbx, nby, kb, c->wx, c->wy, c->red);
  }
  hipLaunchKernelGGL(max_final, dim3(1), dim3(kMaxFinal), 0, s, (const double*)c->red, (int)nb, out);
  return hipGetLastError();
}

hipError_t launch_nusselt(mr_ctx* c, const void* th, const void* w, double* prof, hipStream_t s) {
  const int P = nu_parts(c);
  if (c->nz > kNuMaxFaces) return hipErrorInvalidValue;
  const hipError_t e = ensure_red(c);
  if (e != hipSuccess) return e;
  nusselt_kernels(c, th, w, prof, c->red, P, s);
  return hipGetLastError();
}

int nusselt_fixed(mr_ctx* c, const void* th, const void* w, double* prof, hipStream_t s) {
  const int P = nu_parts(c);
  if (c->nz > kNuMaxFaces || (size_t)c->nz * P * 4 > kNuScratchDoubles) return MR_ESHAPE;
  if (c->device < 0 || c->device >= kMaxDevices) return MR_EINVAL;
  double* part;
  {
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    part = g_scratch[c->device];
  }
  if (!part) return MR_EINVAL;   // mr_init sets it up for the context's device
  nusselt_kernels(c, th, w, prof, part, P, s);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) {
    c->last_err = (int)e;
    return MR_EHIP;
  }
  return MR_OK;
}

hipError_t launch_copy(const void* src, void* dst, int64_t nbytes, hipStream_t s) {
  const int64_t n = nbytes / 16;
  if (n == 0) return hipSuccess;
  const int nb = (int)std::min<int64_t>(65536, (n + 255) / 256);
  hipLaunchKernelGGL(copy_kernel, dim3(nb), dim3(256), 0, s, (const int4*)src, (int4*)dst, n);
  return hipGetLastError();
}

}  // namespace mr
