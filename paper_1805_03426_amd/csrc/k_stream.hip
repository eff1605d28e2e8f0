// Host side of the streaming step: how a context's grid is cut into tiles and
// z segments, and the launches (kernels in stream_kernel.h, instantiated in
// k_stream64.hip and k_stream32.hip).
#include "stream_variant.h"

#include <math.h>

#include <algorithm>

namespace mr {
namespace stream {
extern template hipError_t launch_stream<double, false>(int, int, dim3, const StreamArgs<double>&, hipStream_t);
extern template hipError_t launch_stream<double, true>(int, int, dim3, const StreamArgs<double>&, hipStream_t);
extern template hipError_t launch_stream<float, false>(int, int, dim3, const StreamArgs<float>&, hipStream_t);
extern template hipError_t launch_stream<float, true>(int, int, dim3, const StreamArgs<float>&, hipStream_t);
extern template hipError_t launch_stream_var<double>(int, int, dim3, const VarArgs<double>&, hipStream_t);
extern template hipError_t launch_stream_var<float>(int, int, dim3, const VarArgs<float>&, hipStream_t);
}  // namespace stream

// Tile shape and number of z segments: the pair with the least time by a model
// of what bounds the launch, the longer of
//   - the bytes of all workgroups at the rate that the shape reaches when the
//     GPU is full (wider rows of columns do better), half of the columns past a
//     ragged end counted;
//   - the levels of a walk times what a level takes a CU that holds one
//     workgroup, or as many as the fullest CU gets.
// Timed, for instance (128 x 4 columns: 256^3 in FP64, 144 us with 2 segments,
// one workgroup for each of 256 CUs; 189 us with 1, 177 with 3, half of the CUs
// idle or a second round for half of them).  400^3 FP64: 256 x 4 and 1 segment
// 602 us, 128 x 4 702; 576^3 FP64: 192 x 4 1.87 ms, 256 x 4 2.09; 450 x 300 x
// 200 FP32, 1 segment: 192 x 4 155 us, 128 x 4 190 (300 workgroups on 256 CUs; at
// a reach of few levels the model takes 2 segments, 2% ahead by its figures: 171).
// The estimate that goes with the plan (us) takes a level's time on a CU that holds
// one workgroup (alone_us), or several, from steps timed at 66 grids and four
// look-aheads each (medians by shape); the choice among plans leaves the 64-column
// tiles more than they take alone (one_us), which the estimate must not.  Copies of 4
// bytes take 1.6 times as long (FP64) and 1.1 (FP32).  Look-aheads of 60 levels leave
// a CU two workgroups of 4 wavefronts at a time.
// Variants (walls, fourth order, explicit z): 186^3 FP64 192 x 4 columns and 4
// segments 72 us, 3 segments 77, 64 x 4 and 3 segments 68; 128 x 4 and 5, 85.
StreamPlan stream_plan(int nx, int ny, int nz, bool f64, bool variant, int cus, int depth, const std::vector<int> (&before)[2],
                       const std::vector<int> (&after)[2]) {
  struct Shape {
    double one_us;    // a level of the only workgroup of a CU
    double more_us;   // a level for each workgroup of a CU that holds several
    double rate;      // bytes per us of a full GPU
    double alone_us, shared_us;   // one_us and more_us of the estimate
  };
  static const Shape s64[kStreamShapes] = {{1.40, 1.40, 5.6e6, 1.37, 1.37}, {1.13, 1.13, 5.5e6, 1.13, 1.13},
                                           {0.72, 0.72, 5.35e6, 0.66, 0.66}, {0.60, 0.33, 5.0e6, 0.43, 0.28}};
  static const Shape s32[kStreamShapes] = {{0.70, 0.70, 5.6e6, 0.80, 0.75}, {0.70, 0.60, 5.5e6, 0.67, 0.60},
                                           {0.61, 0.38, 5.35e6, 0.58, 0.44}, {0.55, 0.25, 5.0e6, 0.40, 0.22}};
  // the variants' kernels (three shapes; FP64 with 4-byte copies takes 1.6 times as long a level)
  static const Shape v64[kStreamShapes] = {{}, {0.95, 0.95, 5.5e6, 0.86, 0.86}, {0.68, 0.68, 5.5e6, 0.67, 0.67}, {0.60, 0.42, 5.0e6, 0.57, 0.42}};
  static const Shape v32[kStreamShapes] = {{}, {0.70, 0.62, 5.5e6, 0.70, 0.62}, {0.55, 0.45, 5.35e6, 0.55, 0.44}, {0.48, 0.22, 5.0e6, 0.41, 0.22}};
  const double slow = variant && f64 && nx % 2 ? 1.6 : 1.0;
  const Shape* sh = variant ? (f64 ? v64 : v32) : (f64 ? s64 : s32);
  const double sz = f64 ? 8.0 : 4.0;
  StreamPlan best;
  double best_us = -1.0;
  for (int q = 0; q < kStreamShapes; ++q) {
    const int waves = kStreamShape[q].segs * kStreamShape[q].rows;
    if (!(variant ? stream_var_fits(kStreamDepth[depth], waves) : stream_fits(kStreamDepth[depth], waves))) continue;
    const int tw = 64 * kStreamShape[q].segs, rows = kStreamShape[q].rows;
    const int64_t ntx = (nx + tw - 1) / tw, nty = (ny + rows - 1) / rows;
    const double cols = (double)nx * ny;
    const double loaded = cols + 0.5 * ((double)(ntx * tw) * (nty * rows) - cols);
    for (int nseg = 1; nseg <= kStreamMaxSeg && (nseg == 1 || nz / nseg >= 8); ++nseg) {
      StreamPlan p;
      p.shape = q;
      p.nseg = nseg;
      int levels = 0;
      double walked = 0.0;
      for (int d = 0; d < 2; ++d)
        for (int g = 0; g < nseg; ++g) {
          const int ks = (int)((int64_t)nz * g / nseg), ke = (int)((int64_t)nz * (g + 1) / nseg);
          const int a0 = g ? std::max(0, ks - before[d][ks]) : 0;
          int a1 = std::min(nz, ke + after[d][ke - 1]);
          a1 += (kStreamBlock - (a1 - a0) % kStreamBlock) % kStreamBlock;   // whole blocks
          p.seg[d].insert(p.seg[d].end(), {ks, ke, a0, a1});
          levels = std::max(levels, a1 - a0);
          if (d == 0) walked += a1 - a0;
        }
      const double per_cu = (double)((ntx * nty * nseg + cus - 1) / cus);   // of the fullest CU
      const double mem = (5.0 * walked + nz) * loaded * sz / sh[q].rate;
      const double us = std::max(mem, (levels + 6) * slow * std::max(sh[q].one_us, per_cu * sh[q].more_us));
      if (best_us < 0.0 || us < best_us) {
        best_us = us;
        const double narrow = f64 ? (nx % 2 ? 1.6 : 1.0) : (nx % 4 ? 1.1 : 1.0);
        const bool pairs = kStreamDepth[depth] > 44 && waves == 4 && per_cu > 1.0;   // two at a time on a CU
        const double busy = sh[q].shared_us * (pairs ? 2.0 * ceil(per_cu / 2.0) : per_cu);
        p.us = std::max(mem, (levels + 6) * narrow * std::max(sh[q].alone_us, busy));
        best = p;
      }
    }
  }
  return best;
}

namespace {
using namespace stream;

template <typename T>
const StreamSys<T>& sys(const mr_ctx* c, bool rev, int down, int kind);
template <>
const StreamSys<double>& sys<double>(const mr_ctx* c, bool rev, int down, int kind) { return c->sr64[rev][down][kind]; }
template <>
const StreamSys<float>& sys<float>(const mr_ctx* c, bool rev, int down, int kind) { return c->sr32[rev][down][kind]; }

template <typename T>
const StreamSys<T>& sys_id(const mr_ctx* c);
template <>
const StreamSys<double>& sys_id<double>(const mr_ctx* c) { return c->sid64; }
template <>
const StreamSys<float>& sys_id<float>(const mr_ctx* c) { return c->sid32; }

// Arguments of both directions: f the advected field, p the second field, the
// implicit system of step kind `solve` (transposed in the reverse step; -1: none).
template <typename T, bool REV>
StreamArgs<T> base_args(const mr_ctx* c, bool down, int solve, const void* f, const void* p, void* out, const void* u,
                        const void* v, const void* w) {
  StreamArgs<T> a;
  ::memset((void*)&a, 0, sizeof(a));
  a.f = (const T*)f;
  a.p = (const T*)p;
  a.u = (const T*)u;
  a.v = (const T*)v;
  a.w = (const T*)w;
  a.out = (T*)out;
  a.down = down;
  const StreamSys<T>& sy = solve >= 0 ? sys<T>(c, REV, a.down, solve) : sys_id<T>(c);
  a.row = sy.row;
  a.cb = sy.cb;
  a.seg = c->stream_seg[a.down];
  a.uhx = (T)c->uhx;
  a.uhy = (T)c->uhy;
  a.uxx = (T)(c->uhx * c->uhx);
  a.uyy = (T)(c->uhy * c->uhy);
  a.nx = c->nx;
  a.ny = c->ny;
  a.nz = c->nz;
  const StreamShape sh = kStreamShape[c->stream_shape];
  a.ntx = (c->nx + 64 * sh.segs - 1) / (64 * sh.segs);
  a.nty = (c->ny + sh.rows - 1) / sh.rows;
  // bands of 8 x tiles: 1024 x 1024 x 512 within 1% of 4, 2-6% faster than 1 and 2
  a.band = std::min(8, a.ntx);
  return a;
}

template <typename T, bool REV>
hipError_t launch(const mr_ctx* c, const StreamArgs<T>& a, hipStream_t s) {
  const dim3 grid((unsigned)((int64_t)a.ntx * a.nty * c->stream_nseg));
  return launch_stream<T, REV>(c->stream_shape, c->stream_d - 1, grid, a, s);
}

template <typename T>
hipError_t fwd_t(mr_ctx* c, int64_t n, int q, const void* thp, const void* thc, void* out, const void* u, const void* v,
                 const void* w, hipStream_t s) {
  const int kind = step_kind(n, c->n_avg);
  // FP32 where the column sweeps would run (q >= 0, the step's index in its
  // sequence): their walk direction and their float elimination values, so that
  // the same float results come out (but for the last bit where the doubles
  // behind them differ in theirs)
  const bool as_sweep = sizeof(T) == 4 && q >= 0;
  StreamArgs<T> a = base_args<T, false>(c, as_sweep ? !(q & 1) : (n & 1), kind, thc, thp, out, u, v, w);
  a.as_sweep = as_sweep;
  a.ap = (T)alpha_prev(kind);
  a.ac = (T)alpha_cur(kind);
  a.tau = (T)c->tau[kind];
  a.tk = (T)(c->tau[kind] * c->kappa);
  return launch<T, false>(c, a, s);
}

// Reverse step n: the transposed stencils of step n on mu^n, the lagged
// diffusion of step n+1 on mu^{n+1} (zero weights without one), the transposed
// system of step n-1.  Step 0: no system (the derivative with respect to theta^0),
// and the start-up step's own diffusion.  In us, line solver and this: 256^3 FP32
// 103 and 84, 1024 x 1024 x 512 FP32 4016 and 2451, FP64 8352 and 5172.
template <typename T>
hipError_t bwd_t(mr_ctx* c, int64_t n, const void* mun, const void* muc, void* out, const void* u, const void* v,
                 const void* w, hipStream_t s) {
  const int kind = step_kind(n, c->n_avg);
  StreamArgs<T> a =
      base_args<T, true>(c, n & 1, n > 0 ? step_kind(n - 1, c->n_avg) : -1, muc, mun ? mun : muc, out, u, v, w);
  a.ac = (T)alpha_cur(kind);
  a.tau = (T)c->tau[kind];
  a.tk0 = n == 0 ? (T)(c->tau[kind] * c->kappa) : T(0);
  if (mun) {
    const int k1 = step_kind(n + 1, c->n_avg);
    a.ap = (T)alpha_prev(k1);
    a.tk = (T)(c->tau[k1] * c->kappa);
  }
  return launch<T, true>(c, a, s);
}

template <typename T>
hipError_t var_t(mr_ctx* c, const Geom<T>& g, int64_t n, const void* thp, const void* thc, void* out, const void* u,
                 const void* v, const void* w, hipStream_t s) {
  const int kind = step_kind(n, c->n_avg);
  VarArgs<T> a;
  ::memset((void*)&a, 0, sizeof(a));
  a.f = (const T*)thc;
  a.p = (const T*)thp;
  a.u = (const T*)u;
  a.v = (const T*)v;
  a.w = (const T*)w;
  a.out = (T*)out;
  a.row = (const VarRow<T>*)c->vrow[kind];
  a.cb = c->vcb[kind];
  a.seg = c->stream_seg[0];
  a.c4x = c->face_order == 4 ? g.c4x : nullptr;
  a.c4y = c->face_order == 4 ? g.c4y : nullptr;
  a.ap = (T)alpha_prev(kind);
  a.ac = (T)alpha_cur(kind);
  a.tx = (T)(c->tau[kind] * c->uhx);
  a.ty = (T)(c->tau[kind] * c->uhy);
  a.kx = (T)(c->tau[kind] * c->kappa * c->uhx * c->uhx);
  a.ky = (T)(c->tau[kind] * c->kappa * c->uhy * c->uhy);
  a.nx = c->nx;
  a.ny = c->ny;
  a.nz = c->nz;
  const StreamShape sh = kStreamShape[c->stream_shape];
  a.ntx = (c->nx + 64 * sh.segs - 1) / (64 * sh.segs);
  a.nty = (c->ny + sh.rows - 1) / sh.rows;
  a.band = std::min(8, a.ntx);
  a.wx = c->wx;
  a.wy = c->wy;
  const dim3 grid((unsigned)((int64_t)a.ntx * a.nty * c->stream_nseg));
  return launch_stream_var<T>(c->stream_shape, c->stream_v - 1, grid, a, s);
}

}  // namespace

hipError_t launch_stream_step_var(mr_ctx* c, int64_t n, const void* thp, const void* thc, void* out, const void* u,
                                  const void* v, const void* w, hipStream_t s) {
  return c->precision == MR_FP64 ? var_t<double>(c, c->g64, n, thp, thc, out, u, v, w, s)
                                 : var_t<float>(c, c->g32, n, thp, thc, out, u, v, w, s);
}

hipError_t launch_stream_step(mr_ctx* c, int64_t n, int q, const void* thp, const void* thc, void* out,
                              const void* u, const void* v, const void* w, hipStream_t s) {
  return c->precision == MR_FP64 ? fwd_t<double>(c, n, q, thp, thc, out, u, v, w, s)
                                 : fwd_t<float>(c, n, q, thp, thc, out, u, v, w, s);
}

hipError_t launch_stream_step_backward(mr_ctx* c, int64_t n, const void* mun, const void* muc, void* out,
                                       const void* u, const void* v, const void* w, hipStream_t s) {
  return c->precision == MR_FP64 ? bwd_t<double>(c, n, mun, muc, out, u, v, w, s)
                                 : bwd_t<float>(c, n, mun, muc, out, u, v, w, s);
}

}  // namespace mr
