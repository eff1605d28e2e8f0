// Streaming form of the forward step's variants: side walls, fourth-order face
// values of the advected field, an explicit share of the z diffusion, in any
// combination, on uniform x and y widths.  The walk, the look-ahead, the ring of
// elimination values and the copies into LDS are those of the plain streaming
// step (stream_kernel.h); what differs:
//   - fourth order (ORD4): face values come from four-cell weights on every axis,
//     so the advected field comes with a halo of two rows and at least two columns,
//     and a level is closed by the field two levels ahead.  Second order reads the
//     two cells beside a face only (four cells with weights 0, 1/2, 1/2, 0 let a
//     value that is not finite in two cells further: 0 times it is not 0; 150^3
//     with walls, look-ahead 16: FP64 56.6 us with them, 49.0 without, FP32 35.8 and
//     34.0);
//   - the explicit z share reads the lagged field one level each way, from the
//     column's own values carried along the walk;
//   - a wall's faces have zero weights and carry no velocity, and what the copies
//     bring from beyond it is the chunk or row next to it: the cell itself or one
//     that its other faces weigh, but for FP32 chunks of four columns, where the
//     cell takes its own value instead;
//   - the walk always goes up, and the weights hold registers: workgroups of at
//     most 12 wavefronts.
// Walls and the explicit z share are no template parameters: they cost little.
// On grids that fill the GPU it is bound by the bytes (400 x 300 x 200: FP64 267 us,
// 4.3 TB/s of the 6 values per cell, the line solver 464; FP32 158 and 304; with
// walls alone 258 and 377, 155 and 186), on small ones by a
// level's chain from barrier to barrier (0.6 us with one wavefront per SIMD, 0.9
// with three).  The table row of a level is read at its start, from lines that a
// block's first level has brought into the scalar cache: rows carried in scalar
// registers a level ahead spilled them into vector lanes (140 vector instructions
// a level instead of 66, a third more time at 186^3 FP64: 72 us now, the line
// solver 135).
#pragma once

#include "stream_kernel.h"

namespace mr {
namespace stream {

template <typename T>
struct VarArgs {
  const T* f;          // theta^n
  const T* p;          // theta^{n-1}: x/y diffusion, a_p, explicit z share
  const T* u;
  const T* v;
  const T* w;
  T* out;
  const VarRow<T>* row;   // per walk position
  const double* cb;
  const int* seg;
  const T* c4x;        // face weights of x and y (null: second order)
  const T* c4y;
  T ap, ac, tx, ty;    // tx, ty: tau / h
  T kx, ky;            // tau kappa / h^2
  int nx, ny, nz;
  int ntx, nty, band;
  int wx, wy;
};

// One level of a tile in LDS: as Tile, with two rows of halo for the advected
// field and one for the lagged one, and V >= 2 columns for both.
template <typename T, int TX, int TY, int CH>
struct VarTile {
  static constexpr int W = 64 * TX;
  static constexpr int V = CH / (int)sizeof(T) > 2 ? CH / (int)sizeof(T) : 2;   // columns of halo on each side
  static constexpr int E = CH > (int)sizeof(T) ? CH / (int)sizeof(T) : 1;       // columns of a chunk
  static constexpr int chunks(int cols) { return cols * (int)sizeof(T) / CH; }
  static constexpr int PF = W + 2 * V, PU = W + V;
  static constexpr int cF = chunks(PF), cU = chunks(PU), cW = chunks(W);
  static constexpr int up64(int n) { return (n + 63) / 64; }
  static constexpr int nF = (TY + 4) * cF, nP = (TY + 2) * cF, nU = TY * cU, nV = (TY + 1) * cW, nW = TY * cW;   // chunks
  static constexpr int gP = up64(nF), gU = gP + up64(nP), gV = gU + up64(nU), gW = gV + up64(nV);
  static constexpr int groups = gW + up64(nW);
  static constexpr int slots = (groups + TX * TY - 1) / (TX * TY);
  static constexpr int group = 64 * CH;
  static constexpr int stage = groups * group;
};

// i mod n for any i >= -2 n - 2 .
__device__ __forceinline__ int wrap_any(int i, int n) {
  if (i < 0) {
    i += n;
    if (i < 0) i = (i % n + n) % n;   // axes of one or two cells
  }
  return wrap(i, n);
}

template <typename T, int D, int TX, int TY, int CH, bool ORD4>
__global__ void __launch_bounds__(64 * TX * TY) stream_var_kernel(VarArgs<T> A) {
  constexpr int B = kStreamBlock;
  using L = VarTile<T, TX, TY, CH>;
  constexpr int NSTAGE = 3;
  __shared__ __attribute__((aligned(16))) char buf[NSTAGE * L::stage];
  const int lane = threadIdx.x;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.y);
  const int r = wv / TX, cx = wv - r * TX;
  const int lx = cx * 64 + lane;
  const int nx = A.nx, ny = A.ny, nz = A.nz;
  const int ntile = A.ntx * A.nty;
  const int t = xcd_remap(blockIdx.x, gridDim.x);
  const int sg = t / ntile, g = t - sg * ntile;
  const int per_band = A.band * A.nty;
  const int bnd = g / per_band, rt = g - bnd * per_band;
  const int wb = min(A.band, A.ntx - bnd * A.band);
  const int jt = rt / wb, xt = bnd * A.band + (rt - jt * wb);
  const int i0 = xt * L::W, j0 = jt * TY;
  const int nxy = nx * ny;
  // columns and rows past a ragged end compute a continuation and store nothing
  const bool act = i0 + lx < nx && j0 + r < ny;
  const int i = wrap(i0 + lx, nx), j = wrap(j0 + r, ny);
  constexpr unsigned sz = sizeof(T);
  const unsigned oc = (unsigned)(j * nx + i) * sz;

  const int ks = tab(A.seg, 4 * sg), ke = tab(A.seg, 4 * sg + 1);
  const int k0 = tab(A.seg, 4 * sg + 2), k1 = tab(A.seg, 4 * sg + 3);
  const int64_t plane = (int64_t)nxy * sz;

  const char* base[L::slots];
  unsigned off[L::slots];
#pragma unroll
  for (int q = 0; q < L::slots; ++q) {
    const int gi = min(q * (TX * TY) + wv, L::groups - 1);
    const T* fld = gi < L::gP ? A.f : gi < L::gU ? A.p : gi < L::gV ? A.u : gi < L::gW ? A.v : A.w + nxy;   // w on the face above
    const int g0 = gi < L::gP ? 0 : gi < L::gU ? L::gP : gi < L::gV ? L::gU : gi < L::gW ? L::gV : L::gW;
    const int n = gi < L::gP ? L::nF : gi < L::gU ? L::nP : gi < L::gV ? L::nU : gi < L::gW ? L::nV : L::nW;
    const int cr = gi < L::gU ? L::cF : gi < L::gV ? L::cU : L::cW;
    const int c = min((gi - g0) * 64 + lane, n - 1);
    const int row = c / cr - (gi < L::gP ? 2 : gi < L::gU ? 1 : 0), b = (c % cr) * CH;
    // (across a wall: the chunk or row next to it, whose weight is zero)
    const int ic = i0 - (gi < L::gU ? L::V : 0) + b / (int)sz, jr = j0 + row;
    const int gc = A.wx ? min(max(ic, 0), nx - L::E) : wrap_any(ic, nx), gr = A.wy ? min(max(jr, 0), ny - 1) : wrap_any(jr, ny);
    base[q] = (const char*)(fld + (size_t)k0 * nxy);
    off[q] = (unsigned)(gr * nx + gc) * sz + b % (int)sz;
  }
  const unsigned lds0 = (unsigned)(size_t)(__attribute__((address_space(3))) char*)buf;
  int sn = k0;
  auto issue = [&](int st) {
#pragma unroll
    for (int q = 0; q < L::slots; ++q) copy_lds<CH>(base[q], off[q], lds0 + st * L::stage + min(q * (TX * TY) + wv, L::groups - 1) * L::group);
    const int64_t step = sn + 1 < nz ? plane : 0;
#pragma unroll
    for (int q = 0; q < L::slots; ++q) base[q] += step;
    ++sn;
  };

  // byte offsets inside a stage: the advected field's row - 2, column - 2; the
  // lagged field's row - 1, column - 1; u, v
  const unsigned of = (unsigned)((r * L::PF + lx + L::V - 2) * (int)sz);
  const unsigned op = (unsigned)(L::gP * L::group + (r * L::PF + lx + L::V - 1) * (int)sz);
  const unsigned ou = (unsigned)(L::gU * L::group + (r * L::PU + lx) * (int)sz);
  const unsigned ov = (unsigned)(L::gV * L::group + (r * L::W + lx) * (int)sz);

  // which faces of this cell are walls
  const bool walls = A.wx || A.wy;
  const bool xl = A.wx && i == 0, xh = A.wx && i == nx - 1, yl = A.wy && j == 0, yh = A.wy && j == ny - 1;
  const T kxl = xl ? T(0) : A.kx, kxh = xh ? T(0) : A.kx, kyl = yl ? T(0) : A.ky, kyh = yh ? T(0) : A.ky;
  // fourth order: weights of this column's and row's two faces (0 and n wrap or are walls)
  T xa[4], xb[4], ya[4], yb[4];
  if constexpr (ORD4) {
    const int ih = !A.wx && i + 1 == nx ? 0 : i + 1, jh = !A.wy && j + 1 == ny ? 0 : j + 1;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      xa[q] = A.c4x[4 * i + q];
      xb[q] = A.c4x[4 * ih + q];
      ya[q] = tab(A.c4y, 4 * j + q);
      yb[q] = tab(A.c4y, 4 * jh + q);
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      if (xl) xa[q] = T(0);
      if (xh) xb[q] = T(0);
      if (yl) ya[q] = T(0);
      if (yh) yb[q] = T(0);
    }
  }

  // (the weights of y are wave-uniform: in tiles of 4 wavefronts they go to vector
  // registers, which there are enough of, but for look-aheads of 28 levels, where
  // that would leave a CU two workgroups instead of three)
  if constexpr (ORD4 && TX == 1 && D != 28) {
#pragma unroll
    for (int q = 0; q < 4; ++q) asm("" : "+v"(ya[q]), "+v"(yb[q]));
  }

  double ring[D + B];
#pragma unroll
  for (int q = 0; q < D + B; ++q) ring[q] = 0.0;
  double e = 0.0;
  const T* const fcol = A.f + (size_t)j * nx + i;
  const T* const pcol = A.p + (size_t)j * nx + i;
  // carried along the walk: the advected field one, two and three levels back, the
  // lagged field one and two back, w on the face below and on the one before,
  // the right-hand sides one and two levels back, the flux through the face
  // one level back
  T t1 = fcol[(size_t)max(k0 - 1, 0) * nxy], t2 = fcol[(size_t)max(k0 - 2, 0) * nxy], t3 = T(0);
  T p1 = pcol[(size_t)max(k0 - 1, 0) * nxy], p2 = T(0);
  T w1 = A.w[(size_t)k0 * nxy + (size_t)j * nx + i], w0 = T(0);
  T r1 = T(0), r2 = T(0), fx = T(0);

  struct Row {
    double em, ea, tkb;
    T cz[4], lz[3], tz;
  };
  // FP64 in second order with 16-byte copies: the row is read behind the copies,
  // where fewer scalar registers are in use (moves of spilled ones out of vector
  // lanes: 2 to 477 a kernel before them, 0 to 27 behind)
  constexpr bool LATE = sizeof(T) == 8 && !ORD4 && CH == 16;
  auto load_row = [&](int s) {
    const double* rd = (const double*)(A.row + s);
    const T* rt = (const T*)(rd + 4);
    return Row{tab(rd, 0), tab(rd, 1), tab(rd, 2), {tab(rt, 0), tab(rt, 1), tab(rt, 2), tab(rt, 3)},
               {tab(rt, 4), tab(rt, 5), tab(rt, 6)}, tab(rt, 7)};
  };

  // reads level s, starts the copies `next`, forms level s's x and y terms,
  // completes level s - 1's explicit z share, and closes level s - 2 with the
  // flux through face s - 1; returns that level's elimination value
  auto advance = [&](int s, unsigned sb, int next) {
    const char* b = buf + sb;
    auto at = [&](unsigned o) { return *reinterpret_cast<const T*>(b + o); };
    constexpr unsigned P = L::PF * sz;
    const T fc = at(of + 2 * P + 2 * sz);
    T fxm = at(of + 2 * P + sz), fxp = at(of + 2 * P + 3 * sz), fxm2, fxp2, fym2, fyp2;
    const T fym = at(of + P + 2 * sz), fyp = at(of + 3 * P + 2 * sz);
    if constexpr (ORD4) {
      fxm2 = at(of + 2 * P); fxp2 = at(of + 2 * P + 4 * sz);
      fym2 = at(of + 2 * sz); fyp2 = at(of + 4 * P + 2 * sz);
    }
    const T pc = at(op + P + sz);
    T pxm = at(op + P), pxp = at(op + P + 2 * sz);
    const T pym = at(op + sz), pyp = at(op + 2 * P + sz);
    T u0 = at(ou), u1 = at(ou + sz);
    T v0 = at(ov), v1 = at(ov + L::W * sz);
    const T wn = at(ov + (L::gW - L::gV) * L::group);
    Row rw;
    if constexpr (!LATE) rw = load_row(s);
    issue(next);
    if (walls) {   // wall faces carry no velocity
      u0 = xl ? T(0) : u0;
      u1 = xh ? T(0) : u1;
      v0 = yl ? T(0) : v0;
      v1 = yh ? T(0) : v1;
      if constexpr (L::V > 2) {   // (a chunk of four columns: the one beyond the wall is three columns in)
        fxm = xl ? fc : fxm;
        fxp = xh ? fc : fxp;
        pxm = xl ? pc : pxm;
        pxp = xh ? pc : pxp;
      }
    }
    if constexpr (LATE) rw = load_row(s);
    // face s - 1 (cells s - 3 .. s) and level s - 2
    T fn;
    if constexpr (ORD4) fn = w0 * (rw.cz[0] * t3 + rw.cz[1] * t2 + rw.cz[2] * t1 + rw.cz[3] * fc);
    else fn = w0 * (rw.cz[1] * t2 + rw.cz[2] * t1);
    e = rw.em * ((double)(r2 - rw.tz * (fn - fx)) + rw.tkb) + rw.ea * e;
    asm volatile("" : "+v"(e));   // the level is finished here (keeps the levels' work in order)
    // level s - 1: the explicit z share of the lagged field
    r2 = r1 + (rw.lz[0] * p2 + rw.lz[1] * p1 + rw.lz[2] * pc);
    // level s: x and y
    T fxl, fxh, fyl, fyh;
    if constexpr (ORD4) {
      fxl = xa[0] * fxm2 + xa[1] * fxm + xa[2] * fc + xa[3] * fxp, fxh = xb[0] * fxm + xb[1] * fc + xb[2] * fxp + xb[3] * fxp2;
      fyl = ya[0] * fym2 + ya[1] * fym + ya[2] * fc + ya[3] * fyp, fyh = yb[0] * fym + yb[1] * fc + yb[2] * fyp + yb[3] * fyp2;
    } else {
      const T half = T(0.5);
      fxl = half * (fxm + fc), fxh = half * (fc + fxp), fyl = half * (fym + fc), fyh = half * (fc + fyp);
    }
    r1 = A.ap * pc + A.ac * fc - ((u1 * fxh - u0 * fxl) * A.tx + (v1 * fyh - v0 * fyl) * A.ty) +
         (kxh * (pxp - pc) - kxl * (pc - pxm)) + (kyh * (pyp - pc) - kyl * (pc - pym));
    asm volatile("" : "+v"(r1), "+v"(r2));
    fx = fn;
    t3 = t2; t2 = t1; t1 = fc;
    p2 = p1; p1 = pc;
    w0 = w1; w1 = wn;
    return e;
  };

  // back substitution from the newest position of the ring; writes the oldest
  // block (kx: position of ring[0]); true if that took exactly B stores
  const bool any = __any(act);
  auto emit = [&](int kx) {
    double x = 0.0;
    const bool whole = kx >= ks && kx + B <= ke;
#pragma unroll
    for (int q = D + B - 1; q >= B; --q) x = ring[q] - tab(A.cb, kx + q) * x;
    T xo[B];
#pragma unroll
    for (int q = B - 1; q >= 0; --q) {
      x = ring[q] - tab(A.cb, kx + q) * x;
      xo[q] = (T)x;
    }
    if (whole) {
#pragma unroll
      for (int q = 0; q < B; ++q)
        if (act) st_nt(A.out + (size_t)(kx + q) * nxy, oc, xo[q]);
    } else {
#pragma unroll
      for (int q = 0; q < B; ++q)
        if (act && kx + q >= ks && kx + q < ke) st_nt(A.out + (size_t)(kx + q) * nxy, oc, xo[q]);
    }
    return whole && any;
  };
  auto shift = [&]() {
#pragma unroll
    for (int q = 0; q < D; ++q) ring[q] = ring[q + B];
  };

  // levels k0 .. k1 + 1: level s closes s - 2, whose elimination value enters the
  // ring; the first two close nothing (their values are dropped), the last two
  // only close
#pragma unroll
  for (int s = 0; s < NSTAGE - 1; ++s) issue(s);
  constexpr int N = (NSTAGE - 2) * L::slots;
  wait_barrier<N>();
  advance(k0, 0, NSTAGE - 1);
  wait_barrier<N>();
  advance(k0 + 1, L::stage, 0);
  e = 0.0;
  int st = 1;
  int stored = 0;   // (wave-uniform) the B stores of the block before are younger than the position's copies
  int q = k0;
  for (; q < k1; q += B) {
    // the rows of the block after this one into the scalar cache, all at once: a
    // miss per level would be waited for with that level's LDS reads, and rows held
    // in registers a level ahead spill
    touch_rows(A.row, q + B + 2, nz + kStreamRowPad - 1);
#pragma unroll
    for (int s = 0; s < B; ++s) {
      const int last = st;
      st = st == NSTAGE - 1 ? 0 : st + 1;
      if (s < NSTAGE - 1 && stored) wait_barrier<N + B>();
      else wait_barrier<N>();
      ring[D + s] = advance(q + s + 2, st * L::stage, last);   // (last: the slot read before this barrier)
      __builtin_amdgcn_sched_barrier(0);
    }
    stored = 0;
    if (q + B - D > ks) stored = __builtin_amdgcn_readfirstlane((int)emit(q - D));
    shift();
  }
#pragma unroll
  for (int s = 0; s < B; ++s) ring[D + s] = 0.0;
  for (; q - D < ke; q += B) {
    emit(q - D);
    shift();
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // no copy into LDS outlives the workgroup
}

// Launches the kernel of a context's tile shape and look-ahead.
template <typename T, int TX, int TY, int CH, bool ORD4, int Q>
hipError_t launch_var_depth(int depth, dim3 grid, const VarArgs<T>& a, hipStream_t s) {
  if constexpr (Q < kStreamDepths) {
    constexpr int D = kStreamDepth[Q];
    if (depth != Q) return launch_var_depth<T, TX, TY, CH, ORD4, Q + 1>(depth, grid, a, s);
    if constexpr (stream_var_fits(D, TX * TY)) {
      hipLaunchKernelGGL((stream_var_kernel<T, D, TX, TY, CH, ORD4>), grid, dim3(64, TX * TY), 0, s, a);
      return hipGetLastError();
    }
  }
  return hipErrorInvalidValue;
}

template <typename T, int CH, bool ORD4>
hipError_t launch_var_shape(int shape, int depth, dim3 grid, const VarArgs<T>& a, hipStream_t s) {
  static_assert(kStreamShapes == 4, "one case per shape (the widest holds too many wavefronts)");
  switch (shape) {
    case 1: return launch_var_depth<T, kStreamShape[1].segs, kStreamShape[1].rows, CH, ORD4, 0>(depth, grid, a, s);
    case 2: return launch_var_depth<T, kStreamShape[2].segs, kStreamShape[2].rows, CH, ORD4, 0>(depth, grid, a, s);
    case 3: return launch_var_depth<T, kStreamShape[3].segs, kStreamShape[3].rows, CH, ORD4, 0>(depth, grid, a, s);
  }
  return hipErrorInvalidValue;
}

template <typename T>
hipError_t launch_stream_var(int shape, int depth, dim3 grid, const VarArgs<T>& a, hipStream_t s) {
  const uintptr_t p = (uintptr_t)a.f | (uintptr_t)a.p | (uintptr_t)a.u | (uintptr_t)a.v | (uintptr_t)a.w;
  const bool wide = ((uintptr_t)a.nx * sizeof(T)) % 16 == 0 && p % 16 == 0;
  if (a.c4x)
    return wide ? launch_var_shape<T, 16, true>(shape, depth, grid, a, s) : launch_var_shape<T, 4, true>(shape, depth, grid, a, s);
  return wide ? launch_var_shape<T, 16, false>(shape, depth, grid, a, s) : launch_var_shape<T, 4, false>(shape, depth, grid, a, s);
}

}  // namespace stream
}  // namespace mr
