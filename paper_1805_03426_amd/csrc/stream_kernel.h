// Streaming form of the scalar step and of its reverse (Eqs. 5-7 with the z
// diffusion implicit): one kernel per step, one pass over the fields.
//
// The implicit z system I - tau kappa Lz is diagonally dominant, so the factor
// with which a level's value enters the solution d levels away falls with d
// (each level multiplies it by about r / (1 + 2 r), r = tau kappa / h^2).  A
// workgroup walks a tile of columns in z, level by level: it builds the
// right-hand side, runs the Thomas elimination (in double) and keeps the last
// D + B elimination values in registers.  After every B levels it back-
// substitutes from the newest level and writes the B oldest ones: D levels of
// look-ahead, D taken by the host such that the product of the D factors is at
// most kTruncate64 (FP64) or kTruncate32 (FP32), which is what the solution
// can miss of a value D levels ahead, far below the rounding of the stored
// type.  No elimination value goes to memory and no column is held whole: a
// cell is read as 5 values and written as 1.
//
// The walk may be cut into z segments, each a workgroup of its own: a segment
// starts its elimination the same kind of distance before its first level
// (from zero) and looks ahead past its last one, so segments exchange nothing;
// the levels in between are computed twice.  Grids with few columns fill the
// GPU that way.  Even steps walk up, odd ones down, so that a step finds the
// levels that the step before touched last in the 256 MB Infinity Cache
// (256^3: 3-5% faster in FP64 and FP32 than always upwards).
//
// What bounds it: the bytes from memory.  Each level of the tile (five fields,
// theta and the lagged field with a halo of one row and one chunk of columns)
// is copied straight from memory to LDS, two levels ahead of the one being
// worked on (no registers hold loads in flight, which leaves them to the
// elimination values), and one barrier per level hands it over.  x, y
// neighbours then come from LDS.  Timed per step at 1024 x 1024 x 512 on
// 256 x 4 tiles: 5.18 ms in FP64 (4.97 TB/s of the 6 values per cell; a copy of
// this size reaches 5.3) and 2.44 ms in FP32 (5.3 TB/s), against 6.24 and 2.75 ms
// for the column sweeps, whose elimination values go through memory, and 8.24 and
// 3.89 for the line solver; the reverse step 5.17 and 2.45, 6.30 and 2.77, 8.35 and
// 4.02.  The same walk with loads into registers and neighbours from the cache took
// a fifth (FP64) and a third (FP32) longer than this: 26% and 62% more lines came
// from memory than the five fields have, because the wavefronts drifted apart.
#pragma once

#include <string.h>

#include "mr_internal.h"

namespace mr {
namespace stream {

template <typename T>
struct StreamArgs {
  const T* f;         // theta^n (reverse: mu^n): the advected field
  const T* p;         // theta^{n-1} (reverse: mu^{n+1}): x/y diffusion and a_p
  const T* u;
  const T* v;
  const T* w;
  T* out;
  const StreamRow<T>* row;   // per walk position
  const double* cb;          // per walk position s: x_s = e_s - cb_s x_{s+1}; readable from -kStreamPad
  const int* seg;            // per z segment: first position, end, walk start, walk end
  T ap, ac, tau, tk;
  T tk0;                     // reverse step 0: tau kappa of the start-up step's own diffusion (else 0)
  T uhx, uhy, uxx, uyy;
  int nx, ny, nz;
  int ntx, nty;              // tiles per level
  int band;                  // x tiles per band of the tile walk
  int down;                  // walk downwards
  int as_sweep;              // FP32 forward step: round as the column sweeps do (elimination values in float)
};

__device__ __forceinline__ double fma_(double a, double b, double c) { return __builtin_fma(a, b, c); }
__device__ __forceinline__ float fma_(float a, float b, float c) { return __builtin_fmaf(a, b, c); }

template <typename T>
__device__ __forceinline__ void st_nt(T* base, unsigned off, T v) {
  __builtin_nontemporal_store(v, reinterpret_cast<T*>(reinterpret_cast<char*>(base) + off));
}
// Wave-uniform table reads through the constant address space (scalar loads).
template <typename T>
__device__ __forceinline__ T tab(const T* p, int k) {
  return ((const __attribute__((address_space(4))) T*)(p))[k];
}

// Reads kStreamBlock table rows from row s on (at most row `last`), every 64-byte line of them.
template <typename R>
__device__ __forceinline__ void touch_rows(const R* row, int s, int last) {
  constexpr int N = (int)sizeof(R) / 64;
  static_assert(kStreamBlock == 8 && N >= 1 && N <= 2, "the operands below");
  float x[kStreamBlock][2];
#pragma unroll
  for (int q = 0; q < kStreamBlock; ++q)
#pragma unroll
    for (int l = 0; l < 2; ++l) x[q][l] = tab((const float*)(row + min(s + q, last)), (l < N ? l : 0) * 16);
  asm volatile("" ::"s"(x[0][0]), "s"(x[1][0]), "s"(x[2][0]), "s"(x[3][0]), "s"(x[4][0]), "s"(x[5][0]), "s"(x[6][0]), "s"(x[7][0]));
  if constexpr (N == 2)
    asm volatile("" ::"s"(x[0][1]), "s"(x[1][1]), "s"(x[2][1]), "s"(x[3][1]), "s"(x[4][1]), "s"(x[5][1]), "s"(x[6][1]), "s"(x[7][1]));
}

// Asynchronous copy of one chunk per lane from memory to LDS (lane l's chunk
// lands at dst + l * CH).
template <int CH>
__device__ __forceinline__ void copy_lds(const char* base, unsigned off, unsigned dst) {
  if constexpr (CH == 16)
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(dst), "v"(off), "s"(base) : "memory", "m0");
  else
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, %2" ::"s"(dst), "v"(off), "s"(base) : "memory", "m0");
}
// Waits until at most N memory operations of this wavefront are under way and
// its LDS reads are done, then for the workgroup.
template <int N>
__device__ __forceinline__ void wait_barrier() {
  asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(N) : "memory");
}

// Shape of a tile and of one level of it in LDS: the rows of the five fields
// one after the other, theta and the lagged field with one row and one chunk
// of columns more on each side, u with a chunk more to the right, v with a row
// more above.
template <typename T, int TX, int TY, int CH>
struct Tile {
  static constexpr int W = 64 * TX;
  static constexpr int V = CH < (int)sizeof(T) ? 1 : CH / (int)sizeof(T);   // columns of halo on each side
  static constexpr int chunks(int cols) { return cols * (int)sizeof(T) / CH; }
  static constexpr int PF = W + 2 * V, PU = W + V;                 // row pitches in values
  static constexpr int cF = chunks(PF), cU = chunks(PU), cW = chunks(W);
  // groups of 64 chunks (one copy of a wavefront), each in one field
  static constexpr int up64(int n) { return (n + 63) / 64; }
  static constexpr int nF = (TY + 2) * cF, nU = TY * cU, nV = (TY + 1) * cW, nW = TY * cW;   // chunks
  static constexpr int gP = up64(nF), gU = 2 * gP, gV = gU + up64(nU), gW = gV + up64(nV), groups = gW + up64(nW);
  static constexpr int slots = (groups + TX * TY - 1) / (TX * TY);   // copies of a wavefront per level
  static constexpr int group = 64 * CH;                              // bytes of a group in LDS
  static constexpr int stage = groups * group;                       // bytes of a level in LDS
};

// i mod n for -n <= i, by subtraction where one is enough.
__device__ __forceinline__ int wrap(int i, int n) {
  if (i < 0) i += n;
  if (i >= n) {
    i -= n;
    if (i >= n) i %= n;   // only where the tile is wider than the grid
  }
  return i;
}

template <typename T, int D, bool REV, int TX, int TY, int CH>
__global__ void __launch_bounds__(64 * TX * TY) stream_kernel(StreamArgs<T> A) {
  constexpr int B = kStreamBlock;
  using L = Tile<T, TX, TY, CH>;
  constexpr int NSTAGE = 3;   // levels in LDS: one being worked on, two on their way (four: no faster)
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
  // columns and rows past a ragged end are the periodic continuation: they
  // repeat another tile's columns (the same values) and are not stored
  const bool act = i0 + lx < nx && j0 + r < ny;
  const int i = wrap(i0 + lx, nx), j = wrap(j0 + r, ny);
  constexpr unsigned sz = sizeof(T);
  const unsigned oc = (unsigned)(j * nx + i) * sz;

  const int ks = tab(A.seg, 4 * sg), ke = tab(A.seg, 4 * sg + 1);
  const int k0 = tab(A.seg, 4 * sg + 2), k1 = tab(A.seg, 4 * sg + 3);   // k1 - k0 is whole blocks
  const int64_t plane = (A.down ? -1 : 1) * (int64_t)nxy * sz;          // bytes from a position to the next
  auto level = [&](int s) { return A.down ? nz - 1 - s : s; };

  // this wavefront's groups of a level: the field at position k0 (wave-uniform)
  // and this lane's chunk in it
  const char* base[L::slots];
  unsigned off[L::slots];
#pragma unroll
  for (int q = 0; q < L::slots; ++q) {
    const int gi = min(q * (TX * TY) + wv, L::groups - 1);
    const T* fld = gi < L::gP ? A.f : gi < L::gU ? A.p : gi < L::gV ? A.u : gi < L::gW ? A.v : A.w;
    if (gi >= L::gW && !A.down) fld += nxy;   // w on the face above
    const int g0 = gi < L::gP ? 0 : gi < L::gU ? L::gP : gi < L::gV ? L::gU : gi < L::gW ? L::gV : L::gW;
    const int n = gi < L::gU ? L::nF : gi < L::gV ? L::nU : gi < L::gW ? L::nV : L::nW;      // chunks of the field
    const int cr = gi < L::gU ? L::cF : gi < L::gV ? L::cU : L::cW;                          // and of a row of it
    const int c = min((gi - g0) * 64 + lane, n - 1);
    const int row = c / cr - (gi < L::gU ? 1 : 0), b = (c % cr) * CH;   // tile row, byte inside the row
    const int gc = wrap(i0 - (gi < L::gU ? L::V : 0) + b / (int)sz, nx), gr = wrap(j0 + row, ny);
    base[q] = (const char*)(fld + (size_t)level(k0) * nxy);
    off[q] = (unsigned)(gr * nx + gc) * sz + b % (int)sz;
  }
  const unsigned lds0 = (unsigned)(size_t)(__attribute__((address_space(3))) char*)buf;
  // copies the next position into stage slot `st` and moves on (at the last level stays there)
  int sn = k0;
  auto issue = [&](int st) {
#pragma unroll
    for (int q = 0; q < L::slots; ++q) copy_lds<CH>(base[q], off[q], lds0 + st * L::stage + min(q * (TX * TY) + wv, L::groups - 1) * L::group);
    const int64_t step = sn + 1 < nz ? plane : 0;
#pragma unroll
    for (int q = 0; q < L::slots; ++q) base[q] += step;
    ++sn;
  };

  // values in the tile's own position: byte offsets inside a stage
  const unsigned of = (unsigned)((r * L::PF + lx) * (int)sz + (L::V - 1) * (int)sz);   // (row - 1, column - 1)
  const unsigned ou = (unsigned)(L::gU * L::group + (r * L::PU + lx) * (int)sz);
  const unsigned ov = (unsigned)(L::gV * L::group + (r * L::W + lx) * (int)sz);

  double ring[D + B];
#pragma unroll
  for (int q = 0; q < D + B; ++q) ring[q] = 0.0;
  double e = 0.0;
  const T half = T(0.5);
  // the advected field one position back, w on the face ahead of it, and what
  // is formed of that position's right-hand side (rr; FP32 forward step: the x and y
  // advection pxy, the lagged x/y diffusion lap, the rear face's sum and w)
  T tc = A.f[(size_t)level(max(k0 - 1, 0)) * nxy + (size_t)j * nx + i];
  T wf = A.w[(size_t)(A.down ? level(k0) + 1 : level(k0)) * nxy + (size_t)j * nx + i];
  T rr = T(0), pxy = T(0), lap = T(0), rs = T(0), wr = T(0);

  // the table rows of the position being read and of the one behind it; the
  // next one is loaded a position ahead
  struct Row {
    double em, ea, tkb;
    T c0, c1, c2, c3;
  };
  auto load_row = [&](int s) {
    const double* rd = (const double*)(A.row + s);
    const T* rt = (const T*)(rd + 4);
    return Row{tab(rd, 0), tab(rd, 1), tab(rd, 2), tab(rt, 0), tab(rt, 1), tab(rt, 2), tab(rt, 3)};
  };
  Row rb = load_row(k0 - 1), rc = load_row(k0);

  // reads a position's values, starts the copies `next` and forms all of the
  // position's right-hand side but what the field ahead enters; returns the
  // elimination value of the position behind, which this position's field closes.
  // The FP32 forward step's products and sums are grouped as in the line solver
  // (as_sweep: the column sweeps) by explicit fused multiply-adds, so that its
  // right-hand sides are the same bit for bit; FP64 keeps fewer values for it.
  const bool as_sweep = sizeof(T) == 4 && !REV && A.as_sweep;
  auto advance = [&](int s, unsigned sb, int next) {
    const char* b = buf + sb;
    auto at = [&](unsigned o) { return *reinterpret_cast<const T*>(b + o); };
    const T fym = at(of + sz), fxm = at(of + L::PF * sz), fc = at(of + (L::PF + 1) * sz), fxp = at(of + (L::PF + 2) * sz);
    const T fyp = at(of + (2 * L::PF + 1) * sz);
    constexpr unsigned dp = L::gP * L::group;
    const T pym = at(of + dp + sz), pxm = at(of + dp + L::PF * sz), pc = at(of + dp + (L::PF + 1) * sz);
    const T pxp = at(of + dp + (L::PF + 2) * sz), pyp = at(of + dp + (2 * L::PF + 1) * sz);
    const T u0 = at(ou), u1 = at(ou + sz);
    const T v0 = at(ov), v1 = at(ov + L::W * sz);
    const T wn = at(ov + (L::gW - L::gV) * L::group);
    issue(next);
    const Row rn = load_row(s + 1);
    // close the position behind: the flux through the face ahead of it
    T r0;
    if constexpr (REV) {
      r0 = rr + A.tau * half * (wf * (fc * rb.c0 - tc * rb.c1));
    } else if constexpr (sizeof(T) == 8) {
      r0 = rr - A.tau * half * (rb.c0 * wf * (tc + fc));
    } else {
      const T fs = tc + fc, wa = rb.c0 * wf;
      const T z = A.down ? fma_(rs, wr, -(wa * fs)) : fma_(fs, wa, -(wr * rs));   // (flux above) - (flux below)
      r0 = fma_(A.tk, lap, fma_(-A.tau, half * fma_(rb.c1, z, pxy), rr));
    }
    e = rb.em * ((double)r0 + rb.tkb) + rb.ea * e;
    asm volatile("" : "+v"(e));   // the level is finished here (keeps the levels' work in order)
    // this position's right-hand side: its rear face, x and y
    const T lx2 = fma_(T(-2), pc, pxp + pxm), ly2 = fma_(T(-2), pc, pyp + pym);
    if constexpr (REV || sizeof(T) == 8) {
      T adv;
      if constexpr (REV)
        adv = half * ((u0 * (fc - fxm) + u1 * (fxp - fc)) * A.uhx + (v0 * (fc - fym) + v1 * (fyp - fc)) * A.uhy +
                      wf * (fc * rc.c2 - tc * rc.c3));
      else
        adv = -half * ((u1 * (fc + fxp) - u0 * (fxm + fc)) * A.uhx + (v1 * (fc + fyp) - v0 * (fym + fc)) * A.uhy +
                       rc.c2 * wf * (tc + fc));
      rr = A.ap * pc + A.ac * fc + A.tau * adv + A.tk * (lx2 * A.uxx + ly2 * A.uyy);
      if constexpr (REV)   // the start-up step reads theta^0 for its diffusion too
        if (A.tk0 != T(0))
          rr += A.tk0 * (fma_(T(-2), fc, fxp + fxm) * A.uxx + fma_(T(-2), fc, fyp + fym) * A.uyy);
    } else {
      const T x = fma_(u1, fc + fxp, -(u0 * (fxm + fc))), y = fma_(v1, fc + fyp, -(v0 * (fym + fc)));
      pxy = as_sweep ? fma_(x, A.uhx, y * A.uhy) : fma_(y, A.uhy, x * A.uhx);
      lap = as_sweep ? fma_(lx2, A.uxx, ly2 * A.uyy) : fma_(ly2, A.uyy, lx2 * A.uxx);
      rr = fma_(A.ap, pc, A.ac * fc);
      rs = tc + fc;
      wr = rc.c2 * wf;
      asm volatile("" : "+v"(pxy), "+v"(lap));
    }
    asm volatile("" : "+v"(rr));
    tc = fc;
    wf = wn;
    rb = rc;
    rc = rn;
    return as_sweep ? (double)(T)e : e;
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
        if (act) st_nt(A.out + (size_t)level(kx + q) * nxy, oc, xo[q]);
    } else {
#pragma unroll
      for (int q = 0; q < B; ++q)
        if (act && kx + q >= ks && kx + q < ke) st_nt(A.out + (size_t)level(kx + q) * nxy, oc, xo[q]);
    }
    return whole && any;
  };
  auto shift = [&]() {
#pragma unroll
    for (int q = 0; q < D; ++q) ring[q] = ring[q + B];
  };

  // positions k0 .. k1: position s closes s - 1, whose elimination value enters
  // the ring; the first one closes nothing (its own value is dropped), the last
  // one (k1) only closes
#pragma unroll
  for (int s = 0; s < NSTAGE - 1; ++s) issue(s);
  constexpr int N = (NSTAGE - 2) * L::slots;   // copies still under way when a position's are done
  int st = 0;
  wait_barrier<N>();
  advance(k0, 0, NSTAGE - 1);
  e = 0.0;
  int stored = 0;   // (wave-uniform) the B stores of the block before are younger than the position's copies
  int q = k0;
  for (; q < k1; q += B) {
    // the rows of the block after this one into the scalar cache, all at once: a
    // miss per level would be waited for with that level's LDS reads.  186^3 FP32
    // 45.2 to 42.3 us, 576^3 FP32 897 to 882; FP64 on wider tiles does not need it
    // (256^3 142 us without, 145 with)
    if constexpr (sizeof(T) == 4 || TX == 1) touch_rows(A.row, q + B + 2, nz + kStreamRowPad - 1);
#pragma unroll
    for (int s = 0; s < B; ++s) {
      const int last = st;
      st = st == NSTAGE - 1 ? 0 : st + 1;
      if (s < NSTAGE - 1 && stored) wait_barrier<N + B>();
      else wait_barrier<N>();
      ring[D + s] = advance(q + s + 1, st * L::stage, last);   // (last: the slot read before this barrier)
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
template <typename T, bool REV, int TX, int TY, int CH, int Q>
hipError_t launch_depth(int depth, dim3 grid, const StreamArgs<T>& a, hipStream_t s) {
  if constexpr (Q < kStreamDepths) {
    constexpr int D = kStreamDepth[Q];
    if (depth != Q) return launch_depth<T, REV, TX, TY, CH, Q + 1>(depth, grid, a, s);
    if constexpr (stream_fits(D, TX * TY)) {
      hipLaunchKernelGGL((stream_kernel<T, D, REV, TX, TY, CH>), grid, dim3(64, TX * TY), 0, s, a);
      return hipGetLastError();
    }
  }
  return hipErrorInvalidValue;
}

template <typename T, bool REV, int CH>
hipError_t launch_shape(int shape, int depth, dim3 grid, const StreamArgs<T>& a, hipStream_t s) {
  static_assert(kStreamShapes == 4, "one case per shape");
  switch (shape) {
    case 0: return launch_depth<T, REV, kStreamShape[0].segs, kStreamShape[0].rows, CH, 0>(depth, grid, a, s);
    case 1: return launch_depth<T, REV, kStreamShape[1].segs, kStreamShape[1].rows, CH, 0>(depth, grid, a, s);
    case 2: return launch_depth<T, REV, kStreamShape[2].segs, kStreamShape[2].rows, CH, 0>(depth, grid, a, s);
    case 3: return launch_depth<T, REV, kStreamShape[3].segs, kStreamShape[3].rows, CH, 0>(depth, grid, a, s);
  }
  return hipErrorInvalidValue;
}

// 16-byte copies where every row of every field starts on 16 bytes, else
// 4-byte ones (four times the copies: at 1024 x 1024 x 512 up to 5% more
// time, at 256^3 18% more in FP64 and 12% in FP32; on small grids, bound by a
// level's chain, up to 60%).
template <typename T, bool REV>
hipError_t launch_stream(int shape, int depth, dim3 grid, const StreamArgs<T>& a, hipStream_t s) {
  const uintptr_t p = (uintptr_t)a.f | (uintptr_t)a.p | (uintptr_t)a.u | (uintptr_t)a.v | (uintptr_t)a.w;
  if (((uintptr_t)a.nx * sizeof(T)) % 16 == 0 && p % 16 == 0) return launch_shape<T, REV, 16>(shape, depth, grid, a, s);
  return launch_shape<T, REV, 4>(shape, depth, grid, a, s);
}

}  // namespace stream
}  // namespace mr
