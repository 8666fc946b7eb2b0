// The three passes of one batch of pair Poisson solves (Eq. applyVX):
//
//   A  plane pass, one (pair, z) at a time: rho = conj(psi_j) phi_k on the xy
//      plane, forward FFT along x then y, written to the pair's work volume.
//   B  pencil pass, one (pair, y, x-tile): forward FFT along z, times K at the
//      digit-reversed positions (the table carries -scale/Omega), inverse FFT
//      along z, written back in place.
//   C  plane pass, one (target k, z), looping over the batch's orbitals j in
//      ascending order: inverse FFT along y then x, times psi_j, added to the
//      k-th output plane held in registers.
//
// The first stage that follows a global read and the last before a global
// write move the data themselves, so a pass holds it in LDS only in between.
// The bodies here are __host__ __device__ templates over a barrier policy;
// the host runs them one thread at a time to check plans and tables, the
// device kernels for any grid (vx_gen.hip) many at a time.
#pragma once

#include "fft.hpp"

namespace fx {

struct PassGeom {
  int nx, ny, nz;
  int sx;  // LDS row stride (elements) of an xy plane: nx, or nx + 1 when nx is even
  AxisArg ax, ay, az;
  int hx, hy, hz;  // folded kernel table dims n/2 + 1
  FastDiv dnx, dny, dhx;
};

// LDS elements an xy plane needs (twiddles come after).
FX_HD int plane_lds_elems(const PassGeom& g) { return g.ny * g.sx; }

// The rows and columns of an xy plane as transforms, and where they lie in LDS.
FX_HD Lines plane_rows(const PassGeom& g) { return {g.ny, g.ny, g.dny}; }
FX_HD Lines plane_cols(const PassGeom& g) { return {g.nx, g.nx, g.dnx}; }
template <typename T>
FX_HD Span<T> lds_rows(cpx<T>* s, const PassGeom& g) { return {s, 1, g.sx}; }
template <typename T>
FX_HD Span<T> lds_cols(cpx<T>* s, const PassGeom& g) { return {s, g.sx, 1}; }
template <typename T>
FX_HD Span<T> mem_cols(const cpx<T>* p, const PassGeom& g) { return {const_cast<cpx<T>*>(p), g.nx, 1}; }

// Pass A body.  psi_j / phi_k / out point at plane z (contiguous nx*ny).  The
// caller puts a barrier between two calls on the same LDS.
template <typename T, class Sync>
FX_HD void pass_a_body(const cpx<T>* psi_j, const cpx<T>* phi_k, cpx<T>* out, cpx<T>* s, const cpx<T>* twx,
                       const cpx<T>* twy, const PassGeom& g, int tid, int nthr, Sync sync) {
  const int nxy = g.nx * g.ny;
  // four elements at a time, so that their eight loads are in flight together
  constexpr int U = 4;
  for (int e0 = tid; e0 < nxy; e0 += U * nthr) {
    cpx<T> a[U], b[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int e = e0 + u * nthr < nxy ? e0 + u * nthr : e0;
      a[u] = psi_j[e];
      b[u] = phi_k[e];
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int e = e0 + u * nthr;
      // conj(a) b with the fused multiply-adds written out (left to the
      // compiler, the copies of this line are fused differently); which of the
      // two products of the real part is rounded first is part of the result's
      // bits: a.x b.x on planes of up to 512 points, a.y b.y on larger ones
      const bool xf = nxy <= 512;
      const T p = xf ? a[u].x : a[u].y, q = xf ? b[u].x : b[u].y;
      const T v = xf ? a[u].y : a[u].x, w = xf ? b[u].y : b[u].x;
      if (e < nxy)
        s[e + fdiv(e, g.dnx) * (g.sx - g.nx)] =
            cpx<T>{fmadd(v, w, p * q), fmadd(a[u].x, b[u].y, -(a[u].y * b[u].x))};
    }
  }
  sync();
  const Span<T> rows = lds_rows(s, g), cols = lds_cols(s, g);
  for (int st = 0; st < g.ax.nst; ++st) {
    run_stage<true, false, false, T>(rows, rows, g.ax.st[st], plane_rows(g), twx, tid, nthr);
    sync();
  }
  for (int st = 0; st + 1 < g.ay.nst; ++st) {
    run_stage<true, false, false, T>(cols, cols, g.ay.st[st], plane_cols(g), twy, tid, nthr);
    sync();
  }
  run_stage<true, false, true, T>(cols, mem_cols(out, g), g.ay.st[g.ay.nst - 1], plane_cols(g), twy, tid, nthr);
}

// Factor of the z-convolution: K at (digit-reversed) z position pos and x
// column x0 + f of the tile, from the K slice of this y held in LDS.
template <typename T>
struct KSlice {
  const T* kl;       // hz x hx values at the tile's folded y
  const int* foldx;  // folded frequency of each x position
  const int* foldz;
  int x0, hx;
  FX_HD T operator()(int pos, int f) const { return kl[foldz[pos] * hx + foldx[x0 + f]]; }
};

// Pass B body for the x-tile [x0, x0 + xt) of the xz plane at (digit-reversed)
// y of one pair volume; s holds nz * xt values.  Columns at or past the edge
// are left out.  The first stage takes its twiddles from twz0: the device
// kernel fills its LDS tables (twz, kf) just before and the barrier after the
// first stage publishes them, so the reads of the volume need not wait.
template <typename T, class Sync>
FX_HD void pass_b_body(cpx<T>* vol, int y, int x0, const Lines& tile, cpx<T>* s, const cpx<T>* twz0, const cpx<T>* twz,
                       KSlice<T> kf, const PassGeom& g, int tid, int nthr, Sync sync) {
  const Span<T> mem{vol + (size_t)y * g.nx + x0, g.nx * g.ny, 1}, lds{s, tile.count, 1};
  const Lines ln{tile.count, tile.count < g.nx - x0 ? tile.count : g.nx - x0, tile.dcount};
  const int last = g.az.nst - 1;
  if (last == 0) {
    sync();
    run_mid<true, T>(mem, mem, g.az.st[0], ln, kf, tid, nthr);
    return;
  }
  run_stage<true, true, false, T>(mem, lds, g.az.st[0], ln, twz0, tid, nthr);
  sync();
  for (int st = 1; st < last; ++st) {
    run_stage<true, false, false, T>(lds, lds, g.az.st[st], ln, twz, tid, nthr);
    sync();
  }
  run_mid<false, T>(lds, lds, g.az.st[last], ln, kf, tid, nthr);
  sync();
  for (int st = last - 1; st > 0; --st) {
    run_stage<false, false, false, T>(lds, lds, g.az.st[st], ln, twz, tid, nthr);
    sync();
  }
  run_stage<false, false, true, T>(lds, mem, g.az.st[0], ln, twz, tid, nthr);
}

// Pass C transform part: plane (digit-reversed spectrum in y and x) up to the
// last inverse x stage (stage 0), whose inputs are left in s.  early() runs
// once the plane has been read.
template <typename T, int RMAX = 12, class Sync, class Early>
FX_HD void pass_c_fft(const cpx<T>* plane, cpx<T>* s, const cpx<T>* twx, const cpx<T>* twy, const PassGeom& g, int tid,
                      int nthr, Sync sync, Early early) {
  const Span<T> rows = lds_rows(s, g), cols = lds_cols(s, g);
  run_stage<false, true, false, T, RMAX>(mem_cols(plane, g), cols, g.ay.st[g.ay.nst - 1], plane_cols(g), twy, tid, nthr);
  sync();
  early();
  for (int st = g.ay.nst - 2; st >= 0; --st) {
    run_stage<false, false, false, T, RMAX>(cols, cols, g.ay.st[st], plane_cols(g), twy, tid, nthr);
    sync();
  }
  for (int st = g.ax.nst - 1; st > 0; --st) {
    run_stage<false, false, false, T, RMAX>(rows, rows, g.ax.st[st], plane_rows(g), twx, tid, nthr);
    sync();
  }
}

// Dft<R, 1> with the twiddles of the composite radices 9 and 12 as written-out
// fused multiply-adds: where the outputs stay in registers the compiler orders
// (and so fuses) two of their products differently from the same butterfly
// between two LDS accesses, and the results' last bits with them.
template <int R, typename T>
FX_HD void dft_inv_pinned(cpx<T>* x) {
  if constexpr (R != 9 && R != 12) {
    Dft<R, 1, T>::run(x);
  } else {
    constexpr int A = first_factor<R>::value, B = R / A;
    cpx<T> t[B][A];
#pragma unroll
    for (int m2 = 0; m2 < B; ++m2) {
#pragma unroll
      for (int m1 = 0; m1 < A; ++m1) t[m2][m1] = x[B * m1 + m2];
      Dft<A, 1, T>::run(t[m2]);
#pragma unroll
      for (int k1 = 0; k1 < A; ++k1) {
        const int e = m2 * k1 % R;
        if (e % 3 == 0 && R == 12) {  // a multiple of a quarter turn
          t[m2][k1] = twc<R, T>(t[m2][k1], e);
        } else if (e != 0) {
          const ct::cs w = ct::turn(e, R);
          const T c = (T)w.c, sn = (T)w.s;
          const cpx<T> a = t[m2][k1];
          t[m2][k1] = cpx<T>{fmadd(a.x, c, -(a.y * sn)),
                             w.c > 0 ? fmadd(a.y, c, a.x * sn) : fmadd(a.x, sn, a.y * c)};
        }
      }
    }
#pragma unroll
    for (int k1 = 0; k1 < A; ++k1) {
      cpx<T> b[B];
#pragma unroll
      for (int m2 = 0; m2 < B; ++m2) b[m2] = t[m2][k1];
      Dft<B, 1, T>::run(b);
#pragma unroll
      for (int k2 = 0; k2 < B; ++k2) x[k1 + A * k2] = b[k2];
    }
  }
}

// The last inverse x stage of the rows in s (radix R = that of stage 0), one
// butterfly: thread-consecutive b take consecutive positions i2 of a row, so
// its values lie at plane positions pos + m * span.  Returns them in x.
template <int R, typename T>
FX_HD void row_last_stage(const cpx<T>* s, const cpx<T>* twx, const PassGeom& g, int b, cpx<T> (&x)[R]) {
  const AxisStage& st = g.ax.st[0];
  const int r = fdiv(b, st.dspan), i2 = b - r * st.span;
  const cpx<T>* p = s + (r * g.sx + i2);
#pragma unroll
  for (int m = 0; m < R; ++m) x[m] = p[m * st.span];
  if (st.span > 1) {
#pragma unroll
    for (int k = 1; k < R; ++k) x[k] = cmulc(x[k], twx[i2 * k]);
  }
  dft_inv_pinned<R, T>(x);
}
FX_HD int row_last_pos(const PassGeom& g, int b) {
  const AxisStage& st = g.ax.st[0];
  const int r = fdiv(b, st.dspan);
  return r * g.nx + (b - r * st.span);
}

}  // namespace fx
