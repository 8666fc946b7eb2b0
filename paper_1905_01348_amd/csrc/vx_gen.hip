// V_X pair passes for any supported grid: the bodies of vx_passes.hpp with
// run-time plans, persistent like the compile-time-specialised kernels of the
// cubic workload edges (vx_ct.hip) and with the same batch interface (packed
// diagonal batches, conjugated second role, sum groups, several trajectories).
//
// What bounds them is instruction issue and the latency across the stage
// barriers, not HBM, so: every index is a high multiply by a constant of the
// grid (FastDiv) instead of a division, the stage next to a global read or
// write moves the data itself (no LDS round trip, one barrier fewer), the last
// inverse x stage accumulates from its registers, and thread counts are taken
// so that the butterflies of the stages fill them.
#include <algorithm>

#include "fft.hpp"
#include "item_map.hpp"
#include "pair_order.hpp"
#include "vx.hpp"
#include "vx_passes.hpp"

namespace fx {

constexpr int kGenAThreads = 512;
// most threads of a generic z-pass workgroup (its launch bound)
constexpr int kPencilThreads = 512;

// ---- pass A ------------------------------------------------------------------
template <typename T>
__global__ void __launch_bounds__(kGenAThreads, 4) k_gen_a(const cpx<T>* __restrict__ psi, int64_t ld_psi,
                                                          const cpx<T>* __restrict__ phi, int64_t ld_phi,
                                                          cpx<T>* __restrict__ work, int j0, int nj, int k0, int tri,
                                                          int npairs, PassGeom g, const cpx<T>* __restrict__ twx_g,
                                                          const cpx<T>* __restrict__ twy_g, int split, TrajSegs segs) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  cpx<T>* s = reinterpret_cast<cpx<T>*>(smem_raw);
  cpx<T>* twx = s + plane_lds_elems(g);
  cpx<T>* twy = twx + g.nx;
  const int tid = threadIdx.x, nthr = blockDim.x;
  for (int i = tid; i < g.nx; i += nthr) twx[i] = twx_g[i];
  for (int i = tid; i < g.ny; i += nthr) twy[i] = twy_g[i];
  const int nxy = g.nx * g.ny;
  const size_t nr = (size_t)nxy * g.nz;
  const ItemMap im = item_map(g.nz, npairs, split & 3, gridDim.x, blockIdx.x);
  for (int li = im.first; li < im.total; li += im.step) {
    int p, z;
    im.at(li, &p, &z);
    p = unit_plane(p, npairs, nj, tri, (split >> 2) & 1);
    int jj, kk;
    pair_of(p, nj, tri, &jj, &kk);
    const cpx<T>* a = seg_psi<T>(segs, psi, k0 + kk) + (int64_t)(j0 + jj) * ld_psi + (size_t)z * nxy;
    const cpx<T>* b = phi + (int64_t)(k0 + kk) * ld_phi + (size_t)z * nxy;
    pass_a_body<T>(a, b, work + p * nr + (size_t)z * nxy, s, twx, twy, g, tid, nthr, DeviceSync{});
    __syncthreads();
  }
}

// ---- pass B: one (pair, y, x-tile) per workgroup -------------------------------
template <typename T>
__global__ void __launch_bounds__(kPencilThreads) k_gen_b(cpx<T>* __restrict__ work, Lines tile, int ntx, PassGeom g,
                                                          const cpx<T>* __restrict__ twz_g,
                                                          const T* __restrict__ kfold, const int* __restrict__ foldx_g,
                                                          const int* __restrict__ foldy_g,
                                                          const int* __restrict__ foldz_g) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  cpx<T>* s = reinterpret_cast<cpx<T>*>(smem_raw);
  cpx<T>* twz = s + g.nz * tile.count;
  T* kl = reinterpret_cast<T*>(twz + g.nz);
  int* fxl = reinterpret_cast<int*>(kl + g.hz * g.hx);
  int* fzl = fxl + g.nx;
  const int tid = threadIdx.x, nthr = blockDim.x;
  const int tx = blockIdx.x % ntx;
  const int rest = blockIdx.x / ntx;
  const int y = rest % g.ny;
  const int p = rest / g.ny;
  const int fy = foldy_g[y];
  for (int i = tid; i < g.nz; i += nthr) {
    twz[i] = twz_g[i];
    fzl[i] = foldz_g[i];
  }
  for (int i = tid; i < g.nx; i += nthr) fxl[i] = foldx_g[i];
  for (int i = tid; i < g.hz * g.hx; i += nthr) {
    const int fz = fdiv(i, g.dhx);
    kl[i] = kfold[((size_t)fz * g.hy + fy) * g.hx + (i - fz * g.hx)];
  }
  const int x0 = tx * tile.count;
  const KSlice<T> kf{kl, fxl, fzl, x0, g.hx};
  pass_b_body<T>(work + (size_t)p * g.nx * g.ny * g.nz, y, x0, tile, s, twz_g, twz, kf, g, tid, nthr, DeviceSync{});
}

// ---- pass C ------------------------------------------------------------------
// One item = (target tt of the batch, sum group gr, plane z).  Role 0: targets
// k0 + kk, terms psi_{j0+jj} v_{jk}; role 1: targets j0 + jj, terms psi_{k0+kk}
// conj(v_{jk}); on a diagonal batch role 0 takes jj <= kk, role 1 kk > jj; role
// 2: both (see k_pass_c_ct).  R: radix of the last inverse x stage, IT its
// butterflies per thread; their R IT sums per thread stay in registers over
// the batch's terms.  Two LDS planes, alternating by term, where dbl is set
// (they then take at most 40 KB): a term's first stage need not wait for the
// previous term's last reads.
constexpr int kGenCThreads = 768;  // launch bound: 170 registers a thread

template <typename T, typename A, int R, int IT, int RMAX>
__global__ void __launch_bounds__(kGenCThreads, (sizeof(T) == 4 && R * IT <= 8 ? 4 : 3))
    k_gen_c(const cpx<T>* __restrict__ mult, int64_t ld_mult, const cpx<T>* __restrict__ work, int nj, int nk, int tri,
            int role, int j0, int k0, int units, cpx<A>* acc, int64_t ld_acc, int first_in, void* out, int64_t ld_out,
            int out_c64, int last_in, PassGeom g, const cpx<T>* __restrict__ twx_g, const cpx<T>* __restrict__ twy_g,
            int split, TrajSegs segs, int jsplit, int64_t gstride, int dbl) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  cpx<T>* s = reinterpret_cast<cpx<T>*>(smem_raw);
  const int plane = plane_lds_elems(g);
  cpx<T>* twx = s + (dbl ? 2 : 1) * plane;
  cpx<T>* twy = twx + g.nx;
  const int tid = threadIdx.x, nthr = blockDim.x;
  for (int i = tid; i < g.nx; i += nthr) twx[i] = twx_g[i];
  for (int i = tid; i < g.ny; i += nthr) twy[i] = twy_g[i];
  __syncthreads();
  const int nxy = g.nx * g.ny;
  const size_t nr = (size_t)nxy * g.nz;
  const int total = g.ny * g.ax.st[0].nb, span = g.ax.st[0].span;
  // the orbital values once the transform's registers are free: FP32 with sums
  // of up to 8 values then keeps four waves per SIMD (64^3: 1200 -> 850 us)
  constexpr bool kLate = sizeof(T) == 8 || R * IT > 4;
  int pos[IT];
#pragma unroll
  for (int it = 0; it < IT; ++it) pos[it] = row_last_pos(g, tid + it * nthr);
  const auto owns = [&](int it) __attribute__((always_inline)) { return tid + it * nthr < total; };
  const ItemMap im = item_map(g.nz, units, split, gridDim.x, blockIdx.x);
  int par = 0;
  for (int li = im.first; li < im.total; li += im.step) {
    int u, z;
    im.at(li, &u, &z);
    int tt = u / jsplit;
    const int gr = u - tt * jsplit;
    bool cj0 = role == 1, cj1 = role != 0;
    if (role == 2 && !tri) {
      cj0 = cj1 = tt >= nk;
      if (cj0) tt -= nk;
    }
    const int t = (cj1 ? j0 : k0) + tt;
    const int first = first_in && !cj0, last = last_in && (cj1 || role == 0);
    cpx<A>* accg = acc + gr * gstride + t * ld_acc + (size_t)z * nxy;
    cpx<A> a[IT][R];
#pragma unroll
    for (int it = 0; it < IT; ++it)
#pragma unroll
      for (int m = 0; m < R; ++m) {
        a[it][m] = cpx<A>{0, 0};
        if (!first && owns(it)) a[it][m] = accg[pos[it] + m * span];
      }
    for (int cj = cj0; cj <= (int)cj1; ++cj) {
      const A sgn = cj ? (A)-1 : (A)1;
      // terms lo, lo + jsplit, ... < hi: those whose orbital m0 + l is gr mod jsplit
      const int m0 = cj ? k0 : j0;
      int lo = cj ? (tri ? tt + 1 : 0) : 0;
      const int hi = cj ? nk : (tri ? tt + 1 : nj);
      const int r = (m0 + lo) % jsplit;
      lo += gr >= r ? gr - r : gr - r + jsplit;
      for (int l = lo; l < hi; l += jsplit) {
        const cpx<T>* pm = seg_psi<T>(segs, mult, t) + (int64_t)(m0 + l) * ld_mult + (size_t)z * nxy;
        const int pl = cj ? plane_of(tt, l, nj, tri) : plane_of(l, tt, nj, tri);
        cpx<T>* sl = s + (dbl && par ? plane : 0);
        cpx<T> vp[IT][R];
        const auto orbital = [&]() __attribute__((always_inline)) {
#pragma unroll
          for (int it = 0; it < IT; ++it)
#pragma unroll
            for (int m = 0; m < R; ++m)
              if (owns(it)) vp[it][m] = pm[pos[it] + m * span];
        };
        pass_c_fft<T, RMAX>(work + (size_t)pl * nr + (size_t)z * nxy, sl, twx, twy, g, tid, nthr, DeviceSync{},
                      [&]() __attribute__((always_inline)) {
                        if (!kLate) orbital();
                      });
        cpx<T> x[IT][R];
#pragma unroll
        for (int it = 0; it < IT; ++it)
          if (owns(it)) row_last_stage<R, T>(sl, twx, g, tid + it * nthr, x[it]);
        if (kLate) orbital();
#pragma unroll
        for (int it = 0; it < IT; ++it)
#pragma unroll
          for (int m = 0; m < R; ++m)
            if (owns(it))
              a[it][m] = cfma(a[it][m], cpx<A>{(A)vp[it][m].x, (A)vp[it][m].y},
                              cpx<A>{(A)x[it][m].x, sgn * (A)x[it][m].y});
        if (dbl)
          par ^= 1;
        else
          __syncthreads();
      }
    }
#pragma unroll
    for (int it = 0; it < IT; ++it)
#pragma unroll
      for (int m = 0; m < R; ++m) {
        if (!owns(it)) continue;
        const int e = pos[it] + m * span;
        if (!last) {
          accg[e] = a[it][m];
        } else {
          const size_t off = t * ld_out + (size_t)z * nxy + e;
          if (out_c64)
            reinterpret_cast<cpx<float>*>(out)[off] = cpx<float>{(float)a[it][m].x, (float)a[it][m].y};
          else
            reinterpret_cast<cpx<double>*>(out)[off] = cpx<double>{(double)a[it][m].x, (double)a[it][m].y};
        }
      }
  }
}

constexpr int kFlatThreads = 512;  // launch bound of the form with a thread per plane value

// Item li: plane z of output column t = (first column of its block) + tt, sum
// group gr, roles cj0 .. cj1.
struct GenItem {
  int t, tt, gr, z;
  bool cj0, cj1;
};
__device__ inline GenItem gen_item(const ItemMap& im, int li, int jsplit, int role, int tri, int nk, int j0, int k0) {
  GenItem m;
  int u;
  im.at(li, &u, &m.z);
  m.tt = u / jsplit;
  m.gr = u - m.tt * jsplit;
  m.cj0 = role == 1;
  m.cj1 = role != 0;
  if (role == 2 && !tri) {
    m.cj0 = m.cj1 = m.tt >= nk;
    if (m.cj0) m.tt -= nk;
  }
  m.t = (m.cj1 ? j0 : k0) + m.tt;
  return m;
}
// Its terms in role cj: lo, lo + jsplit, ... < hi, those whose orbital m0 + l is gr mod jsplit.
__device__ inline void gen_terms(const GenItem& m, int cj, int jsplit, int tri, int nj, int nk, int m0, int* lo, int* hi) {
  const int l = cj ? (tri ? m.tt + 1 : 0) : 0;
  *hi = cj ? nk : (tri ? m.tt + 1 : nj);
  const int r = (m0 + l) % jsplit;
  *lo = l + (m.gr >= r ? m.gr - r : m.gr - r + jsplit);
}
template <typename A>
__device__ inline void gen_store(void* out, size_t off, int out_c64, cpx<A> v) {
  if (out_c64)
    reinterpret_cast<cpx<float>*>(out)[off] = cpx<float>{(float)v.x, (float)v.y};
  else
    reinterpret_cast<cpx<double>*>(out)[off] = cpx<double>{(double)v.x, (double)v.y};
}

// The same for an x axis of one stage (edges up to 12) where a butterfly per
// thread leaves most of a wave idle: the last stage, the loads and the sums would
// fall to one thread per row (8 x 8 plane: 8 threads of 64), with the 12 values of
// a radix-12 row in FP64 spilling 400 bytes.  Here a thread owns EPT plane values
// from the load of the work plane to the sums, which it takes from LDS after the
// last stage, and loads the next term's values while the current one is
// transformed (gen_c_flat has the rule).
template <typename T, typename A, int EPT>
__global__ void __launch_bounds__(kFlatThreads, 4)
    k_gen_c_flat(const cpx<T>* __restrict__ mult, int64_t ld_mult, const cpx<T>* __restrict__ work, int nj, int nk,
                 int tri, int role, int j0, int k0, int units, cpx<A>* acc, int64_t ld_acc, int first_in, void* out,
                 int64_t ld_out, int out_c64, int last_in, PassGeom g, const cpx<T>* __restrict__ twx_g,
                 const cpx<T>* __restrict__ twy_g, int split, TrajSegs segs, int jsplit, int64_t gstride) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  cpx<T>* s = reinterpret_cast<cpx<T>*>(smem_raw);  // two planes, alternating by term
  const int plane = plane_lds_elems(g);
  cpx<T>* twx = s + 2 * plane;
  cpx<T>* twy = twx + g.nx;
  const int tid = threadIdx.x, nthr = blockDim.x;
  for (int i = tid; i < g.nx; i += nthr) twx[i] = twx_g[i];
  for (int i = tid; i < g.ny; i += nthr) twy[i] = twy_g[i];
  __syncthreads();
  const int nxy = g.nx * g.ny;
  const size_t nr = (size_t)nxy * g.nz;
  int at[EPT];  // where the thread's values lie in LDS
#pragma unroll
  for (int i = 0; i < EPT; ++i) {
    const int e = tid + i * nthr;
    at[i] = e + fdiv(e, g.dnx) * (g.sx - g.nx);
  }
  const auto owns = [&](int i) __attribute__((always_inline)) { return tid + i * nthr < nxy; };
  const ItemMap im = item_map(g.nz, units, split, gridDim.x, blockIdx.x);
  int par = 0;
  for (int li = im.first; li < im.total; li += im.step) {
    const GenItem m = gen_item(im, li, jsplit, role, tri, nk, j0, k0);
    const int first = first_in && !m.cj0, last = last_in && (m.cj1 || role == 0);
    cpx<A>* accg = acc + m.gr * gstride + m.t * ld_acc + (size_t)m.z * nxy;
    cpx<A> a[EPT];
#pragma unroll
    for (int i = 0; i < EPT; ++i) {
      a[i] = cpx<A>{0, 0};
      if (!first && owns(i)) a[i] = accg[tid + i * nthr];
    }
    for (int cj = m.cj0; cj <= (int)m.cj1; ++cj) {
      const A sgn = cj ? (A)-1 : (A)1;
      const int m0 = cj ? k0 : j0;
      int lo, hi;
      gen_terms(m, cj, jsplit, tri, nj, nk, m0, &lo, &hi);
      cpx<T> next[EPT];
      const auto ahead = [&](int l) __attribute__((always_inline)) {
        const int pl = cj ? plane_of(m.tt, l, nj, tri) : plane_of(l, m.tt, nj, tri);
        const cpx<T>* p = work + (size_t)pl * nr + (size_t)m.z * nxy;
#pragma unroll
        for (int i = 0; i < EPT; ++i)
          if (owns(i)) next[i] = g_load<true>(p + tid + i * nthr);
      };
      if (lo < hi) ahead(lo);
      for (int l = lo; l < hi; l += jsplit) {
        cpx<T>* sl = s + (par ? plane : 0);
#pragma unroll
        for (int i = 0; i < EPT; ++i)
          if (owns(i)) sl[at[i]] = next[i];
        __syncthreads();
        const cpx<T>* pm = seg_psi<T>(segs, mult, m.t) + (int64_t)(m0 + l) * ld_mult + (size_t)m.z * nxy;
        cpx<T> vp[EPT];
#pragma unroll
        for (int i = 0; i < EPT; ++i)
          if (owns(i)) vp[i] = pm[tid + i * nthr];
        if (l + jsplit < hi) ahead(l + jsplit);
        const Span<T> rows = lds_rows(sl, g), cols = lds_cols(sl, g);
        for (int st = g.ay.nst - 1; st >= 0; --st) {
          run_stage<false, false, false, T>(cols, cols, g.ay.st[st], plane_cols(g), twy, tid, nthr);
          __syncthreads();
        }
        for (int st = g.ax.nst - 1; st >= 0; --st) {
          run_stage<false, false, false, T>(rows, rows, g.ax.st[st], plane_rows(g), twx, tid, nthr);
          __syncthreads();
        }
#pragma unroll
        for (int i = 0; i < EPT; ++i)
          if (owns(i)) {
            const cpx<T> v = sl[at[i]];
            a[i] = cfma(a[i], cpx<A>{(A)vp[i].x, (A)vp[i].y}, cpx<A>{(A)v.x, sgn * (A)v.y});
          }
        par ^= 1;
      }
    }
#pragma unroll
    for (int i = 0; i < EPT; ++i) {
      const int e = tid + i * nthr;
      if (!owns(i)) continue;
      if (!last)
        accg[e] = a[i];
      else
        gen_store(out, m.t * ld_out + (size_t)m.z * nxy + e, out_c64, a[i]);
    }
  }
}

// ---- host side ------------------------------------------------------------------
static int round64(int v) { return (v + 63) / 64 * 64; }

// Persistent grid: resident workgroups, a multiple of the XCD count.
template <typename K>
static fx_status gen_grid(fx_ctx* ctx, K kernel, int nthr, size_t lds, int64_t items, int* grid) {
  FX_TRY(allow_dynamic_lds(reinterpret_cast<const void*>(kernel), lds));
  int per_cu = 0;
  FX_HIP(hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, reinterpret_cast<const void*>(kernel), nthr, lds));
  int g = (int)std::max<int64_t>(1, std::min<int64_t>(items, (int64_t)std::max(per_cu, 1) * std::max(ctx->n_cu, 1)));
  if (g >= kXcds) g -= g % kXcds;
  *grid = g;
  return FX_OK;
}

// Threads of a plane-forward workgroup.  A stage of `total` butterflies of
// radix R takes ceil(total / t) rounds of about R + 4 LDS accesses and 4 more
// for its barrier; the workgroups that LDS and registers (at most `waves` per
// CU) let a CU hold overlap each other up to 20 waves, past which the CU's
// issue rate is shared.  On ten planes from 9 x 8 to 96 x 96 in both precisions
// the count with the smallest time per plane so estimated measured within 5%
// of the best of 64, 128, ... 512, which itself is 1.2 to 5 times faster than
// the worst.
static int plane_threads(const PassGeom& g, size_t lds, int waves) {
  int best = 64;
  double best_cost = 0.0;
  for (int t = 64; t <= kGenAThreads; t += 64) {
    double c = (g.nx * g.ny + t - 1) / t + 4.0;
    const auto add = [&](const AxisArg& a, int lines) {
      for (int st = 0; st < a.nst; ++st) c += ((lines * a.st[st].nb + t - 1) / t) * (a.st[st].R + 4.0) + 4.0;
    };
    add(g.ax, g.ny);
    add(g.ay, g.nx);
    const int wg = std::max(1, std::min({(int)((160 << 10) / lds), waves * 64 / t, 32}));
    c *= std::max(1.0, wg * t / 64 / 20.0) / wg;
    if (t == 64 || c < best_cost) {
      best = t;
      best_cost = c;
    }
  }
  return best;
}

template <typename T>
fx_status gen_pass_a(fx_ctx* ctx, hipStream_t st, const PassGeom& g, const GridTables* tb, const CtBatch<T>& b) {
  const size_t lds = ((size_t)plane_lds_elems(g) + g.nx + g.ny) * sizeof(cpx<T>);
  const int nthr = plane_threads(g, lds, sizeof(T) == 4 ? 28 : 16);
  const auto kern = k_gen_a<T>;
  int grid = 0;
  FX_TRY(gen_grid(ctx, kern, nthr, lds, (int64_t)b.npairs * g.nz, &grid));
  hipLaunchKernelGGL(kern, dim3(grid), dim3(nthr), lds, st, b.psi, b.ld_psi, b.phi, b.ld_phi, b.work, b.j0, b.nj, b.k0,
                     b.tri, b.npairs, g, (const cpx<T>*)tb->tw[0], (const cpx<T>*)tb->tw[1],
                     item_split(g.nz, b.npairs, b.zsplit & 1, grid) | (b.zsplit & 4), b.segs);
  FX_LAUNCH_CHECK();
  return FX_OK;
}

fx_status gen_check_tile(const PassGeom& g, int xtile, int most_threads) {
  const int points = g.nz * std::min(g.nx, xtile > 0 ? xtile : 32);
  if (round64((points + 17) / 18) > (most_threads > 0 ? std::min(most_threads, 256) : 256))
    FX_FAIL(FX_ERR_UNSUPPORTED, "pencil tile of %d points is too large", points);
  return FX_OK;
}

template <typename T>
fx_status gen_pass_b(fx_ctx* ctx, hipStream_t st, const PassGeom& g, const GridTables* tb, const CtBatch<T>& b,
                     int xtile, int most_threads) {
  // Columns of a tile: whole x rows (the longest runs in memory) where the
  // tile stays within 56 KB of LDS, so that two workgroups share a CU; else the
  // largest divisor of the edge within 50 KB (a ragged last tile wastes its
  // share of the threads).  48 x 64 x 72 FP64: 32 columns 1566 us, whole rows
  // 1327; 81 x 54 x 64 FP32: 32 1770, 81 1159; 96 x 96 x 64 FP64: whole rows
  // (96 KB) 2127, 48 1909, 32 1807.
  int xt = g.nx;
  if (xtile > 0) {
    xt = std::min(g.nx, xtile);
  } else if ((size_t)g.nz * g.nx * sizeof(cpx<T>) > 56 * 1024) {
    do {
      do --xt;
      while (g.nx % xt != 0);
    } while (xt > 1 && (size_t)g.nz * xt * sizeof(cpx<T>) > 50 * 1024);
  }
  const int ntx = (g.nx + xt - 1) / xt;
  int widest = 0;
  for (int i = 0; i < g.az.nst; ++i) widest = std::max(widest, xt * g.az.st[i].nb);
  const int cap = most_threads > 0 ? std::min(most_threads, kPencilThreads) : kPencilThreads;
  const int nthr = std::min(cap, round64(widest));
  const size_t lds = ((size_t)g.nz * xt + g.nz) * sizeof(cpx<T>) + (size_t)g.hz * g.hx * sizeof(T) +
                     (size_t)(g.nx + g.nz) * sizeof(int);
  const auto kern = k_gen_b<T>;
  FX_TRY(allow_dynamic_lds(reinterpret_cast<const void*>(kern), lds));
  const Lines tile{xt, xt, fast_div(xt)};
  hipLaunchKernelGGL(kern, dim3((unsigned)((int64_t)b.npairs * g.ny * ntx)), dim3(nthr), lds, st, b.work, tile, ntx, g,
                     (const cpx<T>*)tb->tw[2], (const T*)tb->kfold, tb->fold[0], tb->fold[1], tb->fold[2]);
  FX_LAUNCH_CHECK();
  return FX_OK;
}

template <typename T, typename A, int R, int IT, int RMAX>
static fx_status gen_c_launch(fx_ctx* ctx, hipStream_t st, const PassGeom& g, const GridTables* tb, const CtBatch<T>& b,
                              const CtAcc<A>& c, int role) {
  const size_t plane = (size_t)plane_lds_elems(g) * sizeof(cpx<T>), tw = (size_t)(g.nx + g.ny) * sizeof(cpx<T>);
  const int dbl = 2 * plane <= 40 * 1024;
  const size_t lds = (dbl ? 2 : 1) * plane + tw;
  const int total = g.ny * g.ax.st[0].nb;
  const int nthr = round64((total + IT - 1) / IT);
  const int units = (role == 0 ? b.nk : role == 1 ? b.nj : b.tri ? b.nk : b.nk + b.nj) * b.jsplit;
  const auto kern = k_gen_c<T, A, R, IT, RMAX>;
  int grid = 0;
  FX_TRY(gen_grid(ctx, kern, nthr, lds, (int64_t)units * g.nz, &grid));
  hipLaunchKernelGGL(kern, dim3(grid), dim3(nthr), lds, st, role ? b.phi : b.psi, role ? b.ld_phi : b.ld_psi,
                     (const cpx<T>*)b.work, b.nj, b.nk, b.tri, role, b.j0, b.k0, units,
                     c.acc, c.ld_acc, c.first, c.out, c.ld_out, c.out_c64, c.last, g, (const cpx<T>*)tb->tw[0],
                     (const cpx<T>*)tb->tw[1], item_split(g.nz, units, (b.zsplit >> 1) & 1, grid),
                     role ? TrajSegs{} : b.segs, b.jsplit, c.gstride, dbl);
  FX_LAUNCH_CHECK();
  return FX_OK;
}

template <typename T, typename A, int EPT>
static fx_status gen_c_flat_launch(fx_ctx* ctx, hipStream_t st, const PassGeom& g, const GridTables* tb,
                                   const CtBatch<T>& b, const CtAcc<A>& c, int role) {
  const size_t lds = (2 * (size_t)plane_lds_elems(g) + g.nx + g.ny) * sizeof(cpx<T>);
  const int nthr = round64((g.nx * g.ny + EPT - 1) / EPT);
  const int units = (role == 0 ? b.nk : role == 1 ? b.nj : b.tri ? b.nk : b.nk + b.nj) * b.jsplit;
  const auto kern = k_gen_c_flat<T, A, EPT>;
  int grid = 0;
  FX_TRY(gen_grid(ctx, kern, nthr, lds, (int64_t)units * g.nz, &grid));
  hipLaunchKernelGGL(kern, dim3(grid), dim3(nthr), lds, st, role ? b.phi : b.psi, role ? b.ld_phi : b.ld_psi,
                     (const cpx<T>*)b.work, b.nj, b.nk, b.tri, role, b.j0, b.k0, units, c.acc, c.ld_acc, c.first, c.out,
                     c.ld_out, c.out_c64, c.last, g, (const cpx<T>*)tb->tw[0], (const cpx<T>*)tb->tw[1],
                     item_split(g.nz, units, (b.zsplit >> 1) & 1, grid), role ? TrajSegs{} : b.segs, b.jsplit,
                     c.gstride);
  FX_LAUNCH_CHECK();
  return FX_OK;
}

// The form with a thread per plane value: planes of at most 12 rows and 108 values
// (us per apply, 16 orbitals on 64 targets, a butterfly per thread against this
// one: 8 x 8 x 96 FP64 283 / 219, FP32 with FP64 sums 192 / 161; 12 x 9 x 9 98 / 57
// and 53 / 46; past 108 values FP32 loses, 8 x 16 x 16 63 / 66, 9 x 18 x 18 84 /
// 98, and so does FP64, 8 x 24 x 24 131 / 145), and radix-12 rows in FP64 whatever
// their number (12^3, 32 on 8: 54 / 36; 12 x 36 x 36 598 / 462; 12 x 96 x 4 215 /
// 168; FP32 keeps the butterfly: 282 / 349, 114 / 123).
static bool gen_c_flat(const PassGeom& g, size_t real_bytes) {
  return g.ax.nst == 1 && ((g.ny <= 12 && g.nx * g.ny <= 108) || (real_bytes == 8 && g.nx == 12));
}

// IT > 1 only where the first x radix of a tuned schedule leaves more
// butterflies than one per thread of the launch bound.
template <typename T, typename A, int R, int ITM>
static fx_status gen_c_radix(fx_ctx* ctx, hipStream_t st, const PassGeom& g, const GridTables* tb, const CtBatch<T>& b,
                             const CtAcc<A>& c, int role) {
  // radices of the stages that run through LDS; up to 8, the kernel without
  // the wider ones (in FP64 those cost it 100 to 300 bytes of spills)
  int widest = 2;
  for (int i = 1; i < g.ax.nst; ++i) widest = std::max(widest, g.ax.st[i].R);
  for (int i = 0; i < g.ay.nst; ++i) widest = std::max(widest, g.ay.st[i].R);
  if (g.ny * g.ax.st[0].nb <= kGenCThreads)
    return widest <= 8 ? gen_c_launch<T, A, R, 1, 8>(ctx, st, g, tb, b, c, role)
                       : gen_c_launch<T, A, R, 1, 12>(ctx, st, g, tb, b, c, role);
  if constexpr (ITM > 1) return gen_c_launch<T, A, R, ITM, 12>(ctx, st, g, tb, b, c, role);
  FX_FAIL(FX_ERR_UNSUPPORTED, "no plane-inverse kernel for %d butterflies of radix %d", g.ny * g.ax.st[0].nb, R);
}

template <typename T, typename A>
fx_status gen_pass_c(fx_ctx* ctx, hipStream_t st, const PassGeom& g, const GridTables* tb, const CtBatch<T>& b,
                     const CtAcc<A>& c, int role) {
  if (gen_c_flat(g, sizeof(T))) {
    if constexpr (sizeof(T) == 8) {  // up to 12 x 96 values
      if (g.nx * g.ny > 2 * kFlatThreads) return gen_c_flat_launch<T, A, 3>(ctx, st, g, tb, b, c, role);
      if (g.nx * g.ny > kFlatThreads) return gen_c_flat_launch<T, A, 2>(ctx, st, g, tb, b, c, role);
    }
    return gen_c_flat_launch<T, A, 1>(ctx, st, g, tb, b, c, role);
  }
  switch (g.ax.st[0].R) {
    // most butterflies of a stage: 96 rows x 96 / R (radix 9: x 9), so
    // ITM = ceil(9216 / (768 R))
    case 2: return gen_c_radix<T, A, 2, 6>(ctx, st, g, tb, b, c, role);
    case 3: return gen_c_radix<T, A, 3, 4>(ctx, st, g, tb, b, c, role);
    case 4: return gen_c_radix<T, A, 4, 3>(ctx, st, g, tb, b, c, role);
    case 6: return gen_c_radix<T, A, 6, 2>(ctx, st, g, tb, b, c, role);
    case 8: return gen_c_radix<T, A, 8, 2>(ctx, st, g, tb, b, c, role);
    case 9: return gen_c_radix<T, A, 9, 2>(ctx, st, g, tb, b, c, role);
    case 12: return gen_c_radix<T, A, 12, 1>(ctx, st, g, tb, b, c, role);
    default: FX_FAIL(FX_ERR_UNSUPPORTED, "no plane-inverse kernel for radix %d", g.ax.st[0].R);
  }
}

template fx_status gen_pass_a<float>(fx_ctx*, hipStream_t, const PassGeom&, const GridTables*, const CtBatch<float>&);
template fx_status gen_pass_a<double>(fx_ctx*, hipStream_t, const PassGeom&, const GridTables*, const CtBatch<double>&);
template fx_status gen_pass_b<float>(fx_ctx*, hipStream_t, const PassGeom&, const GridTables*, const CtBatch<float>&,
                                     int, int);
template fx_status gen_pass_b<double>(fx_ctx*, hipStream_t, const PassGeom&, const GridTables*, const CtBatch<double>&,
                                      int, int);
template fx_status gen_pass_c<float, double>(fx_ctx*, hipStream_t, const PassGeom&, const GridTables*,
                                             const CtBatch<float>&, const CtAcc<double>&, int);
template fx_status gen_pass_c<float, float>(fx_ctx*, hipStream_t, const PassGeom&, const GridTables*,
                                            const CtBatch<float>&, const CtAcc<float>&, int);
template fx_status gen_pass_c<double, double>(fx_ctx*, hipStream_t, const PassGeom&, const GridTables*,
                                              const CtBatch<double>&, const CtAcc<double>&, int);

}  // namespace fx
