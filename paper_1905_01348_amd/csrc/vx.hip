// fx_apply_vx: V_X applied to a block of targets by batched pair Poisson
// solves (Eq. applyVX; the Fock-application loop of Sec. 3.2 on one GPU's
// band-index share).  Pairs are processed in batches of nk targets x nj
// orbitals; every batch runs the three passes of vx_passes.hpp.
#include <algorithm>
#include <cmath>
#include <cstdlib>
#include <set>

#include "common.hpp"
#include "vx.hpp"
#include "vx_passes.hpp"

namespace fx {

// Columns of one or two blocks converted to another precision: columns c < n0 of
// in0 to out0, the others from in1 to out1.  Bound by memory, or by the launch
// where a call's orbitals and targets are few: one launch for both, a block of
// rows per workgroup with four values in flight per thread and no division
// (us: 27 + 11 columns at 32 x 36 x 24, complex128 to FP32, 5.7 + 4.7 -> 6.1; 1024
// at 96^3 to FP64 4390 -> 3810, 5.7 TB/s).
template <typename TI, typename TO>
__global__ void __launch_bounds__(256) k_convert(const cpx<TI>* __restrict__ in0, int64_t ld0, cpx<TO>* __restrict__ out0,
                                                 int n0, const cpx<TI>* __restrict__ in1, int64_t ld1,
                                                 cpx<TO>* __restrict__ out1, int64_t ld_out, int64_t nr, int ncols) {
  const int64_t r0 = blockIdx.x * (int64_t)1024 + threadIdx.x;
  for (int c = blockIdx.y; c < ncols; c += gridDim.y) {
    const cpx<TI>* in = c < n0 ? in0 + c * ld0 : in1 + (c - n0) * ld1;
    cpx<TO>* out = c < n0 ? out0 + c * ld_out : out1 + (c - n0) * ld_out;
    cpx<TI> v[4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (r0 + 256 * i < nr) v[i] = in[r0 + 256 * i];
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (r0 + 256 * i < nr) out[r0 + 256 * i] = cpx<TO>{(TO)v[i].x, (TO)v[i].y};
  }
}

// E_X: half the sum over the columns of Re <psi_k, w_k>, in FP64 with a fixed
// order.  Bound by the read of psi and w.  A column is cut into ex_parts(nr)
// spans, a workgroup each, and one workgroup adds all the spans' sums: with a
// workgroup per column and one thread adding the columns, 16 columns at 24^3
// took 16.6 + 4.5 us, 85 at 48^3 207 + 9 us; now 4.7 + 4.0 and 53 + 8 us (4.2
// TB/s).  The scratch region of the allocation-free form gets one span per column
// where it cannot hold more.
static int ex_parts(int64_t nr) { return (int)std::min<int64_t>(64, std::max<int64_t>(1, nr / 2048)); }

__device__ inline double block_sum256(double v) {
  __shared__ double red[256];
  red[threadIdx.x] = v;
  __syncthreads();
  for (int h = 128; h > 0; h >>= 1) {
    if ((int)threadIdx.x < h) red[threadIdx.x] += red[threadIdx.x + h];
    __syncthreads();
  }
  return red[0];
}

template <typename TP, typename TW>
__global__ void __launch_bounds__(256) k_dot_cols(const cpx<TP>* __restrict__ psi, int64_t ldp,
                                                  const cpx<TW>* __restrict__ w, int64_t ldw, int64_t nr, int parts,
                                                  double* __restrict__ partial) {
  const int64_t k = blockIdx.x / parts;
  const int s = blockIdx.x - (int)k * parts;
  const int64_t hi = nr * (s + 1) / parts;
  double acc = 0.0;
#pragma unroll 4
  for (int64_t r = nr * s / parts + threadIdx.x; r < hi; r += 256) {
    const cpx<TP> a = psi[k * ldp + r];
    const cpx<TW> b = w[k * ldw + r];
    acc += (double)a.x * (double)b.x + (double)a.y * (double)b.y;
  }
  acc = block_sum256(acc);
  if (threadIdx.x == 0) partial[blockIdx.x] = acc;
}

__global__ void __launch_bounds__(256) k_half_sum(const double* __restrict__ partial, int n, double* __restrict__ out) {
  double s = 0.0;
#pragma unroll 4
  for (int i = threadIdx.x; i < n; i += 256) s += partial[i];
  s = block_sum256(s);
  if (threadIdx.x == 0) *out = 0.5 * s;
}

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------
static AxisArg to_arg(const AxisPlan& p) {
  AxisArg a{};
  a.n = p.n;
  a.nst = p.nst;
  for (int i = 0, L = p.n; i < p.nst; ++i) {
    const int R = p.R[i];
    a.st[i] = AxisStage{R, L, L / R, p.n / L, p.n / R, fast_div(L / R)};
    L /= R;
  }
  return a;
}

PassGeom make_geom(const fx_cell* cell, const PlanSet* plans = nullptr) {
  PassGeom g;
  g.nx = cell->n[0];
  g.ny = cell->n[1];
  g.nz = cell->n[2];
  // odd row stride (in elements) so consecutive rows start in different banks
  g.sx = g.nx % 2 ? g.nx : g.nx + 1;
  PlanSet ps;
  if (plans)
    ps = *plans;
  else
    default_plans(cell, &ps);
  g.ax = to_arg(ps.ax[0]);
  g.ay = to_arg(ps.ax[1]);
  g.az = to_arg(ps.ax[2]);
  g.hx = g.nx / 2 + 1;
  g.hy = g.ny / 2 + 1;
  g.hz = g.nz / 2 + 1;
  g.dnx = fast_div(g.nx);
  g.dny = fast_div(g.ny);
  g.dhx = fast_div(g.hx);
  return g;
}

static size_t work_cap_bytes(fx_ctx* ctx) {
  // pair work volume per batch: 8 GiB (a few percent of HBM) keeps launches
  // long and partial-sum traffic low; capped at a quarter of the budget
  size_t cap = (size_t)8192 << 20;
  if (const char* e = getenv("FX_WORK_MB")) cap = (size_t)atol(e) << 20;
  if (cap > ctx->budget / 4) cap = ctx->budget / 4;
  return cap;
}

// z-pass form of the specialised kernels: the persistent kernel with whole x
// rows is the automatic choice at 96^3, where it measured faster (3.12 vs
// 3.38 ms per launch of 1170 pairs), whole x rows at 72^3 (15.6 vs 16.6 ms
// for 432 orbitals x 8 targets); elsewhere the autotuner decides.
static int ct_b_variant(const VxArgs& a) {
  if (a.b_var >= 1 && a.b_var <= 4) return a.b_var;
  return a.cell->n[0] == 96 ? 4 : (a.cell->n[0] == 72 ? 3 : 1);
}

// Plane-inverse threads of the specialised kernels: the larger count (fewer
// accumulators per thread, more waves per CU) is the automatic choice at
// 96^3, where it measured faster (3.34 vs 3.39 ms per launch of 1170 pairs),
// and at 72^3 (15.1 vs 15.6 ms for 432 orbitals x 8 targets, with whole-row
// z tiles), in its wave-level form (5): 2.75 vs 2.79 ms per launch at 96^3
// in FP32, 2.38 vs 2.50 in FP64.  Elsewhere the autotuner decides.
static int ct_c_variant(const VxArgs& a) {
  if (a.c_var >= 1 && a.c_var <= 5) return a.c_var;
  return a.cell->n[0] == 96 || a.cell->n[0] == 72 ? 5 : 1;
}

// Sum groups of the plane-inverse pass: the terms of orbital j
// go to partial sum j mod S of their target, each in ascending j, and the S
// partial sums are added in order of the group at the end.  With few targets
// the pass has few items (targets x planes); S times as many balance the
// CUs.  The grouping depends on the orbital index only, so a column's result
// is the same whatever the batch size and whichever targets share a launch.
// Automatic: as many groups as give the eight targets of a request the
// workgroups that are resident at once (256 CUs of 12 waves, also in FP32, where
// some kernels hold 16: the precisions then group alike; a plane has about
// ny nx / R butterflies in its last stage, R the first x radix), with at least
// four terms each.  The count of targets must not enter, since served requests
// are merged; the phi == psi form keeps one running sum (its partial sums then
// need no memory beyond `out`), as does the allocation-free form.  Nor must
// memory enter: where it is short, blocks shrink or the groups run one after
// the other (run_batches).
// 27 orbitals x 11 targets at 32 x 36 x 24: one sum leaves 264 items of 27
// terms one after the other, 182 us, four groups 71 and 7 to add them; at 64^3
// two groups gain nothing and their partial sums cost the other passes 130 of
// 2440 us.  Two groups also where eight targets are up to a quarter more than
// the resident workgroups, so that the second round is a short one (planes of 5 or
// 6 waves on 72 planes, of 7 or more on 36; 96 orbitals
// at 48 x 64 x 72 in FP64, 512 resident: 8 targets 4423 -> 4133 us, 16 8107 ->
// 7739, 32 14630 -> 14920; at half more, 96 x 96 x 48, the partial sums cost as
// much as they save).
static int ct_jsplit(const VxArgs& a, const PassGeom& g, bool square) {
  if (a.no_alloc || a.add) return 1;
  if (a.c_split == 1 || a.c_split == 2 || a.c_split == 4 || a.c_split == 8) return a.c_split;
  if (square) return 1;
  // planes of up to 108 points: eight to eleven terms take no longer than the
  // launch that adds two groups (8^3, 8 orbitals on 8 targets 24 / 27 us; 12
  // orbitals 30 / 27)
  if (a.n_psi < 12 && g.nx * g.ny <= 108) return 1;
  const int waves = (g.ny * g.ax.st[0].nb + 63) / 64;
  const int64_t most = std::min<int64_t>(a.n_psi / 4, 256 * std::max(1, 12 / waves) / (8 * g.nz));
  int s = 1;
  while (s < 8 && 2 * s <= most) s *= 2;
  // a second round of workgroups that is nearly empty for eight targets
  const int64_t items = 8 * (int64_t)g.nz, resident = 256 * std::max(1, 12 / waves);
  if (s == 1 && items > resident && 4 * items <= 5 * resident && a.n_psi >= 32) s = 2;
  return s;
}

// Whether the phi == psi form is halved off the workload edges (on them it
// always is).  FP32 transforms with FP64 sums keep every ordered pair's own
// solve: the solve of (k, j) is the conjugate of that of (j, k) only to FP32
// rounding, which the FP64 sums would show.  And the halved passes run one
// after the other over the same planes, so there must be planes enough for the
// resident workgroups (see ct_jsplit) twice over.
static bool gen_halved(const VxArgs& a, const PassGeom& g) {
  const int waves = (g.ny * g.ax.st[0].nb + 63) / 64;
  return a.prec != FX_PREC_FP32_ACC64 && (int64_t)a.n_psi * g.nz >= 2 * 256 * std::max(1, 12 / waves);
}

// out[t] = sum over the groups g = 0, 1, ... of acc[g][t] (targets t0 ..
// t0 + nt - 1), converted to the output type.
template <typename A>
__global__ void k_combine_groups(const cpx<A>* __restrict__ acc, int64_t gstride, int64_t ld_acc, int jsplit, int t0,
                                 int nt, int64_t nr, void* __restrict__ out, int64_t ld_out, int out_c64) {
  const int64_t total = (int64_t)nt * nr;
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < total; i += (int64_t)gridDim.x * blockDim.x) {
    const int64_t t = t0 + i / nr, e = i % nr;
    cpx<A> v = acc[t * ld_acc + e];
    for (int g = 1; g < jsplit; ++g) v = cadd(v, acc[g * gstride + t * ld_acc + e]);
    if (out_c64)
      reinterpret_cast<cpx<float>*>(out)[t * ld_out + e] = cpx<float>{(float)v.x, (float)v.y};
    else
      reinterpret_cast<cpx<double>*>(out)[t * ld_out + e] = cpx<double>{(double)v.x, (double)v.y};
  }
}

template <typename A>
static fx_status combine_groups(fx_ctx* ctx, hipStream_t st, const cpx<A>* acc, int64_t gstride, int64_t ld_acc,
                                int jsplit, int t0, int nt, int64_t nr, void* out, int64_t ld_out, int out_c64) {
  const int64_t total = (int64_t)nt * nr;
  const int blocks = (int)std::max<int64_t>(1, std::min<int64_t>((total + 255) / 256, 8 * std::max(ctx->n_cu, 1)));
  hipLaunchKernelGGL((k_combine_groups<A>), dim3(blocks), dim3(256), 0, st, acc, gstride, ld_acc, jsplit, t0, nt, nr,
                     out, ld_out, out_c64);
  FX_LAUNCH_CHECK();
  return FX_OK;
}

// Work order of the persistent plane passes: how the XCDs share their items (bit
// 0 the plane-forward pass, bit 1 the plane-inverse pass; set: each XCD takes a
// contiguous range of z planes of every unit, clear: a contiguous range of units
// at every z), and with bit 2 the plane-forward pass walks its pairs in blocks of
// 4 orbitals x 16 targets (unit_plane).  With the z split the plane-forward pass
// reads each orbital and target plane once per XCD instead of once per XCD per
// chunk of pairs (3.05 -> 2.82 ms per launch of 1170 pairs at 96^3); the
// plane-inverse pass is slower with it (2.76 against 2.71) and keeps the unit
// split.  Only the order changes, never a result.
static int ct_zsplit() {
  const char* e = getenv("FX_VX_ZSPLIT");
  return e ? atoi(e) : 5;
}

// The three passes of a batch, by the kernels chosen for the grid.
template <typename T, typename A>
struct PairPasses {
  fx_ctx* ctx;
  hipStream_t st;
  bool ct;
  PassGeom g;
  const GridTables* tb;
  int xtile, nthr_b;
  fx_status a(const CtBatch<T>& b) const {
    return ct ? ct_pass_a<T>(ctx, st, g.nx, b) : gen_pass_a<T>(ctx, st, g, tb, b);
  }
  fx_status b(const CtBatch<T>& b) const {
    return ct ? ct_pass_b<T>(ctx, st, g.nx, b) : gen_pass_b<T>(ctx, st, g, tb, b, xtile, nthr_b);
  }
  fx_status c(const CtBatch<T>& b, const CtAcc<A>& c, int role) const {
    return ct ? ct_pass_c<T, A>(ctx, st, g.nx, b, c, role) : gen_pass_c<T, A>(ctx, st, g, tb, b, c, role);
  }
};

// A batch of the call `a`: its launch configuration and tables beside what it covers.
template <typename T>
static CtBatch<T> make_batch(const VxArgs& a, const GridTables* tb, const cpx<T>* psi, int64_t ld_psi, const cpx<T>* phi,
                             int64_t ld_phi, cpx<T>* work, int j0, int nj, int k0, int nk, int npairs, int tri,
                             int jsplit) {
  CtBatch<T> b{psi, ld_psi, phi, ld_phi, work, j0, nj, k0, nk, npairs, reinterpret_cast<const cpx<T>*>(tb->tw[0]),
               reinterpret_cast<const T*>(tb->kfold), tb->fold[0], tri, a.a_pipe > 0 ? 1 : 0, ct_b_variant(a),
               ct_c_variant(a), (a.a_var >= 1 && a.a_var <= 3) ? a.a_var : 0, a.nt_hint != 0 ? 1 : 0, ct_zsplit()};
  b.segs = a.segs;
  b.jsplit = jsplit;
  return b;
}

// Halved apply for phi == psi (all N targets): each unordered pair {j, k} is
// solved once, as (min, max), since v_kj = conj(v_jk) for a real, even kernel.
// Orbitals are cut into blocks of B; block pairs (J <= K) run in ascending
// order of J, then K.  For each, pass C takes both roles: role 0 adds the pairs
// to the targets of block K, role 1 (conjugated) to those of block J.  Every
// output column then receives its terms in ascending j, each term computed
// from the ordered pair (min(j,k), max(j,k)), so the result does not depend
// on B.  Diagonal block pairs hold only the B(B+1)/2 pairs j <= k.
template <typename T, typename A>
static fx_status run_halved(fx_ctx* ctx, Workspace* ws, const VxArgs& a, const PairPasses<T, A>& pass,
                            const GridTables* tb, const cpx<T>* psi, int64_t ld_psi, int64_t pairs_cap, hipStream_t st,
                            VxStats* stats) {
  const int64_t nr = (int64_t)a.cell->n[0] * a.cell->n[1] * a.cell->n[2];
  const size_t pair_bytes = (size_t)nr * sizeof(cpx<T>);
  const int N = a.n_psi;
  int B = (int)std::min<int64_t>(N, std::max<int64_t>(1, (int64_t)std::sqrt((double)pairs_cap)));
  if (a.force_nj > 0) B = std::min(B, a.force_nj);
  const int nblk = (N + B - 1) / B;
  B = (N + nblk - 1) / nblk;
  void* work = nullptr;
  FX_TRY(ws_get(ctx, ws, "vx_work", (size_t)B * B * pair_bytes, &work));
  const bool out_c64 = a.out_dtype == FX_C64;
  const bool out_is_A = (sizeof(A) == 8) == !out_c64;
  const int jsplit = ct_jsplit(a, pass.g, true);
  // partial sums live between the block pairs
  cpx<A>* acc = nullptr;
  int64_t ld_acc = 0, gstride = 0;
  if (out_is_A && jsplit == 1) {
    acc = reinterpret_cast<cpx<A>*>(a.out);
    ld_acc = a.ld_out;
  } else {
    void* p = nullptr;
    FX_TRY(ws_get(ctx, ws, "vx_acc", (size_t)jsplit * N * nr * sizeof(cpx<A>), &p));
    acc = reinterpret_cast<cpx<A>*>(p);
    ld_acc = nr;
    gstride = (int64_t)N * nr;
  }
  const double sz = sizeof(cpx<T>), asz = sizeof(cpx<A>), osz = out_c64 ? 8.0 : 16.0;
  int64_t launches = 0, solves = 0;
  for (int J = 0; J < nblk; ++J) {
    const int j0 = J * B, jb = std::min(B, N - j0);
    for (int K = J; K < nblk; ++K) {
      const int k0 = K * B, kb = std::min(B, N - k0);
      const int tri = J == K;
      const int npairs = tri ? jb * (jb + 1) / 2 : jb * kb;
      const CtBatch<T> cb = make_batch<T>(a, tb, psi, ld_psi, psi, ld_psi, reinterpret_cast<cpx<T>*>(work), j0, jb, k0,
                                          kb, npairs, tri, jsplit);
      const double vol = (double)npairs * nr * sz;
      int slot;
      FX_TRY(prof_begin(ctx, st, FX_K_VX_PLANE_FWD, 2.0 * vol, &slot));
      FX_TRY(pass.a(cb));
      FX_TRY(prof_end(ctx, st, slot));
      FX_TRY(prof_begin(ctx, st, FX_K_VX_PENCIL_Z, 2.0 * vol, &slot));
      FX_TRY(pass.b(cb));
      FX_TRY(prof_end(ctx, st, slot));
      // both roles: the first contribution to the targets of block K is J = 0,
      // the last to those of block J is K = nblk - 1
      {
        const int first = J == 0, last = K == nblk - 1 && jsplit == 1;
        CtAcc<A> ca{acc, ld_acc, first, a.out, a.ld_out, out_c64 ? 1 : 0, last, gstride};
        // a diagonal batch's targets take both roles in one sum
        const double in = (double)((tri ? 0 : jb) + (first ? 0 : kb)) * asz;
        const double outb = (double)jb * (last ? osz : asz) + (tri ? 0.0 : kb * asz);
        const double planes = tri ? 2.0 * npairs - jb : 2.0 * npairs;
        FX_TRY(prof_begin(ctx, st, FX_K_VX_PLANE_INV, 2.0 * planes * nr * sz + (in + outb) * nr * jsplit, &slot));
        FX_TRY(pass.c(cb, ca, 2));
        FX_TRY(prof_end(ctx, st, slot));
      }
      launches += 3;
      solves += npairs;
    }
  }
  if (jsplit > 1) {
    int slot;
    FX_TRY(prof_begin(ctx, st, FX_K_REDUCE, (double)N * nr * (jsplit * asz + osz), &slot));
    FX_TRY(combine_groups<A>(ctx, st, acc, gstride, ld_acc, jsplit, 0, N, nr, a.out, a.ld_out, out_c64 ? 1 : 0));
    FX_TRY(prof_end(ctx, st, slot));
    ++launches;
  }
  if (stats) {
    stats->nk = B;
    stats->nj = B;
    stats->launches = launches;
    stats->solves = solves;
  }
  return FX_OK;
}

// total += x over one target, written to `out` (the total's own column, or the result's)
template <typename A>
__global__ void __launch_bounds__(256) k_add_group(const cpx<A>* total, const cpx<A>* x, int64_t nr, void* out,
                                                   int out_c64) {
  for (int64_t e = blockIdx.x * (int64_t)256 + threadIdx.x; e < nr; e += (int64_t)gridDim.x * 256) {
    const cpx<A> v = cadd(total[e], x[e]);
    if (out_c64)
      reinterpret_cast<cpx<float>*>(out)[e] = cpx<float>{(float)v.x, (float)v.y};
    else
      reinterpret_cast<cpx<double>*>(out)[e] = cpx<double>{(double)v.x, (double)v.y};
  }
}

// Sum groups where a quarter of the budget cannot hold a pair volume and the S
// partial sums of one target: target by target and group by group, a pair at a
// time, each group's running sum added to the total when it is complete.  The
// same additions in the same order as with all groups at once, so the same
// bits, in one partial sum of memory (two where `out` is of another type).
template <typename T, typename A>
static fx_status run_groups_in_turn(fx_ctx* ctx, Workspace* ws, const VxArgs& a, const PairPasses<T, A>& pass,
                                    const GridTables* tb, const cpx<T>* psi, int64_t ld_psi, const cpx<T>* phi,
                                    int64_t ld_phi, int jsplit, hipStream_t st, VxStats* stats) {
  const int64_t nr = (int64_t)a.cell->n[0] * a.cell->n[1] * a.cell->n[2];
  const int out_c64 = a.out_dtype == FX_C64, A_c64 = sizeof(A) == 4;
  const int nsum = out_c64 == A_c64 ? 1 : 2;
  const double sz = sizeof(cpx<T>), asz = sizeof(cpx<A>);
  void* work = nullptr;
  FX_TRY(ws_get(ctx, ws, "vx_work", (size_t)nr * (nsum * sizeof(cpx<A>) + sizeof(cpx<T>)), &work));
  cpx<A>* const x = reinterpret_cast<cpx<A>*>(work);
  cpx<T>* const vol = reinterpret_cast<cpx<T>*>(x + nsum * nr);
  const int blocks = (int)std::max<int64_t>(1, std::min<int64_t>((nr + 255) / 256, 8 * std::max(ctx->n_cu, 1)));
  const int groups = std::min(jsplit, a.n_psi);  // (any others are empty)
  int64_t launches = 0;
  for (int k = 0; k < a.n_phi; ++k) {
    char* const col = (char*)a.out + (size_t)k * a.ld_out * dtype_size(a.out_dtype);
    cpx<A>* const total = nsum == 1 ? reinterpret_cast<cpx<A>*>(col) : x + nr;
    for (int g = 0; g < groups; ++g) {
      // (the passes find a target's sum by its column k)
      CtAcc<A> ca{(g ? x : total) - k * nr, nr, 1, a.out, a.ld_out, out_c64, 0};
      int slot;
      for (int j = g; j < a.n_psi; j += jsplit, ca.first = 0) {
        const CtBatch<T> cb = make_batch<T>(a, tb, psi, ld_psi, phi, ld_phi, vol, j, 1, k, 1, 1, 0, 1);
        FX_TRY(prof_begin(ctx, st, FX_K_VX_PLANE_FWD, 2.0 * nr * sz, &slot));
        FX_TRY(pass.a(cb));
        FX_TRY(prof_end(ctx, st, slot));
        FX_TRY(prof_begin(ctx, st, FX_K_VX_PENCIL_Z, 2.0 * nr * sz, &slot));
        FX_TRY(pass.b(cb));
        FX_TRY(prof_end(ctx, st, slot));
        FX_TRY(prof_begin(ctx, st, FX_K_VX_PLANE_INV, nr * (2.0 * sz + (ca.first ? asz : 2.0 * asz)), &slot));
        FX_TRY(pass.c(cb, ca, 0));
        FX_TRY(prof_end(ctx, st, slot));
        launches += 3;
      }
      if (g == 0) continue;
      const bool end = g == groups - 1;
      FX_TRY(prof_begin(ctx, st, FX_K_REDUCE, 3.0 * nr * asz, &slot));
      hipLaunchKernelGGL((k_add_group<A>), dim3(blocks), dim3(256), 0, st, (const cpx<A>*)total, (const cpx<A>*)x, nr,
                         end ? (void*)col : (void*)total, end ? out_c64 : A_c64);
      FX_LAUNCH_CHECK();
      FX_TRY(prof_end(ctx, st, slot));
      ++launches;
    }
  }
  if (stats) {
    stats->nk = 1;
    stats->nj = 1;
    stats->launches = launches;
    stats->solves = (int64_t)a.n_psi * a.n_phi;
  }
  return FX_OK;
}

template <typename T, typename A>
static fx_status run_batches(fx_ctx* ctx, Workspace* ws, const VxArgs& a, const GridTables* tb,
                             const cpx<T>* psi, int64_t ld_psi, const cpx<T>* phi, int64_t ld_phi, hipStream_t st,
                             VxStats* stats) {
  const PassGeom g = make_geom(a.cell, a.plans_set ? &a.plans : nullptr);
  const int64_t nr = (int64_t)g.nx * g.ny * g.nz;
  const size_t pair_bytes = (size_t)nr * sizeof(cpx<T>);
  size_t cap = a.work_cap ? std::min(a.work_cap, ctx->budget / 4) : work_cap_bytes(ctx);
  const int64_t pairs_cap = (int64_t)std::max<size_t>(1, cap / pair_bytes);
  // cubic grids of the workload edges run the compile-time-specialised
  // kernels unless the generic family or another radix schedule is asked for
  bool use_ct = ct_supported(a.cell) && a.kernels != 2;
  if (use_ct && a.plans_set) {
    PlanSet d;
    default_plans(a.cell, &d);
    use_ct = same_plans(a.plans, d);
  }
  if (a.kernels == 1 && !use_ct)
    FX_FAIL(FX_ERR_UNSUPPORTED, "no specialised kernels for grid %dx%dx%d with this radix schedule", g.nx, g.ny,
            g.nz);
  if (a.segs.n > 0 && (!use_ct || psi == phi))
    FX_FAIL(FX_ERR_UNSUPPORTED, "multi-trajectory launches need the specialised kernels and phi != psi");
  if (!use_ct) FX_TRY(gen_check_tile(g, a.xtile, a.nthr_b));
  const PairPasses<T, A> pass{ctx, st, use_ct, g, tb, a.xtile, a.nthr_b};
  const bool square = psi == phi && ld_psi == ld_phi && a.n_psi == a.n_phi;
  if (square && a.halve != 0 && (use_ct || a.halve > 0 || (!a.served && gen_halved(a, g))))
    return run_halved<T, A>(ctx, ws, a, pass, tb, psi, ld_psi, pairs_cap, st, stats);
  const bool out_c64 = a.out_dtype == FX_C64;
  const bool out_is_A = (sizeof(A) == 8) == !out_c64;
  const int jsplit = a.n_psi > 1 ? ct_jsplit(a, g, false) : 1;
  // (a multiple of 256, so that the pair volumes behind them are aligned)
  const size_t sum_bytes = jsplit > 1 ? ((size_t)jsplit * nr * sizeof(cpx<A>) + 255) & ~(size_t)255 : 0;
  // Batch shape: up to 16 orbitals per batch first (the plane-inverse pass
  // reads and writes its partial sums once per batch), then as many targets
  // as fit, balanced over the target blocks, then any leftover capacity
  // back to orbitals.  With sum groups a target also takes sum_bytes of `room`.
  int nj = 0, nk = 0;
  const auto shape = [&](size_t room) {  // (0: without the groups' sums)
    nj = (int)std::min<int64_t>(a.n_psi, std::min<int64_t>(16, pairs_cap));
    if (room) nj = (int)std::min<int64_t>(nj, (int64_t)((room - sum_bytes) / pair_bytes));
    if (a.force_nj > 0) nj = std::min(nj, a.force_nj);
    int64_t nk_max = std::max<int64_t>(1, pairs_cap / nj);
    if (room) nk_max = std::min<int64_t>(nk_max, (int64_t)(room / (nj * pair_bytes + sum_bytes)));
    const int64_t kblocks = (a.n_phi + nk_max - 1) / nk_max;
    nk = (int)((a.n_phi + kblocks - 1) / kblocks);
    if (a.force_nj > 0) return;
    int64_t pairs = pairs_cap;
    if (room) pairs = std::min<int64_t>(pairs, (int64_t)((room - nk * sum_bytes) / pair_bytes));
    nj = (int)std::min<int64_t>(a.n_psi, std::max<int64_t>(nj, pairs / nk));
  };
  // Groups in rounds (ROUNDS of k_pass_c_ct) where all orbitals fit one batch and
  // the targets' planes alone occupy half the resident workgroups (24^3: 32
  // targets, where both forms take the same time).
  int rounds = 0;
  if (jsplit > 1 && use_ct && ct_rounds_supported(g.nx, ct_c_variant(a)) && a.n_psi >= jsplit) {
    shape(0);
    const int waves = (g.ny * g.ax.st[0].nb + 63) / 64;
    rounds = nj == a.n_psi && 2 * (int64_t)nk * g.nz >= 256 * std::max(1, 12 / waves);
  }
  // The groups' partial sums of a block of targets lie before its pair volumes in
  // the work buffer.  Where the two do not fit a quarter of the budget, what is
  // left of it, or under capture the buffer that is there, a block has fewer
  // targets or orbitals, never fewer groups: the bits do not depend on memory.
  // (With less left than the pairs alone need the request stands, and is
  // FX_ERR_OOM: a server then hands back idle workspaces.)
  if (jsplit > 1 && !rounds) {
    const size_t left = ws_room(ctx, ws, "vx_work");
    const size_t least = (size_t)std::min<int64_t>(pairs_cap, (int64_t)a.n_psi * a.n_phi) * pair_bytes;
    size_t room = ctx->budget / 4;
    if (ctx->capturing || least <= left) room = std::min(room, left);
    if (sum_bytes + pair_bytes > room)
      return run_groups_in_turn<T, A>(ctx, ws, a, pass, tb, psi, ld_psi, phi, ld_phi, jsplit, st, stats);
    shape(room);
  } else if (!rounds) {
    shape(0);
  }
  const size_t sums = rounds ? 0 : nk * sum_bytes;
  void* work = nullptr;
  FX_TRY(ws_get(ctx, ws, "vx_work", sums + (size_t)nk * nj * pair_bytes, &work));
  cpx<T>* const volumes = reinterpret_cast<cpx<T>*>((char*)work + sums);
  const bool multi_j = nj < a.n_psi;
  cpx<A>* acc = nullptr;
  int64_t ld_acc = 0, gstride = 0;
  const bool grouped = jsplit > 1 && !rounds;  // partial sums in memory
  if (grouped) {
    // added into out after a block's last batch
    acc = reinterpret_cast<cpx<A>*>(work);
    ld_acc = nr;
    gstride = (int64_t)nk * nr;
  } else if (a.add) {
    // the one batch of each target starts from the caller's columns
    if (multi_j || sizeof(A) != 8) FX_FAIL(FX_ERR_INVALID, "a start value needs one orbital and FP64 sums");
    acc = reinterpret_cast<cpx<A>*>(const_cast<void*>(a.add));
    ld_acc = a.ld_add;
  } else if (multi_j) {
    if (out_is_A) {
      acc = reinterpret_cast<cpx<A>*>(a.out);
      ld_acc = a.ld_out;
    } else {
      void* p = nullptr;
      FX_TRY(ws_get(ctx, ws, "vx_acc", (size_t)a.n_phi * nr * sizeof(cpx<A>), &p));
      acc = reinterpret_cast<cpx<A>*>(p);
      ld_acc = nr;
    }
  }
  int64_t launches = 0;
  for (int k0 = 0; k0 < a.n_phi; k0 += nk) {
    const int kb = std::min(nk, a.n_phi - k0);
    for (int j0 = 0; j0 < a.n_psi; j0 += nj) {
      const int jb = std::min(nj, a.n_psi - j0);
      const int first = j0 == 0 && !a.add, last = j0 + jb >= a.n_psi;
      const int npairs = kb * jb;
      // algorithmic bytes of each pass, per pair and grid point: plane-forward
      // psi_j + T (phi_k is reused from cache across the batch's orbitals),
      // z-pass T read + write, plane-inverse T + psi_j, plus the partial sums
      // read and written once per batch and target
      const double vol = (double)npairs * nr * sizeof(cpx<T>);
      const double accb = (double)kb * nr *
                          ((first ? 0.0 : (double)sizeof(cpx<A>)) +
                           (last ? (out_c64 ? 8.0 : 16.0) : (double)sizeof(cpx<A>)));
      int slot;
      CtBatch<T> cb = make_batch<T>(a, tb, psi, ld_psi, phi, ld_phi, volumes, j0, jb, k0, kb, npairs, 0, jsplit);
      cb.rounds = rounds;
      CtAcc<A> ca{grouped ? acc - (int64_t)k0 * ld_acc : acc, ld_acc, first, a.out, a.ld_out, out_c64 ? 1 : 0,
                  grouped ? 0 : last, gstride};
      FX_TRY(prof_begin(ctx, st, FX_K_VX_PLANE_FWD, 2.0 * vol, &slot));
      FX_TRY(pass.a(cb));
      FX_TRY(prof_end(ctx, st, slot));
      FX_TRY(prof_begin(ctx, st, FX_K_VX_PENCIL_Z, 2.0 * vol, &slot));
      FX_TRY(pass.b(cb));
      FX_TRY(prof_end(ctx, st, slot));
      FX_TRY(prof_begin(ctx, st, FX_K_VX_PLANE_INV, 2.0 * vol + accb, &slot));
      FX_TRY(pass.c(cb, ca, 0));
      FX_TRY(prof_end(ctx, st, slot));
      launches += 3;
      if (grouped && last) {
        const double osz = out_c64 ? 8.0 : 16.0;
        FX_TRY(prof_begin(ctx, st, FX_K_REDUCE, (double)kb * nr * (jsplit * sizeof(cpx<A>) + osz), &slot));
        FX_TRY(combine_groups<A>(ctx, st, ca.acc, gstride, ld_acc, jsplit, k0, kb, nr, a.out, a.ld_out, out_c64 ? 1 : 0));
        FX_TRY(prof_end(ctx, st, slot));
        ++launches;
      }
    }
  }
  if (stats) {
    stats->nk = nk;
    stats->nj = nj;
    stats->launches = launches;
    stats->solves = (int64_t)a.n_psi * a.n_phi;
  }
  return FX_OK;
}

template <typename TI, typename TO>
static fx_status convert2(const void* in0, int64_t ld0, void* out0, int n0, const void* in1, int64_t ld1, void* out1,
                          int n1, int64_t ld_out, int64_t nr, hipStream_t st) {
  const dim3 grid((unsigned)((nr + 1023) / 1024), (unsigned)std::min<int64_t>((int64_t)n0 + n1, 65535));
  hipLaunchKernelGGL((k_convert<TI, TO>), grid, dim3(256), 0, st, reinterpret_cast<const cpx<TI>*>(in0), ld0,
                     reinterpret_cast<cpx<TO>*>(out0), n0, reinterpret_cast<const cpx<TI>*>(in1), ld1,
                     reinterpret_cast<cpx<TO>*>(out1), ld_out, nr, n0 + n1);
  FX_LAUNCH_CHECK();
  return FX_OK;
}

template <typename TI, typename TO>
static fx_status convert(const void* in, int64_t ld_in, void* out, int64_t ld_out, int64_t nr, int ncols,
                         hipStream_t st) {
  return convert2<TI, TO>(in, ld_in, out, ncols, nullptr, 0, nullptr, 0, ld_out, nr, st);
}

fx_status convert_cols(const void* in, fx_dtype din, int64_t ld_in, void* out, fx_dtype dout, int64_t ld_out,
                       int64_t nr, int ncols, hipStream_t st) {
  if (din == FX_C128 && dout == FX_C128) return convert<double, double>(in, ld_in, out, ld_out, nr, ncols, st);
  if (din == FX_C128) return convert<double, float>(in, ld_in, out, ld_out, nr, ncols, st);
  if (dout == FX_C128) return convert<float, double>(in, ld_in, out, ld_out, nr, ncols, st);
  return convert<float, float>(in, ld_in, out, ld_out, nr, ncols, st);
}

fx_status check_vx_args(const VxArgs& a) {
  FX_TRY(check_cell(a.cell));
  FX_TRY(check_kernel(a.kern, a.internal_kernel));
  const int64_t nr = (int64_t)a.cell->n[0] * a.cell->n[1] * a.cell->n[2];
  if (!a.psi || !a.phi || !a.out) FX_FAIL(FX_ERR_INVALID, "psi, phi and out must be non-NULL device pointers");
  if (a.n_psi <= 0 || a.n_phi <= 0) FX_FAIL(FX_ERR_INVALID, "n_psi = %d and n_phi = %d must be positive", a.n_psi, a.n_phi);
  if (a.ld_psi < nr || a.ld_phi < nr || a.ld_out < nr)
    FX_FAIL(FX_ERR_INVALID, "leading dimensions (%lld, %lld, %lld) must be >= N_r = %lld", (long long)a.ld_psi,
            (long long)a.ld_phi, (long long)a.ld_out, (long long)nr);
  if (a.in_dtype != FX_C128 && a.in_dtype != FX_C64) FX_FAIL(FX_ERR_UNSUPPORTED, "unknown in_dtype %d", a.in_dtype);
  if (a.out_dtype != FX_C128 && a.out_dtype != FX_C64) FX_FAIL(FX_ERR_UNSUPPORTED, "unknown out_dtype %d", a.out_dtype);
  if (a.prec != FX_PREC_FP64 && a.prec != FX_PREC_FP32 && a.prec != FX_PREC_FP32_ACC64)
    FX_FAIL(FX_ERR_UNSUPPORTED, "precision %d is not a V_X precision", a.prec);
  // aliasing of out with the inputs
  const size_t isz = dtype_size(a.in_dtype), osz = dtype_size(a.out_dtype);
  const char* o0 = (const char*)a.out;
  const char* o1 = o0 + ((size_t)(a.n_phi - 1) * a.ld_out + nr) * osz;
  const char* ins[2] = {(const char*)a.psi, (const char*)a.phi};
  const size_t ilen[2] = {((size_t)(a.n_psi - 1) * a.ld_psi + nr) * isz, ((size_t)(a.n_phi - 1) * a.ld_phi + nr) * isz};
  for (int i = 0; i < 2; ++i)
    if (o0 < ins[i] + ilen[i] && ins[i] < o1) FX_FAIL(FX_ERR_INVALID, "out overlaps an input array");
  if (a.ex_dev && !(a.phi == a.psi && a.ld_phi == a.ld_psi && a.n_phi <= a.n_psi))
    FX_FAIL(FX_ERR_INVALID, "ex_energy_dev requires phi == psi (same pointer and ld, n_phi <= n_psi)");
  return FX_OK;
}

bool plans_from_radix(const fx_cell* cell, const int32_t radix[3][4], PlanSet* ps, bool* any) {
  default_plans(cell, ps);
  *any = false;
  for (int x = 0; x < 3; ++x) {
    if (radix[x][0] == 0) continue;
    AxisPlan p;
    p.n = cell->n[x];
    p.nst = 0;
    for (int i = 0; i < 4; ++i) p.R[i] = 1;
    for (int i = 0; i < 4 && radix[x][i] != 0; ++i) p.R[p.nst++] = radix[x][i];
    for (int i = p.nst; i < 4; ++i)
      if (radix[x][i] != 0) return false;
    if (!valid_axis_plan(p)) return false;
    ps->ax[x] = p;
    *any = true;
  }
  return true;
}

std::array<int, 5> vx_tune_key(const fx_cell* cell, fx_prec prec, bool square) {
  return {cell->n[0], cell->n[1], cell->n[2], (int)prec, square ? 1 : 0};
}

void resolve_vx_config(fx_ctx* ctx, VxArgs* a) {
  // environment overrides, for experiments and comparisons
  if (const char* e = getenv("FX_VX_NJ")) a->force_nj = atoi(e);
  if (const char* e = getenv("FX_VX_XT")) a->xtile = atoi(e);
  if (const char* e = getenv("FX_VX_NTHR_B")) a->nthr_b = atoi(e);
  if (const char* e = getenv("FX_VX_HALVE")) a->halve = atoi(e);
  if (const char* e = getenv("FX_VX_A_PIPE")) a->a_pipe = atoi(e);
  if (const char* e = getenv("FX_VX_B_VAR")) a->b_var = atoi(e);
  if (const char* e = getenv("FX_VX_C_VAR")) a->c_var = atoi(e);
  if (const char* e = getenv("FX_VX_A_VAR")) a->a_var = atoi(e);
  if (const char* e = getenv("FX_VX_NT")) a->nt_hint = atoi(e);
  if (const char* e = getenv("FX_VX_C_SPLIT")) a->c_split = atoi(e);
  if (getenv("FX_VX_GENERIC")) a->kernels = 2;
  if (const char* e = getenv("FX_WORK_MB")) a->work_cap = (size_t)atol(e) << 20;
  if (!ctx) return;
  auto it = ctx->vx_tuning.find(vx_tune_key(a->cell, a->prec, vx_square_form(*a)));
  if (it == ctx->vx_tuning.end()) return;
  const fx_vx_config& c = it->second;
  if (!a->kernels) a->kernels = c.kernels;
  if (!a->work_cap && c.work_mb > 0) a->work_cap = (size_t)c.work_mb << 20;
  if (a->a_pipe < 0 && c.a_prefetch >= 0) a->a_pipe = c.a_prefetch;
  if (!a->b_var) a->b_var = c.b_variant;
  if (!a->c_var) a->c_var = c.c_variant;
  if (!a->a_var) a->a_var = c.a_variant;
  if (a->nt_hint < 0 && c.nt_hint >= 0) a->nt_hint = c.nt_hint;
  if (!a->c_split) a->c_split = c.c_split;
  if (!a->xtile) a->xtile = c.b_xtile;
  if (!a->nthr_b) a->nthr_b = c.b_threads;
  if (!a->plans_set) {
    bool any = false;
    PlanSet ps;
    if (plans_from_radix(a->cell, c.radix, &ps, &any) && any) {
      a->plans = ps;
      a->plans_set = true;
    }
  }
}

fx_status vx_apply(fx_ctx* ctx, Workspace* ws, const VxArgs& a_in, hipStream_t st, VxStats* stats) {
  FX_TRY(check_vx_args(a_in));
  VxArgs a = a_in;
  resolve_vx_config(ctx, &a);
  const int64_t nr = (int64_t)a.cell->n[0] * a.cell->n[1] * a.cell->n[2];
  const bool t64 = a.prec == FX_PREC_FP64;
  const bool same = a.phi == a.psi && a.ld_phi == a.ld_psi;
  const bool need_conv = (a.in_dtype == FX_C128) != t64;
  const GridTables* tb = nullptr;
  GridTables tb_scratch;
  if (a.segs.n > 0 && need_conv)
    FX_FAIL(FX_ERR_UNSUPPORTED, "multi-trajectory launches take orbitals in the compute type");
  int parts = ex_parts(nr);
  if (a.no_alloc) {
    if (!ws->arena) FX_FAIL(FX_ERR_INVALID, "allocation-free call without a scratch region");
    if (need_conv)
      FX_FAIL(FX_ERR_UNSUPPORTED, "the allocation-free form takes %s inputs for this precision (no conversion)",
              t64 ? "complex128" : "complex64");
    a.halve = 0;
    FX_TRY(scratch_tables(ws, a.cell, a.kern, t64 ? 0 : 1, a.plans_set ? &a.plans : nullptr, st, &tb_scratch));
    tb = &tb_scratch;
    // what the scratch region must still hold besides the pair volume: partial
    // sums when out cannot hold them, and the energy partials
    const size_t asz = a.prec == FX_PREC_FP32 ? 8 : 16;
    const size_t used = (ws->arena_used + 255) & ~(size_t)255;
    const size_t pair_bytes = (size_t)nr * (t64 ? 16 : 8);
    size_t reserve = 0, room = 0;
    for (parts = ex_parts(nr);; parts = 1) {
      reserve = (dtype_size(a.out_dtype) != asz ? (size_t)a.n_phi * nr * asz : 0) +
                (a.ex_dev ? (size_t)a.n_phi * parts * sizeof(double) : 0) + 3 * 256;
      room = ws->arena_bytes > used + reserve ? ws->arena_bytes - used - reserve : 0;
      if (room >= pair_bytes || parts == 1) break;
    }
    if (room < pair_bytes)
      FX_FAIL(FX_ERR_INVALID,
              "the %zu-byte scratch region cannot hold one pair volume (%zu bytes) besides %zu bytes of tables and "
              "%zu of partial sums; the call is too large for the allocation-free form",
              ws->arena_bytes, pair_bytes, used, reserve);
    a.work_cap = a.work_cap ? std::min(a.work_cap, room) : room;
  } else {
    FX_TRY(grid_tables(ctx, a.cell, a.kern, t64 ? 0 : 1, a.plans_set ? &a.plans : nullptr, &tb));
  }
  const void* psi = a.psi;
  const void* phi = a.phi;
  int64_t ld_psi = a.ld_psi, ld_phi = a.ld_phi;
  if (need_conv) {
    const int ncp = same ? std::max(a.n_psi, a.n_phi) : a.n_psi;
    const size_t tsz = t64 ? 16 : 8;
    void* p = nullptr;
    FX_TRY(ws_get(ctx, ws, "vx_psiT", (size_t)ncp * nr * tsz, &p));
    void* q = p;
    if (!same) FX_TRY(ws_get(ctx, ws, "vx_phiT", (size_t)a.n_phi * nr * tsz, &q));
    const int ncq = same ? 0 : a.n_phi;
    if (t64)
      FX_TRY((convert2<float, double>(a.psi, a.ld_psi, p, ncp, a.phi, a.ld_phi, q, ncq, nr, nr, st)));
    else
      FX_TRY((convert2<double, float>(a.psi, a.ld_psi, p, ncp, a.phi, a.ld_phi, q, ncq, nr, nr, st)));
    psi = p;
    phi = q;
    ld_psi = ld_phi = nr;
  }
  if (a.prec == FX_PREC_FP64) {
    FX_TRY((run_batches<double, double>(ctx, ws, a, tb, (const cpx<double>*)psi, ld_psi, (const cpx<double>*)phi,
                                        ld_phi, st, stats)));
  } else if (a.prec == FX_PREC_FP32_ACC64) {
    FX_TRY((run_batches<float, double>(ctx, ws, a, tb, (const cpx<float>*)psi, ld_psi, (const cpx<float>*)phi, ld_phi,
                                       st, stats)));
  } else {
    FX_TRY((run_batches<float, float>(ctx, ws, a, tb, (const cpx<float>*)psi, ld_psi, (const cpx<float>*)phi, ld_phi,
                                      st, stats)));
  }
  if (a.ex_dev) {
    // the spans' sums in the work buffer, which the passes no longer need: no
    // allocation whose failure could change their number, and with it the bits
    void* part = nullptr;
    FX_TRY(ws_get(ctx, ws, "vx_work", (size_t)a.n_phi * parts * sizeof(double), &part));
    const bool p64 = a.in_dtype == FX_C128, o64 = a.out_dtype == FX_C128;
    dim3 grid((unsigned)(a.n_phi * parts)), blk(256);
    if (p64 && o64)
      hipLaunchKernelGGL((k_dot_cols<double, double>), grid, blk, 0, st, (const cpx<double>*)a.psi, a.ld_psi,
                         (const cpx<double>*)a.out, a.ld_out, nr, parts,
                         (double*)part);
    else if (p64)
      hipLaunchKernelGGL((k_dot_cols<double, float>), grid, blk, 0, st, (const cpx<double>*)a.psi, a.ld_psi,
                         (const cpx<float>*)a.out, a.ld_out, nr, parts,
                         (double*)part);
    else if (o64)
      hipLaunchKernelGGL((k_dot_cols<float, double>), grid, blk, 0, st, (const cpx<float>*)a.psi, a.ld_psi,
                         (const cpx<double>*)a.out, a.ld_out, nr, parts,
                         (double*)part);
    else
      hipLaunchKernelGGL((k_dot_cols<float, float>), grid, blk, 0, st, (const cpx<float>*)a.psi, a.ld_psi,
                         (const cpx<float>*)a.out, a.ld_out, nr, parts,
                         (double*)part);
    FX_LAUNCH_CHECK();
    hipLaunchKernelGGL(k_half_sum, dim3(1), dim3(256), 0, st, (const double*)part, a.n_phi * parts, a.ex_dev);
    FX_LAUNCH_CHECK();
  }
  return FX_OK;
}

// Host run of the pass bodies for one pair: v = (-scale/Omega) *
// IFFT_u[K FFT_u(conj(psi_j) phi_k)], with the device code's plans, twiddles,
// folded kernel table and z-tiling, in FP64 (prec 0) or FP32 (prec 1).
// Inputs and outputs are host arrays of N_r interleaved complex doubles.
template <typename T>
static void host_pair(const fx_cell* cell, const HostTables& h, const double* psi_j, const double* phi_k, double* v,
                      int xtile, const PlanSet* plans) {
  const PassGeom g = make_geom(cell, plans);
  const size_t nxy = (size_t)g.nx * g.ny, nr = nxy * g.nz;
  std::vector<cpx<T>> a(nr), b(nr), vol(nr);
  for (size_t i = 0; i < nr; ++i) {
    a[i] = {(T)psi_j[2 * i], (T)psi_j[2 * i + 1]};
    b[i] = {(T)phi_k[2 * i], (T)phi_k[2 * i + 1]};
  }
  std::vector<cpx<T>> tw[3];
  for (int ax = 0; ax < 3; ++ax)
    for (auto& c : h.tw[ax]) tw[ax].push_back({(T)c.x, (T)c.y});
  const int xt = std::max(1, std::min(g.nx, xtile));
  std::vector<cpx<T>> s((size_t)std::max(plane_lds_elems(g), g.nz * xt));
  for (int z = 0; z < g.nz; ++z)
    pass_a_body<T>(a.data() + z * nxy, b.data() + z * nxy, vol.data() + z * nxy, s.data(), tw[0].data(), tw[1].data(),
                   g, 0, 1, HostSync{});
  std::vector<T> kl((size_t)g.hz * g.hx);
  for (int y = 0; y < g.ny; ++y) {
    const int fy = h.fold[1][y];
    for (int fz = 0; fz < g.hz; ++fz)
      for (int fx = 0; fx < g.hx; ++fx) kl[fz * g.hx + fx] = (T)h.kfold[((size_t)fz * g.hy + fy) * g.hx + fx];
    const Lines tile{xt, xt, fast_div(xt)};
    for (int x0 = 0; x0 < g.nx; x0 += xt) {
      const KSlice<T> kf{kl.data(), h.fold[0].data(), h.fold[2].data(), x0, g.hx};
      pass_b_body<T>(vol.data(), y, x0, tile, s.data(), tw[2].data(), tw[2].data(), kf, g, 0, 1, HostSync{});
    }
  }
  for (int z = 0; z < g.nz; ++z) {
    pass_c_fft<T>(vol.data() + z * nxy, s.data(), tw[0].data(), tw[1].data(), g, 0, 1, HostSync{}, [] {});
    const Span<T> rows = lds_rows(s.data(), g);
    run_stage<false, false, false, T>(rows, rows, g.ax.st[0], plane_rows(g), tw[0].data(), 0, 1);
    for (size_t e = 0; e < nxy; ++e) {
      const int y = (int)(e / g.nx), x = (int)(e - (size_t)y * g.nx);
      v[2 * (z * nxy + e)] = (double)s[(size_t)y * g.sx + x].x;
      v[2 * (z * nxy + e) + 1] = (double)s[(size_t)y * g.sx + x].y;
    }
  }
}

}  // namespace fx

using namespace fx;

extern "C" {

fx_status fx_apply_vx(fx_ctx* ctx, const fx_cell* cell, const fx_kernel* kernel, const void* psi, int32_t n_psi,
                      int64_t ld_psi, const void* phi, int32_t n_phi, int64_t ld_phi, void* out, int64_t ld_out,
                      fx_dtype in_dtype, fx_dtype out_dtype, fx_prec prec, void* stream, double* ex_energy_dev) {
  clear_error();
  if (!ctx) FX_FAIL(FX_ERR_INVALID, "ctx is NULL");
  std::lock_guard<std::recursive_mutex> lk(ctx->mu);
  FX_HIP(hipSetDevice(ctx->device));
  VxArgs a;
  a.cell = cell;
  a.kern = kernel;
  a.psi = psi;
  a.n_psi = n_psi;
  a.ld_psi = ld_psi;
  a.phi = phi;
  a.n_phi = n_phi;
  a.ld_phi = ld_phi;
  a.out = out;
  a.ld_out = ld_out;
  a.in_dtype = in_dtype;
  a.out_dtype = out_dtype;
  a.prec = prec;
  a.ex_dev = ex_energy_dev;
  hipStream_t st = (hipStream_t)stream;
  FX_TRY(note_capture(ctx, st));
  if (ctx->graph_max <= 0) return vx_apply(ctx, &ctx->ws, a, st, nullptr);
  if (!cell || !kernel) FX_FAIL(FX_ERR_INVALID, "cell and kernel must be non-NULL");
  KeyBytes k;
  k.add(0).add(cell->n[0]).add(cell->n[1]).add(cell->n[2]).add(cell->len[0]).add(cell->len[1]).add(cell->len[2]);
  k.add(kernel->kind).add(kernel->omega).add(kernel->scale).add(psi).add(n_psi).add(ld_psi).add(phi).add(n_phi);
  k.add(ld_phi).add(out).add(ld_out).add(in_dtype).add(out_dtype).add(prec).add(ex_energy_dev);
  return graph_call(ctx, k.b, st, [&](hipStream_t s) { return vx_apply(ctx, &ctx->ws, a, s, nullptr); });
}

fx_status fx_debug_host_pair_plan(const fx_cell* cell, const fx_kernel* kernel, int prec, const int32_t* radix,
                                  const double* psi_j, const double* phi_k, double* v) {
  int xtile = cell ? cell->n[0] : 1;
  if (const char* e = getenv("FX_VX_XT")) xtile = atoi(e);
  clear_error();
  FX_TRY(check_cell(cell));
  FX_TRY(check_kernel(kernel));
  if (!psi_j || !phi_k || !v) FX_FAIL(FX_ERR_INVALID, "NULL host pointer");
  PlanSet ps;
  bool any = false;
  if (radix && !plans_from_radix(cell, reinterpret_cast<const int32_t(*)[4]>(radix), &ps, &any))
    FX_FAIL(FX_ERR_INVALID, "invalid radix schedule");
  const PlanSet* pp = radix ? &ps : nullptr;
  HostTables h;
  host_tables(cell, kernel, &h, pp);
  if (prec == 0)
    host_pair<double>(cell, h, psi_j, phi_k, v, xtile, pp);
  else
    host_pair<float>(cell, h, psi_j, phi_k, v, xtile, pp);
  return FX_OK;
}

fx_status fx_debug_host_pair(const fx_cell* cell, const fx_kernel* kernel, int prec, const double* psi_j,
                             const double* phi_k, double* v) {
  return fx_debug_host_pair_plan(cell, kernel, prec, nullptr, psi_j, phi_k, v);
}

fx_status fx_debug_axis_plans(int32_t n, int32_t max_plans, int32_t* radix_out, int32_t* count) {
  clear_error();
  if (!radix_out || !count || max_plans <= 0) FX_FAIL(FX_ERR_INVALID, "bad output arguments");
  if (!supported_edge(n)) FX_FAIL(FX_ERR_UNSUPPORTED, "edge %d is not 2^a 3^b in [2, 96]", n);
  std::vector<AxisPlan> ps((size_t)max_plans);
  const int k = enumerate_axis_plans(n, ps.data(), max_plans);
  for (int i = 0; i < k; ++i)
    for (int r = 0; r < 4; ++r) radix_out[4 * i + r] = r < ps[i].nst ? ps[i].R[r] : 0;
  *count = k;
  return FX_OK;
}

}  // extern "C"
