// FP64 complex dense linear algebra for the ACE operator (hand-written HIP):
//   zgemm   C = alpha op(A) op(B) + beta C, op in {N, C}, batched, split over K
//           with a fixed-order FP64 reduction of the split partial sums;
//   potrf   blocked Cholesky of a Hermitian positive definite matrix (lower);
//   trinv   inverse of a lower triangular matrix (recursive 2x2 blocking);
//   herm    Hermitised copy, its negation and half its trace.
// All matrices are column-major complex double: element (i, j) at P[i + j*ld].
#include <algorithm>
#include <cstdlib>
#include <cmath>
#include <cstdio>
#include <type_traits>
#include <vector>

#include "common.hpp"
#include "fft.hpp"
#include "linalg.hpp"

namespace fx {

using z = cpx<double>;

FX_HD z zconj(z a) { return {a.x, -a.y}; }
// acc + a*b as four fused multiply-adds (written as `acc += a.x*b.x - a.y*b.y`
// the compiler emits a multiply, a fused multiply-add and an add per
// component: six FP64 instructions instead of four)
FX_HD z zfma(z acc, z a, z b) {
  acc.x = __builtin_fma(a.x, b.x, acc.x);
  acc.x = __builtin_fma(-a.y, b.y, acc.x);
  acc.y = __builtin_fma(a.x, b.y, acc.y);
  acc.y = __builtin_fma(a.y, b.x, acc.y);
  return acc;
}

// ---------------------------------------------------------------------------
// zgemm on the FP64 matrix cores (v_mfma_f64_16x16x4: 68-73 TFLOP/s in a loop
// of its own on this GPU, about the vector FMA rate, but its operands feed
// 16x16 outputs each, so the LDS reads that held a vector-FMA kernel to 49-52
// TFLOP/s are a tenth of the time here).  2 x WNW waves; output tile (32 WM) x
// (16 WN WNW), K steps of 8 through a double-buffered LDS with one barrier
// per step; the next step's global loads are in registers while the current
// one is multiplied.  A wave owns the 16x16 tiles (wm + 2 i, wn + WNW j), so
// that the columns left over at an edge are shared by the waves of a row, and
// skips those that lie outside.
// 64 x 64 tiles at four waves per SIMD: 58-61 TFLOP/s of executed products
// (N = 432 at 72^3: Psi^H H Psi 15.0 -> 10.3 ms, Psi S 12.2 -> 9.3 ms against
// the vector-FMA kernel).  128 x 64 at two waves per SIMD measured 2-6%
// slower, 128 x 128 with steps of 16 at one workgroup per CU 14-20% (the
// barriers are exposed).
// The matrix instruction is given B's columns as its rows and A's rows as its
// columns: lane l then holds C(m = l % 16, n = 4 e + l / 16) of a tile, so
// stores run along m.  A complex product is four real ones (re: b.x a.x, then
// -b.y a.y; im: b.y a.x, then b.x a.y).  The sum of an element runs over k in
// order, whatever the tile, so results do not depend on the tile chosen.
//
// Split over K: split s covers [s*kchunk, min(K, (s+1)*kchunk)).  With a
// partial buffer the raw sum of split s goes to partial[(batch*nsplit + s) *
// M*N] (ld M); without one (nsplit == 1) C = alpha*sum + beta*C is written
// directly.  Blocks are dealt so that each XCD works on neighbouring tiles
// (n fastest) of the same split and shares their operands in its L2, where their
// number is a multiple of 8 (runs for any number measured within 1%).
// ---------------------------------------------------------------------------
constexpr int ZK = 8;
typedef double doublex4 __attribute__((ext_vector_type(4)));

struct ZgArgs {
  int M, N, K;
  const z* A;
  int64_t lda, sA;
  const z* B;
  int64_t ldb, sB;
  z* C;
  int64_t ldc, sC;
  z alpha, beta;
  int nsplit, kchunk, tiles_m, tiles_n;
  z* partial;
  ZgShape shape;
  ZgResidual res;
};

template <int WM, int WN, int WNW>
struct ZgTile {
  static constexpr int BM = 32 * WM, BN = 16 * WN * WNW, NT = 128 * WNW;
  // rows of BM + 1 (BN + T::PAD) values: the k of one m that op C stores from
  // neighbouring lanes fall on distinct banks
  static constexpr int PAD = 16 / ZK;
  static constexpr int LA = ZK * (BM + PAD), LB = ZK * (BN + PAD);
  static constexpr size_t kLds = 2 * (LA + LB) * sizeof(z);
};

template <int OPA, int OPB, int WM, int WN, int WNW>
__global__ void __launch_bounds__(128 * WNW, WM * WN <= 4 ? 4 : 2) k_zgemm(const ZgArgs g) {
  using T = ZgTile<WM, WN, WNW>;
  constexpr int BM = T::BM, BN = T::BN, NT = T::NT;
  constexpr int UA = BM * ZK / NT, UB = BN * ZK / NT;
  extern __shared__ __align__(16) unsigned char smem_raw[];
  z* const As = reinterpret_cast<z*>(smem_raw);
  z* const Bs = As + 2 * T::LA;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave & 1, wn = wave >> 1;
  const int nblk = gridDim.x, bid = blockIdx.x;
  const int lid = nblk % 8 == 0 ? (bid % 8) * (nblk / 8) + bid / 8 : bid;
  const int tn = lid % g.tiles_n, r1 = lid / g.tiles_n;
  const int tm = r1 % g.tiles_m, bz = r1 / g.tiles_m;
  const int batch = bz / g.nsplit, split = bz - batch * g.nsplit;
  const int m0 = tm * BM, n0 = tn * BN, N = g.N;
  const int M = g.shape.mlim > 0 ? min(g.M, g.shape.mlim - batch * g.shape.mstep) : g.M;
  if (m0 >= M || ((g.shape.flags & kZgHermitian) && m0 + BM <= n0)) return;
  const z* A = g.A + batch * g.sA;
  const z* B = g.B + batch * g.sB;
  int kbeg = split * g.kchunk, kend = min(g.K, kbeg + g.kchunk);
  if (g.shape.flags & kZgALower) kend = min(kend, min(M, m0 + BM));
  if (g.shape.flags & kZgBLower) kbeg = max(kbeg, n0);
  // staged loads: UA elements of the A tile and UB of the B tile per thread;
  // op C reads along k (the stored matrix's column)
  const auto a_m = [tid](int u) { return OPA == 0 ? (tid + NT * u) % BM : (tid + NT * u) / ZK; };
  const auto a_k = [tid](int u) { return OPA == 0 ? (tid + NT * u) / BM : (tid + NT * u) % ZK; };
  const auto b_n = [tid](int u) { return OPB == 0 ? (tid + NT * u) / ZK : (tid + NT * u) % BN; };
  const auto b_k = [tid](int u) { return OPB == 0 ? (tid + NT * u) % ZK : (tid + NT * u) / BN; };
  // Out-of-range rows and columns load a clamped one (they only reach outputs
  // that are not written); k past the end is set to zero on the way to LDS.
  // Loads stand outside branches and op C's sign is applied after them, so
  // that nothing waits for a load before its step is stored.
  z ra[UA], rb[UB];
  const z *pa[UA], *pb[UB];
  const int64_t da = OPA == 0 ? g.lda : 1, db = OPB == 0 ? 1 : g.ldb;
#pragma unroll
  for (int u = 0; u < UA; ++u) pa[u] = A + (int64_t)min(m0 + a_m(u), M - 1) * (OPA == 0 ? 1 : g.lda);
#pragma unroll
  for (int u = 0; u < UB; ++u) pb[u] = B + (int64_t)min(n0 + b_n(u), N - 1) * (OPB == 0 ? g.ldb : 1);
  const auto gload = [&](int k0) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < UA; ++u) ra[u] = pa[u][min(k0 + a_k(u), kend - 1) * da];
#pragma unroll
    for (int u = 0; u < UB; ++u) rb[u] = pb[u][min(k0 + b_k(u), kend - 1) * db];
  };
  const auto sstore = [&](int b, int k0) __attribute__((always_inline)) {
    const bool tail = k0 + ZK > kend;
#pragma unroll
    for (int u = 0; u < UA; ++u) {
      z v = OPA == 0 ? ra[u] : zconj(ra[u]);
      if (tail && k0 + a_k(u) >= kend) v = z{0.0, 0.0};
      As[b * T::LA + a_k(u) * (BM + T::PAD) + a_m(u)] = v;
    }
#pragma unroll
    for (int u = 0; u < UB; ++u) {
      z v = OPB == 0 ? rb[u] : zconj(rb[u]);
      if (tail && k0 + b_k(u) >= kend) v = z{0.0, 0.0};
      Bs[b * T::LB + b_k(u) * (BN + T::PAD) + b_n(u)] = v;
    }
  };
  doublex4 cr[WM][WN], ci[WM][WN];
#pragma unroll
  for (int i = 0; i < WM; ++i)
#pragma unroll
    for (int j = 0; j < WN; ++j) {
      cr[i][j] = doublex4{0.0, 0.0, 0.0, 0.0};
      ci[i][j] = doublex4{0.0, 0.0, 0.0, 0.0};
    }
  // 16-wide tiles of this wave that hold any output
  const int nti = min(WM, max(0, ((M - m0 + 15) / 16 - wm + 1) / 2));
  const int ntj = min(WN, max(0, ((N - n0 + 15) / 16 - wn + WNW - 1) / WNW));
  const int l16 = lane & 15, lk = lane >> 4;
  const auto mac = [&](int buf, auto full) __attribute__((always_inline)) {
    const z* as = As + buf * T::LA + lk * (BM + T::PAD) + wm * 16 + l16;
    const z* bs = Bs + buf * T::LB + lk * (BN + T::PAD) + wn * 16 + l16;
#pragma unroll
    for (int kk = 0; kk < ZK / 4; ++kk) {
      z a[WM], b[WN];
#pragma unroll
      for (int i = 0; i < WM; ++i) a[i] = as[4 * kk * (BM + T::PAD) + 32 * i];
#pragma unroll
      for (int j = 0; j < WN; ++j) b[j] = bs[4 * kk * (BN + T::PAD) + 16 * WNW * j];
#pragma unroll
      for (int i = 0; i < WM; ++i)
#pragma unroll
        for (int j = 0; j < WN; ++j)
          if (full.value || (i < nti && j < ntj)) {
            cr[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(b[j].x, a[i].x, cr[i][j], 0, 0, 0);
            ci[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(b[j].y, a[i].x, ci[i][j], 0, 0, 0);
            if (!full.value) {
              cr[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(-b[j].y, a[i].y, cr[i][j], 0, 0, 0);
              ci[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(b[j].x, a[i].y, ci[i][j], 0, 0, 0);
            }
          }
      if (full.value) {
#pragma unroll
        for (int i = 0; i < WM; ++i)
#pragma unroll
          for (int j = 0; j < WN; ++j) {
            cr[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(-b[j].y, a[i].y, cr[i][j], 0, 0, 0);
            ci[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(b[j].x, a[i].y, ci[i][j], 0, 0, 0);
          }
      }
    }
  };
  const auto kloop = [&](auto full) __attribute__((always_inline)) {
    if (kbeg < kend) {
      gload(kbeg);
      sstore(0, kbeg);
    }
    __syncthreads();
    int buf = 0;
    for (int k0 = kbeg; k0 < kend; k0 += ZK) {
      const bool more = k0 + ZK < kend;
      if (more) gload(k0 + ZK);
      mac(buf, full);
      if (more) sstore(buf ^ 1, k0 + ZK);
      __syncthreads();
      buf ^= 1;
    }
  };
  if (m0 + BM <= M && n0 + BN <= N)
    kloop(std::true_type{});
  else
    kloop(std::false_type{});
  z* P = g.partial ? g.partial + (int64_t)bz * M * N : nullptr;
  z* Cb = g.C + batch * g.sC;
  const bool bz0 = g.beta.x == 0.0 && g.beta.y == 0.0;
#pragma unroll
  for (int i = 0; i < WM; ++i)
#pragma unroll
    for (int j = 0; j < WN; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int m = m0 + (wm + 2 * i) * 16 + l16, n = n0 + (wn + WNW * j) * 16 + 4 * e + lk;
        if (m >= M || n >= N) continue;
        const z s = {cr[i][j][e], ci[i][j][e]};
        if (P) {
          P[m + (int64_t)n * M] = s;
        } else if (g.res.psi) {
          // psi - half + i hdt (h - s), s = (Psi S)(m, n)
          const z p = g.res.psi[m + (int64_t)n * g.res.ldp], f = g.res.half[m + (int64_t)n * g.res.ldf];
          const z h = g.res.h[m + (int64_t)n * g.res.ldh];
          Cb[m + (int64_t)n * g.ldc] = z{p.x - f.x - g.res.hdt * (h.y - s.y), p.y - f.y + g.res.hdt * (h.x - s.x)};
        } else {
          z r = cmul(g.alpha, s);
          if (!bz0) r = cadd(r, cmul(g.beta, Cb[m + (int64_t)n * g.ldc]));
          Cb[m + (int64_t)n * g.ldc] = r;
        }
      }
}

// C = alpha * sum_s partial_s + beta * C.  A block adds the splits of 16
// neighbouring elements: group q of 16 threads takes splits q, q + 16, ... in
// ascending order, then the 16 sums are added in order of q.  (One thread per
// element left a 128 x 100 result on 50 workgroups.)
__global__ void __launch_bounds__(256) k_split_reduce(int M, int N, int nsplit, int nbatch,
                                                      const z* __restrict__ partial, z* C, int64_t ldc, int64_t sC,
                                                      z alpha, z beta) {
  __shared__ z red[16][17];
  const int64_t MN = (int64_t)M * N;
  const int el = threadIdx.x & 15, q = threadIdx.x >> 4;
  for (int64_t base = (int64_t)blockIdx.x * 16; base < MN * nbatch; base += (int64_t)gridDim.x * 16) {
    const int64_t i = base + el;
    const int64_t b = i / MN, e = i - b * MN;
    z s = {0.0, 0.0};
    if (b < nbatch) {
#pragma unroll 4
      for (int t = q; t < nsplit; t += 16) s = cadd(s, partial[(b * nsplit + t) * MN + e]);
    }
    red[q][el] = s;
    __syncthreads();
    if (q == 0 && b < nbatch) {
      for (int t = 1; t < 16; ++t) s = cadd(s, red[t][el]);
      z r = cmul(alpha, s);
      z* c = C + b * sC + e % M + (e / M) * ldc;
      if (!(beta.x == 0.0 && beta.y == 0.0)) r = cadd(r, cmul(beta, *c));
      *c = r;
    }
    __syncthreads();
  }
}

static unsigned reduce_blocks(int64_t elems) { return (unsigned)std::max<int64_t>(1, std::min<int64_t>((elems + 15) / 16, 16384)); }

fx_status zgemm(fx_ctx* ctx, Workspace* ws, hipStream_t st, int opa, int opb, int M, int N, int K, z alpha,
                const void* A, int64_t lda, const void* B, int64_t ldb, z beta, void* C, int64_t ldc, int batch,
                int64_t sA, int64_t sB, int64_t sC, int nsplit_hint, ZgShape shape, ZgResidual res) {
  if (M <= 0 || N <= 0) return FX_OK;
  if (K <= 0) {
    // empty sum: C = beta C (no splits to add)
    hipLaunchKernelGGL(k_split_reduce, dim3(reduce_blocks((int64_t)M * N * batch)), dim3(256), 0, st, M, N, 0, batch,
                       (const z*)nullptr, (z*)C, ldc, sC, alpha, beta);
    FX_LAUNCH_CHECK();
    return FX_OK;
  }
  const int n_cu = std::max(ctx->n_cu, 1);
  const auto tiles_of = [&](int bm, int bn) { return (int64_t)((M + bm - 1) / bm) * ((N + bn - 1) / bn) * batch; };
  int nsplit = nsplit_hint;
  if (nsplit <= 0) {
    // enough workgroups to fill the chip twice (four 64 x 64 tiles are resident
    // per CU), each with at least 16 K steps
    int per_cu = 8;
    if (const char* e = getenv("FX_ZGEMM_PER_CU")) per_cu = std::max(1, std::min(64, atoi(e)));
    const int64_t want = std::max<int64_t>(1, per_cu * n_cu / tiles_of(64, 64));
    nsplit = (int)std::max<int64_t>(1, std::min<int64_t>(want, K / 128));
  }
  int kchunk = (K + nsplit - 1) / nsplit;
  kchunk = (kchunk + ZK - 1) / ZK * ZK;
  nsplit = (K + kchunk - 1) / kchunk;
  z* part = nullptr;
  if (nsplit > 1 && batch == 1) {
    // Partial sums that the budget cannot hold: the product in blocks of columns
    // with the same splits, and so the same bits.
    const size_t col = sizeof(z) * (size_t)M * nsplit, room = ws_room(ctx, ws, "zgemm_part");
    if (col * N > room && N > 1) {
      const int nc = (int)std::max<size_t>(1, room / col);
      shape.flags &= ~kZgHermitian;  // (a block's columns do not start at the diagonal: all its tiles)
      for (int n0 = 0; n0 < N; n0 += nc)
        FX_TRY(zgemm(ctx, ws, st, opa, opb, M, std::min(nc, N - n0), K, alpha, A, lda,
                     (const z*)B + (opb ? n0 : n0 * ldb), ldb, beta, (z*)C + n0 * ldc, ldc, 1, 0, 0, 0, nsplit, shape,
                     res));
      return FX_OK;
    }
  }
  if (nsplit > 1) {
    void* p = nullptr;
    FX_TRY(ws_get(ctx, ws, "zgemm_part", sizeof(z) * (size_t)M * N * nsplit * batch, &p));
    part = (z*)p;
  }
  // 64 x 64 tiles where they occupy the chip; below that 32 x 32, whose
  // workgroups are a quarter of the work each (N x N products of the
  // factorisations)
  const bool big = tiles_of(64, 64) * nsplit >= n_cu;
  const int bm = big ? 64 : 32, bn = bm;
  ZgArgs g{M, N, K, (const z*)A, lda, sA, (const z*)B, ldb, sB, (z*)C, ldc, sC, alpha, beta, nsplit, kchunk,
           (M + bm - 1) / bm, (N + bn - 1) / bn, part, shape, res};
  const dim3 grid((unsigned)(tiles_of(bm, bn) * nsplit));
  int slot;
  FX_TRY(prof_begin(ctx, st, opa ? FX_K_GEMM_CN : FX_K_GEMM_NN, 8.0 * M * N * (double)K * batch, &slot));
#define FX_ZG(a, b)                                                                     \
  if (big) {                                                                            \
    const auto kern = k_zgemm<a, b, 2, 2, 2>;                                           \
    FX_TRY(allow_dynamic_lds((const void*)kern, ZgTile<2, 2, 2>::kLds));                \
    hipLaunchKernelGGL(kern, grid, dim3(ZgTile<2, 2, 2>::NT), (ZgTile<2, 2, 2>::kLds), st, g);          \
  } else {                                                                              \
    const auto kern = k_zgemm<a, b, 1, 1, 2>;                                           \
    hipLaunchKernelGGL(kern, grid, dim3(256), (ZgTile<1, 1, 2>::kLds), st, g);          \
  }
  if (opa == 0 && opb == 0) {
    FX_ZG(0, 0)
  } else if (opa == 0) {
    FX_ZG(0, 1)
  } else if (opb == 0) {
    FX_ZG(1, 0)
  } else {
    FX_ZG(1, 1)
  }
#undef FX_ZG
  FX_LAUNCH_CHECK();
  FX_TRY(prof_end(ctx, st, slot));
  if (nsplit > 1) {
    FX_TRY(prof_begin(ctx, st, FX_K_REDUCE, 16.0 * M * N * batch * (nsplit + 2.0), &slot));
    hipLaunchKernelGGL(k_split_reduce, dim3(reduce_blocks((int64_t)M * N * batch)), dim3(256), 0, st, M, N, nsplit,
                       batch, (const z*)part, (z*)C, ldc, sC, alpha, beta);
    FX_LAUNCH_CHECK();
    FX_TRY(prof_end(ctx, st, slot));
  }
  return FX_OK;
}

// ---------------------------------------------------------------------------
// Hermitisation: H = (M + M^H)/2, Aneg = -H, ex = 1/2 Re tr H.
// ---------------------------------------------------------------------------
__global__ void k_herm(int n, const z* __restrict__ M, int64_t ldm, z* __restrict__ H, z* __restrict__ Aneg) {
  const int64_t nn = (int64_t)n * n;
  for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < nn; e += (int64_t)gridDim.x * blockDim.x) {
    const int i = (int)(e % n), j = (int)(e / n);
    const z a = M[i + (int64_t)j * ldm], b = M[j + (int64_t)i * ldm];
    z h = {0.5 * (a.x + b.x), 0.5 * (a.y - b.y)};
    if (i == j) h.y = 0.0;
    H[e] = h;
    Aneg[e] = z{-h.x, -h.y};
  }
}

// half the trace: 64 strided sums in ascending order, added in order of the lane
__global__ void __launch_bounds__(64) k_half_trace(int n, const z* __restrict__ H, double* out) {
  __shared__ double red[64];
  double s = 0.0;
  for (int i = threadIdx.x; i < n; i += 64) s += H[i + (int64_t)i * n].x;
  red[threadIdx.x] = s;
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int t = 1; t < 64; ++t) s += red[t];
    *out = 0.5 * s;
  }
}

// ---------------------------------------------------------------------------
// Blocked Cholesky, lower: A = L L^H, in blocks of CB columns.  Three launches
// per block: the diagonal block (factor and inverse, one workgroup), the rows
// below it (substitution) and the trailing update; the inverses are kept for
// ztrinv.  What bounds it is the chain of small launches, so a block is
// as large as one workgroup holds in registers: with 32-wide blocks solved by
// one thread per row, factor and inverse of 432 columns took 2.1 ms in 70
// launches (now 0.5 ms in 27).
// ---------------------------------------------------------------------------
constexpr int CB = kCholBlock;

// Diagonal block (nb <= CB columns at (k, k)): right-looking elimination with
// the 4 x 4 elements (tr + 16 i, ts + 16 j) of a thread in registers, column
// by column.  S becomes U D U^H with U unit lower: column c publishes S(:, c)
// (not yet scaled) and row c of X = U^{-1}, each element then takes its
// update, and one barrier per column suffices with two buffers.  At the end
// L = U D^{1/2} and L^{-1} = D^{-1/2} X.  Past nb the block is the identity.
// A non-positive or non-finite pivot records column + 1 in *info (first one
// wins) and is replaced by 1 so the rest stays finite.
__global__ void __launch_bounds__(256) k_potrf_diag(int n, z* A, int64_t lda, int k, z* __restrict__ dinv, int* info) {
  __shared__ z col[2][CB], row[2][CB];
  __shared__ double piv[CB];
  const int nb = min(CB, n - k);
  const int tr = threadIdx.x & 15, ts = threadIdx.x >> 4;
  z S[4][4], X[4][4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int r = tr + 16 * i, s = ts + 16 * j;
      X[i][j] = z{r == s ? 1.0 : 0.0, 0.0};
      S[i][j] = X[i][j];
      if (r < nb && s <= r) S[i][j] = A[(k + r) + (int64_t)(k + s) * lda];
    }
#pragma unroll
  for (int cj = 0; cj < 4; ++cj) {
    for (int cc = 0; cc < 16; ++cc) {
      const int c = 16 * cj + cc, buf = c & 1;
      if (ts == cc) {
#pragma unroll
        for (int i = 0; i < 4; ++i) col[buf][tr + 16 * i] = S[i][cj];
      }
      if (tr == cc) {
#pragma unroll
        for (int j = 0; j < 4; ++j) row[buf][ts + 16 * j] = X[cj][j];
      }
      __syncthreads();
      double d = col[buf][c].x;
      if (!(d > 0.0) || !isfinite(d)) {
        if (threadIdx.x == 0 && *info == 0) *info = k + c + 1;
        d = 1.0;
      }
      if (threadIdx.x == 0) piv[c] = d;
      const double inv = 1.0 / d;
      z m[4], x[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int s = ts + 16 * j;
        m[j] = s > c ? zconj(col[buf][s]) : z{0.0, 0.0};
        x[j] = row[buf][s];
      }
#pragma unroll
      for (int i = cj; i < 4; ++i) {
        const int r = tr + 16 * i;
        const z v = col[buf][r];
        const z l = r > c ? z{-v.x * inv, -v.y * inv} : z{0.0, 0.0};
#pragma unroll
        for (int j = cj; j < 4; ++j) S[i][j] = zfma(S[i][j], l, m[j]);
#pragma unroll
        for (int j = 0; j <= cj; ++j) X[i][j] = zfma(X[i][j], l, x[j]);
      }
    }
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int r = tr + 16 * i, s = ts + 16 * j;
      const double ir = 1.0 / sqrt(piv[r]), is = 1.0 / sqrt(piv[s]);
      dinv[r + CB * s] = z{X[i][j].x * ir, X[i][j].y * ir};
      if (r < nb && s < nb)
        A[(k + r) + (int64_t)(k + s) * lda] =
            r > s ? z{S[i][j].x * is, S[i][j].y * is} : z{r == s ? sqrt(piv[s]) : 0.0, 0.0};
    }
}

// Rows below the diagonal block at (k, k): X L_kk^H = A21 by substitution, column
// by column.  (The product with the explicit inverse of the block is a matrix
// product, but its error grows with the block's condition: an orbital that
// differs from another by 1e-6 left |M - L L^H| at 5e-12 |M| instead of 1e-15.)
// What bounds it is the chain over the 64 columns, so a row is shared by 16 lanes,
// lane q with the columns q + 16 i in registers: the lane that owns column c hands
// x_c to the others, and each takes it off its later columns.  The loop over a
// lane's columns stays rolled: unrolled over all 64 it is 40 KB of code that runs
// once, 150 us of instruction fetches; this is 17 us for up to 368 rows, 12 as a
// product.  L_kk lies in LDS by column.
__global__ void __launch_bounds__(256) k_potrf_panel(int n, z* A, int64_t lda, int k) {
  __shared__ z L[CB][CB];
  for (int e = threadIdx.x; e < CB * CB; e += 256) L[e / CB][e % CB] = A[(k + e % CB) + (int64_t)(k + e / CB) * lda];
  const int q = threadIdx.x & 15, row = k + CB + blockIdx.x * 16 + (threadIdx.x >> 4);
  z* const a = A + min(row, n - 1) + (int64_t)(k + q) * lda;
  z x[CB / 16];
#pragma unroll
  for (int i = 0; i < CB / 16; ++i) x[i] = a[(int64_t)16 * i * lda];
  __syncthreads();
  // 1 / L(c, c) in the diagonal's imaginary part
  if (threadIdx.x < CB) L[threadIdx.x][threadIdx.x].y = 1.0 / L[threadIdx.x][threadIdx.x].x;
  __syncthreads();
  // v / d for real d: the product with its reciprocal, corrected once
  const auto over = [](double v, z d) __attribute__((always_inline)) {
    const double t = v * d.y;
    return __builtin_fma(__builtin_fma(-t, d.x, v), d.y, t);
  };
#pragma unroll
  for (int i = 0; i < CB / 16; ++i) {
#pragma unroll 2
    for (int s = 0; s < 16; ++s) {
      const int c = 16 * i + s;
      const z d = L[c][c], v = {over(x[i].x, d), over(x[i].y, d)};
      const z m = {-__shfl(v.x, s, 16), -__shfl(v.y, s, 16)};
      // column 16 i + q is x_c itself for lane s and a later one for lanes q > s
      const z f = zfma(x[i], m, zconj(L[c][16 * i + q]));
      x[i].x = q == s ? v.x : q > s ? f.x : x[i].x;
      x[i].y = q == s ? v.y : q > s ? f.y : x[i].y;
#pragma unroll
      for (int j = i + 1; j < CB / 16; ++j) x[j] = zfma(x[j], m, zconj(L[c][16 * j + q]));
    }
  }
  if (row < n)
#pragma unroll
    for (int i = 0; i < CB / 16; ++i) a[(int64_t)16 * i * lda] = x[i];
}

__global__ void k_zero_upper(int n, z* A, int64_t lda) {
  const int64_t nn = (int64_t)n * n;
  for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < nn; e += (int64_t)gridDim.x * blockDim.x) {
    const int i = (int)(e % n), j = (int)(e / n);
    if (i < j) A[i + (int64_t)j * lda] = z{0.0, 0.0};
  }
}

// the pairs of a level of ztrinv hold s x s each: never more than n x n together
static fx_status trinv_workspace(fx_ctx* ctx, Workspace* ws, int n, void** T) {
  *T = nullptr;
  return n <= CB ? FX_OK : ws_get(ctx, ws, "trinv_T", sizeof(z) * (size_t)n * n, T);
}

fx_status chol_workspace(fx_ctx* ctx, Workspace* ws, int n, void** dinv) {
  void* T = nullptr;
  FX_TRY(trinv_workspace(ctx, ws, n, &T));
  return ws_get(ctx, ws, "chol_dinv", sizeof(z) * CB * ((n + CB - 1) / CB * CB), dinv);
}

fx_status zpotrf(fx_ctx* ctx, Workspace* ws, hipStream_t st, int n, void* A, int64_t lda, void* dinv, int* info_dev) {
  z* a = (z*)A;
  for (int k = 0; k < n; k += CB) {
    const int nb = std::min(CB, n - k);
    z* di = (z*)dinv + (int64_t)k * CB;
    hipLaunchKernelGGL(k_potrf_diag, dim3(1), dim3(256), 0, st, n, a, lda, k, di, info_dev);
    FX_LAUNCH_CHECK();
    const int rest = n - k - nb;
    if (rest <= 0) break;
    z* L21 = a + (k + nb) + (int64_t)k * lda;
    z* A22 = a + (k + nb) + (int64_t)(k + nb) * lda;
    // rows below: L21 = A21 L_kk^{-H}, in place (rows are left only below whole blocks)
    hipLaunchKernelGGL(k_potrf_panel, dim3((unsigned)((rest + 15) / 16)), dim3(256), 0, st, n, a, lda, k);
    FX_LAUNCH_CHECK();
    // trailing update A22 -= L21 L21^H, lower part
    FX_TRY(zgemm(ctx, ws, st, 0, 1, rest, rest, nb, z{-1.0, 0.0}, L21, lda, L21, lda, z{1.0, 0.0}, A22, lda, 1, 0,
                 0, 0, 1, ZgShape{kZgHermitian}));
  }
  hipLaunchKernelGGL(k_zero_upper, dim3(std::min(((int64_t)n * n + 255) / 256, (int64_t)4096)), dim3(256), 0, st, n,
                     a, lda);
  FX_LAUNCH_CHECK();
  return FX_OK;
}

// ---------------------------------------------------------------------------
// Inverse of a lower triangular matrix, in place, from the inverses of its CB x
// CB diagonal blocks: neighbouring blocks of s = CB, 2 CB, ... are joined by
// inv([[P, 0], [Q, R]]) = [[inv P, 0], [-inv R Q inv P, inv R]], all pairs of a
// level in one batched product each (two launches per level).
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(256) k_place_diag(int n, z* A, int64_t lda, const z* __restrict__ dinv) {
  const int k = blockIdx.x * CB, nb = min(CB, n - k);
  for (int e = threadIdx.x; e < CB * CB; e += 256) {
    const int i = e % CB, j = e / CB;
    if (i < nb && j < nb) A[(k + i) + (int64_t)(k + j) * lda] = dinv[(int64_t)k * CB + e];
  }
}

fx_status ztrinv(fx_ctx* ctx, Workspace* ws, hipStream_t st, int n, void* Av, int64_t lda, const void* dinv) {
  z* A = (z*)Av;
  hipLaunchKernelGGL(k_place_diag, dim3((n + CB - 1) / CB), dim3(256), 0, st, n, A, lda, (const z*)dinv);
  FX_LAUNCH_CHECK();
  if (n <= CB) return FX_OK;
  void* T = nullptr;
  FX_TRY(trinv_workspace(ctx, ws, n, &T));
  for (int s = CB; s < n; s *= 2) {
    const int pairs = (n - s + 2 * s - 1) / (2 * s);
    const int64_t step = (int64_t)2 * s * (1 + lda);
    // rows of Q and R of pair p: min(s, n - s - 2 s p)
    z* Q = A + s;
    z* R = A + s + (int64_t)s * lda;
    FX_TRY(zgemm(ctx, ws, st, 0, 0, s, s, s, z{1.0, 0.0}, Q, lda, A, lda, z{0.0, 0.0}, T, s, pairs, step, step,
                 (int64_t)s * s, 1, ZgShape{kZgBLower, n - s, 2 * s}));
    FX_TRY(zgemm(ctx, ws, st, 0, 0, s, s, s, z{-1.0, 0.0}, R, lda, T, s, z{0.0, 0.0}, Q, lda, pairs, step,
                 (int64_t)s * s, step, 1, ZgShape{kZgALower, n - s, 2 * s}));
  }
  return FX_OK;
}

fx_status zherm(hipStream_t st, int n, const void* M, int64_t ldm, void* H, void* Aneg, double* ex_dev) {
  hipLaunchKernelGGL(k_herm, dim3(std::min(((int64_t)n * n + 255) / 256, (int64_t)4096)), dim3(256), 0, st, n,
                     (const z*)M, ldm, (z*)H, (z*)Aneg);
  FX_LAUNCH_CHECK();
  if (ex_dev) {
    hipLaunchKernelGGL(k_half_trace, dim3(1), dim3(64), 0, st, n, (const z*)H, ex_dev);
    FX_LAUNCH_CHECK();
  }
  return FX_OK;
}

// X <- X U with U = Linv^H upper triangular.  Columns n0 .. n0 + 63 of the result
// need columns k < n0 + 64 of X only, so the column blocks go from the last to
// the first, and within a launch a workgroup reads only its own 64 rows and
// stores the block after its last read.  Half the products of the square form
// and no second array: at 72^3, 432 columns, product and copy back took 9.3 +
// 1.1 ms.
fx_status zmul_upper_inplace(fx_ctx* ctx, hipStream_t st, int M, int n, void* X, int64_t ldx, const void* Linv,
                             int64_t ldl) {
  using T = ZgTile<2, 2, 2>;
  const auto kern = k_zgemm<0, 1, 2, 2, 2>;
  FX_TRY(allow_dynamic_lds((const void*)kern, T::kLds));
  z* x = (z*)X;
  int slot;
  FX_TRY(prof_begin(ctx, st, FX_K_GEMM_NN, 4.0 * M * (double)n * (n + 1.0), &slot));
  for (int n0 = (n - 1) / T::BN * T::BN; n0 >= 0; n0 -= T::BN) {
    const int nb = std::min(T::BN, n - n0), K = n0 + nb;
    ZgArgs g{M, nb, K, x, ldx, 0, (const z*)Linv + n0, ldl, 0, x + (int64_t)n0 * ldx, ldx, 0, z{1.0, 0.0}, z{0.0, 0.0},
             1, (K + ZK - 1) / ZK * ZK, (M + T::BM - 1) / T::BM, 1, nullptr, ZgShape{}};
    hipLaunchKernelGGL(kern, dim3((unsigned)g.tiles_m), dim3(T::NT), T::kLds, st, g);
    FX_LAUNCH_CHECK();
  }
  FX_TRY(prof_end(ctx, st, slot));
  return FX_OK;
}

}  // namespace fx
