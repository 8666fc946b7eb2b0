// K_ACE phi = -xi (xi^H phi) on the matrix cores.
//
// Both projections are written as real GEMMs whose two operands are
// contiguous along the reduction dimension ("TN"), on the interleaved
// (re, im) real view of the complex arrays:
//
//   C = xi^H phi  : D (N x 2R) = A B^T, A row m = column m of xi (2 N_r reals),
//                   B row 2n = phi_n, B row 2n+1 = (-i phi_n) = (im, -re) pairs;
//                   Re C(m,n) = D(m, 2n), Im C(m,n) = D(m, 2n+1).  The reduction
//                   (2 N_r long) is split across workgroups; split partial sums
//                   are added in FP64 in a fixed order.
//   y = -xi C     : D (N_r x 2R) = A B^T, A row r = row r of xi (2 N reals),
//                   B row 2n = (Re C, -Im C) pairs, B row 2n+1 = (Im C, Re C);
//                   y(r,n) = -(D(r,2n), D(r,2n+1)).
//
// Precision forms: every operand X is split as X_p = round(X) and
// r_X = round(X - X_p) (FP32, BF16 or FP16), and with the residual step the
// GEMM computes A_p B_p (main accumulator) and A_p r_B + r_A B_p (correction
// accumulator), both in FP32 on the matrix cores, added in FP64 at the end.
// FP16 operands are scaled by powers of two first (xi by one factor, each
// right-hand side and each column of C by its own) so that the largest
// magnitude lands in [2^13, 2^14): the 11-bit significand then holds the
// values and their residuals without overflow or loss to subnormals, and the
// exact power-of-two factors are divided out in FP64 afterwards.
#include <algorithm>
#include <cstdint>
#include <type_traits>

#include "fft.hpp"
#include "item_map.hpp"
#include "mfma_gemm.hpp"
#include "vx.hpp"

namespace fx {

typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef _Float16 halfx8 __attribute__((ext_vector_type(8)));

// ---- rounding ---------------------------------------------------------------
// float -> bfloat16, round to nearest even (NaN kept quiet)
__device__ inline uint16_t f2bf(float f) {
  uint32_t u = __float_as_uint(f);
  if ((u & 0x7fffffffu) > 0x7f800000u) return (uint16_t)((u >> 16) | 0x40u);
  u += 0x7fffu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}
__device__ inline float bf2f(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

template <typename S>
struct Prec;
template <>
struct Prec<float> {
  static constexpr int BK = 32;   // K elements per tile step (128 bytes per row)
  static constexpr int PAD = 4;   // LDS row padding (elements)
  __device__ static float round(double x) { return (float)x; }
  __device__ static double widen(float s) { return (double)s; }
  __device__ static float round_f(float x) { return x; }
  __device__ static float widen_f(float s) { return s; }
};
template <>
struct Prec<uint16_t> {
  static constexpr int BK = 64;
  static constexpr int PAD = 8;
  __device__ static uint16_t round(double x) { return f2bf((float)x); }
  __device__ static double widen(uint16_t s) { return (double)bf2f(s); }
  __device__ static uint16_t round_f(float x) { return f2bf(x); }
  __device__ static float widen_f(uint16_t s) { return bf2f(s); }
};

template <>
struct Prec<_Float16> {
  static constexpr int BK = 64;
  static constexpr int PAD = 8;
  __device__ static _Float16 round(double x) { return (_Float16)x; }
  __device__ static double widen(_Float16 s) { return (double)s; }
  __device__ static _Float16 round_f(float x) { return (_Float16)x; }
  __device__ static float widen_f(_Float16 s) { return (float)s; }
};

// Power-of-two factor that takes a largest magnitude m (as FP32 bits; m >= 0)
// into [2^13, 2^14); 1 for the FP32 and BF16 forms (no maxima) and for m = 0.
__device__ inline double scale_of(const unsigned* maxbits, int i) {
  if (!maxbits) return 1.0;
  const float m = __uint_as_float(maxbits[i]);
  if (!(m > 0.f) || !isfinite(m)) return 1.0;
  int e = 0;
  (void)frexpf(m, &e);  // m = f 2^e, f in [0.5, 1)
  return ldexp(1.0, 14 - e);
}

// Largest |x| of each column (per_col) or of all columns, as FP32 bits
// (monotone for non-negative floats, so an integer max merges blocks);
// `out` must hold zeros first.  x: complex columns of nr values, column c at
// x + c * ld.  Read-bound: four complex loads in flight per thread, and blocks
// of at most 2048 values (with 32768, the 8 columns of a request at 48^3 ran in
// 32 workgroups, 55 us).
template <typename T>
__global__ void __launch_bounds__(256) k_absmax(const cpx<T>* __restrict__ x, int64_t ld, int64_t nr, int per_col,
                                                unsigned* __restrict__ out) {
  __shared__ float red[4];
  const int c = blockIdx.y;
  const cpx<T>* col = x + (int64_t)c * ld;
  float m = 0.f;
  const int64_t step = (int64_t)gridDim.x * 256;
  for (int64_t i0 = blockIdx.x * (int64_t)256 + threadIdx.x; i0 < nr; i0 += 4 * step) {
    cpx<T> v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) v[u] = col[i0 + u * step < nr ? i0 + u * step : i0];
#pragma unroll
    for (int u = 0; u < 4; ++u) m = fmaxf(m, fmaxf((float)fabs((double)v[u].x), (float)fabs((double)v[u].y)));
  }
  for (int w = 32; w > 0; w >>= 1) m = fmaxf(m, __shfl_xor(m, w));
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = m;
  __syncthreads();
  if (threadIdx.x == 0)
    atomicMax(out + (per_col ? c : 0), __float_as_uint(fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]))));
}
static unsigned absmax_blocks(int64_t nr, int cols) {
  return (unsigned)std::max<int64_t>(1, std::min<int64_t>((nr + 2047) / 2048, std::max(1, 8192 / cols)));
}

__global__ void k_zero_u32(unsigned* __restrict__ p, int n) {
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) p[i] = 0u;
}

constexpr int KPAD = 64;  // reduction dims of split arrays are padded to this
static int64_t roundk(int64_t k) { return (k + KPAD - 1) / KPAD * KPAD; }

// (a, b) pairs -> (b, -a) on a 16-byte vector: multiplication by -i of the
// complex values it holds.
__device__ inline uint4 times_minus_i(uint4 v, int elem_bytes) {
  if (elem_bytes == 4) {
    return uint4{v.y, v.x ^ 0x80000000u, v.w, v.z ^ 0x80000000u};
  }
  // bf16: 4 pairs, each 32-bit word holds (lo = a, hi = b)
  uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const uint32_t a = w[i] & 0xffffu, b = w[i] >> 16;
    w[i] = b | ((a ^ 0x8000u) << 16);
  }
  return uint4{w[0], w[1], w[2], w[3]};
}

// ---------------------------------------------------------------------------
// TN GEMM on matrix cores, FP32 operands (k_tn_pair takes the 2-byte types).
// 256 threads = 4 waves in a 2x2 arrangement, each wave a 64x64 block of D made
// of 2x2 MFMA 32x32 tiles.  Workgroup tile 128 x 128, K step BK.  Held to two
// waves per SIMD (accumulators in the unified register file), so that two
// workgroups share a CU and one's barriers and loads overlap the other's matrix
// work: at 96^3, N = R = 1024 this took the products with the residual from
// 67-68% to 73-82% of the FP32 peak (the output product spills a few registers).
//   A: rows m (M of them), A[m*lda + k];  B: rows n (N of them), B[n*ldb + k].
//   BDOUBLE: B holds N/2 source rows; LDS row 2c is source row c and row
//            2c+1 is source row c times -i (see header comment).
//   MODE 0: write FP64 partial sums, partial[(split*M + m)*N + n].
//   MODE 1: write y(r=m, n/2) component n&1 = -alpha * D to a complex output.
// ---------------------------------------------------------------------------
constexpr int TBM = 128, TBN = 128;

// Order of a wave's own LDS accesses across lanes: the wave's LDS
// instructions execute in issue order, so only the compiler has to be kept
// from moving accesses across this point.
__device__ inline void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Epilogue of the TN GEMM kernels: D tile element e of MFMA tile (i, j) of a
// wave is row i*32 + 8*(e/4) + 4*(lane/32) + e%4, column j*32 + lane%32 of the
// wave's 64x64 block.  MODE 0 writes FP64 partial sums; MODE 1 turns each
// 32x32 tile around in the wave's own 32 x 33 doubles of `smem_raw` (the
// caller's LDS, idle by then) and writes y = -alpha * D along r.
template <bool REFINE, int MODE>
__device__ inline void tn_epilogue(floatx16 (&acc)[2][2], floatx16 (&cor)[2][2], unsigned char* smem_raw, int lane,
                                   int wave, int wm, int wn, int m0, int n0, int M, int N, int split,
                                   double* __restrict__ partial, void* __restrict__ out, int64_t ldo, int out_c64,
                                   double alpha, const double* __restrict__ colalpha) {
  if (MODE == 0) {
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const int n = n0 + wn * 64 + j * 32 + (lane & 31);
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          const int m = m0 + wm * 64 + i * 32 + 8 * (e >> 2) + 4 * (lane >> 5) + (e & 3);
          if (m >= M || n >= N) continue;
          partial[((int64_t)split * M + m) * N + n] = (double)acc[i][j][e] + (REFINE ? (double)cor[i][j][e] : 0.0);
        }
      }
    return;
  }
  // MODE 1: the output runs along m (r) for each target, the tile along n:
  // each wave turns its 32x32 tiles around in its own slice of the (now idle)
  // LDS, then writes 32 consecutive r of one target per half-wave.
  constexpr int SL = 33;  // padded row of the staged tile (doubles)
  double* stg = reinterpret_cast<double*>(smem_raw) + wave * 32 * SL;
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) {
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const int ml = 8 * (e >> 2) + 4 * (lane >> 5) + (e & 3);
        stg[ml * SL + (lane & 31)] = (double)acc[i][j][e] + (REFINE ? (double)cor[i][j][e] : 0.0);
      }
      wave_lds_sync();
      const int ml = lane & 31;
      const int m = m0 + wm * 64 + i * 32 + ml;
#pragma unroll
      for (int it = 0; it < 8; ++it) {
        const int tl = (lane >> 5) + 2 * it;  // target within the tile's 16
        const int n = n0 + wn * 64 + j * 32 + 2 * tl;
        const double re = stg[ml * SL + 2 * tl], im = stg[ml * SL + 2 * tl + 1];
        if (m < M && n < N) {
          const int64_t idx = (int64_t)(n >> 1) * ldo + m;
          const double al = colalpha ? colalpha[n >> 1] : alpha;
          if (out_c64)
            reinterpret_cast<float2*>(out)[idx] = make_float2((float)(-al * re), (float)(-al * im));
          else
            reinterpret_cast<double2*>(out)[idx] = make_double2(-al * re, -al * im);
        }
      }
      wave_lds_sync();
    }
}

template <typename S, bool REFINE, bool BDOUBLE, int MODE>
__global__ void __launch_bounds__(256, 2) k_tn_mfma(int M, int N, int K, int kchunk, const S* __restrict__ Ap,
                                                 const S* __restrict__ Ar, int64_t lda, const S* __restrict__ Bp,
                                                 const S* __restrict__ Br, int64_t ldb, double* __restrict__ partial,
                                                 void* __restrict__ out, int64_t ldo, int out_c64, double alpha,
                                                 const double* __restrict__ colalpha, int tiles_m, int tiles_n) {
  static_assert(sizeof(S) == 4, "FP32 operands");
  constexpr int BK = Prec<S>::BK;
  constexpr int LDK = BK + Prec<S>::PAD;
  constexpr int EPV = 16 / sizeof(S);  // elements per 16-byte vector
  constexpr int VPR = BK / EPV;        // vectors per tile row (8)
  constexpr int NT = REFINE ? 4 : 2;
  extern __shared__ __align__(16) unsigned char smem_raw[];
  S* sm = reinterpret_cast<S*>(smem_raw);
  S* sAp = sm;
  S* sBp = sm + TBM * LDK;
  S* sAr = sm + 2 * TBM * LDK;
  S* sBr = sm + 3 * TBM * LDK;

  const int lid = xcd_run(gridDim.x, blockIdx.x);  // n tiles fastest, then m, then splits
  const int tn = lid % tiles_n;
  const int rest = lid / tiles_n;
  const int tm = rest % tiles_m;
  const int split = rest / tiles_m;
  const int m0 = tm * TBM, n0 = tn * TBN;
  const int kbeg = split * kchunk;
  const int kend = min(K, kbeg + kchunk);

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave & 1, wn = wave >> 1;

  floatx16 acc[2][2], cor[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) {
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        acc[i][j][e] = 0.f;
        cor[i][j][e] = 0.f;
      }
    }

  // register staging of one K step: 4 vectors per thread per A tile; B tile
  // rows: 128 (plain) or 64 source rows (BDOUBLE, 2 vectors per thread)
  constexpr int BV = BDOUBLE ? 2 : 4;
  uint4 ra[2][4], rb[2][BV];
  // rows past the edge load a clamped (valid) row and are zeroed by value,
  // so the loads need no branches
  auto zsel = [](uint4 v, bool keep) __attribute__((always_inline)) {
    return uint4{keep ? v.x : 0u, keep ? v.y : 0u, keep ? v.z : 0u, keep ? v.w : 0u};
  };
  auto gload = [&](int k0) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int v = tid + 256 * u, row = v / VPR, c = v % VPR;
      const int m = m0 + row;
      const int mc = m < M ? m : M - 1;
      const int64_t off = (int64_t)mc * lda + k0 + c * EPV;
      ra[0][u] = zsel(*reinterpret_cast<const uint4*>(Ap + off), m < M);
      if (REFINE) ra[1][u] = zsel(*reinterpret_cast<const uint4*>(Ar + off), m < M);
    }
#pragma unroll
    for (int u = 0; u < BV; ++u) {
      const int v = tid + 256 * u, row = v / VPR, c = v % VPR;
      const int n = BDOUBLE ? n0 / 2 + row : n0 + row;
      const int nlim = BDOUBLE ? N / 2 : N;
      const int nc = n < nlim ? n : nlim - 1;
      const int64_t off = (int64_t)nc * ldb + k0 + c * EPV;
      rb[0][u] = zsel(*reinterpret_cast<const uint4*>(Bp + off), n < nlim);
      if (REFINE) rb[1][u] = zsel(*reinterpret_cast<const uint4*>(Br + off), n < nlim);
    }
  };
  auto sstore = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int v = tid + 256 * u, row = v / VPR, c = v % VPR;
      *reinterpret_cast<uint4*>(sAp + row * LDK + c * EPV) = ra[0][u];
      if (REFINE) *reinterpret_cast<uint4*>(sAr + row * LDK + c * EPV) = ra[1][u];
    }
#pragma unroll
    for (int u = 0; u < BV; ++u) {
      const int v = tid + 256 * u, row = v / VPR, c = v % VPR;
      if (BDOUBLE) {
        *reinterpret_cast<uint4*>(sBp + (2 * row) * LDK + c * EPV) = rb[0][u];
        *reinterpret_cast<uint4*>(sBp + (2 * row + 1) * LDK + c * EPV) = times_minus_i(rb[0][u], sizeof(S));
        if (REFINE) {
          *reinterpret_cast<uint4*>(sBr + (2 * row) * LDK + c * EPV) = rb[1][u];
          *reinterpret_cast<uint4*>(sBr + (2 * row + 1) * LDK + c * EPV) = times_minus_i(rb[1][u], sizeof(S));
        }
      } else {
        *reinterpret_cast<uint4*>(sBp + row * LDK + c * EPV) = rb[0][u];
        if (REFINE) *reinterpret_cast<uint4*>(sBr + row * LDK + c * EPV) = rb[1][u];
      }
    }
  };

  if (kbeg < kend) gload(kbeg);
  for (int k0 = kbeg; k0 < kend; k0 += BK) {
    sstore();
    __syncthreads();
    if (k0 + BK < kend) gload(k0 + BK);
    const int ar = wm * 64 + (lane & 31);
    const int br = wn * 64 + (lane & 31);
    // MFMA u of group q takes k = 4q + u (lanes 0-31) and BK/2 + 4q + u
    // (lanes 32-63): any order of the step's k terms gives the same sum up
    // to rounding, and this one lets each lane fetch the operands of four
    // MFMAs with one 16-byte LDS read (rows 36 floats apart fill the 32
    // banks in each group of 8 lanes; 4-byte reads of 32 rows did not)
#pragma unroll
    for (int q = 0; q < BK / 8; ++q) {
      const int kc = (lane >> 5) * (BK / 2) + 4 * q;
      float4 a[2], b[2], a2[2], b2[2];
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        a[t] = *reinterpret_cast<const float4*>(reinterpret_cast<const float*>(sAp) + (ar + 32 * t) * LDK + kc);
        b[t] = *reinterpret_cast<const float4*>(reinterpret_cast<const float*>(sBp) + (br + 32 * t) * LDK + kc);
        if (REFINE) {
          a2[t] = *reinterpret_cast<const float4*>(reinterpret_cast<const float*>(sAr) + (ar + 32 * t) * LDK + kc);
          b2[t] = *reinterpret_cast<const float4*>(reinterpret_cast<const float*>(sBr) + (br + 32 * t) * LDK + kc);
        }
      }
#pragma unroll
      for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int j = 0; j < 2; ++j) {
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[i][u], b[j][u], acc[i][j], 0, 0, 0);
            if (REFINE) {
              cor[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[i][u], b2[j][u], cor[i][j], 0, 0, 0);
              cor[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(a2[i][u], b[j][u], cor[i][j], 0, 0, 0);
            }
          }
    }
    __syncthreads();
  }

  tn_epilogue<REFINE, MODE>(acc, cor, smem_raw, lane, wave, wm, wn, m0, n0, M, N, split, partial, out, ldo, out_c64,
                            alpha, colalpha);
}

// ---------------------------------------------------------------------------
// The TN GEMM for the 2-byte operand types (BF16, FP16), real and imaginary
// part of a right-hand side together.  256 threads = 4 waves, 2 x 2; workgroup
// tile 128 rows of A by 64 right-hand sides, a wave 64 by 32.  Only the source
// rows of B (row ldb * c of right-hand side c) are stored and read: the second
// column tile of a wave multiplies the same fragments turned in registers,
// (a, b) -> (b, -a) in MODE 0 and (-b, a) in MODE 1, so that tile j = 0 holds
// the real and j = 1 the imaginary parts, lane by lane.
// Per K step of 64 a wave has 48 matrix instructions (1540 cycles) and reads 24
// fragments (32 with both parts stored), one 16-deep slice ahead of their use;
// the next step's tiles are loaded into registers meanwhile, and two workgroups
// a CU cover each other's barriers.  (Tiles loaded straight to LDS instead need
// all fragments of a step in registers first, since an LDS read waits for such
// loads: with steps of 64 they spill, with 32 the loads have too little time.)
// A tile row is 128 bytes, eight 16-byte chunks without padding; row r keeps
// global chunk g in slot g ^ ((r >> 1) & 7), so that the reads of 16
// consecutive rows fall on distinct banks.  Waves whose rows or right-hand
// sides are all past the edge load, but multiply nothing (432 factors fill 3.4
// row tiles).
//   MODE 0: FP64 partial sums, partial[(split*M + m)*N + 2c], + 1 (as a pair).
//   MODE 1: y(r = m, c) = -colalpha[c] D.
// The k terms of an element run in order, 16 per matrix instruction, as in
// k_tn_skinny.
// What bounds it now is the chip's power: 432 factors and right-hand sides at
// 72^3 in FP16 with the residual, first product 2627 -> 2053 us, output product
// 2423 -> 1766 (875 and 1020 TFLOP/s executed; a large library product in BF16
// reaches 1190).  The last 11% of cycles saved went into a lower clock (1.92 ->
// 1.83 GHz).  Without the residual 1250 -> 704 and 1010 -> 739 us.
// ---------------------------------------------------------------------------
constexpr int PBK = 64, PROWB = 128;                     // K step: elements, bytes of a row
constexpr int kPairA = TBM * PROWB, kPairB = 64 * PROWB;  // one operand tile

template <bool REFINE>
constexpr size_t pair_lds_bytes() {
  return std::max<size_t>((size_t)(REFINE ? 2 : 1) * (kPairA + kPairB), (size_t)4 * 16 * 33 * sizeof(double2));
}

template <typename S>
__device__ inline floatx16 mfma16(u32x4 a, u32x4 b, floatx16 c) {
  if constexpr (std::is_same<S, _Float16>::value)
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(halfx8, a), __builtin_bit_cast(halfx8, b), c, 0,
                                                  0, 0);
  else
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0,
                                                   0, 0);
}

template <typename S, bool REFINE, int MODE>
__global__ void __launch_bounds__(256, 2) k_tn_pair(int M, int R, int K, int kchunk, const S* __restrict__ Ap,
                                                    const S* __restrict__ Ar, int64_t lda, const S* __restrict__ Bp,
                                                    const S* __restrict__ Br, int64_t ldb,
                                                    double* __restrict__ partial, void* __restrict__ out, int64_t ldo,
                                                    int out_c64, const double* __restrict__ colalpha, int tiles_m,
                                                    int tiles_n) {
  static_assert(sizeof(S) == 2, "2-byte operands");
  constexpr int NOPS = REFINE ? 2 : 1;
  extern __shared__ __align__(16) unsigned char smem_raw[];
  unsigned char* tA = smem_raw;
  unsigned char* tB = smem_raw + NOPS * kPairA;

  const int lid = xcd_run(gridDim.x, blockIdx.x);  // n tiles fastest, then m, then splits
  const int tn = lid % tiles_n, rest = lid / tiles_n;
  const int tm = rest % tiles_m, split = rest / tiles_m;
  const int m0 = tm * TBM, c0 = tn * 64;
  const int kbeg = split * kchunk, kend = min(K, kbeg + kchunk);

  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave & 1, wn = wave >> 1;
  const int half = lane >> 5, l32 = lane & 31;
  // nothing of this wave's tile is part of the output
  const bool idle = c0 + wn * 32 >= R || m0 + wm * 64 >= M;

  floatx16 acc[2][2], cor[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        acc[i][j][e] = 0.f;
        cor[i][j][e] = 0.f;
      }

  // each wave instruction fills 1 KB (8 rows): lane l lands in row l / 8, slot
  // l % 8 of it.  Rows past the edge load a clamped, valid row: they only reach
  // outputs that are not written.
  // (byte offsets within a tile: rows are at most 2 * 96^3 elements, so 32 bits hold them)
  uint32_t offa[4], offb[2];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int row = (wave + 4 * q) * 8 + (lane >> 3), slot = (lane & 7) ^ ((row >> 1) & 7);
    offa[q] = (uint32_t)min(row, M - 1 - m0) * (uint32_t)lda * 2u + slot * 16u;
    if (q < 2) offb[q] = (uint32_t)min(row, R - 1 - c0) * (uint32_t)ldb * 2u + slot * 16u;
  }
  // (buffer addressing: one offset register per row instead of a 64-bit pointer
  // per row and operand)
  const auto rsrc = [](const S* base) __attribute__((always_inline)) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<S*>(base), 0, 0xffffffff, 0x00027000);
  };
  const __amdgpu_buffer_rsrc_t gA[2] = {rsrc(Ap + (int64_t)m0 * lda), rsrc((REFINE ? Ar : Ap) + (int64_t)m0 * lda)};
  const __amdgpu_buffer_rsrc_t gB[2] = {rsrc(Bp + (int64_t)c0 * ldb), rsrc((REFINE ? Br : Bp) + (int64_t)c0 * ldb)};
  u32x4 ra[NOPS][4], rb[NOPS][2];
  const auto gload = [&](int k0) __attribute__((always_inline)) {
#pragma unroll
    for (int o = 0; o < NOPS; ++o) {
#pragma unroll
      for (int q = 0; q < 4; ++q) ra[o][q] = __builtin_amdgcn_raw_buffer_load_b128(gA[o], offa[q], k0 * 2, 0);
#pragma unroll
      for (int q = 0; q < 2; ++q) rb[o][q] = __builtin_amdgcn_raw_buffer_load_b128(gB[o], offb[q], k0 * 2, 0);
    }
  };
  const auto sstore = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int o = 0; o < NOPS; ++o) {
#pragma unroll
      for (int q = 0; q < 4; ++q)
        *reinterpret_cast<u32x4*>(tA + o * kPairA + (wave + 4 * q) * 1024 + lane * 16) = ra[o][q];
#pragma unroll
      for (int q = 0; q < 2; ++q)
        *reinterpret_cast<u32x4*>(tB + o * kPairB + (wave + 4 * q) * 1024 + lane * 16) = rb[o][q];
    }
  };
  const auto frag = [&](const unsigned char* t, int row, int g) __attribute__((always_inline)) {
    return *reinterpret_cast<const u32x4*>(t + row * PROWB + ((g ^ ((row >> 1) & 7)) << 4));
  };
  const auto turned = [](u32x4 v) __attribute__((always_inline)) {
    constexpr uint32_t sign = MODE == 0 ? 0x80000000u : 0x8000u;
    return (v << 16 | v >> 16) ^ sign;
  };

  if (kbeg < kend) gload(kbeg);
  for (int k0 = kbeg; idle && k0 < kend; k0 += PBK) {
    sstore();
    __syncthreads();
    if (k0 + PBK < kend) gload(k0 + PBK);
    __syncthreads();
  }
  u32x4 a[2][2][NOPS], b[2][NOPS];  // [kk & 1]: fragments, read one 16-deep slice ahead
  const auto fread = [&](int kk) __attribute__((always_inline)) {
#pragma unroll
    for (int o = 0; o < NOPS; ++o) {
      b[kk & 1][o] = frag(tB + o * kPairB, wn * 32 + l32, kk * 2 + half);
#pragma unroll
      for (int i = 0; i < 2; ++i)
        a[kk & 1][i][o] = frag(tA + o * kPairA, wm * 64 + 32 * i + l32, kk * 2 + half);
    }
  };
  for (int k0 = kbeg; !idle && k0 < kend; k0 += PBK) {
    sstore();
    __syncthreads();
    fread(0);
    if (k0 + PBK < kend) gload(k0 + PBK);
#pragma unroll
    for (int kk = 0; kk < PBK / 16; ++kk) {
      if (kk + 1 < PBK / 16) fread(kk + 1);
      __builtin_amdgcn_sched_barrier(0);
      const int f = kk & 1;
      u32x4 bt[NOPS];
#pragma unroll
      for (int o = 0; o < NOPS; ++o) bt[o] = turned(b[f][o]);
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        acc[i][0] = mfma16<S>(a[f][i][0], b[f][0], acc[i][0]);
        if constexpr (REFINE) cor[i][0] = mfma16<S>(a[f][i][0], b[f][1], cor[i][0]);
      }
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        acc[i][1] = mfma16<S>(a[f][i][0], bt[0], acc[i][1]);
        if constexpr (REFINE) cor[i][1] = mfma16<S>(a[f][i][0], bt[1], cor[i][1]);
      }
      if constexpr (REFINE) {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          cor[i][0] = mfma16<S>(a[f][i][1], b[f][0], cor[i][0]);
          cor[i][1] = mfma16<S>(a[f][i][1], bt[0], cor[i][1]);
        }
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    __syncthreads();
  }

  const int c = c0 + wn * 32 + l32;
  const auto value = [&](int i, int j, int e) __attribute__((always_inline)) {
    return (double)acc[i][j][e] + (REFINE ? (double)cor[i][j][e] : 0.0);
  };
  if (MODE == 0) {
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const int m = m0 + wm * 64 + i * 32 + 8 * (e >> 2) + 4 * half + (e & 3);
        if (m < M && c < R)
          *reinterpret_cast<double2*>(partial + (((int64_t)split * M + m) * R + c) * 2) =
              double2{value(i, 0, e), value(i, 1, e)};
      }
    return;
  }
  // the output runs along m (r) for each target: each wave turns its tiles
  // around, 16 rows at a time, in its own slice of the (now idle) LDS
  const double al = c < R ? (colalpha ? colalpha[c] : 1.0) : 0.0;
  double2* stg = reinterpret_cast<double2*>(smem_raw) + wave * 16 * 33;
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int h = 0; h < 2; ++h) {
#pragma unroll
      for (int e = 8 * h; e < 8 * h + 8; ++e)
        stg[(8 * ((e >> 2) & 1) + 4 * half + (e & 3)) * 33 + l32] = double2{-al * value(i, 0, e), -al * value(i, 1, e)};
      wave_lds_sync();
      const int ml = lane & 15, m = m0 + wm * 64 + i * 32 + 16 * h + ml;
#pragma unroll
      for (int it = 0; it < 8; ++it) {
        const int tl = (lane >> 4) + 4 * it, t = c0 + wn * 32 + tl;
        const double2 v = stg[ml * 33 + tl];
        if (m < M && t < R) {
          const int64_t idx = (int64_t)t * ldo + m;
          if (out_c64)
            reinterpret_cast<float2*>(out)[idx] = make_float2((float)v.x, (float)v.y);
          else
            reinterpret_cast<double2*>(out)[idx] = v;
        }
      }
      wave_lds_sync();
    }
}

// ---------------------------------------------------------------------------
// The TN GEMM for few right-hand sides (N <= 64 real columns): one wave per 32
// rows of A, no LDS and no barrier.  Such a product is bound by reading A (xi
// in p and r form: 113 MB at 48^3, 128 factors); in 128 x 128 tiles seven
// eighths of the matrix work is padding and 128 workgroups with two barriers
// per step leave half the chip idle (70 us for 8 right-hand sides, 1.6 TB/s).
// Each lane reads its operands straight from memory: the four 16-byte pieces
// of a step of row l % 32 that lane l multiplies (of p and of r), so a wave
// uses whole 128-byte lines over a step, A three steps ahead (one for two
// column tiles and for the short reductions of MODE 1), B, a few rows in L2,
// one.  CT: 32-wide column tiles (1 or 2).
// The k terms of an element run in the order of the tile kernels (k_tn_mfma in
// FP32, k_tn_pair in the 2-byte types) over the same split
// chunks, so a right-hand side's bits do not depend on which kernel ran.
// MODE 0 as theirs.  MODE 1 gives the matrix instruction B as its rows: lane
// l then holds y(r = l % 32) of several targets, and stores run along r.
// ---------------------------------------------------------------------------
template <typename S>
__device__ inline floatx16 mfma_vec(uint4 a, uint4 b, floatx16 c) {
  if constexpr (std::is_same<S, float>::value) {
    const float4 x = __builtin_bit_cast(float4, a), y = __builtin_bit_cast(float4, b);
    c = __builtin_amdgcn_mfma_f32_32x32x2f32(x.x, y.x, c, 0, 0, 0);
    c = __builtin_amdgcn_mfma_f32_32x32x2f32(x.y, y.y, c, 0, 0, 0);
    c = __builtin_amdgcn_mfma_f32_32x32x2f32(x.z, y.z, c, 0, 0, 0);
    return __builtin_amdgcn_mfma_f32_32x32x2f32(x.w, y.w, c, 0, 0, 0);
  } else {
    return mfma16<S>(__builtin_bit_cast(u32x4, a), __builtin_bit_cast(u32x4, b), c);
  }
}

template <typename S, bool REFINE, bool BDOUBLE, int MODE, int CT>
__global__ void __launch_bounds__(64, (MODE == 1 ? 3 : 2)) k_tn_skinny(int M, int N, int kchunk, int K, const S* __restrict__ Ap,
                                                     const S* __restrict__ Ar, int64_t lda, const S* __restrict__ Bp,
                                                     const S* __restrict__ Br, int64_t ldb,
                                                     double* __restrict__ partial, void* __restrict__ out, int64_t ldo,
                                                     int out_c64, const double* __restrict__ colalpha, int tiles_m) {
  constexpr int BK = Prec<S>::BK;  // 128 bytes of a row
  constexpr int DA = CT == 1 && MODE == 0 ? 4 : 2;  // A buffers: steps in flight plus one
  const int lane = threadIdx.x, l32 = lane & 31, half = lane >> 5;
  const int tm = blockIdx.x % tiles_m, split = blockIdx.x / tiles_m;
  const int m0 = tm * 32;
  const int kbeg = split * kchunk, kend = min(K, kbeg + kchunk);
  // piece v of a step: bytes [off(v), off(v) + 16) of the row's 128 (the tile
  // kernels' lane layout: 2-byte types k = 16 v + 8 half, FP32 k = 16 half + 4 v)
  const auto off = [half](int v) { return sizeof(S) == 4 ? 16 * half + 4 * v : 16 * v + 8 * half; };
  const int64_t arow = (int64_t)min(m0 + l32, M - 1) * lda;
  const S* ap = Ap + arow;
  const S* ar = Ar + arow;
  const S *bp[CT], *br[CT];
  bool odd[CT];
#pragma unroll
  for (int t = 0; t < CT; ++t) {
    const int n = min(32 * t + l32, N - 1);
    const int64_t row = (int64_t)(BDOUBLE ? n >> 1 : n) * ldb;
    odd[t] = BDOUBLE && (n & 1);
    bp[t] = Bp + row;
    br[t] = Br + row;
  }
  uint4 fa[DA][REFINE ? 8 : 4], fb[2][CT][REFINE ? 8 : 4];
  const auto load_a = [&](int k0, uint4 (&f)[REFINE ? 8 : 4]) __attribute__((always_inline)) {
    const int k = min(k0, kend - BK);  // past the end: a valid step, not used
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      f[v] = *reinterpret_cast<const uint4*>(ap + k + off(v));
      if (REFINE) f[4 + v] = *reinterpret_cast<const uint4*>(ar + k + off(v));
    }
  };
  const auto load_b = [&](int k0, uint4 (&f)[CT][REFINE ? 8 : 4]) __attribute__((always_inline)) {
    const int k = min(k0, kend - BK);
#pragma unroll
    for (int t = 0; t < CT; ++t)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        f[t][v] = *reinterpret_cast<const uint4*>(bp[t] + k + off(v));
        if (REFINE) f[t][4 + v] = *reinterpret_cast<const uint4*>(br[t] + k + off(v));
      }
  };
  const auto turned = [&](uint4 v, bool o) __attribute__((always_inline)) {
    if (!BDOUBLE) return v;
    const uint4 w = times_minus_i(v, sizeof(S));
    return uint4{o ? w.x : v.x, o ? w.y : v.y, o ? w.z : v.z, o ? w.w : v.w};
  };
  floatx16 acc[CT], cor[CT];
#pragma unroll
  for (int t = 0; t < CT; ++t)
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      acc[t][e] = 0.f;
      cor[t][e] = 0.f;
    }
  const auto mul = [&](const uint4& x, const uint4& y, const floatx16& c) __attribute__((always_inline)) {
    return MODE == 0 ? mfma_vec<S>(x, y, c) : mfma_vec<S>(y, x, c);
  };
  const auto step = [&](const uint4 (&a)[REFINE ? 8 : 4], const uint4 (&b)[CT][REFINE ? 8 : 4])
      __attribute__((always_inline)) {
#pragma unroll
    for (int v = 0; v < 4; ++v)
#pragma unroll
      for (int t = 0; t < CT; ++t) {
        const uint4 x = turned(b[t][v], odd[t]);
        if constexpr (REFINE && std::is_same<S, float>::value) {
          // k_tn_mfma interleaves the three products k by k
          const uint4 x2 = turned(b[t][4 + v], odd[t]);
          const float4 fa4 = __builtin_bit_cast(float4, a[v]), fr4 = __builtin_bit_cast(float4, a[4 + v]);
          const float4 fb4 = __builtin_bit_cast(float4, x), fs4 = __builtin_bit_cast(float4, x2);
          const float av[4] = {fa4.x, fa4.y, fa4.z, fa4.w}, rv[4] = {fr4.x, fr4.y, fr4.z, fr4.w};
          const float bv[4] = {fb4.x, fb4.y, fb4.z, fb4.w}, sv[4] = {fs4.x, fs4.y, fs4.z, fs4.w};
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            const auto m = [&](float p, float q, floatx16 c) __attribute__((always_inline)) {
              return MODE == 0 ? __builtin_amdgcn_mfma_f32_32x32x2f32(p, q, c, 0, 0, 0)
                               : __builtin_amdgcn_mfma_f32_32x32x2f32(q, p, c, 0, 0, 0);
            };
            acc[t] = m(av[u], bv[u], acc[t]);
            cor[t] = m(av[u], sv[u], cor[t]);
            cor[t] = m(rv[u], bv[u], cor[t]);
          }
        } else {
          acc[t] = mul(a[v], x, acc[t]);
          if constexpr (REFINE) {
            cor[t] = mul(a[v], turned(b[t][4 + v], odd[t]), cor[t]);
            cor[t] = mul(a[4 + v], x, cor[t]);
          }
        }
      }
  };
  if (kbeg < kend) {
#pragma unroll
    for (int d = 0; d < DA - 1; ++d) load_a(kbeg + d * BK, fa[d]);
    load_b(kbeg, fb[0]);
    // DA steps per round, so that every buffer index is a constant
    for (int k0 = kbeg; k0 < kend; k0 += DA * BK) {
#pragma unroll
      for (int d = 0; d < DA; ++d) {
        load_a(k0 + (d + DA - 1) * BK, fa[(d + DA - 1) % DA]);
        load_b(k0 + (d + 1) * BK, fb[(d + 1) & 1]);
        if (k0 + d * BK < kend) step(fa[d], fb[d & 1]);
      }
    }
  }
  if (MODE == 0) {
#pragma unroll
    for (int t = 0; t < CT; ++t) {
      const int n = 32 * t + l32;
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const int m = m0 + 8 * (e >> 2) + 4 * half + (e & 3);
        if (m < M && n < N)
          partial[((int64_t)split * M + m) * N + n] = (double)acc[t][e] + (REFINE ? (double)cor[t][e] : 0.0);
      }
    }
  } else {
    const int m = m0 + l32;
#pragma unroll
    for (int t = 0; t < CT; ++t)
#pragma unroll
      for (int e = 0; e < 16; e += 2) {
        const int n = 32 * t + 8 * (e >> 2) + 4 * half + (e & 3);
        if (m >= M || n >= N) continue;
        const double re = (double)acc[t][e] + (REFINE ? (double)cor[t][e] : 0.0);
        const double im = (double)acc[t][e + 1] + (REFINE ? (double)cor[t][e + 1] : 0.0);
        const int64_t idx = (int64_t)(n >> 1) * ldo + m;
        const double al = colalpha ? colalpha[n >> 1] : 1.0;
        if (out_c64)
          reinterpret_cast<float2*>(out)[idx] = make_float2((float)(-al * re), (float)(-al * im));
        else
          reinterpret_cast<double2*>(out)[idx] = make_double2(-al * re, -al * im);
      }
  }
}

// ---- split kernels ----------------------------------------------------------
// xi (complex double, N_r x N, ld N_r) -> col form: row m = interleaved column m.
template <typename S>
__global__ void k_split_col(const double* __restrict__ xi, int64_t nr, int n, int64_t kc, S* __restrict__ p,
                            S* __restrict__ r, const unsigned* __restrict__ smax) {
  const int64_t total = (int64_t)n * kc;
  const double sc = scale_of(smax, 0);
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < total; i += (int64_t)gridDim.x * blockDim.x) {
    const int64_t m = i / kc, k = i - m * kc;
    const double v = k < 2 * nr ? sc * xi[m * 2 * nr + k] : 0.0;
    const S hp = Prec<S>::round(v);
    p[i] = hp;
    r[i] = Prec<S>::round(v - Prec<S>::widen(hp));
  }
}

// xi -> row form: row r = interleaved row r of xi (N complex values), padded
// to kn.  64 grid points x 32 orbitals per block through LDS.
template <typename S>
__global__ void __launch_bounds__(256) k_split_row(const double* __restrict__ xi, int64_t nr, int n, int64_t kn,
                                                   S* __restrict__ p, S* __restrict__ r,
                                                   const unsigned* __restrict__ smax) {
  __shared__ double2 t[32][65];
  const double sc = scale_of(smax, 0);
  const int64_t r0 = (int64_t)blockIdx.x * 64;
  const int m0 = blockIdx.y * 32;
  for (int e = threadIdx.x; e < 32 * 64; e += 256) {
    const int mi = e / 64, ri = e % 64;
    const int64_t rr = r0 + ri;
    const int m = m0 + mi;
    double2 v = {0.0, 0.0};
    if (m < n && rr < nr) v = reinterpret_cast<const double2*>(xi)[(int64_t)m * nr + rr];
    t[mi][ri] = v;
  }
  __syncthreads();
  for (int e = threadIdx.x; e < 64 * 64; e += 256) {
    const int ri = e / 64, kk = e % 64;  // kk: position in the 64-wide k window
    const int64_t rr = r0 + ri;
    if (rr >= nr) continue;
    const double2 v = t[kk >> 1][ri];
    const double x = sc * ((kk & 1) ? v.y : v.x);
    const int64_t idx = rr * kn + 2 * (int64_t)m0 + kk;
    const S hp = Prec<S>::round(x);
    p[idx] = hp;
    r[idx] = Prec<S>::round(x - Prec<S>::widen(hp));
  }
}

// phi (complex, ld) -> B source rows: row n = interleaved phi_n, padded to kc.
// Memory-bound; a thread makes one 16-byte vector of each of p and r (one value
// per thread with a 64-bit division each ran at 2.5 TB/s: 1037 us for 432
// columns at 72^3 in FP16).
template <typename S, typename TI>
__device__ inline void split_column(const cpx<TI>* __restrict__ col, int n, int64_t nr, int64_t kc, S* __restrict__ p,
                                    S* __restrict__ r, const unsigned* __restrict__ smax) {
  constexpr int V = 16 / sizeof(S);
  const double sc = scale_of(smax, n);
  // FP32 input: the scaled value and its residual are exact in FP32 (a
  // power-of-two factor that stays finite; X - round(X) of an FP32 X), so the
  // split is the same as in FP64, at FP32 speed
  const bool exact32 = std::is_same<TI, float>::value && sc < 0x1p100;
  for (int64_t k = (blockIdx.x * (int64_t)256 + threadIdx.x) * V; k < kc; k += (int64_t)gridDim.x * 256 * V) {
    alignas(16) S hp[V], hr[V];
#pragma unroll
    for (int u = 0; u < V / 2; ++u) {
      const int64_t i = k / 2 + u;
      const cpx<TI> v = i < nr ? col[i] : cpx<TI>{0, 0};
      const TI xv[2] = {v.x, v.y};
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        if (exact32) {
          const float x = (float)sc * (float)xv[q];
          hp[2 * u + q] = Prec<S>::round_f(x);
          hr[2 * u + q] = Prec<S>::round_f(x - Prec<S>::widen_f(hp[2 * u + q]));
        } else {
          const double x = sc * (double)xv[q];
          hp[2 * u + q] = Prec<S>::round(x);
          hr[2 * u + q] = Prec<S>::round(x - Prec<S>::widen(hp[2 * u + q]));
        }
      }
    }
    *reinterpret_cast<uint4*>(p + n * kc + k) = *reinterpret_cast<const uint4*>(hp);
    *reinterpret_cast<uint4*>(r + n * kc + k) = *reinterpret_cast<const uint4*>(hr);
  }
}
template <typename S, typename TI>
__global__ void __launch_bounds__(256) k_split_phi(const cpx<TI>* __restrict__ phi, int64_t ld, int64_t nr, int R,
                                                   int64_t kc, S* __restrict__ p, S* __restrict__ r,
                                                   const unsigned* __restrict__ smax) {
  for (int n = blockIdx.y; n < R; n += gridDim.y) split_column<S, TI>(phi + (int64_t)n * ld, n, nr, kc, p, r, smax);
}

// Sum of element i over the split partials, partial viewed as [nsplit][count]:
// 16 threads of a block (q = 0 .. 15) add splits q, q + 16, ... of the same
// element in ascending order, then their sums are added in order of q.  Every
// thread of the block must call it; the sum is valid where q == 0.
__device__ inline double2 sum_splits(const double2* __restrict__ partial, int64_t count, int nsplit, int64_t i,
                                     double2 (&red)[16][17]) {
  const int el = threadIdx.x & 15, q = threadIdx.x >> 4;
  double2 s = {0.0, 0.0};
  if (i < count) {
#pragma unroll 4
    for (int t = q; t < nsplit; t += 16) {
      const double2 v = partial[t * count + i];
      s.x += v.x;
      s.y += v.y;
    }
  }
  red[q][el] = s;
  __syncthreads();
  if (q == 0)
    for (int t = 1; t < 16; ++t) {
      s.x += red[t][el].x;
      s.y += red[t][el].y;
    }
  __syncthreads();
  return s;
}
static unsigned sum_blocks(int64_t count) { return (unsigned)std::min<int64_t>((count + 15) / 16, 16384); }

// Fixed-order FP64 sum of the C = xi^H phi split partials, written as the B
// operand of y = -xi C: row 2n = (Re C(k,n), -Im C(k,n)) pairs, row 2n+1 =
// (Im C(k,n), Re C(k,n)) pairs, padded to kn; split p / r.
template <typename S>
__global__ void __launch_bounds__(256) k_reduce_cn(const double2* __restrict__ partial, int nsplit, int n, int R,
                                                   int64_t kn, S* __restrict__ p, S* __restrict__ r) {
  __shared__ double2 red[16][17];
  const int64_t count = (int64_t)n * R;
  // neighbouring elements are neighbouring right-hand sides of the same k; the
  // padding k >= n follows them
  for (int64_t b0 = blockIdx.x * (int64_t)16; b0 < (int64_t)R * (kn / 2); b0 += (int64_t)gridDim.x * 16) {
    const int64_t i = b0 + (threadIdx.x & 15);
    const double2 c = sum_splits(partial, count, nsplit, i, red);
    if (threadIdx.x >= 16 || i >= (int64_t)R * (kn / 2)) continue;
    const int64_t k = i / R, nc = i - k * R;
    const double v[4] = {c.x, -c.y, c.y, c.x};
    const int64_t base0 = (2 * nc) * kn + 2 * k, base1 = (2 * nc + 1) * kn + 2 * k;
    const int64_t idx[4] = {base0, base0 + 1, base1, base1 + 1};
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const S hp = Prec<S>::round(v[q]);
      p[idx[q]] = hp;
      r[idx[q]] = Prec<S>::round(v[q] - Prec<S>::widen(hp));
    }
  }
}

// The same for scaled FP16 operands, in two passes.  First
// C(k, nc) = (fixed-order FP64 sum of the partials) / (s_xi s_nc), exact
// since the factors are powers of two, into an FP64 buffer, with each
// right-hand side's largest magnitude merged into cmax[nc] (zeroed first).
// Then the split of t_nc C with t_nc the power of two of cmax[nc], and
// colalpha[nc] = 1 / (s_xi t_nc) for the epilogue of y = -xi C.
__global__ void __launch_bounds__(256) k_sum_cn_scaled(const double2* __restrict__ partial, int nsplit, int n, int R,
                                                       const unsigned* __restrict__ xmax,
                                                       const unsigned* __restrict__ pmax, double2* __restrict__ c64,
                                                       unsigned* __restrict__ cmax) {
  __shared__ double2 red[16][17];
  const double sx = scale_of(xmax, 0);
  const int64_t count = (int64_t)n * R;
  for (int64_t b0 = blockIdx.x * (int64_t)16; b0 < count; b0 += (int64_t)gridDim.x * 16) {
    const int64_t i = b0 + (threadIdx.x & 15);
    const double2 c = sum_splits(partial, count, nsplit, i, red);
    if (threadIdx.x >= 16 || i >= count) continue;
    const int nc = (int)(i % R);
    const double f = 1.0 / (sx * scale_of(pmax, nc));
    c64[i] = double2{c.x * f, c.y * f};
    atomicMax(cmax + nc, __float_as_uint((float)fmax(fabs(c.x * f), fabs(c.y * f))));
  }
}

template <typename S>
__global__ void k_split_cn_scaled(const double2* __restrict__ c64, int n, int R, int64_t kn,
                                  const unsigned* __restrict__ xmax, const unsigned* __restrict__ cmax,
                                  S* __restrict__ p, S* __restrict__ r, double* __restrict__ colalpha) {
  const double sx = scale_of(xmax, 0);
  const int64_t total = (int64_t)R * (kn / 2);
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < total; i += (int64_t)gridDim.x * blockDim.x) {
    const int64_t nc = i / (kn / 2), k = i - nc * (kn / 2);
    const double t = scale_of(cmax, (int)nc);
    if (k == 0) colalpha[nc] = 1.0 / (sx * t);
    double cr = 0.0, ci = 0.0;
    if (k < n) {
      const double2 c = c64[k * R + nc];
      cr = c.x * t;
      ci = c.y * t;
    }
    const double v[4] = {cr, -ci, ci, cr};
    const int64_t base0 = (2 * nc) * kn + 2 * k, base1 = (2 * nc + 1) * kn + 2 * k;
    const int64_t idx[4] = {base0, base0 + 1, base1, base1 + 1};
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const S hp = Prec<S>::round(v[q]);
      p[idx[q]] = hp;
      r[idx[q]] = Prec<S>::round(v[q] - Prec<S>::widen(hp));
    }
  }
}

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------
// FP16 operands are scaled by powers of two (see the header comment).
template <typename S>
constexpr bool kScaled = std::is_same<S, _Float16>::value;

// workspace names per element size: {phi p, phi r, B p, B r}
template <typename S>
static const char* split_name(int which) {
  static const char* n32[4] = {"mf_phi_p32", "mf_phi_r32", "mf_bnn_p32", "mf_bnn_r32"};
  static const char* n16[4] = {"mf_phi_p16", "mf_phi_r16", "mf_bnn_p16", "mf_bnn_r16"};
  return sizeof(S) == 4 ? n32[which] : n16[which];
}

template <typename K>
static fx_status allow_lds_mfma(K kernel, size_t bytes) {
  return allow_dynamic_lds(reinterpret_cast<const void*>(kernel), bytes);
}

template <typename S>
static fx_status prepare_split_t(fx_ace* a, AceSplit* sp, hipStream_t st) {
  if (sp->ready) return FX_OK;
  const int64_t nr = a->nr;
  const int n = a->n;
  sp->kc = roundk(2 * nr);
  sp->kn = roundk(2 * (int64_t)n);
  const size_t cb = sizeof(S) * (size_t)n * sp->kc, rb = sizeof(S) * (size_t)nr * sp->kn;
  FX_TRY(ace_alloc(a, cb, &sp->col_p));
  FX_TRY(ace_alloc(a, cb, &sp->col_r));
  FX_TRY(ace_alloc(a, rb, &sp->row_p));
  FX_TRY(ace_alloc(a, rb, &sp->row_r));
  const unsigned* smax = nullptr;
  if (kScaled<S>) {
    // one power-of-two factor for all of xi, from its largest magnitude
    FX_TRY(ace_alloc(a, 256, &sp->smax));
    hipLaunchKernelGGL(k_zero_u32, dim3(1), dim3(64), 0, st, (unsigned*)sp->smax, 1);
    FX_LAUNCH_CHECK();
    hipLaunchKernelGGL((k_absmax<double>), dim3(absmax_blocks(nr, n), (unsigned)n), dim3(256), 0, st,
                       (const cpx<double>*)a->xi, nr, nr, 0, (unsigned*)sp->smax);
    FX_LAUNCH_CHECK();
    smax = (const unsigned*)sp->smax;
  }
  const int64_t tc = (int64_t)n * sp->kc;
  hipLaunchKernelGGL((k_split_col<S>), dim3((unsigned)std::min<int64_t>((tc + 255) / 256, 16384)), dim3(256), 0, st,
                     (const double*)a->xi, nr, n, sp->kc, (S*)sp->col_p, (S*)sp->col_r, smax);
  FX_LAUNCH_CHECK();
  hipLaunchKernelGGL((k_split_row<S>), dim3((unsigned)((nr + 63) / 64), (unsigned)(sp->kn / 64)), dim3(256), 0, st,
                     (const double*)a->xi, nr, n, sp->kn, (S*)sp->row_p, (S*)sp->row_r, smax);
  FX_LAUNCH_CHECK();
  sp->ready = true;
  return FX_OK;
}

fx_status ace_prepare_split(fx_ace* a, fx_prec prec, hipStream_t st) {
  if (prec == FX_PREC_ACE_FP32R || prec == FX_PREC_ACE_FP32) return prepare_split_t<float>(a, &a->f32, st);
  if (prec == FX_PREC_ACE_BF16R || prec == FX_PREC_ACE_BF16) return prepare_split_t<uint16_t>(a, &a->b16, st);
  if (prec == FX_PREC_ACE_FP16R || prec == FX_PREC_ACE_FP16) return prepare_split_t<_Float16>(a, &a->f16, st);
  return FX_OK;
}

template <typename S, bool REFINE>
static fx_status apply_t(fx_ctx* ctx, Workspace* ws, fx_ace* a, AceSplit* sp, const void* phi, int R, int64_t ld_phi,
                         void* out, int64_t ld_out, fx_dtype in_dtype, fx_dtype out_dtype, hipStream_t st) {
  constexpr int BK = Prec<S>::BK;
  constexpr int LDK = BK + Prec<S>::PAD;
  const int64_t nr = a->nr;
  const int n = a->n;
  FX_TRY(prepare_split_t<S>(a, sp, st));
  // phi split (FP16: each right-hand side scaled by its own power of two)
  void *php = nullptr, *phr = nullptr;
  const size_t pb = sizeof(S) * (size_t)R * sp->kc;
  FX_TRY(ws_get(ctx, ws, split_name<S>(0), pb, &php));
  FX_TRY(ws_get(ctx, ws, split_name<S>(1), pb, &phr));
  unsigned *pmax = nullptr, *cmax = nullptr;
  double* colalpha = nullptr;
  if (kScaled<S>) {
    void* t = nullptr;
    // largest magnitudes: R of phi, then R of C
    FX_TRY(ws_get(ctx, ws, "mf_phimax", 2 * sizeof(unsigned) * (size_t)R, &t));
    pmax = (unsigned*)t;
    cmax = pmax + R;
    FX_TRY(ws_get(ctx, ws, "mf_colalpha", sizeof(double) * (size_t)R, &t));
    colalpha = (double*)t;
    hipLaunchKernelGGL(k_zero_u32, dim3((unsigned)std::min(64, (2 * R + 255) / 256)), dim3(256), 0, st, pmax, 2 * R);
    FX_LAUNCH_CHECK();
    const dim3 g(absmax_blocks(nr, R), (unsigned)R);
    if (in_dtype == FX_C128)
      hipLaunchKernelGGL((k_absmax<double>), g, dim3(256), 0, st, (const cpx<double>*)phi, ld_phi, nr, 1, pmax);
    else
      hipLaunchKernelGGL((k_absmax<float>), g, dim3(256), 0, st, (const cpx<float>*)phi, ld_phi, nr, 1, pmax);
    FX_LAUNCH_CHECK();
  }
  int slot;
  FX_TRY(prof_begin(ctx, st, FX_K_SPLIT, (double)R * nr * (in_dtype == FX_C128 ? 16 : 8) + 2.0 * pb, &slot));
  {
    constexpr int64_t kPerBlock = 256 * (16 / sizeof(S));
    const dim3 g((unsigned)std::min<int64_t>((sp->kc + kPerBlock - 1) / kPerBlock, 4096),
                 (unsigned)std::min(R, 32768));
    if (in_dtype == FX_C128)
      hipLaunchKernelGGL((k_split_phi<S, double>), g, dim3(256), 0, st, (const cpx<double>*)phi, ld_phi, nr, R, sp->kc,
                         (S*)php, (S*)phr, (const unsigned*)pmax);
    else
      hipLaunchKernelGGL((k_split_phi<S, float>), g, dim3(256), 0, st, (const cpx<float>*)phi, ld_phi, nr, R, sp->kc,
                         (S*)php, (S*)phr, (const unsigned*)pmax);
  }
  FX_LAUNCH_CHECK();
  FX_TRY(prof_end(ctx, st, slot));

  [[maybe_unused]] const size_t lds = (size_t)(REFINE ? 4 : 2) * TBM * LDK * sizeof(S);
  // C = xi^H phi: M = n, N = 2R, K = kc, split over K
  {
    const int tiles_m = (n + TBM - 1) / TBM, tiles_n = (2 * R + TBN - 1) / TBN;
    const int tiles = tiles_m * tiles_n;
    const int64_t ksteps = sp->kc / BK;
    // the split depends on the reduction length only, so a column's result
    // does not depend on how many right-hand sides share the launch
    // (up to 128 chunks of at least 16 steps: enough workgroups for a few
    // right-hand sides, where the output has only a handful of tiles)
    int nsplit = (int)std::max<int64_t>(1, std::min<int64_t>(128, ksteps / 16));
    if (const char* e = getenv("FX_ACE_NSPLIT")) nsplit = std::max(1, atoi(e));
    int64_t kchunk = (ksteps + nsplit - 1) / nsplit * BK;
    nsplit = (int)((sp->kc + kchunk - 1) / kchunk);
    void* part = nullptr;
    FX_TRY(ws_get(ctx, ws, "mf_partial", sizeof(double) * (size_t)nsplit * n * 2 * R, &part));
    // Few right-hand sides by a wave per 32 rows instead of workgroup tiles.  FP32:
    // up to 32 (us, waves against tiles: 432 factors at 72^3, 8 of them 795 / 2350,
    // 32: 1694 / 2350).  2-byte types, up to 16: while the tiles leave half the chip
    // idle (with the residual: 128 factors at 48^3, 8: 31 / 43, 216 at 72^3 193 /
    // 166, 432 336 / 264; without it the waves hold out longer, 216 84 / 97, 432
    // 147 / 136); 17 to 32: while the waves do (64 factors at 48^3, 24: 34 / 42,
    // 128 51 / 46).
    const int tms = (n + 31) / 32;
    const bool waves_cn = sizeof(S) == 4 ? R <= 32
                          : R <= 16     ? tiles * nsplit < (REFINE ? 192 : 384)
                                        : R <= 32 && tms * nsplit < 512;
    FX_TRY(prof_begin(ctx, st, FX_K_GEMM_CN, (REFINE ? 3.0 : 1.0) * 2.0 * n * 2.0 * R * (double)sp->kc, &slot));
    if (waves_cn) {
      const auto kern = R <= 16 ? k_tn_skinny<S, REFINE, true, 0, 1> : k_tn_skinny<S, REFINE, true, 0, 2>;
      hipLaunchKernelGGL(kern, dim3((unsigned)(tms * nsplit)), dim3(64), 0, st, n, 2 * R, (int)kchunk, (int)sp->kc,
                         (const S*)sp->col_p, (const S*)sp->col_r, sp->kc, (const S*)php, (const S*)phr, sp->kc,
                         (double*)part, (void*)nullptr, (int64_t)0, 0, (const double*)nullptr, tms);
    } else {
      const auto launch = [&](auto kern, size_t bytes, auto... rest) -> fx_status {
        FX_TRY(allow_lds_mfma(kern, bytes));
        hipLaunchKernelGGL(kern, dim3((unsigned)(tiles * nsplit)), dim3(256), bytes, st, n, sizeof(S) == 2 ? R : 2 * R,
                           (int)sp->kc, (int)kchunk, (const S*)sp->col_p, (const S*)sp->col_r, sp->kc, (const S*)php,
                           (const S*)phr, sp->kc, (double*)part, (void*)nullptr, (int64_t)0, 0, rest..., tiles_m,
                           tiles_n);
        return FX_OK;
      };
      const double* no_scale = nullptr;
      if constexpr (sizeof(S) == 2)
        FX_TRY(launch(k_tn_pair<S, REFINE, 0>, pair_lds_bytes<REFINE>(), no_scale));
      else
        FX_TRY(launch(k_tn_mfma<S, REFINE, true, 0>, lds, 1.0, no_scale));
    }
    FX_LAUNCH_CHECK();
    FX_TRY(prof_end(ctx, st, slot));
    // reduce -> B operand of the second product
    void *bp = nullptr, *br = nullptr;
    const size_t bb = sizeof(S) * (size_t)2 * R * sp->kn;
    FX_TRY(ws_get(ctx, ws, split_name<S>(2), bb, &bp));
    FX_TRY(ws_get(ctx, ws, split_name<S>(3), bb, &br));
    const int64_t tr = (int64_t)R * (sp->kn / 2);
    FX_TRY(prof_begin(ctx, st, FX_K_REDUCE, 8.0 * nsplit * n * 2.0 * R + 2.0 * bb, &slot));
    if (kScaled<S>) {
      void* c64 = nullptr;
      FX_TRY(ws_get(ctx, ws, "mf_c64", 16 * (size_t)n * R, &c64));
      hipLaunchKernelGGL(k_sum_cn_scaled, dim3(sum_blocks((int64_t)n * R)), dim3(256), 0, st, (const double2*)part,
                         nsplit, n, R, (const unsigned*)sp->smax, (const unsigned*)pmax, (double2*)c64, cmax);
      FX_LAUNCH_CHECK();
      hipLaunchKernelGGL((k_split_cn_scaled<S>), dim3((unsigned)std::min<int64_t>((tr + 255) / 256, 16384)),
                         dim3(256), 0, st, (const double2*)c64, n, R, sp->kn, (const unsigned*)sp->smax,
                         (const unsigned*)cmax, (S*)bp, (S*)br, colalpha);
    } else {
      hipLaunchKernelGGL((k_reduce_cn<S>), dim3(sum_blocks(tr)), dim3(256), 0, st, (const double2*)part, nsplit, n, R,
                         sp->kn, (S*)bp, (S*)br);
    }
    FX_LAUNCH_CHECK();
    FX_TRY(prof_end(ctx, st, slot));
    // y = -xi C: M = nr, N = 2R, K = kn
    FX_TRY(prof_begin(ctx, st, FX_K_GEMM_NN, (REFINE ? 3.0 : 1.0) * 2.0 * (double)nr * 2.0 * R * (double)sp->kn, &slot));
    // FP32, up to 32 right-hand sides: by waves too (8 right-hand sides with 432
    // factors at 72^3 2233 -> 1020 us, 32 of them 2296 -> 1980); the 2-byte types
    // keep the tiles (8, FP16 with the residual: 281 against 417 us)
    bool waves_out = false;
    if constexpr (sizeof(S) == 4) {
      waves_out = R <= 32;
      if (waves_out) {
        const int tms = (int)((nr + 31) / 32);
        const auto kern = R <= 16 ? k_tn_skinny<S, REFINE, false, 1, 1> : k_tn_skinny<S, REFINE, false, 1, 2>;
        hipLaunchKernelGGL(kern, dim3((unsigned)tms), dim3(64), 0, st, (int)nr, 2 * R, (int)sp->kn, (int)sp->kn,
                           (const S*)sp->row_p, (const S*)sp->row_r, sp->kn, (const S*)bp, (const S*)br, sp->kn,
                           (double*)nullptr, out, ld_out, out_dtype == FX_C64 ? 1 : 0, (const double*)colalpha, tms);
      }
    }
    if (!waves_out) {
      const int tm2 = (int)((nr + TBM - 1) / TBM), tn2 = (2 * R + TBN - 1) / TBN;
      const dim3 grid((unsigned)(tm2 * tn2)), blk(256);
      const int c64 = out_dtype == FX_C64 ? 1 : 0;
      if constexpr (sizeof(S) == 2) {
        const auto kern = k_tn_pair<S, REFINE, 1>;
        const size_t bytes = pair_lds_bytes<REFINE>();
        FX_TRY(allow_lds_mfma(kern, bytes));
        // (row 2c of B: the even rows)
        hipLaunchKernelGGL(kern, grid, blk, bytes, st, (int)nr, R, (int)sp->kn, (int)sp->kn, (const S*)sp->row_p,
                           (const S*)sp->row_r, sp->kn, (const S*)bp, (const S*)br, 2 * sp->kn, (double*)nullptr, out,
                           ld_out, c64, (const double*)colalpha, tm2, tn2);
      } else {
        const auto kern = k_tn_mfma<S, REFINE, false, 1>;
        // the epilogue turns each wave's 32x32 tiles around in 32 x 33 doubles of LDS
        const size_t bytes = std::max(lds, (size_t)4 * 32 * 33 * sizeof(double));
        FX_TRY(allow_lds_mfma(kern, bytes));
        hipLaunchKernelGGL(kern, grid, blk, bytes, st, (int)nr, 2 * R, (int)sp->kn, (int)sp->kn, (const S*)sp->row_p,
                           (const S*)sp->row_r, sp->kn, (const S*)bp, (const S*)br, sp->kn, (double*)nullptr, out,
                           ld_out, c64, 1.0, (const double*)colalpha, tm2, tn2);
      }
    }
    FX_LAUNCH_CHECK();
    FX_TRY(prof_end(ctx, st, slot));
  }
  return FX_OK;
}

fx_status ace_apply_mfma(fx_ctx* ctx, Workspace* ws, fx_ace* a, const void* phi, int nphi, int64_t ld_phi, void* out,
                         int64_t ld_out, fx_dtype in_dtype, fx_dtype out_dtype, fx_prec prec, hipStream_t st) {
  switch (prec) {
    case FX_PREC_ACE_FP32R:
      return apply_t<float, true>(ctx, ws, a, &a->f32, phi, nphi, ld_phi, out, ld_out, in_dtype, out_dtype, st);
    case FX_PREC_ACE_FP32:
      return apply_t<float, false>(ctx, ws, a, &a->f32, phi, nphi, ld_phi, out, ld_out, in_dtype, out_dtype, st);
    case FX_PREC_ACE_BF16R:
      return apply_t<uint16_t, true>(ctx, ws, a, &a->b16, phi, nphi, ld_phi, out, ld_out, in_dtype, out_dtype, st);
    case FX_PREC_ACE_BF16:
      return apply_t<uint16_t, false>(ctx, ws, a, &a->b16, phi, nphi, ld_phi, out, ld_out, in_dtype, out_dtype, st);
    case FX_PREC_ACE_FP16R:
      return apply_t<_Float16, true>(ctx, ws, a, &a->f16, phi, nphi, ld_phi, out, ld_out, in_dtype, out_dtype, st);
    case FX_PREC_ACE_FP16:
      return apply_t<_Float16, false>(ctx, ws, a, &a->f16, phi, nphi, ld_phi, out, ld_out, in_dtype, out_dtype, st);
    default:
      FX_FAIL(FX_ERR_UNSUPPORTED, "precision %d is not a matrix-core ACE precision", prec);
  }
}

}  // namespace fx
