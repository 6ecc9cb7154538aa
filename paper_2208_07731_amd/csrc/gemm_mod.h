// FP64 products C = A B^T on the 8-bit matrix cores of gfx950, by residues.
//
//   C(m, n) = sum_k A(m, k) B(n, k), A and B K-contiguous, FP64 results.
//
// Each row of A and of B is scaled by a power of two to a 2-norm below 2^65
// and rounded to integers (mod_split), so that every entry of the integer
// product is below 2^130 (Cauchy-Schwarz) whatever K is.  The integer product
// is computed exactly modulo 17 pairwise coprime moduli of at most 8 bits
// (their product P is 2^133.0) with one int8 matrix product per modulus
// (mod_gemm), and put together by the Chinese remainder theorem (mod_crt):
// with w_i = ((P / p_i)^-1 mod p_i) / p_i, C / P = sum_i r_i w_i modulo 1.
// The only errors are the rounding of the operands (absolute, up to 2^-65 of the
// row's 2-norm per entry: entries down to 2^-12 of the norm keep all their 53
// bits, and at K = 16384 terms the typical one is 2^-7 of it) and the last
// rounding of C.  Two moduli fewer, 2^58, round the typical entry of K = 2048
// and lose the tails of localised orbitals first: a worst entry 3 times as far
// off as an FP64 sum's at a density range of 1e3, a ninth of it with these.
// The guarantee stays relative to the product of the (balanced) rows' norms, an
// FP64 sum's is relative to the sum of moduli of its own terms.  Residue
// products are the idea of Ozaki's scheme for matrix multiplication through
// integer arithmetic; this form is derived from the remainder theorem above.
//
// Why: the FP64 matrix cores do 78.6 TFLOP/s, the int8 ones 64 times as much,
// so 17 int8 products have 3.7 times the rate to spend; splitting and putting
// together move 25 bytes per operand and per result element, which K N / (K +
// N) has to pay for (mod_pays).  Measured: 32768 x 8192 x 8192 69.0 ms FP64 (64
// TFLOP/s), 34.2 by residues; 65536 x 2048 x 2048 8.6 and 6.1; the 2-norm error
// against extended precision is 6.5e-17, that of rounding the result, where the
// FP64 kernel's is 1.1e-15 to 3.2e-15.
//
// A common power of two per k is moved from one operand to the other
// (A(m, k) d_k, B(n, k) / d_k, exact), which takes out the range that the
// density at the interpolation points gives the columns (six orders of magnitude
// and more) and that a row's scale cannot.  With B = (C C^H)^-1 that is d_k =
// sqrt(B(k, k)) (mod_diag); products with Phi_mu or Psi_mu take it from the mean
// exponents of both operands' columns (mod_means), since Abar and V grow where
// the orbitals are small: Abar Phi_mu at a density range of 1e6 is off by 2e-14
// without it, where an FP64 sum is off by 5e-16, and by 2e-17 with it.
//
// A row that is not finite, or whose norm is outside 2^+-460, raises a flag;
// the residue kernels then do nothing and the FP64 kernel launched behind them
// (GemmShape::only) computes the panel as it always did.
#pragma once

#include "gemm.h"

namespace isdf {
namespace {

constexpr int MOD_N = 17;
constexpr int MOD_BITS = 65;      // a scaled row's 2-norm is at most 2^65
constexpr int MOD_KMAX = 16384;   // |sum| < K 2^14 <= 2^28, the bound of mod_reduce
constexpr int MOD_T = 256;        // output tile edge
constexpr int MOD_BK = 128;       // K bytes per LDS stage
constexpr int MOD_THREADS = 512;  // 8 wavefronts, 2 (m) x 4 (n), 128 x 64 outputs each

// Product of n moduli (below 2^160) as P + Plo, two doubles of 53 bits each.
struct ModProduct {
  double P, Plo;
};
constexpr ModProduct mod_product(const int* p, int n) {
  unsigned limb[5] = {1, 0, 0, 0, 0};
  for (int i = 0; i < n; ++i) {
    unsigned long long carry = 0;
    for (unsigned& l : limb) {
      const unsigned long long t = (unsigned long long)l * (unsigned)p[i] + carry;
      l = (unsigned)t;
      carry = t >> 32;
    }
  }
  ModProduct r{0.0, 0.0};
  int seen = 0;  // bits from the first one on
  for (int b = 159; b >= 0; --b) {
    r.P *= 2.0;
    r.Plo *= 2.0;
    const int bit = limb[b / 32] >> (b % 32) & 1;
    if (bit || seen) ++seen;
    if (!bit) continue;
    if (seen <= 53) r.P += 1.0;
    else if (seen <= 106) r.Plo += 1.0;
  }
  return r;
}
// (product of the other moduli) mod p[i]
constexpr int mod_others(const int* p, int n, int i) {
  int m = 1;
  for (int j = 0; j < n; ++j)
    if (j != i) m = m * p[j] % p[i];
  return m;
}

struct ModTab {
  int p[MOD_N];
  int c14[MOD_N];    // 2^14 mod p, in (-p/2, p/2]
  float fip[MOD_N];  // 1 / p
  double ip[MOD_N];
  // w = w1 + w2, w1 a multiple of 2^-42: sums of r_i w1_i are exact
  double w1[MOD_N], w2[MOD_N];
  double P, Plo;     // product of the moduli, P + Plo to 106 bits
};

constexpr ModTab make_mod_tab() {
  ModTab t{};
  const int p[MOD_N] = {256, 255, 253, 251, 247, 241, 239, 233, 229, 227, 223, 217, 211, 199, 197, 193, 191};
  for (int i = 0; i < MOD_N; ++i) {
    const int m = mod_others(p, MOD_N, i);
    int q = 1;
    while (q * m % p[i] != 1) ++q;
    if (2 * q > p[i]) q -= p[i];
    const long long num = (long long)q * (1ll << 42);
    t.p[i] = p[i];
    t.c14[i] = 16384 % p[i] > p[i] / 2 ? 16384 % p[i] - p[i] : 16384 % p[i];
    t.fip[i] = 1.0f / (float)p[i];
    t.ip[i] = 1.0 / p[i];
    t.w1[i] = (double)(num / p[i]) / (double)(1ll << 42);
    t.w2[i] = ((double)(num % p[i]) / p[i]) / (double)(1ll << 42);
  }
  t.P = mod_product(p, MOD_N).P;
  t.Plo = mod_product(p, MOD_N).Plo;
  return t;
}
constexpr ModTab MOD_TAB = make_mod_tab();
static __device__ __constant__ ModTab mod_tab = make_mod_tab();

// Complex products: modulo p = 1 (mod 4) (or a product of such primes) there is
// an s with s^2 = -1, and x + i y -> (x + s y, x - s y) turns the complex
// product into two independent real ones instead of four, exactly.  18 such
// moduli of at most 241 have the product 2^130.3, for rows of a 2-norm below
// 2^64; 36 planes against the 68 of the real 2 x 2 block form.  Conjugation
// swaps the two planes.  108000 x 1201 x 1201 complex: 22.5 ms on the FP64
// matrix cores, 10.2 this way (with two moduli fewer the int8 products took 11.2
// in the real form and 6.9 this way).
constexpr int MOD_NC = 18;
constexpr int MOD_BITS_C = 64;

struct ModTabC {
  int p[MOD_NC];
  int c14[MOD_NC];
  float fp[MOD_NC], fip[MOD_NC];
  float s[MOD_NC];   // a square root of -1
  double dp[MOD_NC], ip[MOD_NC];
  // weights of u + v (real part) and u - v (imaginary part), split as in ModTab
  double w1r[MOD_NC], w2r[MOD_NC], w1i[MOD_NC], w2i[MOD_NC];
  double P, Plo;
};

constexpr int mod_inverse(int a, int p) {
  int q = 1;
  while (q * a % p != 1) ++q;
  return q;
}

constexpr ModTabC make_mod_tab_c() {
  ModTabC t{};
  const int p[MOD_NC] = {241, 233, 229, 221, 205, 197, 193, 181, 173, 157, 149, 137, 113, 109, 101, 97, 89, 73};
  for (int i = 0; i < MOD_NC; ++i) {
    const int m = mod_others(p, MOD_NC, i);
    int s = 1;
    while ((s * s + 1) % p[i] != 0) ++s;
    const int q0 = mod_inverse(m, p[i]);
    int qr = q0 * mod_inverse(2, p[i]) % p[i], qi = q0 * mod_inverse(2 * s % p[i], p[i]) % p[i];
    if (2 * qr > p[i]) qr -= p[i];
    if (2 * qi > p[i]) qi -= p[i];
    const long long nr = (long long)qr * (1ll << 42), ni = (long long)qi * (1ll << 42);
    t.p[i] = p[i];
    t.c14[i] = 16384 % p[i] > p[i] / 2 ? 16384 % p[i] - p[i] : 16384 % p[i];
    t.fp[i] = (float)p[i];
    t.fip[i] = 1.0f / (float)p[i];
    t.s[i] = (float)s;
    t.dp[i] = p[i];
    t.ip[i] = 1.0 / p[i];
    t.w1r[i] = (double)(nr / p[i]) / (double)(1ll << 42);
    t.w2r[i] = ((double)(nr % p[i]) / p[i]) / (double)(1ll << 42);
    t.w1i[i] = (double)(ni / p[i]) / (double)(1ll << 42);
    t.w2i[i] = ((double)(ni % p[i]) / p[i]) / (double)(1ll << 42);
  }
  t.P = mod_product(p, MOD_NC).P;
  t.Plo = mod_product(p, MOD_NC).Plo;
  return t;
}
constexpr ModTabC MOD_TAB_C = make_mod_tab_c();
static __device__ __constant__ ModTabC mod_tab_c = make_mod_tab_c();

typedef int i4v __attribute__((ext_vector_type(4)));
typedef int i16v __attribute__((ext_vector_type(16)));

// A panel is left to the FP64 kernel when either operand raised its flag.
__device__ __forceinline__ bool mod_off(const int* abort, const int* bflag, const int* aflag) {
  return (abort && *abort) || *bflag || *aflag;
}

// ------------------------------------------------------------------ scales
// d[k] = 2^round(log2 sqrt(B(k, k))) and its reciprocal (1 where the diagonal
// is not a normal positive number); step 2: of the real 2 x 2 blocks of a
// complex matrix.
__global__ void mod_diag(const double* __restrict__ B, int64_t ldb, int K, int step, double* __restrict__ d,
                         double* __restrict__ di) {
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= K) return;
  const double v = B[(int64_t)k * step * (ldb + 1)];
  int e = 0;
  if (v > 1e-280 && v < 1e280) {
    frexp(v, &e);
    e >>= 1;
  }
  d[k] = ldexp(1.0, e);
  di[k] = ldexp(1.0, -e);
}

// d[k] = 2^round((b - a) / 2) and its reciprocal, with a and b the mean binary
// exponents of the nonzero finite entries of column k of A (M rows) and of B (N
// rows; both complex, re and im side by side, lda and ldb in reals), from at
// most MEANS rows of each.  A mean of exponents and not a norm: one large entry
// would take its column's digits from all the other rows.  32 columns by 8
// groups of rows per workgroup; 2 MEANS rows are read, 8 MB of 16384 x 2048.
constexpr int MEANS = 128;
template <class TA>
__global__ __launch_bounds__(256) void mod_means(const TA* __restrict__ A, int64_t lda, int M,
                                                 const double* __restrict__ B, int64_t ldb, int N, int K,
                                                 double* __restrict__ d, double* __restrict__ di) {
  __shared__ int sum[2][8][32], cnt[2][8][32];
  const int c = threadIdx.x & 31, g = threadIdx.x >> 5;
  const int k = blockIdx.x * 32 + c, kc = k < K ? k : K - 1;
  const auto column = [&](auto* x, int64_t ld, int rows, int which) {
    const int n = rows < MEANS ? rows : MEANS;
    int s = 0, m = 0;
#pragma unroll 8
    for (int i = g; i < n; i += 8) {
      const double2 z = Cplx<std::remove_const_t<std::remove_pointer_t<decltype(x)>>>::load(
          x + (int64_t)i * rows / n * ld + 2 * kc);
      const int e = __double2hiint(fmax(fabs(z.x), fabs(z.y))) >> 20 & 0x7ff;
      if (e != 0 && e != 0x7ff) {
        s += e;
        ++m;
      }
    }
    sum[which][g][c] = s;
    cnt[which][g][c] = m;
  };
  column(A, lda, M, 0);
  column(B, ldb, N, 1);
  __syncthreads();
  if (g != 0 || k >= K) return;
  int s[2] = {0, 0}, m[2] = {0, 0};
#pragma unroll
  for (int w = 0; w < 2; ++w)
    for (int i = 0; i < 8; ++i) {
      s[w] += sum[w][i][c];
      m[w] += cnt[w][i][c];
    }
  int e = 0;
  if (m[0] && m[1]) e = (int)rintf(0.5f * ((float)s[1] / (float)m[1] - (float)s[0] / (float)m[0]));
  e = e < -400 ? -400 : e > 400 ? 400 : e;
  d[k] = ldexp(1.0, e);
  di[k] = ldexp(1.0, -e);
}

__global__ void mod_clear(int* flags, int n) {
  for (int i = threadIdx.x; i < n; i += blockDim.x) flags[i] = 0;
}

// ------------------------------------------------------------------- split
// Row blockIdx.x of X (K entries, times ks[k]): its scale and the
// residues of its scaled integers, planes [MOD_N][rows][kpad] (zero past K).
// One workgroup per row, the row held in registers between the norm and the
// residues (4 IT per thread).  Bound by HBM: 8 bytes read and 17 written per
// entry; a residue costs 7 FP64 operations.
// r mod p of an integer |x| <= 2^65 held in a double: the quotient is off by up
// to 2^-52 |x| / p, which leaves a first remainder below 2^13 + p (an integer,
// so exact); the second step takes that to [-p/2, p/2].
__device__ __forceinline__ unsigned mod_byte(double x, double p, double ip) {
  const double r = fma(-__builtin_rint(x * ip), p, x);
  const double y = fma(-__builtin_rint(r * ip), p, r + 6755399441055744.0);  // + 1.5 2^52: integer in the low word
  return (unsigned)__double2loint(y) & 0xffu;
}

// Low bytes of four words.
__device__ __forceinline__ unsigned mod_pack(unsigned a, unsigned b, unsigned c, unsigned d) {
  return __builtin_amdgcn_perm(__builtin_amdgcn_perm(d, c, 0x0c0c0400u), __builtin_amdgcn_perm(b, a, 0x0c0c0400u),
                               0x05040100u);
}

// The power of two that takes a row of squared 2-norm n2 to at most 2^bits (0 for a zero row); its reciprocal into *rscale; a row out of range (`some`:
// not all zero) raises the flag.
__device__ __forceinline__ double mod_scale(double n2, int some, int bits, int tid, double* rscale, int* flag) {
  double up = 0.0, down = 0.0;
  if (n2 > 1e-280 && n2 < 1e280) {
    int e2 = 0;
    frexp(n2, &e2);  // n2 < 2^e2
    const int e = bits - ((e2 + 1) >> 1);
    up = ldexp(1.0, e);
    down = ldexp(1.0, -e);
  } else if (some) {
    if (tid == 0) atomicOr(flag, 1);
  }
  if (tid == 0) *rscale = down;
  return up;
}

template <class TS, int IT>
__global__ __launch_bounds__(256) void mod_split(const TS* __restrict__ X, int64_t ld, int rows, int K, int kpad,
                                                 const double* __restrict__ ks, int vec, int8_t* __restrict__ out,
                                                 int64_t pstride, double* __restrict__ rscale, int* flag,
                                                 const int* abort) {
  if (abort && *abort) return;
  __shared__ double red[256 / ISDF_WAVE];
  const int tid = threadIdx.x;
  const int64_t row = blockIdx.x;
  const TS* x = X + row * ld;
  double v[IT][4];
  double n2 = 0.0;
  bool any = false;
#pragma unroll
  for (int it = 0; it < IT; ++it) {
    const int k = 4 * (tid + 256 * it);
    if (vec && k + 4 <= K) {
      load_pair<TS>(x + k, v[it][0], v[it][1]);
      load_pair<TS>(x + k + 2, v[it][2], v[it][3]);
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) v[it][e] = k + e < K ? (double)x[k + e] : 0.0;
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      any |= v[it][e] != 0.0;  // true for NaN
      v[it][e] *= k + e < K ? ks[k + e] : 0.0;
      n2 = fma(v[it][e], v[it][e], n2);
    }
  }
  n2 = wave_sum(n2);
  if ((tid & 63) == 0) red[tid >> 6] = n2;
  const int some = __syncthreads_or(any);
  n2 = (red[0] + red[1]) + (red[2] + red[3]);
  const double up = mod_scale(n2, some, MOD_BITS, tid, rscale + row, flag);
  int8_t* o = out + row * kpad;
#pragma unroll
  for (int it = 0; it < IT; ++it) {
    const int k = 4 * (tid + 256 * it);
    if (k >= kpad) continue;
    double s[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) s[e] = __builtin_rint(v[it][e] * up);
#pragma unroll
    for (int i = 0; i < MOD_N; ++i) {
      unsigned w = 0;
#pragma unroll
      for (int e = 0; e < 4; ++e) w |= mod_byte(s[e], MOD_TAB.p[i], MOD_TAB.ip[i]) << (8 * e);
      *reinterpret_cast<unsigned*>(o + i * pstride + k) = w;
    }
  }
}

// Row blockIdx.x of a complex X (K entries, real and imaginary parts side by
// side, ld in reals), scaled by the 2-norm of its 2 K reals: planes
// [2 MOD_NC][rows][kpad] of x + s y and x - s y modulo each modulus (`conj`:
// the other way round).  x and y leave FP64 as remainders below 2^12 + p (as in
// mod_byte), the rest is exact in FP32 (s < p / 2, so |x + s y| < 2^20).
template <class TS, int IT>
__global__ __launch_bounds__(256) void mod_split_c(const TS* __restrict__ X, int64_t ld, int rows, int K, int kpad,
                                                   const double* __restrict__ ks, int vec, int conj,
                                                   int8_t* __restrict__ out, int64_t pstride,
                                                   double* __restrict__ rscale, int* flag, const int* abort) {
  if (abort && *abort) return;
  __shared__ double red[256 / ISDF_WAVE];
  const int tid = threadIdx.x;
  const int64_t row = blockIdx.x;
  const TS* x = X + row * ld;
  double v[IT][8];
  double n2 = 0.0;
  bool any = false;
#pragma unroll
  for (int it = 0; it < IT; ++it) {
    const int k = 4 * (tid + 256 * it);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      double a = 0.0, b = 0.0;
      if (k + e < K) {
        if (vec) {
          load_pair<TS>(x + 2 * (k + e), a, b);
        } else {
          a = (double)x[2 * (k + e)];
          b = (double)x[2 * (k + e) + 1];
        }
        any |= a != 0.0 || b != 0.0;  // true for NaN
        a *= ks[k + e];
        b *= ks[k + e];
      }
      v[it][2 * e] = a;
      v[it][2 * e + 1] = b;
      n2 = fma(a, a, fma(b, b, n2));
    }
  }
  n2 = wave_sum(n2);
  if ((tid & 63) == 0) red[tid >> 6] = n2;
  const int some = __syncthreads_or(any);
  n2 = (red[0] + red[1]) + (red[2] + red[3]);
  const double up = mod_scale(n2, some, MOD_BITS_C, tid, rscale + row, flag);
  int8_t* o = out + row * kpad;
#pragma unroll
  for (int it = 0; it < IT; ++it) {
    const int k = 4 * (tid + 256 * it);
    if (k >= kpad) continue;
    double s[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) s[e] = __builtin_rint(v[it][e] * up);
#pragma unroll
    for (int i = 0; i < MOD_NC; ++i) {
      unsigned wu[4], wv[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float rx = (float)fma(-__builtin_rint(s[2 * e] * MOD_TAB_C.ip[i]), MOD_TAB_C.dp[i], s[2 * e]);
        const float ry = (float)fma(-__builtin_rint(s[2 * e + 1] * MOD_TAB_C.ip[i]), MOD_TAB_C.dp[i], s[2 * e + 1]);
        const float u = fmaf(MOD_TAB_C.s[i], ry, rx), w = fmaf(-MOD_TAB_C.s[i], ry, rx);
        // + 1.5 2^23: the integer in the low bits, a multiple of 256 beside it
        wu[e] = __float_as_uint(fmaf(-__builtin_rintf(u * MOD_TAB_C.fip[i]), MOD_TAB_C.fp[i], u + 12582912.0f));
        wv[e] = __float_as_uint(fmaf(-__builtin_rintf(w * MOD_TAB_C.fip[i]), MOD_TAB_C.fp[i], w + 12582912.0f));
      }
      *reinterpret_cast<unsigned*>(o + (2 * i + conj) * pstride + k) = mod_pack(wu[0], wu[1], wu[2], wu[3]);
      *reinterpret_cast<unsigned*>(o + (2 * i + 1 - conj) * pstride + k) = mod_pack(wv[0], wv[1], wv[2], wv[3]);
    }
  }
}

// -------------------------------------------------------------------- GEMM
// A word whose low byte is acc mod p in [-p/2, p/2] (the byte wraps for p =
// 256): 14 low bits and the rest times 2^14 mod p give |t| <= 2^21 + 2^14,
// whose quotient by p one FP32 multiply-add rounds to the nearest integer
// (its error, 2^-25 t / p, is below the 1 / (2 p) between t / p and a half
// integer); the 1.5 2^23 that puts the integer into the low bits is a
// multiple of 256 and drops out of the byte.
__device__ __forceinline__ unsigned mod_reduce(int acc, int p, int c14, float fip) {
  const int t = __mul24(acc >> 14, c14 - 16384) + acc;
  const int q = __float_as_int(fmaf((float)t, fip, 12582912.0f));
  return (unsigned)(t - __mul24(q, p));
}
// The same where K <= MOD_KQUICK and p <= 241: the residues are at most (p + 1) /
// 2, so the sum is exact to half a unit of its FP32 rounding; with the rounding
// of 1 / p the quotient is off by little enough that the remainder still fits
// the byte (mod_quick_bound).
constexpr int MOD_KQUICK = 4096;
constexpr double mod_quick_bound() {
  double worst = 0.0;
  for (int i = 0; i < MOD_NC; ++i) {
    const double p = MOD_TAB_C.p[i], r = (p + 1.0) / 2.0, acc = r * r * MOD_KQUICK;
    double half = 0.5;  // half a unit in the last place of acc in FP32
    for (double t = acc; t >= 16777216.0; t /= 2.0) half *= 2.0;
    if (acc < 16777216.0) half = 0.0;
    const double off = (double)MOD_TAB_C.fip[i] * p - 1.0;
    const double bound = p / 2.0 + half + acc * (off < 0.0 ? -off : off);
    worst = bound > worst ? bound : worst;
  }
  return worst;
}
static_assert(mod_quick_bound() < 127.5, "the remainder fits a byte");
__device__ __forceinline__ unsigned mod_reduce_quick(int acc, int p, float fip) {
  const int q = __float_as_int(fmaf((float)acc, fip, 12582912.0f));
  return (unsigned)(acc - __mul24(q, p));
}

// Residue planes of A B^T: R [planes][M][ldr] from A [planes][M][ld] and B
// [planes][N][ld] (CPLX: two planes per modulus) (ld a multiple of 128 bytes, ldr of 256).  256 x 256 tiles of
// eight wavefronts (128 x 64 each: 128 accumulator registers), 128-byte K
// stages in two LDS buffers (128 KB, one workgroup per CU), the next stage
// but one in flight in registers.  v_mfma_i32_32x32x32_i8 takes B's rows as
// its row operand, so that a lane's four consecutive accumulators are four
// consecutive n of one m and leave as one word.  An LDS row is its 8 chunks of
// 16 bytes at chunk ^ (row / 2 % 8): the 32 lanes of a fragment read (32 rows,
// one chunk) hit 16 different 16-byte slots modulo 512 bytes, two lanes each.
template <bool CPLX>
__global__ __launch_bounds__(MOD_THREADS, 2) void mod_gemm(const int8_t* __restrict__ A, int64_t astride,
                                                           const int8_t* __restrict__ B, int64_t bstride, int ld, int M,
                                                           int N, int8_t* __restrict__ R, int64_t rstride, int ldr,
                                                           const int* abort, const int* bflag, const int* aflag) {
  if (mod_off(abort, bflag, aflag)) return;
  constexpr int STAGE = 2 * MOD_T * MOD_BK;
  __shared__ __attribute__((aligned(16))) int8_t smem[2 * STAGE];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int wm = wv >> 2, wn = wv & 3;
  const int tiles_m = (M + MOD_T - 1) / MOD_T, tiles_n = (N + MOD_T - 1) / MOD_T;
  const int ntiles = tiles_m * tiles_n;
  const int logical = xcd_remap(blockIdx.x, gridDim.x);
  const int mod = logical / ntiles, tile = logical % ntiles;
  // column by column within groups of 4 row blocks: the 32 tiles of an XCD
  // then need 4 row and 8 column panels of A and B
  constexpr int GR = 4;
  const int first = (tile / (GR * tiles_n)) * GR;
  const int rows_in = tiles_m - first < GR ? tiles_m - first : GR;
  const int local = tile % (GR * tiles_n);
  const int m0 = (first + local % rows_in) * MOD_T, n0 = (local / rows_in) * MOD_T;
  A += mod * astride;
  B += mod * bstride;

  // staging: chunk `id` of a stage is 16 bytes of row id / 8
  constexpr int PER = MOD_T * MOD_BK / 16 / MOD_THREADS;
  int64_t offa[PER], offb[PER];
  int dst[PER];
#pragma unroll
  for (int c = 0; c < PER; ++c) {
    const int id = tid + c * MOD_THREADS, r = id >> 3, ch = id & 7;
    const int ra = m0 + r < M ? m0 + r : M - 1, rb = n0 + r < N ? n0 + r : N - 1;  // past the edge: any valid row
    offa[c] = (int64_t)ra * ld + 16 * ch;
    offb[c] = (int64_t)rb * ld + 16 * ch;
    dst[c] = r * MOD_BK + 16 * (ch ^ ((r >> 1) & 7));
  }
  i4v sa[PER], sb[PER];
  auto load_a = [&](int c, int k) { sa[c] = *reinterpret_cast<const i4v*>(A + offa[c] + k); };
  auto load_b = [&](int c, int k) { sb[c] = *reinterpret_cast<const i4v*>(B + offb[c] + k); };
  auto store_a = [&](int c, int8_t* buf) { *reinterpret_cast<i4v*>(buf + dst[c]) = sa[c]; };
  auto store_b = [&](int c, int8_t* buf) { *reinterpret_cast<i4v*>(buf + MOD_T * MOD_BK + dst[c]) = sb[c]; };
  const int half = lane >> 5, sw = ((lane & 31) >> 1) & 7;
  const int arow = (wm * 128 + (lane & 31)) * MOD_BK;
  const int brow = MOD_T * MOD_BK + (wn * 64 + (lane & 31)) * MOD_BK;
  i4v fa[2][4], fb[2][2];
  // fragment t of sub-step s (32 of the stage's K bytes): B 0, A 0..3, B 1 in
  // the order the products want them
  auto frag = [&](int t, const int8_t* buf, int s, int to) {
    const int ch = 16 * ((2 * s + half) ^ sw);
    if (t == 0) fb[to][0] = *reinterpret_cast<const i4v*>(buf + brow + ch);
    else if (t == 5) fb[to][1] = *reinterpret_cast<const i4v*>(buf + brow + 32 * MOD_BK + ch);
    else fa[to][t - 1] = *reinterpret_cast<const i4v*>(buf + arow + (t - 1) * 32 * MOD_BK + ch);
  };
  i16v acc[2][4];
#pragma unroll
  for (int j = 0; j < 2; ++j)
#pragma unroll
    for (int i = 0; i < 4; ++i) acc[j][i] = i16v{0};

  const int klast = ld - MOD_BK;
  const int k1 = MOD_BK < klast ? MOD_BK : klast;
#pragma unroll
  for (int c = 0; c < PER; ++c) {
    load_a(c, 0);
    load_b(c, 0);
  }
#pragma unroll
  for (int c = 0; c < PER; ++c) {
    store_a(c, smem);
    store_b(c, smem);
  }
#pragma unroll
  for (int c = 0; c < PER; ++c) load_a(c, k1);
#pragma unroll
  for (int c = 0; c < PER; ++c) load_b(c, k1);
  __syncthreads();
#pragma unroll
  for (int t = 0; t < 6; ++t) frag(t, smem, 0, 0);
  int cur = 0;
  for (int k = 0; k < ld; k += MOD_BK) {
    // the last steps load, store and read a stage that nothing uses (the last
    // one again), which keeps the loop free of branches
    const int8_t* cbuf = smem + cur * STAGE;
    int8_t* nbuf = smem + (cur ^ 1) * STAGE;
    const int k2 = k + 2 * MOD_BK < klast ? k + 2 * MOD_BK : klast;
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const int now = s & 1;
      if (s == 3) __syncthreads();  // the next stage is stored by every wave; this buffer's reads are done
      __builtin_amdgcn_s_setprio(1);
      // one product, then at most one LDS read, LDS write and load: a wave's
      // instructions issue in order, and a run of LDS accesses would hold
      // back the products behind it while the LDS serves the other waves
#pragma unroll
      for (int t = 0; t < 8; ++t) {
        const int j = t >> 2, i = t & 3;
        acc[j][i] = __builtin_amdgcn_mfma_i32_32x32x32_i8(fb[now][j], fa[now][i], acc[j][i], 0, 0, 0);
        if (t < 6) frag(t, s < 3 ? cbuf : nbuf, (s + 1) & 3, now ^ 1);
        // the next stage goes into the other buffer (its last reads ended
        // before the previous barrier), A's half under sub-step 0, B's under 1
        if (t & 1) {
          if (s == 0) {
            store_a(t >> 1, nbuf);
            load_a(t >> 1, k2);
          }
          if (s == 1) {
            store_b(t >> 1, nbuf);
            load_b(t >> 1, k2);
          }
        }
        __builtin_amdgcn_sched_barrier(0);
      }
      __builtin_amdgcn_s_setprio(0);
    }
    cur ^= 1;
  }

  // residues to memory: a wave's 128 x 64 bytes through its own LDS rows (80
  // bytes apart), 16-byte stores of 64-byte row segments
  __syncthreads();
  const int p = CPLX ? mod_tab_c.p[mod >> 1] : mod_tab.p[mod], c14 = CPLX ? mod_tab_c.c14[mod >> 1] : mod_tab.c14[mod];
  const float fip = CPLX ? mod_tab_c.fip[mod >> 1] : mod_tab.fip[mod];
  const bool quick = CPLX && ld <= MOD_KQUICK;
  int8_t* mine = smem + wv * 128 * 80;
#pragma unroll
  for (int j = 0; j < 2; ++j)
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        unsigned w[4];
#pragma unroll
        for (int e = 0; e < 4; ++e)
          w[e] = quick ? mod_reduce_quick(acc[j][i][4 * q + e], p, fip) : mod_reduce(acc[j][i][4 * q + e], p, c14, fip);
        *reinterpret_cast<unsigned*>(mine + (i * 32 + (lane & 31)) * 80 + j * 32 + 8 * q + 4 * half) =
            mod_pack(w[0], w[1], w[2], w[3]);
      }
  __builtin_amdgcn_wave_barrier();
  int8_t* r = R + mod * rstride;
#pragma unroll
  for (int t = 0; t < 8; ++t) {
    const int row = 16 * t + (lane >> 2), m = m0 + wm * 128 + row;
    const i4v v = *reinterpret_cast<const i4v*>(mine + row * 80 + 16 * (lane & 3));
    if (m < M) *reinterpret_cast<i4v*>(r + (int64_t)m * ldr + n0 + wn * 64 + 16 * (lane & 3)) = v;
  }
}

// --------------------------------------------------------------------- CRT
// C(m, n .. n + 3) from the residues of one row m, in FP64: f = sum_i r_i w_i
// modulo 1 is C / P (|C| < P / 3, so the fraction nearest zero), exact in its
// first part (r_i w1_i are multiples of 2^-42, their sum below 2^11).
__device__ __forceinline__ void mod_combine(const int8_t* __restrict__ R, int64_t rstride, double scale,
                                            const double* __restrict__ cs, int n, int N, double (&c)[4]) {
  int w[MOD_N];
#pragma unroll
  for (int i = 0; i < MOD_N; ++i) w[i] = *reinterpret_cast<const int*>(R + i * rstride);
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    double h = 0.0, l = 0.0;
#pragma unroll
    for (int i = 0; i < MOD_N; ++i) {
      const double r = (double)(int8_t)(w[i] >> (8 * e));
      h = fma(r, MOD_TAB.w1[i], h);
      l = fma(r, MOD_TAB.w2[i], l);
    }
    const double f = (h - __builtin_rint(h)) + l;
    c[e] = fma(f, MOD_TAB.P, f * MOD_TAB.Plo) * scale * cs[n + e < N ? n + e : N - 1];
  }
}

// One thread per Epi::REP runs of 4 consecutive outputs of a row; workgroups
// of 256 threads over the panel's rows x ceil(N / 4).  HBM-bound: 17 residue
// bytes read per output beside what the epilogue moves.
template <class Epi>
__global__ __launch_bounds__(256) void mod_crt(const int8_t* __restrict__ R, int64_t rstride, int ldr, int M, int N,
                                               const double* __restrict__ rs, const double* __restrict__ cs,
                                               const int* abort, const int* bflag, const int* aflag, Epi epi) {
  if (mod_off(abort, bflag, aflag)) {
    epi.off();
    return;
  }
  const int n4 = (N + 3) / 4;
  const int64_t total = (int64_t)M * n4;
  typename Epi::Sum sum{};
#pragma unroll 1
  for (int u = 0; u < Epi::REP; ++u) {
    const int64_t e = ((int64_t)blockIdx.x * Epi::REP + u) * 256 + threadIdx.x;
    if (e < total) {
      const int m = (int)(e / n4), n = 4 * (int)(e % n4);
      const auto in = epi.load(m, n);
      double c[4];
      mod_combine(R + (int64_t)m * ldr + n, rstride, rs[m], cs, n, N, c);
      epi(m, n, c, in, sum);
    }
  }
  epi.finish(sum);
}

// Complex outputs nu .. nu + 3 of row m, re and im side by side, from the
// residues of u and v: u + v = 2 re, u - v = 2 s im (factors in the weights).
__device__ __forceinline__ void mod_combine_c(const int8_t* __restrict__ R, int64_t rstride, double scale,
                                              const double* __restrict__ cs, int nu, int N, double (&c)[8]) {
  int u[MOD_NC], v[MOD_NC];
#pragma unroll
  for (int i = 0; i < MOD_NC; ++i) {
    u[i] = *reinterpret_cast<const int*>(R + 2 * i * rstride);
    v[i] = *reinterpret_cast<const int*>(R + (2 * i + 1) * rstride);
  }
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    double h = 0.0, l = 0.0, hi = 0.0, li = 0.0;
#pragma unroll
    for (int i = 0; i < MOD_NC; ++i) {
      const int a = (int8_t)(u[i] >> (8 * e)), b = (int8_t)(v[i] >> (8 * e));
      const double p = (double)(a + b), q = (double)(a - b);
      h = fma(p, MOD_TAB_C.w1r[i], h);
      l = fma(p, MOD_TAB_C.w2r[i], l);
      hi = fma(q, MOD_TAB_C.w1i[i], hi);
      li = fma(q, MOD_TAB_C.w2i[i], li);
    }
    const double f = (h - __builtin_rint(h)) + l, g = (hi - __builtin_rint(hi)) + li;
    const double t = scale * cs[nu + e < N ? nu + e : N - 1];
    c[2 * e] = fma(f, MOD_TAB_C.P, f * MOD_TAB_C.Plo) * t;
    c[2 * e + 1] = fma(g, MOD_TAB_C.P, g * MOD_TAB_C.Plo) * t;
  }
}

// mod_crt for complex outputs: N complex columns, the epilogue sees pairs of
// them as 4 reals of a row of 2 N.
template <class Epi>
__global__ __launch_bounds__(256) void mod_crt_c(const int8_t* __restrict__ R, int64_t rstride, int ldr, int M, int N,
                                                 const double* __restrict__ rs, const double* __restrict__ cs,
                                                 const int* abort, const int* bflag, const int* aflag, Epi epi) {
  if (mod_off(abort, bflag, aflag)) {
    epi.off();
    return;
  }
  const int n4 = (N + 3) / 4;
  const int64_t total = (int64_t)M * n4;
  typename Epi::Sum sum{};
#pragma unroll 1
  for (int u = 0; u < Epi::REP; ++u) {
    const int64_t e = ((int64_t)blockIdx.x * Epi::REP + u) * 256 + threadIdx.x;
    if (e < total) {
      const int m = (int)(e / n4), nu = 4 * (int)(e % n4);
      const auto in = epi.load(m, 2 * nu);
      double c[8];
      mod_combine_c(R + (int64_t)m * ldr + nu, rstride, rs[m], cs, nu, N, c);
      const double lo[4] = {c[0], c[1], c[2], c[3]}, up[4] = {c[4], c[5], c[6], c[7]};
      epi(m, 2 * nu, lo, in, sum);
      if (nu + 2 < N) epi(m, 2 * nu + 4, up, epi.load(m, 2 * nu + 4), sum);
    }
  }
  epi.finish(sum);
}

// C(m, n) = alpha c
template <class TC>
struct ModStore {
  static constexpr int REP = 1;
  struct Sum {};
  TC* C;
  int64_t ldc;
  int N;
  double alpha;
  int vec;  // pairs of a row aligned
  struct In {};
  __device__ __forceinline__ In load(int, int) const { return {}; }
  __device__ __forceinline__ void operator()(int m, int n, const double (&c)[4], const In&, Sum&) const {
    TC* p = C + (int64_t)m * ldc + n;
    if (vec && n + 4 <= N) {
      typedef TC v2 __attribute__((ext_vector_type(2)));
      reinterpret_cast<v2*>(p)[0] = v2{(TC)(alpha * c[0]), (TC)(alpha * c[1])};
      reinterpret_cast<v2*>(p)[1] = v2{(TC)(alpha * c[2]), (TC)(alpha * c[3])};
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (n + e < N) p[e] = (TC)(alpha * c[e]);
    }
  }
  __device__ __forceinline__ void off() const {}
  __device__ __forceinline__ void finish(const Sum&) const {}
};

// -------------------------------------------------------------------- host
// Buffers of a product with up to `rows` rows of A per call, processed in
// panels of `mp` rows (planes of a panel: 17 bytes per entry of A and of C, 36
// per complex one).
struct ModWork {
  int8_t *a, *b, *r;
  double *ra, *rb, *d, *di;
  int* flags;  // [nflags]: [0] B, [1 + i] panel i
  int nflags;
  int64_t mp;  // 0: no buffers
  int kpad, ldr;
  int cplx;    // complex products
};

constexpr int64_t MOD_PANEL = 16384;
constexpr int MOD_KMAX_C = 8192;  // entries of a complex row held in registers by mod_split_c

// Whether the buffers are carved (the line that workspace sizes were given by).
static bool mod_room(int64_t M, int64_t N, int64_t K) {
  return M >= 2048 && K <= MOD_KMAX && K * N >= 512 * (K + N);
}
static bool mod_room_c(int64_t M, int64_t N, int64_t K) {
  return M >= 2048 && K <= MOD_KMAX_C && K * N >= 160 * (K + N);
}
// Whether residues beat the FP64 kernel, by the modelled time of a row of C: the
// FP64 product takes 2 K N / 66 TFLOP/s on whole 128-wide tiles; the residues 34
// K N / 2.4 POP/s on whole 256-wide tiles, with a prologue and an epilogue worth
// 256 terms, and 25 (K + N) bytes at 4.4 TB/s.  FP64 over residues at 16384
// rows: 1024 x 1024 1.03 measured, 1.05 modelled; 1100 1.25, 1.04; 1280 1.21,
// 1.17; 2048 1.40, 1.41.  A modelled gain below MOD_GAIN goes to the clock, which
// the int8 products lower for what runs beside them: the residual of 64^3 x 1024
// points 14.3 ms with the FP64 product, 15.5 with the residues.
constexpr double MOD_GAIN = 1.06;
static bool mod_pays(int64_t M, int64_t N, int64_t K) {
  const double fp64 = 2.0 * (double)K * (double)(ceil_div(N, 128) * 128) / 66e12;
  const double mod = 34.0 * (double)(K + 256) * (double)(ceil_div(N, MOD_T) * MOD_T) / 2.4e15 +
                     25.0 * (double)(K + N) / 4.4e12;
  return mod_room(M, N, K) && MOD_GAIN * mod <= fp64;
}
// The same for a complex product of N columns and K terms: 8 K N operations
// (tiles of 64 complex columns) against 72 K N and 52 K + 88 N bytes.  384 x 384
// 0.78 measured, 0.81 modelled; 448 1.02, 0.97; 512 1.13, 1.13; 768 1.60, 1.49.
static bool mod_pays_c(int64_t M, int64_t N, int64_t K) {
  const double fp64 = 8.0 * (double)K * (double)(ceil_div(N, 64) * 64) / 66e12;
  const double mod = 72.0 * (double)(K + 256) * (double)(ceil_div(N, MOD_T) * MOD_T) / 2.4e15 +
                     (52.0 * (double)K + 88.0 * (double)N) / 4.4e12;
  return mod_room_c(M, N, K) && MOD_GAIN * mod <= fp64;
}

static ModWork carve_planes(Carver& c, int64_t rows, int64_t N, int64_t K, int cplx) {
  ModWork w{};
  const int planes = cplx ? 2 * MOD_NC : MOD_N;
  w.cplx = cplx;
  w.mp = rows < MOD_PANEL ? rows : MOD_PANEL;
  w.kpad = (int)ceil_div(K, MOD_BK) * MOD_BK;
  w.ldr = (int)ceil_div(N, MOD_T) * MOD_T;
  w.nflags = (int)(1 + ceil_div(rows > N ? rows : N, w.mp));
  w.flags = c.take<int>(w.nflags);
  w.d = c.take<double>(K);
  w.di = c.take<double>(K);
  w.ra = c.take<double>(w.mp);
  w.rb = c.take<double>(N);
  w.b = c.take<int8_t>((size_t)planes * N * w.kpad);
  w.a = c.take<int8_t>((size_t)planes * w.mp * w.kpad);
  w.r = c.take<int8_t>((size_t)planes * w.mp * w.ldr);
  return w;
}
static ModWork carve_mod(Carver& c, int64_t rows, int64_t N, int64_t K) {
  return mod_room(rows, N, K) ? carve_planes(c, rows, N, K, 0) : ModWork{};
}
static ModWork carve_mod_c(Carver& c, int64_t rows, int64_t N, int64_t K) {
  return mod_room_c(rows, N, K) ? carve_planes(c, rows, N, K, 1) : ModWork{};
}
// Buffers of the products with an N1 x N1 operand: complex ones of half the
// order where the two orbital sets differ.
static ModWork carve_mod_for(Carver& c, int64_t rows, int64_t n1, bool aliased) {
  return aliased ? carve_mod(c, rows, n1, n1) : carve_mod_c(c, rows, n1 / 2, n1 / 2);
}

// Residues of the rows of X into planes `out`; complex rows when w.cplx.
template <class TS>
static bool mod_rows(const TS* X, int64_t ld, int rows, int K, const ModWork& w, const double* ks, bool conj,
                     int8_t* out, double* rscale, int* flag, const int* abort, hipStream_t s) {
  const int vec = ld % 2 == 0 && (uintptr_t)X % (2 * sizeof(TS)) == 0;
  const int kpad = w.kpad;
  const int64_t ps = (int64_t)rows * kpad;
  const dim3 grid((unsigned)rows), block(256);
  const auto launch = [&](auto it) {
    constexpr int IT = decltype(it)::value;
    if (w.cplx)
      hipLaunchKernelGGL((mod_split_c<TS, IT>), grid, block, 0, s, X, ld, rows, K, kpad, ks, vec, conj ? 1 : 0, out, ps,
                         rscale, flag, abort);
    else
      hipLaunchKernelGGL((mod_split<TS, IT>), grid, block, 0, s, X, ld, rows, K, kpad, ks, vec, out, ps, rscale, flag,
                         abort);
  };
  if (kpad <= 1024) launch(std::integral_constant<int, 1>());
  else if (kpad <= 2048) launch(std::integral_constant<int, 2>());
  else if (kpad <= 4096) launch(std::integral_constant<int, 4>());
  else if (kpad <= 8192) launch(std::integral_constant<int, 8>());
  else
    hipLaunchKernelGGL((mod_split<TS, 16>), grid, block, 0, s, X, ld, rows, K, kpad, ks, vec, out, ps, rscale, flag,
                       abort);
  return launch_ok();
}

// Where the powers of two come from that are moved between the operands: the
// diagonal of one of them (symmetric of order K), or the columns of both.
enum { MOD_DIAG_A = 1, MOD_DIAG_B = 2, MOD_MEANS = 3 };

// Raises the flag unless B (order 2 K) is the real 2 x 2 block form of a complex
// matrix, [[re, im], [-im, re]] per entry, whose even rows say it all: exactly
// for results in double (block_form makes the library's own matrices exact), to
// `tol` of the diagonals' geometric mean for results stored in single.  Any other
// matrix keeps the FP64 kernel.
constexpr double MOD_TOL_SINGLE = 0x1p-24;
__global__ __launch_bounds__(256) void mod_blocks(const double* __restrict__ B, int64_t ldb, int K, double tol,
                                                  int* flag) {
  const int i = blockIdx.y;
  const double* r0 = B + 2 * i * ldb;
  const double* r1 = r0 + ldb;
  const double di = r0[2 * i];
  for (int j = blockIdx.x * blockDim.x + threadIdx.x; j < K; j += gridDim.x * blockDim.x) {
    const double e = fabs(r0[2 * j] - r1[2 * j + 1]) + fabs(r0[2 * j + 1] + r1[2 * j]);
    if (!(e <= tol * sqrt(fabs(di * B[2 * j * (ldb + 1)])))) atomicOr(flag, 1);
  }
}

// Powers of two and residues of B (N x K), once per call; A: the other operand
// (M rows).  Complex (w.cplx): B is the real 2 x 2 block form of a complex N x K
// matrix, whose rows are the even ones, and the product is A B^H (bal =
// MOD_DIAG_B: N = K, checked by mod_blocks to `tol`).  MOD_MEANS: complex only.
template <class TA>
static bool mod_prepare(const TA* A, int64_t lda, int M, const double* B, int64_t ldb, int N, int K, int bal,
                        double tol, const ModWork& w, const int* abort, hipStream_t s) {
  const int step = w.cplx ? 2 : 1;
  hipLaunchKernelGGL(mod_clear, dim3(1), dim3(256), 0, s, w.flags, w.nflags);
  if (bal == MOD_MEANS) {
    hipLaunchKernelGGL((mod_means<TA>), dim3((unsigned)ceil_div(K, 32)), dim3(256), 0, s, A, lda, M, B, 2 * ldb, N, K,
                       w.d, w.di);
  } else {
    const double* m = bal == MOD_DIAG_A ? (const double*)A : B;
    hipLaunchKernelGGL(mod_diag, dim3((unsigned)ceil_div(K, 256)), dim3(256), 0, s, m, bal == MOD_DIAG_A ? lda : ldb, K,
                       step, w.d, w.di);
  }
  if (w.cplx && bal == MOD_DIAG_B)
    hipLaunchKernelGGL(mod_blocks, dim3((unsigned)ceil_div(K, 1024), (unsigned)K), dim3(256), 0, s, B, ldb, K, tol,
                       w.flags);
  return mod_rows<double>(B, step * ldb, N, K, w, bal == MOD_DIAG_A ? w.d : w.di, true, w.b, w.rb, w.flags, abort, s);
}

// Another product with the same B: the panels' flags of the last one go (a flag
// left there would keep these panels on the FP64 kernel).
static bool mod_next(const ModWork& w, hipStream_t s) {
  hipLaunchKernelGGL(mod_clear, dim3(1), dim3(256), 0, s, w.flags + 1, w.nflags - 1);
  return launch_ok();
}

template <class Epi>
static int64_t mod_crt_blocks(int64_t rows, int64_t N) {
  return ceil_div(rows * ceil_div(N, 4), 256 * Epi::REP);
}

// One panel (at most w.mp rows): residues of its rows of A, the residue
// products, and the results through `epi`.  N, K in complex entries when
// w.cplx.
template <class TA, class Epi>
static bool mod_panel(const TA* A, int64_t lda, int rows, int N, int K, int bal, int panel, const ModWork& w,
                      const Epi& epi, const int* abort, hipStream_t s) {
  int* aflag = w.flags + 1 + panel;
  if (!mod_rows<TA>(A, lda, rows, K, w, bal == MOD_DIAG_A ? w.di : w.d, false, w.a, w.ra, aflag, abort, s))
    return false;
  const int64_t tiles = ceil_div(rows, MOD_T) * ceil_div(N, MOD_T);
  const dim3 grid((unsigned)(tiles * (w.cplx ? 2 * MOD_NC : MOD_N)));
  const dim3 crt((unsigned)mod_crt_blocks<Epi>(rows, N));
  const int64_t as = (int64_t)rows * w.kpad, bs = (int64_t)N * w.kpad, rs = (int64_t)rows * w.ldr;
  const int8_t *a = w.a, *b = w.b, *r = w.r;
  const int *bf = w.flags, *af = aflag;
  const double *ra = w.ra, *rb = w.rb;
  if (w.cplx) {
    hipLaunchKernelGGL(mod_gemm<true>, grid, dim3(MOD_THREADS), 0, s, a, as, b, bs, w.kpad, rows, N, w.r, rs, w.ldr,
                       abort, bf, af);
    hipLaunchKernelGGL((mod_crt_c<Epi>), crt, dim3(256), 0, s, r, rs, w.ldr, rows, N, ra, rb, abort, bf, af, epi);
  } else {
    hipLaunchKernelGGL(mod_gemm<false>, grid, dim3(MOD_THREADS), 0, s, a, as, b, bs, w.kpad, rows, N, w.r, rs, w.ldr,
                       abort, bf, af);
    hipLaunchKernelGGL((mod_crt<Epi>), crt, dim3(256), 0, s, r, rs, w.ldr, rows, N, ra, rb, abort, bf, af, epi);
  }
  return launch_ok();
}

}  // namespace
}  // namespace isdf
