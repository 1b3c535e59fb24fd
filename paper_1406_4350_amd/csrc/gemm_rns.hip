// Large FP64 complex products on the INT8 matrix cores, by exact integer arithmetic in a residue number system.
//
// The FP64 matrix cores do 78.6 TFLOP/s and the INT8 ones about 5 POP/s, 64 times as much. Each operand vector (a row
// of op(A), a column of B) is scaled by a power of two to a 2-norm in [2^60, 2^61) and rounded to integers; the
// product of the integer matrices is computed exactly, modulo kRnsMods pairwise coprime numbers p below 2^8, as one
// int8 x int8 -> int32 product per modulus and real product; the Chinese remainder theorem gives the integers back.
// By Cauchy-Schwarz every entry (real or imaginary) is below 2^122 <= prod p / 4 in magnitude, so nothing overflows
// whatever the data, and the only errors are the roundings of the operands (at most 1/2 in integers of norm 2^60 ... 2^61,
// 2^-61.3 |a| |b| per entry in the mean square at most) and one rounding of the result. They are relative to the norms,
// where those of an FP64 product follow sum |a_k b_k|: a chain of K / 4 FP64 MFMAs leaves about 2^-53 0.3 sqrt(chain / K)
// |a| |b| (chain: the K range that one accumulator sums) where the two vectors overlap, and less where they do not. A
// column of B therefore takes this route only if sum_k |a_k b_k| >= kRnsOverlap |a| |b| for every row a, which the
// envelope env_k = min over the rows of |a_k| / |a|, kept with A's planes, bounds from below by sum_k env_k |b_k|: its
// error is then in the mean square at most 2^-61.3 / 2^-8 = 2^-53.3 of sum |a_k b_k|, what FP64 leaves too. The other
// columns, flagged, take the FP64 product. Blocks of a plane-wave calculation pass: the envelope bounds measured 0.03 to
// 0.27 for P^H x (the overlaps themselves 0.16 to 0.67) and 0.007 to 0.2 for P w (0.04 to 0.46), from random smooth
// blocks to converged ones. There, entry by entry against extended precision (17 077 plane waves, 832 projectors, 512
// bands), in units of 2^-53 sum |a_k b_k|: largest error 0.06 to 0.25 and 0.018 to 0.032 in the mean square (mostly the
// rounding of the result), from the FP64 product 3.1 to 20 and 0.58 to 1.5. With 15 moduli (2^57) the same bound would
// need an overlap 16 times as large, which the envelope bounds of P w do not reach.
//
// The scheme (residues of scaled integers, one INT8 product per modulus, Chinese remaindering) is the one that Ozaki,
// Uchino and Imamura published as Ozaki scheme II (arXiv:2504.08009); moduli, splitting, kernels and guard are this file's.
//
// A complex product takes three real ones, P1 = a_r b_r, P2 = a_i b_i, P3 = (a_r + s a_i)(b_r + b_i), re = P1 - s P2,
// im = P3 - P1 - s P2 (s = -1 for conj(a) b, 1 for a b): exact here, since everything is modulo p.
// Operands arrive as int8 planes (per modulus: residues of the real parts, of the imaginary parts and of the sum),
// K contiguous; the projectors' planes are laid out once with the plan, the other operand's per call.
#include <algorithm>
#include <cmath>
#include <cstdlib>

#include "gemm_common.h"
#include "kernels.h"

namespace chebfd {
namespace {

constexpr int L = kRnsMods;
// 256, then the largest numbers below 242 that are pairwise coprime. The split leaves residues of the odd ones within
// +-kResMax (one above (p - 1) / 2 at 241: its reduction rounds in float), and the one-step reductions of their products
// (error at most 6) stay inside the int8 range.
constexpr int kP[16] = {256, 241, 239, 235, 233, 229, 227, 223, 221, 217, 211, 209, 199, 197, 193, 191};
static_assert(L <= 16, "moduli");

typedef unsigned __int128 u128;
constexpr u128 rns_modulus() {
  u128 m = 1;
  for (int l = 0; l < L; ++l) m *= u128(kP[l]);
  return m;
}
constexpr int rns_bits() {  // M < 2^bits
  int b = 0;
  for (u128 m = rns_modulus(); m; m >>= 1) ++b;
  return b;
}
constexpr bool rns_coprime() {
  for (int i = 0; i < L; ++i)
    for (int j = 0; j < i; ++j) {
      int a = kP[i], b = kP[j];
      while (b) { const int t = a % b; a = b; b = t; }
      if (a != 1) return false;
    }
  return true;
}
static_assert(rns_coprime(), "moduli must be pairwise coprime");
// operand norms: 2^kNormExp per operand, twice that two bits below M
constexpr int kNormExp = (rns_bits() - 1 - 2) / 2;
static_assert(kNormExp <= 61, "the split takes integers up to 2^61");

constexpr double u128_to_double(u128 v) {  // exact for values of at most 53 significant bits
  double r = 0.0, f = 1.0;
  for (; v; v >>= 32, f *= 4294967296.0) r += f * double(unsigned(v & 0xffffffffu));
  return r;
}
// Weights w_l = (M / p_l) ((M / p_l)^-1 mod p_l) of the Chinese remainder theorem in two parts of 40 bits, w1 a
// multiple of 2^(bits - 40) and w2 of 2^(bits - 80). What is left out (below 2^45 per weight, 2^57.6 in a sum, of results
// up to 2^122 |a| |b|) is a few per cent of the rounding of the operands. Sums of kRnsMods such parts times residues (at
// most 384 in magnitude) are exact in FP64.
struct Crt {
  double w1[L], w2[L], m1, m2, minv;
};
constexpr Crt make_crt() {
  Crt c{};
  const u128 M = rns_modulus();
  constexpr int s1 = rns_bits() - 40, s2 = rns_bits() - 80;
  for (int l = 0; l < L; ++l) {
    const u128 q = M / u128(kP[l]);
    const int r = int(q % u128(kP[l]));
    int inv = 1;
    while ((r * inv) % kP[l] != 1) ++inv;
    const u128 w = q * u128(inv);
    c.w1[l] = u128_to_double((w >> s1) << s1);
    c.w2[l] = u128_to_double(((w & ((u128(1) << s1) - 1)) >> s2) << s2);
  }
  c.m1 = u128_to_double((M >> s1) << s1);
  c.m2 = u128_to_double(((M & ((u128(1) << s1) - 1)) >> s2) << s2);
  c.minv = 1.0 / (c.m1 + c.m2);
  return c;
}
constexpr Crt kCrt = make_crt();
constexpr int sym_mod(long long v, int p) {
  int r = int(v % p);
  if (r < 0) r += p;
  return r > p / 2 ? r - p : r;
}

struct ModTab { int p[L]; float inv[L]; int c16[L]; };  // c16 = 2^16 mod p
constexpr ModTab make_tab() {
  ModTab t{};
  for (int l = 0; l < L; ++l) { t.p[l] = kP[l]; t.inv[l] = 1.0f / float(kP[l]); t.c16[l] = sym_mod(1 << 16, kP[l]); }
  return t;
}
__constant__ ModTab kTab = make_tab();

// x - p round(x / p) for |x| < 2^22 p: the float product added to 1.5 2^23 leaves the rounded quotient in the low
// mantissa bits. Exact up to the rounding of x to float: |result| <= p / 2 + 2^-24 |x| + |x - float(x)|.
constexpr float kMagic = 12582912.0f;
constexpr int kMagicBits = 0x4B400000;
__host__ __device__ __forceinline__ int mul24(int a, int b) {
#ifdef __HIP_DEVICE_COMPILE__
  return __mul24(a, b);
#else
  return a * b;
#endif
}
__host__ __device__ __forceinline__ int mod_step(int x, int p, float inv) {
  const int q = __builtin_bit_cast(int, fmaf(float(x), inv, kMagic)) - kMagicBits;
  return x - mul24(q, p);
}
// the low byte of the same: the constant of kMagicBits drops out modulo 256
__device__ __forceinline__ unsigned mod_byte(int x, int p, float inv) {
  return unsigned(x - mul24(__builtin_bit_cast(int, fmaf(float(x), inv, kMagic)), p));
}
__device__ __forceinline__ unsigned pack4(unsigned a, unsigned b, unsigned c, unsigned d) {  // low bytes
  const unsigned lo = __builtin_amdgcn_perm(b, a, 0x0c0c0400u), hi = __builtin_amdgcn_perm(d, c, 0x04000c0cu);
  return lo | hi;
}

// ---- scales ------------------------------------------------------------------------------------------------
// A vector of norm f 2^x (f in [1/2, 1)) is scaled by 2^(kNormExp - x). Returns whether it is fit for the integers: not
// one with a NaN or Inf, or whose largest entry is not 0 and outside [1e-130, 1e130].
__device__ __forceinline__ bool set_scale(double ss, double mx, double* scale, double* inv) {
  const bool zero = mx == 0.0 && ss == 0.0;
  const bool ok = zero || (mx >= 1e-130 && mx <= 1e130 && ss < 1e300);
  int x = 0;
  if (ok && !zero) (void)frexp(sqrt(ss), &x);
  *scale = ldexp(1.0, kNormExp - x);
  *inv = ldexp(1.0, x - kNormExp);
  return ok;
}
// 1 / norm, 0 for a vector of zeros (which the envelopes leave out)
__device__ __forceinline__ double rnorm_of(double ss) { return ss > 0.0 ? 1.0 / sqrt(ss) : 0.0; }

// flag[n] = 1 for a column that is not fit or, with env, whose overlap with some row of A may be below kRnsOverlap (the
// larger component stands for the modulus); *any = 1 if one is. Bound by memory; env stays in L2.
constexpr int NST = 1024;
template <typename E>
__global__ __launch_bounds__(NST) void k_rns_colnorm(long K, const cx<E>* __restrict__ B, long ldb,
                                                     const double* __restrict__ env, double* scale, double* inv,
                                                     double* rnorm, int* flag, int* any) {
  __shared__ double rs[NST / 64], rm[NST / 64], ro[NST / 64];
  const cx<E>* col = B + long(blockIdx.x) * ldb;
  double ss = 0.0, mx = 0.0, ov = 0.0;
  for (long i = threadIdx.x; i < K; i += NST) {
    const cx<E> v = col[i];
    const double x = fabs(double(v.x)), y = fabs(double(v.y)), m = fmax(x, y);
    ss += x * x + y * y;
    mx = fmax(mx, m);
    if (env) ov = fma(env[i], m, ov);
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    ss += __shfl_xor(ss, o, 64);
    mx = fmax(mx, __shfl_xor(mx, o, 64));
    ov += __shfl_xor(ov, o, 64);
  }
  if ((threadIdx.x & 63) == 0) { rs[threadIdx.x >> 6] = ss; rm[threadIdx.x >> 6] = mx; ro[threadIdx.x >> 6] = ov; }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < NST / 64; ++w) { ss += rs[w]; mx = fmax(mx, rm[w]); ov += ro[w]; }
    const int n = blockIdx.x;
    bool ok = set_scale(ss, mx, scale + n, inv + n);
    if (env && mx != 0.0) ok = ok && ov >= kRnsOverlap * sqrt(ss);
    if (rnorm) rnorm[n] = rnorm_of(ss);
    if (flag) flag[n] = ok ? 0 : 1;
    if (any && !ok) *any = 1;
  }
}

// rows of an M x K matrix stored with the rows contiguous: one thread per row; with the columns' 1 / norms also the
// columns' envelope, env[m] = min_k |A[m][k]| / |column k|
template <typename E>
__global__ __launch_bounds__(256) void k_rns_rownorm(long M, int K, const cx<E>* __restrict__ A, long lda,
                                                     double* scale, double* inv, double* rnorm,
                                                     const double* __restrict__ cnorm, double* env, int* any) {
  const long m = long(blockIdx.x) * 256 + threadIdx.x;
  if (m >= M) return;
  double ss = 0.0, mx = 0.0, lo = 1.0;
#pragma unroll 8
  for (int k = 0; k < K; ++k) {
    const cx<E> v = A[m + long(k) * lda];
    const double x = double(v.x), y = double(v.y), q = x * x + y * y, c = cnorm[k];
    ss += q;
    mx = fmax(mx, fmax(fabs(x), fabs(y)));
    lo = c > 0.0 ? fmin(lo, q * c * c) : lo;
  }
  if (!set_scale(ss, mx, scale + m, inv + m)) *any = 1;
  rnorm[m] = rnorm_of(ss);
  env[m] = sqrt(lo);
}
// the rows' envelope, env[k] = min_m |A[m][k]| / |row m|: one block per column
template <typename E>
__global__ __launch_bounds__(NST) void k_rns_rowenv(long M, const cx<E>* __restrict__ A, long lda,
                                                    const double* __restrict__ rnorm, double* env) {
  __shared__ double red[NST / 64];
  const cx<E>* col = A + long(blockIdx.x) * lda;
  double lo = 1.0;
  for (long m = threadIdx.x; m < M; m += NST) {
    const cx<E> v = col[m];
    const double x = double(v.x), y = double(v.y), c = rnorm[m];
    lo = c > 0.0 ? fmin(lo, (x * x + y * y) * c * c) : lo;
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) lo = fmin(lo, __shfl_xor(lo, o, 64));
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = lo;
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < NST / 64; ++w) lo = fmin(lo, red[w]);
    env[blockIdx.x] = sqrt(lo);
  }
}
// the overlap that an envelope leaves a vector of K equal entries
__global__ __launch_bounds__(NST) void k_rns_flat(long K, const double* __restrict__ env, double* out) {
  __shared__ double red[NST / 64];
  double s = 0.0;
  for (long k = threadIdx.x; k < K; k += NST) s += env[k];
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < NST / 64; ++w) s += red[w];
    *out = s / sqrt(double(K));
  }
}

// ---- operands to residues ------------------------------------------------------------------------------------
// y = d3 2^48 + d2 2^32 + d1 2^16 + d0 with |d3| <= 2^13 and |d2|, |d1|, |d0| <= 2^15 for |y| <= 2^61, y rounded to an
// integer: sums of digits times residues stay exact as floats
struct Digits { int d3, d2, d1, d0; };
__device__ __forceinline__ Digits digits(double y) {
  const double h = rint(y * 0x1p-48);
  const double r = fma(-h, 0x1p48, y);
  const double g = rint(r * 0x1p-32);
  const double q = fma(-g, 0x1p32, r);
  const double f = rint(q * 0x1p-16);
  return {int(h), int(g), int(f), int(rint(fma(-f, 0x1p16, q)))};
}
// residues modulo kP[l] of NV complex integers, as bytes packed by four: re, im and re + im or (DIFF) re - im. |sum of digits times powers| <= split_max < 2^24, of which one step leaves at most
// kResMax modulo the odd numbers (p / 2 + 1/2 + 2^-24 split_max: 121 modulo 241).
constexpr int split_max(int p) {
  int s = 1 << 15;
  for (int e = 1; e < 4; ++e) {
    const int c = sym_mod(1ll << (16 * e), p);
    s += (c < 0 ? -c : c) * (1 << (e == 3 ? 13 : 15));
  }
  return s;
}
constexpr int kResMax = 121;
template <int NV, bool DIFF>
__device__ __forceinline__ void residues(int l, const Digits (&re)[NV], const Digits (&im)[NV], unsigned (&pr)[NV / 4],
                                         unsigned (&pi)[NV / 4], unsigned (&pt)[NV / 4]) {
  const int p = kP[l];
  const float inv = 1.0f / float(p);
  const int c3 = sym_mod(1ll << 48, p), c2 = sym_mod(1ll << 32, p), c1 = sym_mod(1ll << 16, p);
#pragma unroll
  for (int g = 0; g < NV / 4; ++g) {
    int r[4], i[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const Digits& a = re[4 * g + j];
      const Digits& b = im[4 * g + j];
      r[j] = mod_step(mul24(a.d3, c3) + mul24(a.d2, c2) + mul24(a.d1, c1) + a.d0, p, inv);
      i[j] = mod_step(mul24(b.d3, c3) + mul24(b.d2, c2) + mul24(b.d1, c1) + b.d0, p, inv);
    }
    pr[g] = pack4(unsigned(r[0]), unsigned(r[1]), unsigned(r[2]), unsigned(r[3]));
    pi[g] = pack4(unsigned(i[0]), unsigned(i[1]), unsigned(i[2]), unsigned(i[3]));
    int t[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) t[j] = DIFF ? r[j] - i[j] : r[j] + i[j];
    pt[g] = pack4(mod_byte(t[0], p, inv), mod_byte(t[1], p, inv), mod_byte(t[2], p, inv), mod_byte(t[3], p, inv));
  }
}

// Vectors contiguous along k (columns of B, columns of A under a conjugate transpose): 4 k per thread, so a wave
// reads 4 KB and writes 256 bytes of each plane. Bound by memory: 16 bytes read, 3 kRnsMods written per element. A column
// n with flag[n fs] set is left unwritten (its products are not used).
template <typename E, bool DIFF>
__global__ __launch_bounds__(256) void k_rns_split(long K, const cx<E>* __restrict__ B, long ldb,
                                                   const double* __restrict__ scale, int8_t* __restrict__ base,
                                                   int8_t* __restrict__ third, long plane, long ld, const int* __restrict__ flag, int fs) {
  const long k = (long(blockIdx.x) * 256 + threadIdx.x) * 4;
  const long n = blockIdx.y;
  if (k >= ld || flag[n * fs]) return;
  const double s = scale[n];
  const cx<E>* col = B + n * ldb;
  Digits re[4], im[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const cx<E> v = col[min(k + j, K - 1)];
    const bool in = k + j < K;
    re[j] = digits(in ? double(v.x) * s : 0.0);
    im[j] = digits(in ? double(v.y) * s : 0.0);
  }
  const long at = n * ld + k;
#pragma unroll
  for (int l = 0; l < L; ++l) {
    unsigned pr[1], pi[1], pt[1];
    residues<4, DIFF>(l, re, im, pr, pi, pt);
    if (base) {
      *reinterpret_cast<unsigned*>(base + (2 * l) * plane + at) = pr[0];
      *reinterpret_cast<unsigned*>(base + (2 * l + 1) * plane + at) = pi[0];
    }
    *reinterpret_cast<unsigned*>(third + l * plane + at) = pt[0];
  }
}

// Vectors strided along k (rows of A, stored with the rows contiguous): a block takes 64 rows by 64 k, lane = row,
// 16 k per thread, so reads are 1 KB per wave and k, and each row of each plane is written 16 bytes at a time.
template <typename E>
__global__ __launch_bounds__(256) void k_rns_split_rows(long M, int K, const cx<E>* __restrict__ A, long lda,
                                                        const double* __restrict__ scale, int8_t* __restrict__ base,
                                                        int8_t* __restrict__ sum, long plane, long ld,
                                                        const int* __restrict__ flag) {
  if (*flag) return;
  const long m = long(blockIdx.x) * 64 + (threadIdx.x & 63);
  const int k0 = int(blockIdx.y) * 64 + (threadIdx.x >> 6) * 16;
  if (m >= M || k0 >= ld) return;
  const double s = scale[m];
  Digits re[16], im[16];
#pragma unroll
  for (int j = 0; j < 16; ++j) {
    const cx<E> v = A[m + long(min(k0 + j, K - 1)) * lda];
    const bool in = k0 + j < K;
    re[j] = digits(in ? double(v.x) * s : 0.0);
    im[j] = digits(in ? double(v.y) * s : 0.0);
  }
  const long at = m * ld + k0;
#pragma unroll
  for (int l = 0; l < L; ++l) {
    unsigned pr[4], pi[4], ps[4];
    residues<16, false>(l, re, im, pr, pi, ps);
    *reinterpret_cast<uint4*>(base + (2 * l) * plane + at) = uint4{pr[0], pr[1], pr[2], pr[3]};
    *reinterpret_cast<uint4*>(base + (2 * l + 1) * plane + at) = uint4{pi[0], pi[1], pi[2], pi[3]};
    *reinterpret_cast<uint4*>(sum + l * plane + at) = uint4{ps[0], ps[1], ps[2], ps[3]};
  }
}

// ---- the int8 products ---------------------------------------------------------------------------------------
typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef int i32x16 __attribute__((ext_vector_type(16)));

constexpr int RT = 256;         // output tile (both ways), 4 waves of 128 x 128
constexpr int RK = kRnsKTile;   // k per LDS stage
constexpr int RCH = RK / 16;    // 16-byte chunks of a stage row
constexpr int kStageBytes = 2 * RT * RK;
// |accumulator| <= kResMax^2 k (modulo 256 it may wrap): K up to kRnsMaxK fits int32, and up to kDirectK the one-byte
// reduction takes it as it is; beyond, its upper half is folded first: |x| <= 2^15 120 + 2^16, exact as a float
constexpr int kDirectK = 4480;
static_assert(long(kRnsMaxK) * kResMax * kResMax < (1l << 31), "accumulator range");
static_assert(long(kDirectK) * kResMax * kResMax <= (1l << 26), "accumulator range of the one-byte reduction");

// chunk c of stage row r sits at chunk c ^ (r / 2 % 8): 16 consecutive rows read at one c touch all 64 LDS banks
__device__ __forceinline__ int stage_at(int r, int c) { return r * RK + ((c ^ ((r >> 1) & 7)) << 4); }

// C[z][n][m] (residues as int8, m contiguous, ldc) = sum_k A_z[m][k] B_z[n][k] modulo kP[z / 3], z = 3 l + product.
// One wave per SIMD holds a 128 x 128 tile (256 accumulators) on the 32x32x32 int8 MFMA; the LDS holds two stages of
// 128 k. While tile t is multiplied, tile t + 1 goes from registers to the other stage and tile t + 2 is requested
// from memory, one 16-byte access behind each MFMA (sched_group_barrier), and the fragments of the next 32 k are read
// one step ahead, across the one barrier of the tile: the MFMAs never wait on a whole group of loads. Measured at
// 3328 x 512 x 32768, 45 products (15 moduli): 2070 TOP/s against 1890 without the two stages as separate arrays (the compiler
// then orders reads behind writes), 1560 without the interleaving, and 3100 for the MFMAs alone: power is
// the limit (in a filter of 2048 bands at 128^3 the matrix cores are 81% busy at 1.36 GHz in P^H x and 64% at 1.61 GHz in
// P w, whose tiles of 3328 k are short). Loads straight to LDS measured 5% slower; persistent blocks that request
// the next output tile's operands during the last k tiles of this one left too few registers for the reduction of the
// accumulators and took 31 instead of 22 us per tile at 1024 k.
__global__ __launch_bounds__(256, 1) void k_rns_gemm(int M, int N, int nt, RnsOperand A, RnsOperand B,
                                                     int8_t* __restrict__ C, long ldc, long zc,
                                                     const int* __restrict__ flag) {
  __shared__ __align__(16) int8_t S0[kStageBytes], S1[kStageBytes];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int tm = (M + RT - 1) / RT, tn = (N + RT - 1) / RT;
  // one contiguous run of tiles per XCD, the N tile fastest: the blocks an XCD holds at once share their operands in L2
  int bx, by, z;
  gemm_tile_of(blockIdx.x, gridDim.x, tm, tn, 1, bx, by, z);
  const int m0 = bx * RT, n0 = by * RT, l = z / 3, c3 = z - 3 * l;
  bool some = false;  // a column of the tile takes this route
#pragma unroll
  for (int i = 0; i < RT; i += 64) some = some || (n0 + i + lane < N && flag[n0 + i + lane] == 0);
  if (!__any(some)) return;
  const int8_t* Az = c3 < 2 ? A.base + (2 * l + c3) * A.plane : A.third + l * A.third_plane;
  const int8_t* Bz = c3 < 2 ? B.base + (2 * l + c3) * B.plane : B.third + l * B.third_plane;

  // loaders: 16-byte chunk tid % 8 of rows tid / 8 + 32 i of each tile, rows past M or N clamped (they feed only outputs
  // that are not used); 32-bit offsets from the tiles' first rows
  constexpr int NL = 2 * RT * RCH / 256;
  static_assert(RCH == 8 && NL == 16, "loader roles");
  const int8_t* Ab = Az + long(m0) * A.ld;
  const int8_t* Bb = Bz + long(n0) * B.ld;
  unsigned src[NL];
#pragma unroll
  for (int i = 0; i < NL; ++i) {
    const int row = (i & 7) * 32 + (tid >> 3);
    src[i] = unsigned(i < 8 ? min(row, M - 1 - m0) : min(row, N - 1 - n0)) * unsigned(A.ld) + (tid & 7) * 16;
  }
  const int dst = stage_at(tid >> 3, tid & 7);  // + 32 i rows: the swizzle repeats every 16 rows
  i32x4 g[NL];
  const int wm = (wave & 1) * 128, wn = (wave >> 1) * 128, fr = lane & 31, fh = lane >> 5;
  constexpr int KS = RK / 32;
  i32x16 acc[4][4];
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int b = 0; b < 4; ++b)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[a][b][v] = 0;
  auto load_i = [&](int i, int k0) { g[i] = *reinterpret_cast<const i32x4*>((i < 8 ? Ab : Bb) + k0 + src[i]); };
  auto put_i = [&](int i, int8_t* S) { *reinterpret_cast<i32x4*>(S + dst + i * 32 * RK) = g[i]; };
  // the int8 MFMA takes row (lane % 32) of either operand at 16 (lane / 32) ... + 15 of its 32 k
  auto frag = [&](const int8_t* S, int ks, i32x4(&fa)[4], i32x4(&fb)[4]) {
#pragma unroll
    for (int a = 0; a < 4; ++a)
      fa[a] = *reinterpret_cast<const i32x4*>(S + stage_at(wm + 32 * a + fr, 2 * ks + fh));
#pragma unroll
    for (int a = 0; a < 4; ++a)
      fb[a] = *reinterpret_cast<const i32x4*>(S + stage_at(RT + wn + 32 * a + fr, 2 * ks + fh));
  };
  auto mul = [&](const i32x4(&fa)[4], const i32x4(&fb)[4]) {
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
      for (int b = 0; b < 4; ++b) acc[a][b] = __builtin_amdgcn_mfma_i32_32x32x32_i8(fa[a], fb[b], acc[a][b], 0, 0, 0);
  };
#pragma unroll
  for (int i = 0; i < NL; ++i) load_i(i, 0);
#pragma unroll
  for (int i = 0; i < NL; ++i) put_i(i, S0);
#pragma unroll
  for (int i = 0; i < NL; ++i) load_i(i, min(1, nt - 1) * RK);
  __syncthreads();
  i32x4 fa[2][4], fb[2][4];
  frag(S0, 0, fa[0], fb[0]);
  // tile t from stage Sa; the last tiles request (and store) the last tile again, which nothing reads
  auto step = [&](int t, int8_t* Sa, int8_t* Sb) {
    const int kn = min(t + 2, nt - 1) * RK;
    constexpr int PER = (NL + KS - 2) / (KS - 1);
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      if (ks + 1 < KS) {
        frag(Sa, ks + 1, fa[(ks + 1) & 1], fb[(ks + 1) & 1]);
#pragma unroll
        for (int i = ks * PER; i < (ks + 1) * PER && i < NL; ++i) { put_i(i, Sb); load_i(i, kn); }
        mul(fa[ks & 1], fb[ks & 1]);
#pragma unroll
        for (int q = 0; q < 8; ++q) {  // MFMA, LDS read, MFMA, LDS write, global load
          __builtin_amdgcn_sched_group_barrier(0x8, 1, 0);
          __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
          __builtin_amdgcn_sched_group_barrier(0x8, 1, 0);
          __builtin_amdgcn_sched_group_barrier(0x200, 1, 0);
          __builtin_amdgcn_sched_group_barrier(0x20, 1, 0);
        }
      } else {
        __syncthreads();
        frag(Sb, 0, fa[(ks + 1) & 1], fb[(ks + 1) & 1]);
        mul(fa[ks & 1], fb[ks & 1]);
#pragma unroll
        for (int q = 0; q < 8; ++q) {
          __builtin_amdgcn_sched_group_barrier(0x8, 2, 0);
          __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
        }
      }
    }
  };
  const int p = kTab.p[l];
  const float inv = kTab.inv[l];
  int it = 0;
  for (; it + 1 < nt; it += 2) { step(it, S0, S1); step(it + 1, S1, S0); }
  if (it < nt) step(it, S0, S1);

  // bytes through the wave's own 16 KB of LDS (row n: 8 chunks of 16 m) to 128-byte rows.
  // Accumulator v of a lane: row 8 (v / 4) + 4 (lane / 32) + v % 4, column lane % 32 of its 32 x 32 block.
  __syncthreads();
  int8_t* W = S0 + wave * 128 * 128;
  const int c16 = kTab.c16[l];
  auto bytes = [&](auto fold) {
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
      for (int b = 0; b < 4; ++b) {
#pragma unroll
        for (int v = 0; v < 16; v += 4) {
          unsigned x[4];
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            int y = acc[a][b][v + j];
            if constexpr (decltype(fold)::value) y = mul24(y >> 16, c16) + (y & 0xffff);
            x[j] = mod_byte(y, p, inv);
          }
          const int m = 32 * a + 2 * v + 4 * fh, n = 32 * b + fr;
          *reinterpret_cast<unsigned*>(W + stage_at(n, m >> 4) + (m & 15)) = pack4(x[0], x[1], x[2], x[3]);
        }
        __builtin_amdgcn_sched_barrier(0);  // one block at a time: all 256 at once would not fit the registers
      }
  };
  if (nt * RK > kDirectK) bytes(std::true_type{});
  else bytes(std::false_type{});
  __syncthreads();
  const int cc = lane & 7, rr = lane >> 3;
  const long m = m0 + wm + 16 * cc;
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    const int n = 8 * i + rr;
    const i32x4 v = *reinterpret_cast<const i32x4*>(W + stage_at(n, cc));
    if (n0 + wn + n < N && m < ldc) *reinterpret_cast<i32x4*>(C + z * zc + long(n0 + wn + n) * ldc + m) = v;
  }
}
static_assert(kStageBytes == 4 * 128 * 128, "the output bytes of a block fill one stage");

// ---- residues to results -------------------------------------------------------------------------------------
// 4 m per thread from the 3 kRnsMods planes (256 bytes of each per wave), then the epilogue with m across the lanes
// (through LDS). Bound by memory.
template <typename EO>
__global__ __launch_bounds__(256) void k_rns_finish(int M, int N, const int8_t* __restrict__ C, long ldc, long zc,
                                                    const double* __restrict__ ia, const double* __restrict__ ib,
                                                    int sg, Epi<EO> epi, const int* __restrict__ flag) {
  __shared__ c128 buf[1024];
  const long mb = long(blockIdx.x) * 1024, n = blockIdx.y;
  if (flag[n]) return;
  const int t = threadIdx.x;
  const long m4 = mb + 4 * t;
  if (m4 < ldc) {
    const int8_t* c = C + n * ldc + m4;
    unsigned w[3 * L];
#pragma unroll
    for (int z = 0; z < 3 * L; ++z) w[z] = *reinterpret_cast<const unsigned*>(c + z * zc);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      double r1 = 0.0, r2 = 0.0, i1 = 0.0, i2 = 0.0;
#pragma unroll
      for (int l = 0; l < L; ++l) {
        const int x1 = int(w[3 * l] << (24 - 8 * j)) >> 24, x2 = sg * (int(w[3 * l + 1] << (24 - 8 * j)) >> 24),
                  x3 = int(w[3 * l + 2] << (24 - 8 * j)) >> 24;
        const double re = double(x1 - x2), im = double(x3 - x1 - x2);
        r1 = fma(re, kCrt.w1[l], r1);
        r2 = fma(re, kCrt.w2[l], r2);
        i1 = fma(im, kCrt.w1[l], i1);
        i2 = fma(im, kCrt.w2[l], i2);
      }
      const double qr = rint(r1 * kCrt.minv), qi = rint(i1 * kCrt.minv);
      buf[4 * t + j] = c128{fma(-qr, kCrt.m1, r1) + fma(-qr, kCrt.m2, r2), fma(-qi, kCrt.m1, i1) + fma(-qi, kCrt.m2, i2)};
    }
  }
  __syncthreads();
  const double sb = ib[n];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const long m = mb + 256 * j + t;
    if (m < M) {
      const double s = ia[m];
      const c128 v = buf[256 * j + t];
      epi_store(epi, m, n, v.x * s * sb, v.y * s * sb);
    }
  }
}

}  // namespace

int rns_residue_largest(int l, int x0, int x1) {
  const int p = kP[l];
  const float inv = 1.0f / float(p);
  int big = 0;
  for (int x = x0; x < x1; ++x) big = std::max(big, std::abs(mod_step(x, p, inv)));
  return big;
}
void rns_residue_limits(int* modulus, int l, int* sum, int* residue) {
  *modulus = kP[l];
  *sum = split_max(kP[l]);
  *residue = kP[l] % 2 ? kResMax : 128;
}

// Microseconds of both routes, from what they measured. FP64: one 64 x 64 tile of a CU's takes 0.0955 us per k, the tiles
// of a CU share its matrix cores (whole tiles per CU, from the tiles and splits that gemm() launches), then the split-K
// partials. INT8: a 256 x 256 tile takes 0.0138 us per k and 3.5 us to fill and empty, in rounds of 256 tiles (the first
// ones faster: few blocks leave the clock higher), or the A planes read once at 4.2 TB/s where few columns share them; the
// operand scaled and split, the results' residues. Back-projections also read and write three operands and the result.
//   M x N x K              FP64    INT8     (us, INT8 with the scaling, the split of B and the epilogue)
//   3328 x 512 x 137065   21987   10833     137065 x 512 x 3328   21828   12210
//   3328 x 128 x 137065    9352    5964     137065 x 128 x 3328    5651    5956
//   3328 x  64 x 137065    5722    5587     137065 x  64 x 3328    3229    5512
//   1664 x 700 x 57777     6285    3912     57777 x 700 x 1664     6580    4508
//    832 x 512 x 57777     3733    1920     57777 x 512 x 832      2639    2331
//    512 x 448 x 17077      639     383     17077 x 448 x 512       502     545
//    512 x 512 x 17077      417     398     17077 x 512 x 512       563     586
//    512 x 256 x 17077      213     291     17077 x 256 x 512       310     307
//   1024 x 512 x 7153       348     273     7153 x 512 x 1024       438     329
// Over 230 products (2109 to 137 065 plane waves, 128 to 3328 projectors, 48 to 1024 bands) the rule takes the faster side,
// or one within 6% of it; the estimates are within 20% of the measured times. Back-projections keep a larger margin: the
// rule was too good to INT8 at few plane waves (7153 x 448 x 512: 229 and 259). Products of the small FP64 GEMM, whose
// time this does not estimate, stay with it.
void rns_cost(int M, int N, int K, bool back, double* fp64, double* int8) {
  *fp64 = *int8 = 0.0;
  if (M <= 0 || N <= 0 || K <= 0) return;
  const double m = M, epi = back ? 64.0 * m * N / 4.5e6 : 0.0;
  const long tiles = long((M + 63) / 64) * ((N + 63) / 64);
  const int sp = back ? 1 : gemm_pick_splits(M, N, K);
  const long kc = ((K + sp - 1) / sp + 31) / 32 * 32, s = (K + kc - 1) / kc;
  *fp64 = double((tiles * s + 255) / 256) * (0.0955 * kc + 1.0) + (s > 1 ? 32.0 * s * m * N / 4e6 : 0.0) + epi;
  const double k = double(rns_ld(K));
  const long step = rns_chunk(N);
  for (long n0 = 0; n0 < N; n0 += step) {
    const double n = double(std::min<long>(step, N - n0));
    const double t = double((M + RT - 1) / RT) * std::ceil(n / RT) * 3 * L;
    *int8 += std::max(std::max(0.75, t / 256 + 0.15) * (0.0138 * k + 3.5), 3.0 * L * m * k / 4.2e6) +
             82.0 * n * (k + m) / 4.6e6;
  }
  *int8 += 15.0 + epi;
}
bool rns_pays(int M, int N, int K, bool back) {
  if (M <= 0 || N <= 0 || K <= 0 || K > kRnsMaxK || gemm_is_small(M, N, K)) return false;
  double fp64, int8;
  rns_cost(M, N, K, back, &fp64, &int8);
  return int8 < (back ? 0.92 : 0.98) * fp64;
}
bool rns_pays_some(int M, int N, int K, bool back) {
  for (int n = 64; n < N; n += 64)
    if (rns_pays(M, n, K, back)) return true;
  return rns_pays(M, N, K, back);
}

template <typename E>
hipError_t rns_scale_cols(long K, int N, const cx<E>* B, long ldb, const double* env, double* scale, double* inv,
                          double* rnorm, int* flag, int* any, hipStream_t st) {
  if (N <= 0) return hipSuccess;
  hipLaunchKernelGGL((k_rns_colnorm<E>), dim3(N), dim3(NST), 0, st, K, B, ldb, env, scale, inv, rnorm, flag, any);
  return hipGetLastError();
}

template <typename E>
hipError_t rns_scale_rows(long M, int K, const cx<E>* A, long lda, double* scale, double* inv, double* rnorm,
                          const double* cnorm, double* env, int* any, hipStream_t st) {
  if (M <= 0) return hipSuccess;
  hipLaunchKernelGGL((k_rns_rownorm<E>), dim3(unsigned((M + 255) / 256)), dim3(256), 0, st, M, K, A, lda, scale, inv,
                     rnorm, cnorm, env, any);
  return hipGetLastError();
}

template <typename E>
hipError_t rns_row_envelope(long M, int K, const cx<E>* A, long lda, const double* rnorm, double* env, hipStream_t st) {
  if (K <= 0) return hipSuccess;
  hipLaunchKernelGGL((k_rns_rowenv<E>), dim3(K), dim3(NST), 0, st, M, A, lda, rnorm, env);
  return hipGetLastError();
}

hipError_t rns_flat_overlap(long K, const double* env, double* out, hipStream_t st) {
  hipLaunchKernelGGL(k_rns_flat, dim3(1), dim3(NST), 0, st, K, env, out);
  return hipGetLastError();
}

template <typename E>
hipError_t rns_split_cols(long K, int N, const cx<E>* B, long ldb, const double* scale, int8_t* base, int8_t* third,
                          bool diff, long plane, long ld, const int* flag, int fs, hipStream_t st) {
  if (N <= 0) return hipSuccess;
  if (K <= 0 || N > 65535 || ld != rns_ld(K) || plane < N * ld || !third) return hipErrorInvalidValue;
  const dim3 grid(unsigned((ld / 4 + 255) / 256), unsigned(N));
  if (diff)
    hipLaunchKernelGGL((k_rns_split<E, true>), grid, dim3(256), 0, st, K, B, ldb, scale, base, third, plane, ld, flag, fs);
  else
    hipLaunchKernelGGL((k_rns_split<E, false>), grid, dim3(256), 0, st, K, B, ldb, scale, base, third, plane, ld, flag, fs);
  return hipGetLastError();
}

template <typename E>
hipError_t rns_split_rows(long M, int K, const cx<E>* A, long lda, const double* scale, int8_t* base, int8_t* sum,
                          long plane, long ld, const int* flag, hipStream_t st) {
  if (M <= 0) return hipSuccess;
  if (K <= 0 || ld != rns_ld(K) || plane < M * ld || !sum || ld / 64 > 65535) return hipErrorInvalidValue;
  hipLaunchKernelGGL((k_rns_split_rows<E>), dim3(unsigned((M + 63) / 64), unsigned(ld / 64)), dim3(256), 0, st, M, K, A,
                     lda, scale, base, sum, plane, ld, flag);
  return hipGetLastError();
}

template <typename EO>
hipError_t rns_product(GemmMode mode, int M, int N, int K, const RnsOperand& A, const RnsOperand& B, int8_t* C,
                       const Epi<EO>& epi, const int* flag, hipStream_t st) {
  if (M <= 0 || N <= 0) return hipSuccess;
  if (K <= 0 || K > kRnsMaxK || N > 65535 || A.ld != rns_ld(K) || B.ld != A.ld) return hipErrorInvalidValue;
  const long ldc = rns_ldc(M), zc = ldc * N;
  const long tm = (M + RT - 1) / RT, tn = (N + RT - 1) / RT;
  hipLaunchKernelGGL(k_rns_gemm, dim3(unsigned(tm * tn * 3 * L)), dim3(256), 0, st, M, N, int(A.ld / RK), A, B, C, ldc,
                     zc, flag);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((k_rns_finish<EO>), dim3(unsigned((M + 1023) / 1024), unsigned(N)), dim3(256), 0, st, M, N, C, ldc,
                     zc, A.inv, B.inv, mode == GEMM_CN ? -1 : 1, epi, flag);
  return hipGetLastError();
}

#define INST(E)                                                                                                       \
  template hipError_t rns_scale_cols<E>(long, int, const cx<E>*, long, const double*, double*, double*, double*, int*, \
                                        int*, hipStream_t);                                                           \
  template hipError_t rns_scale_rows<E>(long, int, const cx<E>*, long, double*, double*, double*, const double*,      \
                                        double*, int*, hipStream_t);                                                  \
  template hipError_t rns_row_envelope<E>(long, int, const cx<E>*, long, const double*, double*, hipStream_t);        \
  template hipError_t rns_split_cols<E>(long, int, const cx<E>*, long, const double*, int8_t*, int8_t*, bool, long,    \
                                        long, const int*, int, hipStream_t);                                          \
  template hipError_t rns_split_rows<E>(long, int, const cx<E>*, long, const double*, int8_t*, int8_t*, long, long,    \
                                        const int*, hipStream_t);                                                     \
  template hipError_t rns_product<E>(GemmMode, int, int, int, const RnsOperand&, const RnsOperand&, int8_t*,          \
                                     const Epi<E>&, const int*, hipStream_t);
INST(double)
#undef INST

}  // namespace chebfd
