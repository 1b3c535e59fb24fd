// Complex GEMM on CDNA4 matrix cores: three (FP64) or four (FP32) real 16x16x4 MFMAs per complex product block,
// and a hi/lo split FP16 form for the projector products of the mixed-precision filter.
//
// Used for every O(Npw x Nprojs) contraction of the filter (projections P^H psi and back-projection
// P w, Alg. 1; the reuse trick of Sec. 5.1 leaves one of each per filter step), for the Rayleigh-Ritz
// subspace matrices Y^H H Y, Y^H S Y and the rotation Y Z (Alg. 2), and for the small projector-space
// products with P^H P and the capacitance inverse (Sec. 5.1).
#include <algorithm>
#include <type_traits>

#include "gemm_common.h"
#include "kernels.h"

namespace chebfd {
namespace {

template <typename T> struct Mfma;
template <> struct Mfma<double> {
  typedef double acc __attribute__((ext_vector_type(4)));
  __device__ __forceinline__ static acc run(double a, double b, acc c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
  }
};
template <> struct Mfma<float> {
  typedef float acc __attribute__((ext_vector_type(4)));
  __device__ __forceinline__ static acc run(float a, float b, acc c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
  }
};

// split-K chunks are multiples of BK = 32; LDS rows padded by one element (a padding of 16 puts the transposed tile
// stores on one bank)
constexpr int BM = 64, BN = 64, BK = 32, PAD = 1, NT = 256;

inline int tile_group(int M, int K) { return K >= M ? kTileGroup : 1; }

// Epilogue operands moved into the leading slots (L, then U, then W) and counted: 0, 1 or 3 slots in use, a
// second operand without a third repeated in the third slot with weight 0 (it is a finite input). The tiled
// kernels take the count as a template parameter and read every used slot without a branch.
template <typename E> int epi_slots(Epi<E>& e) {
  const cx<E>* p[3] = {e.L, e.U, e.W};
  long l[3] = {e.ldl, e.ldu, e.ldw};
  double b[3] = {e.bL, e.bU, e.bW};
  int c = 0;
  for (int s = 0; s < 3; ++s)
    if (p[s]) { p[c] = p[s]; l[c] = l[s]; b[c] = b[s]; ++c; }
  for (int s = c; s < 3; ++s) { p[s] = nullptr; l[s] = 0; b[s] = 0.0; }
  if (c == 2) { p[2] = p[1]; l[2] = l[1]; b[2] = 0.0; c = 3; }
  e.L = p[0]; e.ldl = l[0]; e.bL = b[0];
  e.U = p[1]; e.ldu = l[1]; e.bU = b[1];
  e.W = p[2]; e.ldw = l[2]; e.bW = b[2];
  return c;
}

// Epilogue of one wave's NI x NJ MFMA blocks of 16 x 16 (T accumulators, the combined real and imaginary parts in
// cr, ci; rows of accumulator v given by row_of(v); column block j scaled by scale[j]). The NE operands of block
// b + 1 are requested, at clamped in-range indices, before the stores of block b, so that every thread keeps a
// block of loads in flight instead of waiting on each element in turn. PRED: only columns n with pred[n] set are stored.
template <int NE, bool PRED = false, int NI, int NJ, typename E, typename Acc, typename RowOf>
__device__ __forceinline__ void epi_blocks(const Epi<E>& epi, int M, int N, long mb, long nb, int li,
                                           const Acc (&cr)[NI][NJ], const Acc (&ci)[NI][NJ],
                                           const double (&scale)[NJ], RowOf row_of, const int* pred = nullptr) {
  constexpr int NS = NE > 0 ? NE : 1, NBLK = NI * NJ;
  const cx<E>* src[3] = {epi.L, epi.U, epi.W};
  const long lds[3] = {epi.ldl, epi.ldu, epi.ldw};
  const double bet[3] = {epi.bL, epi.bU, epi.bW};
  cx<E> buf[2][NS][4];
  auto eload = [&](int b, cx<E>(&dst)[NS][4]) {
    const int i = b / NJ, j = b % NJ;
    const long n = min(nb + 16 * j + li, long(N) - 1);
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const long m = min(mb + 16 * i + row_of(v), long(M) - 1);
#pragma unroll
      for (int s = 0; s < NS; ++s)
        if constexpr (NE > 0) dst[s][v] = src[s][m + n * lds[s]];
    }
  };
  if constexpr (NE > 0) eload(0, buf[0]);
#pragma unroll
  for (int b = 0; b < NBLK; ++b) {
    if constexpr (NE > 0)
      if (b + 1 < NBLK) eload(b + 1, buf[(b + 1) & 1]);
    const int i = b / NJ, j = b % NJ;
    const long n = nb + 16 * j + li;
    bool keep = n < N;
    if constexpr (PRED) keep = keep && pred[n];
    const double f = epi.alpha * scale[j];
    // values of all four elements first, then the guarded stores: a value computed only under the guard would
    // let the compiler move its loads there and wait on them
    cx<E> val[4];
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      double xr = f * double(cr[i][j][v]), xi = f * double(ci[i][j][v]);
#pragma unroll
      for (int s = 0; s < NS; ++s)
        if constexpr (NE > 0) {
          xr += bet[s] * double(buf[b & 1][s][v].x);
          xi += bet[s] * double(buf[b & 1][s][v].y);
        }
      val[v] = cx<E>{E(xr), epi.real_only ? E(0) : E(xi)};
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const long m = mb + 16 * i + row_of(v);
      if (m < M && keep) epi.out[m + n * epi.ldo] = val[v];
    }
  }
}

// One 64 x 64 complex output tile per block of 4 waves; wave w owns the 32 x 32 quadrant
// (w & 1, w >> 1) as 2 x 2 MFMA blocks. FP64 tiles take three real products per complex product
// (P1 = a_r b_r, P2 = a_i b_i, P3 = (a_r + s a_i)(b_r + b_i) with s = 1 for a b and s = -1 for conj(a) b:
// re = P1 - s P2, im = P3 - P1 - s P2), the sums formed in registers from the real and imaginary parts
// (storing them as two more LDS planes measured 9% slower), or two where FORM says so (FORM_RE: only the real part is
// wanted, P1 and P2; FORM_B_REAL: b is real, a_r b_r and a_i b_r); FP32 tiles keep the four-product form, whose
// rounding does not grow with the magnitude of the other component.
//
// The LDS holds two stages of GK = 16 k (separate arrays, so that the compiler need not order the reads of one behind
// the writes of the other; two blocks per CU). While tile t is multiplied, tile t + 1 goes from registers to the other
// stage and tile t + 2 is requested from memory, each access behind an MFMA (sched_group_barrier), and the fragments of
// the next 4 k are read one step ahead, across the one barrier of the tile: small products, with one or two waves per
// SIMD, have nobody else to hide these latencies behind. Against one stage of 32 k filled between two barriers:
// 256 x 256 x 7153 (16 splits) 66 -> 49 us, 7153 x 256 x 256 with three epilogue operands 80 -> 77 us (its operands'
// traffic, 146 MB, is not overlapped: all its blocks are resident at once); the two-product forms at 64^3, Gamma point:
// 512 x 301 x 8539 262 -> 176 us, 8539 x 301 x 512 210 -> 145 us.
// ROLE only separates kernel names per use (projection, back-projection, small, subspace) for profiling.
constexpr int GK = 16;
static_assert(BK % GK == 0, "splits are whole tiles");
template <typename T, typename EA, typename EB, typename EO, int MODE, int ROLE, int NE, int FORM, bool PRED>
__global__ __launch_bounds__(NT, 2) void k_gemm(int M, int N, int K, int kchunk, const cx<EA>* __restrict__ A,
                                             long lda, const cx<EB>* __restrict__ B, long ldb, Epi<EO> epi,
                                             c128* __restrict__ part, int grp,
                                             const int* __restrict__ pred) {
  constexpr bool G3 = sizeof(T) == 8;
  static_assert(G3 || FORM == FORM_FULL, "the two-product forms are FP64");
  constexpr int SZ = GK * (BM + PAD);
  static_assert(BM == BN, "one stage layout");
  __shared__ cx<T> A0[SZ], B0[SZ], A1[SZ], B1[SZ];
  using acc_t = typename Mfma<T>::acc;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int li = lane & 15, lk = lane >> 4;
  const int wm = (wave & 1) * 32, wn = (wave >> 1) * 32;
  int bx, by, bz;
  gemm_tile_of(blockIdx.x, gridDim.x, (M + BM - 1) / BM, (N + BN - 1) / BN, grp, bx, by, bz);
  const long m0 = long(bx) * BM, n0 = long(by) * BN;
  static_assert(BN == 64, "a lane per column");
  if (PRED && !__any(n0 + lane < N && pred[min(n0 + lane, long(N) - 1)])) return;
  const int kbeg = bz * kchunk;
  const int kend = min(K, kbeg + kchunk);
  const int nt = (kend - kbeg + GK - 1) / GK;

  acc_t cr[2][2], ci[2][2], c3[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int v = 0; v < 4; ++v) { cr[i][j][v] = T(0); ci[i][j][v] = T(0); c3[i][j][v] = T(0); }

  // global -> registers for one K tile (raw storage type), registers -> LDS converted to the MFMA type. Rows past M
  // and columns past N are read clamped (they feed only outputs that are not stored), k past the end clamped and
  // zeroed by value: a load under a condition would be waited for before the MFMAs.
  constexpr int RL = (BM * GK) / NT;
  cx<EA> va[RL];
  cx<EB> vb[RL];
  // A: k fastest for a conjugate transpose (as stored), row fastest else; B: k fastest
  const int ak = MODE == GEMM_CN ? tid % GK : tid / BM, am = MODE == GEMM_CN ? tid / GK : tid % BM;
  constexpr int AKS = MODE == GEMM_CN ? 0 : NT / BM, AMS = MODE == GEMM_CN ? NT / GK : 0;
  const int bk = tid % GK, bn = tid / GK;
  const cx<EA>* arow[RL];
  const cx<EB>* bcol[RL];
#pragma unroll
  for (int r = 0; r < RL; ++r) {
    const long gm = min(m0 + am + r * AMS, long(M) - 1);
    arow[r] = MODE == GEMM_CN ? A + gm * lda : A + gm;
    bcol[r] = B + min(n0 + bn + r * (NT / GK), long(N) - 1) * ldb;
  }
  auto load_r = [&](int r, int k0) {
    const int ka = min(k0 + ak + r * AKS, kend - 1), kb = min(k0 + bk, kend - 1);
    va[r] = MODE == GEMM_CN ? arow[r][ka] : arow[r][long(ka) * lda];
    vb[r] = bcol[r][kb];
  };
  auto put_r = [&](int r, int k0, cx<T>* As, cx<T>* Bs) {
    const bool oa = k0 + ak + r * AKS < kend, ob = k0 + bk < kend;
    As[(ak + r * AKS) * (BM + PAD) + am + r * AMS] = cx<T>{oa ? T(va[r].x) : T(0), oa ? T(va[r].y) : T(0)};
    Bs[bk * (BN + PAD) + bn + r * (NT / GK)] = cx<T>{ob ? T(vb[r].x) : T(0), ob ? T(vb[r].y) : T(0)};
  };
  auto frag = [&](const cx<T>* As, const cx<T>* Bs, int ks, cx<T>(&a)[2], cx<T>(&b)[2]) {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      a[i] = As[(4 * ks + lk) * (BM + PAD) + wm + 16 * i + li];
      b[i] = Bs[(4 * ks + lk) * (BN + PAD) + wn + 16 * i + li];
    }
  };
  auto mul = [&](const cx<T>(&a)[2], const cx<T>(&b)[2]) {
    if constexpr (G3) {
      // cr <- P1, ci <- P2, c3 <- P3
      T as[2], bs[2];
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        as[i] = MODE == GEMM_CN ? a[i].x - a[i].y : a[i].x + a[i].y;
        bs[i] = b[i].x + b[i].y;
      }
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          cr[i][j] = Mfma<T>::run(a[i].x, b[j].x, cr[i][j]);
          ci[i][j] = Mfma<T>::run(a[i].y, FORM == FORM_B_REAL ? b[j].x : b[j].y, ci[i][j]);
          if constexpr (FORM == FORM_FULL) c3[i][j] = Mfma<T>::run(as[i], bs[j], c3[i][j]);
        }
    } else {
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          if (MODE == GEMM_CN) {  // conj(a) b
            cr[i][j] = Mfma<T>::run(a[i].x, b[j].x, cr[i][j]);
            cr[i][j] = Mfma<T>::run(a[i].y, b[j].y, cr[i][j]);
            ci[i][j] = Mfma<T>::run(a[i].x, b[j].y, ci[i][j]);
            ci[i][j] = Mfma<T>::run(-a[i].y, b[j].x, ci[i][j]);
          } else {  // a b
            cr[i][j] = Mfma<T>::run(a[i].x, b[j].x, cr[i][j]);
            cr[i][j] = Mfma<T>::run(-a[i].y, b[j].y, cr[i][j]);
            ci[i][j] = Mfma<T>::run(a[i].x, b[j].y, ci[i][j]);
            ci[i][j] = Mfma<T>::run(a[i].y, b[j].x, ci[i][j]);
          }
        }
    }
  };

  if (nt > 0) {
    constexpr int KS = GK / 4;
    static_assert(KS == 4 && RL == 4, "interleaving below");
    auto at = [&](int t) { return kbeg + min(t, nt - 1) * GK; };
#pragma unroll
    for (int r = 0; r < RL; ++r) load_r(r, kbeg);
#pragma unroll
    for (int r = 0; r < RL; ++r) put_r(r, kbeg, A0, B0);
#pragma unroll
    for (int r = 0; r < RL; ++r) load_r(r, at(1));
    __syncthreads();
    cx<T> fa[2][2], fb[2][2];
    frag(A0, B0, 0, fa[0], fb[0]);
    // tile t from stage (As, Bs); the last tiles request (and store) the last tile again, which nothing reads
    auto step = [&](int t, cx<T>* As, cx<T>* Bs, cx<T>* An, cx<T>* Bn) {
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        if (ks + 1 < KS) {
          frag(As, Bs, ks + 1, fa[(ks + 1) & 1], fb[(ks + 1) & 1]);
#pragma unroll
          for (int r = ks; r < RL; r += KS - 1)
            if (r < RL) { put_r(r, at(t + 1), An, Bn); load_r(r, at(t + 2)); }
          mul(fa[ks & 1], fb[ks & 1]);
#pragma unroll
          for (int q = 0; q < 4; ++q) {  // MFMA, LDS read, MFMA, LDS write, MFMA, global load
            __builtin_amdgcn_sched_group_barrier(0x8, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
            if constexpr (FORM == FORM_FULL) __builtin_amdgcn_sched_group_barrier(0x8, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x200, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x8, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x20, 1, 0);
          }
        } else {
          __syncthreads();
          frag(An, Bn, 0, fa[(ks + 1) & 1], fb[(ks + 1) & 1]);
          mul(fa[ks & 1], fb[ks & 1]);
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            __builtin_amdgcn_sched_group_barrier(0x8, 2, 0);
            __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
          }
        }
      }
    };
    int it = 0;
    for (; it + 1 < nt; it += 2) { step(it, A0, B0, A1, B1); step(it + 1, A1, B1, A0, B0); }
    if (it < nt) step(it, A0, B0, A1, B1);
  }

  if constexpr (G3) {
    constexpr T sg = MODE == GEMM_CN ? T(-1) : T(1);
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const T p1 = cr[i][j][v], p2 = ci[i][j][v], p3 = c3[i][j][v];
          if constexpr (FORM == FORM_B_REAL) {
            ci[i][j][v] = sg * p2;  // a_i b_r, negated under conj(a)
          } else {
            cr[i][j][v] = p1 - sg * p2;
            ci[i][j][v] = FORM == FORM_FULL ? p3 - p1 - sg * p2 : T(0);
          }
        }
  }
  // accumulator v of a lane holds column li of each 16 x 16 block, row 4*lk + v for the f32 MFMA and
  // row lk + 4*v for the f64 MFMA (lane layouts of the two 16x16x4 instructions differ)
  auto row_of = [&](int v) { return sizeof(T) == 8 ? lk + 4 * v : 4 * lk + v; };
  if (part) {
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const long m = m0 + wm + 16 * i + row_of(v);
          const long n = n0 + wn + 16 * j + li;
          if (m < M && n < N) part[(long(bz) * N + n) * M + m] = c128{double(cr[i][j][v]), double(ci[i][j][v])};
        }
  } else {
    const double one[2] = {1.0, 1.0};
    epi_blocks<NE, PRED>(epi, M, N, m0 + wm, n0 + wn, li, cr, ci, one, row_of, pred);
  }
}

// upper: only the elements of tiles bx <= by (the others' partials were not written)
template <typename EO>
__global__ __launch_bounds__(256) void k_reduce(int M, int N, int splits, const c128* __restrict__ part, Epi<EO> epi,
                                                int upper = 0, const int* __restrict__ pred = nullptr) {
  const long total = long(M) * N;
  for (long t = blockIdx.x * long(blockDim.x) + threadIdx.x; t < total; t += long(gridDim.x) * blockDim.x) {
    const long n = t / M, m = t - n * M;
    if ((upper && m / BM > n / BN) || (pred && !pred[n])) continue;
    double re = 0.0, im = 0.0;
    // eight partials in flight at a time, added in order
    for (int s0 = 0; s0 < splits; s0 += 8) {
      c128 v[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) v[j] = part[long(min(s0 + j, splits - 1)) * total + t];
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        re = s0 + j < splits ? re + v[j].x : re;
        im = s0 + j < splits ? im + v[j].y : im;
      }
    }
    epi_store(epi, m, n, re, im);
  }
}

// ---- small complex FP64 GEMM ----------------------------------------------------------------------------
// Products with at most a few hundred 16 x 16 output blocks and K of at most a thousand (the projector-space
// matrices of Sec. 5.1 and the subspace matrices of the Rayleigh-Ritz step) fill only a few dozen 64 x 64 tiles:
// the tiled kernel above then runs one wave per SIMD and needs split-K with a second reduction launch. Here one
// block of SW waves computes one 16 x 16 output block. Wave w takes the w-th part of K and reads its operand
// fragments straight from global memory (a few MB that stay in L2), the next load group in flight during the
// MFMAs of the current one; the partial blocks meet in LDS and are summed in a fixed order, so that the result does not depend on timing.
//
// Within a load group of 16 k, lane (li, lk) holds k = k0 + 4 s + lk for MFMA step s (the instruction's own k
// order): the 4 lanes of one B column (and of one A column for conj(A)^T) read 64 contiguous bytes per load.
//
// Few blocks with a longer K (the projections and Grams of the small spheres) leave the chip idle while each block pulls
// its whole K through one CU: K is then split over blocks too, and the partial blocks summed by k_reduce, or by the kernel
// that reads the product next where it can (gemm_small_parts) (65 x 41 x 925,
// 15 blocks: 15.1 us in one launch, also with 16 waves per block; 8.4 us with 14 splits, the reduction included). Filters of
// 4 steps at 24^3, 4 to 130 projectors and 1 to 100 bands, take 145 to 206 us instead of 150 to 238; Rayleigh-Ritz of 1 to
// 100 bands there 231 to 272 instead of 276 to 319; with 832 projectors (their K in projector space) 1 to 8 bands gain 1%.
constexpr int SKG = 16, SKMAX = 1024, SBLKMAX = 1024, SLD = 17, SW = 4;  // 8 waves per block measured slower at 256^3
static_assert(SW >= 4, "the epilogue takes one thread per element of the 16 x 16 block");

template <typename EO, int MODE>
__global__ __launch_bounds__(64 * SW) void k_gemm_s(int M, int N, int K, int kchunk, const c128* __restrict__ A,
                                                long lda, const c128* __restrict__ B, long ldb, Epi<EO> epi,
                                                c128* __restrict__ part) {
  __shared__ c128 red[SW][16 * SLD];
  using acc_t = Mfma<double>::acc;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int li = lane & 15, lk = lane >> 4;
  int bx, by, bz;
  gemm_tile_of(blockIdx.x, gridDim.x, (M + 15) / 16, (N + 15) / 16, 1, bx, by, bz);
  const long m0 = long(bx) * 16, n0 = long(by) * 16;
  // rows of A past M and columns of B past N are read clamped: they feed only output rows and columns that are
  // never stored
  const long amc = min(m0 + li, long(M) - 1), bnc = min(n0 + li, long(N) - 1);
  const c128* __restrict__ Ab = MODE == GEMM_CN ? A + amc * lda : A + amc;
  const long ask = MODE == GEMM_CN ? 1 : lda;  // A stride along k
  const c128* __restrict__ Bb = B + bnc * ldb;
  const int kb = (bz * SW + wave) * kchunk, ke = min(K, kb + kchunk);
  const int kfull = kb + (max(ke - kb, 0) / SKG) * SKG;  // end of the whole load groups

  acc_t p1, p2, p3;
#pragma unroll
  for (int v = 0; v < 4; ++v) { p1[v] = 0.0; p2[v] = 0.0; p3[v] = 0.0; }

  // whole groups load without conditions (a load under a branch would make the compiler wait for every load
  // in flight before the MFMAs); only the last partial group zeroes k >= ke by value
  c128 a0[4], b0[4], a1[4], b1[4];
  auto load = [&](int k0, c128(&a)[4], c128(&b)[4]) {
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const int k = k0 + 4 * s + lk;
      a[s] = Ab[long(k) * ask];
      b[s] = Bb[k];
    }
  };
  auto load_tail = [&](int k0, c128(&a)[4], c128(&b)[4]) {
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const int k = k0 + 4 * s + lk;
      const bool kok = k < ke;
      const int kc = kok ? k : ke - 1;
      const c128 va = Ab[long(kc) * ask], vb = Bb[kc];
      a[s] = kok ? va : c128{0.0, 0.0};
      b[s] = kok ? vb : c128{0.0, 0.0};
    }
  };
  // P1 = a_r b_r, P2 = a_i b_i, P3 = (a_r + s a_i)(b_r + b_i), s = -1 for conj(a) b
  auto mul = [&](const c128(&a)[4], const c128(&b)[4]) {
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const double as = MODE == GEMM_CN ? a[s].x - a[s].y : a[s].x + a[s].y;
      p1 = Mfma<double>::run(a[s].x, b[s].x, p1);
      p2 = Mfma<double>::run(a[s].y, b[s].y, p2);
      p3 = Mfma<double>::run(as, b[s].x + b[s].y, p3);
    }
  };
  int k0 = kb;
  if (ke - kb == 4 * SKG) {
    // exactly four whole groups (K = 256 over 4 waves, the projector-space and subspace products): every load of
    // the wave issued before the first MFMA, one memory latency instead of four
    c128 a4[4][4], b4[4][4];
#pragma unroll
    for (int g = 0; g < 4; ++g) load(kb + g * SKG, a4[g], b4[g]);
#pragma unroll
    for (int g = 0; g < 4; ++g) mul(a4[g], b4[g]);
    k0 = ke;
  }
  // otherwise the next group is always requested (clamped to the last whole group, which the final pass reads
  // twice) and rotated into place after the MFMAs of this one: a request under a condition, or one consumed only
  // past a branch, is waited for or moved by the compiler before the MFMAs
  if (k0 < kfull) load(k0, a0, b0);
  for (; k0 < kfull; k0 += SKG) {
    load(min(k0 + SKG, kfull - SKG), a1, b1);
    mul(a0, b0);
#pragma unroll
    for (int s = 0; s < 4; ++s) { a0[s] = a1[s]; b0[s] = b1[s]; }
  }
  if (k0 < ke) {
    load_tail(k0, a0, b0);
    mul(a0, b0);
  }

  // accumulator v of a lane holds row lk + 4 v, column li of the 16 x 16 block
  constexpr double sg = MODE == GEMM_CN ? -1.0 : 1.0;
#pragma unroll
  for (int v = 0; v < 4; ++v)
    red[wave][(lk + 4 * v) + SLD * li] = c128{p1[v] - sg * p2[v], p3[v] - p1[v] - sg * p2[v]};
  __syncthreads();
  if (tid < 256) {
    const int r = tid & 15, c = tid >> 4;
    double re = 0.0, im = 0.0;
#pragma unroll
    for (int w = 0; w < SW; ++w) {
      const c128 x = red[w][r + SLD * c];
      re += x.x;
      im += x.y;
    }
    const long m = m0 + r, n = n0 + c;
    if (m < M && n < N) {
      if (part) part[(long(bz) * N + n) * M + m] = c128{re, im};
      else epi_store(epi, m, n, re, im);
    }
  }
}

// ---- FP16 hi/lo split GEMM ------------------------------------------------------------------------------
typedef _Float16 h8 __attribute__((ext_vector_type(8)));
typedef float f4 __attribute__((ext_vector_type(4)));

constexpr int HBK = 32, HLD = HBK + 8;  // LDS rows of 40 halves (80 bytes): 16-byte aligned, rows spread over banks

__device__ __forceinline__ f4 mfma_h(h8 a, h8 b, f4 c) { return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0); }
// acc += x * y with x = xh + xl, y = yh + yl, dropping xl * yl
__device__ __forceinline__ f4 mul3(h8 xh, h8 xl, h8 yh, h8 yl, f4 acc) {
  acc = mfma_h(xh, yh, acc);
  acc = mfma_h(xh, yl, acc);
  return mfma_h(xl, yh, acc);
}

// FP16 tiles: TB x TB complex outputs per block (TB = 64: 4 waves, TB = 128: 8 waves), each wave a (16 NI) x 32
// sub-tile of NI x 2 MFMA blocks; the waves form a 2 x (TB / 32) grid. Every thread loads one row (A) and one column
// (B) group of 8 k per K tile of 32, so a block has 4 TB threads. The 128 tiles read each LDS fragment for twice the
// MFMA work of the 64 tiles (a 64 x 32 wave sub-tile against 32 x 32), halving the LDS traffic per product, which
// bounds the 64 tiles on the large projector products.
template <int TB> struct HTile {
  static constexpr int NI = TB / 32, NJ = 2, WM = 2, WN = TB / 32, NT = 64 * WM * WN;
  static_assert(NT == 4 * TB, "one loader row per 4 threads");
};

// The 16x16x32 FP16 MFMA takes, in lane l, row l % 16 of A and column l % 16 of B at k = 8 (l / 16) ...
// 8 (l / 16) + 7, and returns row 4 (l / 16) + v, column l % 16 in accumulator element v.
// BPRE: B arrives as pre-split planes Bp [4][brows][bld] (see scale_split_columns) and is copied to LDS as it is.
template <int TB, typename EB, typename EO, int MODE, int ROLE, int NE, bool BPRE>
__global__ __launch_bounds__(HTile<TB>::NT) void k_gemm_h(int M, int N, int K, int kchunk,
                                                           const _Float16* __restrict__ Ap, long arows, long ald,
                                                           double ainv, const cx<EB>* __restrict__ B, long ldb,
                                                           const _Float16* __restrict__ Bp, long brows, long bld,
                                                           const float* __restrict__ bsc, Epi<EO> epi,
                                                           c128* __restrict__ part, int grp) {
  using HT = HTile<TB>;
  constexpr int NI = HT::NI, NJ = HT::NJ;
  // The 128 tiles (one block per CU) take two LDS stages: tile t is multiplied from one while tile t + 1 is
  // converted and written to the other, so the MFMAs just issued run on while the wave waits for the next tile's
  // loads, and one barrier per tile suffices. The 64 tiles keep one stage and more resident blocks.
  constexpr int NS = TB == 128 ? 2 : 1;
  __shared__ __align__(16) _Float16 As[NS][4][TB][HLD];
  __shared__ __align__(16) _Float16 Bs[NS][4][TB][HLD];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int li = lane & 15, lk = lane >> 4;
  const int wm = (wave % HT::WM) * 16 * NI, wn = (wave / HT::WM) * 16 * NJ;
  int bx, by, bz;
  gemm_tile_of(blockIdx.x, gridDim.x, (M + TB - 1) / TB, (N + TB - 1) / TB, grp, bx, by, bz);
  const long m0 = long(bx) * TB, n0 = long(by) * TB;
  const int kbeg = bz * kchunk;
  const int kend = min(K, kbeg + kchunk);

  f4 cr[NI][NJ], ci[NI][NJ];
#pragma unroll
  for (int i = 0; i < NI; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j) { cr[i][j] = f4{0.f, 0.f, 0.f, 0.f}; ci[i][j] = f4{0.f, 0.f, 0.f, 0.f}; }

  // loader roles: TB rows (A) / columns (B) x 4 groups of 8 k per tile, one group per thread
  const int lrow = tid >> 2, lgrp = tid & 3;
  const long gm = m0 + lrow, gn = n0 + lrow;
  const float sc = gn < N ? bsc[gn] : 1.f;
  // raw registers of one K tile (A planes as stored, B in its storage type), converted and split only when
  // written to LDS, so that the loads of the next tile stay in flight during the MFMAs of this one
  h8 ra[4], rb[4];
  cx<EB> vb[8];
  auto load_tile = [&](int k0) {
    const int kk = k0 + 8 * lgrp;
#pragma unroll
    for (int pl = 0; pl < 4; ++pl) {
      h8 v = {};
      if (gm < M) v = *reinterpret_cast<const h8*>(Ap + (pl * arows + gm) * ald + kk);  // K padded to 32: in bounds
      ra[pl] = v;
    }
    if constexpr (BPRE) {
#pragma unroll
      for (int pl = 0; pl < 4; ++pl) {
        h8 v = {};
        if (gn < N) v = *reinterpret_cast<const h8*>(Bp + (pl * brows + gn) * bld + kk);  // padded with zeros
        rb[pl] = v;
      }
    } else {
      const cx<EB>* col = B + (gn < N ? gn : 0) * ldb;
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        cx<EB> v = {EB(0), EB(0)};
        if (gn < N && kk + j < kend) v = col[kk + j];
        vb[j] = v;
      }
    }
  };
  auto store_tile = [&](int sg) {
#pragma unroll
    for (int pl = 0; pl < 4; ++pl) *reinterpret_cast<h8*>(&As[sg][pl][lrow][8 * lgrp]) = ra[pl];
    if constexpr (BPRE) {
#pragma unroll
      for (int pl = 0; pl < 4; ++pl) *reinterpret_cast<h8*>(&Bs[sg][pl][lrow][8 * lgrp]) = rb[pl];
      return;
    }
    h8 rh, rl, ih, il;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const float xr = float(vb[j].x * EB(sc)), xi = float(vb[j].y * EB(sc));
      const _Float16 hr = _Float16(xr), hi = _Float16(xi);
      rh[j] = hr;
      ih[j] = hi;
      rl[j] = _Float16(xr - float(hr));
      il[j] = _Float16(xi - float(hi));
    }
    *reinterpret_cast<h8*>(&Bs[sg][0][lrow][8 * lgrp]) = rh;
    *reinterpret_cast<h8*>(&Bs[sg][1][lrow][8 * lgrp]) = rl;
    *reinterpret_cast<h8*>(&Bs[sg][2][lrow][8 * lgrp]) = ih;
    *reinterpret_cast<h8*>(&Bs[sg][3][lrow][8 * lgrp]) = il;
  };

  if (kbeg < kend) {
    load_tile(kbeg);
    store_tile(0);
  }
  __syncthreads();
  int sg = 0;
  for (int k0 = kbeg; k0 < kend; k0 += HBK) {
    const bool more = k0 + HBK < kend;
    if (more) load_tile(k0 + HBK);  // in flight while this tile is multiplied
    h8 b[NJ][4];
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
      for (int pl = 0; pl < 4; ++pl) b[j][pl] = *reinterpret_cast<const h8*>(&Bs[NS == 2 ? sg : 0][pl][wn + 16 * j + li][8 * lk]);
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      h8 a[4];
#pragma unroll
      for (int pl = 0; pl < 4; ++pl) a[pl] = *reinterpret_cast<const h8*>(&As[NS == 2 ? sg : 0][pl][wm + 16 * i + li][8 * lk]);
      const h8 nih = -a[2], nil = -a[3];
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        cr[i][j] = mul3(a[0], a[1], b[j][0], b[j][1], cr[i][j]);
        ci[i][j] = mul3(a[0], a[1], b[j][2], b[j][3], ci[i][j]);
        if (MODE == GEMM_CN) {  // conj(a) b: re += ar br + ai bi, im += ar bi - ai br
          cr[i][j] = mul3(a[2], a[3], b[j][2], b[j][3], cr[i][j]);
          ci[i][j] = mul3(nih, nil, b[j][0], b[j][1], ci[i][j]);
        } else {  // a b: re += ar br - ai bi, im += ar bi + ai br
          cr[i][j] = mul3(nih, nil, b[j][2], b[j][3], cr[i][j]);
          ci[i][j] = mul3(a[2], a[3], b[j][0], b[j][1], ci[i][j]);
        }
      }
    }
    if constexpr (NS == 2) {
      if (more) store_tile(sg ^ 1);  // that stage was last read before the previous barrier
      __syncthreads();
      sg ^= 1;
    } else {
      __syncthreads();
      if (more) {
        store_tile(0);
        __syncthreads();
      }
    }
  }

  // column scales of the lane's columns (undo the per-band power-of-two scaling of B and the A scale)
  double fs[NJ];
#pragma unroll
  for (int j = 0; j < NJ; ++j) {
    const long n = n0 + wn + 16 * j + li;
    fs[j] = n < N ? ainv / double(bsc[n]) : 0.0;
  }
  auto row_of = [&](int v) { return 4 * lk + v; };
  if (part) {
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        const long n = n0 + wn + 16 * j + li;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const long m = m0 + wm + 16 * i + row_of(v);
          if (m < M && n < N)
            part[(long(bz) * N + n) * M + m] = c128{fs[j] * double(cr[i][j][v]), fs[j] * double(ci[i][j][v])};
        }
      }
  } else {
    epi_blocks<NE>(epi, M, N, m0 + wm, n0 + wn, li, cr, ci, fs, row_of);
  }
}

// ---- the 128 tiles with both operands as planes -----------------------------------------------------------------
// Same products as k_gemm_h for TB = 128, pre-split B. One wave per SIMD holds a 64 x 64 complex tile (2 x 2 blocks of the
// 32x32x16 MFMA, 128 accumulators); the LDS holds two stages of 32 k (1024 plane rows of 64 bytes, 64 KB each). While
// tile t is multiplied, tile t + 1 goes from registers to the other stage and tile t + 2 is requested from memory, one
// 16-byte access behind each MFMA or two (sched_group_barrier), and the fragments of the next 16 k are read one step
// ahead, across the one barrier of the tile. The epilogue passes through LDS so that its operands are read and written
// with m across the lanes. Bound by power: the matrix cores are 63 to 67% busy at 1.57 to 1.65 GHz (8 waves of 64 x 32 tiles
// without the interleaving: 45 to 50% at 1.9 to 2.0 GHz), 1.06 PFLOP/s executed. 3328 x 1024 x 137065 12.0 -> 10.6 ms,
// 137065 x 1024 x 3328 with three epilogue operands 12.4 -> 10.6 ms.
constexpr int PT = 128, PKB = 2 * HBK;       // output tile; bytes of a stage row
constexpr int kPStage = 2 * 4 * PT * PKB;    // A planes, then B planes
// chunk c (16 bytes) of stage row r sits at chunk c ^ (r / 4 % 4): 16 consecutive rows read at one c touch all 64 banks
__device__ __forceinline__ int pstage_at(int r, int c) { return r * PKB + ((c ^ ((r >> 2) & 3)) << 4); }
typedef float f16v __attribute__((ext_vector_type(16)));
__device__ __forceinline__ f16v mul3(h8 xh, h8 xl, h8 yh, h8 yl, f16v acc) {
  acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(xh, yh, acc, 0, 0, 0);
  acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(xh, yl, acc, 0, 0, 0);
  return __builtin_amdgcn_mfma_f32_32x32x16_f16(xl, yh, acc, 0, 0, 0);
}

template <typename EO, int MODE, int ROLE, int NE>
__global__ __launch_bounds__(256, 1) void k_gemm_hp(int M, int N, int K, int kchunk, const _Float16* __restrict__ Ap,
                                                   long arows, long ald, double ainv, const _Float16* __restrict__ Bp,
                                                   long brows, long bld, const float* __restrict__ bsc, Epi<EO> epi,
                                                   c128* __restrict__ part, int grp) {
  __shared__ __align__(16) int8_t S0[kPStage], S1[kPStage];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  int bx, by, bz;
  gemm_tile_of(blockIdx.x, gridDim.x, (M + PT - 1) / PT, (N + PT - 1) / PT, grp, bx, by, bz);
  const int m0 = bx * PT, n0 = by * PT;
  const int kbeg = bz * kchunk;
  const int nt = (min(K, kbeg + kchunk) - kbeg + HBK - 1) / HBK;  // K is padded with zeros to whole tiles

  // loaders: chunk tid % 4 of rows tid / 4 + 64 (i % 2) of plane i / 2 of A, then of B, rows past M or N clamped (they
  // feed only outputs that are not stored)
  constexpr int NL = 16;
  const int8_t* base[8];
#pragma unroll
  for (int pl = 0; pl < 4; ++pl) {
    base[pl] = reinterpret_cast<const int8_t*>(Ap + (pl * arows + m0) * ald + kbeg);
    base[4 + pl] = reinterpret_cast<const int8_t*>(Bp + (pl * brows + n0) * bld + kbeg);
  }
  unsigned off[4];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int row = 64 * h + (tid >> 2);
    off[h] = unsigned(min(row, M - 1 - m0)) * unsigned(2 * ald) + (tid & 3) * 16;
    off[2 + h] = unsigned(min(row, N - 1 - n0)) * unsigned(2 * bld) + (tid & 3) * 16;
  }
  const int dst = pstage_at(tid >> 2, tid & 3);  // + 64 i rows: the swizzle repeats every 16 rows
  h8 g[NL];
  auto load_i = [&](int i, int t) {
    g[i] = *reinterpret_cast<const h8*>(base[i >> 1] + t * PKB + off[(i >> 3) * 2 + (i & 1)]);
  };
  auto put_i = [&](int i, int8_t* S) { *reinterpret_cast<h8*>(S + dst + i * 64 * PKB) = g[i]; };
  const int wm = (wave & 1) * 64, wn = (wave >> 1) * 64, fr = lane & 31, fh = lane >> 5;
  f16v cr[2][2], ci[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) { cr[i][j][v] = 0.f; ci[i][j][v] = 0.f; }
  // lane l of the MFMA holds row l % 32 at k = 8 (l / 32) ... + 7 of its 16
  auto frag = [&](const int8_t* S, int ks, h8(&fa)[2][4], h8(&fb)[2][4]) {
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int pl = 0; pl < 4; ++pl) {
        fa[i][pl] = *reinterpret_cast<const h8*>(S + pstage_at(pl * PT + wm + 32 * i + fr, 2 * ks + fh));
        fb[i][pl] = *reinterpret_cast<const h8*>(S + pstage_at((4 + pl) * PT + wn + 32 * i + fr, 2 * ks + fh));
      }
  };
  auto mul = [&](const h8(&fa)[2][4], const h8(&fb)[2][4]) {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const h8 nih = -fa[i][2], nil = -fa[i][3];
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        cr[i][j] = mul3(fa[i][0], fa[i][1], fb[j][0], fb[j][1], cr[i][j]);
        ci[i][j] = mul3(fa[i][0], fa[i][1], fb[j][2], fb[j][3], ci[i][j]);
        if (MODE == GEMM_CN) {  // conj(a) b: re += ar br + ai bi, im += ar bi - ai br
          cr[i][j] = mul3(fa[i][2], fa[i][3], fb[j][2], fb[j][3], cr[i][j]);
          ci[i][j] = mul3(nih, nil, fb[j][0], fb[j][1], ci[i][j]);
        } else {  // a b: re += ar br - ai bi, im += ar bi + ai br
          cr[i][j] = mul3(nih, nil, fb[j][2], fb[j][3], cr[i][j]);
          ci[i][j] = mul3(fa[i][2], fa[i][3], fb[j][0], fb[j][1], ci[i][j]);
        }
      }
    }
  };
  if (nt > 0) {
#pragma unroll
    for (int i = 0; i < NL; ++i) load_i(i, 0);
#pragma unroll
    for (int i = 0; i < NL; ++i) put_i(i, S0);
#pragma unroll
    for (int i = 0; i < NL; ++i) load_i(i, min(1, nt - 1));
    __syncthreads();
    h8 fa[2][2][4], fb[2][2][4];
    frag(S0, 0, fa[0], fb[0]);
    // tile t from stage Sa; the last tiles request (and store) the last tile again, which nothing reads
    auto step = [&](int t, int8_t* Sa, int8_t* Sb) {
      const int tn = min(t + 2, nt - 1);
      frag(Sa, 1, fa[1], fb[1]);
#pragma unroll
      for (int i = 0; i < NL; ++i) { put_i(i, Sb); load_i(i, tn); }
      mul(fa[0], fb[0]);
#pragma unroll
      for (int q = 0; q < 16; ++q) {
        __builtin_amdgcn_sched_group_barrier(0x8, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x8, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x200, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x8, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x20, 1, 0);
      }
      __syncthreads();
      frag(Sb, 0, fa[0], fb[0]);
      mul(fa[1], fb[1]);
#pragma unroll
      for (int q = 0; q < 16; ++q) {
        __builtin_amdgcn_sched_group_barrier(0x8, 3, 0);
        __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
      }
    };
    int it = 0;
    for (; it + 1 < nt; it += 2) { step(it, S0, S1); step(it + 1, S1, S0); }
    if (it < nt) step(it, S0, S1);
    __syncthreads();
  }

  // 32 columns at a time through the wave's own 32 KB: element (m, n) at float2 64 n + (m ^ (n % 16) * 2), so that the
  // 32 columns written at one m spread over the banks. Accumulator v of a lane: row 8 (v / 4) + 4 (lane / 32) + v % 4,
  // column lane % 32 of its 32 x 32 block.
  float2* W = reinterpret_cast<float2*>((wave & 2 ? S1 : S0) + (wave & 1) * (kPStage / 2));
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int m = 32 * i + 8 * (v >> 2) + 4 * fh + (v & 3), n = 32 * j + fr;
        W[64 * n + (m ^ ((n & 15) * 2))] = float2{cr[i][j][v], ci[i][j][v]};
      }
  __syncthreads();
  const long m = m0 + wm + lane;
  const long mc = min(m, long(M) - 1);
  const int nn = min(64, N - n0 - wn);
  constexpr int NS = NE > 0 ? NE : 1, NU = 4;
  const cx<EO>* src[3] = {epi.L, epi.U, epi.W};
  const long lds[3] = {epi.ldl, epi.ldu, epi.ldw};
  const double bet[3] = {epi.bL, epi.bU, epi.bW};
  for (int q = 0; q < nn; q += NU) {
    cx<EO> in[NU][NS];
#pragma unroll
    for (int u = 0; u < NU; ++u) {
      const long n = n0 + wn + min(q + u, nn - 1);
#pragma unroll
      for (int s = 0; s < NS; ++s)
        if constexpr (NE > 0) in[u][s] = src[s][mc + n * lds[s]];
    }
#pragma unroll
    for (int u = 0; u < NU; ++u) {
      const int c = min(q + u, nn - 1);
      const long n = n0 + wn + c;
      const float2 x = W[64 * c + (lane ^ ((c & 15) * 2))];
      const double f = ainv / double(bsc[n]);
      if (part) {
        if (m < M && q + u < nn) part[(long(bz) * N + n) * M + m] = c128{f * double(x.x), f * double(x.y)};
      } else {
        const double fa = epi.alpha * f;
        double xr = fa * double(x.x), xi = fa * double(x.y);
#pragma unroll
        for (int s = 0; s < NS; ++s)
          if constexpr (NE > 0) { xr += bet[s] * double(in[u][s].x); xi += bet[s] * double(in[u][s].y); }
        if (m < M && q + u < nn) epi.out[m + n * epi.ldo] = cx<EO>{EO(xr), epi.real_only ? EO(0) : EO(xi)};
      }
    }
  }
}

// largest |Re|, |Im| of a column in the block, and the column's power-of-two scale: mx = f 2^e, f in [0.5, 1), is taken
// to [2^13, 2^14)
constexpr int CST = 1024;
__device__ __forceinline__ double block_max(double mx, double* red) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) mx = fmax(mx, __shfl_xor(mx, o, 64));
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = mx;
  __syncthreads();
  mx = red[0];
  for (int w = 1; w < CST / 64; ++w) mx = fmax(mx, red[w]);
  return mx;
}
__device__ __forceinline__ float column_scale(double mx) {
  int e = 0;
  const bool ok = mx > 0.0 && mx < 1e300;
  if (ok) (void)frexp(mx, &e);
  return ok ? ldexpf(1.f, min(kHalfTopExp - e, 126)) : 1.f;
}

// one 1024-thread block per column (16 waves per CU keep enough loads in flight), max over lanes by shuffles
template <typename E>
__global__ __launch_bounds__(CST) void k_colscale(long rows, const cx<E>* __restrict__ B, long ldb, float* bsc,
                                                  double* maxout) {
  __shared__ double red[CST / 64];
  const cx<E>* col = B + long(blockIdx.x) * ldb;
  double mx = 0.0;
  for (long i = threadIdx.x; i < rows; i += blockDim.x) {
    const cx<E> v = col[i];
    mx = fmax(mx, fmax(fabs(double(v.x)), fabs(double(v.y))));
  }
  mx = block_max(mx, red);
  if (threadIdx.x == 0) {
    if (maxout) maxout[blockIdx.x] = mx;
    if (bsc) bsc[blockIdx.x] = column_scale(mx);
  }
}

// the hi and lo planes of one scaled element (the same operations as the on-the-fly split in k_gemm_h)
template <typename E>
__device__ __forceinline__ void split_store(cx<E> v, E sc, _Float16* P, long total, long t) {
  const float xr = float(v.x * sc), xi = float(v.y * sc);
  const _Float16 hr = _Float16(xr), hi = _Float16(xi);
  P[t] = hr;
  P[total + t] = _Float16(xr - float(hr));
  P[2 * total + t] = hi;
  P[3 * total + t] = _Float16(xi - float(hi));
}

// Scale and planes of a column of at most kScaleSplit elements in one go, the column in the block's registers: one read
// and one launch where k_colscale and k_split_columns take two (256 bands of 7153: 7.0 us instead of 4.8 + 7.2).
constexpr int kScaleSplit = 8 * CST;
template <typename E>
__global__ __launch_bounds__(CST) void k_scale_split(int K, const cx<E>* __restrict__ B, long ldb, float* bsc,
                                                     _Float16* __restrict__ P, long pld, long total) {
  __shared__ double red[CST / 64];
  constexpr int NE = kScaleSplit / CST;
  const long n = blockIdx.x;
  const cx<E>* col = B + n * ldb;
  cx<E> v[NE];
  double mx = 0.0;
#pragma unroll
  for (int j = 0; j < NE; ++j) {
    const int k = threadIdx.x + j * CST;
    const cx<E> x = col[min(k, K - 1)];
    v[j] = cx<E>{k < K ? x.x : E(0), k < K ? x.y : E(0)};
    mx = fmax(mx, fmax(fabs(double(v[j].x)), fabs(double(v[j].y))));
  }
  const float sc = column_scale(block_max(mx, red));
  if (threadIdx.x == 0) bsc[n] = sc;
#pragma unroll
  for (int j = 0; j < NE; ++j) {
    const int k = threadIdx.x + j * CST;
    if (k < pld) split_store<E>(v[j], E(sc), P, total, n * pld + k);
  }
}

__global__ void k_split_planes(const c128* __restrict__ X, long ldx, int ksrc, bool transpose, double scale,
                               _Float16* __restrict__ P, long prow, long pld) {
  const long total = prow * pld;
  for (long t = blockIdx.x * long(blockDim.x) + threadIdx.x; t < total; t += long(gridDim.x) * blockDim.x) {
    const long r = t / pld, k = t - r * pld;
    c128 v = {0.0, 0.0};
    if (k < ksrc) v = transpose ? X[r + k * ldx] : X[k + r * ldx];
    const double xr = v.x * scale, xi = v.y * scale;
    const _Float16 hr = _Float16(float(xr)), hi = _Float16(float(xi));
    P[t] = hr;
    P[total + t] = _Float16(float(xr - double(float(hr))));
    P[2 * total + t] = hi;
    P[3 * total + t] = _Float16(float(xi - double(float(hi))));
  }
}

template <typename E>
__global__ void k_split_columns(int K, int N, const cx<E>* __restrict__ B, long ldb, const float* __restrict__ bsc,
                                _Float16* __restrict__ P, long pld) {
  const long total = long(N) * pld;
  for (long t = blockIdx.x * long(blockDim.x) + threadIdx.x; t < total; t += long(gridDim.x) * blockDim.x) {
    const long n = t / pld, k = t - n * pld;
    cx<E> v = {E(0), E(0)};
    if (k < K) v = B[k + n * ldb];
    split_store<E>(v, E(bsc[n]), P, total, t);
  }
}

}  // namespace

// Split count that minimises the rounds of resident blocks per unit of K work, ceil(tiles s / slots) / s, over
// s in [1, smax] (the smallest such s): a launch of tiles slightly above a multiple of the resident blocks
// otherwise leaves most of the GPU idle in its last round.
long quantized_splits(long tiles, long slots, long smax, long smin = 1) {
  if (smin < 1) smin = 1;
  if (smax < smin) smax = smin;
  long best = smin;
  double cost = double((tiles * smin + slots - 1) / slots) / double(smin);
  for (long s = smin + 1; s <= smax; ++s) {
    const double c = double((tiles * s + slots - 1) / slots) / double(s);
    if (c < cost - 1e-12) { cost = c; best = s; }
  }
  return best;
}

int gemm_pick_splits(int M, int N, int K) {
  if (M <= 0 || N <= 0 || K <= 0) return 1;
  const long tiles = long((M + BM - 1) / BM) * ((N + BN - 1) / BN);
  const long kblocks = (K + BK - 1) / BK;
  long smax = std::min<long>(32, kblocks / 2);  // at least two K tiles per split
  if (smax < 1) smax = 1;
  long s;
  if (tiles < 256) {
    // about one block per CU: measured on the paw48 projector shapes, the tall NN products (448 tiles) run best
    // without split-K and the 256 x 256 x 7153 reductions with 16 splits (28 and 56 slower)
    s = std::min((256 + tiles - 1) / tiles, smax);
  } else {
    // two resident blocks per CU on 256 CUs (the 3328 x 2048 x 137065 projection: 1664 tiles, 4 splits)
    s = quantized_splits(tiles, 512, std::min<long>(smax, 8));
  }
  return int(std::max<long>(s, 1));
}

bool gemm_is_small(int M, int N, int K) { return K <= SKMAX && long((M + 15) / 16) * ((N + 15) / 16) <= SBLKMAX; }

// K of a wave with s splits, and K over blocks as well where few of them meet a longer K: up to a block per CU, at least
// 64 k each
static int gemm_small_chunk(int K, int s) {
  const int kc = (std::max(K, 0) + SW * s - 1) / (SW * s);
  return std::max(SKG, ((kc + SKG - 1) / SKG) * SKG);
}
int gemm_small_splits(int M, int N, int K, int splits) {
  const long blocks = long((M + 15) / 16) * ((N + 15) / 16);
  if (K < 512 || blocks > 64) return 1;
  const int s = int(std::min<long>({long(std::max(splits, 1)), 256 / blocks, long(K / 64)}));
  const int kc = gemm_small_chunk(K, s);
  return std::max(1, (K + SW * kc - 1) / (SW * kc));
}
template <typename EO>
static hipError_t gemm_small_launch(GemmMode mode, int M, int N, int K, const c128* A, long lda, const c128* B, long ldb,
                                    int s, const Epi<EO>& epi, c128* part, hipStream_t st) {
  const dim3 grid(unsigned(long((M + 15) / 16) * ((N + 15) / 16) * s));
  const int kc = gemm_small_chunk(K, s);
  if (mode == GEMM_CN)
    hipLaunchKernelGGL((k_gemm_s<EO, GEMM_CN>), grid, dim3(64 * SW), 0, st, M, N, K, kc, A, lda, B, ldb, epi, part);
  else
    hipLaunchKernelGGL((k_gemm_s<EO, GEMM_NN>), grid, dim3(64 * SW), 0, st, M, N, K, kc, A, lda, B, ldb, epi, part);
  return hipGetLastError();
}
hipError_t gemm_small_parts(GemmMode mode, int M, int N, int K, const c128* A, long lda, const c128* B, long ldb,
                            int count, c128* part, hipStream_t st) {
  if (M <= 0 || N <= 0) return hipSuccess;
  if (!part || !gemm_is_small(M, N, K)) return hipErrorInvalidValue;
  return gemm_small_launch<double>(mode, M, N, K, A, lda, B, ldb, count, Epi<double>{}, part, st);
}

template <typename T, typename EA, typename EB, typename EO>
hipError_t gemm(GemmMode mode, int M, int N, int K, const cx<EA>* A, long lda, const cx<EB>* B, long ldb,
                const Epi<EO>& epi, int splits, c128* part, hipStream_t st, GemmRole role, bool upper,
                const int* pred, GemmForm form) {
  if (M <= 0 || N <= 0) return hipSuccess;
  if (upper && M != N) return hipErrorInvalidValue;
  if (role == ROLE_PROJECT ? mode != GEMM_CN : role == ROLE_BACKPROJECT && mode != GEMM_NN) return hipErrorInvalidValue;
  constexpr bool kPred = std::is_same<T, double>::value && std::is_same<EA, double>::value && std::is_same<EB, double>::value;
  if (pred && !(kPred && form == FORM_FULL && (role == ROLE_PROJECT || role == ROLE_BACKPROJECT))) return hipErrorInvalidValue;
  if constexpr (std::is_same<T, double>::value && std::is_same<EA, double>::value && std::is_same<EB, double>::value) {
    if (gemm_is_small(M, N, K)) {
      if (pred) return hipErrorInvalidValue;  // too small for a product that has another route
      const int s = part ? gemm_small_splits(M, N, K, splits) : 1;
      const hipError_t e = gemm_small_launch(mode, M, N, K, A, lda, B, ldb, s, epi, s > 1 ? part : nullptr, st);
      if (e != hipSuccess || s == 1) return e;
      const long total = long(M) * N;
      hipLaunchKernelGGL((k_reduce<EO>), dim3(unsigned((total + 255) / 256)), dim3(256), 0, st, M, N, s, part, epi);
      return hipGetLastError();
    }
  }
  if (splits < 1) splits = 1;
  int kchunk = (K + splits - 1) / splits;
  kchunk = ((kchunk + BK - 1) / BK) * BK;
  if (kchunk < BK) kchunk = BK;
  splits = K > 0 ? (K + kchunk - 1) / kchunk : 1;
  const bool use_part = splits > 1;
  if (use_part && !part) return hipErrorInvalidValue;
  const long tm = (M + BM - 1) / BM;
  dim3 grid(unsigned((upper ? tm * (tm + 1) / 2 : tm * ((N + BN - 1) / BN)) * splits));
  const int grp = upper ? kUpperTiles : tile_group(M, K);
  c128* pp = use_part ? part : nullptr;
  Epi<EO> en = epi;
  const int ne = epi_slots(en);
  auto go = [&](auto modec, auto rolec, auto nec, auto formc, auto predc) {
    constexpr int MO = decltype(modec)::value, RO = decltype(rolec)::value, NEC = decltype(nec)::value,
                  FO = decltype(formc)::value;
    constexpr bool PR = decltype(predc)::value;
    hipLaunchKernelGGL((k_gemm<T, EA, EB, EO, MO, RO, NEC, FO, PR>), grid, dim3(NT), 0, st, M, N, K, kchunk, A, lda, B, ldb,
                       en, pp, grp, pred);
  };
  auto launch = [&](auto modec, auto rolec) {
    constexpr int MO = decltype(modec)::value, RO = decltype(rolec)::value;
    auto by_ne = [&](auto formc, auto predc) {
      if (ne == 0 || use_part) go(modec, rolec, std::integral_constant<int, 0>{}, formc, predc);
      else if (ne == 1) go(modec, rolec, std::integral_constant<int, 1>{}, formc, predc);
      else go(modec, rolec, std::integral_constant<int, 3>{}, formc, predc);
    };
    // the FP64 side of the INT8 products
    if constexpr (std::is_same<EA, double>::value && std::is_same<EB, double>::value &&
                  (RO == ROLE_PROJECT || RO == ROLE_BACKPROJECT)) {
      if (pred) return by_ne(std::integral_constant<int, FORM_FULL>{}, std::true_type{});
    }
    // real parts of projections and Grams, real right sides of back-projections
    if constexpr (sizeof(T) == 8 && MO == GEMM_CN && (RO == ROLE_PROJECT || RO == ROLE_SUBSPACE)) {
      if (form == FORM_RE) return by_ne(std::integral_constant<int, FORM_RE>{}, std::false_type{});
    } else if constexpr (sizeof(T) == 8 && RO == ROLE_BACKPROJECT) {
      if (form == FORM_B_REAL) return by_ne(std::integral_constant<int, FORM_B_REAL>{}, std::false_type{});
    }
    by_ne(std::integral_constant<int, FORM_FULL>{}, std::false_type{});
  };
  using CN = std::integral_constant<int, GEMM_CN>;
  using NNm = std::integral_constant<int, GEMM_NN>;
  switch (role) {
    case ROLE_PROJECT: launch(CN{}, std::integral_constant<int, ROLE_PROJECT>{}); break;
    case ROLE_BACKPROJECT: launch(NNm{}, std::integral_constant<int, ROLE_BACKPROJECT>{}); break;
    case ROLE_SUBSPACE: mode == GEMM_CN ? launch(CN{}, std::integral_constant<int, 3>{}) : launch(NNm{}, std::integral_constant<int, 3>{}); break;
    default: mode == GEMM_CN ? launch(CN{}, std::integral_constant<int, 0>{}) : launch(NNm{}, std::integral_constant<int, 0>{}); break;
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || !use_part) return e;
  const long total = long(M) * N;
  int blocks = int((total + 255) / 256);
  if (blocks > 4096) blocks = 4096;
  hipLaunchKernelGGL((k_reduce<EO>), dim3(blocks), dim3(256), 0, st, M, N, splits, part, epi, upper ? 1 : 0,
                     pred);
  return hipGetLastError();
}

// split count of an upper-triangle product (tm (tm + 1) / 2 tiles): the fewest rounds of 512 resident blocks per
// unit of K work, at most 8 splits and two K tiles per split
int gemm_upper_splits(int N, int K) {
  if (N <= 0 || K <= 0) return 1;
  const long tm = (N + BM - 1) / BM;
  const long kblocks = (K + BK - 1) / BK;
  const long smax = std::max<long>(1, std::min<long>(8, kblocks / 2));
  return int(quantized_splits(tm * (tm + 1) / 2, 512, smax));
}

__global__ void k_hermitian_lower(int n, c128* __restrict__ A, long lda) {
  const long total = long(n) * n;
  for (long t = blockIdx.x * long(blockDim.x) + threadIdx.x; t < total; t += long(gridDim.x) * blockDim.x) {
    const long j = t / n, i = t - j * n;
    if (i > j) {
      const c128 v = A[j + i * lda];
      A[i + j * lda] = c128{v.x, -v.y};
    }
  }
}

hipError_t hermitian_lower(int n, c128* A, long lda, hipStream_t st) {
  if (n <= 1) return hipSuccess;
  const long total = long(n) * n;
  const int blocks = int(std::min<long>((total + 255) / 256, 4096));
  hipLaunchKernelGGL(k_hermitian_lower, dim3(blocks), dim3(256), 0, st, n, A, lda);
  return hipGetLastError();
}

void gemm_block_item(int i, int total, int tm, int tn, int grp, int& bx, int& by, int& bz) {
  gemm_tile_of(i, total, tm, tn, grp, bx, by, bz);
}

// upper bound of the split counts any GEMM kernel here picks for an M x N x K product (partial-buffer sizing):
// 512 target blocks, two K tiles of 32 per split, at most 32 splits; gemm_pick_splits and gemm_h_pick_splits
// never exceed it
int gemm_split_bound(int M, int N, int K) {
  if (M <= 0 || N <= 0 || K <= 0) return 1;
  const long tiles = long((M + BM - 1) / BM) * ((N + BN - 1) / BN);
  long s = (512 + tiles - 1) / tiles;
  const long kblocks = (K + BK - 1) / BK;
  if (s > kblocks / 2) s = kblocks / 2;
  if (s > 32) s = 32;
  if (s < 1) s = 1;
  return int(std::max<long>(s, std::max(gemm_pick_splits(M, N, K), gemm_h_pick_splits(M, N, K))));
}

// Tile and split-K count of the FP16 split GEMM. The FP32 accumulators of one split sum K / splits products in
// sequence, and their rounding error grows like eps32 sqrt(K / splits): long reductions (the projections P^H x over
// all plane waves) are split into chunks of at most kHalfChunk, summed in FP64 by the reduction (at K = 57777 in one
// chunk the error set a residual floor of the mixed outer loop near 1e-5). The 128 tiles (one block of 8 waves per
// CU) are used when the launch fills at least one round of resident blocks, with the split count that wastes least
// of the last round; else the 64 tiles with about one block per CU (measured best on the paw48 shapes, where the
// 512-block target was 5% slower on the 256 x 256 x 7153 projection: twice the partial traffic).
// allow_split = false: one split (the caller bounds K).
constexpr long kHalfChunk = 4096;

void h_plan(int M, int N, int K, bool allow_split, int* tb, int* splits) {
  const long kblocks = (K + HBK - 1) / HBK;
  const long smin = allow_split ? (K + kHalfChunk - 1) / kHalfChunk : 1;
  long smax = allow_split ? std::max<long>(std::min<long>(64, kblocks / 2), smin) : 1;
  const long t128 = long((M + 127) / 128) * ((N + 127) / 128);
  // at least 16 K tiles per split of the 128 tiles, whose prologue and epilogue are long
  const long smax128 = std::max(std::min(smax, kblocks / 16), smin);
  const long s128 = quantized_splits(t128, 256, smax128, smin);
  if (t128 * s128 >= 256) {
    *tb = 128;
    *splits = int(s128);
    return;
  }
  const long tiles = long((M + 63) / 64) * ((N + 63) / 64);
  long s = (256 + tiles - 1) / tiles;
  s = std::max(std::min(s, smax), smin);
  *tb = 64;
  *splits = int(std::max<long>(s, 1));
}

int gemm_h_pick_splits(int M, int N, int K) {
  if (M <= 0 || N <= 0 || K <= 0) return 1;
  int tb = 64, s = 1;
  h_plan(M, N, K, true, &tb, &s);
  return s;
}

bool gemm_h_pre_128(int M, int N, int K, int splits) {
  int tb = 64, s = 1;
  h_plan(M, N, K, splits > 1, &tb, &s);
  return tb == 128;
}

template <typename EB, typename EO>
hipError_t gemm_h(GemmMode mode, int M, int N, int K, const HalfPlanes& A, const cx<EB>* B, long ldb,
                  const float* bscale, const Epi<EO>& epi, int splits, c128* part, hipStream_t st, GemmRole role) {
  if (M <= 0 || N <= 0) return hipSuccess;
  if (!A.p || A.rows < M || A.ld % HBK || A.ld < ((K + HBK - 1) / HBK) * HBK) return hipErrorInvalidValue;
  int tb = 64, planned = 1;
  h_plan(M, N, K, true, &tb, &planned);
  if (splits < 1) splits = 1;
  int kchunk = (K + splits - 1) / splits;
  kchunk = ((kchunk + HBK - 1) / HBK) * HBK;
  if (kchunk < HBK) kchunk = HBK;
  splits = K > 0 ? (K + kchunk - 1) / kchunk : 1;
  const bool use_part = splits > 1;
  if (use_part && !part) return hipErrorInvalidValue;
  c128* pp = use_part ? part : nullptr;
  Epi<EO> en = epi;
  const int ne = epi_slots(en);
  const _Float16* nb16 = nullptr;
  auto launch = [&](auto tbc, auto modec, auto rolec) {
    constexpr int T = decltype(tbc)::value, MO = decltype(modec)::value, RO = decltype(rolec)::value;
    const dim3 grid(((M + T - 1) / T) * ((N + T - 1) / T) * splits), block(HTile<T>::NT);
    const int grp = tile_group(M, K);
    if (ne == 0 || use_part)
      hipLaunchKernelGGL((k_gemm_h<T, EB, EO, MO, RO, 0, false>), grid, block, 0, st, M, N, K, kchunk, A.p, A.rows,
                         A.ld, A.inv_scale, B, ldb, nb16, 0L, 0L, bscale, en, pp, grp);
    else if (ne == 1)
      hipLaunchKernelGGL((k_gemm_h<T, EB, EO, MO, RO, 1, false>), grid, block, 0, st, M, N, K, kchunk, A.p, A.rows,
                         A.ld, A.inv_scale, B, ldb, nb16, 0L, 0L, bscale, en, pp, grp);
    else
      hipLaunchKernelGGL((k_gemm_h<T, EB, EO, MO, RO, 3, false>), grid, block, 0, st, M, N, K, kchunk, A.p, A.rows,
                         A.ld, A.inv_scale, B, ldb, nb16, 0L, 0L, bscale, en, pp, grp);
  };
  using CN = std::integral_constant<int, GEMM_CN>;
  using NNm = std::integral_constant<int, GEMM_NN>;
  using R1 = std::integral_constant<int, 1>;
  using R2 = std::integral_constant<int, 2>;
  auto by_tile = [&](auto modec, auto rolec) {
    if (tb == 128) launch(std::integral_constant<int, 128>{}, modec, rolec);
    else launch(std::integral_constant<int, 64>{}, modec, rolec);
  };
  if (mode == GEMM_CN) by_tile(CN{}, R1{});
  else by_tile(NNm{}, R2{});
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || !use_part) return e;
  const long total = long(M) * N;
  int blocks = int((total + 255) / 256);
  if (blocks > 4096) blocks = 4096;
  hipLaunchKernelGGL((k_reduce<EO>), dim3(blocks), dim3(256), 0, st, M, N, splits, part, epi);
  return hipGetLastError();
}

template <typename E>
hipError_t scale_split_columns(int K, int N, const cx<E>* B, long ldb, float* bscale, _Float16* planes, long pld,
                               hipStream_t st) {
  if (N <= 0) return hipSuccess;
  if (K <= 0 || pld < K || pld % HBK || ldb < K) return hipErrorInvalidValue;
  const long total = long(N) * pld;
  if (pld <= kScaleSplit) {
    hipLaunchKernelGGL((k_scale_split<E>), dim3(unsigned(N)), dim3(CST), 0, st, K, B, ldb, bscale, planes, pld, total);
    return hipGetLastError();
  }
  hipLaunchKernelGGL((k_colscale<E>), dim3(unsigned(N)), dim3(CST), 0, st, long(K), B, ldb, bscale, nullptr);
  const long blocks = std::min<long>((total + 255) / 256, 65536);
  hipLaunchKernelGGL((k_split_columns<E>), dim3(unsigned(blocks)), dim3(256), 0, st, K, N, B, ldb, bscale, planes,
                     pld);
  return hipGetLastError();
}

template <typename EO>
hipError_t gemm_h_pre(GemmMode mode, int M, int N, int K, const HalfPlanes& A, const HalfPlanes& Bp,
                      const float* bscale, const Epi<EO>& epi, int splits, c128* part, hipStream_t st, GemmRole role) {
  if (M <= 0 || N <= 0) return hipSuccess;
  const long kp = ((std::max(K, 0) + HBK - 1) / HBK) * HBK;
  if (!A.p || A.rows < M || A.ld % HBK || A.ld < kp) return hipErrorInvalidValue;
  if (!Bp.p || Bp.rows != N || Bp.ld % HBK || Bp.ld < kp) return hipErrorInvalidValue;
  int tb = 64, s = 1;
  h_plan(M, N, K, splits > 1, &tb, &s);
  if (splits < 1) splits = 1;
  int kchunk = (K + splits - 1) / splits;
  kchunk = ((kchunk + HBK - 1) / HBK) * HBK;
  if (kchunk < HBK) kchunk = HBK;
  splits = K > 0 ? (K + kchunk - 1) / kchunk : 1;
  const bool use_part = splits > 1;
  if (use_part && !part) return hipErrorInvalidValue;
  Epi<EO> en = epi;
  const int ne = epi_slots(en);
  const cx<double>* nb64 = nullptr;
  c128* np = use_part ? part : nullptr;
  auto launch = [&](auto tbc, auto modec, auto rolec) {
    constexpr int T = decltype(tbc)::value, MO = decltype(modec)::value, RO = decltype(rolec)::value;
    const dim3 grid(((M + T - 1) / T) * ((N + T - 1) / T) * splits);
    const int grp = tile_group(M, K);
    auto go = [&](auto nec) {
      constexpr int NEC = decltype(nec)::value;
      if constexpr (T == PT)
        hipLaunchKernelGGL((k_gemm_hp<EO, MO, RO, NEC>), grid, dim3(256), 0, st, M, N, K, kchunk, A.p, A.rows, A.ld,
                           A.inv_scale, Bp.p, Bp.rows, Bp.ld, bscale, en, np, grp);
      else
        hipLaunchKernelGGL((k_gemm_h<T, double, EO, MO, RO, NEC, true>), grid, dim3(HTile<T>::NT), 0, st, M, N, K,
                           kchunk, A.p, A.rows, A.ld, A.inv_scale, nb64, 0L, Bp.p, Bp.rows, Bp.ld, bscale, en, np, grp);
    };
    if (ne == 0 || use_part) go(std::integral_constant<int, 0>{});
    else if (ne == 1) go(std::integral_constant<int, 1>{});
    else go(std::integral_constant<int, 3>{});
  };
  using CN = std::integral_constant<int, GEMM_CN>;
  using NNm = std::integral_constant<int, GEMM_NN>;
  using R1 = std::integral_constant<int, 1>;
  using R2 = std::integral_constant<int, 2>;
  auto by_tile = [&](auto modec, auto rolec) {
    if (tb == 128) launch(std::integral_constant<int, 128>{}, modec, rolec);
    else launch(std::integral_constant<int, 64>{}, modec, rolec);
  };
  if (mode == GEMM_CN) by_tile(CN{}, R1{});
  else by_tile(NNm{}, R2{});
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || !use_part) return e;
  const long total = long(M) * N;
  int blocks = int((total + 255) / 256);
  if (blocks > 4096) blocks = 4096;
  hipLaunchKernelGGL((k_reduce<EO>), dim3(blocks), dim3(256), 0, st, M, N, splits, part, epi);
  return hipGetLastError();
}

template <typename E>
hipError_t column_scales(long rows, int ncols, const cx<E>* B, long ldb, float* bscale, hipStream_t st) {
  if (ncols <= 0) return hipSuccess;
  hipLaunchKernelGGL((k_colscale<E>), dim3(ncols), dim3(CST), 0, st, rows, B, ldb, bscale, nullptr);
  return hipGetLastError();
}

hipError_t column_maxabs(long rows, int ncols, const c128* X, long ldx, double* out, hipStream_t st) {
  if (ncols <= 0) return hipSuccess;
  hipLaunchKernelGGL((k_colscale<double>), dim3(ncols), dim3(CST), 0, st, rows, X, ldx, nullptr, out);
  return hipGetLastError();
}

hipError_t split_planes(const c128* X, long ldx, int rows_x, int cols_x, bool transpose, double scale,
                        _Float16* planes, long prow, long pld, hipStream_t st) {
  const int ksrc = transpose ? cols_x : rows_x;
  if (prow != (transpose ? rows_x : cols_x) || pld < ksrc) return hipErrorInvalidValue;
  const long total = prow * pld;
  if (total <= 0) return hipSuccess;
  const long blocks = std::min<long>((total + 255) / 256, 65536);
  hipLaunchKernelGGL(k_split_planes, dim3(unsigned(blocks)), dim3(256), 0, st, X, ldx, ksrc, transpose, scale, planes,
                     prow, pld);
  return hipGetLastError();
}

template hipError_t gemm_h<float, double>(GemmMode, int, int, int, const HalfPlanes&, const c64*, long, const float*,
                                          const Epi<double>&, int, c128*, hipStream_t, GemmRole);
template hipError_t gemm_h_pre<float>(GemmMode, int, int, int, const HalfPlanes&, const HalfPlanes&, const float*,
                                       const Epi<float>&, int, c128*, hipStream_t, GemmRole);
template hipError_t gemm_h_pre<double>(GemmMode, int, int, int, const HalfPlanes&, const HalfPlanes&, const float*,
                                        const Epi<double>&, int, c128*, hipStream_t, GemmRole);
template hipError_t scale_split_columns<float>(int, int, const c64*, long, float*, _Float16*, long, hipStream_t);
template hipError_t scale_split_columns<double>(int, int, const c128*, long, float*, _Float16*, long, hipStream_t);
template hipError_t column_scales<float>(long, int, const c64*, long, float*, hipStream_t);
template hipError_t column_scales<double>(long, int, const c128*, long, float*, hipStream_t);

#define INST(T, EA, EB, EO)                                                                               \
  template hipError_t gemm<T, EA, EB, EO>(GemmMode, int, int, int, const cx<EA>*, long, const cx<EB>*, long, \
                                          const Epi<EO>&, int, c128*, hipStream_t, GemmRole, bool, const int*, GemmForm);
INST(double, double, double, double)
INST(float, float, float, float)
INST(float, float, double, float)
INST(float, float, float, double)
INST(double, float, float, double)
INST(double, float, double, float)
#undef INST

}  // namespace chebfd
