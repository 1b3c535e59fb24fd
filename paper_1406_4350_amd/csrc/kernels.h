// Internal launchers of the chebfd HIP kernels (not part of the public C ABI).
#pragma once
#include "common.h"

namespace chebfd {

// Output epilogue shared by the GEMMs and the split-K reduction:
//   out = alpha * (A B) + bL * L + bU * U + bW * W      (element-wise, any of L/U/W may be null)
// `out` may alias W (the Chebyshev recurrence writes psi^i over psi^(i-2)).
template <typename E> struct Epi {
  cx<E>* out = nullptr; long ldo = 0;
  double alpha = 1.0;
  const cx<E>* L = nullptr; long ldl = 0; double bL = 0.0;
  const cx<E>* U = nullptr; long ldu = 0; double bU = 0.0;
  const cx<E>* W = nullptr; long ldw = 0; double bW = 0.0;
  bool real_only = false;  // keep the real part (inner products of real functions, Gamma point)
};

enum GemmMode { GEMM_CN = 0, GEMM_NN = 1 };
// FORM_RE: the caller keeps only the real part of conj(A)^T B (the imaginary part of the result is 0); FORM_B_REAL: the
// imaginary part of B in A B is 0 or to be taken as 0. Two real products per complex one instead of three; FORM_RE is taken
// by the tiled FP64 projections and Grams, FORM_B_REAL by the back-projections, both ignored (the full product) elsewhere.
enum GemmForm { FORM_FULL = 0, FORM_RE = 1, FORM_B_REAL = 2 };
// separate kernel instances per use, so that profiles tell them apart; projections are GEMM_CN, back-projections GEMM_NN
enum GemmRole { ROLE_SMALL = 0, ROLE_PROJECT = 1, ROLE_BACKPROJECT = 2, ROLE_SUBSPACE = 3 };

// C (M x N) = op(A) B, complex, column-major operands.
//   GEMM_CN: A stored K x M (lda), op = conjugate transpose;  GEMM_NN: A stored M x K (lda).
//   B stored K x N (ldb).
// T is the MFMA arithmetic type; EA/EB are the storage types of A and B (converted on load).
// splits > 1: K is split, FP64 partial products go to `part` (splits * M * N complex doubles) and a
// deterministic reduction applies the epilogue; splits == 1: the epilogue is applied directly.
// upper = true (M = N, a Hermitian result): only the 64 x 64 output tiles with row tile <= column tile are
// computed (the others are not written; hermitian_lower fills them), splits from gemm_upper_splits.
// pred (device, N ints): only the columns n with pred[n] not 0 are computed (the others took rns_product;
// full FP64 projections and back-projections; hipErrorInvalidValue elsewhere and at the sizes of the small GEMM, which
// have no other route).
template <typename T, typename EA, typename EB, typename EO>
hipError_t gemm(GemmMode mode, int M, int N, int K, const cx<EA>* A, long lda, const cx<EB>* B, long ldb,
                const Epi<EO>& epi, int splits, c128* part, hipStream_t st, GemmRole role = ROLE_SMALL,
                bool upper = false, const int* pred = nullptr, GemmForm form = FORM_FULL);
int gemm_upper_splits(int N, int K);
// whether an FP64 product of FP64 operands takes the small GEMM (one 16 x 16 block of the result per workgroup)
bool gemm_is_small(int M, int N, int K);
// The splits that such a product takes where `splits` partials have room, and the product left as that many partials
// (count x M x N in part, ld M) for a kernel that adds them itself (diag_parts, block_diag_parts).
int gemm_small_splits(int M, int N, int K, int splits);
hipError_t gemm_small_parts(GemmMode mode, int M, int N, int K, const c128* A, long lda, const c128* B, long ldb,
                            int count, c128* part, hipStream_t st);
// A[i][j] = conj(A[j][i]) for i > j (n x n, column-major)
hipError_t hermitian_lower(int n, c128* A, long lda, hipStream_t st);

// number of K splits the launcher would like for an (M, N, K) product on 256 CUs
int gemm_pick_splits(int M, int N, int K);

// ---- FP16 hi/lo split complex GEMM (FP32 accumulation) ---------------------------------------------------
// A is held as four FP16 planes (Re hi, Re lo, Im hi, Im lo) of sA * A, each row m holding its K values
// contiguously (row stride ld halves, a multiple of 8; K padded with zeros to a multiple of 32). sA is a power of
// two chosen so that max |sA A| is in [2^13, 2^14) (2^kHalfTopExp, near the top of the FP16 range):
// hi = fp16(sA a), lo = fp16(sA a - hi), so hi + lo carries about 22 significant bits for every entry down to
// about 2^-17 of the largest, both halves being normal FP16 numbers there. Products of such operands reach 2^28
// and their sums over K stay far inside the FP32 range of the accumulators.
constexpr int kHalfTopExp = 14;
struct HalfPlanes {
  const _Float16* p = nullptr;  // [4][rows][ld]: Re hi, Re lo, Im hi, Im lo
  long rows = 0, ld = 0;
  double inv_scale = 1.0;  // 1 / sA
};
// out (M x N) = op(A) B with op(A)[m][k] = A[m][k] (GEMM_NN) or conj(A[m][k]) (GEMM_CN, A = the conjugate-
// transposed operand stored row m = output row). B (K x N, column-major, ldb) is split on the fly after
// scaling column n by bscale[n] (a power of two, see column_scales); each product is hi*hi + hi*lo + lo*hi on
// the 16x16x32 FP16 MFMA. Splits and epilogue as for gemm().
template <typename EB, typename EO>
hipError_t gemm_h(GemmMode mode, int M, int N, int K, const HalfPlanes& A, const cx<EB>* B, long ldb,
                  const float* bscale, const Epi<EO>& epi, int splits, c128* part, hipStream_t st, GemmRole role);
// B scaled and split once, exactly as column_scales and the on-the-fly split of gemm_h: bscale[n], and planes [4][N][pld]
// of bscale[n] B[k][n] (Re hi, Re lo, Im hi, Im lo; zero for K <= k < pld), pld >= K a multiple of 32
template <typename E>
hipError_t scale_split_columns(int K, int N, const cx<E>* B, long ldb, float* bscale, _Float16* planes, long pld,
                               hipStream_t st);
// gemm_h with B given as such planes (Bp.rows = N, Bp.ld = pld, Bp.inv_scale unused); splits > 1 sums split-K
// partials in part as gemm_h does. The products are those of gemm_h; its 64 x 64 tiles sum them in the same order, the
// 128 x 128 tiles (k_gemm_hp) in another, so that results agree to the rounding of the FP32 sums.
template <typename EO>
hipError_t gemm_h_pre(GemmMode mode, int M, int N, int K, const HalfPlanes& A, const HalfPlanes& Bp,
                      const float* bscale, const Epi<EO>& epi, int splits, c128* part, hipStream_t st, GemmRole role);
int gemm_h_pick_splits(int M, int N, int K);
// whether gemm_h_pre takes its 128 x 128 tiles with these splits
bool gemm_h_pre_128(int M, int N, int K, int splits);
// upper bound of both split rules, for sizing split-K partial buffers
int gemm_split_bound(int M, int N, int K);
// the work item (M tile bx, N tile by, split bz) the tiled kernels give block i of a `total`-block launch
void gemm_block_item(int i, int total, int tm, int tn, int grp, int& bx, int& by, int& bz);
// bscale[n] = 2^-e with max_k |B[k][n]| (over Re and Im) in [2^(e-1), 2^e); 1 for a zero column
template <typename E> hipError_t column_scales(long rows, int ncols, const cx<E>* B, long ldb, float* bscale,
                                               hipStream_t st);
// per-column max |Re|, |Im| of a complex128 matrix (FP64), for the global scale of the split planes
hipError_t column_maxabs(long rows, int ncols, const c128* X, long ldx, double* out, hipStream_t st);
// planes of sA * X for a complex128 X (rows_x x cols_x, ld ldx). transpose = false: plane row r = column r of X
// (k runs down X's column); transpose = true: plane row r = row r of X (k runs along X's row).
hipError_t split_planes(const c128* X, long ldx, int rows_x, int cols_x, bool transpose, double scale,
                        _Float16* planes, long prow, long pld, hipStream_t st);

// ---- large FP64 complex products on the INT8 matrix cores ---------------------------------------------------
// Operands as residues modulo kRnsMods coprime numbers (see gemm_rns.hip): int8 planes [2 l] (real parts) and
// [2 l + 1] (imaginary parts) at base + i plane, the sums' (or differences') plane l at third + l third_plane; row r of a
// plane at r ld, its K values contiguous and padded with zeros to ld = rns_ld(K). inv[r] undoes the row's scale.
constexpr int kRnsMods = 16, kRnsKTile = 128, kRnsMaxK = 146560;
inline long rns_ld(long K) { return (K + kRnsKTile - 1) / kRnsKTile * kRnsKTile; }
inline long rns_ldc(long M) { return (M + 15) / 16 * 16; }
struct RnsOperand {
  const int8_t* base = nullptr;
  const int8_t* third = nullptr;
  long plane = 0, third_plane = 0, ld = 0;
  const double* inv = nullptr;
  const double* env = nullptr;  // A: min over its rows of |entry k| / |row|, K values
};
constexpr double kRnsOverlap = 1.0 / 256;  // smallest sum_k |a_k b_k| / (|a| |b|) of a column that takes the INT8 route
// Host arithmetic, the operations of the kernels: modulus number l, the largest |integer| that its split reduces and the
// largest |residue| that kRnsMaxK counts on; the largest |residue| left of x0 <= x < x1.
void rns_residue_limits(int* modulus, int l, int* sum, int* residue);
int rns_residue_largest(int l, int x0, int x1);
// Columns taken at a time by a product on the INT8 matrix cores, whose residue planes (48 bytes per complex entry of
// the operand and of the result) are scratch: about equal pieces of at most kRnsChunk columns, whole tiles of 256.
constexpr int kRnsChunk = 1024;
inline long rns_chunk(long n) {
  const long pieces = (n + kRnsChunk - 1) / kRnsChunk, per = (n + pieces - 1) / pieces, whole = (per + 255) / 256 * 256;
  return n < whole ? n : whole;
}
// Estimated times (us) of an M x N x K product, P^H x or (back) P w with its vector epilogue, on the FP64 and on the INT8
// matrix cores with A already split; whether INT8 is the faster, at N columns or at some width up to N
void rns_cost(int M, int N, int K, bool back, double* fp64, double* int8);
bool rns_pays(int M, int N, int K, bool back);
bool rns_pays_some(int M, int N, int K, bool back);
// Power-of-two scales of the columns (K x N, ldb) and their inverses, and where asked for 1 / norms (0 for a column of
// zeros), flag[n] = 1 (else 0) for a column not fit for the integers (NaN, Inf, entries beyond 1e+-130) or, with A's
// envelope, of too small an overlap with A's rows; *any = 1 (else untouched) if one is not. rns_product leaves flagged
// columns to gemm() with pred = flag.
template <typename E>
hipError_t rns_scale_cols(long K, int N, const cx<E>* B, long ldb, const double* env, double* scale, double* inv,
                          double* rnorm, int* flag, int* any, hipStream_t st);
// the same of the rows (M x K, lda), with the envelope of the columns, whose 1 / norms are cnorm, over the rows
template <typename E>
hipError_t rns_scale_rows(long M, int K, const cx<E>* A, long lda, double* scale, double* inv, double* rnorm,
                          const double* cnorm, double* env, int* any, hipStream_t st);
// the envelope of the rows over the columns; the overlap that an envelope leaves a vector of K equal entries
template <typename E>
hipError_t rns_row_envelope(long M, int K, const cx<E>* A, long lda, const double* rnorm, double* env, hipStream_t st);
hipError_t rns_flat_overlap(long K, const double* env, double* out, hipStream_t st);
// Residue planes of scaled columns (row n of a plane = column n; base null: not written) with the sums re + im or, with
// diff, the differences re - im as third planes, nothing for a column n with flag[n fs] set, and of scaled rows (row m = row
// m) with the sums (nothing if *flag is set).
template <typename E>
hipError_t rns_split_cols(long K, int N, const cx<E>* B, long ldb, const double* scale, int8_t* base, int8_t* third,
                          bool diff, long plane, long ld, const int* flag, int fs, hipStream_t st);
template <typename E>
hipError_t rns_split_rows(long M, int K, const cx<E>* A, long lda, const double* scale, int8_t* base, int8_t* sum,
                          long plane, long ld, const int* flag, hipStream_t st);
// out (M x N) = conj(A)^T B (GEMM_CN, A's third planes the differences) or A B (GEMM_NN, the sums; B's always the
// sums) with the epilogue of gemm(), the columns with flag[n] set left alone. C: 3 kRnsMods N rns_ldc(M) bytes of
// scratch. N <= 65535.
template <typename EO>
hipError_t rns_product(GemmMode mode, int M, int N, int K, const RnsOperand& A, const RnsOperand& B, int8_t* C,
                       const Epi<EO>& epi, const int* flag, hipStream_t st);

// ---- FFT passes (per batch of bands) -------------------------------------------------------------------
struct FftGeom {
  int n, ncol, npw, rx;
  const int4* col;  // per column: {x-line index gx + rx, y = gy mod n, first sphere entry, length}
  const int* ent;   // per sphere entry: (column << 8) | (gz mod n)
  const int4* xline;  // per x-line xi = gx + rx: {first column, lowest gy, number of columns (consecutive gy), 0}
  bool narrow = false;  // every |gx| and |gy| <= n / 4
};
template <typename T>
hipError_t fft_col_inverse(const FftGeom& g, const cx<T>* tw, const cx<T>* X, long ldx, int nb, cx<T>* colbuf,
                           hipStream_t st);
template <typename T>
hipError_t fft_plane(const FftGeom& g, const cx<T>* tw, const T* Vt, const cx<T>* cin, cx<T>* cout, int nb,
                     hipStream_t st);
template <typename T>
hipError_t fft_col_forward(const FftGeom& g, const cx<T>* tw, const cx<T>* colbuf, const cx<T>* X, long ldx,
                           const T* kin, cx<T>* out, long ldo, int nb, hipStream_t st);
// the three passes in one launch, one block per band, where fft_band_fits (small boxes); kin null: no kinetic term
template <typename T> bool fft_band_fits(const FftGeom& g);
template <typename T>
hipError_t fft_band(const FftGeom& g, const cx<T>* tw, const T* Vt, const cx<T>* X, long ldx, const T* kin, cx<T>* out,
                    long ldo, int nb, hipStream_t st);
hipError_t fft_prepare_attributes();
// dV[x][y][z] += coef n^-3 sum_b w_b Re(conj(a_b(r)) psi_b(r)) for nband bands of z-transformed disk columns ca, cb
// (w = null: all weights 1); part: cross_density_part_doubles(n, nband) doubles of scratch. For n > 64 and ca != cb,
// scale[b] = (|psi_b| / |a_b|)^(1/2) balances the two fields of the polarisation form (balance_scales); else unused.
template <typename T>
hipError_t cross_density(const FftGeom& g, const cx<T>* tw, const cx<T>* ca, const cx<T>* cb, int nband,
                         const double* wts, const double* scale, double coef, double* part, double* dV,
                         hipStream_t st);
// s[b] = (pp[b].re / aa[b].re)^(1/4) from squared norms (col_dots of a with a and of psi with psi); 1 if degenerate
hipError_t balance_scales(int nb, const c128* aa, const c128* pp, double* s, hipStream_t st);
size_t cross_density_part_doubles(int n, int nband);
size_t fft_xdens_lds_bytes(int n, int rx, bool dbl);
// dynamic LDS bytes of the plane pass for box n, x-line half-width rx (0 if n unsupported)
size_t fft_plane_lds_bytes(int n, int rx, bool dbl);
// blocks of the plane pass resident on the current device at once (its persistent grid for large batches)
int fft_plane_blocks(int n, int rx, bool narrow, bool dbl);
// Row stride (in elements) of the disk-column buffers [band][z][column]: the column count rounded up to 16, so
// that every z-row starts on a 128-byte line (the column passes read 16 or 32 neighbouring columns of a row)
__host__ __device__ inline int col_stride(int ncol) { return (ncol + 15) & ~15; }
// Gamma point: U[:, j] = bands 2j + i 2j+1 expanded to the whole sphere (gmap: half index | conj << 30, h0 the
// half index of G = 0 or -1); out = the two bands separated from the transformed W, scaled back, + K X
template <typename T>
hipError_t gamma_pack(int npf, int nb, const int* gmap, int h0, const cx<T>* X, long ldx, cx<T>* U, long ldu,
                      hipStream_t st);
template <typename T>
hipError_t gamma_split(int nh, int nb, const int2* pair, int h0, const cx<T>* W, long ldw, const T* kin,
                       const cx<T>* X, long ldx, cx<T>* out, long ldo, hipStream_t st);

// ---- small projector-space and vector kernels -------------------------------------------------------------
// out[:, b] = blockdiag(D) in[:, b]; pinfo[i] = {first row of i's atom, block size, offset of the block in D}
hipError_t block_diag_apply(int nproj, int nb, const int4* pinfo, const double* D, const c128* in, long ldi,
                            c128* out, long ldo, hipStream_t st);
// out[i, b] = d[i] * in[i, b]
// Minv (packed like D, complex) = inverses of the atom diagonal blocks of the HPD matrix C (blocks up to 32;
// bad[0] = 1 otherwise). Preconditioner of the iterative capacitance solve (Sec. 5.1).
hipError_t block_inverse(int nproj, const int4* pinfo, const c128* C, long ldc, c128* Minv, int* bad, hipStream_t st);
// out = blockdiag(M) in (+ out if accumulate), complex packed blocks
hipError_t block_diag_apply_c(int nproj, int nb, const int4* pinfo, const c128* M, const c128* in, long ldi, c128* out,
                              long ldo, bool accumulate, hipStream_t st);
hipError_t diag_apply(int nproj, int nb, const double* d, const c128* in, long ldi, c128* out, long ldo,
                      hipStream_t st);
// The same (d, blockdiag(D), and a dense nproj x nproj A up to kDensePartsProj) of a sum of `parts` partials (nproj x nb each, ld nproj), their real parts with real_only
hipError_t diag_parts(int nproj, int nb, const double* d, int parts, const c128* part, bool real_only, c128* out,
                      long ldo, hipStream_t st);
hipError_t block_diag_parts(int nproj, int nb, const int4* pinfo, const double* D, int parts, const c128* part,
                            bool real_only, c128* out, long ldo, hipStream_t st);
// 192: one block per band pulls all of A through its CU. S^-1 X at 24^3, 8 bands, waited for one by one (and in a row), with
// this kernel and with a reduction launch and k_gemm_s: 29.3 and 32.0 us (16.4, 19.5) at 65 projectors, 32.9 and 34.3 (16.7,
// 19.8) at 169, 35.1 and 33.8 (18.1, 19.7) at 208.
constexpr int kDensePartsProj = 192;
hipError_t dense_parts(int nproj, int nb, const c128* A, int parts, const c128* part, bool real_only, c128* out, long ldo,
                       hipStream_t st);
// Projector space of a filter step with an overlap (S = I + P Q P^H, Q diagonal, C = Q^-1 + P^H P): open: dp = D cur and
// qdp = Q^-1 D cur (both ld ldd); close: out = s1 (Q^-1 (dp - w) - c cur) - s2 prev (prev may be null or out), and with
// next the open of out for the following step. atom: projectors of the largest atom.
hipError_t overlap_open(int nproj, int nb, int atom, const int4* pinfo, const double* D, const double* Q,
                        const c128* cur, long ldc, c128* dp, c128* qdp, long ldd, hipStream_t st);
hipError_t overlap_close(int nproj, int nb, int atom, const int4* pinfo, const double* D, const double* Q, c128* dp,
                         c128* qdp, long ldd, const c128* w, long ldw, double s1, double c, const c128* cur, long ldc, double s2,
                         const c128* prev, long ldp, c128* out, long ldo, bool next, hipStream_t st);
// out = a x + b y (+ c z), complex, any storage type
template <typename E>
hipError_t axpbypcz(long rows, int nb, double a, const cx<E>* x, long ldx, double b, const cx<E>* y, long ldy,
                    double c, const cx<E>* z, long ldz, cx<E>* out, long ldo, hipStream_t st);
template <typename EO, typename EI>
hipError_t convert_copy(long rows, int nb, const cx<EI>* in, long ldi, cx<EO>* out, long ldo, hipStream_t st);
// per column: out[b] = sum_i conj(x[i,b]) y[i,b]  (deterministic, FP64 accumulation)
template <typename E>
hipError_t col_dots(long rows, int nb, const cx<E>* x, long ldx, const cx<E>* y, long ldy, c128* out,
                    hipStream_t st);
// per column: out[b] = || R[:, b] - lam[b] U[:, b] ||_2
template <typename E>
hipError_t col_resid_norms(long rows, int nb, const cx<E>* R, long ldr, const cx<E>* U, long ldu,
                           const double* lam, double* out, hipStream_t st);
// H, S (n x n): symmetric scaling by 1/sqrt(S_ii), Hermitisation; writes scale d; bad[0] = 1 if some
// S_ii is not positive, bad[1] = 1 if an entry is not finite (plain stores, bad must be cleared first)
hipError_t rr_prepare(int n, c128* H, c128* S, double* d, int* bad, hipStream_t st);
// Z[i, j] *= d[i]
hipError_t scale_rows(int n, int ncols, c128* Z, long ldz, const double* d, hipStream_t st);
// full Hermitian matrix from its lower triangle
hipError_t hermitian_from_lower(int n, c128* A, long lda, hipStream_t st);
// C = diag(1/q) + G
hipError_t capacitance(int n, const c128* G, const double* q, c128* C, hipStream_t st);
// V [x][y][z] (FP64) -> Vt [z][y][x] in T
template <typename T> hipError_t transpose_potential(int n, const double* V, T* Vt, hipStream_t st);
template <typename E> hipError_t fill_zero(cx<E>* p, long count, hipStream_t st);
// dst[:, didx ? didx[j] : j] = src[:, sidx ? sidx[j] : j] for j < ncols (gather / scatter of band columns)
template <typename E>
hipError_t permute_cols(long rows, int ncols, const cx<E>* src, long lds, const int* sidx, cx<E>* dst, long ldd,
                        const int* didx, hipStream_t st);
// out[:, j] = a[:, j] - lam[j] b[:, j]  (contiguous rows x nb, complex128)
hipError_t sub_scaled_cols(int rows, int nb, const c128* a, const c128* b, const double* lam, c128* out,
                           hipStream_t st);
// out[e] += alpha sum_b w_b Re(conj(x[k,b]) y[l,b] + conj(x[l,b]) y[k,b]) for packed block entry e = (k, l)
hipError_t block_grad(int dsize, const int2* dent, int nb, const c128* x, long ldx, const c128* y, long ldy,
                      const double* wts, double alpha, double* out, hipStream_t st);
// B[i + j nk] = w_i conj(Z[j + i ldz]), i < nk, j < nb
hipError_t weighted_adjoint(int nk, int nb, const double* w, const c128* Z, long ldz, c128* B, hipStream_t st);
// R[:, i] -= lam[i] U[:, i] for i < ncols
template <typename E>
hipError_t sub_lambda_cols(long rows, int ncols, cx<E>* R, long ldr, const cx<E>* U, long ldu, const double* lam,
                           hipStream_t st);
template <typename E> hipError_t fill_zero_real(E* p, long count, hipStream_t st);
// Warm-started refinement of H X = S X Lambda (n x n, FP64): given M1 = X^H S X, M2 = X^H H X, the correction
// X <- X (I + F) with F_ij = (M2_ij - lam_j M1_ij)/(lam_j - lam_i), F_ii = (1 - M1_ii)/2, lam_i = M2_ii/M1_ii;
// absF = off-diagonal |F| (1e300 for an unresolvable near-degenerate pair); bmax[b] = the maximum of block b's
// entries (NaN if one is NaN) for b < refine_blocks(n) <= kRefineBlocksMax; with flag, *flag_out = *flag. bmax and
// flag_out may be pinned host memory, to be read behind an event on st
constexpr int kRefineBlocksMax = 256;
int refine_blocks(int n);
hipError_t refine_update(int n, const c128* M1, long ld1, const c128* M2, long ld2, c128* F, double* lam, double* absF,
                         double* bmax, hipStream_t st, const int* flag = nullptr, int* flag_out = nullptr);
// res[0] = max |M1 - I|, res[1] = max off-diagonal |M2| / max(1, max |diag M2|) (NaN if an entry is NaN); part
// holds 3 kRefineCheckBlocks doubles of per-block maxima
constexpr int kRefineCheckBlocks = 64;
static_assert(3 * kRefineCheckBlocks <= kRefineBlocksMax, "the block maxima of the check fit the refinement's");
hipError_t refine_check(int n, const c128* M1, long ld1, const c128* M2, long ld2, double* part, double* res,
                        hipStream_t st);
hipError_t identity_matrix(int n, c128* X, hipStream_t st);
// ascending sort of lam (n <= 2048) -> ritz, perm; Z[:, k] = d .* X[:, perm[k]]
hipError_t sort_eigen(int n, const double* lam, double* ritz, int* perm, const c128* X, const double* d, c128* Z,
                      hipStream_t st);
// LOBPCG: W[:, j] = K(t / E_kin(x_a)) (HX - lambda_a SX)[:, a], a = act[j], with the rational kinetic
// preconditioner K(x) = (27 + 18x + 12x^2 + 8x^3) / (27 + 18x + 12x^2 + 8x^3 + 16x^4)
template <typename E>
hipError_t lobpcg_precondition(long rows, int nact, const E* kin, const cx<E>* X, const cx<E>* HX, const cx<E>* SX,
                               long ld, const double* lam, const int* act, cx<E>* W, long ldw, hipStream_t st);
// R = Re A; A = R + 0 i (real symmetric eigenproblems of the Gamma point)
hipError_t real_part(long rows, int cols, const c128* A, long lda, double* R, long ldr, hipStream_t st);
hipError_t complex_from_real(long rows, int cols, const double* R, long ldr, c128* A, long lda, hipStream_t st);
// flag[0] = 1 if any entry of A (rows x cols, ld lda) is NaN or Inf (plain stores of 1, no atomics)
hipError_t flag_nonfinite(long rows, int cols, const c128* A, long lda, int* flag, hipStream_t st);
// flag[0] = 1 if any of x[0 .. count) is NaN or Inf (plain stores of 1, no atomics)
hipError_t flag_nonfinite_real(long count, const double* x, int* flag, hipStream_t st);
// Z[:, j] *= 1 / sqrt(s[j])
hipError_t scale_cols_isqrt(int n, int ncols, c128* Z, long ldz, const double* s, hipStream_t st);
// out[i] = Re a[i] / Re b[i]
hipError_t ratio_real(int nb, const c128* a, const c128* b, double* out, hipStream_t st);
// out[j] = ||a_j - b_j|| / ||b_j|| over the rows of column j (projector-space blocks, FP64)
hipError_t col_rel_diff(int rows, int nb, const c128* a, long lda, const c128* b, long ldb, double* out,
                        hipStream_t st);

// Clusters of the Rayleigh-Ritz refinement: bits[i W + w] bit b set when |F_ij| > tau, j = 32 w + b, i != j
// (W = ceil(n / 32)). cluster_eig solves each cluster's pencil (M2_CC, M1_CC), members idx[off[c] ..
// off[c+1]) with 2 <= size <= kClusterMax, and writes its eigenvectors into the block (C, C) of Q, which must
// hold the identity elsewhere; flag[0] = 1 if an M1_CC is not positive definite.
constexpr int kClusterMax = 48;
hipError_t coupling_bits(int n, const double* absF, double tau, unsigned* bits, hipStream_t st);
hipError_t cluster_eig(int nclusters, const c128* M1, long ld1, const c128* M2, long ld2, const int* idx, const int* off,
                       c128* Q, long ldq, int* flag, hipStream_t st);

}  // namespace chebfd
