// Device pieces shared by the complex GEMMs: placement of the output tiles on the XCDs, the vector epilogue.
#pragma once
#include "kernels.h"

namespace chebfd {
namespace {

// Block placement. The hardware deals the blocks of a launch to the 8 XCDs in turn (block i to XCD i mod 8),
// each XCD with its own L2. Physical block i takes the logical item that gives each XCD one contiguous run of
// items. Items are numbered split by split; inside a split, in groups of `grp` M tiles, and inside a group with
// the M tile fastest. With grp = 8 the blocks an XCD holds at once (32 to 64) cover a square-ish patch of up to 8
// M tiles by 4 to 8 N tiles, so each slice of A and of B they read is shared by several resident blocks in the
// XCD's L2: the rule for long contractions (K >= M: projections, Gram matrices), where both operands stream
// K-long slices. With grp = 1 the N tile runs fastest and each M tile's slice of A is read once, by all N tiles
// at the same time: the rule for tall, short-K products (back-projection, rotation), whose A dwarfs B.
constexpr int kTileGroup = 8;
constexpr int kUpperTiles = -1;  // group value of the upper-triangle tile order (Hermitian products)
__host__ __device__ inline void gemm_tile_of(int i, int total, int tm, int tn, int grp, int& bx, int& by, int& bz) {
  const int q = total / 8, rem = total % 8, k = i % 8, j = i / 8;
  const int L = (k < rem ? k * (q + 1) : rem * (q + 1) + (k - rem) * q) + j;
  if (grp == kUpperTiles) {  // the tiles bx <= by of a square grid, column by column: t = by (by + 1) / 2 + bx
    const int per = tm * (tm + 1) / 2;
    bz = L / per;
    const int t = L - bz * per;
    int c = int((sqrt(8.0 * t + 1.0) - 1.0) * 0.5);
    while (c * (c + 1) / 2 > t) --c;
    while ((c + 1) * (c + 2) / 2 <= t) ++c;
    by = c;
    bx = t - c * (c + 1) / 2;
    return;
  }
  const int per = tm * tn;
  bz = L / per;
  const int t = L - bz * per;
  const int first = (t / (grp * tn)) * grp;
  const int gm = tm - first < grp ? tm - first : grp;  // M tiles in this group (fewer in the last)
  const int r = t - first * tn;
  bx = first + r % gm;
  by = r / gm;
}

template <typename E>
__device__ __forceinline__ void epi_store(const Epi<E>& e, long m, long n, double re, double im) {
  double xr = e.alpha * re, xi = e.alpha * im;
  if (e.L) { cx<E> v = e.L[m + n * e.ldl]; xr += e.bL * double(v.x); xi += e.bL * double(v.y); }
  if (e.U) { cx<E> v = e.U[m + n * e.ldu]; xr += e.bU * double(v.x); xi += e.bU * double(v.y); }
  if (e.W) { cx<E> v = e.W[m + n * e.ldw]; xr += e.bW * double(v.x); xi += e.bW * double(v.y); }
  e.out[m + n * e.ldo] = cx<E>{E(xr), e.real_only ? E(0) : E(xi)};
}

}  // namespace
}  // namespace chebfd
