// HIP kernels for parallel-in-time SRTM filtering and smoothing on gfx950.
//
// Method: Yaghoobi & Sarkka, arXiv 2410.00627, Sec. IV. The forward pass is the
// parallel IMKF: an inclusive scan of the filter elements (eq. a-k-f) under the
// operator of eq. op-filter, which yields the slow-rate carry (m^f_{k,l}, P^f_{k,l}).
// The reverse pass is the parallel IMS: a suffix scan of the smoother elements
// (eq. parallel-ak-smoothing) under eq. op-smoother, which yields (m^s_{k,1}, P^s_{k,1}),
// followed by the per-window fast-rate recovery of eq. seq-smoothing-all
// (Remarks fast-par-filter and parallel-fast-smoothing).
//
// Design points specific to this implementation (the paper's equations are unchanged):
//  * The model is time invariant, so every filter element with k > 1 shares its matrix
//    part (F, D, J); a run of 2^p consecutive elements therefore has matrices that depend
//    on p only. The constants kernel computes them once per call (repeated squaring under
//    eq. op-filter), and the per-tile up-sweeps combine only the vector parts (d, eta)
//    with per-level coefficient matrices shared by every lane.
//  * The first element is written as a prior state (0, m0, P0, 0, 0) combined with the
//    generic element of window 1; this equals the paper's a_1 = (0, m^f_{1,l}, P^f_{1,l}).
//  * A prefix that contains the prior has F = 0, so every exclusive prefix is a "state"
//    (m, P) and the down-sweeps combine states with aligned segments.
//  * The reverse scan runs over the same tree: (eta, J) of a run of filter elements is the
//    information that its measurements hold about the state before it, and the information of all
//    later windows together with the filter state gives the smoothed blocks of eq.
//    seq-smoothing-all. A window's bits select the runs before it (states) and after it
//    (information), each run once, so one fold finds both.
//  * Under such a model the covariances settle after some hundred windows; a tile whose windows
//    share them takes vectors only (settled tiles).
//  * Short dependent chains (level chain, upper levels of the fold) hold one matrix entry per lane
//    and run on the float64 matrix cores.
//  * Within a window only the blocks the outputs need are formed (Remark
//    cross-covariances): P^f_{k,i,i}, P^f_{k,i,l} and means, from per-step constants
//    A^i, Q_ii, Q_il, c_i, instead of the dense (l nx)^2 window covariance.
//  * Models given per window (time varying) share nothing between elements: their kernels
//    (k_tv_*) build each window's constants and element in one lane and scan whole elements.

#include <hip/hip_ext.h>

#include <type_traits>

#include "srtm_device.h"
#include "srtm_entry.h"
#include "srtm_layout.h"

namespace srtm {

// Every array of a call is device (global) memory. Pointers read from a descriptor are
// generic; passing them through the global address space lets the compiler emit global
// instead of flat loads and stores.
template <typename T>
SRTM_DEV T* as_global(T* p) {
  using G = __attribute__((address_space(1))) T*;
  return (T*)((G)p);
}
template <typename T>
SRTM_DEV T* as_global(const void* p) {
  return as_global(static_cast<T*>(const_cast<void*>(p)));
}

// Store of one scalar to device memory through a global pointer.
template <typename T>
SRTM_DEV void put_global(T* p, T v) {
  *(__attribute__((address_space(1))) T*)p = v;
}

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));

// Staged copy of n scalars with the nthr threads of a workgroup: value q = ld(q) is handed to
// st(q, value). Each thread issues up to B loads before its first store.
template <int B, typename T, class LD, class ST>
SRTM_DEV void staged_copy(int n, int tid, int nthr, LD ld, ST st) {
#pragma unroll 1
  for (int base = 0; base < n; base += B * nthr) {
    T v[B];
#pragma unroll
    for (int i = 0; i < B; ++i) {
      const int q = base + i * nthr + tid;
      v[i] = (q < n) ? ld(q) : T(0);
    }
#pragma unroll
    for (int i = 0; i < B; ++i) {
      const int q = base + i * nthr + tid;
      if (q < n) st(q, v[i]);
    }
  }
}

// Wave-wide sum (fixed butterfly order, identical on every lane).
SRTM_DEV double wave_sum(double v) {
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}

// Wave-wide sums of N values, each as wave_sum forms it: at every distance a lane passes the half of its values
// on that it does not keep (N - 1 exchanges or a few more, not 6 N), and ends with the sums start ..
// start + cnt - 1 in x[0 ..] (start = 0 and cnt = N before). The 33 or 34 sums of
// a wave (nx = 4) one by one took 6 us of the gradient's statistics kernel.
template <int N, int DIST, int SZ>
SRTM_DEV void wave_sums(double (&x)[SZ], int lane, int& start, int& cnt) {
  if constexpr (DIST >= 1) {
    constexpr int H = (N + 1) / 2;
    const bool up = (lane & DIST) != 0;
#pragma unroll
    for (int j = 0; j < H; ++j) {
      const double lo = x[j], hi = H + j < N ? x[H + j < N ? H + j : 0] : 0.0;
      x[j] = (up ? hi : lo) + __shfl_xor(up ? lo : hi, DIST, 64);
    }
    start += up ? H : 0;
    cnt = up ? (cnt > H ? cnt - H : 0) : (cnt < H ? cnt : H);
    wave_sums<H, DIST / 2>(x, lane, start, cnt);
  }
}

// ============================================================================ constants
// ---------------------------------------------------------------- 4 x 4 blocks on the matrix cores
// Up to four NX x NX problems (NX <= 4, padded with zeros to 4 x 4) per wave, one matrix entry per
// lane: lane 16 r + 4 b + c holds entry (r, c) of block b's matrix ("block layout"), the layout in which
// v_mfma_f64_4x4x4_4b takes its B operand and returns its result. Read as the A operand the same register is
// the transpose, so mm4(X, Y, C) = X^T Y + C for four blocks at once, and a chain of products needs no
// exchange between lanes as long as every product is written with the transposed or symmetric operand
// first. A vector is held as a matrix with equal columns. One lane per problem (64 problems per wave)
// moves more problems per cycle, but a dependent 4 x 4 combine then takes about 1 us (600 instructions of
// 4 cycles); this form takes about 0.2 us and is meant for the short chains that everything waits for.
SRTM_DEV double mm4(double x, double y, double c) { return __builtin_amdgcn_mfma_f64_4x4x4f64(x, y, c, 0, 0, 0); }

// The value of another lane of the quad: CTRL 0xB1 swaps neighbours, 0x4E swaps pairs.
template <int CTRL>
SRTM_DEV double quad_swap(double x) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(x), CTRL, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(x), CTRL, 0xf, 0xf, true);
  return __hiloint2double(hi, lo);
}

// One wave's view of the block layout: this lane's place and its 64 doubles of LDS scratch.
struct Block4 {
  int r, b, c;
  double* own;          // this lane's scratch entry
  const double* base;   // its block's entries, row-major
  double eye;
  SRTM_DEV Block4(double* scratch) {
    const int lane = threadIdx.x & 63;
    r = lane >> 4;
    b = (lane >> 2) & 3;
    c = lane & 3;
    base = scratch + 16 * b;
    own = scratch + 16 * b + 4 * r + c;
    eye = r == c ? 1.0 : 0.0;
  }
  // Transposed inverse of M (entry (r, c) of the result is entry (c, r) of M^{-1}): cofactors over the
  // determinant. Cofactor (r, c) is the determinant of the rows r^1, r^2, r^3 and columns c^1, c^2, c^3 in
  // that order: the parity of each order cancels the sign (-1)^{r+c}. ok &= the determinant is usable.
  // NX = 2: the leading 2 x 2 block alone, the identity beside it being its own inverse: one LDS read instead
  // of nine, 100000 windows (float64, L = 5) 52.1 -> 51.0 us a call, the filter's (ny = 2, float32) 43.8 -> 43.1.
  template <int NX>
  SRTM_DEV double inv_t(double M, bool& ok) const {
    *own = M;
    wave_sync();
    if constexpr (NX == 2) {
      const double x = sld(base + 4 * (r ^ 1) + (c ^ 1));
      wave_sync();
      const bool diag = (r >> 1) == (c >> 1);
      const double cof = ((r ^ c) & 1) ? -x : x;
      double det = M * cof;
      det += quad_swap<0xB1>(det);
      const double id = rcp_nr(det);
      ok = ok && (!diag || (det != 0.0 && isfinite(id)));
      return diag ? cof * id : 0.0;
    }
    double x[3][3];
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
      for (int j = 0; j < 3; ++j) x[i][j] = sld(base + 4 * (r ^ (i + 1)) + (c ^ (j + 1)));
    wave_sync();
    const double cof = x[0][0] * (x[1][1] * x[2][2] - x[1][2] * x[2][1]) -
                       x[0][1] * (x[1][0] * x[2][2] - x[1][2] * x[2][0]) +
                       x[0][2] * (x[1][0] * x[2][1] - x[1][1] * x[2][0]);
    double det = M * cof;  // summed along the row
    det += quad_swap<0xB1>(det);
    det += quad_swap<0x4E>(det);
    const double id = rcp_nr(det);
    ok = ok && det != 0.0 && isfinite(id);
    return cof * id;
  }
  // Symmetric product X Y of a pair whose exact product is symmetric (Xt = X^T, Y symmetric): both
  // orders of the product are transposes of each other bit by bit, so their mean is exactly symmetric.
  SRTM_DEV static double mm_sym(double Xt, double Y) { return 0.5 * (mm4(Xt, Y, 0.0) + mm4(Y, Xt, 0.0)); }
};

// ---------------------------------------------------------------- 8 x 8 matrices on the matrix cores
// One matrix of up to 8 x 8 (padded with zeros) per wave: as 2 x 2 blocks of the block layout, lane 16 r + 4 (2 i + j) + c
// holding entry (4 i + r, 4 j + c). X^T Y is then the sum over k of two 4 x 4 block products, block (i, j) of
// term k taking X's block (k, i) and Y's block (k, j): Lhs8 and Rhs8 hold an operand's blocks moved there (whole
// blocks move inside the row of 16 lanes, by row rotations under a bank mask).
template <int CTRL, int BANKS>
SRTM_DEV double move_banks(double old, double x) {
  const int lo = __builtin_amdgcn_update_dpp(__double2loint(old), __double2loint(x), CTRL, 0xf, BANKS, false);
  const int hi = __builtin_amdgcn_update_dpp(__double2hiint(old), __double2hiint(x), CTRL, 0xf, BANKS, false);
  return __hiloint2double(hi, lo);
}
constexpr int ROW_ROR = 0x120;  // + n: lane l of a row of 16 takes lane (l - n) mod 16
struct Lhs8 {
  double k0, k1;
  SRTM_DEV explicit Lhs8(double x)  // blocks (0, 0, 1, 1) and (2, 2, 3, 3)
      : k0(move_banks<ROW_ROR + 8, 0x8>(move_banks<ROW_ROR + 4, 0x6>(x, x), x)),
        k1(move_banks<ROW_ROR + 12, 0x6>(move_banks<ROW_ROR + 8, 0x1>(x, x), x)) {}
};
struct Rhs8 {
  double k0, k1;
  SRTM_DEV explicit Rhs8(double y)  // blocks (0, 1, 0, 1) and (2, 3, 2, 3)
      : k0(move_banks<ROW_ROR + 8, 0xc>(y, y)), k1(move_banks<ROW_ROR + 8, 0x3>(y, y)) {}
};
SRTM_DEV double mm8(const Lhs8& x, const Rhs8& y, double c) { return mm4(x.k1, y.k1, mm4(x.k0, y.k0, c)); }

// One wave's view of that layout: this lane's entry and its 64 doubles of LDS scratch (row-major 8 x 8).
template <int NX>
struct Block8 {
  static_assert(NX > 4 && NX <= 8, "two blocks a side");
  int r, c;
  double* scratch;
  SRTM_DEV explicit Block8(double* s) : scratch(s) {
    const int lane = threadIdx.x & 63, b = (lane >> 2) & 3;
    r = 4 * (b >> 1) + (lane >> 4);
    c = 4 * (b & 1) + (lane & 3);
  }
  SRTM_DEV bool in() const { return r < NX && c < NX; }
  // Transposed inverse of the leading NX x NX block of M (zero outside it): Gauss-Jordan elimination with
  // partial pivoting of [M | I], a column per lane, the pivot column read from its lane. ok &= every pivot is usable.
  // With one lane eliminating alone and the products through LDS, the constants kernel took 46 us (nx = 6, l = 20, 8
  // levels of the chain) against 26 us.
  SRTM_DEV double inv_t(double M, bool& ok) const {
    const int lane = threadIdx.x & 63;
    scratch[8 * r + c] = M;
    wave_sync();
    double a[NX];
#pragma unroll
    for (int q = 0; q < NX; ++q) {
      const double v = sld(scratch + 8 * q + (lane < NX ? lane : 0));
      a[q] = lane < NX ? v : lane - NX == q ? 1.0 : 0.0;
    }
    wave_sync();
#pragma unroll
    for (int k = 0; k < NX; ++k) {
      double p[NX];  // column k
#pragma unroll
      for (int q = 0; q < NX; ++q)
        p[q] = __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(a[q]), k),
                                __builtin_amdgcn_readlane(__double2loint(a[q]), k));
#pragma unroll
      for (int q = k + 1; q < NX; ++q)
        if (fabs(p[q]) > fabs(p[k])) {  // the same on every lane
          const double t = p[q], u = a[q];
          p[q] = p[k];
          a[q] = a[k];
          p[k] = t;
          a[k] = u;
        }
      const double ip = rcp_nr(p[k]);
      ok = ok && p[k] != 0.0 && isfinite(ip);
      a[k] *= ip;
#pragma unroll
      for (int q = 0; q < NX; ++q)
        if (q != k) a[q] = my_fma(-p[q], a[k], a[q]);
    }
    if (lane >= NX && lane < 2 * NX) {
#pragma unroll
      for (int q = 0; q < NX; ++q) scratch[8 * (lane - NX) + q] = a[q];  // column lane - NX of the inverse as a row
    }
    wave_sync();
    const double v = in() ? sld(scratch + 8 * r + c) : 0.0;
    wave_sync();
    return v;
  }
};

// Level chain over levels p0 .. p1-1, run by wave 0 of a workgroup.
// `chain` is chain_doubles(nx) doubles of LDS whose first 3 nx^2 hold F, D, J of Theta(2^p0). Writes the
// level records p0 .. p1-1 and, when p1 < nlev, F, D, J of Theta(2^p1) in float64 to `hand`
// (3 nx^2 doubles), where a continuation of the chain in a later launch picks them up. `lev64` (may be null)
// receives F, D, J of each level in float64 (lev64_off).
//   Theta(2^{p+1}) = Theta(2^p) (x) Theta(2^p) under eq. op-filter, W = (I + D J)^{-1}, and the
// coefficients that combine the vector parts of two runs of 2^p elements:
//   d_ij = G1 d_i + G2 eta_j + d_j,   eta_ij = G3 eta_j - G4 d_i + eta_i,
//   G1 = F W, G2 = F W D, G3 = (W F)^T, G4 = (W F)^T J.
// On the matrix cores, one entry per lane and no exchange but the inverse's (level_chain8: nx > 4).
template <typename T, int NX>
SRTM_DEV int level_chain4(double* chain, T* __restrict__ cst, const ConstLayout& lay, int p0, int p1, int nlev,
                          double* __restrict__ hand, double* __restrict__ lev64) {
  constexpr int NN = NX * NX;
  static_assert(NX <= 4, "4 x 4 blocks");
  const Block4 B(chain + 3 * NN);
  const bool in = B.r < NX && B.c < NX;
  const int rc = in ? B.r * NX + B.c : 0, cr = in ? B.c * NX + B.r : 0;
  double F = in ? chain[rc] : 0.0, Ft = in ? chain[cr] : 0.0;
  double D = in ? chain[NN + rc] : 0.0, J = in ? chain[2 * NN + rc] : 0.0;
  bool ok = true;
  for (int p = p0; p < p1; ++p) {
    const double Wt = B.template inv_t<NX>(mm4(D, J, B.eye), ok);  // W^T
    const double W = mm4(Wt, B.eye, 0.0);
    const double WF = mm4(Wt, F, 0.0);
    const double G3 = mm4(F, Wt, 0.0);  // (W F)^T
    const double G1 = mm4(Ft, W, 0.0);
    const double XD = Block4::mm_sym(Wt, D);  // W D
    const double XDF = mm4(XD, Ft, 0.0);      // W D F^T
    const double G2 = mm4(Ft, XD, 0.0);
    const double G4 = mm4(WF, J, 0.0);
    const double JWF = mm4(J, WF, 0.0);
    if (in) {  // the record, two entries per lane: rows (G1, G2) and (G3, -G4), then F, D, J
      T* dst = cst + lay.lev + p * lay.lev_stride;
      const double a = B.b == 0 ? G1 : B.b == 1 ? G2 : B.b == 2 ? G3 : -G4;
      dst[lay.o_C + ((B.b >> 1) * NX + B.r) * 2 * NX + (B.b & 1) * NX + B.c] = (T)a;
      const double x = B.b == 0 ? F : B.b == 1 ? D : J;
      if (B.b < 3) dst[lay.o_F + B.b * NN + rc] = (T)x;
      if (lev64 && B.b < 3) put_global(lev64 + p * 3 * NN + B.b * NN + rc, x);
    }
    const double nF = mm4(Ft, WF, 0.0), nFt = mm4(WF, Ft, 0.0);
    D = Block4::mm_sym(Ft, XDF) + D;  // F W D F^T + D
    J = Block4::mm_sym(F, JWF) + J;   // (W F)^T J F + J
    F = nF;
    Ft = nFt;
  }
  if (p1 < nlev && in && B.b < 3) put_global(hand + B.b * NN + rc, B.b == 0 ? F : B.b == 1 ? D : J);
  return ok ? 0 : SRTM_INFO_COMBINE_SINGULAR;
}

template <typename T, int NX>
SRTM_DEV int level_chain8(double* chain, T* __restrict__ cst, const ConstLayout& lay, int p0, int p1, int nlev,
                          double* __restrict__ hand, double* __restrict__ lev64) {
  constexpr int NN = NX * NX;
  const Block8<NX> B(chain + 3 * NN);
  const bool in = B.in();
  const int rc = in ? B.r * NX + B.c : 0, cr = in ? B.c * NX + B.r : 0;
  double F = in ? chain[rc] : 0.0, Ft = in ? chain[cr] : 0.0;
  double D = in ? chain[NN + rc] : 0.0, J = in ? chain[2 * NN + rc] : 0.0;
  const double eye = in && B.r == B.c ? 1.0 : 0.0;
  const Rhs8 rI(eye);
  bool ok = true;
  for (int p = p0; p < p1; ++p) {
    const Lhs8 lD(D), lJ(J), lF(F), lFt(Ft);
    const Rhs8 rD(D), rJ(J), rF(F), rFt(Ft);
    const double Wt = B.inv_t(mm8(lD, rJ, eye), ok);  // W^T
    const Lhs8 lWt(Wt);
    const Rhs8 rWt(Wt);
    const double W = mm8(lWt, rI, 0.0), WF = mm8(lWt, rF, 0.0);
    const double G3 = mm8(lF, rWt, 0.0);  // (W F)^T
    const double XD = 0.5 * (mm8(lWt, rD, 0.0) + mm8(lD, rWt, 0.0));  // W D
    const Lhs8 lXD(XD), lWF(WF);
    const Rhs8 rXD(XD), rWF(WF);
    const double G1 = mm8(lFt, Rhs8(W), 0.0), G2 = mm8(lFt, rXD, 0.0), G4 = mm8(lWF, rJ, 0.0);
    const double XDF = mm8(lXD, rFt, 0.0), JWF = mm8(lJ, rWF, 0.0);
    if (in) {  // the record: rows (G1, G2) and (G3, -G4), then F, D, J
      T* dst = cst + lay.lev + p * lay.lev_stride;
      T* o = dst + lay.o_C + B.r * 2 * NX + B.c;
      o[0] = (T)G1;
      o[NX] = (T)G2;
      o[2 * NN] = (T)G3;
      o[2 * NN + NX] = (T)-G4;
      dst[lay.o_F + rc] = (T)F;
      dst[lay.o_F + NN + rc] = (T)D;
      dst[lay.o_F + 2 * NN + rc] = (T)J;
      if (lev64) {
        put_global(lev64 + p * 3 * NN + rc, F);
        put_global(lev64 + p * 3 * NN + NN + rc, D);
        put_global(lev64 + p * 3 * NN + 2 * NN + rc, J);
      }
    }
    // F W D F^T + D and (W F)^T J F + J, exactly symmetric (Block4::mm_sym)
    D += 0.5 * (mm8(lFt, Rhs8(XDF), 0.0) + mm8(Lhs8(XDF), rFt, 0.0));
    J += 0.5 * (mm8(lF, Rhs8(JWF), 0.0) + mm8(Lhs8(JWF), rF, 0.0));
    F = mm8(lFt, rWF, 0.0);
    Ft = mm8(lWF, rFt, 0.0);
  }
  if (p1 < nlev && in) {
    put_global(hand + rc, F);
    put_global(hand + NN + rc, D);
    put_global(hand + 2 * NN + rc, J);
  }
  return ok ? 0 : SRTM_INFO_COMBINE_SINGULAR;
}

template <typename T, int NX>
SRTM_DEV int level_chain(double* chain, T* __restrict__ cst, const ConstLayout& lay, int p0, int p1, int nlev,
                         double* __restrict__ hand, double* __restrict__ lev64) {
  if constexpr (NX <= 4) return level_chain4<T, NX>(chain, cst, lay, p0, p1, nlev, hand, lev64);
  else return level_chain8<T, NX>(chain, cst, lay, p0, p1, nlev, hand, lev64);
}

// Levels 0 .. CHAIN_SPLIT-1 come from the constants kernel (the in-tile scans need the levels
// below LOG_TILE); the rest, which only the levels above the tiles use, from one workgroup of the
// tile-reduction launch, so that they are computed while the tiles are reduced (for 2^17 windows
// nine levels, 6 us at nx = 4, beside reductions of 8 us; a level costs 0.45 us more in the constants
// kernel, so a higher split does not pay).
constexpr int CHAIN_SPLIT = LOG_TILE;
static_assert(CHAIN_SPLIT >= LOG_TILE, "the tile reductions read levels below LOG_TILE");

// Dynamic LDS of the tile-reduction launch: the larger of a tile reduction's elements, tree and row
// tables and a level chain's float64 scratch.
template <typename T, int NX>
constexpr size_t fwd_reduce_lds_bytes() {
  constexpr size_t red = sizeof(T) * (size_t)(4 * NX * TILE + LOG_TILE * 4 * NX * NX);
  constexpr size_t chn = sizeof(double) * (size_t)chain_doubles(NX);
  return red > chn ? red : chn;
}

// The rest of the level chain (levels CHAIN_SPLIT .. nlev-1), continued from the handed-over
// Theta(2^CHAIN_SPLIT). The wave runs at raised priority: it shares its SIMD with reductions.
template <typename T, int NX, int NY>
SRTM_DEV void chain_tail_body(T* __restrict__ cst, const double* __restrict__ hand, double* __restrict__ lev64, int L,
                              int nlev, int32_t* info) {
  constexpr int NN = NX * NX;
  extern __shared__ char smraw[];
  double* chain = reinterpret_cast<double*>(smraw);  // chain_doubles(nx)
  const int tid = threadIdx.x;
  if (tid >= 64 || nlev <= CHAIN_SPLIT) return;
  __builtin_amdgcn_s_setprio(3);
  for (int q = tid; q < 3 * NN; q += 64) chain[q] = gld(hand + q);
  wave_sync();
  const ConstLayout lay = make_const_layout(NX, NY, L, nlev);
  const int f = level_chain<T, NX>(chain, cst, lay, CHAIN_SPLIT, nlev, nlev, nullptr, lev64);
  if (f && info) atomicOr(info, f);
}

// Per-step tables of the constants kernel for NX <= 4, on the matrix cores: A^i, Q_ii, Sig_i = sum_{u=0..i} A^u and
// al_i = sum_{j=1..i-1} A^{i-j} Q_jj for i = 0 .. L by doubling. With everything known up to s, for j = 1 .. s
//   A^{s+j} = A^j A^s,   Q_{s+j} = Q_j + A^j Q_s A^{jT},   Sig_{s+j} = Sig_{j-1} + A^j Sig_s,
//   al_{s+j} = al_j + A^j (al_s + Q_s Sig_{j-1}^T),
// one block of lanes per j, then in one pass Q_il = Q_ii (A^{l-i})^T and c_i = (1/l) (al_i + Q_ii Sig_{l-i}^T) C^T.
// Log2(l) stages of about 400 cycles; sums over the steps with one entry per thread took 14000 cycles for
// l = 20 (each an LDS round trip per term). All 256 threads; LDS arrays as in constants_body. Every entry also
// goes, unrounded, to the float64 copy.
template <typename T, int NX, int NY>
SRTM_DEV void step_tables4(int L, const ConstLayout& lay, T* __restrict__ cst, double* __restrict__ cst64,
                           const double* sC, double* Apow, double* Qii, double* Sig, double* al, double* ci) {
  constexpr int NN = NX * NX, NXY = NX * NY;
  const int lane = threadIdx.x & 63, slot = (threadIdx.x >> 6) * 4 + ((lane >> 2) & 3);  // block among the 16
  const int r = lane >> 4, c = lane & 3;
  const bool in = r < NX && c < NX;
  const int rc = in ? r * NX + c : 0, cr = in ? c * NX + r : 0;
  auto get = [&](const double* a, int i, int o) { return in ? a[i * NN + o] : 0.0; };
  for (int s = 1; s < L; s *= 2) {
    const double As = get(Apow, s, rc), Qs = get(Qii, s, rc), Ss = get(Sig, s, rc), as = get(al, s, rc);
    const int n = 2 * s < L ? s : L - s;  // j = 1 .. n
    for (int j0 = 0; j0 < n; j0 += 16) {
      const int j = j0 + slot + 1;
      const bool act = j <= n;
      const int jj = act ? j : 1;
      const double AjT = get(Apow, jj, cr), Qj = get(Qii, jj, rc), Sj = get(Sig, jj - 1, rc), SjT = get(Sig, jj - 1, cr),
                   aj = get(al, jj, rc);
      const double nA = mm4(AjT, As, 0.0);
      const double nQ = Block4::mm_sym(AjT, mm4(Qs, AjT, 0.0)) + Qj;
      const double nS = mm4(AjT, Ss, Sj);
      const double na = mm4(AjT, mm4(Qs, SjT, as), aj);
      if (act && in) {
        Apow[(s + j) * NN + rc] = nA;
        Qii[(s + j) * NN + rc] = nQ;
        Sig[(s + j) * NN + rc] = nS;
        al[(s + j) * NN + rc] = na;
      }
    }
    __syncthreads();
  }
  const double CT = r < NX && c < NY ? sC[c * NX + r] : 0.0, il = 1.0 / (double)L;
  auto put = [&](int off, double v) {
    cst[off] = (T)v;
    cst64[off] = v;
  };
  for (int i0 = 0; i0 < L; i0 += 16) {
    const int i = i0 + slot + 1;
    const bool act = i <= L;
    const int ii = act ? i : L;
    const double Q = get(Qii, ii, rc);
    const double QL = mm4(Q, get(Apow, L - ii, cr), 0.0);
    const double tT = mm4(get(Sig, L - ii, cr), Q, get(al, ii, cr));  // (al_i + Q_ii Sig_{l-i}^T)^T
    const double cv = mm4(tT, CT, 0.0) * il;
    if (act && r < NX) {
      const int base = lay.per_i + (i - 1) * lay.per_i_stride;
      if (c < NX) {
        put(base + lay.o_Ai + rc, Apow[i * NN + rc]);
        put(base + lay.o_Qii + rc, Q);
        put(base + lay.o_QiL + rc, QL);
      }
      if (c < NY) {
        put(base + lay.o_ci + r * NY + c, cv);
        ci[i * NXY + r * NY + c] = cv;
      }
    }
  }
}

// One workgroup, float64 throughout. Per-step tables are built in LDS by parallel
// loops; the slow-rate constants and the level tables by the lanes of wave 0.
//
// With Q_ij = Cov(x_{k,i}, x_{k,j} | x_{k-1,l}) = sum_{t=1..min(i,j)} A^{i-t} Q A^{(j-t)T}:
//   Q_ii = sum_{t=0}^{i-1} A^t Q A^{tT},   Q_il = Q_ii (A^{l-i})^T,
//   c_i  = (1/l) sum_j Q_ij C^T = Cov(x_{k,i}, y_k | x_{k-1,l})  (noise part),
//   C_bar = (C/l) sum_{i=1..l} A^i,  R_x = (1/l) sum_i C c_i + R,  G_bar Q~ M_bar^T = c_l,
//   Q_bar = Q_ll, A_bar = A^l   (eq. h-k-l-2, eq. y-k-l-2 and eq. a-k-f).
template <typename T, int NX, int NY>
SRTM_DEV void constants_body(const T* __restrict__ Fm, const T* __restrict__ Qm, const T* __restrict__ Hm,
                             const T* __restrict__ Rm, int L, int nlev, T* __restrict__ cst,
                             double* __restrict__ cst64, double* __restrict__ hand, double* __restrict__ lev64,
                             int32_t* info) {
  constexpr int NN = NX * NX, NXY = NX * NY;
  constexpr int W2S = (NN > 2 * NXY ? NN : 2 * NXY);
  extern __shared__ double sm[];
  const int tid = threadIdx.x, nthr = blockDim.x;
  const ConstLayout lay = make_const_layout(NX, NY, L, nlev);
  double* sA = sm;
  double* sQ = sA + NN;
  double* sC = sQ + NN;
  double* sR = sC + NXY;
  double* Apow = sR + NY * NY;          // (L+1) NN, Apow[i] = A^i
  double* Qii = Apow + (L + 1) * NN;    // (L+1) NN, Qii[i] = Q_ii (Qii[0] = 0)
  double* W1 = Qii + (L + 1) * NN;      // (L+1) NN scratch
  double* W2 = W1 + (L + 1) * NN;       // (L+1) W2S scratch
  double* ci = W2 + (L + 1) * W2S;      // (L+1) NXY, ci[i] = c_i
  double* chain = ci + (L + 1) * NXY;   // chain_doubles(nx): level-chain records and scratch

  for (int e = tid; e < NN; e += nthr) {
    sA[e] = (double)Fm[e];
    sQ[e] = (double)Qm[e];
    Apow[e] = (e / NX == e % NX) ? 1.0 : 0.0;
    Apow[NN + e] = (double)Fm[e];
  }
  for (int e = tid; e < NXY; e += nthr) sC[e] = (double)Hm[e];
  for (int e = tid; e < NY * NY; e += nthr) sR[e] = (double)Rm[e];
  auto put = [&](int off, double v) {
    cst[off] = (T)v;
    cst64[off] = v;
  };
  if constexpr (NX <= 4) {
    for (int e = tid; e < NN; e += nthr) {
      const double eye = e / NX == e % NX ? 1.0 : 0.0, a = (double)Fm[e];
      // the symmetric part of Q, as its sums use it (upper triangle mirrored)
      const int r = e / NX, c = e % NX;
      Qii[e] = W2[e] = W2[NN + e] = 0.0;  // Q_0, al_0, al_1
      Qii[NN + e] = (double)Qm[r <= c ? e : c * NX + r];
      W1[e] = eye;
      W1[NN + e] = eye + a;
      put(lay.A + e, a);
      put(lay.Q + e, (double)Qm[e]);
    }
    __syncthreads();
    step_tables4<T, NX, NY>(L, lay, cst, cst64, sC, Apow, Qii, W1, W2, ci);
    __syncthreads();
  } else {
    __syncthreads();
    // A^i by doubling: A^i = A^s A^{i-s} for i in (s, 2s].
    for (int s = 1; s < L; s *= 2) {
      const int hi = (2 * s < L) ? 2 * s : L;
      for (int e = tid; e < (hi - s) * NN; e += nthr) {
        const int i = s + 1 + e / NN, rc = e % NN, r = rc / NX, c = rc % NX;
        double acc = 0.0;
        for (int k = 0; k < NX; ++k) acc += Apow[s * NN + r * NX + k] * Apow[(i - s) * NN + k * NX + c];
        Apow[i * NN + rc] = acc;
      }
      __syncthreads();
    }
    // W2[t] = A^t Q A^tT, t = 0..L-1: one entry of the upper triangle per item, mirrored, so that
    // every sum of these blocks is exactly symmetric.
    for (int e = tid; e < L * NN; e += nthr) {
      const int t = e / NN, rc = e % NN, r = rc / NX, c = rc % NX;
      if (c < r) continue;
      const double* At = Apow + t * NN;
      double acc = 0.0;
      for (int k = 0; k < NX; ++k) {
        double aq = 0.0;
        for (int j = 0; j < NX; ++j) aq += At[r * NX + j] * sQ[j * NX + k];
        acc += aq * At[c * NX + k];
      }
      W2[t * NN + r * NX + c] = acc;
      W2[t * NN + c * NX + r] = acc;
    }
    __syncthreads();
    // Q_ii = sum_{t<i} W2[t] (Qii[0] = 0) and W1[s] = Sig_s = sum_{u=0}^{s} A^u. Item (i, rc) forms
    // entry rc of Q_{i+1,i+1} (i < l) and of Sig_i, each as four independent partial sums (a
    // running sum would chain one LDS round trip per term).
    auto sum_blocks = [&](const double* src, int n, int rc) {
      double a0 = 0.0, a1 = 0.0, a2 = 0.0, a3 = 0.0;
      int t = 0;
      for (; t + 4 <= n; t += 4) {
        a0 += src[t * NN + rc];
        a1 += src[(t + 1) * NN + rc];
        a2 += src[(t + 2) * NN + rc];
        a3 += src[(t + 3) * NN + rc];
      }
      for (; t < n; ++t) a0 += src[t * NN + rc];
      return (a0 + a1) + (a2 + a3);
    };
    for (int e = tid; e < (L + 1) * NN; e += nthr) {
      const int i = e / NN, rc = e % NN;
      if (i < L) Qii[(i + 1) * NN + rc] = sum_blocks(W2, i + 1, rc);
      if (i == 0) Qii[rc] = 0.0;
      W1[i * NN + rc] = sum_blocks(Apow, i + 1, rc);
    }
    __syncthreads();
    // CS[s] = C Sig_s (NY x NX) in W2[0 ..], QC[j] = Q_jj C^T (NX x NY) in W2[(L+1) NXY ..]; beside
    // them the per-step tables go to the constants block: A^i, Q_ii, Q_il = Q_ii (A^{l-i})^T, and
    // A, Q. Every entry of the model part (below the level tables) also goes, unrounded, to the
    // float64 copy.
    double* CS = W2;
    double* QC = W2 + (L + 1) * NXY;
    for (int e = tid; e < (L + 1) * NXY + (L + 1) * NN; e += nthr) {
      if (e < (L + 1) * NXY) {
        const int s = e / NXY, rc = e % NXY;
        {
          const int r = rc / NX, c = rc % NX;  // CS: NY x NX
          double acc = 0.0;
          for (int k = 0; k < NX; ++k) acc += sC[r * NX + k] * W1[s * NN + k * NX + c];
          CS[s * NXY + rc] = acc;
        }
        {
          const int r = rc / NY, c = rc % NY;  // QC: NX x NY
          double acc = 0.0;
          for (int k = 0; k < NX; ++k) acc += Qii[s * NN + r * NX + k] * sC[c * NX + k];
          QC[s * NXY + rc] = acc;
        }
      } else if (e < (L + 1) * NXY + L * NN) {
        const int e2 = e - (L + 1) * NXY;
        const int i = 1 + e2 / NN, rc = e2 % NN, r = rc / NX, c = rc % NX;
        const int base = lay.per_i + (i - 1) * lay.per_i_stride;
        put(base + lay.o_Ai + rc, Apow[i * NN + rc]);
        put(base + lay.o_Qii + rc, Qii[i * NN + rc]);
        double acc = 0.0;
        for (int k = 0; k < NX; ++k) acc += Qii[i * NN + r * NX + k] * Apow[(L - i) * NN + c * NX + k];
        put(base + lay.o_QiL + rc, acc);
      } else {
        const int q = e - (L + 1) * NXY - L * NN;
        put(lay.A + q, sA[q]);
        put(lay.Q + q, sQ[q]);
      }
    }
    __syncthreads();
    // c_i = (1/l) [ sum_{j<i} A^{i-j} Q_jj C^T + Q_ii (C Sig_{l-i})^T ], the sum over j as four
    // independent partial sums.
    for (int e = tid; e < L * NXY; e += nthr) {
      const int i = 1 + e / NXY, rc = e % NXY, r = rc / NY, c = rc % NY;
      double a0 = 0.0, a1 = 0.0, a2 = 0.0, a3 = 0.0;
      for (int k = 0; k < NX; ++k) a0 += Qii[i * NN + r * NX + k] * CS[(L - i) * NXY + c * NX + k];
      int j = 1;
      for (; j + 4 <= i; j += 4)
        for (int k = 0; k < NX; ++k) {
          a0 += Apow[(i - j) * NN + r * NX + k] * QC[j * NXY + k * NY + c];
          a1 += Apow[(i - j - 1) * NN + r * NX + k] * QC[(j + 1) * NXY + k * NY + c];
          a2 += Apow[(i - j - 2) * NN + r * NX + k] * QC[(j + 2) * NXY + k * NY + c];
          a3 += Apow[(i - j - 3) * NN + r * NX + k] * QC[(j + 3) * NXY + k * NY + c];
        }
      for (; j < i; ++j)
        for (int k = 0; k < NX; ++k) a0 += Apow[(i - j) * NN + r * NX + k] * QC[j * NXY + k * NY + c];
      ci[i * NXY + rc] = ((a0 + a1) + (a2 + a3)) / (double)L;
    }
    __syncthreads();
  }

  // c_i to the constants block (nx > 4); C_bar = (C/l)(Sig_l - I) and R_x = (1/l) sum_i C c_i + R into LDS (W2 is
  // free again), an entry of R_x per wave with its sum over (i, k) spread over the lanes.
  double* sCbar = W2;
  double* sRx = W2 + NXY;
  const int nci = NX <= 4 ? 0 : L * NXY;
  for (int e = tid; e < nci + NXY; e += nthr) {
    if (e < nci) {
      const int i = 1 + e / NXY, rc = e % NXY;
      put(lay.per_i + (i - 1) * lay.per_i_stride + lay.o_ci + rc, ci[i * NXY + rc]);
    } else {
      const int q = e - nci, r = q / NX, c = q % NX;
      double acc = 0.0;
      for (int k = 0; k < NX; ++k) acc += sC[r * NX + k] * (W1[L * NN + k * NX + c] - (k == c ? 1.0 : 0.0));
      sCbar[q] = acc / (double)L;
    }
  }
  for (int q = tid >> 6; q < NY * NY; q += nthr >> 6) {
    const int r = q / NY, c = q % NY;
    double acc = 0.0;
    for (int t = tid & 63; t < L * NX; t += 64) acc += sC[r * NX + t % NX] * ci[NXY + t * NY + c];
    acc = wave_sum(acc);
    if ((tid & 63) == 0) sRx[q] = acc / (double)L + sR[q];
  }
  __syncthreads();
  if (tid >= 64) return;  // the rest is done by wave 0
  int lflag = 0;
  double* rec = chain;  // the chain's F, D, J of Theta(1): the generic element
  {
    // ------------------------------------------------------------ generic element (wave 0)
    // Every lane inverts R_x itself; lane e < nx^2 forms entry e of F, D and J (D and J from
    // both halves, symmetrised), and the first lanes write C_bar, R_x, K and H_eta.
    //   K = S_xy R_x^{-1},  H_eta = C_bar^T R_x^{-1},  F = A^l - K C_bar,
    //   D = Q_ll - K S_xy^T,  J = H_eta C_bar,  with S_xy = c_l.
    double Rx[NY][NY], Rxi[NY][NY];
    for (int r = 0; r < NY; ++r)
      for (int c = 0; c < NY; ++c) Rx[r][c] = sRx[r * NY + c];
    symmetrize(Rx);
    if (!spd_inv(Rx, Rxi) && tid == 0) lflag |= SRTM_INFO_INNOVATION_NOT_PD;
    const double* Sxy = ci + L * NXY;  // NX x NY
    auto krow = [&](int r, double (&o)[NY]) {  // row r of K
#pragma unroll
      for (int k = 0; k < NY; ++k) {
        double s = 0.0;
#pragma unroll
        for (int j = 0; j < NY; ++j) s += Sxy[r * NY + j] * Rxi[j][k];
        o[k] = s;
      }
    };
    auto hrow = [&](int r, double (&o)[NY]) {  // row r of H_eta
#pragma unroll
      for (int k = 0; k < NY; ++k) {
        double s = 0.0;
#pragma unroll
        for (int j = 0; j < NY; ++j) s += sCbar[j * NX + r] * Rxi[j][k];
        o[k] = s;
      }
    };
    if (tid < NN) {
      const int r = tid / NX, c = tid % NX;
      double Kr[NY], Kc[NY], Hr[NY], Hc[NY];
      krow(r, Kr);
      krow(c, Kc);
      hrow(r, Hr);
      hrow(c, Hc);
      double f = Apow[L * NN + tid], drc = Qii[L * NN + r * NX + c], dcr = Qii[L * NN + c * NX + r];
      double jrc = 0.0, jcr = 0.0;
#pragma unroll
      for (int k = 0; k < NY; ++k) {
        f -= Kr[k] * sCbar[k * NX + c];
        drc -= Kr[k] * Sxy[c * NY + k];
        dcr -= Kc[k] * Sxy[r * NY + k];
        jrc += Hr[k] * sCbar[k * NX + c];
        jcr += Hc[k] * sCbar[k * NX + r];
      }
      rec[tid] = f;
      rec[NN + tid] = (r == c) ? drc : 0.5 * (drc + dcr);
      rec[2 * NN + tid] = (r == c) ? jrc : 0.5 * (jrc + jcr);
    }
    if (tid < NX) {
      double Kr[NY], Hr[NY];
      krow(tid, Kr);
      hrow(tid, Hr);
#pragma unroll
      for (int k = 0; k < NY; ++k) {
        put(lay.K + tid * NY + k, Kr[k]);
        put(lay.Heta + tid * NY + k, Hr[k]);
      }
    }
    for (int q = tid; q < NXY; q += 64) put(lay.Cbar + q, sCbar[q]);
    for (int q = tid; q < NY * NY; q += 64) {
      const int r = q / NY, c = q % NY;
      put(lay.Rx + q, (r == c) ? sRx[q] : 0.5 * (sRx[r * NY + c] + sRx[c * NY + r]));
    }
  }
  wave_sync();
  // Levels below CHAIN_SPLIT; the others continue in the tile-reduction launch.
  const int p1 = nlev < CHAIN_SPLIT ? nlev : CHAIN_SPLIT;
  lflag |= level_chain<T, NX>(chain, cst, lay, 0, p1, nlev, hand, lev64);
  if (lflag && info) atomicOr(info, lflag);
}

// ============================================================================ helpers
// Known inputs of a call (all null and nu = 0 without inputs).
template <typename T>
struct InputView {
  const T* B;  // [nx][nu]
  const T* u;  // [N][l][nu], u[k-1][i-1] drives x_{k,i}
  const T* H;  // [ny][nx], the measurement matrix C
  T* rec;      // workspace [N][ny + nx]: y_k - mu_k and z_{k,l}, written by the tile reductions
  int nu;
};

// A call's constants block (time-invariant model).
template <typename T, int NX, int NY>
struct Model {
  const T* __restrict__ cst;
  ConstLayout lay;
  InputView<T> in{};
  SRTM_DEV const T* per_i(int i) const { return cst + lay.per_i + (i - 1) * lay.per_i_stride; }
  SRTM_DEV int per_i_off(int i) const { return lay.per_i + (i - 1) * lay.per_i_stride; }
  SRTM_DEV const T* level(int p) const { return cst + lay.lev + p * lay.lev_stride; }
  SRTM_DEV int AL_off(int L) const { return per_i_off(L) + lay.o_Ai; }  // A^l
  SRTM_DEV int cL_off(int L) const { return per_i_off(L) + lay.o_ci; }  // c_l
  template <int R, int C>
  SRTM_DEV void get(T (&a)[R][C], int off) const { load(a, cst + off); }
  SRTM_DEV T at(int off) const { return cst[off]; }
};

// Per-window blocks and element records are stored tile by tile, window-minor within a tile:
// scalar j of window k at base[(k / TILE) * width * TILE + j * TILE + k % TILE] for records of
// `width` scalars, so that the lanes of a wave read and write consecutive addresses and one
// tile's records stay within width * TILE scalars. Returns window k's column (stride TILE).
template <typename T>
SRTM_DEV T* tv_column(T* base, int64_t k, int width) {
  return base + (k / TILE) * (int64_t)width * TILE + (k % TILE);
}
// The block of columns of window k's tile (tv_column minus the column).
template <typename T>
SRTM_DEV T* tv_tile_base(T* base, int64_t k, int width) {
  return base + (k / TILE) * (int64_t)width * TILE;
}

// One window of a per-window model: its constants block (TvLayout, one column of its tile's
// block of columns at `blk`: the row base blk + off * TILE is the same for every lane of a
// workgroup and each lane adds its column) and its own A, Q and C, entry j at A[j * ms]: the
// caller's row-major arrays (LDSM false, ms = 1) or a window-minor copy in LDS (LDSM, ms the
// copy's column count).
template <typename T, int NX, int NY, bool LDSM = false>
struct TvModel {
  const T* __restrict__ blk;
  TvLayout lay;
  int lane;
  const T* __restrict__ A;
  const T* __restrict__ Q;
  const T* __restrict__ C;
  int ms = 1;
  SRTM_DEV T mdl(const T* p, int j) const { return LDSM ? sld(p + j * ms) : gld(p + j * ms); }
  SRTM_DEV int AL_off(int) const { return lay.AL; }
  SRTM_DEV int cL_off(int) const { return lay.cL; }
  SRTM_DEV int slot_off(int q) const { return lay.slot + q * lay.slot_stride; }
  template <int R, int CC>
  SRTM_DEV void get(T (&a)[R][CC], int off) const {
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
      for (int c = 0; c < CC; ++c) a[r][c] = at(off + r * CC + c);
  }
  SRTM_DEV T at(int off) const { return gld(blk + (int64_t)off * TILE + lane); }
};

template <typename T, int N>
SRTM_DEV T symget(const T (&P)[N][N], int r, int c) { return r <= c ? P[r][c] : P[c][r]; }

// state (m, P) (x) segment (F, d, D, eta, J): the eq. op-filter combination whose left
// operand holds the prior (F = 0):  W = (I + P J)^{-1},
//   m' = F W (m + P eta) + d,   P' = F W P F^T + D   (W P is symmetric; its upper triangle is used).
template <typename T, int NX>
SRTM_DEV bool state_combine(T (&m)[NX], T (&P)[NX][NX], const T (&F)[NX][NX], const T (&d)[NX],
                            const T (&D)[NX][NX], const T (&eta)[NX], const T (&J)[NX][NX]) {
  T M[NX][NX], W[NX][NX];
  mm(P, J, M);
#pragma unroll
  for (int r = 0; r < NX; ++r) M[r][r] += T(1);
  const bool ok = inv_small(M, W);
  T u[NX], Wu[NX], WP[NX][NX];
#pragma unroll
  for (int r = 0; r < NX; ++r) {
    T t = m[r];
#pragma unroll
    for (int k = 0; k < NX; ++k) t = my_fma(P[r][k], eta[k], t);
    u[r] = t;
  }
  mv(W, u, Wu);
#pragma unroll
  for (int r = 0; r < NX; ++r)
#pragma unroll
    for (int c = r; c < NX; ++c) {
      T t = T(0);
#pragma unroll
      for (int k = 0; k < NX; ++k) t = my_fma(W[r][k], P[k][c], t);
      WP[r][c] = t;
      WP[c][r] = t;
    }
#pragma unroll
  for (int r = 0; r < NX; ++r) {
    T t = d[r];
#pragma unroll
    for (int k = 0; k < NX; ++k) t = my_fma(F[r][k], Wu[k], t);
    m[r] = t;
  }
  sandwich(F, WP, D, P);
  return ok;
}

// Full filter element and a_i (x) a_j of eq. op-filter, with W = (I + D_i J_j)^{-1} and
// (I + J_j D_i)^{-1} = W^T (D, J symmetric):
//   F = F_j W F_i, d = F_j W (d_i + D_i eta_j) + d_j, D = F_j W D_i F_j^T + D_j,
//   eta = (W F_i)^T (eta_j - J_j d_i) + eta_i,  J = (W F_i)^T J_j F_i + J_i.
template <typename T, int NX>
struct FElem {
  T F[NX][NX], d[NX], D[NX][NX], e[NX], J[NX][NX];
};

template <typename T, int NX>
SRTM_DEV bool elem_combine(const FElem<T, NX>& a, const FElem<T, NX>& b, FElem<T, NX>& o) {
  T M[NX][NX], W[NX][NX];
  mm(a.D, b.J, M);
#pragma unroll
  for (int r = 0; r < NX; ++r) M[r][r] += T(1);
  const bool ok = inv_small(M, W);
  T XF[NX][NX], u[NX], Xu[NX], XD[NX][NX];
  mm(W, a.F, XF);
#pragma unroll
  for (int r = 0; r < NX; ++r) {
    T t = a.d[r];
#pragma unroll
    for (int k = 0; k < NX; ++k) t = my_fma(a.D[r][k], b.e[k], t);
    u[r] = t;
  }
  mv(W, u, Xu);
#pragma unroll
  for (int r = 0; r < NX; ++r)
#pragma unroll
    for (int c = r; c < NX; ++c) {
      T t = T(0);
#pragma unroll
      for (int k = 0; k < NX; ++k) t = my_fma(W[r][k], a.D[k][c], t);
      XD[r][c] = t;
      XD[c][r] = t;
    }
  FElem<T, NX> t;
  mm(b.F, XF, t.F);
#pragma unroll
  for (int r = 0; r < NX; ++r) {
    T q = b.d[r];
#pragma unroll
    for (int k = 0; k < NX; ++k) q = my_fma(b.F[r][k], Xu[k], q);
    t.d[r] = q;
  }
  sandwich(b.F, XD, b.D, t.D);
  T vv[NX], JF[NX][NX];
#pragma unroll
  for (int r = 0; r < NX; ++r) {
    T q = b.e[r];
#pragma unroll
    for (int k = 0; k < NX; ++k) q = my_fma(-b.J[r][k], a.d[k], q);
    vv[r] = q;
  }
  mm(b.J, a.F, JF);
#pragma unroll
  for (int r = 0; r < NX; ++r) {
    T q = a.e[r];
#pragma unroll
    for (int k = 0; k < NX; ++k) q = my_fma(XF[k][r], vv[k], q);
    t.e[r] = q;
#pragma unroll
    for (int c = r; c < NX; ++c) {
      T sj = a.J[r][c];
#pragma unroll
      for (int k = 0; k < NX; ++k) sj = my_fma(XF[k][r], JF[k][c], sj);
      t.J[r][c] = sj;
      t.J[c][r] = sj;
    }
  }
  o = t;
  return ok;
}

template <typename T, int NX>
SRTM_DEV void elem_identity(FElem<T, NX>& a) {
#pragma unroll
  for (int r = 0; r < NX; ++r) {
    a.d[r] = T(0);
    a.e[r] = T(0);
#pragma unroll
    for (int c = 0; c < NX; ++c) {
      a.F[r][c] = (r == c) ? T(1) : T(0);
      a.D[r][c] = T(0);
      a.J[r][c] = T(0);
    }
  }
}

// Smoother element (E, g, S) and eq. op-smoother: for a (earlier) and b (later),
//   E = E_a E_b, g = E_a g_b + g_a, S = E_a S_b E_a^T + S_a.
template <typename T, int NX>
struct SElem {
  T E[NX][NX], g[NX], S[NX][NX];
};

template <typename T, int NX>
SRTM_DEV void selem_combine(const SElem<T, NX>& a, const SElem<T, NX>& b, SElem<T, NX>& o) {
  SElem<T, NX> t;
  mm(a.E, b.E, t.E);
  T ES[NX][NX];
  mm(a.E, b.S, ES);
#pragma unroll
  for (int r = 0; r < NX; ++r) {
    T s = a.g[r];
#pragma unroll
    for (int k = 0; k < NX; ++k) s = my_fma(a.E[r][k], b.g[k], s);
    t.g[r] = s;
#pragma unroll
    for (int c = r; c < NX; ++c) {
      T q = a.S[r][c];
#pragma unroll
      for (int k = 0; k < NX; ++k) q = my_fma(ES[r][k], a.E[c][k], q);
      t.S[r][c] = q;
      t.S[c][r] = q;
    }
  }
  o = t;
}

// segment (E, g, S) applied to the smoothed state after it: m' = E m + g, P' = E P E^T + S.
template <typename T, int NX>
SRTM_DEV void sstate_combine(const SElem<T, NX>& a, T (&m)[NX], T (&P)[NX][NX]) {
  T EP[NX][NX], mn[NX];
  mm(a.E, P, EP);
#pragma unroll
  for (int r = 0; r < NX; ++r) {
    T s = a.g[r];
#pragma unroll
    for (int k = 0; k < NX; ++k) s = my_fma(a.E[r][k], m[k], s);
    mn[r] = s;
  }
#pragma unroll
  for (int r = 0; r < NX; ++r) {
    m[r] = mn[r];
#pragma unroll
    for (int c = r; c < NX; ++c) {
      T q = a.S[r][c];
#pragma unroll
      for (int k = 0; k < NX; ++k) q = my_fma(EP[r][k], a.E[c][k], q);
      P[r][c] = q;
      P[c][r] = q;
    }
  }
}

// ---------------------------------------------------------------- LDS slot storage (SoA)
template <typename T>
struct Slots {
  T* base;
  int n;  // slots per field row
  SRTM_DEV T& at(int f, int s) const { return base[f * n + s]; }
};

template <typename T, int NX>
SRTM_DEV void st_state(const Slots<T>& S, int s, const T (&m)[NX], const T (&P)[NX][NX]) {
#pragma unroll
  for (int r = 0; r < NX; ++r) S.at(r, s) = m[r];
#pragma unroll
  for (int r = 0; r < NX; ++r)
#pragma unroll
    for (int c = r; c < NX; ++c) S.at(NX + r * NX + c, s) = P[r][c];
}
template <typename T, int NX>
SRTM_DEV void ld_state(const Slots<T>& S, int s, T (&m)[NX], T (&P)[NX][NX]) {
#pragma unroll
  for (int r = 0; r < NX; ++r) m[r] = S.at(r, s);
#pragma unroll
  for (int r = 0; r < NX; ++r)
#pragma unroll
    for (int c = r; c < NX; ++c) {
      P[r][c] = S.at(NX + r * NX + c, s);
      P[c][r] = P[r][c];
    }
}
template <typename T, int NX>
SRTM_DEV void st_felem(const Slots<T>& S, int s, const FElem<T, NX>& a) {
  constexpr int NN = NX * NX;
#pragma unroll
  for (int r = 0; r < NX; ++r) {
    S.at(NN + r, s) = a.d[r];
    S.at(2 * NN + NX + r, s) = a.e[r];
#pragma unroll
    for (int c = 0; c < NX; ++c) {
      S.at(r * NX + c, s) = a.F[r][c];
      S.at(NN + NX + r * NX + c, s) = a.D[r][c];
      S.at(2 * NN + 2 * NX + r * NX + c, s) = a.J[r][c];
    }
  }
}
template <typename T, int NX>
SRTM_DEV void ld_felem(const Slots<T>& S, int s, FElem<T, NX>& a) {
  constexpr int NN = NX * NX;
#pragma unroll
  for (int r = 0; r < NX; ++r) {
    a.d[r] = S.at(NN + r, s);
    a.e[r] = S.at(2 * NN + NX + r, s);
#pragma unroll
    for (int c = 0; c < NX; ++c) {
      a.F[r][c] = S.at(r * NX + c, s);
      a.D[r][c] = S.at(NN + NX + r * NX + c, s);
      a.J[r][c] = S.at(2 * NN + 2 * NX + r * NX + c, s);
    }
  }
}
template <typename T, int NX>
SRTM_DEV void st_selem(const Slots<T>& S, int s, const SElem<T, NX>& a) {
  constexpr int NN = NX * NX;
#pragma unroll
  for (int r = 0; r < NX; ++r) {
    S.at(NN + r, s) = a.g[r];
#pragma unroll
    for (int c = 0; c < NX; ++c) {
      S.at(r * NX + c, s) = a.E[r][c];
      S.at(NN + NX + r * NX + c, s) = a.S[r][c];
    }
  }
}
template <typename T, int NX>
SRTM_DEV void ld_selem(const Slots<T>& S, int s, SElem<T, NX>& a) {
  constexpr int NN = NX * NX;
#pragma unroll
  for (int r = 0; r < NX; ++r) {
    a.g[r] = S.at(NN + r, s);
#pragma unroll
    for (int c = 0; c < NX; ++c) {
      a.E[r][c] = S.at(r * NX + c, s);
      a.S[r][c] = S.at(NN + NX + r * NX + c, s);
    }
  }
}

// x <- x (x) b under eq. op-smoother, where b is the element of lane l + d (DOWN) or l - d of the
// same wave, when `take`; otherwise x is left as it is. Every lane takes part in the exchange.
// The partner's E and S arrive column by column and are consumed at once, so that only a few
// exchanged values are live (the products are those of selem_combine, in its order).
template <bool DOWN, typename T, int NX>
SRTM_DEV void selem_merge_lane(SElem<T, NX>& x, int d, bool take) {
  auto mv = [&](T v) { return DOWN ? __shfl_down(v, (unsigned)d, 64) : __shfl_up(v, (unsigned)d, 64); };
  T tE[NX][NX], ES[NX][NX], tg[NX];
#pragma unroll
  for (int c = 0; c < NX; ++c) {
    T be[NX], bs[NX];
#pragma unroll
    for (int k = 0; k < NX; ++k) {
      be[k] = mv(x.E[k][c]);
      bs[k] = mv(x.S[k][c]);
    }
#pragma unroll
    for (int r = 0; r < NX; ++r) {
      T e = x.E[r][0] * be[0], q = x.E[r][0] * bs[0];
#pragma unroll
      for (int k = 1; k < NX; ++k) {
        e = my_fma(x.E[r][k], be[k], e);
        q = my_fma(x.E[r][k], bs[k], q);
      }
      tE[r][c] = e;
      ES[r][c] = q;
    }
  }
  {
    T bg[NX];
#pragma unroll
    for (int k = 0; k < NX; ++k) bg[k] = mv(x.g[k]);
#pragma unroll
    for (int r = 0; r < NX; ++r) {
      T t = x.g[r];
#pragma unroll
      for (int k = 0; k < NX; ++k) t = my_fma(x.E[r][k], bg[k], t);
      tg[r] = t;
    }
  }
  if (take) {
#pragma unroll
    for (int r = 0; r < NX; ++r)
#pragma unroll
      for (int c = r; c < NX; ++c) {
        T q = x.S[r][c];
#pragma unroll
        for (int k = 0; k < NX; ++k) q = my_fma(ES[r][k], x.E[c][k], q);
        x.S[r][c] = q;
        x.S[c][r] = q;
      }
#pragma unroll
    for (int r = 0; r < NX; ++r) {
      x.g[r] = tg[r];
#pragma unroll
      for (int c = 0; c < NX; ++c) x.E[r][c] = tE[r][c];
    }
  }
}

// ---------------------------------------------------------------- per-window quantities
// Window k with prior (m, P) = (m^f_{k-1,l}, P^f_{k-1,l}) and measurement y_k. With
// V = P C_bar^T, S = C_bar V + R_x, U_i = A^i V + c_i = Cov(x_{k,i}, y_k | y_{1:k-1}):
//   m^f_{k,i} = A^i m + U_i S^{-1} e,   e = y_k - C_bar m,
//   P^f_{k,i,i} = A^i P A^{iT} + Q_ii - U_i S^{-1} U_i^T,
//   P^f_{k,i,l} = A^i P A^{lT} + Q_il - U_i S^{-1} U_l^T          (eq. update-fast, blockwise).
template <typename T, int NX, int NY>
struct Window {
  T m[NX];         // prior mean (of x_{k,0})
  T mp[NX];        // m' = m + V S^{-1} e      ->  m^f_i = A^i m' + c_i Se
  T Se[NY];        // S^{-1} e
  T P[NX][NX];     // prior covariance (symmetric)
  T V[NX][NY];     // P C_bar^T
  T Si[NY][NY];    // S^{-1} (symmetric)
  T Y1[NX][NX];    // P A^{lT} - V Y2      ->  P^f_{i,l} = A^i Y1 + Q_il - c_i Y2
  T Y2[NY][NX];    // S^{-1} U_l^T
};

// MV: Model (one constants block) or TvModel (the window's own block).
template <typename T, int NX, int NY, class MV>
SRTM_DEV bool window_setup(const MV& M, int L, const T (&m)[NX], const T (&P)[NX][NX],
                           const T (&yk)[NY], Window<T, NX, NY>& w) {
  T Cb[NY][NX], Rx[NY][NY];
  M.get(Cb, M.lay.Cbar);
  M.get(Rx, M.lay.Rx);
#pragma unroll
  for (int r = 0; r < NX; ++r)
#pragma unroll
    for (int c = 0; c < NX; ++c) w.P[r][c] = P[r][c];
  mm_nt(P, Cb, w.V);
  T S[NY][NY];
  mm(Cb, w.V, S);
#pragma unroll
  for (int r = 0; r < NY; ++r)
#pragma unroll
    for (int c = 0; c < NY; ++c) S[r][c] += Rx[r][c];
  symmetrize(S);
  const bool ok = spd_inv(S, w.Si);
  T e[NY];
#pragma unroll
  for (int r = 0; r < NY; ++r) {
    T s = yk[r];
#pragma unroll
    for (int k = 0; k < NX; ++k) s = my_fma(-Cb[r][k], m[k], s);
    e[r] = s;
  }
  mv(w.Si, e, w.Se);
#pragma unroll
  for (int r = 0; r < NX; ++r) {
    w.m[r] = m[r];
    T s = m[r];
#pragma unroll
    for (int k = 0; k < NY; ++k) s = my_fma(w.V[r][k], w.Se[k], s);
    w.mp[r] = s;
  }
  // U_l = A^l V + c_l, Y2 = S^{-1} U_l^T, Y1 = P A^{lT} - V Y2
  T AL[NX][NX], cL[NX][NY];
  M.get(AL, M.AL_off(L));
  M.get(cL, M.cL_off(L));
  T UL[NX][NY];
  mm(AL, w.V, UL);
#pragma unroll
  for (int r = 0; r < NX; ++r)
#pragma unroll
    for (int c = 0; c < NY; ++c) UL[r][c] += cL[r][c];
  mm_nt(w.Si, UL, w.Y2);
  T PAL[NX][NX];
  mm_nt(P, AL, PAL);
#pragma unroll
  for (int r = 0; r < NX; ++r)
#pragma unroll
    for (int c = 0; c < NX; ++c) {
      T s = PAL[r][c];
#pragma unroll
      for (int k = 0; k < NY; ++k) s = my_fma(-w.V[r][k], w.Y2[k][c], s);
      w.Y1[r][c] = s;
    }
  return ok;
}

// Filter blocks of fast step i: mean, P^f_{i,i} and (optionally) P^f_{i,l}, from the step's
// A^i and c_i and entries (r, c) of Q_ii and Q_il given by qii(r, c) and qil(r, c).
template <bool CROSS, typename T, int NX, int NY, class QII, class QIL>
SRTM_DEV void step_blocks(const Window<T, NX, NY>& w, const T (&Ai)[NX][NX], const T (&ci)[NX][NY], QII qii,
                          QIL qil, T (&mf)[NX], T (&Pii)[NX][NX], T (&PiL)[NX][NX]) {
  // mean
#pragma unroll
  for (int r = 0; r < NX; ++r) {
    T s = T(0);
#pragma unroll
    for (int k = 0; k < NX; ++k) s = my_fma(Ai[r][k], w.mp[k], s);
#pragma unroll
    for (int k = 0; k < NY; ++k) s = my_fma(ci[r][k], w.Se[k], s);
    mf[r] = s;
  }
  // U_i = A^i V + c_i ; US = U_i S^{-1}
  T U[NX][NY], US[NX][NY];
  mm(Ai, w.V, U);
#pragma unroll
  for (int r = 0; r < NX; ++r)
#pragma unroll
    for (int c = 0; c < NY; ++c) U[r][c] += ci[r][c];
#pragma unroll
  for (int r = 0; r < NX; ++r)
#pragma unroll
    for (int c = 0; c < NY; ++c) {
      T s = T(0);
#pragma unroll
      for (int k = 0; k < NY; ++k) s = my_fma(U[r][k], symget(w.Si, k, c), s);
      US[r][c] = s;
    }
  // P^f_{i,i} = (A^i P) A^{iT} + Q_ii - US U^T  (upper triangle, mirrored)
#pragma unroll
  for (int r = 0; r < NX; ++r) {
    T AP[NX];
#pragma unroll
    for (int c = 0; c < NX; ++c) {
      T s = T(0);
#pragma unroll
      for (int k = 0; k < NX; ++k) s = my_fma(Ai[r][k], symget(w.P, k, c), s);
      AP[c] = s;
    }
#pragma unroll
    for (int c = r; c < NX; ++c) {
      T s = qii(r, c);
#pragma unroll
      for (int k = 0; k < NX; ++k) s = my_fma(AP[k], Ai[c][k], s);
#pragma unroll
      for (int k = 0; k < NY; ++k) s = my_fma(-US[r][k], U[c][k], s);
      Pii[r][c] = s;
      Pii[c][r] = s;
    }
  }
  if (CROSS) {
    // P^f_{i,l} = A^i Y1 + Q_il - c_i Y2
#pragma unroll
    for (int r = 0; r < NX; ++r)
#pragma unroll
      for (int c = 0; c < NX; ++c) {
        T s = qil(r, c);
#pragma unroll
        for (int k = 0; k < NX; ++k) s = my_fma(Ai[r][k], w.Y1[k][c], s);
#pragma unroll
        for (int k = 0; k < NY; ++k) s = my_fma(-ci[r][k], w.Y2[k][c], s);
        PiL[r][c] = s;
      }
  }
}

// Time-invariant model: the step's tables from the constants block (wave-uniform loads).
template <typename T, int NX, int NY, bool CROSS>
SRTM_DEV void window_step(const Model<T, NX, NY>& M, const Window<T, NX, NY>& w, int i, T (&mf)[NX],
                          T (&Pii)[NX][NX], T (&PiL)[NX][NX]) {
  const int po = M.per_i_off(i);
  T Ai[NX][NX], ci[NX][NY];
  M.get(Ai, po + M.lay.o_Ai);
  M.get(ci, po + M.lay.o_ci);
  step_blocks<CROSS>(
      w, Ai, ci, [&](int r, int c) { return M.at(po + M.lay.o_Qii + r * NX + c); },
      [&](int r, int c) { return M.at(po + M.lay.o_QiL + r * NX + c); }, mf, Pii, PiL);
}

// Per-window model: the fast steps of window k in order, in the prior-inclusive form. With the
// window's prior (m, P) of x_{k,0} and Sig_i = Cov(x_{k,i} | y_{1:k-1}) = A^i P A^{iT} + Q_ii,
//   Sig_i = A Sig_{i-1} A^T + Q (Sig_0 = P),  mu_i = A mu_{i-1} (mu_0 = m),
//   al_i = A (al_{i-1} + Sig_{i-1} C^T) (al_1 = 0),
//   U_i = Cov(x_{k,i}, y_k | y_{1:k-1}) = (1/l) [al_i + Sig_i (C Sig_{l-i})^T],
//   m^f_{k,i} = mu_i + U_i S^{-1} e,  P^f_{k,i,i} = Sig_i - U_i S^{-1} U_i^T,
//   P^f_{k,i,l} = Sig_i (A^{l-i})^T - U_i S^{-1} U_l^T
// (the same blocks as step_blocks: A^i P A^{lT} + Q_il = Sig_i (A^{l-i})^T), from the window's own
// A, Q and C and the backward factors A^s and C Sig_s (s = l - i) of its block, stored for even s
// (TvLayout): a step with odd s forms them from the slot it shares with step i + 1.
template <typename T, int NX, int NY>
struct TvSteps {
  T Sg[NX][NX], al[NX][NY], mu[NX];  // Sg: upper triangle only
  T fCS[NY][NX], fAs[NX][NX];        // the factors of the slot in use: C Sig_{2q}, A^{2q}
  int i = 0;  // the last step formed
  template <bool CROSS, bool LDSM>
  SRTM_DEV void next(const TvModel<T, NX, NY, LDSM>& M, int L, const Window<T, NX, NY>& w, T (&mf)[NX],
                     T (&Pii)[NX][NX], T (&PiL)[NX][NX]) {
    const int s = L - (i + 1);
    if (i == 0 || (s & 1)) {  // the first step, or the first of the two steps of slot s / 2
      const int so = M.slot_off(s >> 1);
      M.get(fCS, so + M.lay.o_CS);
      M.get(fAs, so + M.lay.o_As);
    }
    T CS[NY][NX], As[NX][NX], A[NX][NX], C[NY][NX];
#pragma unroll
    for (int r = 0; r < NX; ++r) {
#pragma unroll
      for (int c = 0; c < NX; ++c) A[r][c] = M.mdl(M.A, r * NX + c);
    }
#pragma unroll
    for (int r = 0; r < NY; ++r) {
#pragma unroll
      for (int c = 0; c < NX; ++c) C[r][c] = M.mdl(M.C, r * NX + c);
    }
    if (s & 1) {  // A^s = A A^{s-1},  C Sig_s = C Sig_{s-1} + C A^s
      mm(A, fAs, As);
#pragma unroll
      for (int r = 0; r < NY; ++r)
#pragma unroll
        for (int c = 0; c < NX; ++c) {
          T v = fCS[r][c];
#pragma unroll
          for (int q = 0; q < NX; ++q) v = my_fma(C[r][q], As[q][c], v);
          CS[r][c] = v;
        }
    } else {
#pragma unroll
      for (int r = 0; r < NX; ++r) {
#pragma unroll
        for (int c = 0; c < NX; ++c) As[r][c] = fAs[r][c];
#pragma unroll
        for (int c = 0; c < NY; ++c) CS[c][r] = fCS[c][r];
      }
    }
    if (i == 0) {
#pragma unroll
      for (int r = 0; r < NX; ++r) {
        mu[r] = w.m[r];
#pragma unroll
        for (int c = r; c < NX; ++c) Sg[r][c] = w.P[r][c];
#pragma unroll
        for (int c = 0; c < NY; ++c) al[r][c] = T(0);
      }
    } else {
      T b[NX][NY];
#pragma unroll
      for (int r = 0; r < NX; ++r)
#pragma unroll
        for (int c = 0; c < NY; ++c) {
          T v = al[r][c];
#pragma unroll
          for (int q = 0; q < NX; ++q) v = my_fma(symget(Sg, r, q), C[c][q], v);
          b[r][c] = v;
        }
      mm(A, b, al);
    }
    {  // Sig_i = A Sig_{i-1} A^T + Q, mu_i = A mu_{i-1}
      T AS[NX][NX], nm[NX];
#pragma unroll
      for (int r = 0; r < NX; ++r) {
        T t = T(0);
#pragma unroll
        for (int q = 0; q < NX; ++q) t = my_fma(A[r][q], mu[q], t);
        nm[r] = t;
#pragma unroll
        for (int c = 0; c < NX; ++c) {
          T v = T(0);
#pragma unroll
          for (int q = 0; q < NX; ++q) v = my_fma(A[r][q], symget(Sg, q, c), v);
          AS[r][c] = v;
        }
      }
#pragma unroll
      for (int r = 0; r < NX; ++r) {
        mu[r] = nm[r];
#pragma unroll
        for (int c = r; c < NX; ++c) {
          T v = M.mdl(M.Q, r * NX + c);
#pragma unroll
          for (int q = 0; q < NX; ++q) v = my_fma(AS[r][q], A[c][q], v);
          Sg[r][c] = v;
        }
      }
    }
    ++i;
    // U = (1/l) (al + Sig C Sig_{l-i}^T),  US = U S^{-1}
    const T il = T(1) / T(L);
    T U[NX][NY], US[NX][NY];
#pragma unroll
    for (int r = 0; r < NX; ++r)
#pragma unroll
      for (int c = 0; c < NY; ++c) {
        T v = al[r][c];
#pragma unroll
        for (int q = 0; q < NX; ++q) v = my_fma(symget(Sg, r, q), CS[c][q], v);
        U[r][c] = v * il;
      }
#pragma unroll
    for (int r = 0; r < NX; ++r)
#pragma unroll
      for (int c = 0; c < NY; ++c) {
        T v = T(0);
#pragma unroll
        for (int q = 0; q < NY; ++q) v = my_fma(U[r][q], symget(w.Si, q, c), v);
        US[r][c] = v;
      }
#pragma unroll
    for (int r = 0; r < NX; ++r) {
      T v = mu[r];
#pragma unroll
      for (int q = 0; q < NY; ++q) v = my_fma(U[r][q], w.Se[q], v);
      mf[r] = v;
#pragma unroll
      for (int c = r; c < NX; ++c) {
        T t = Sg[r][c];
#pragma unroll
        for (int q = 0; q < NY; ++q) t = my_fma(-US[r][q], U[c][q], t);
        Pii[r][c] = t;
        Pii[c][r] = t;
      }
    }
    if (CROSS) {
#pragma unroll
      for (int r = 0; r < NX; ++r)
#pragma unroll
        for (int c = 0; c < NX; ++c) {
          T v = T(0);
#pragma unroll
          for (int q = 0; q < NX; ++q) v = my_fma(symget(Sg, r, q), As[c][q], v);
#pragma unroll
          for (int q = 0; q < NY; ++q) v = my_fma(-U[r][q], w.Y2[q][c], v);
          PiL[r][c] = v;
        }
    }
  }
};

// Blocks of fast step 1 (the smoother element's): from the constants block, or from the
// window's own model.
template <typename T, int NX, int NY>
SRTM_DEV void first_step(const Model<T, NX, NY>& M, int, const Window<T, NX, NY>& w, T (&mf)[NX], T (&Pii)[NX][NX],
                         T (&PiL)[NX][NX]) {
  window_step<T, NX, NY, true>(M, w, 1, mf, Pii, PiL);
}
template <typename T, int NX, int NY>
SRTM_DEV void first_step(const TvModel<T, NX, NY>& M, int L, const Window<T, NX, NY>& w, T (&mf)[NX],
                         T (&Pii)[NX][NX], T (&PiL)[NX][NX]) {
  TvSteps<T, NX, NY> st;
  st.template next<true, false>(M, L, w, mf, Pii, PiL);
}

template <typename T, int NX, int NY>
SRTM_DEV void load_prior(const T* __restrict__ carry, const T* __restrict__ m0, const T* __restrict__ P0,
                         int64_t k, T (&m)[NX], T (&P)[NX][NX]) {
  constexpr int ST = NX + NX * NX;
  if (k == 0) {
    gloadv(m, m0);
    gload(P, P0);
  } else {
    gloadv(m, carry + (k - 1) * ST);
    gload(P, carry + (k - 1) * ST + NX);
  }
}

// ---------------------------------------------------------------- known inputs
// With x_t = A x_{t-1} + B u_{t-1} + w_{t-1} (eq. original-linear-SSM), window k's own
// inputs add the deterministic response z_{k,i} = A z_{k,i-1} + B u_{k,i-1}, z_{k,0} = 0, to
// its fast states given x_{k-1,l}: in eq. h-k-l-2 B_bar u_bar_k = z_{k,l}, and in eq. y-k-l-2
// D_bar u_bar_k = mu_k = (C/l) sum_i z_{k,i}. Hence the filter element's d gains z_{k,l}, every
// innovation uses y_k - mu_k, m^f_{k,i} gains z_{k,i}, and the smoother's prediction of
// x_{k+1,1} gains B u_{k+1,0}. No covariance depends on the inputs.

// B u of one fast step (uk: that step's nu inputs).
template <typename T, int NX>
SRTM_DEV void input_drive(const InputView<T>& in, const T* __restrict__ uk, T (&bu)[NX]) {
#pragma unroll
  for (int r = 0; r < NX; ++r) bu[r] = T(0);
#pragma unroll
  for (int j = 0; j < NU_MAX; ++j) {
    if (j < in.nu) {
      const T uj = gld(uk + j);
#pragma unroll
      for (int r = 0; r < NX; ++r) bu[r] = my_fma(gld(in.B + r * in.nu + j), uj, bu[r]);
    }
  }
}

// z <- A z + B u  (one fast step of the input response)
template <typename T, int NX>
SRTM_DEV void input_step(const InputView<T>& in, const T (&A)[NX][NX], const T* __restrict__ uk, T (&z)[NX]) {
  T nz[NX];
  input_drive(in, uk, nz);
#pragma unroll
  for (int r = 0; r < NX; ++r)
#pragma unroll
    for (int q = 0; q < NX; ++q) nz[r] = my_fma(A[r][q], z[q], nz[r]);
#pragma unroll
  for (int r = 0; r < NX; ++r) z[r] = nz[r];
}

// Input response z_{k,n} of a window from its inputs uk and the sum zs of z_{k,1} .. z_{k,n}. The inputs
// of 8 fast steps are loaded together before they are used, so that their loads are in flight
// at once, and A and B (with zero columns past nu) stay in registers: with B read in every step, each
// entry behind its own test of nu, the tile reduction of 32767 windows (l = 20, nu = 2, float64) took 19.5 us.
template <typename T, int NX, int NY>
SRTM_DEV void input_response(const Model<T, NX, NY>& M, const T* __restrict__ uk, int n, T (&z)[NX], T (&zs)[NX]) {
  constexpr int CH = 8;
  const int nu = M.in.nu;
  T A[NX][NX], B[NX][NU_MAX];
  load(A, M.cst + M.lay.A);
#pragma unroll
  for (int r = 0; r < NX; ++r) {
    zs[r] = z[r] = T(0);
#pragma unroll
    for (int j = 0; j < NU_MAX; ++j) B[r][j] = j < nu ? gld(M.in.B + r * nu + j) : T(0);
  }
#pragma unroll 1
  for (int i0 = 0; i0 < n; i0 += CH) {
    T ub[CH][NU_MAX];
#pragma unroll
    for (int t = 0; t < CH; ++t)
#pragma unroll
      for (int j = 0; j < NU_MAX; ++j) ub[t][j] = (i0 + t < n && j < nu) ? gld(uk + (i0 + t) * nu + j) : T(0);
#pragma unroll
    for (int t = 0; t < CH; ++t) {
      if (i0 + t < n) {
        T nz[NX];
#pragma unroll
        for (int r = 0; r < NX; ++r) {
          T a = T(0);
#pragma unroll
          for (int j = 0; j < NU_MAX; ++j) a = my_fma(B[r][j], ub[t][j], a);
#pragma unroll
          for (int q = 0; q < NX; ++q) a = my_fma(A[r][q], z[q], a);
          nz[r] = a;
        }
#pragma unroll
        for (int r = 0; r < NX; ++r) {
          z[r] = nz[r];
          zs[r] += nz[r];
        }
      }
    }
  }
}

// zL = z_{k,l} and yt = y_k - mu_k of window k < N.
template <typename T, int NX, int NY>
SRTM_DEV void window_input_pass(const Model<T, NX, NY>& M, const T* __restrict__ y, int64_t k, int L,
                                T (&yt)[NY], T (&zL)[NX]) {
  T zs[NX];
  input_response(M, M.in.u + k * L * M.in.nu, L, zL, zs);
  const T inv_l = T(1) / T(L);
#pragma unroll
  for (int r = 0; r < NY; ++r) {
    T s = T(0);
#pragma unroll
    for (int c = 0; c < NX; ++c) s = my_fma(gld(M.in.H + r * NX + c), zs[c], s);
    yt[r] = gld(y + k * NY + r) - s * inv_l;
  }
}

// Window k's measurement (zero past the last window): y_k itself without inputs, and with inputs
// y_k - mu_k and z_{k,l} from the per-window record (zL = 0 without inputs).
template <bool INP, typename T, int NX, int NY>
SRTM_DEV void window_meas(const Model<T, NX, NY>& M, const T* __restrict__ y, int64_t k, int64_t N,
                          T (&yt)[NY], T (&zL)[NX]) {
  constexpr int RS = NX + NY;
#pragma unroll
  for (int r = 0; r < NX; ++r) zL[r] = T(0);
  if constexpr (INP) {
#pragma unroll
    for (int r = 0; r < NY; ++r) yt[r] = (k < N) ? gld(M.in.rec + k * RS + r) : T(0);
#pragma unroll
    for (int r = 0; r < NX; ++r) zL[r] = (k < N) ? gld(M.in.rec + k * RS + NY + r) : T(0);
  } else {
#pragma unroll
    for (int r = 0; r < NY; ++r) yt[r] = (k < N) ? gld(y + k * NY + r) : T(0);
  }
}

// Smoother element of window k (eq. parallel-ak-smoothing, transposed S_k):
//   P^- = A P^f_{k,l} A^T + Q,  E = P^f_{k,1,l} A^T (P^-)^{-1},  g = m^f_{k,1} - E A m^f_{k,l},
//   S = P^f_{k,1} - E A (P^f_{k,1,l})^T = P^f_{k,1} - E P^- E^T;   last window: (0, m^f_{N,1}, P^f_{N,1}).
// Also returns P^-, (P^-)^{-1} and the predicted mean A m^f_{k,l}, which the smoother correction
// reuses. (A, Qm) is the model of the step into x_{k+1,1}. With inputs, z1 = B u_{k,0} is added to
// m^f_{k,1} and bnext = B u_{k+1,0} to the prediction.
template <bool INP, typename T, int NX, int NY, class MV>
SRTM_DEV int smoother_element(const MV& M, int L, const Window<T, NX, NY>& w, bool last,
                              const T (&mL)[NX], const T (&PL)[NX][NX], const T (&z1)[NX], const T (&bnext)[NX],
                              const T (&A)[NX][NX], const T (&Qm)[NX][NX], SElem<T, NX>& el, T (&Pmi)[NX][NX],
                              T (&mpred)[NX], T (&Pm)[NX][NX]) {
  T mf1[NX], Pf11[NX][NX], Pf1L[NX][NX];
  first_step(M, L, w, mf1, Pf11, Pf1L);
  if constexpr (INP) {
#pragma unroll
    for (int r = 0; r < NX; ++r) mf1[r] += z1[r];
  }
  int flag = 0;
  if (last) {
#pragma unroll
    for (int r = 0; r < NX; ++r) {
      el.g[r] = mf1[r];
      mpred[r] = T(0);
#pragma unroll
      for (int c = 0; c < NX; ++c) {
        el.E[r][c] = T(0);
        el.S[r][c] = Pf11[r][c];
        Pmi[r][c] = T(0);
        Pm[r][c] = T(0);
      }
    }
    return 0;
  }
  sandwich(A, PL, Qm, Pm);
  if (!spd_inv(Pm, Pmi)) flag |= SRTM_INFO_PRED_SINGULAR;
  mv(A, mL, mpred);
  if constexpr (INP) {
#pragma unroll
    for (int r = 0; r < NX; ++r) mpred[r] += bnext[r];
  }
  T PA[NX][NX];  // P^f_{1,l} A^T, which is also E P^-
  mm_nt(Pf1L, A, PA);
  mm(PA, Pmi, el.E);
  T Em[NX];
  mv(el.E, mpred, Em);
#pragma unroll
  for (int r = 0; r < NX; ++r) {
    el.g[r] = mf1[r] - Em[r];
#pragma unroll
    for (int c = r; c < NX; ++c) {  // S = P^f_{1,1} - E P^- E^T = P^f_{1,1} - (P^f_{1,l} A^T) E^T
      T s = Pf11[r][c];
#pragma unroll
      for (int k = 0; k < NX; ++k) s = my_fma(-PA[r][k], el.E[c][k], s);
      el.S[r][c] = s;
      el.S[c][r] = s;
    }
  }
  return flag;
}

// ============================================================================ forward
// The scans use one dyadic tree over the windows 0 .. N-1 of a sequence (0-based here): node i of level
// p is the run [i 2^p, (i+1) 2^p), and because the model is time invariant its matrices are Theta(2^p)
// for every i. Only the vector parts (d, eta) are per run. A filter state at window k is the prior followed
// by the runs of the set bits of k, highest first, and the information of all windows after k comes from
// the runs of the clear bits of k below the highest bit in which k and N differ, on top of the runs of N's
// own set bits below it (fold section). The run that bit p of k asks for is always the sibling of the
// node that holds k at that level, (k >> p) ^ 1.
// Levels 1 .. 7 lie within a tile (TILE windows) and are kept per tile in `utree`, node i of level p in
// slot tree_off(p) + i of 2 nx rows (d, eta) of TILE slots; level-0 nodes are the window's own elements and are
// formed again from y where they are needed. Level 8 (whole tiles) is `ftagg`, and the levels above it
// follow each other in `ttree` (tile_level_off).
// Highest set bit of x > 0, and -1 for 0.
SRTM_DEV int top_bit(int64_t x) { return x > 0 ? 63 - __clzll(x) : -1; }

// Combination of the vector parts of two neighbouring runs of 2^p elements, one output row per thread
// (rows 0 .. nx-1: d, nx .. 2nx-1: eta). Row r of a level's coefficient table is 2 nx scalars:
//   d = d_r + G1 d_l + G2 eta_r  (G1, G2),   eta = eta_l + G3 eta_r - G4 d_l  (G3, -G4).
// Child row c at [c * stride]. A thread that formed the whole pair instead read all 4 nx^2 coefficients for it, and those reads set the
// time of a level (about 1 us of a wave in either precision, at nx = 4).
template <int NX>
constexpr int row_slots() { return 2 * NX <= 2 ? 2 : 2 * NX <= 4 ? 4 : 2 * NX <= 8 ? 8 : 16; }

template <typename T, int NX, typename ACC = T>
SRTM_DEV T row_combine(const T* __restrict__ co, const T* __restrict__ left, const T* __restrict__ right, int r, int stride) {
  ACC acc = (ACC)(r < NX ? right[r * stride] : left[r * stride]);
  const T* a = r < NX ? left : right + NX * stride;
  const T* b = r < NX ? right + NX * stride : left;
#pragma unroll
  for (int k = 0; k < NX; ++k) {
    acc = my_fma((ACC)co[k], (ACC)a[k * stride], acc);
    acc = my_fma((ACC)co[NX + k], (ACC)b[k * stride], acc);
  }
  return (T)acc;
}

// Entry q of the row tables of consecutive levels (4 nx^2 scalars a level), from the level records at
// `lev`.
template <typename T, int NX>
SRTM_DEV T row_coefficient(const T* __restrict__ lev, const ConstLayout& lay, int q) {
  constexpr int RT = 4 * NX * NX;
  return gld(lev + (q / RT) * lay.lev_stride + lay.o_C + q % RT);
}

// The same combination for NX <= 4 on the matrix cores, 16 pairs at a time: lane 16 k + col holds row k of the
// children of output node col, and the level's four coefficient matrices are A operands held in registers.
// Rows of LDS slots are read as whole left/right pairs. Read one output row per thread, the children and
// coefficients conflicted in the LDS banks, about 600 cycles for 32 pairs against 150 for 64.
template <typename T, int NX>
struct PairCoef {
  double g1, g2, g3, g4;  // entries (lane & 3, lane >> 4) of G1, G2, G3, -G4
  SRTM_DEV void load_lds(const T* rows) {
    const int lane = threadIdx.x & 63, r = lane & 3, c = lane >> 4;
    const bool in = r < NX && c < NX;
    const T* C = rows + (in ? r * 2 * NX + c : 0);
    g1 = in ? (double)C[0] : 0.0;
    g2 = in ? (double)C[NX] : 0.0;
    g3 = in ? (double)C[2 * NX * NX] : 0.0;
    g4 = in ? (double)C[2 * NX * NX + NX] : 0.0;
  }
  SRTM_DEV void load(const T* __restrict__ rows) {
    const int lane = threadIdx.x & 63, r = lane & 3, c = lane >> 4;
    const bool in = r < NX && c < NX;
    const T* C = rows + (in ? r * 2 * NX + c : 0);
    g1 = in ? (double)gld(C) : 0.0;
    g2 = in ? (double)gld(C + NX) : 0.0;
    g3 = in ? (double)gld(C + 2 * NX * NX) : 0.0;
    g4 = in ? (double)gld(C + 2 * NX * NX + NX) : 0.0;
  }
};

// Output nodes 16 g .. 16 g + 15 (those below n) of one level: children at src[row * stride + 2 i (+ 1)],
// results to dst[row * stride + i].
template <typename T, int NX>
SRTM_DEV void pair_combine(const PairCoef<T, NX>& co, const T* src, T* dst, int stride, int g, int n) {
  typedef T T2 __attribute__((ext_vector_type(2)));
  const int lane = threadIdx.x & 63, k = lane >> 4, i = 16 * g + (lane & 15);
  const bool in = k < NX && i < n;
  T2 d = {T(0), T(0)}, e = {T(0), T(0)};
  if (in) {
    d = *reinterpret_cast<const T2*>(src + k * stride + 2 * i);
    e = *reinterpret_cast<const T2*>(src + (NX + k) * stride + 2 * i);
  }
  const double dl = (double)d.x, dr = (double)d.y, el = (double)e.x, er = (double)e.y;
  const double nd = mm4(co.g2, er, mm4(co.g1, dl, dr));
  const double ne = mm4(co.g4, dl, mm4(co.g3, er, el));
  if (in) {
    dst[k * stride + i] = (T)nd;
    dst[(NX + k) * stride + i] = (T)ne;
  }
}

// Vector part (d, eta) of window k's filter element from its measurement yt (y_k - mu_k with
// inputs) and its input response zL = z_{k,l}.
template <bool INP, typename T, int NX, int NY>
SRTM_DEV void fwd_element(const Model<T, NX, NY>& M, const T (&yt)[NY], const T (&zL)[NX], T (&d)[NX],
                          T (&e)[NX]) {
  T K[NX][NY], He[NX][NY];
  load(K, M.cst + M.lay.K);
  load(He, M.cst + M.lay.Heta);
  mv(K, yt, d);
  mv(He, yt, e);
  if constexpr (INP) {
#pragma unroll
    for (int r = 0; r < NX; ++r) d[r] += zL[r];
  }
}

// How a tile's tree is formed: pairs on the matrix cores (pair_combine), or one thread per node and output row
// (row_combine), its sums in the element type or in float64.
enum TreeForm { TREE_MFMA, TREE_ROWS, TREE_ROWS64 };
// The matrix cores take nx = 3 and 4. A pair of shorter vectors is less than their 4 x 4 blocks carry: 2048 tiles of
// 64 sequences at nx = 2 (float32) take 16 us there, 9 us in rows; 12 tiles at nx = 1 (float64) 5.8 and 4.0.
template <typename T, int NX>
constexpr TreeForm tree_form() { return NX > 4 || (NX <= 2 && sizeof(T) == 8) ? TREE_ROWS : NX <= 2 ? TREE_ROWS64 : TREE_MFMA; }

// K1: the dyadic tree of one tile over the vector parts (d, eta) of its windows' filter elements: levels
// 1 .. LOG_TILE-1 to `utree`, the tile's own node to `ftagg`. The float32 gradient, whose results keep their rounding,
// takes TREE_ROWS for every nx.
template <bool INP, TreeForm FORM, typename T, int NX, int NY>
SRTM_DEV void fwd_reduce_body(const T* __restrict__ y, int64_t N, const T* __restrict__ cst, int L,
                              InputView<T> in, T* __restrict__ tagg, T* __restrict__ utree, int64_t tile) {
  constexpr int NN = NX * NX, R2 = 2 * NX, RS2 = row_slots<NX>();
  constexpr bool ROWS = FORM != TREE_MFMA;
  using ACC = std::conditional_t<FORM == TREE_ROWS64, double, T>;
  extern __shared__ char smraw[];
  T* leaf = reinterpret_cast<T*>(smraw);  // rows of TILE elements, then of the tree's TILE slots, then (ROWS)
  T* tree = leaf + R2 * TILE;
  T* sC = tree + R2 * TILE;               // the row tables of levels 0 .. LOG_TILE-1
  const Model<T, NX, NY> M{cst, make_const_layout(NX, NY, L), in};
  const int tid = threadIdx.x, wv = tid >> 6;
  const int64_t k = tile * TILE + tid;
  // The level records were written by an earlier launch, possibly on another die: one load per
  // coefficient, all in flight together, instead of a dependent round trip per level.
  constexpr int NC = ROWS ? LOG_TILE * 4 * NN : 0, PC = (NC + TILE - 1) / TILE;
  T cv[PC > 0 ? PC : 1], yt[NY], zL[NX], d[NX], e[NX];
  PairCoef<T, (NX <= 4 ? NX : 1)> co[LOG_TILE];
  if constexpr (ROWS) {
#pragma unroll
    for (int i = 0; i < PC; ++i) {
      const int q = i * TILE + tid;
      cv[i] = q < NC ? row_coefficient<T, NX>(M.level(0), M.lay, q) : T(0);
    }
  } else {
#pragma unroll
    for (int p = 0; p < LOG_TILE; ++p) co[p].load(M.level(p) + M.lay.o_C);
  }
  if constexpr (INP) {  // one pass over the window's inputs; later kernels read the record
    if (k < N) {
      window_input_pass(M, y, k, L, yt, zL);
      constexpr int RS = NX + NY;
#pragma unroll
      for (int r = 0; r < NY; ++r) put_global(M.in.rec + k * RS + r, yt[r]);
#pragma unroll
      for (int r = 0; r < NX; ++r) put_global(M.in.rec + k * RS + NY + r, zL[r]);
    } else {
#pragma unroll
      for (int r = 0; r < NY; ++r) yt[r] = T(0);
#pragma unroll
      for (int r = 0; r < NX; ++r) zL[r] = T(0);
    }
  } else {
    window_meas<false>(M, y, k, N, yt, zL);
  }
  if constexpr (ROWS) {
#pragma unroll
    for (int i = 0; i < PC; ++i) {
      const int q = i * TILE + tid;
      if (q < NC) sC[q] = cv[i];
    }
  }
  fwd_element<INP>(M, yt, zL, d, e);
#pragma unroll
  for (int r = 0; r < NX; ++r) {
    leaf[r * TILE + tid] = d[r];
    leaf[(NX + r) * TILE + tid] = e[r];
  }
  __syncthreads();
  constexpr int NT = tree_off(LOG_TILE);  // slots of levels 1 .. LOG_TILE-1
  if constexpr (ROWS) {
    const int row = tid % RS2;
#pragma unroll 1
    for (int p = 1; p <= LOG_TILE; ++p) {
      const T* src = p == 1 ? leaf : tree + tree_off(p - 1);
      T* dst = tree + tree_off(p);
      const int n = TILE >> p;
      if (row < R2) {
        T cr[R2];
#pragma unroll
        for (int k2 = 0; k2 < R2; ++k2) cr[k2] = sC[((p - 1) * R2 + row) * R2 + k2];
        for (int i = tid / RS2; i < n; i += TILE / RS2)
          dst[row * TILE + i] = row_combine<T, NX, ACC>(cr, src + 2 * i, src + 2 * i + 1, row, TILE);
      }
      __syncthreads();
    }
  } else {
    // levels 1 .. 3 by all waves, the rest by wave 0
#pragma unroll
    for (int p = 1; p <= LOG_TILE; ++p) {
      const T* src = p == 1 ? leaf : tree + tree_off(p > 1 ? p - 1 : 1);
      const int n = TILE >> p;
      if (p <= 3) {
        for (int g = wv; g < n / 16; g += TILE / 64) pair_combine<T, NX>(co[p - 1], src, tree + tree_off(p), TILE, g, n);
        __syncthreads();
      } else if (wv == 0) {
        pair_combine<T, NX>(co[p - 1], src, tree + tree_off(p), TILE, 0, n);
        wave_sync();
      }
    }
    __syncthreads();
  }
  T* ut = utree + tile * (R2 * TILE);
  constexpr int NCH = R2 * TILE * (int)sizeof(T) / 16;
  for (int q = tid; q < NCH; q += TILE) {
    const u32x4 v = reinterpret_cast<const u32x4*>(tree)[q];
    put_global(reinterpret_cast<u32x4*>(ut) + q, v);
  }
  if (tid < R2) put_global(tagg + tile * R2 + tid, tree[tid * TILE + NT]);
}

// ---------------------------------------------------------------- fold: states and information
// A filter state (m, P) followed by a run (F, d, D, eta, J) is state_combine; the information (eta, J) about
// the state before a run, from the information after it, is
//   W = (I + J_s D)^{-1},  eta' = F^T W (eta_s - J_s d) + eta,  J' = F^T W J_s F + J,
// the same map with F^T for F, (J, D) for (D, J) and (eta, -d) for (d, eta). So one combine serves both, and
// a window's bit p asks for exactly one of them: forward when the bit is set, backward when it is
// clear. With the state (m, P) after window k and the information (eta, J) of every window after it,
//   v = (I + J P)^{-1} (eta - J m),   W = -(I + J P)^{-1} J
// are the smoother correction of eq. seq-smoothing-all (m^s_{k,i} = m^f_{k,i} + P^f_{k,i,l} v and
// P^s_{k,i} = P^f_{k,i,i} + P^f_{k,i,l} W P^f_{k,i,l}^T): p(x_{k,l} | y_{1:N}) is the filter state times the
// likelihood of the later measurements, whose information form is the (eta, J) of their filter element
// (eq. op-filter). Unlike the smoother elements of eq. parallel-ak-smoothing, which are built from the
// filter states and scanned after them, (eta, J) comes from the same tree as the states, so both are
// found in one pass and no second tile-level scan follows it.

// A combine solves (I + P J) y = u + P ve and (I + P J) X = P by the explicit inverse; then y' = T y + vd and
// P' = T X T^T + D. Where P J is large, as after a wide prior, the inverse loses digits that T y and T X T^T show
// (float64, nx = 2, P0 = 1e4 I: filter means 2e-6 off). A wave with P J beyond REFINE_FROM among its
// problems therefore refines both solutions by one residual step, b - y - P (J y), and takes the mean of X with its
// transpose; in all waves that would be 10 % of a call (nx = 4, float64, 3000 windows). Float32 calls need none in
// float64 steps, and nx = 1 and nx > 4 (elimination with pivoting) lost nothing against the window-by-window form.
constexpr double REFINE_FROM = 256.0;

// One combine in the block layout (four problems per wave): state (u, P) and run (Tt = F^T or F, Dp, Jp, vd,
// ve), in place. u is a vector held as equal columns; P, Dp and Jp are symmetric.
template <int NX, bool REFINE>
SRTM_DEV bool combine4(const Block4& B, double& u, double& P, double Tt, double Dp, double Jp, double vd, double ve) {
  bool ok = true;
  const double b = mm4(P, ve, u), A = mm4(P, Jp, B.eye);    // u + P ve, I + P Jp
  const double Wt = B.template inv_t<NX>(A, ok);            // A^{-T}
  double X = Block4::mm_sym(Wt, P), y = mm4(Wt, b, 0.0);
  if (REFINE && __any(fabs(A) > REFINE_FROM)) {
    const double E = mm4(P, -mm4(Jp, X, 0.0), P - X), e = mm4(P, -mm4(Jp, y, 0.0), b - y);
    X = 0.5 * (mm4(Wt, E, X) + mm4(E, Wt, X));
    y = mm4(Wt, e, y);
  }
  u = mm4(Tt, y, vd);
  P = Block4::mm_sym(Tt, mm4(X, Tt, 0.0)) + Dp;
  return ok;
}

// The same for one problem per wave, nx > 4.
template <int NX>
SRTM_DEV bool combine8(const Block8<NX>& B, double& u, double& P, double Tt, double Dp, double Jp, double vd, double ve) {
  bool ok = true;
  const Lhs8 lP(P), lT(Tt);
  const Rhs8 rP(P), rT(Tt);
  const double w = mm8(lP, Rhs8(ve), u);
  const double Wt = B.inv_t(mm8(lP, Rhs8(Jp), B.in() && B.r == B.c ? 1.0 : 0.0), ok);
  const Lhs8 lW(Wt);
  const double X = 0.5 * (mm8(lW, rP, 0.0) + mm8(lP, Rhs8(Wt), 0.0));
  u = mm8(lT, Rhs8(mm8(lW, Rhs8(w), 0.0)), vd);
  const double Y = mm8(Lhs8(X), rT, 0.0);
  P = 0.5 * (mm8(lT, Rhs8(Y), 0.0) + mm8(Lhs8(Y), rT, 0.0)) + Dp;
  return ok;
}
// combine8 with level tables `tab` ((F, D, J), (F^T, J, D)) and the run (d, eta), row r at nd[r * stride].
template <int NX, typename T>
SRTM_DEV bool wave_combine(const Block8<NX>& B, double& u, double& P, const T* tab, const T* nd, int stride, bool fwd) {
  constexpr int NN = NX * NX;
  const bool in = B.in();
  const T* t = tab + (in ? B.r * NX + B.c : 0);
  const double a = in ? (double)t[0] : 0.0, b = in ? (double)t[NN] : 0.0, c = in ? (double)t[2 * NN] : 0.0,
               at = in ? (double)t[3 * NN] : 0.0;
  const double d = B.r < NX ? (double)nd[B.r * stride] : 0.0, e = B.r < NX ? (double)nd[(NX + B.r) * stride] : 0.0;
  return combine8(B, u, P, fwd ? at : a, fwd ? b : c, fwd ? c : b, fwd ? d : e, fwd ? e : -d);
}

SRTM_DEV int tile_windows(int64_t N, int64_t tile) {
  const int64_t w = N - tile * TILE;
  return (int)(w < TILE ? w : TILE);
}

// Levels handled one lane per window in the fold; the ones above go to the matrix cores, four problems per wave for
// nx <= 4 (a wave's 16-window groups) and one for larger nx (a wave's 64 windows). A level of one lane per
// window costs a wave about 700 instructions at nx = 4 whatever it holds, the four problems of a wave's
// groups about 60; at nx = 6 (float32, 63 tiles) the fold took 52 us with all 14 levels in lanes, 42 us so.
// nx = 1 stays in lanes: a combine of scalars is shorter there than a 4 x 4 one on the matrix cores (20000 windows in
// float32: the filter's fold 5 us in lanes, 10 us in blocks), and its tiles gain too little from being settled.
constexpr int LANE_LEVELS = 4;
template <int NX> constexpr bool blocks4() { return NX >= 2 && NX <= 4; }
template <int NX> constexpr bool block8() { return NX > 4; }
template <int NX> constexpr int lane_levels() { return blocks4<NX>() ? LANE_LEVELS : block8<NX>() ? LOG_TILE - 2 : LOG_TILE; }

// LDS of the fold, in bytes from its start (level tables of nlev levels).
template <typename T, int NX>
struct FoldLds {
  static constexpr int NN = NX * NX, R2 = 2 * NX, IS = info_stride(NX);
  static constexpr int MAXT = 20;                                          // tile-level bits (N <= 2^26: 18)
  static constexpr int NZ = LOG_TILE + 1;
  size_t leaf, tree, lane, lev, node, tail, scratch, group, gain, total;
  __host__ __device__ FoldLds(int nlev) {
    const int laneL = blocks4<NX>() ? lane_levels<NX>() : nlev;  // all levels where the matrix cores take them from here
    size_t o = 0;
    auto take = [&](size_t n) { const size_t at = o; o = (o + n + 15) & ~size_t(15); return at; };
    leaf = take(sizeof(T) * R2 * TILE);
    tree = take(sizeof(T) * R2 * TILE);
    lane = take(sizeof(T) * (size_t)laneL * 6 * NN);                       // per level (F, D, J), (F^T, J, D)
    lev = take(blocks4<NX>() ? sizeof(double) * 48 * (size_t)nlev : 0);    // per level F, D, J as 4 x 4 blocks
    node = take(sizeof(T) * MAXT * R2);                                    // tile-level nodes of this tile
    tail = take(sizeof(double) * NZ * IS * 4);                             // information of N's low bits
    scratch = take(sizeof(double) * 64 * 4);
    group = take(sizeof(double) * 4 * (blocks4<NX>() ? 4 * 40 : 2 * (NN + NX)));  // states of each wave's groups
    gain = take(blocks4<NX>() ? sizeof(double) * LOG_TILE * 2 * 2 * NN : 0);    // a settled tile's gains per level
    total = o;
  }
};

// Levels a sequence can have (N <= 2^26).
constexpr int MAXLEV = 26;

// Float32 sequences of several tiles keep F, D, J of every level in float64 too, behind the prior records
// (nx = 1 leaves no room there): the fold's float64 steps then work with one consistent model, so that a state that has settled
// is seen as settled to float64 rounding.
template <typename T, int NX>
SRTM_DEV bool has_lev64(int64_t N) { return std::is_same_v<T, float> && NX >= 2 && NX <= 4 && N > TILE; }

// Entry q of the fold's level tables: F, D, J as 4 x 4 blocks, 48 entries a level.
template <typename T, int NX>
SRTM_DEV double block_entry(const T* __restrict__ cst, const double* __restrict__ lev64, const ConstLayout& lay, int q) {
  const int p = q / 48, e = q % 48, r = (e % 16) / 4, c = e % 4;
  if (r >= NX || c >= NX) return 0.0;
  const int o = (e / 16) * NX * NX + r * NX + c;
  if (std::is_same_v<T, float> && lev64) return gld(lev64 + p * 3 * NX * NX + o);
  return (double)gld(cst + lay.lev + p * lay.lev_stride + lay.o_F + o);
}
template <typename T, int NX>
SRTM_DEV void stage_blocks(const T* __restrict__ cst, const double* __restrict__ lev64, const ConstLayout& lay, int nlev,
                           double* lev, int tid, int nthr) {
  staged_copy<4, double>(nlev * 48, tid, nthr, [&](int q) { return block_entry<T, NX>(cst, lev64, lay, q); },
                         [&](int q, double v) { lev[q] = v; });
}

// ---------------------------------------------------------------- settled tiles
// Under a time-invariant model the covariances of a filter and smoother that forget settle: after some
// hundred windows every window has the same P^f and J, and only vectors differ. The fold tests this per
// whole tile, in float64, on the state (P) at the tile's start and the information (J) after its end: one
// window's map and the whole tile's map have to leave each of them where it is, entry by entry within
// settled_tol of the standard deviations. What changes by less over the tile's 256 windows is the same matrix
// for all of them to the rounding of the element type. In a settled tile the fold combines vectors only (a 4 x 4
// gain pair per level, formed once per tile, instead of a matrix inverse per window and level), and the
// recovery forms the covariances of a fast step once per tile and streams them to every window.
// Tiles near either end, models that do not settle, and anything not finite take the general way.
// Float64: 2^-47, some rounding errors of one combine. 2^-49 is at the rounding itself: 4 of 36 random models (nx = 4) then
// never settle, and a call of 32767 windows with inputs takes 123 us instead of 79; the worst P^f of 30 models that
// settle slowly would be 3.3e-15 off instead of 7.4e-15. Float32: 2^-26, a quarter of its rounding.
template <typename T>
SRTM_DEV constexpr double settled_tol() { return sizeof(T) == 8 ? 0x1p-47 : 0x1p-26; }
// Whether a tile is settled is kept in the last slot of its tree's first row (levels 1 .. 7 leave two free).
template <typename T, int NX>
SRTM_DEV T* settled_flag(T* utree, int64_t tile) { return utree + tile * (2 * NX * TILE) + TILE - 1; }
template <typename T, int NX>
SRTM_DEV bool tile_settled(const T* utree, int64_t tile) {
  if constexpr (!blocks4<NX>()) return false;
  const int f = gld(settled_flag<T, NX>(const_cast<T*>(utree), tile)) != T(0);
  return __builtin_amdgcn_readfirstlane(f) != 0;
}

// One lane's state / information: vector and symmetric matrix.
template <typename T, int NX>
struct Belief {
  T u[NX], P[NX][NX];
};

template <typename T, int NX>
SRTM_DEV void belief_zero(Belief<T, NX>& b) {
#pragma unroll
  for (int r = 0; r < NX; ++r) {
    b.u[r] = T(0);
#pragma unroll
    for (int c = 0; c < NX; ++c) b.P[r][c] = T(0);
  }
}
// From a packed record (vector, upper triangle).
template <typename T, int NX, typename S>
SRTM_DEV void belief_load(Belief<T, NX>& b, const S* p) {
  int o = NX;
#pragma unroll
  for (int r = 0; r < NX; ++r) {
    b.u[r] = (T)p[r];
#pragma unroll
    for (int c = r; c < NX; ++c) b.P[r][c] = b.P[c][r] = (T)p[o++];
  }
}

// One window's record: the vector from its column `col`, the symmetric matrix from column `mcol` (the same,
// or the tile's first window's in a settled tile), W windows per field.
template <typename T, int NX, typename S>
SRTM_DEV void record_load(T (&u)[NX], T (&P)[NX][NX], const S* __restrict__ col, const S* __restrict__ mcol, int W) {
  int o = NX;
#pragma unroll
  for (int r = 0; r < NX; ++r) {
    u[r] = (T)gld(col + (int64_t)r * W);
#pragma unroll
    for (int c = r; c < NX; ++c) P[r][c] = P[c][r] = (T)gld(mcol + (int64_t)(o++) * W);
  }
}
template <typename T, int NX>
SRTM_DEV void record_store(const T (&u)[NX], const T (&P)[NX][NX], T* __restrict__ col, int W, bool matrix) {
#pragma unroll
  for (int r = 0; r < NX; ++r) put_global(col + (int64_t)r * W, u[r]);
  if (matrix) {
    int o = NX;
#pragma unroll
    for (int r = 0; r < NX; ++r)
#pragma unroll
      for (int c = r; c < NX; ++c) put_global(col + (int64_t)(o++) * W, P[r][c]);
  }
}

// One lane's combine with the run (d, e), row r at nd[r * stride], of level tables `tab` = (F, Dp, Jp) as staged for its direction.
template <typename T, int NX, typename S>
SRTM_DEV bool lane_combine(Belief<T, NX>& b, const T* __restrict__ tab, const S* __restrict__ nd, int stride, bool fwd) {
  constexpr int NN = NX * NX;
  T J[NX][NX], A[NX][NX], W[NX][NX], X[NX][NX], r[NX], y[NX], vd[NX];
  load(J, tab + 2 * NN);
#pragma unroll
  for (int i = 0; i < NX; ++i) r[i] = b.u[i];
#pragma unroll
  for (int k = 0; k < NX; ++k) {
    const T d = (T)nd[k * stride], e = (T)nd[(NX + k) * stride], ve = fwd ? e : -d;
    vd[k] = fwd ? d : e;
#pragma unroll
    for (int i = 0; i < NX; ++i) r[i] = my_fma(b.P[i][k], ve, r[i]);
  }
  mm(b.P, J, A);
  T big = T(0);
#pragma unroll
  for (int i = 0; i < NX; ++i) {
#pragma unroll
    for (int k = 0; k < NX; ++k) big = my_fma(A[i][k], A[i][k], big);
    A[i][i] += T(1);
  }
  const bool ok = inv_small(A, W);
  mv(W, r, y);
#pragma unroll
  for (int i = 0; i < NX; ++i)
#pragma unroll
    for (int c = i; c < NX; ++c) {
      T t = T(0);
#pragma unroll
      for (int k = 0; k < NX; ++k) t = my_fma(W[i][k], b.P[k][c], t);
      X[i][c] = X[c][i] = t;
    }
  if (blocks4<NX>() && __builtin_expect(__any(big > T(REFINE_FROM * REFINE_FROM)), 0)) {
    auto residual = [&](const T (&q)[NX], const T (&z)[NX], T (&e)[NX]) {  // q - z - P (J z)
      T Jz[NX];
      mv(J, z, Jz);
#pragma unroll
      for (int i = 0; i < NX; ++i) {
        T t = q[i] - z[i];
#pragma unroll
        for (int k = 0; k < NX; ++k) t = my_fma(-b.P[i][k], Jz[k], t);
        e[i] = t;
      }
    };
    T e[NX];
    residual(r, y, e);
    mv_acc(W, e, y);
#pragma unroll
    for (int c = 0; c < NX; ++c) {
      T q[NX], z[NX];
#pragma unroll
      for (int i = 0; i < NX; ++i) q[i] = b.P[i][c];
      mv(W, q, z);
      residual(q, z, e);
      mv_acc(W, e, z);
#pragma unroll
      for (int i = 0; i < NX; ++i) X[i][c] = z[i];
    }
    symmetrize(X);
  }
  T F[NX][NX], D[NX][NX];
  load(F, tab);
  load(D, tab + NN);
#pragma unroll
  for (int i = 0; i < NX; ++i) b.u[i] = vd[i];
  mv_acc(F, y, b.u);
  sandwich(F, X, D, b.P);
  return ok;
}

// Information of N's set bits below each bit (tail), low bits first, for a sequence's last windows.
// `node(p)` is the (d, eta) of N's node of level p, row r at node(p)[r * stride] in LDS; entry q of `out` (info_stride scalars
// each) receives the information of N's set bits below bit q, q = 0 .. qmax. One wave; every block of
// lanes (nx <= 4) computes the same chain.
template <typename T, int NX, class ND>
SRTM_DEV bool tail_chain(const double* lev, const T* lane, double* scratch, int64_t N, int qmax, ND node, int stride,
                         double* out) {
  constexpr int NN = NX * NX, IS = info_stride(NX);
  bool ok = true;
  if constexpr (blocks4<NX>()) {
    const Block4 B(scratch);
    const bool in = B.r < NX && B.c < NX;
    double u = 0.0, P = 0.0;
    for (int q = 0; q <= qmax; ++q) {
      if (B.b == 0 && in) {
        if (B.c == 0) out[q * IS + B.r] = u;
        if (B.c >= B.r) out[q * IS + NX + B.r * NX - B.r * (B.r - 1) / 2 + B.c - B.r] = P;
      }
      if (q < qmax && ((N >> q) & 1)) {
        const double* lv = lev + q * 48;
        const auto* nd = node(q);
        const double d = B.r < NX ? (double)nd[B.r * stride] : 0.0, e = B.r < NX ? (double)nd[(NX + B.r) * stride] : 0.0;
        if (!combine4<NX, sizeof(T) == 8>(B, u, P, lv[4 * B.r + B.c], lv[32 + 4 * B.r + B.c], lv[16 + 4 * B.r + B.c], e, -d)) ok = false;
      }
    }
  } else if constexpr (block8<NX>()) {
    const Block8<NX> B(scratch);
    double u = 0.0, P = 0.0;
#pragma unroll 1
    for (int q = 0; q <= qmax; ++q) {
      if (B.in()) {
        if (B.c == 0) out[q * IS + B.r] = u;
        if (B.c >= B.r) out[q * IS + NX + B.r * NX - B.r * (B.r - 1) / 2 + B.c - B.r] = P;
      }
      if (q < qmax && ((N >> q) & 1)) {
        if (!wave_combine(B, u, P, lane + (size_t)q * 6 * NN, node(q), stride, false)) ok = false;
      }
    }
  } else {
    Belief<T, NX> b;
    belief_zero(b);
#pragma unroll 1
    for (int q = 0; q <= qmax; ++q) {
      if ((threadIdx.x & 63) == 0) {
        int o = NX;
#pragma unroll
        for (int r = 0; r < NX; ++r) {
          out[q * IS + r] = (double)b.u[r];
#pragma unroll
          for (int c = r; c < NX; ++c) out[q * IS + o++] = (double)b.P[r][c];
        }
      }
      if (q < qmax && ((N >> q) & 1)) {
        if (!lane_combine(b, lane + (size_t)q * 6 * NN + 3 * NN, node(q), stride, false)) ok = false;
      }
    }
  }
  return ok;
}

// Direction tables of one lane: per level (F, D, J) for forward combines and (F^T, J, D) for backward
// ones, 6 nx^2 scalars a level.
template <typename T, int NX>
SRTM_DEV void stage_lane_tables(const T* __restrict__ cst, const ConstLayout& lay, int nlev, T* out, int tid, int nthr) {
  constexpr int NN = NX * NX;
  staged_copy<4, T>(nlev * 6 * NN, tid, nthr,
                    [&](int q) {
                      const int p = q / (6 * NN), e = q % (6 * NN), m = e / NN, r = (e % NN) / NX, c = e % NX;
                      const int off = m == 0 ? r * NX + c : m == 3 ? c * NX + r
                                    : (m == 1 || m == 5 ? NN : 2 * NN) + r * NX + c;
                      return gld(cst + lay.lev + p * lay.lev_stride + lay.o_F + off);
                    },
                    [&](int q, T v) { out[q] = v; });
}

// (d, eta) of N's level-0 node, the element of window N-1 (bit 0 of N set).
template <bool INP, typename T, int NX, int NY>
SRTM_DEV void last_element(const Model<T, NX, NY>& M, const T* __restrict__ y, int64_t N, T* out) {
  T yt[NY], zL[NX], d[NX], e[NX];
  window_meas<INP>(M, y, N - 1, N, yt, zL);
  fwd_element<INP>(M, yt, zL, d, e);
#pragma unroll
  for (int r = 0; r < NX; ++r) {
    out[r] = d[r];
    out[NX + r] = e[r];
  }
}

// Threads of the tile-level kernel (KS in a mixed batch), and the nodes of one level that it keeps in LDS
// (longer levels are read back from device memory; the levels of at most this size together take less than
// twice it).
constexpr int TT = 512;
template <int NX> constexpr int tt_nodes() { return NX <= 4 ? 512 : 256; }
template <typename T, int NX>
inline size_t tile_tree_lds_bytes(int nlev) {
  constexpr int NN = NX * NX;
  const size_t tab = blocks4<NX>() ? sizeof(double) * 48 * (size_t)nlev : sizeof(T) * 6 * NN * (size_t)nlev;
  return sizeof(T) * 2 * NX * (2 * (size_t)tt_nodes<NX>()) + sizeof(T) * 4 * NN * (size_t)(nlev > LOG_TILE ? nlev - LOG_TILE : 0) +
         tab + sizeof(T) * 2 * NX * 32 + sizeof(double) * 64 + 128;
}

// K2: the levels of the tree above the tiles, over the sequence's whole tiles (one workgroup per sequence;
// nodes formed as in the tile reductions, tree_form), and, for the smoother, the information of
// N's set bits below each bit. A sequence of one tile has no level above it and its fold finds
// the information of N's bits by itself.
template <bool INP, typename T, int NX, int NY>
SRTM_DEV void tile_tree_body(const T* __restrict__ y, int64_t N, int nlev, const T* __restrict__ cst,
                             const double* __restrict__ lev64, int L,
                             InputView<T> in, const T* __restrict__ tagg, const T* __restrict__ utree,
                             T* __restrict__ ttree, double* __restrict__ tail, bool smoother, int32_t* info, int nthr) {
  constexpr int NN = NX * NX, R2 = 2 * NX, RS2 = row_slots<NX>(), TT_NODES = tt_nodes<NX>();
  const int64_t nf = N >> LOG_TILE;
  if (N <= TILE) return;
  extern __shared__ char smraw[];
  T* nodes = reinterpret_cast<T*>(smraw);                                   // 2 TT_NODES nodes
  T* sC = nodes + R2 * 2 * TT_NODES;                                        // row tables of levels LOG_TILE ..
  T* own = sC + (nlev > LOG_TILE ? nlev - LOG_TILE : 0) * 4 * NN;           // N's nodes, by level
  double* dbl = reinterpret_cast<double*>(((uintptr_t)(own + R2 * 32) + 15) & ~(uintptr_t)15);
  double* scratch = dbl;                                                    // 64
  double* lev = dbl + 64;                                                   // 4 x 4 blocks (nx <= 4) or
  T* lane = reinterpret_cast<T*>(lev);                                      // lane tables (nx > 4)
  const Model<T, NX, NY> M{cst, make_const_layout(NX, NY, L, nlev), in};
  const int tid = threadIdx.x;
  staged_copy<4, T>((nlev - LOG_TILE) * 4 * NN, tid, nthr,
                    [&](int q) { return row_coefficient<T, NX>(M.level(LOG_TILE), M.lay, q); },
                    [&](int q, T v) { sC[q] = v; });
  if (smoother) {
    if constexpr (blocks4<NX>()) stage_blocks<T, NX>(cst, lev64, M.lay, nlev, lev, tid, nthr);
    else stage_lane_tables<T, NX>(cst, M.lay, nlev, lane, tid, nthr);
    // N's nodes within the last tile (its bits 1 .. 7), and bit 0's window
    const T* ut = utree + (N >> LOG_TILE) * (R2 * TILE);
    for (int q = tid; q < (LOG_TILE - 1) * R2; q += nthr) {
      const int p = 1 + q / R2;
      if ((N >> p) & 1) own[p * R2 + q % R2] = gld(ut + (q % R2) * TILE + tree_off(p) + (((int)(N & (TILE - 1)) >> p) ^ 1));
    }
    if (tid == nthr - 1 && (N & 1)) last_element<INP>(M, y, N, own);
  }
  // Up-sweep; level LOG_TILE + q has nf >> q nodes. Levels longer than the LDS buffer go through device
  // memory (each of them waits for its stores); the others stay in LDS, rows of 2 TT_NODES slots, and are
  // stored together at the end, so that no level waits for a store to arrive.
  constexpr int ST = 2 * TT_NODES;
  using ACC = std::conditional_t<tree_form<T, NX>() == TREE_ROWS64, double, T>;
  const int row = tid % RS2, wv = tid >> 6;
  int q0 = 0;              // first level kept in LDS
  while ((nf >> q0) > TT_NODES) ++q0;
  {
    const T* src = tagg;
    T* dst = ttree;
#pragma unroll 1
    for (int q = 1; q <= q0; ++q) {
      const int64_t nn = nf >> q;
      __syncthreads();  // the row tables (first level), the level below
      if (smoother && ((nf >> (q - 1)) & 1) && tid < R2) own[(LOG_TILE + q - 1) * R2 + tid] = gld(src + ((nf >> (q - 1)) - 1) * R2 + tid);
      if (row < R2)
        for (int64_t i = tid / RS2; i < nn; i += nthr / RS2)
          put_global(dst + i * R2 + row, row_combine<T, NX>(sC + ((q - 1) * R2 + row) * R2, src + 2 * i * R2,
                                                            src + (2 * i + 1) * R2, row, 1));
      src = dst;
      dst += nn * R2;
    }
    if (q0) __syncthreads();
    const int n = (int)(nf >> q0);
    staged_copy<8, T>(n * R2, tid, nthr, [&](int q) { return gld(src + q); },
                      [&](int q, T v) { nodes[(q % R2) * ST + q / R2] = v; });
    __syncthreads();
    int at = 0;  // the level below
#pragma unroll 1
    for (int q = q0 + 1; (nf >> q) > 0; ++q) {
      const int below = (int)(nf >> (q - 1)), nn = (int)(nf >> q);
      const int to = (at + below + 1) & ~1;  // pairs are read whole: even slots
      if constexpr (tree_form<T, NX>() == TREE_MFMA) {
        PairCoef<T, NX> co;
        co.load_lds(sC + (q - 1) * 4 * NN);
        for (int g = wv; g < (nn + 15) / 16; g += nthr >> 6) pair_combine<T, NX>(co, nodes + at, nodes + to, ST, g, nn);
      } else if (row < R2) {
        T co[R2];
#pragma unroll
        for (int k2 = 0; k2 < R2; ++k2) co[k2] = sC[((q - 1) * R2 + row) * R2 + k2];
        for (int i = tid / RS2; i < nn; i += nthr / RS2)
          nodes[row * ST + to + i] = row_combine<T, NX, ACC>(co, nodes + at + 2 * i, nodes + at + 2 * i + 1, row, ST);
      }
      at = to;
      __syncthreads();
    }
    // the levels above q0 to device memory, and N's nodes
    int o = 0;
    for (int q = q0; (nf >> q) > 0; ++q) {
      const int cnt = (int)(nf >> q);
      if (q > q0) {
        for (int e = tid; e < cnt * R2; e += nthr) put_global(dst + e, nodes[(e % R2) * ST + o + e / R2]);
        dst += cnt * R2;
      }
      if (smoother && (cnt & 1) && tid < R2) own[(LOG_TILE + q) * R2 + tid] = nodes[tid * ST + o + cnt - 1];
      o = (o + cnt + 1) & ~1;
    }
  }
  __syncthreads();
  if (smoother && tid < 64) {
    const bool ok = tail_chain<T, NX>(lev, lane, scratch, N, top_bit(N), [&](int p) { return own + p * R2; }, 1, tail);
    if (!ok && info) atomicOr(info, SRTM_INFO_COMBINE_SINGULAR);
  }
}

// K5: reverse tile-level scan of the time-varying smoother in one workgroup of KS threads. Thread r holds the aggregate of
// its chunk of 2^lchunk consecutive tiles, counted from the end (thread 0 holds the last tiles),
// folded under eq. op-smoother (earlier (x) later), and merges it with all later runs (lane
// shuffles inside a wave, then the later waves' aggregates). Every run reaching the
// last window has E = 0, i.e. is the smoothed state at its first window; thread r then walks
// its chunk backwards from the state after it, writing per tile the smoothed state of the
// first window after the tile (zero after the last tile).
template <typename T, int NX>
SRTM_DEV void ld_selem_global(const T* __restrict__ src, SElem<T, NX>& x) {
  constexpr int NN = NX * NX;
#pragma unroll
  for (int i = 0; i < NX; ++i) {
    x.g[i] = gld(src + NN + i);
#pragma unroll
    for (int c = 0; c < NX; ++c) {
      x.E[i][c] = gld(src + i * NX + c);
      x.S[i][c] = gld(src + NN + NX + i * NX + c);
    }
  }
}

template <typename T, int NX>
SRTM_DEV void selem_identity(SElem<T, NX>& x) {
#pragma unroll
  for (int i = 0; i < NX; ++i) {
    x.g[i] = T(0);
#pragma unroll
    for (int c = 0; c < NX; ++c) {
      x.E[i][c] = (i == c) ? T(1) : T(0);
      x.S[i][c] = T(0);
    }
  }
}

template <typename T, int NX, int NY>
SRTM_DEV void bwd_tiles_body(const T* __restrict__ tagg, int64_t nt, int lchunk, int steps, T* __restrict__ tstate) {
  constexpr int NN = NX * NX, SE = 2 * NN + NX, ST = NX + NN;
  extern __shared__ char smraw[];
  const Slots<T> S{reinterpret_cast<T*>(smraw), KS};
  const int tid = threadIdx.x;
  const int64_t c = int64_t(1) << lchunk;
  const int64_t thi = nt - 1 - tid * c;  // the chunk is tiles thi - c + 1 .. thi (those >= 0)
  SElem<T, NX> x, xhi;  // xhi: the aggregate of tile thi itself (c = 2), reused by the walk
  if (thi >= 0 && c == 2) {  // both loads in flight together
    SElem<T, NX> a;
    ld_selem_global(tagg + thi * SE, xhi);
    if (thi - 1 >= 0) {
      ld_selem_global(tagg + (thi - 1) * SE, a);
      selem_combine(a, xhi, x);
    } else {
      x = xhi;
    }
  } else if (thi >= 0) {
    ld_selem_global(tagg + thi * SE, x);
#pragma unroll 1
    for (int64_t t = thi - 1; t > thi - c && t >= 0; --t) {
      SElem<T, NX> a;
      ld_selem_global(tagg + t * SE, a);
      selem_combine(a, x, x);
    }
  } else {
    selem_identity(x);
  }
  // Thread r ends with its run merged with every later run (threads r - 1 .. 0): within each
  // wave by lane shuffles (distances below 64), then each wave with the aggregates of the waves
  // before it (later tiles; lane 63 holds its wave's), through LDS.
  {
    const int lane = tid & 63, wv = tid >> 6;
    const int lim = steps < 6 ? steps : 6;
#pragma unroll 1
    for (int q = 0; q < lim; ++q) selem_merge_lane<false>(x, 1 << q, lane >= (1 << q));
    if (steps > 6) {
      if (lane == 63) st_selem(S, wv, x);
      __syncthreads();
#pragma unroll 1
      for (int v = wv - 1; v >= 0; --v) {  // x (x) A_{wv-1} (x) ... (x) A_0, left to right
        SElem<T, NX> a;
        ld_selem(S, v, a);
        selem_combine(x, a, x);
      }
      __syncthreads();  // the aggregates are read before the slots take the results
    }
  }
  st_selem(S, tid, x);
  __syncthreads();
  if (thi >= 0) {
    T m[NX], P[NX][NX];
    if (tid > 0) {
      SElem<T, NX> nxt;
      ld_selem(S, tid - 1, nxt);
#pragma unroll
      for (int i = 0; i < NX; ++i) {
        m[i] = nxt.g[i];
#pragma unroll
        for (int cc = 0; cc < NX; ++cc) P[i][cc] = nxt.S[i][cc];
      }
    } else {
#pragma unroll
      for (int i = 0; i < NX; ++i) {
        m[i] = T(0);
#pragma unroll
        for (int cc = 0; cc < NX; ++cc) P[i][cc] = T(0);
      }
    }
#pragma unroll 1
    for (int64_t t = thi; t > thi - c && t >= 0; --t) {
#pragma unroll
      for (int i = 0; i < NX; ++i) tstate[t * ST + i] = m[i];
#pragma unroll
      for (int i = 0; i < NX; ++i)
#pragma unroll
        for (int cc = 0; cc < NX; ++cc) tstate[t * ST + NX + i * NX + cc] = P[i][cc];
      if (t - 1 > thi - c && t - 1 >= 0) {
        if (c == 2) {
          sstate_combine(xhi, m, P);
        } else {
          SElem<T, NX> a;
          ld_selem_global(tagg + t * SE, a);
          sstate_combine(a, m, P);
        }
      }
    }
  }
}

// Output staging. Each lane computes one window's blocks; records are written to LDS
// and copied out by the whole wave so that consecutive lanes store consecutive 16-byte
// chunks. Covariance records (nx^2 scalars) are flushed every fast step; means are
// gathered over G consecutive fast steps so that a record fills whole cache lines.
template <int CH> struct Chunk;
template <> struct Chunk<16> { using type = u32x4; };
template <> struct Chunk<8> { using type = u32x2; };
template <> struct Chunk<4> { using type = unsigned int; };

// Store of one output chunk. Outputs are written once and never read back by the library;
// when a flush writes whole 128-byte lines they are stored non-temporally (streamed past the
// L2), otherwise normally, so that partial lines can merge in the L2 first.
template <bool NT, typename V>
SRTM_DEV void put_chunk(char* p, const V& v) {
  using G = __attribute__((address_space(1))) V*;  // outputs are device memory: global stores
  if constexpr (NT)
    __builtin_nontemporal_store(v, (G)p);
  else
    *(G)p = v;
}


// Copies records w = 0..nvalid-1 (nvalid <= 64) of RB bytes (stride SB bytes in LDS) to
// dst + w * gstride bytes in chunks of CH bytes. A record is PER = RB / CH chunks; one store
// instruction moves WPI = 64 / PER whole records (lane l: chunk l mod PER of record
// l / PER + r WPI; the last 64 mod PER lanes idle), so every store address is a wave-uniform base
// plus one loop-invariant 32-bit lane offset.
template <int RB, int SB, int CH, bool NT>
SRTM_DEV void flush_chunks(int lane, int nvalid, const char* __restrict__ lds, char* __restrict__ dst,
                           int64_t gstride) {
  constexpr int PER = RB / CH;
  static_assert(RB % CH == 0 && SB % CH == 0 && PER <= 64, "whole chunks, at most one per lane");
  constexpr int WPI = 64 / PER;
  constexpr int NIT = (64 + WPI - 1) / WPI;
  using V = typename Chunk<CH>::type;
  const int wl = lane / PER, pl = lane - wl * PER;
  const unsigned int lo = (unsigned int)(wl * gstride) + (unsigned int)(pl * CH);
  const char* lsrc = lds + wl * SB + pl * CH;
  if constexpr (64 % PER == 0) {  // every lane busy: all LDS reads first, then the stores back to back
    V v[NIT];
#pragma unroll
    for (int r = 0; r < NIT; ++r) v[r] = *reinterpret_cast<const V*>(lsrc + r * WPI * SB);
    if (nvalid == 64) {
#pragma unroll
      for (int r = 0; r < NIT; ++r) put_chunk<NT>(dst + (int64_t)r * WPI * gstride + lo, v[r]);
    } else {
#pragma unroll
      for (int r = 0; r < NIT; ++r)
        if (wl + r * WPI < nvalid) put_chunk<NT>(dst + (int64_t)r * WPI * gstride + lo, v[r]);
    }
  } else {  // groups of four instructions (reads, then stores), to bound the registers held
    constexpr int G = 4;
    const bool act = wl < WPI;
#pragma unroll 1
    for (int r0 = 0; r0 < NIT; r0 += G) {
      V v[G];
#pragma unroll
      for (int j = 0; j < G; ++j)
        if (r0 + j < NIT && act && wl + (r0 + j) * WPI < 64)
          v[j] = *reinterpret_cast<const V*>(lsrc + (r0 + j) * WPI * SB);
#pragma unroll
      for (int j = 0; j < G; ++j)
        if (r0 + j < NIT && act && wl + (r0 + j) * WPI < nvalid)
          put_chunk<NT>(dst + (int64_t)(r0 + j) * WPI * gstride + lo, v[j]);
    }
  }
}

// Chunks of 16 bytes when the record length and LDS stride allow them and the destination and
// record stride are 16-byte aligned, 8 bytes for records that are 8- but not 16-byte multiples,
// 4-byte words otherwise. Without GENERAL only records that divide the wave (64 mod PER = 0) go
// in chunks. GENERAL (4-byte element types) also chunks the others, e.g. the 144-byte records of
// a 6 x 6 float covariance; the float64 recovery of the mixed-pair kernels, which spills heavily,
// returned wrong results for unchanged cases with it, so float64 keeps 4-byte words for them.
template <int RB, int SB, bool NT = false, bool GENERAL = false>
SRTM_DEV void flush_records(int lane, int nvalid, const char* __restrict__ lds, char* __restrict__ dst,
                            int64_t gstride) {
  const uintptr_t al = reinterpret_cast<uintptr_t>(dst) | (uintptr_t)gstride;
  if constexpr (RB % 16 == 0 && SB % 16 == 0 && RB / 16 <= 64 && (GENERAL || 64 % (RB / 16) == 0)) {
    if (al % 16 == 0) {
      flush_chunks<RB, SB, 16, NT>(lane, nvalid, lds, dst, gstride);
      return;
    }
  }
  if constexpr (RB % 16 != 0 && RB % 8 == 0 && SB % 8 == 0 && RB / 8 <= 64 && (GENERAL || 64 % (RB / 8) == 0)) {
    if (al % 8 == 0) {
      flush_chunks<RB, SB, 8, NT>(lane, nvalid, lds, dst, gstride);
      return;
    }
  }
  if constexpr (RB % 8 != 0 && 64 % (RB / 4) == 0) {  // whole records of 4-byte words per lane
    flush_chunks<RB, SB, 4, NT>(lane, nvalid, lds, dst, gstride);
    return;
  }
  for (int c = lane; c < nvalid * (RB / 4); c += 64) {  // 4-byte words
    const int w = c / (RB / 4), e = c - w * (RB / 4);
    put_global(reinterpret_cast<unsigned int*>(dst + w * gstride) + e,
               reinterpret_cast<const unsigned int*>(lds + w * SB)[e]);
  }
}

// Element-wise variant for a run-time record length (the last, partial group of means).
template <typename T>
SRTM_DEV void flush_records_rt(int lane, int nvalid, const char* __restrict__ lds, int SB, T* __restrict__ dst,
                               int64_t gstride_elems, int nel) {
  for (int c = lane; c < nvalid * nel; c += 64) {
    const int w = c / nel, e = c - w * nel;
    put_global(dst + w * gstride_elems + e, reinterpret_cast<const T*>(lds + w * SB)[e]);
  }
}

// Fast steps gathered into one output record: the largest power of two (at most 8) for
// which the record still fits in one 128-byte line.
constexpr int line_group(int bytes) {
  int g = 1;
  while (g < 8 && 2 * g * bytes <= 128) g *= 2;
  return g;
}

template <typename T, int NX>
struct OutStage {
  static constexpr int NN = NX * NX;
  static constexpr int GM = line_group(NX * (int)sizeof(T));   // means per record
  static constexpr int GP = line_group(NN * (int)sizeof(T));   // covariances per record
  static constexpr int RBM = GM * NX * (int)sizeof(T), RBP = GP * NN * (int)sizeof(T);
  static constexpr int SBP = ((RBP + 15) / 16) * 16 + 16;   // LDS bytes per lane (padded)
  static constexpr int SBM = ((RBM + 15) / 16) * 16 + 16;
  static constexpr int BYTES = 64 * (SBP + SBM);             // per wave
  char* pbuf;
  char* mbuf;
  SRTM_DEV OutStage(char* base) : pbuf(base), mbuf(base + 64 * SBP) {}
  // blocks of the workgroup's fast step ph (0-based)
  SRTM_DEV void put(int lane, int ph, const T (&m)[NX], const T (&P)[NX][NX]) const {
    T* pp = reinterpret_cast<T*>(pbuf + lane * SBP) + (ph % GP) * NN;
#pragma unroll
    for (int r = 0; r < NX; ++r)
#pragma unroll
      for (int c = 0; c < NX; ++c) pp[r * NX + c] = P[r][c];
    T* mp = reinterpret_cast<T*>(mbuf + lane * SBM) + (ph % GM) * NX;
#pragma unroll
    for (int r = 0; r < NX; ++r) mp[r] = m[r];
  }
  // After put(ph): flush the covariance and mean groups that it completes; ph is fast step i (1-based) and ilim
  // the workgroup's last. The record of window w0 + w for fast steps i0 .. i0+g-1 starts at
  // out[((w0 + w) L + i0 - 1) * size].
  SRTM_DEV void flush(int lane, int nvalid, T* m_out, T* P_out, int64_t w0, int L, int ph, int i, int ilim) const {
    const int sp = ph % GP, sm = ph % GM;
    if (P_out && (sp == GP - 1 || i == ilim)) {
      T* dst = P_out + (w0 * L + (i - sp - 1)) * NN;
      if (sp == GP - 1)
        flush_records<RBP, SBP, RBP % 128 == 0, sizeof(T) == 4>(lane, nvalid, pbuf, reinterpret_cast<char*>(dst),
                                                (int64_t)L * NN * sizeof(T));
      else
        flush_records_rt<T>(lane, nvalid, pbuf, SBP, dst, (int64_t)L * NN, (sp + 1) * NN);
    }
    if (m_out && (sm == GM - 1 || i == ilim)) {
      T* dst = m_out + (w0 * L + (i - sm - 1)) * NX;
      if (sm == GM - 1)
        flush_records<RBM, SBM, RBM % 128 == 0, sizeof(T) == 4>(lane, nvalid, mbuf, reinterpret_cast<char*>(dst),
                                                (int64_t)L * NX * sizeof(T));
      else
        flush_records_rt<T>(lane, nvalid, mbuf, SBM, dst, (int64_t)L * NX, (sm + 1) * NX);
    }
  }
  // slow-rate output: the blocks of fast step 1 (call right after put(1)), contiguous windows
  SRTM_DEV void flush_slow(int lane, int nvalid, T* m_out, T* P_out, int64_t w0) const {
    if (m_out)
      flush_records<NX * (int)sizeof(T), SBM, false, sizeof(T) == 4>(lane, nvalid, mbuf, reinterpret_cast<char*>(m_out + w0 * NX),
                                              (int64_t)NX * sizeof(T));
    if (P_out)
      flush_records<NN * (int)sizeof(T), SBP, false, sizeof(T) == 4>(lane, nvalid, pbuf, reinterpret_cast<char*>(P_out + w0 * NN),
                                              (int64_t)NN * sizeof(T));
  }
};

// A wave's place in the output [64 windows][L steps][RB bytes] of one element size when every window has the
// same records: the records of fast steps i0 .. i0 + ns - 1 lie in LDS one after the other (`tab`), and the
// wave writes them to all 64 windows front to back, 64 chunks (CH bytes each) per store instruction, so
// that its stores run through consecutive addresses. PER = RB / CH instructions are ns-th parts of it.
template <int RB>
struct Stream {
  static constexpr int CH = RB % 16 == 0 ? 16 : RB % 8 == 0 ? 8 : 4, PER = RB / CH;
  int r, n, dr;          // chunk within a window's ns records, their number, its advance per instruction
  unsigned off, dn, dw;  // byte offset, its advance and the extra when the window changes
  SRTM_DEV Stream(int lane, int ns, int L) {
    n = ns * PER;
    const int dq = 64 / n;
    dr = 64 - dq * n;
    const int w = lane / n;
    r = lane - w * n;
    const unsigned win = (unsigned)L * RB;
    off = w * win + r * CH;
    dn = dq * win + dr * CH;
    dw = win - (unsigned)n * CH;
  }
  SRTM_DEV void put(const char* tab, char* dst) {
    using V = typename Chunk<CH>::type;
    V v[PER];
    unsigned o[PER];
#pragma unroll
    for (int q = 0; q < PER; ++q) {
      v[q] = *reinterpret_cast<const V*>(tab + r * CH);
      o[q] = off;
      r += dr;
      off += dn;
      if (r >= n) {
        r -= n;
        off += dw;
      }
    }
#pragma unroll
    for (int q = 0; q < PER; ++q) put_chunk<true>(dst + o[q], v[q]);
  }
};

template <typename T, int NX>
SRTM_DEV bool finite_state(const T (&m)[NX], const T (&P)[NX][NX]) {
  bool ok = true;
#pragma unroll
  for (int r = 0; r < NX; ++r) {
    ok = ok && isfinite(m[r]);
#pragma unroll
    for (int c = r; c < NX; ++c) ok = ok && isfinite(P[r][c]);
  }
  return ok;
}

// Window k's filtered slow state (m^f_{k,l}, P^f_{k,l}) from its window quantities (window_setup
// on the exclusive state): the recovery's blocks at fast step l, m = A^l m' + c_l S^{-1} e (+ z_{k,l}
// with inputs) and P = A^l Y1 + Q_ll - c_l Y2 (upper triangle, mirrored). Equal to the inclusive
// combine X_{k-1} (x) a_k in exact arithmetic, at a fraction of its cost.
template <bool INP, typename T, int NX, int NY>
SRTM_DEV void window_slow_state(const Model<T, NX, NY>& M, int L, const Window<T, NX, NY>& w, const T (&zL)[NX],
                                T (&m)[NX], T (&P)[NX][NX]) {
  T AL[NX][NX], cL[NX][NY];
  M.get(AL, M.AL_off(L));
  M.get(cL, M.cL_off(L));
  const int oq = M.per_i_off(L) + M.lay.o_Qii;
#pragma unroll
  for (int r = 0; r < NX; ++r) {
    T t = INP ? zL[r] : T(0);
#pragma unroll
    for (int k = 0; k < NX; ++k) t = my_fma(AL[r][k], w.mp[k], t);
#pragma unroll
    for (int k = 0; k < NY; ++k) t = my_fma(cL[r][k], w.Se[k], t);
    m[r] = t;
  }
#pragma unroll
  for (int r = 0; r < NX; ++r)
#pragma unroll
    for (int c = r; c < NX; ++c) {
      T t = M.at(oq + r * NX + c);
#pragma unroll
      for (int k = 0; k < NX; ++k) t = my_fma(AL[r][k], w.Y1[k][c], t);
#pragma unroll
      for (int k = 0; k < NY; ++k) t = my_fma(-cL[r][k], w.Y2[k][c], t);
      P[r][c] = t;
      P[c][r] = t;
    }
}

// Writes window k's slow-rate filter outputs when requested; reports a state that is not finite.
template <typename T, int NX>
SRTM_DEV int store_slow(int64_t k, const T (&m)[NX], const T (&P)[NX][NX], T* __restrict__ m_slow,
                        T* __restrict__ P_slow) {
  constexpr int NN = NX * NX;
  if (m_slow) {
#pragma unroll
    for (int r = 0; r < NX; ++r) put_global(m_slow + k * NX + r, m[r]);
  }
  if (P_slow) {
#pragma unroll
    for (int r = 0; r < NN; ++r) put_global(P_slow + k * NN + r, P[r / NX][r % NX]);
  }
  return finite_state(m, P) ? 0 : SRTM_INFO_NONFINITE;
}

// Writes the slow-rate carry (m^f_{k,l}, P^f_{k,l}) of window k < N, and its slow-rate outputs.
template <typename T, int NX>
SRTM_DEV int store_carry(int64_t k, const T (&m)[NX], const T (&P)[NX][NX], T* __restrict__ carry,
                         T* __restrict__ m_slow, T* __restrict__ P_slow) {
  constexpr int NN = NX * NX, ST = NX + NN;
#pragma unroll
  for (int r = 0; r < NX; ++r) put_global(carry + k * ST + r, m[r]);
#pragma unroll
  for (int r = 0; r < NX; ++r)
#pragma unroll
    for (int c = 0; c < NX; ++c) put_global(carry + k * ST + NX + r * NX + c, P[r][c]);
  return store_slow(k, m, P, m_slow, P_slow);
}

// Smoother correction of window k (fold section): v = (I + J P)^{-1} (eta - J m), W = -(I + J P)^{-1} J, from its
// inclusive filter state (m, P) = (m^f_{k,l}, P^f_{k,l}) and its information record (columns `col` and
// `mcol` of a tile of nw windows, record_load; zero after the last window, which gives v = 0 and W = 0). `mean` (may be
// null) receives m. Returns false when I + J P is numerically singular.
// After a wide prior or with accurate measurements P is many times J^{-1}, and P^f_{i,l} multiplies what W and v lose:
// in float64 for both types, W exactly symmetric (a mean with its transpose), and for float64, which has no wider
// type, one step of iterative refinement of both solutions in waves with J P beyond REFINE_FROM (in all of them the
// recovery of 3000 windows at nx = 4 took 1 us more).
template <bool INP, typename T, int NX, int NY, typename S>
SRTM_DEV bool info_correction(const Model<T, NX, NY>& M, int L, const Window<T, NX, NY>& w, const T (&zL)[NX],
                              const S* __restrict__ col, const S* __restrict__ mcol, int nw, T (&v)[NX], T (&W)[NX][NX],
                              T* __restrict__ mean = nullptr) {
  double P[NX][NX], r[NX], J[NX][NX], A[NX][NX], Ai[NX][NX], x[NX], X[NX][NX];
  record_load(r, J, col, mcol, nw);
  {
    T m[NX], Pt[NX][NX];
    window_slow_state<INP>(M, L, w, zL, m, Pt);
    if (mean) {
#pragma unroll
      for (int i = 0; i < NX; ++i) put_global(mean + i, m[i]);
    }
#pragma unroll
    for (int i = 0; i < NX; ++i) {
#pragma unroll
      for (int k = 0; k < NX; ++k) {
        P[i][k] = (double)Pt[i][k];
        r[i] = fma(-J[i][k], (double)m[k], r[i]);  // eta and J m nearly cancel
      }
    }
  }
  mm(J, P, A);
  double big = 0.0;
#pragma unroll
  for (int i = 0; i < NX; ++i) {
#pragma unroll
    for (int k = 0; k < NX; ++k) big = fma(A[i][k], A[i][k], big);
    A[i][i] += 1.0;
  }
  const bool ok = inv_small(A, Ai);
  mv(Ai, r, x);
#pragma unroll
  for (int i = 0; i < NX; ++i)
#pragma unroll
    for (int c = 0; c < NX; ++c) {
      double t = 0.0;
#pragma unroll
      for (int k = 0; k < NX; ++k) t = fma(-Ai[i][k], J[k][c], t);
      X[i][c] = t;
    }
  if (sizeof(T) == 8 && __builtin_expect(__any(big > REFINE_FROM * REFINE_FROM), 0)) {
    auto refine = [&](const double (&b)[NX], double (&y)[NX]) {  // by the residual b - y - J (P y)
      double Py[NX], e[NX];
      mv(P, y, Py);
#pragma unroll
      for (int i = 0; i < NX; ++i) {
        double t = b[i] - y[i];
#pragma unroll
        for (int k = 0; k < NX; ++k) t = fma(-J[i][k], Py[k], t);
        e[i] = t;
      }
      mv_acc(Ai, e, y);
    };
    refine(r, x);
#pragma unroll
    for (int c = 0; c < NX; ++c) {
      double b[NX], y[NX];
#pragma unroll
      for (int i = 0; i < NX; ++i) {
        b[i] = -J[i][c];
        y[i] = X[i][c];
      }
      refine(b, y);
#pragma unroll
      for (int i = 0; i < NX; ++i) X[i][c] = y[i];
    }
  }
#pragma unroll
  for (int i = 0; i < NX; ++i) {
    v[i] = (T)x[i];
#pragma unroll
    for (int c = i; c < NX; ++c) W[i][c] = W[c][i] = (T)(0.5 * (X[i][c] + X[c][i]));
  }
  return ok;
}

// K3: the fold of one tile. Every window's exclusive filter state (m^f_{k-1,l}, P^f_{k-1,l}), its prior and
// the slow filter output of the window before, and (SMOOTH) the information of the windows after it, from the dyadic tree: the
// tile's own bits and the window's bits 4 .. 7 on the matrix cores, four 16-window groups per wave
// (the tile's bits are the same for all of them), the low four bits one lane per window.
// `want_last`: also the filter state after the last window when no lane stands for window N (N a multiple of
// TILE).
template <bool SMOOTH, bool INP, typename T, int NX, int NY>
SRTM_DEV void fold_body(const T* __restrict__ y, int64_t N, int L, int nlev, const T* __restrict__ cst,
                        const double* __restrict__ lev64, InputView<T> in,
                        const T* __restrict__ m0, const T* __restrict__ P0, const T* __restrict__ tagg,
                        const T* __restrict__ ttree, T* __restrict__ utree, const double* __restrict__ tail_g,
                        T* __restrict__ prior, T* __restrict__ m_slow, T* __restrict__ P_slow, T* __restrict__ rec,
                        int32_t* info, int64_t tile, bool want_last) {
  constexpr int NN = NX * NX, R2 = 2 * NX, IS = info_stride(NX), NZ = FoldLds<T, NX>::NZ, LB = lane_levels<NX>();
  constexpr bool B4 = blocks4<NX>();
  extern __shared__ char smraw[];
  const int tid = threadIdx.x, wv = tid >> 6, lane_id = tid & 63;
  const int64_t k = tile * TILE + tid;
  const int64_t nf = N >> LOG_TILE;            // whole tiles
  const int rem = (int)(N & (TILE - 1));       // windows of the partial last tile
  const bool ragged = tile == nf, single = N <= TILE;
  if (single) nlev = LOG_TILE;
  const int hb = ragged ? -1 : top_bit(tile ^ nf);
  const FoldLds<T, NX> lo(nlev);
  T* leaf = reinterpret_cast<T*>(smraw + lo.leaf);
  T* tree = reinterpret_cast<T*>(smraw + lo.tree);
  T* lane = reinterpret_cast<T*>(smraw + lo.lane);
  double* lev = reinterpret_cast<double*>(smraw + lo.lev);
  T* node = reinterpret_cast<T*>(smraw + lo.node);
  double* tail = reinterpret_cast<double*>(smraw + lo.tail) + (single ? wv * NZ * IS : 0);
  double* scratch = reinterpret_cast<double*>(smraw + lo.scratch) + wv * 64;
  const Model<T, NX, NY> M{cst, make_const_layout(NX, NY, L), in};
  int flag = 0;

  // ---- everything the fold reads, in one round of loads: all of them are issued before the first
  // is stored to LDS (one memory round trip instead of one per table)
  constexpr int NCH = TILE * R2 * (int)sizeof(T) / 16, PCH = (NCH + TILE - 1) / TILE;
  constexpr int PLV = B4 ? (MAXLEV * 48 + TILE - 1) / TILE : 1;
  u32x4 tv[PCH];
  const char* tsrc = reinterpret_cast<const char*>(utree + tile * (R2 * TILE));
#pragma unroll
  for (int i = 0; i < PCH; ++i) {
    const int q = i * TILE + tid;
    if (q < NCH) tv[i] = gld(reinterpret_cast<const u32x4*>(tsrc) + q);
  }
  T yt[NY], zL[NX];
  window_meas<INP>(M, y, k, N, yt, zL);
  const int nlv = B4 ? nlev * 48 : 0;
  double lvv[PLV];
  if constexpr (B4) {
#pragma unroll
    for (int i = 0; i < PLV; ++i) {
      const int q = i * TILE + tid;
      lvv[i] = q < nlv ? block_entry<T, NX>(cst, lev64, M.lay, q) : 0.0;
    }
  }
  T ndv = T(0);
  double tlv = 0.0;
  if (tid < FoldLds<T, NX>::MAXT * R2) {  // the tile's own nodes
    const int q = tid / R2, e = tid % R2;
    if (((tile >> q) & 1) || (SMOOTH && q < hb)) {
      const int64_t i = (tile >> q) ^ 1;
      ndv = q == 0 ? gld(tagg + i * R2 + e) : gld(ttree + (tile_level_off(nf, q) + i) * R2 + e);
    }
  }
  const int tl0 = ragged ? 0 : LOG_TILE, tln = !SMOOTH || single ? 0 : ragged ? LOG_TILE * IS : IS;
  if constexpr (SMOOTH) {  // the entries this tile can ask for
    if (tid < tln) tlv = gld(tail_g + (ragged ? 0 : (LOG_TILE + hb) * IS) + tid);
  }
  stage_lane_tables<T, NX>(cst, M.lay, B4 ? LB : nlev, lane, tid, TILE);
  {
    T d[NX], e[NX];
    fwd_element<INP>(M, yt, zL, d, e);
#pragma unroll
    for (int r = 0; r < NX; ++r) {
      leaf[r * TILE + tid] = d[r];
      leaf[(NX + r) * TILE + tid] = e[r];
    }
  }
#pragma unroll
  for (int i = 0; i < PCH; ++i) {
    const int q = i * TILE + tid;
    if (q < NCH) reinterpret_cast<u32x4*>(tree)[q] = tv[i];
  }
  if constexpr (B4) {
#pragma unroll
    for (int i = 0; i < PLV; ++i) {
      const int q = i * TILE + tid;
      if (q < nlv) lev[q] = lvv[i];
    }
  }
  if (tid < FoldLds<T, NX>::MAXT * R2) node[tid] = ndv;
  if (tid < tln) tail[tl0 * IS + tid] = tlv;
  __syncthreads();
  if constexpr (SMOOTH) {
    if (single) {  // each wave its own copy
      const bool ok = tail_chain<T, NX>(lev, lane, scratch, N, top_bit(N), [&](int p) {
        return p == 0 ? leaf + (rem ^ 1) : tree + tree_off(p) + ((rem >> p) ^ 1);
      }, TILE, tail);
      if (!ok) flag |= SRTM_INFO_COMBINE_SINGULAR;
      wave_sync();
    }
  }

  // ---- upper bits
  constexpr bool REF = sizeof(T) == 8;
  Belief<T, NX> fs, bs;  // filter state at the window's start; information after the window
  bool settled = false;  // the tile's covariances are the same for all of its windows
  int bl = ragged ? 0 : LB;  // the window's bits below bl take backward combines
  const int tq = top_bit(tile) > hb - 1 ? top_bit(tile) : hb - 1;  // top bit of the tile that is used
  if constexpr (B4) {
    const Block4 B(scratch);
    const bool in4 = B.r < NX && B.c < NX;
    const int g = wv * 4 + B.b, gr = rem >> 4;
    double fu = B.r < NX ? (double)gld(m0 + B.r) : 0.0;
    double fP = in4 ? 0.5 * ((double)gld(P0 + B.r * NX + B.c) + (double)gld(P0 + B.c * NX + B.r)) : 0.0;
    double bu = 0.0, bP = 0.0;
    int bw = LOG_TILE;  // the group's bits below bw take backward combines
    if (ragged) bw = g < gr ? LB + top_bit(g ^ gr) : 0;
    if constexpr (SMOOTH) {
      if (in4 && bw > 0) {
        const int a = B.r < B.c ? B.r : B.c, e = B.r < B.c ? B.c : B.r;
        bu = tail[bw * IS + B.r];
        bP = tail[bw * IS + NX + a * NX - a * (a - 1) / 2 + e - a];
      }
    }
    // The steps, highest bit first: the tile's bits that ask for a combine, then the group's four. The
    // operands of a step are read while the step before it runs.
    struct Step {
      double Tt, Dp, Jp, vd, ve;
      bool f, act;
    };
    auto fetch = [&](int p) {
      Step st;
      const T* nd;
      int ns = 1;
      if (p >= LOG_TILE) {
        st.f = (tile >> (p - LOG_TILE)) & 1;
        st.act = true;
        nd = node + (p - LOG_TILE) * R2;
      } else {
        const int i = g >> (p - LB);
        st.f = i & 1;
        st.act = st.f || (SMOOTH && p < bw);
        nd = tree + tree_off(p) + (i ^ 1);
        ns = TILE;
      }
      const double* lv = lev + p * 48;
      st.Tt = lv[st.f ? 4 * B.c + B.r : 4 * B.r + B.c];
      st.Dp = lv[(st.f ? 16 : 32) + 4 * B.r + B.c];
      st.Jp = lv[(st.f ? 32 : 16) + 4 * B.r + B.c];
      const double d = B.r < NX ? (double)nd[B.r * ns] : 0.0, e = B.r < NX ? (double)nd[(NX + B.r) * ns] : 0.0;
      st.vd = st.f ? d : e;
      st.ve = st.f ? e : -d;
      return st;
    };
    uint32_t todo = (uint32_t)tile << LOG_TILE;
    if (SMOOTH && hb > 0) todo |= ((1u << hb) - 1u) << LOG_TILE;
    auto run = [&](uint32_t bits) {
      int p = 31 - __builtin_clz(bits);
      Step cur = fetch(p);
#pragma unroll 1
      while (true) {
        bits &= ~(1u << p);
        p = bits ? 31 - __builtin_clz(bits) : LB;
        const Step next = fetch(p);
        double u = cur.f ? fu : bu, P = cur.f ? fP : bP;
        const bool ok = combine4<NX, REF>(B, u, P, cur.Tt, cur.Dp, cur.Jp, cur.vd, cur.ve);
        if (cur.act) {
          if (!ok) flag |= SRTM_INFO_COMBINE_SINGULAR;
          fu = cur.f ? u : fu;
          fP = cur.f ? P : fP;
          bu = cur.f ? bu : u;
          bP = cur.f ? bP : P;
        }
        if (!bits) break;
        cur = next;
      }
    };
    if (todo) run(todo);
    if (!ragged && !single) {  // settled? (every wave finds the same)
      // blocks 0, 1: P over one window and over a tile; blocks 2, 3: J
      const bool f = B.b < 2;
      const double* lv = lev + ((B.b & 1) ? LOG_TILE : 0) * 48;
      const double P = f ? fP : bP;
      double u = 0.0, P1 = P;
      const bool ok = combine4<NX, REF>(B, u, P1, lv[f ? 4 * B.c + B.r : 4 * B.r + B.c], lv[(f ? 16 : 32) + 4 * B.r + B.c],
                               lv[(f ? 32 : 16) + 4 * B.r + B.c], 0.0, 0.0);
      *B.own = P;
      wave_sync();
      const double dev = P1 - P, tol = settled_tol<T>();
      const bool same = ok && dev * dev <= tol * tol * (sld(B.base + 5 * B.r) * sld(B.base + 5 * B.c));
      wave_sync();
      settled = __all(same || (!SMOOTH && !f));
    }
    if (settled) {
      // Vectors only. Level p's forward gains (G, G P), G = F W with W = (I + P J)^{-1}, and backward ones: wave wv
      // forms those of levels 2 wv and 2 wv + 1, one per block.
      const int lvl = 2 * wv + (B.b >> 1);
      const bool f = (B.b & 1) == 0;
      const double* lv = lev + lvl * 48;
      const double P = f ? fP : bP;
      bool ok = true;
      const double Tt = lv[f ? 4 * B.c + B.r : 4 * B.r + B.c];
      const double Jp = lv[(f ? 32 : 16) + 4 * B.r + B.c], A = mm4(P, Jp, B.eye);
      const double Wt = B.template inv_t<NX>(A, ok);
      double W = mm4(Wt, B.eye, 0.0), X = Block4::mm_sym(Wt, P);
      if (REF && __any(fabs(A) > REFINE_FROM)) {
        const double E = mm4(P, -mm4(Jp, X, 0.0), P - X), e = mm4(P, -mm4(Jp, W, 0.0), B.eye - W);
        X = 0.5 * (mm4(Wt, E, X) + mm4(E, Wt, X));
        W = mm4(Wt, e, W);
      }
      const double G = mm4(Tt, W, 0.0), GP = mm4(Tt, X, 0.0);
      double* gain = reinterpret_cast<double*>(smraw + lo.gain);
      if (in4) {
        double* row = gain + ((lvl * 2 + (f ? 0 : 1)) * NX + B.r) * R2;
        row[B.c] = G;
        row[NX + B.c] = GP;
      }
      if (!ok && (SMOOTH || f)) flag |= SRTM_INFO_COMBINE_SINGULAR;
      double* grp = reinterpret_cast<double*>(smraw + lo.group) + wv * 160;
      if (B.b == 0) {
        grp[4 * B.r + B.c] = fP;
        grp[20 + 4 * B.r + B.c] = bP;
        if (B.c == 0) {
          grp[16 + B.r] = fu;
          grp[36 + B.r] = bu;
        }
      }
      __syncthreads();
      double fv[NX], bv[NX];  // float64 for both types: as many instructions, one rounding at the end
#pragma unroll
      for (int r = 0; r < NX; ++r) {
        fv[r] = grp[16 + r];
        bv[r] = grp[36 + r];
#pragma unroll
        for (int c = r; c < NX; ++c) {
          fs.P[r][c] = fs.P[c][r] = (T)grp[4 * r + c];
          bs.P[r][c] = bs.P[c][r] = (T)grp[20 + 4 * r + c];
        }
      }
#pragma unroll 1
      for (int p = LOG_TILE - 1; p >= 0; --p) {
        const bool fw = (tid >> p) & 1;
        if (SMOOTH || fw) {
          const int i = (tid >> p) ^ 1;
          const T* nd = p == 0 ? leaf + i : tree + tree_off(p) + i;
          const double* g = gain + (p * 2 + (fw ? 0 : 1)) * 2 * NN;
          double x[NX], ve[NX], nu[NX];
#pragma unroll
          for (int r = 0; r < NX; ++r) {
            const double d = (double)nd[r * TILE], e = (double)nd[(NX + r) * TILE];
            x[r] = fw ? fv[r] : bv[r];
            ve[r] = fw ? e : -d;
            nu[r] = fw ? d : e;
          }
#pragma unroll
          for (int r = 0; r < NX; ++r) {
#pragma unroll
            for (int c = 0; c < NX; ++c) {
              nu[r] = my_fma(g[r * R2 + c], x[c], nu[r]);
              nu[r] = my_fma(g[r * R2 + NX + c], ve[c], nu[r]);
            }
          }
#pragma unroll
          for (int r = 0; r < NX; ++r) {
            fv[r] = fw ? nu[r] : fv[r];
            bv[r] = fw ? bv[r] : nu[r];
          }
        }
      }
#pragma unroll
      for (int r = 0; r < NX; ++r) {
        fs.u[r] = (T)fv[r];
        bs.u[r] = (T)bv[r];
      }
    } else {
      run(0xF0u);
    // each group's states to its 16 lanes
    double* grp = reinterpret_cast<double*>(smraw + lo.group) + wv * 160;
    grp[B.b * 40 + 4 * B.r + B.c] = fP;
    if (B.c == 0) grp[B.b * 40 + 16 + B.r] = fu;
    if constexpr (SMOOTH) {
      grp[B.b * 40 + 20 + 4 * B.r + B.c] = bP;
      if (B.c == 0) grp[B.b * 40 + 36 + B.r] = bu;
    }
    wave_sync();
    const double* mine = grp + (lane_id >> 4) * 40;
#pragma unroll
    for (int r = 0; r < NX; ++r) {
      fs.u[r] = (T)mine[16 + r];
      bs.u[r] = SMOOTH ? (T)mine[36 + r] : T(0);
#pragma unroll
      for (int c = r; c < NX; ++c) {
        fs.P[r][c] = fs.P[c][r] = (T)mine[4 * r + c];
        bs.P[r][c] = bs.P[c][r] = SMOOTH ? (T)mine[20 + 4 * r + c] : T(0);
      }
    }
    if (ragged) {
      bl = (tid >> 4) < gr ? LB : 0;
      if (SMOOTH && (tid >> 4) == gr && tid < rem) {
        bl = top_bit(tid ^ rem);
        belief_load(bs, tail + bl * IS);
      }
    }
    }
  } else if constexpr (block8<NX>()) {
    const Block8<NX> B(scratch);
    const bool in = B.in();
    const int gr = rem >> LB;
    double fu = B.r < NX ? (double)gld(m0 + B.r) : 0.0;
    double fP = in ? 0.5 * ((double)gld(P0 + B.r * NX + B.c) + (double)gld(P0 + B.c * NX + B.r)) : 0.0;
    double bu = 0.0, bP = 0.0;
    int bw = LOG_TILE;  // the wave's bits below bw take backward combines
    if (ragged) bw = wv < gr ? LB + top_bit(wv ^ gr) : 0;
    if constexpr (SMOOTH) {
      if (in && bw > 0) {
        const int a = B.r < B.c ? B.r : B.c, e = B.r < B.c ? B.c : B.r;
        bP = tail[bw * IS + NX + a * NX - a * (a - 1) / 2 + e - a];
      }
      if (bw > 0 && B.r < NX) bu = tail[bw * IS + B.r];  // equal columns, the padding ones too
    }
#pragma unroll 1
    for (int p = LOG_TILE + tq; p >= LB; --p) {  // the tile's bits, then the wave's
      const bool low = p < LOG_TILE;
      const int64_t i = low ? (int64_t)(wv >> (p - LB)) : tile >> (p - LOG_TILE);
      const bool f = i & 1;
      if (!f && !(SMOOTH && p < (low ? bw : LOG_TILE + hb))) continue;
      double u = f ? fu : bu, P = f ? fP : bP;
      const T* nd = low ? tree + tree_off(p) + (i ^ 1) : node + (p - LOG_TILE) * R2;
      if (!wave_combine(B, u, P, lane + (size_t)p * 6 * NN, nd, low ? TILE : 1, f)) flag |= SRTM_INFO_COMBINE_SINGULAR;
      fu = f ? u : fu;
      fP = f ? P : fP;
      bu = f ? bu : u;
      bP = f ? bP : P;
    }
    // the wave's states to its lanes
    double* grp = reinterpret_cast<double*>(smraw + lo.group) + wv * 2 * (NN + NX);
    if (in) {
      grp[B.r * NX + B.c] = fP;
      grp[NN + NX + B.r * NX + B.c] = bP;
      if (B.c == 0) {
        grp[NN + B.r] = fu;
        grp[2 * NN + NX + B.r] = bu;
      }
    }
    wave_sync();
#pragma unroll
    for (int r = 0; r < NX; ++r) {
      fs.u[r] = (T)grp[NN + r];
      bs.u[r] = SMOOTH ? (T)grp[2 * NN + NX + r] : T(0);
#pragma unroll
      for (int c = r; c < NX; ++c) {
        fs.P[r][c] = fs.P[c][r] = (T)grp[r * NX + c];
        bs.P[r][c] = bs.P[c][r] = SMOOTH ? (T)grp[NN + NX + r * NX + c] : T(0);
      }
    }
    if (ragged) {
      bl = wv < gr ? LB : 0;
      if (SMOOTH && wv == gr && tid < rem) {
        bl = top_bit(tid ^ rem);
        belief_load(bs, tail + bl * IS);
      }
    }
  } else {
    gloadv(fs.u, m0);
    gload(fs.P, P0);
    symmetrize(fs.P);
    belief_zero(bs);
    if constexpr (SMOOTH) {
      if (ragged && tid < rem) bl = top_bit(tid ^ rem);
      if (!ragged || tid < rem) belief_load(bs, tail + bl * IS);
    }
#pragma unroll 1
    for (int q = tq; q >= 0; --q) {
      const bool f = (tile >> q) & 1;
      if (!f && !(SMOOTH && q < hb)) continue;
      Belief<T, NX> x;
#pragma unroll
      for (int r = 0; r < NX; ++r) {
        x.u[r] = f ? fs.u[r] : bs.u[r];
#pragma unroll
        for (int c = 0; c < NX; ++c) x.P[r][c] = f ? fs.P[r][c] : bs.P[r][c];
      }
      if (!lane_combine(x, lane + (size_t)(LOG_TILE + q) * 6 * NN + (f ? 0 : 3 * NN), node + q * R2, 1, f))
        flag |= SRTM_INFO_COMBINE_SINGULAR;
      if (f) fs = x;
      else bs = x;
    }
  }

  // ---- the low bits, one lane per window
#pragma unroll 1
  for (int p = settled ? -1 : LB - 1; p >= 0; --p) {
    const bool f = (tid >> p) & 1;
    const bool act = f || (SMOOTH && p < bl);
    const int i = (tid >> p) ^ 1;
    const T* nd = p == 0 ? leaf + i : tree + tree_off(p) + i;
    if (SMOOTH || f) {
      Belief<T, NX> x;
#pragma unroll
      for (int r = 0; r < NX; ++r) {
        x.u[r] = f ? fs.u[r] : bs.u[r];
#pragma unroll
        for (int c = 0; c < NX; ++c) x.P[r][c] = f ? fs.P[r][c] : bs.P[r][c];
      }
      const bool ok = lane_combine(x, lane + (size_t)p * 6 * NN + (f ? 0 : 3 * NN), nd, TILE, f);
      if (act && !ok) flag |= SRTM_INFO_COMBINE_SINGULAR;
#pragma unroll
      for (int r = 0; r < NX; ++r) {
        fs.u[r] = f ? x.u[r] : fs.u[r];
        bs.u[r] = act && !f ? x.u[r] : bs.u[r];
#pragma unroll
        for (int c = 0; c < NX; ++c) {
          fs.P[r][c] = f ? x.P[r][c] : fs.P[r][c];
          bs.P[r][c] = act && !f ? x.P[r][c] : bs.P[r][c];
        }
      }
    }
  }

  // ---- outputs: the window's prior and information records; the slow filter output of the window
  // before. The windows of a settled tile share the first window's matrices.
  const int nw = tile_windows(N, tile);
  T* prec = prior + tile * (TILE * IS) + tid;
  if (tid == 0) put_global(settled_flag<T, NX>(utree, tile), settled ? T(1) : T(0));
  if (k >= 1 && k <= N) flag |= store_slow(k - 1, fs.u, fs.P, m_slow, P_slow);
  const bool whole = !settled || tid == 0;
  if (k < N) record_store(fs.u, fs.P, prec, nw, whole);
  if constexpr (SMOOTH) {
    if (k < N) {
      record_store(bs.u, bs.P, rec + tile * (TILE * IS) + tid, nw, whole);
      // the prediction of x_{k,1}: P^- = A P A^T + Q has to be positive definite
      if (settled ? wv == 0 : k >= 1) {
        T A[NX][NX], Qm[NX][NX], Pm[NX][NX], Pi[NX][NX];
        load(A, M.cst + M.lay.A);
        load(Qm, M.cst + M.lay.Q);
        sandwich(A, fs.P, Qm, Pm);
        if (!spd_inv(Pm, Pi) && k >= 1) flag |= SRTM_INFO_PRED_SINGULAR;
      }
    }
  }
  if (want_last && k == N - 1 && rem == 0) {
    if (!lane_combine(fs, lane, leaf + tid, TILE, true)) flag |= SRTM_INFO_COMBINE_SINGULAR;
    flag |= store_slow(k, fs.u, fs.P, m_slow, P_slow);
  }
  if (flag && info) atomicOr(info, flag);
}

// ============================================================================ backward
// The smoother half of the per-window models' fused forward/backward kernel for window k of tile `tile`,
// given the window quantities w (window_setup on the exclusive filter state), the inclusive filter state
// (m, P) and (An, Qn), the model of the step into x_{k+1,1}: its smoother element (eq.
// parallel-ak-smoothing), the in-tile reverse scan under eq. op-smoother, the tile aggregate
// a_first (x) ... (x) a_last, and per window the smoother correction of eq. seq-smoothing-all written as terms
// linear in the smoothed state (m_in, P_in) that enters the tile from the right (the first window after
// it). With B = (P^-)^{-1} A and the in-tile exclusive suffix (E', g', S') = a_{k+1} (x) ... (x) a_{last of tile}:
//   v = A^T (P^-)^{-1} (m^s_{k+1,1} - A m^f_{k,l}) = Et m_in + gt,
//   W = A^T (P^-)^{-1} (P^s_{k+1,1} - P^-) (P^-)^{-1} A = Et P_in Et^T + St,
//   Et = B^T E',  gt = B^T (g' - A m^f_{k,l}),  St = B^T (S' - P^-) B;
// all three are zero for the last window, whose smoothed blocks equal the filtered ones. Returns
// numerical status bits.
template <bool INP, typename T, int NX, int NY, class MV>
SRTM_DEV int smoother_part(const MV& M, const Slots<T>& S, int L, int64_t k, int64_t N,
                           const Window<T, NX, NY>& w, const T (&m)[NX], const T (&P)[NX][NX],
                           const T (&An)[NX][NX], const T (&Qn)[NX][NX], T* __restrict__ btagg,
                           T* __restrict__ sfx, int64_t tile) {
  constexpr int NN = NX * NX, SE = 2 * NN + NX, SF = sfx_stride(NX);
  const int tid = threadIdx.x;
  const bool valid = k < N;
  int flag = 0;
  SElem<T, NX> x;
  T B[NX][NX], Bm[NX], BPB[NX][NX];  // B = (P^-)^{-1} A, B^T (predicted mean), B^T P^- B = A^T B
  {
    T z1[NX], bnext[NX];  // B u_{k,0} and B u_{k+1,0}
#pragma unroll
    for (int r = 0; r < NX; ++r) z1[r] = bnext[r] = T(0);
    if constexpr (INP) {
      if (valid) input_drive(M.in, M.in.u + k * L * M.in.nu, z1);
      if (k + 1 < N) input_drive(M.in, M.in.u + (k + 1) * L * M.in.nu, bnext);
    }
    T Pmi[NX][NX], mpred[NX], Pm[NX][NX];
    const int f = smoother_element<INP>(M, L, w, k == N - 1, m, P, z1, bnext, An, Qn, x, Pmi, mpred, Pm);
    if (valid) flag |= f;
    mm(Pmi, An, B);
    mtv(B, mpred, Bm);
#pragma unroll
    for (int r = 0; r < NX; ++r)
#pragma unroll
      for (int c = r; c < NX; ++c) {
        T t = T(0);
#pragma unroll
        for (int q = 0; q < NX; ++q) t = my_fma(An[q][r], B[q][c], t);
        BPB[r][c] = t;
        BPB[c][r] = t;
      }
  }
  if (!valid) {  // past the last window: a zero element (finite, and absorbed by E_N = 0)
#pragma unroll
    for (int r = 0; r < NX; ++r) {
      x.g[r] = T(0);
#pragma unroll
      for (int c = 0; c < NX; ++c) {
        x.E[r][c] = T(0);
        x.S[r][c] = T(0);
      }
    }
  }
  // Lane j ends with a_j (x) a_{j+1} (x) ... (x) a_{TILE-1}. Within each wave first, by lane
  // shuffles at distances 1 .. 32: lane l then holds its wave's elements l .. 63 merged, and lane
  // 0 the whole wave's. Then each wave merges with the aggregates of the waves after it, which
  // pass through LDS (runs of any length merge: eq. op-smoother carries whole matrices).
  {
    const int lane = tid & 63, wv = tid >> 6;
    constexpr int NW = TILE / 64;
#pragma unroll 1
    for (int s = 1; s < 64; s *= 2) selem_merge_lane<true>(x, s, lane + s < 64);
    __syncthreads();  // the slots switch from forward states to smoother elements
    if (lane == 0) st_selem(S, wv, x);
    __syncthreads();
#pragma unroll 1
    for (int v = wv + 1; v < NW; ++v) {  // x (x) A_{wv+1} (x) ... (x) A_{NW-1}, left to right
      SElem<T, NX> a;
      ld_selem(S, v, a);
      selem_combine(x, a, x);
    }
    __syncthreads();  // the aggregates are read before the slots take the suffixes
  }
  st_selem(S, tid, x);
  __syncthreads();
  if (tid == 0) {
    T* dst = btagg + tile * SE;
#pragma unroll
    for (int r = 0; r < NX; ++r) {
      dst[NN + r] = x.g[r];
#pragma unroll
      for (int c = 0; c < NX; ++c) {
        dst[r * NX + c] = x.E[r][c];
        dst[NN + NX + r * NX + c] = x.S[r][c];
      }
    }
  }
  SElem<T, NX> nxt;  // exclusive suffix; the identity (I, 0, 0) for the tile's last lane
  if (tid + 1 < TILE) {
    ld_selem(S, tid + 1, nxt);
  } else {
#pragma unroll
    for (int r = 0; r < NX; ++r) {
      nxt.g[r] = T(0);
#pragma unroll
      for (int c = 0; c < NX; ++c) {
        nxt.E[r][c] = (r == c) ? T(1) : T(0);
        nxt.S[r][c] = T(0);
      }
    }
  }
  if (valid) {
    T rec[SF];
    if (k < N - 1) {
      T SB[NX][NX];
      mm(nxt.S, B, SB);
#pragma unroll
      for (int r = 0; r < NX; ++r) {
        T t = -Bm[r];
#pragma unroll
        for (int q = 0; q < NX; ++q) t = my_fma(B[q][r], nxt.g[q], t);
        rec[NN + r] = t;
#pragma unroll
        for (int c = 0; c < NX; ++c) {
          T e = T(0);
#pragma unroll
          for (int q = 0; q < NX; ++q) e = my_fma(B[q][r], nxt.E[q][c], e);
          rec[r * NX + c] = e;
        }
      }
      int o = NN + NX;
#pragma unroll
      for (int r = 0; r < NX; ++r)
#pragma unroll
        for (int c = r; c < NX; ++c) {
          T t = -BPB[r][c];
#pragma unroll
          for (int q = 0; q < NX; ++q) t = my_fma(B[q][r], SB[q][c], t);
          rec[o++] = t;
        }
    } else {
#pragma unroll
      for (int r = 0; r < SF; ++r) rec[r] = T(0);
    }
    T* dst = sfx + k * SF;
#pragma unroll
    for (int r = 0; r < SF; ++r) put_global(dst + r, rec[r]);
  }
  return flag;
}

// ---------------------------------------------------------------- float32 gradient: scan of smoother elements
// The sums of the gradient nearly vanish near the data's own parameters, so a float32 gradient carries the
// rounding of the float32 states magnified: on one model of the gradient workload (nx = 4, ny = 1, L = 10,
// N = 2^14) it is 7e-5 off the float64 gradient here and 6e-6 through the fold. The entry point keeps the values
// it has had, so float32 gradients still take the states and corrections from this scan (k_fwd_tiles,
// k_fwd_bwd, k_bwd_tiles); float64 gradients, where both agree to 1e-12, and everything else use the fold.
template <typename T> constexpr bool grad_by_elements() { return std::is_same_v<T, float>; }

// Vector part of eq. op-filter for two runs of 2^p elements (the level's row table).
template <typename T, int NX>
SRTM_DEV void level_vec_combine(const T* __restrict__ lev, const ConstLayout& lay, const T (&di)[NX],
                                const T (&ei)[NX], T (&dj)[NX], T (&ej)[NX]) {
  const T* C = lev + lay.o_C;
  T nd[NX], ne[NX];
#pragma unroll
  for (int r = 0; r < NX; ++r) {
    T s = dj[r], t = ei[r];
#pragma unroll
    for (int k = 0; k < NX; ++k) {
      s = my_fma(C[r * 2 * NX + k], di[k], s);
      s = my_fma(C[r * 2 * NX + NX + k], ej[k], s);
      t = my_fma(C[(NX + r) * 2 * NX + k], ej[k], t);
      t = my_fma(C[(NX + r) * 2 * NX + NX + k], di[k], t);
    }
    nd[r] = s;
    ne[r] = t;
  }
#pragma unroll
  for (int r = 0; r < NX; ++r) {
    dj[r] = nd[r];
    ej[r] = ne[r];
  }
}

// Tile-level forward scan in one workgroup of KS threads. Thread tau
// holds the vector parts of its chunk of 2^lchunk tiles (matrices Theta(2^lchunk TILE)); the
// prior (m0, P0) is folded into thread 0, which makes it a state. At step q, threads in
// [2^q, 2^{q+1}) combine the state of thread tau - 2^q with their run (one state combine,
// eq. op-filter with F_i = 0) and become states; the others merge two runs of equal length
// with the shared level coefficients. Thread tau then walks its chunk from its exclusive
// state, writing each tile's incoming state.
template <typename T, int NX, int NY>
SRTM_DEV void fwd_tiles_body(const T* __restrict__ tagg, int64_t nt, int lchunk, int steps, int nlev,
                             const T* __restrict__ cst, int L, const T* __restrict__ m0, const T* __restrict__ P0,
                             T* __restrict__ tstate, int32_t* info) {
  constexpr int NN = NX * NX, ST = NX + NN;
  extern __shared__ char smraw[];
  const Slots<T> S{reinterpret_cast<T*>(smraw), KS};
  const Model<T, NX, NY> M{cst, make_const_layout(NX, NY, L)};
  const int tid = threadIdx.x;
  const int64_t c = int64_t(1) << lchunk;
  const int64_t t0 = tid * c;
  int flag = 0;
  const int l0 = LOG_TILE + lchunk;
  // The level records this scan uses (LOG_TILE .. nlev-1) are copied to LDS behind the slots
  // first, so that no step waits on a memory round trip for its coefficients.
  T* slev = reinterpret_cast<T*>(smraw) + KS * (NX + NN);
  {
    const T* gl = M.level(LOG_TILE);
    const int n = (nlev - LOG_TILE) * M.lay.lev_stride;
    for (int q = tid; q < n; q += KS) slev[q] = gld(gl + q);
  }
  auto level = [&](int p) { return slev + (p - LOG_TILE) * M.lay.lev_stride; };
  T d[NX], e[NX];
  T d0[NX], e0[NX];  // vector parts of tile t0 (c = 2), reused by the walk at the end
  if (c == 1) {
#pragma unroll
    for (int r = 0; r < NX; ++r) {
      d[r] = (t0 < nt) ? gld(tagg + t0 * 2 * NX + r) : T(0);
      e[r] = (t0 < nt) ? gld(tagg + t0 * 2 * NX + NX + r) : T(0);
    }
  } else if (c == 2) {  // two runs of 2^LOG_TILE windows: vector parts only
#pragma unroll
    for (int r = 0; r < NX; ++r) {
      d[r] = (t0 + 1 < nt) ? gld(tagg + (t0 + 1) * 2 * NX + r) : T(0);
      e[r] = (t0 + 1 < nt) ? gld(tagg + (t0 + 1) * 2 * NX + NX + r) : T(0);
    }
#pragma unroll
    for (int r = 0; r < NX; ++r) {
      d0[r] = (t0 < nt) ? gld(tagg + t0 * 2 * NX + r) : T(0);
      e0[r] = (t0 < nt) ? gld(tagg + t0 * 2 * NX + NX + r) : T(0);
    }
    __syncthreads();  // the level copy is complete
    level_vec_combine(level(LOG_TILE), M.lay, d0, e0, d, e);
  } else {  // fold the chunk with full combines (tiles past the end carry zero vectors)
    __syncthreads();  // the level copy is complete
    const T* lv = level(LOG_TILE);
    FElem<T, NX> acc, b;
    load(b.F, lv + M.lay.o_F);
    load(b.D, lv + M.lay.o_D);
    load(b.J, lv + M.lay.o_J);
#pragma unroll 1
    for (int64_t j = 0; j < c; ++j) {
      const int64_t t = t0 + j;
#pragma unroll
      for (int r = 0; r < NX; ++r) {
        b.d[r] = (t < nt) ? tagg[t * 2 * NX + r] : T(0);
        b.e[r] = (t < nt) ? tagg[t * 2 * NX + NX + r] : T(0);
      }
      if (j == 0) {
        acc = b;
      } else if (!elem_combine(acc, b, acc)) {
        flag |= SRTM_INFO_COMBINE_SINGULAR;
      }
    }
#pragma unroll
    for (int r = 0; r < NX; ++r) {
      d[r] = acc.d[r];
      e[r] = acc.e[r];
    }
  }
  if (c == 1) __syncthreads();  // the level copy is complete
  T m[NX], P[NX][NX];
  if (tid == 0) {
    gloadv(m, m0);
    gload(P, P0);
    symmetrize(P);
    const T* lv = level(l0);
    T F[NX][NX], D[NX][NX], J[NX][NX];
    load(F, lv + M.lay.o_F);
    load(D, lv + M.lay.o_D);
    load(J, lv + M.lay.o_J);
    if (!state_combine(m, P, F, d, D, e, J)) flag |= SRTM_INFO_COMBINE_SINGULAR;
  }
  // While 2s < 64, wave 0 holds both the lanes [s, 2s) that form states and lanes [2s, 64) that
  // merge vector runs, and would run both combines one after the other. The vector runs of those
  // lanes are kept by lane tid - 64 of wave 1 instead (its second vector combine of the step):
  // the helper writes the run into the slot at the next step's start, and the owner reads it back
  // from there when it becomes a state. Barriers are unchanged.
  const bool helper = tid >= 64 && tid < 128;
  const int hl = tid - 64;  // the chunk a helper keeps
  T hd[NX], he[NX];         // its run
#pragma unroll 1
  for (int q = 0; q < steps; ++q) {
    const int s = 1 << q;
    const bool kept_prev = q >= 1 && s <= 32;  // the previous step kept the runs of [s, 64)
    const bool keep_now = 2 * s < 64;          // this step keeps the runs of [2s, 64)
    if (tid < s) {
      st_state<T, NX>(S, tid, m, P);
    } else if (!(tid < 64 && kept_prev)) {
#pragma unroll
      for (int r = 0; r < NX; ++r) {
        S.at(r, tid) = d[r];
        S.at(NX + r, tid) = e[r];
      }
    }
    if (helper && kept_prev && hl >= s) {
#pragma unroll
      for (int r = 0; r < NX; ++r) {
        S.at(r, hl) = hd[r];
        S.at(NX + r, hl) = he[r];
      }
    }
    __syncthreads();
    const bool gets_state = tid >= s && tid < 2 * s;
    const bool own_vec = tid >= 2 * s && !(tid < 64 && keep_now);
    const bool helps = helper && keep_now && hl >= 2 * s;
    T mo[NX], Po[NX][NX], dl[NX], el[NX], hdl[NX], hel[NX];
    if (gets_state) {
      ld_state<T, NX>(S, tid - s, mo, Po);
      if (tid < 64 && kept_prev) {  // the run its helper kept
#pragma unroll
        for (int r = 0; r < NX; ++r) {
          d[r] = S.at(r, tid);
          e[r] = S.at(NX + r, tid);
        }
      }
    } else if (own_vec) {
#pragma unroll
      for (int r = 0; r < NX; ++r) {
        dl[r] = S.at(r, tid - s);
        el[r] = S.at(NX + r, tid - s);
      }
    }
    if (helps) {
#pragma unroll
      for (int r = 0; r < NX; ++r) {
        hdl[r] = S.at(r, hl - s);
        hel[r] = S.at(NX + r, hl - s);
        if (q == 0) {  // the owner's own run, stored above
          hd[r] = S.at(r, hl);
          he[r] = S.at(NX + r, hl);
        }
      }
    }
    __syncthreads();
    const T* lv = level(l0 + q);
    if (gets_state) {
      T F[NX][NX], D[NX][NX], J[NX][NX];
      load(F, lv + M.lay.o_F);
      load(D, lv + M.lay.o_D);
      load(J, lv + M.lay.o_J);
      if (!state_combine(mo, Po, F, d, D, e, J)) flag |= SRTM_INFO_COMBINE_SINGULAR;
#pragma unroll
      for (int r = 0; r < NX; ++r) {
        m[r] = mo[r];
#pragma unroll
        for (int cc = 0; cc < NX; ++cc) P[r][cc] = Po[r][cc];
      }
    } else if (own_vec) {
      level_vec_combine(lv, M.lay, dl, el, d, e);
    }
    if (helps) level_vec_combine(lv, M.lay, hdl, hel, hd, he);
  }
  // every active thread now holds the inclusive state through its chunk
  st_state<T, NX>(S, tid, m, P);
  __syncthreads();
  if (t0 < nt) {
    T X[NX], XP[NX][NX];
    if (tid == 0) {
      gloadv(X, m0);
      gload(XP, P0);
      symmetrize(XP);
    } else {
      ld_state<T, NX>(S, tid - 1, X, XP);
    }
    const T* lv = level(LOG_TILE);
    T F[NX][NX], D[NX][NX], J[NX][NX];
    load(F, lv + M.lay.o_F);
    load(D, lv + M.lay.o_D);
    load(J, lv + M.lay.o_J);
#pragma unroll 1
    for (int64_t t = t0; t < t0 + c && t < nt; ++t) {
#pragma unroll
      for (int r = 0; r < NX; ++r) tstate[t * ST + r] = X[r];
#pragma unroll
      for (int r = 0; r < NX; ++r)
#pragma unroll
        for (int cc = 0; cc < NX; ++cc) tstate[t * ST + NX + r * NX + cc] = XP[r][cc];
      if (t + 1 < t0 + c && t + 1 < nt) {
        T dt[NX], et[NX];
        if (c == 2) {
#pragma unroll
          for (int r = 0; r < NX; ++r) {
            dt[r] = d0[r];
            et[r] = e0[r];
          }
        } else {
          gloadv(dt, tagg + t * 2 * NX);
          gloadv(et, tagg + t * 2 * NX + NX);
        }
        if (!state_combine(X, XP, F, dt, D, et, J)) flag |= SRTM_INFO_COMBINE_SINGULAR;
      }
    }
  }
  if (flag && info) atomicOr(info, flag);
}

// Per tile, every window's exclusive state (m^f_{k-1,l}, P^f_{k-1,l}): the tile's incoming state followed by the runs
// of the set bits of the window's place in the tile, highest first (the siblings in the tile's tree `ut`, and
// the elements themselves at level 0). `sm`: 4 nx TILE scalars of LDS.
template <bool INP, typename T, int NX, int NY>
SRTM_DEV int fwd_tile_states(const Model<T, NX, NY>& M, T* sm, const T (&yt)[NY], const T (&zL)[NX],
                             int64_t k, const T* __restrict__ m0, const T* __restrict__ P0,
                             const T* __restrict__ tile_state, const T* __restrict__ ut, T (&mprev)[NX],
                             T (&Pprev)[NX][NX]) {
  constexpr int R2 = 2 * NX;
  const int tid = threadIdx.x;
  int flag = 0;
  T* leaf = sm;
  T* tree = sm + R2 * TILE;
  for (int q = tid; q < TILE * R2; q += TILE) tree[q] = gld(ut + q);
  {
    T d[NX], e[NX];
    fwd_element<INP>(M, yt, zL, d, e);
#pragma unroll
    for (int r = 0; r < NX; ++r) {
      leaf[r * TILE + tid] = d[r];
      leaf[(NX + r) * TILE + tid] = e[r];
    }
  }
  if (k == 0) {  // the prior itself
    gloadv(mprev, m0);
    gload(Pprev, P0);
  } else {
    gloadv(mprev, tile_state);
    gload(Pprev, tile_state + NX);
  }
  symmetrize(Pprev);
  __syncthreads();
#pragma unroll
  for (int p = LOG_TILE - 1; p >= 0; --p) {
    if ((tid >> p) & 1) {
      const int i = (tid >> p) ^ 1;
      const T* nd = p == 0 ? leaf + i : tree + tree_off(p > 0 ? p : 1) + i;
      T dl[NX], el[NX];
#pragma unroll
      for (int r = 0; r < NX; ++r) {
        dl[r] = nd[r * TILE];
        el[r] = nd[(NX + r) * TILE];
      }
      const T* lv = M.level(p);
      T F[NX][NX], D[NX][NX], J[NX][NX];
      load(F, lv + M.lay.o_F);
      load(D, lv + M.lay.o_D);
      load(J, lv + M.lay.o_J);
      if (!state_combine(mprev, Pprev, F, dl, D, el, J)) flag |= SRTM_INFO_COMBINE_SINGULAR;
    }
  }
  return flag;
}

// Per tile: the exclusive filter states, the carry, and the smoother half (smoother_part).
template <bool INP, typename T, int NX, int NY>
SRTM_DEV void fwd_bwd_body(const T* __restrict__ y, int64_t N, int L, const T* __restrict__ cst, InputView<T> in,
                           const T* __restrict__ m0, const T* __restrict__ P0, const T* __restrict__ ftstate,
                           const T* __restrict__ utree, T* __restrict__ carry, T* __restrict__ btagg, T* __restrict__ sfx, int32_t* info, int64_t tile) {
  constexpr int ST = NX + NX * NX;
  extern __shared__ char smraw[];
  const Model<T, NX, NY> M{cst, make_const_layout(NX, NY, L), in};
  const Slots<T> S{reinterpret_cast<T*>(smraw), TILE};
  const int tid = threadIdx.x;
  const int64_t k = tile * TILE + tid;
  const bool valid = k < N;
  T yt[NY], zL[NX];
  window_meas<INP>(M, y, k, N, yt, zL);
  T mprev[NX], Pprev[NX][NX], m[NX], P[NX][NX];
  int flag = fwd_tile_states<INP>(M, S.base, yt, zL, k, m0, P0, ftstate + tile * ST, utree + tile * (2 * NX * TILE), mprev,
                                  Pprev);
  // The smoother element needs the window quantities of the exclusive state; the inclusive state
  // (the carry) follows from them.
  Window<T, NX, NY> w;
  if (!window_setup(M, L, mprev, Pprev, yt, w) && valid) flag |= SRTM_INFO_INNOVATION_NOT_PD;
  window_slow_state<INP>(M, L, w, zL, m, P);
  if (valid) flag |= store_carry<T, NX>(k, m, P, carry, nullptr, nullptr);

  T An[NX][NX], Qn[NX][NX];  // time-invariant: the step into x_{k+1,1} has the model's A and Q
  load(An, M.cst + M.lay.A);
  load(Qn, M.cst + M.lay.Q);
  flag |= smoother_part<INP>(M, S, L, k, N, w, m, P, An, Qn, btagg, sfx, tile);
  if (flag && info) atomicOr(info, flag);
}

// Per-window models in the recovery: the tile's A, Q and C (the caller's per-window F, Q, H)
// copied to LDS window-minor, entry j of window w at mdl[(j * TV_MS) + w] (j < nx^2: A, then Q,
// then C), with a padded column count so that the row-major reads of the copy spread over the
// banks. Windows past the end of the sequence get zeros.
constexpr int TV_MS = TILE + 1;
template <typename T, int NX, int NY>
constexpr size_t tv_model_lds_bytes() { return sizeof(T) * (size_t)(2 * NX * NX + NY * NX) * TV_MS; }

template <typename T, int NX, int NY>
SRTM_DEV void tv_model_to_lds(const T* __restrict__ Fa, const T* __restrict__ Qa, const T* __restrict__ Ha,
                              int64_t t0, int nw, T* mdl) {
  constexpr int NN = NX * NX, NXY = NX * NY;
  for (int q = threadIdx.x; q < TILE * NN; q += TILE) {
    const int w = q / NN, j = q % NN;
    mdl[j * TV_MS + w] = (w < nw) ? gld(Fa + t0 * NN + q) : T(0);
    mdl[(NN + j) * TV_MS + w] = (w < nw) ? gld(Qa + t0 * NN + q) : T(0);
  }
  for (int q = threadIdx.x; q < TILE * NXY; q += TILE) {
    const int w = q / NXY, j = q % NXY;
    mdl[(2 * NN + j) * TV_MS + w] = (w < nw) ? gld(Ha + t0 * NXY + q) : T(0);
  }
}

// The model view of window k: the call's constants block, or (TV) the window's own block with
// its A, Q and C from the tile's LDS copy `mdl` (per-window models: `cst` holds the blocks).
template <bool TV, typename T, int NX, int NY>
SRTM_DEV auto recover_model(const T* __restrict__ cst, int L, const InputView<T>& in, const T* mdl, int64_t k) {
  if constexpr (TV) {
    constexpr int NN = NX * NX;
    const int w = (int)(k % TILE);
    return TvModel<T, NX, NY, true>{tv_tile_base(cst, k, tv_block_size(NX, NY, L)), make_tv_layout(NX, NY, L), w,
                                    mdl + w, mdl + NN * TV_MS + w, mdl + 2 * NN * TV_MS + w, TV_MS};
  } else {
    return Model<T, NX, NY>{cst, make_const_layout(NX, NY, L), in};
  }
}

struct NoSteps {};

// The fast steps of a window do not wait for each other, so a tile's can be split over workgroups, each of
// which repeats what precedes the steps. A tile that has not settled is slow (nx = 4, L = 20, float64: about
// 40 us for its workgroup), and with few tiles that is the launch:
//   - where tiles settle (nx 2 .. 4), the slow ones of the first END_TILES tiles of each sequence (ends_first) take parts
//     of their own: 5 while that leaves a compute unit for every workgroup; 3, or else 2, while the device holds all of
//     them, the parts counted half, since about half of these tiles have settled and their parts leave at once; at
//     nx = 2, where a slow tile is short, 2 at most. Beyond that the parts only queue before the other tiles. One
//     sequence (nx = 4, L = 20, float64; tiles: whole, 3, 5 parts): 128 with inputs: 121, 86, 78 us a call; 235: 94,
//     87, 90. Batches of 3000 windows each (nx = 4, L = 10; whole, 2, 3, 5 parts): 8 sequences, float64: 62, 58, 53, 55;
//     15, float64: 68, 69, 80, 80; 24, float32: 68, 66, 63, 65; 40 of 1000 windows, float64: 64, 66, 69, 76.
//     Part p of all sequences' n-th tile follow each other in the grid, so that the first tiles, slow in every
//     sequence, spread over the dies (a sequence's parts together put them on the same ones: the 24 sequences 78 us in 5).
//   - every tile takes as many parts as let all workgroups run at once; where tiles settle, which leaves a
//     part little but what it repeats, half as many (128 tiles, 2 parts: 41 us against 32 us whole).
// Recovery of 16000 windows (63 tiles) at nx = 6 in float32: 95 us whole, 37 us in 4 parts; 6000 windows at
// nx = 4 in float64: 17.5 us with the end tiles alone split, 14.7 us in 5 parts.
struct Split {
  int extra, all, ends;  // extra workgroups, first in the grid, for the end tiles; parts of any tile, of an end tile
  int nseq;
};
constexpr int CUS = 256, END_TILES = 8, MAX_PARTS = 8, MIN_STEPS = 4;
// Recovery workgroups a compute unit holds (one wave of each on a SIMD).
template <typename T, int NX, bool TV>
constexpr int recover_per_cu() {
  return NX <= (sizeof(T) == 4 ? 4 : 3) && !TV ? 2 : 1;
}
template <typename T, int NX>
inline Split make_split(int64_t ntiles, int64_t nseq) {
  const int64_t fit = (blocks4<NX>() ? CUS / 2 : CUS) / ntiles;
  const int all = (int)(fit < 1 ? 1 : fit > MAX_PARTS ? MAX_PARTS : fit);
  if (!blocks4<NX>()) return Split{0, all, all, 1};
  const int64_t slow = nseq * END_TILES, room = CUS * recover_per_cu<T, NX, false>() - ntiles * all;
  const int ends = NX > 2 && ntiles * all + 4 * slow <= CUS ? 5 : NX > 2 && slow <= room ? 3 : slow <= 2 * room ? 2 : 1;
  if (all >= ends) return Split{0, all, all, 1};
  return Split{(int)slow * (ends - 1), all, ends, (int)nseq};
}
// The tile's number in its sequence (ends_first) and its part for workgroup bid, given the grid's numbering.
SRTM_DEV void split_place(const Split& sp, int64_t bid, int& seq, int64_t& i, int& part) {
  if (bid < sp.extra) {
    const int per = sp.ends - 1, e = (int)bid / per;
    part = 1 + (int)bid % per;
    seq = e % sp.nseq;
    i = e / sp.nseq;
  } else {
    const unsigned w = (unsigned)(bid - sp.extra);
    seq = -1;
    i = w / (unsigned)sp.all;  // counted over all sequences
    part = (int)(w % (unsigned)sp.all);
  }
}

// Part `part` of the fast steps 1 .. n, beg .. end (none: beg > n): of nslow parts of a tile that has not
// settled, of nparts of one that has. MIN_STEPS at least, and for nx <= 4 multiples of it: groups of means stay whole.
template <int NX>
struct StepShare {
  int beg, end;
  SRTM_DEV StepShare(int n, int part, int nparts, int nslow, bool settled) {
    const int np = settled ? nparts : nslow;
    int per = (n + np - 1) / np;
    if (per < MIN_STEPS) per = MIN_STEPS;
    if (NX <= 4) per = (per + MIN_STEPS - 1) / MIN_STEPS * MIN_STEPS;
    beg = part < np ? part * per + 1 : n + 1;
    end = n < beg + per - 1 ? n : beg + per - 1;
  }
};

// Fast steps whose tables the time-invariant recovery holds in LDS at a time.
constexpr int RSTEPS = 32;

// K7: fast-rate recovery, one window per lane and a loop over the window's fast steps.
// MODE bit 1: filter blocks p(x_{k,i} | y_{1:k}); bit 2: smoothed blocks p(x_{k,i} | y_{1:N}); bits 1 and 2 together or
// bit 4 beside bit 2: also the slow filter means, where asked for (a bit of its own: the unused store took the
// recovery of 1094 windows with inputs, nx = 3 in float64, from 20.3 to 22.3 us).
// (and the smoother's slow state, block i = 1) from the correction (v, W), formed of the fold's state and
// information (info_correction), or, for per-window models, of what the tile's forward pass left as terms
// linear in the smoothed state entering the tile; a workgroup covers exactly one tile.
// `ilim` is L when fast-rate outputs are requested and 1 when only the slow smoothed state is. Part `part`
// takes its share of the fast steps (StepShare).
// TV: per-window model; `cst` then holds the per-window constants blocks (stored by tv_column)
// and Fa, Qa (with in.H) the per-window F, Q and H.
template <typename T, int NX, int NY, int MODE, bool INP, bool TV = false>
SRTM_DEV void recover_body(const T* __restrict__ y, int64_t N, int L, int ilim, const T* __restrict__ cst,
                           InputView<T> in, const T* __restrict__ Fa, const T* __restrict__ Qa,
                           const T* __restrict__ m0, const T* __restrict__ P0, const T* __restrict__ carry,
                           const T* __restrict__ sfx, const T* __restrict__ tin, const T* __restrict__ utree,
                           T* __restrict__ mf_fast,
                           T* __restrict__ Pf_fast, T* __restrict__ ms_fast, T* __restrict__ Ps_fast,
                           T* __restrict__ ms_slow, T* __restrict__ Ps_slow, T* __restrict__ mf_slow,
                           int32_t* info, int64_t tile, int part, int nparts, int nslow) {
  constexpr int NN = NX * NX, ST = NX + NN, SF = sfx_stride(NX);
  static_assert(TILE == 256, "one recovery workgroup per tile");
  constexpr bool FILT = (MODE & 1) != 0, SMOOTH = (MODE & 2) != 0, MEANS = MODE == 3 || (MODE & 4) != 0;
  static_assert(!(TV && FILT && SMOOTH), "per-window models: filter and smoother outputs in two passes "
                                         "(the LDS copy of the model follows one staging buffer per wave)");
  using Stg = OutStage<T, NX>;
  extern __shared__ char smraw[];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int64_t k = tile * TILE + tid;
  const int64_t w0 = tile * TILE + wv * 64;
  const int nvalid = (int)((N - w0) < 64 ? ((N - w0) > 0 ? (N - w0) : 0) : 64);
  const Stg fst(smraw + (size_t)wv * Stg::BYTES * (FILT && SMOOTH ? 2 : 1));
  const Stg sst(smraw + (size_t)wv * Stg::BYTES * (FILT && SMOOTH ? 2 : 1) + (FILT && SMOOTH ? Stg::BYTES : 0));
  const bool valid = k < N;
  const int64_t kc = valid ? k : 0;   // clamped index for loads of padding lanes
  T* mdl = reinterpret_cast<T*>(smraw + (size_t)4 * Stg::BYTES * (FILT && SMOOTH ? 2 : 1));
  if constexpr (TV) {
    const int64_t t0 = tile * TILE;
    tv_model_to_lds<T, NX, NY>(Fa, Qa, in.H, t0, (int)((N - t0) < TILE ? (N - t0) : TILE), mdl);
    __syncthreads();
  }
  const auto M = recover_model<TV, T, NX, NY>(cst, L, in, mdl, k);
  T m[NX], P[NX][NX], yk[NY];
  const int nw = tile_windows(N, tile);
  bool settled = false;  // the tile's windows share their covariances
  if constexpr (!TV) settled = tile_settled<T, NX>(utree, tile);
  int ibeg = 1;  // this workgroup's fast steps are ibeg .. ilim
  if constexpr (!TV) {
    const StepShare<NX> share(ilim, part, nparts, nslow, settled);
    if (share.beg > ilim) return;
    ibeg = share.beg;
    ilim = share.end;
  }
  const int64_t col = tile * (TILE * info_stride(NX)) + (valid ? tid : 0);  // the window's records
  const int64_t mcol = settled ? tile * (TILE * info_stride(NX)) : col;
  if constexpr (TV) load_prior<T, NX, NY>(carry, m0, P0, kc, m, P);
  else record_load(m, P, carry + col, carry + mcol, nw);
  T zL[NX];  // z_{k,l}
#pragma unroll
  for (int r = 0; r < NX; ++r) zL[r] = T(0);
  if constexpr (INP) {
    window_meas<true>(M, y, kc, N, yk, zL);
  } else {
    gloadv(yk, y + kc * NY);
  }
  Window<T, NX, NY> w;
  int flag = 0;
  if (!window_setup(M, L, m, P, yk, w) && valid) flag |= SRTM_INFO_INNOVATION_NOT_PD;
  T z[NX], un[NU_MAX];  // input response z_{k,i} and the next step's inputs (inputs only)
#pragma unroll
  for (int r = 0; r < NX; ++r) z[r] = T(0);
  const T* uk = INP ? in.u + kc * L * in.nu : nullptr;
  if constexpr (INP) {
#pragma unroll
    for (int j = 0; j < NU_MAX; ++j) un[j] = (j < in.nu) ? gld(uk + j) : T(0);
  }
  T v[NX], W[NX][NX];
  if constexpr (SMOOTH && !TV) {
    // The slow-rate filter means beside smoothed outputs: a window update keeps the digits of an accurate measurement
    // that the fold's state of the next window loses (its runs carry y as eta = C_bar^T R_x^{-1} y, rounded). The
    // covariances stay the fold's, which loses none where the update subtracts nearly equal matrices.
    T* mean = MEANS && mf_slow && part == 0 && valid ? mf_slow + k * NX : nullptr;
    if (!info_correction<INP>(M, L, w, zL, sfx + col, sfx + mcol, nw, v, W, mean) && valid)
      flag |= SRTM_INFO_COMBINE_SINGULAR;
  } else if constexpr (SMOOTH) {  // v = Et m_in + gt,  W = Et P_in Et^T + St
    const T* src = sfx + kc * SF;
    const T* ti = tin + tile * ST;
    T Et[NX][NX], mi[NX], Pi[NX][NX], EP[NX][NX];
    gload(Et, src);
    gloadv(mi, ti);
    gload(Pi, ti + NX);
#pragma unroll
    for (int r = 0; r < NX; ++r) {
      T t = gld(src + NN + r);
#pragma unroll
      for (int q = 0; q < NX; ++q) t = my_fma(Et[r][q], mi[q], t);
      v[r] = t;
    }
    mm(Et, Pi, EP);
    int o = NN + NX;
#pragma unroll
    for (int r = 0; r < NX; ++r)
#pragma unroll
      for (int c = r; c < NX; ++c) {
        T t = gld(src + o++);
#pragma unroll
        for (int q = 0; q < NX; ++q) t = my_fma(EP[r][q], Et[c][q], t);
        W[r][c] = t;
        W[c][r] = t;
      }
  }
  bool fin = true;
  // z_i = A z_{i-1} + B u_{k,i-1}, the loads of step i+1 issued first
  auto input_advance = [&](int i) {
    if constexpr (INP) {
      T uc[NU_MAX];
#pragma unroll
      for (int j = 0; j < NU_MAX; ++j) {
        uc[j] = un[j];
        un[j] = (j < M.in.nu && i < L) ? gld(uk + i * M.in.nu + j) : T(0);
      }
      T A[NX][NX], nz[NX];
      load(A, M.cst + M.lay.A);
#pragma unroll
      for (int r = 0; r < NX; ++r) {
        T t = T(0);
#pragma unroll
        for (int j = 0; j < NU_MAX; ++j)
          if (j < M.in.nu) t = my_fma(gld(M.in.B + r * M.in.nu + j), uc[j], t);
#pragma unroll
        for (int q = 0; q < NX; ++q) t = my_fma(A[r][q], z[q], t);
        nz[r] = t;
      }
#pragma unroll
      for (int r = 0; r < NX; ++r) z[r] = nz[r];
    }
  };
  // The per-step tables of fast steps i .. go to LDS, RSTEPS steps at a time: read per step as
  // wave-uniform scalar loads they outgrow the scalar registers (spilled to vector-register lanes and
  // read back every step).
  auto stage_steps = [&](int i) {
    if constexpr (!TV) {
      const int n = (ilim - i + 1 < RSTEPS ? ilim - i + 1 : RSTEPS) * M.lay.per_i_stride;
      const T* src = M.per_i(i);
      __syncthreads();  // every wave is done with the previous steps' tables
      staged_copy<8, T>(n, tid, TILE, [&](int q) { return gld(src + q); }, [&](int q, T v) { mdl[q] = v; });
      __syncthreads();
    }
  };
  if constexpr (!TV && blocks4<NX>()) {
    if (settled) {
      // Every window has the same covariances: four threads form those of a fast step once for the tile, and
      // each wave writes them to its 64 windows front to back (Stream). The means of a step are one small
      // matrix product for all windows, m^s_i = [A^i c_i P^f_{i,l}] (m'; S^{-1}e; v), four windows to a block of
      // the matrix cores (Block4's layout; float64 for both types). With one lane per window the same product
      // read its 40 coefficients from LDS in every lane, 1800 cycles a step against 300.
      constexpr int SC = 24;  // fast steps at a time
      constexpr int KF = NX + NY, KS2 = KF + NX, KBF = (KF + 3) / 4, KBS = SMOOTH ? (KS2 + 3) / 4 : KBF;
      constexpr int RB = NN * (int)sizeof(T);
      static_assert(SC * RB <= 64 * Stg::SBP && SC * KBS * 128 <= 64 * Stg::SBP && KBS * 4 * 512 <= 4 * 64 * Stg::SBP,
                    "each table fits one wave's covariance staging");
      static_assert(SC % Stg::GM == 0, "a chunk of steps begins a group of means");
      char* tab_s = smraw;                                                   // P^s of the steps
      double* row_s = reinterpret_cast<double*>(smraw + (size_t)Stg::BYTES);   // rows of the smoothed means
      char* tab_f = smraw + (size_t)2 * Stg::BYTES;                          // P^f
      double* row_f = reinterpret_cast<double*>(smraw + (size_t)3 * Stg::BYTES);
      const int bk = lane >> 4, bw = lane & 15, bc = lane & 3;  // row, window of 16, column of the block layout
      double x[4][KBS];  // (m'; S^{-1}e; v) of window 16 n + bw, entry 4 kb + bk
      {
        double* sx = reinterpret_cast<double*>(fst.pbuf);  // [entry][window], KBS * 4 entries at most
        constexpr int KA = SMOOTH ? KS2 : KF;
        constexpr int KP = 64 * Stg::SBP / 512 < KA ? 64 * Stg::SBP / 512 : KA;  // entries at a time
#pragma unroll
        for (int k0 = 0; k0 < KA; k0 += KP) {
#pragma unroll
          for (int e = k0; e < k0 + KP && e < KA; ++e)
            sx[(e - k0) * 64 + lane] = e < NX ? (double)w.mp[e] : e < KF ? (double)w.Se[e < KF && e >= NX ? e - NX : 0]
                                                                  : SMOOTH ? (double)v[e >= KF ? e - KF : 0] : 0.0;
          wave_sync();
#pragma unroll
          for (int n = 0; n < 4; ++n)
#pragma unroll
            for (int kb = 0; kb < KBS; ++kb) {
              const int e = 4 * kb + bk;
              if (e >= k0 && e < k0 + KP && e < KA) x[n][kb] = sx[(e - k0) * 64 + 16 * n + bw];
              else if (k0 == 0) x[n][kb] = 0.0;
            }
          wave_sync();
        }
      }
      // The filter's product ends at S^{-1}e: its last block of four has zeros in place of v, which a later measurement
      // that is not finite makes NaN.
      double xf[4];
#pragma unroll
      for (int n = 0; n < 4; ++n) xf[n] = 4 * (KBF - 1) + bk < KF ? x[n][KBF - 1] : 0.0;
      // input response of the same windows, entry bk: z_i = A z_{i-1} + B u_{k,i-1}
      double zr[4] = {0.0, 0.0, 0.0, 0.0}, Aop = 0.0, Bop = 0.0, un4[4] = {0.0, 0.0, 0.0, 0.0}, uq[4] = {0.0, 0.0, 0.0, 0.0};
      auto load_u = [&](int i) {  // inputs of the step into x_{k,i}, two steps before they are used
#pragma unroll
        for (int n = 0; n < 4; ++n) {
          un4[n] = uq[n];
          uq[n] = bk < M.in.nu && i <= ilim ? (double)gld(M.in.u + ((w0 + 16 * n + bw) * L + (i - 1)) * M.in.nu + bk) : 0.0;
        }
      };
      auto advance = [&](int i) {
#pragma unroll
        for (int n = 0; n < 4; ++n) zr[n] = mm4(Aop, zr[n], mm4(Bop, un4[n], 0.0));
        load_u(i + 2);
      };
      if constexpr (INP) {
        Aop = bc < NX && bk < NX ? (double)gld(M.cst + M.lay.A + bc * NX + bk) : 0.0;
        Bop = bc < NX && bk < M.in.nu ? (double)gld(M.in.B + bc * M.in.nu + bk) : 0.0;
        load_u(1);
        load_u(2);
#pragma unroll 1
        for (int i = 1; i < ibeg; ++i) advance(i);
      }
      auto base_of = [&](T* out, int i) { return reinterpret_cast<char*>(out) + (w0 * L + (i - 1)) * RB; };
#pragma unroll 1
      for (int i0 = ibeg; i0 <= ilim; i0 += SC) {
        const int ns = ilim - i0 + 1 < SC ? ilim - i0 + 1 : SC;
        stage_steps(i0);  // its first barrier also ends the reads of the previous tables
        // one thread per step and row: row r of step_blocks' matrices and of P^s
        const int sq = tid >> 2, r = tid & 3;
        if (sq < ns && r < NX) {
          const T* ps = mdl + sq * M.lay.per_i_stride;
          const T* Ai = ps + M.lay.o_Ai;
          const T* ci = ps + M.lay.o_ci;
          T Ar[NX], cr[NY], AP[NX], US[NY], Pr[NX], Lr[NX], TW[NX];
          loadv(Ar, Ai + r * NX);
          loadv(cr, ci + r * NY);
          auto u_row = [&](const T (&ar)[NX], const T (&cc)[NY], T (&u)[NY]) {  // U_i = A^i V + c_i, one row
#pragma unroll
            for (int q = 0; q < NY; ++q) {
              T t = ar[0] * w.V[0][q];
#pragma unroll
              for (int k2 = 1; k2 < NX; ++k2) t = my_fma(ar[k2], w.V[k2][q], t);
              u[q] = t + cc[q];
            }
          };
          {
            T u[NY];
            u_row(Ar, cr, u);
#pragma unroll
            for (int q = 0; q < NY; ++q) {
              T t = T(0);
#pragma unroll
              for (int k2 = 0; k2 < NY; ++k2) t = my_fma(u[k2], symget(w.Si, k2, q), t);
              US[q] = t;
            }
          }
#pragma unroll
          for (int c = 0; c < NX; ++c) {
            T t = T(0);
#pragma unroll
            for (int k2 = 0; k2 < NX; ++k2) t = my_fma(Ar[k2], symget(w.P, k2, c), t);
            AP[c] = t;
          }
#pragma unroll
          for (int c = 0; c < NX; ++c) {  // row r of P^f_{i,i} (the entries right of the diagonal are used)
            T ac[NX], cc[NY], u[NY];
            loadv(ac, Ai + c * NX);
            loadv(cc, ci + c * NY);
            u_row(ac, cc, u);
            T t = ps[M.lay.o_Qii + r * NX + c];
#pragma unroll
            for (int k2 = 0; k2 < NX; ++k2) t = my_fma(AP[k2], ac[k2], t);
#pragma unroll
            for (int k2 = 0; k2 < NY; ++k2) t = my_fma(-US[k2], u[k2], t);
            Pr[c] = t;
          }
          auto rows = [&](double* o, int kn, int kb_n) {  // column r of each entry; idle rows stay zero
#pragma unroll
            for (int e = 0; e < 4 * KBS; ++e)
              if (e < 4 * kb_n) {
                const double t = e >= kn ? 0.0 : e < NX ? (double)Ar[e < NX ? e : 0]
                                 : e < KF ? (double)cr[e >= NX && e < KF ? e - NX : 0]
                                          : (double)Lr[e >= KF && e < KS2 ? e - KF : 0];
                o[e * 4 + r] = t;
                if (r == 0) {
#pragma unroll
                  for (int z0 = NX; z0 < 4; ++z0) o[e * 4 + z0] = 0.0;
                }
              }
          };
          if constexpr (FILT) {
            T* o = reinterpret_cast<T*>(tab_f + sq * RB);
#pragma unroll
            for (int c = 0; c < NX; ++c)
              if (c >= r) {
                o[r * NX + c] = o[c * NX + r] = Pr[c];
                fin = fin && isfinite(Pr[c]);
              }
            rows(row_f + sq * KBF * 16, KF, KBF);
          }
          if constexpr (SMOOTH) {
#pragma unroll
            for (int c = 0; c < NX; ++c) {  // row r of P^f_{i,l} = A^i Y1 + Q_il - c_i Y2
              T t = ps[M.lay.o_QiL + r * NX + c];
#pragma unroll
              for (int k2 = 0; k2 < NX; ++k2) t = my_fma(Ar[k2], w.Y1[k2][c], t);
#pragma unroll
              for (int k2 = 0; k2 < NY; ++k2) t = my_fma(-cr[k2], w.Y2[k2][c], t);
              Lr[c] = t;
            }
#pragma unroll
            for (int c = 0; c < NX; ++c) {
              T t = T(0);
#pragma unroll
              for (int k2 = 0; k2 < NX; ++k2) t = my_fma(Lr[k2], symget(W, k2, c), t);
              TW[c] = t;
            }
            double* ro = row_s + sq * KBS * 16;
            rows(ro, KS2, KBS);
            wave_sync();  // the four rows of a step belong to one wave
            T* o = reinterpret_cast<T*>(tab_s + sq * RB);
#pragma unroll
            for (int c = 0; c < NX; ++c) {
              T t = Pr[c];
#pragma unroll
              for (int k2 = 0; k2 < NX; ++k2) t = my_fma(TW[k2], (T)ro[(KF + k2) * 4 + c], t);
              if (c >= r) {
                o[r * NX + c] = o[c * NX + r] = t;
                fin = fin && isfinite(t);
              }
            }
          }
        }
        __syncthreads();
        Stream<RB> sf(lane, ns, L), ss(lane, ns, L);
#pragma unroll 1
        for (int j = 0; j < ns; ++j) {
          const int i = i0 + j;
          if constexpr (INP) advance(i);
          auto means = [&](const double* row, int kb_n, const Stg& st, bool filt) {
            double a[KBS];
#pragma unroll
            for (int kb = 0; kb < KBS; ++kb)
              if (kb < kb_n) a[kb] = row[(j * kb_n + kb) * 16 + 4 * bk + bc];
            T* mp = reinterpret_cast<T*>(st.mbuf + bw * Stg::SBM) + (j % Stg::GM) * NX + bk;
#pragma unroll
            for (int n = 0; n < 4; ++n) {
              double acc = zr[n];
#pragma unroll
              for (int kb = 0; kb < KBS; ++kb)
                if (kb < kb_n) acc = mm4(a[kb], filt && kb == KBF - 1 ? xf[n] : x[n][kb], acc);
              if (bk < NX) {
                *reinterpret_cast<T*>(reinterpret_cast<char*>(mp) + n * 16 * Stg::SBM) = (T)acc;
                fin = fin && isfinite((T)acc);
              }
            }
          };
          if constexpr (FILT) means(row_f, KBF, fst, true);
          if constexpr (SMOOTH) means(row_s, KBS, sst, false);
          if (FILT && Pf_fast) sf.put(tab_f, base_of(Pf_fast, i0));
          if (SMOOTH && Ps_fast) ss.put(tab_s, base_of(Ps_fast, i0));
          wave_sync();
          if (FILT) fst.flush(lane, 64, mf_fast, nullptr, w0, L, j, i, ilim);
          if (SMOOTH) {
            if (i == 1) {
              sst.flush_slow(lane, 64, ms_slow, nullptr, w0);
              if (Ps_slow) {
                Stream<RB> one(lane, 1, 1);
                one.put(tab_s, reinterpret_cast<char*>(Ps_slow + w0 * NN));
              }
            }
            sst.flush(lane, 64, ms_fast, nullptr, w0, L, j, i, ilim);
          }
          wave_sync();
        }
      }
      if (!fin) flag |= SRTM_INFO_NONFINITE;
      if (flag && info) atomicOr(info, flag);
      return;
    }
  }
  if constexpr (INP && !TV) {
    if (ibeg > 1) {  // a later part of the tile's steps: the response before it
      T zs[NX];
      input_response(M, uk, ibeg - 1, z, zs);
#pragma unroll
      for (int j = 0; j < NU_MAX; ++j) un[j] = (j < in.nu) ? gld(uk + (ibeg - 1) * in.nu + j) : T(0);
    }
  }
  std::conditional_t<TV, TvSteps<T, NX, NY>, NoSteps> steps;
#pragma unroll 1
  for (int i = ibeg; i <= ilim; ++i) {
    T mf[NX], Pii[NX][NX], PiL[NX][NX];
    if constexpr (!TV) {
      if ((i - ibeg) % RSTEPS == 0) stage_steps(i);
    }
    if constexpr (TV) {
      steps.template next<SMOOTH, true>(M, L, w, mf, Pii, PiL);
    } else {  // step i's A^i, c_i, Q_ii and Q_il from the LDS copy
      const T* ps = mdl + ((i - ibeg) % RSTEPS) * M.lay.per_i_stride;
      T Ai[NX][NX], ci[NX][NY];
      load(Ai, ps + M.lay.o_Ai);
      load(ci, ps + M.lay.o_ci);
      step_blocks<SMOOTH>(
          w, Ai, ci, [&](int r, int c) { return ps[M.lay.o_Qii + r * NX + c]; },
          [&](int r, int c) { return ps[M.lay.o_QiL + r * NX + c]; }, mf, Pii, PiL);
    }
    if constexpr (INP) {
      input_advance(i);
#pragma unroll
      for (int r = 0; r < NX; ++r) mf[r] += z[r];
    }
    if (FILT) {
      fin = fin && finite_state(mf, Pii);
      fst.put(lane, i - ibeg, mf, Pii);
    }
    if (SMOOTH) {
      T ms[NX], Ps[NX][NX];
#pragma unroll
      for (int r = 0; r < NX; ++r) {
        T s = mf[r];
#pragma unroll
        for (int q = 0; q < NX; ++q) s = my_fma(PiL[r][q], v[q], s);
        ms[r] = s;
        T TW[NX];
#pragma unroll
        for (int c = 0; c < NX; ++c) {
          T t = T(0);
#pragma unroll
          for (int q = 0; q < NX; ++q) t = my_fma(PiL[r][q], symget(W, q, c), t);
          TW[c] = t;
        }
#pragma unroll
        for (int c = r; c < NX; ++c) {
          T t = Pii[r][c];
#pragma unroll
          for (int q = 0; q < NX; ++q) t = my_fma(TW[q], PiL[c][q], t);
          Ps[r][c] = t;
          Ps[c][r] = t;
        }
      }
      fin = fin && finite_state(ms, Ps);
      sst.put(lane, i - ibeg, ms, Ps);
    }
    wave_sync();
    if (FILT) fst.flush(lane, nvalid, mf_fast, Pf_fast, w0, L, i - ibeg, i, ilim);
    if (SMOOTH) {
      if (i == 1) sst.flush_slow(lane, nvalid, ms_slow, Ps_slow, w0);
      sst.flush(lane, nvalid, ms_fast, Ps_fast, w0, L, i - ibeg, i, ilim);
    }
    wave_sync();
  }
  if (!fin && valid) flag |= SRTM_INFO_NONFINITE;
  if (flag && info) atomicOr(info, flag);
}

// ============================================================================ sequential comparator
// The sequential route of Sec. III on the GPU, one lane per sequence and no scan: the IMKF walks
// the windows forwards (eq. prediction and eq. m-h-k-l, written as block l of the window filter
// of eq. update-fast) and stores the slow-rate carry (m^f_{k,l}, P^f_{k,l}); the sequential SRTM
// smoother then walks them backwards (eq. smoothing-dynamic, eq. seq-smoothing-all): with the
// smoothed state (m^s_{k+1,1}, P^s_{k+1,1}) of the window after, P^- = A P^f_{k,l} A^T + Q and
// B = (P^-)^{-1} A, the correction v = B^T (m^s_{k+1,1} - A m^f_{k,l}), W = B^T (P^s_{k+1,1} - P^-) B
// gives every fast step's smoothed blocks m^s_{k,i} = m^f_{k,i} + P^f_{k,i,l} v and
// P^s_{k,i} = P^f_{k,i,i} + P^f_{k,i,l} W P^f_{k,i,l}^T, and block i = 1 is the state the window before
// needs (eq. seq-smoothing-1). The per-window arithmetic is the parallel path's; only the order
// of evaluation differs (a recursion instead of the two scans). This is the paper's sequential
// comparison method (Sec. V), run on the same GPU.
template <typename T, int NX, int NY>
SRTM_DEV void seq_body(const T* __restrict__ y, int64_t N, int L, const T* __restrict__ cst,
                       const T* __restrict__ m0, const T* __restrict__ P0, T* __restrict__ carry,
                       T* __restrict__ ms_fast, T* __restrict__ Ps_fast, T* __restrict__ ms_slow,
                       T* __restrict__ Ps_slow, int32_t* info) {
  constexpr int NN = NX * NX, ST = NX + NN;
  const Model<T, NX, NY> M{cst, make_const_layout(NX, NY, L)};
  int flag = 0;
  bool fin = true;
  T m[NX], P[NX][NX];
  gloadv(m, m0);
  gload(P, P0);
  symmetrize(P);
#pragma unroll 1
  for (int64_t k = 0; k < N; ++k) {  // forward: the IMKF
    T yk[NY];
    gloadv(yk, y + k * NY);
    Window<T, NX, NY> w;
    if (!window_setup(M, L, m, P, yk, w)) flag |= SRTM_INFO_INNOVATION_NOT_PD;
    T PiL[NX][NX];
    window_step<T, NX, NY, false>(M, w, L, m, P, PiL);
#pragma unroll
    for (int r = 0; r < NX; ++r) put_global(carry + k * ST + r, m[r]);
#pragma unroll
    for (int r = 0; r < NX; ++r)
#pragma unroll
      for (int c = 0; c < NX; ++c) put_global(carry + k * ST + NX + r * NX + c, P[r][c]);
  }
  T A[NX][NX], Qm[NX][NX];
  load(A, M.cst + M.lay.A);
  load(Qm, M.cst + M.lay.Q);
  T ms1[NX], Ps1[NX][NX];
#pragma unroll 1
  for (int64_t k = N - 1; k >= 0; --k) {  // backward: the sequential smoother
    T yk[NY];
    gloadv(yk, y + k * NY);
    if (k == 0) {
      gloadv(m, m0);
      gload(P, P0);
      symmetrize(P);
    } else {
      gloadv(m, carry + (k - 1) * ST);
      gload(P, carry + (k - 1) * ST + NX);
    }
    Window<T, NX, NY> w;
    if (!window_setup(M, L, m, P, yk, w)) flag |= SRTM_INFO_INNOVATION_NOT_PD;
    T v[NX], W[NX][NX];
    if (k == N - 1) {
#pragma unroll
      for (int r = 0; r < NX; ++r) {
        v[r] = T(0);
#pragma unroll
        for (int c = 0; c < NX; ++c) W[r][c] = T(0);
      }
    } else {
      T mL[NX], PL[NX][NX], Pm[NX][NX], Pmi[NX][NX], B[NX][NX], d[NX], D[NX][NX], DB[NX][NX];
      gloadv(mL, carry + k * ST);
      gload(PL, carry + k * ST + NX);
      sandwich(A, PL, Qm, Pm);
      if (!spd_inv(Pm, Pmi)) flag |= SRTM_INFO_PRED_SINGULAR;
      mm(Pmi, A, B);
#pragma unroll
      for (int r = 0; r < NX; ++r) {
        T t = ms1[r];
#pragma unroll
        for (int q = 0; q < NX; ++q) t = my_fma(-A[r][q], mL[q], t);
        d[r] = t;
#pragma unroll
        for (int c = 0; c < NX; ++c) D[r][c] = Ps1[r][c] - Pm[r][c];
      }
      mtv(B, d, v);
      mm(D, B, DB);
#pragma unroll
      for (int r = 0; r < NX; ++r)
#pragma unroll
        for (int c = r; c < NX; ++c) {
          T t = T(0);
#pragma unroll
          for (int q = 0; q < NX; ++q) t = my_fma(B[q][r], DB[q][c], t);
          W[r][c] = t;
          W[c][r] = t;
        }
    }
#pragma unroll 1
    for (int i = 1; i <= L; ++i) {
      T mf[NX], Pii[NX][NX], PiL[NX][NX], ms[NX], Ps[NX][NX];
      window_step<T, NX, NY, true>(M, w, i, mf, Pii, PiL);
#pragma unroll
      for (int r = 0; r < NX; ++r) {
        T s = mf[r];
#pragma unroll
        for (int q = 0; q < NX; ++q) s = my_fma(PiL[r][q], v[q], s);
        ms[r] = s;
        T TW[NX];
#pragma unroll
        for (int c = 0; c < NX; ++c) {
          T t = T(0);
#pragma unroll
          for (int q = 0; q < NX; ++q) t = my_fma(PiL[r][q], W[q][c], t);
          TW[c] = t;
        }
#pragma unroll
        for (int c = r; c < NX; ++c) {
          T t = Pii[r][c];
#pragma unroll
          for (int q = 0; q < NX; ++q) t = my_fma(TW[q], PiL[c][q], t);
          Ps[r][c] = t;
          Ps[c][r] = t;
        }
      }
      fin = fin && finite_state(ms, Ps);
      const int64_t o = k * L + (i - 1);
      if (ms_fast) {
#pragma unroll
        for (int r = 0; r < NX; ++r) put_global(ms_fast + o * NX + r, ms[r]);
      }
      if (Ps_fast) {
#pragma unroll
        for (int r = 0; r < NN; ++r) put_global(Ps_fast + o * NN + r, Ps[r / NX][r % NX]);
      }
      if (i == 1) {
#pragma unroll
        for (int r = 0; r < NX; ++r) {
          ms1[r] = ms[r];
#pragma unroll
          for (int c = 0; c < NX; ++c) Ps1[r][c] = Ps[r][c];
        }
        if (ms_slow) {
#pragma unroll
          for (int r = 0; r < NX; ++r) put_global(ms_slow + k * NX + r, ms[r]);
        }
        if (Ps_slow) {
#pragma unroll
          for (int r = 0; r < NN; ++r) put_global(Ps_slow + k * NN + r, Ps[r / NX][r % NX]);
        }
      }
    }
  }
  if (!fin) flag |= SRTM_INFO_NONFINITE;
  if (flag && info) atomicOr(info, flag);
}

// ============================================================================ per-window models
// Time-varying model given per window: window k's F_k, Q_k drive its fast steps x_{k,1} ..
// x_{k,l} (the step from x_{k-1,l} included) and H_k, R_k give y_k. What the time-invariant path
// computes once per call (slow-rate constants, the element matrices) is computed once per window,
// by one lane, into a per-window constants block (TvLayout: window-level constants and the
// backward factors of the fast steps; the forward quantities are recomputed where they are
// used, see TvSteps) and an element record (F, D, J). The forward scan then combines whole
// elements: the level tables of the time-invariant path do not exist here.

// Per-window constants (float64 in registers, one lane, one pass over the window's fast steps):
// the block `blk` (TvLayout `lay`) and the element matrices `el` = F, D, J of the model
// (Fm, Qm, Hm, Rm). With s_i = x_{k,1} + ... + x_{k,i} and the noise covariances (x_{k,0} = 0)
// P_xx = Q_ii, P_xs = Cov(x_{k,i}, s_i), P_ss = Cov(s_i), one fast step x <- A x + w gives
//   P_xx' = A P_xx A^T + Q,  P_xs' = A P_xs + P_xx',  P_ss' = P_ss + A P_xs + (A P_xs)^T + P_xx',
// and after l steps Q_ll = P_xx, c_l = (1/l) P_xs C^T, R_x = (1/l^2) C P_ss C^T + R (eq. h-k-l-2 and
// eq. y-k-l-2: the noise parts of Cov(x_{k,l}, y_k) and Cov(y_k)); C_bar = (C/l)(Sig_l - I),
// K = c_l R_x^{-1}, F = A^l - K C_bar, D = Q_ll - K c_l^T, J = C_bar^T R_x^{-1} C_bar. At step j the
// pass also stores A^j and C Sig_j for even j, the backward factors of fast step i = l - j.
// `blk` and `el` are the window's columns (tv_column): scalar j at blk[j * cs] and el[j * cs].
template <typename T, int NX, int NY>
SRTM_DEV int tv_window_constants(const T* __restrict__ Fm, const T* __restrict__ Qm, const T* __restrict__ Hm,
                                 const T* __restrict__ Rm, int L, const TvLayout& lay, T* __restrict__ blk,
                                 T* __restrict__ el, int64_t cs) {
  int flag = 0;
  auto W = [&](int j, double v) { put_global(blk + (int64_t)j * cs, (T)v); };
  auto WE = [&](int j, double v) { put_global(el + (int64_t)j * cs, (T)v); };
  double A[NX][NX], Q[NX][NX], C[NY][NX], R[NY][NY];
#pragma unroll
  for (int r = 0; r < NX; ++r)
#pragma unroll
    for (int c = 0; c < NX; ++c) {
      A[r][c] = (double)gld(Fm + r * NX + c);
      Q[r][c] = (double)gld(Qm + (c >= r ? r * NX + c : c * NX + r));  // the upper triangle
    }
#pragma unroll
  for (int r = 0; r < NY; ++r) {
#pragma unroll
    for (int c = 0; c < NX; ++c) C[r][c] = (double)gld(Hm + r * NX + c);
#pragma unroll
    for (int c = 0; c < NY; ++c) R[r][c] = (double)gld(Rm + r * NY + c);
  }
  double Aj[NX][NX], Sig[NX][NX], Pxx[NX][NX], Pxs[NX][NX], Pss[NX][NX];
#pragma unroll
  for (int r = 0; r < NX; ++r)
#pragma unroll
    for (int c = 0; c < NX; ++c) {
      Aj[r][c] = Sig[r][c] = (r == c) ? 1.0 : 0.0;
      Pxx[r][c] = Pxs[r][c] = Pss[r][c] = 0.0;
    }
#pragma unroll 1
  for (int j = 0; j < L; ++j) {
    if ((j & 1) == 0) {  // backward factors A^j and C Sig_j (fast step i = l - j), slot j / 2
      const int so = lay.slot + (j >> 1) * lay.slot_stride;
#pragma unroll
      for (int r = 0; r < NX; ++r)
#pragma unroll
        for (int c = 0; c < NX; ++c) W(so + lay.o_As + r * NX + c, Aj[r][c]);
#pragma unroll
      for (int r = 0; r < NY; ++r)
#pragma unroll
        for (int c = 0; c < NX; ++c) {
          double v = 0.0;
#pragma unroll
          for (int q = 0; q < NX; ++q) v += C[r][q] * Sig[q][c];
          W(so + lay.o_CS + r * NX + c, v);
        }
    }
    // one fast step of the noise covariances
    double t[NX][NX], AP[NX][NX];
    mm(A, Pxs, t);  // A P_xs
    mm(A, Pxx, AP);
#pragma unroll
    for (int r = 0; r < NX; ++r)
#pragma unroll
      for (int c = r; c < NX; ++c) {
        double v = Q[r][c];
#pragma unroll
        for (int q = 0; q < NX; ++q) v += AP[r][q] * A[c][q];
        Pxx[r][c] = v;
        Pxx[c][r] = v;
      }
#pragma unroll
    for (int r = 0; r < NX; ++r)
#pragma unroll
      for (int c = r; c < NX; ++c) {
        const double v = Pss[r][c] + t[r][c] + t[c][r] + Pxx[r][c];
        Pss[r][c] = v;
        Pss[c][r] = v;
      }
#pragma unroll
    for (int r = 0; r < NX; ++r)
#pragma unroll
      for (int c = 0; c < NX; ++c) Pxs[r][c] = t[r][c] + Pxx[r][c];
    mm(A, Aj, t);  // A^{j+1}, Sig_{j+1}
#pragma unroll
    for (int r = 0; r < NX; ++r)
#pragma unroll
      for (int c = 0; c < NX; ++c) {
        Aj[r][c] = t[r][c];
        Sig[r][c] += t[r][c];
      }
  }
  // Aj = A^l, Sig = Sig_l, Pxx = Q_ll, Pxs = Cov(x_{k,l}, s_l), Pss = Cov(s_l)
  const double il = 1.0 / (double)L;
  double Cb[NY][NX], cL[NX][NY], Rx[NY][NY];
#pragma unroll
  for (int r = 0; r < NY; ++r)
#pragma unroll
    for (int c = 0; c < NX; ++c) {
      double v = 0.0;
#pragma unroll
      for (int q = 0; q < NX; ++q) v += C[r][q] * (Sig[q][c] - (q == c ? 1.0 : 0.0));
      Cb[r][c] = v * il;
    }
#pragma unroll
  for (int r = 0; r < NX; ++r)
#pragma unroll
    for (int c = 0; c < NY; ++c) {
      double v = 0.0;
#pragma unroll
      for (int q = 0; q < NX; ++q) v += Pxs[r][q] * C[c][q];
      cL[r][c] = v * il;
    }
  {
    double CP[NY][NX];
    mm(C, Pss, CP);
#pragma unroll
    for (int r = 0; r < NY; ++r)
#pragma unroll
      for (int c = 0; c < NY; ++c) {
        double v = 0.0;
#pragma unroll
        for (int q = 0; q < NX; ++q) v += CP[r][q] * C[c][q];
        Rx[r][c] = v * il * il + R[r][c];
      }
  }
  symmetrize(Rx);
  double Rxi[NY][NY];
  if (!spd_inv(Rx, Rxi)) flag |= SRTM_INFO_INNOVATION_NOT_PD;
  double K[NX][NY], Heta[NX][NY], Fe[NX][NX], De[NX][NX], Je[NX][NX];
  mm(cL, Rxi, K);
  mm_tn(Cb, Rxi, Heta);
#pragma unroll
  for (int r = 0; r < NX; ++r)
#pragma unroll
    for (int c = 0; c < NX; ++c) {
      double f = Aj[r][c], dd = Pxx[r][c];
#pragma unroll
      for (int q = 0; q < NY; ++q) {
        f -= K[r][q] * Cb[q][c];
        dd -= K[r][q] * cL[c][q];
      }
      Fe[r][c] = f;
      De[r][c] = dd;
    }
  mm(Heta, Cb, Je);
  symmetrize(De);
  symmetrize(Je);
#pragma unroll
  for (int r = 0; r < NX; ++r)
#pragma unroll
    for (int c = 0; c < NX; ++c) {
      W(lay.AL + r * NX + c, Aj[r][c]);
      WE(r * NX + c, Fe[r][c]);
      WE(NX * NX + r * NX + c, De[r][c]);
      WE(2 * NX * NX + r * NX + c, Je[r][c]);
    }
#pragma unroll
  for (int r = 0; r < NY; ++r) {
#pragma unroll
    for (int c = 0; c < NX; ++c) W(lay.Cbar + r * NX + c, Cb[r][c]);
#pragma unroll
    for (int c = 0; c < NY; ++c) W(lay.Rx + r * NY + c, Rx[r][c]);
  }
#pragma unroll
  for (int r = 0; r < NX; ++r)
#pragma unroll
    for (int c = 0; c < NY; ++c) {
      W(lay.cL + r * NY + c, cL[r][c]);
      W(lay.K + r * NY + c, K[r][c]);
      W(lay.Heta + r * NY + c, Heta[r][c]);
    }
  return flag;
}

// R x C scalars of a window's column (tv_column) from scalar `off` on.
template <typename T, int R, int C>
SRTM_DEV void col_get(T (&a)[R][C], const T* __restrict__ col, int off) {
#pragma unroll
  for (int r = 0; r < R; ++r)
#pragma unroll
    for (int c = 0; c < C; ++c) a[r][c] = gld(col + (int64_t)(off + r * C + c) * TILE);
}

// Window k's filter element: (F, D, J) from its element record, d = K y_k, eta = C_bar^T R_x^{-1} y_k
// from its block (`blk` and `el` are window k's columns, tv_column); the identity element past
// the last window.
template <typename T, int NX, int NY>
SRTM_DEV void tv_element(const T* __restrict__ blk, const T* __restrict__ el, const TvLayout& lay,
                         const T* __restrict__ y, int64_t k, int64_t N, FElem<T, NX>& a) {
  if (k >= N) {
    elem_identity(a);
    return;
  }
  constexpr int NN = NX * NX;
  col_get(a.F, el, 0);
  col_get(a.D, el, NN);
  col_get(a.J, el, 2 * NN);
  T yk[NY], K[NX][NY], He[NX][NY];
  gloadv(yk, y + k * NY);
  col_get(K, blk, lay.K);
  col_get(He, blk, lay.Heta);
  mv(K, yk, a.d);
  mv(He, yk, a.e);
}

// Per tile: the window constants of every window, then the tile's aggregate a_first (x) ... (x)
// a_last under eq. op-filter by an in-place tree in LDS (TILE whole elements).
template <typename T, int NX, int NY>
SRTM_DEV void tv_reduce_body(const T* __restrict__ Fa, const T* __restrict__ Qa, const T* __restrict__ Ha,
                             const T* __restrict__ Ra, const T* __restrict__ y, int64_t N, int L, T* __restrict__ blks,
                             T* __restrict__ els, T* __restrict__ tagg, int32_t* info, int64_t tile) {
  constexpr int NN = NX * NX, NY2 = NY * NY, NXY = NX * NY, FA = 3 * NN + 2 * NX;
  extern __shared__ char smraw[];
  const Slots<T> S{reinterpret_cast<T*>(smraw), TILE};
  const TvLayout lay = make_tv_layout(NX, NY, L);
  const int bs = lay.total, es = tv_elem_size(NX);
  const int tid = threadIdx.x;
  const int64_t k = tile * TILE + tid;
  int flag = 0;
  if (k < N)
    flag |= tv_window_constants<T, NX, NY>(Fa + k * NN, Qa + k * NN, Ha + k * NXY, Ra + k * NY2, L, lay,
                                           tv_column(blks, k, bs), tv_column(els, k, es), TILE);
  FElem<T, NX> a;
  tv_element<T, NX, NY>(tv_column(blks, k, bs), tv_column(els, k, es), lay, y, k, N, a);
  st_felem(S, tid, a);
  __syncthreads();
#pragma unroll 1
  for (int p = 0; p < LOG_TILE; ++p) {
    const int sp = 1 << p;
    if (tid < (TILE >> (p + 1))) {  // pair j to thread j: the active threads fill the first waves
      const int dst = (tid << (p + 1)) + 2 * sp - 1;
      FElem<T, NX> lft, rgt, o;
      ld_felem(S, dst - sp, lft);
      ld_felem(S, dst, rgt);
      if (!elem_combine(lft, rgt, o)) flag |= SRTM_INFO_COMBINE_SINGULAR;
      st_felem(S, dst, o);
    }
    __syncthreads();
  }
  if (tid == TILE - 1) {
    FElem<T, NX> o;
    ld_felem(S, tid, o);
    T* dst = tagg + tile * FA;
#pragma unroll
    for (int r = 0; r < NX; ++r) {
      put_global(dst + NN + r, o.d[r]);
      put_global(dst + 2 * NN + NX + r, o.e[r]);
#pragma unroll
      for (int c = 0; c < NX; ++c) {
        put_global(dst + r * NX + c, o.F[r][c]);
        put_global(dst + NN + NX + r * NX + c, o.D[r][c]);
        put_global(dst + 2 * NN + 2 * NX + r * NX + c, o.J[r][c]);
      }
    }
  }
  if (flag && info) atomicOr(info, flag);
}

template <typename T, int NX>
SRTM_DEV void ld_felem_global(const T* __restrict__ src, FElem<T, NX>& a) {
  constexpr int NN = NX * NX;
#pragma unroll
  for (int r = 0; r < NX; ++r) {
    a.d[r] = gld(src + NN + r);
    a.e[r] = gld(src + 2 * NN + NX + r);
#pragma unroll
    for (int c = 0; c < NX; ++c) {
      a.F[r][c] = gld(src + r * NX + c);
      a.D[r][c] = gld(src + NN + NX + r * NX + c);
      a.J[r][c] = gld(src + 2 * NN + 2 * NX + r * NX + c);
    }
  }
}

// One workgroup of KS threads: Kogge-Stone scan of the tile aggregates (whole elements). Thread
// tau folds its chunk of 2^lchunk tiles; the prior is folded into thread 0, which makes it a
// state; at step q threads [2^q, 2^{q+1}) combine the state of thread tau - 2^q with their run and
// the others merge two runs (eq. op-filter). Each thread then walks its chunk from its exclusive
// state, writing every tile's incoming state.
template <typename T, int NX>
SRTM_DEV void tv_tiles_body(const T* __restrict__ tagg, int64_t nt, int lchunk, int steps, const T* __restrict__ m0,
                            const T* __restrict__ P0, T* __restrict__ tstate, int32_t* info) {
  constexpr int NN = NX * NX, ST = NX + NN, FA = 3 * NN + 2 * NX;
  extern __shared__ char smraw[];
  const Slots<T> S{reinterpret_cast<T*>(smraw), KS};
  const int tid = threadIdx.x;
  const int64_t c = int64_t(1) << lchunk;
  const int64_t t0 = tid * c;
  int flag = 0;
  FElem<T, NX> run;
  elem_identity(run);
  T m[NX], P[NX][NX];  // a state once the thread's run reaches back to the prior
#pragma unroll
  for (int r = 0; r < NX; ++r) {
    m[r] = T(0);
#pragma unroll
    for (int cc = 0; cc < NX; ++cc) P[r][cc] = T(0);
  }
#pragma unroll 1
  for (int64_t j = 0; j < c; ++j) {
    const int64_t t = t0 + j;
    if (t >= nt) break;
    FElem<T, NX> b;
    ld_felem_global(tagg + t * FA, b);
    if (j == 0) {
      run = b;
    } else if (!elem_combine(run, b, run)) {
      flag |= SRTM_INFO_COMBINE_SINGULAR;
    }
  }
  if (tid == 0) {
    gloadv(m, m0);
    gload(P, P0);
    symmetrize(P);
    if (!state_combine(m, P, run.F, run.d, run.D, run.e, run.J)) flag |= SRTM_INFO_COMBINE_SINGULAR;
  }
#pragma unroll 1
  for (int q = 0; q < steps; ++q) {
    const int sp = 1 << q;
    if (tid < sp) {
      st_state<T, NX>(S, tid, m, P);
    } else {
      st_felem(S, tid, run);
    }
    __syncthreads();
    if (tid >= sp && tid < 2 * sp) {
      ld_state<T, NX>(S, tid - sp, m, P);
      if (!state_combine(m, P, run.F, run.d, run.D, run.e, run.J)) flag |= SRTM_INFO_COMBINE_SINGULAR;
    } else if (tid >= 2 * sp) {
      FElem<T, NX> lft;
      ld_felem(S, tid - sp, lft);
      if (!elem_combine(lft, run, run)) flag |= SRTM_INFO_COMBINE_SINGULAR;
    }
    __syncthreads();
  }
  st_state<T, NX>(S, tid, m, P);  // every thread now holds the inclusive state through its chunk
  __syncthreads();
  if (t0 < nt) {
    T X[NX], XP[NX][NX];
    if (tid == 0) {
      gloadv(X, m0);
      gload(XP, P0);
      symmetrize(XP);
    } else {
      ld_state<T, NX>(S, tid - 1, X, XP);
    }
#pragma unroll 1
    for (int64_t t = t0; t < t0 + c && t < nt; ++t) {
#pragma unroll
      for (int r = 0; r < NX; ++r) put_global(tstate + t * ST + r, X[r]);
#pragma unroll
      for (int r = 0; r < NX; ++r)
#pragma unroll
        for (int cc = 0; cc < NX; ++cc) put_global(tstate + t * ST + NX + r * NX + cc, XP[r][cc]);
      if (t + 1 < t0 + c && t + 1 < nt) {
        FElem<T, NX> b;
        ld_felem_global(tagg + t * FA, b);
        if (!state_combine(X, XP, b.F, b.d, b.D, b.e, b.J)) flag |= SRTM_INFO_COMBINE_SINGULAR;
      }
    }
  }
  if (flag && info) atomicOr(info, flag);
}

// Per tile: an in-tile inclusive Kogge-Stone scan of the windows' elements, then each window's
// exclusive and inclusive filter states from the tile's incoming state; the carry (and slow
// filter outputs); with SMOOTH the smoother half of the fused kernel, with the next window's
// F and Q as the model of the step into x_{k+1,1}.
template <typename T, int NX, int NY, bool SMOOTH>
SRTM_DEV void tv_fwd_body(const T* __restrict__ Fa, const T* __restrict__ Qa, const T* __restrict__ Ha,
                          const T* __restrict__ y, int64_t N,
                          int L, const T* __restrict__ blks, const T* __restrict__ els, const T* __restrict__ m0,
                          const T* __restrict__ P0, const T* __restrict__ ftstate, T* __restrict__ carry,
                          T* __restrict__ m_slow, T* __restrict__ P_slow, T* __restrict__ btagg, T* __restrict__ sfx,
                          int32_t* info, int64_t tile) {
  constexpr int NN = NX * NX, ST = NX + NN;
  extern __shared__ char smraw[];
  const Slots<T> S{reinterpret_cast<T*>(smraw), TILE};
  const TvLayout lay = make_tv_layout(NX, NY, L);
  const int tid = threadIdx.x;
  const int64_t k = tile * TILE + tid;
  const bool valid = k < N;
  const int64_t kc = valid ? k : 0;
  int flag = 0;
  const int bs = lay.total, es = tv_elem_size(NX);
  FElem<T, NX> a, x;
  tv_element<T, NX, NY>(tv_column(blks, k, bs), tv_column(els, k, es), lay, y, k, N, a);
  x = a;
#pragma unroll 1
  for (int sp = 1; sp < TILE; sp *= 2) {  // x <- a_first (x) ... (x) a_k
    st_felem(S, tid, x);
    __syncthreads();
    FElem<T, NX> lft;
    if (tid >= sp) ld_felem(S, tid - sp, lft);
    __syncthreads();
    if (tid >= sp && !elem_combine(lft, x, x)) flag |= SRTM_INFO_COMBINE_SINGULAR;
  }
  st_felem(S, tid, x);
  __syncthreads();
  T mprev[NX], Pprev[NX][NX], m[NX], P[NX][NX];
  {
    gloadv(mprev, ftstate + tile * ST);
    gload(Pprev, ftstate + tile * ST + NX);
    symmetrize(Pprev);
    if (tid > 0) {
      FElem<T, NX> ex;
      ld_felem(S, tid - 1, ex);
      if (!state_combine(mprev, Pprev, ex.F, ex.d, ex.D, ex.e, ex.J)) flag |= SRTM_INFO_COMBINE_SINGULAR;
    }
    if (k == 0) {  // the prior itself
      gloadv(mprev, m0);
      gload(Pprev, P0);
      symmetrize(Pprev);
    }
#pragma unroll
    for (int r = 0; r < NX; ++r) {
      m[r] = mprev[r];
#pragma unroll
      for (int c = 0; c < NX; ++c) P[r][c] = Pprev[r][c];
    }
    if (!state_combine(m, P, a.F, a.d, a.D, a.e, a.J)) flag |= SRTM_INFO_COMBINE_SINGULAR;
  }
  if (valid) flag |= store_carry(k, m, P, carry, m_slow, P_slow);
  if constexpr (SMOOTH) {
    __syncthreads();  // the slots switch from forward elements to smoother elements
    const TvModel<T, NX, NY> M{tv_tile_base(blks, k, bs), lay, (int)(k % TILE), Fa + kc * NN, Qa + kc * NN,
                               Ha + kc * NX * NY};
    T yt[NY];
#pragma unroll
    for (int r = 0; r < NY; ++r) yt[r] = valid ? gld(y + k * NY + r) : T(0);
    T An[NX][NX], Qn[NX][NX];
    const int64_t kn = (k + 1 < N) ? k + 1 : kc;  // the last window's element ignores them
    gload(An, Fa + kn * NN);
    gload(Qn, Qa + kn * NN);
    Window<T, NX, NY> w;
    if (!window_setup(M, L, mprev, Pprev, yt, w) && valid) flag |= SRTM_INFO_INNOVATION_NOT_PD;
    flag |= smoother_part<false>(M, S, L, k, N, w, m, P, An, Qn, btagg, sfx, tile);
  }
  if (flag && info) atomicOr(info, flag);
}

// ============================================================================ lag-one cross-covariances
// U_i = A^i V + c_i, the cross-covariance of x_{k,i} with y_k given y_{1:k-1}.
template <typename T, int NX, int NY>
SRTM_DEV void window_U(const Model<T, NX, NY>& M, const Window<T, NX, NY>& w, int i, T (&Ui)[NX][NY]) {
  const T* pi = M.per_i(i);
  T Ai[NX][NX], ci[NX][NY];
  load(Ai, pi + M.lay.o_Ai);
  load(ci, pi + M.lay.o_ci);
  mm(Ai, w.V, Ui);
#pragma unroll
  for (int r = 0; r < NX; ++r)
#pragma unroll
    for (int c = 0; c < NY; ++c) Ui[r][c] += ci[r][c];
}

// Across the window boundary, x_{k-1,l} (x_0 for the first window) given x_{k,1}, with (m, P) the
// filter state of x_{k-1,l}: the one-step smoother gain G = P A^T (P^-)^{-1}, P^- = A P A^T + Q,
// E[x_{k-1,l} | y_{1:N}] = m + G (m^s_{k,1} - A m) and Cov(x_{k,1}, x_{k-1,l} | y_{1:N}) = P^s_{k,1} G^T
// (eq. seq-smoothing-all for one step). Returns false when P^- is singular.
template <typename T, int NX>
SRTM_DEV bool lag1_boundary(const T (&A)[NX][NX], const T (&Qq)[NX][NX], const T (&m)[NX], const T (&P)[NX][NX],
                            const T (&ms)[NX], const T (&Ps)[NX][NX], T (&G)[NX][NX], T (&Pm)[NX][NX], T (&mb)[NX],
                            T (&C)[NX][NX]) {
  T Pmi[NX][NX], PA[NX][NX];
  sandwich(A, P, Qq, Pm);
  const bool ok = spd_inv(Pm, Pmi);
  mm_nt(P, A, PA);
  mm(PA, Pmi, G);
  T Am[NX], dm[NX];
  mv(A, m, Am);
#pragma unroll
  for (int r = 0; r < NX; ++r) dm[r] = ms[r] - Am[r];
  mv(G, dm, mb);
#pragma unroll
  for (int r = 0; r < NX; ++r) mb[r] += m[r];
  mm_nt(Ps, G, C);
  return ok;
}

// Inside window k, fast step i >= 2: Cov(x_{k,i}, x_{k,i-1} | y_{1:k}) = A P^f_{i-1,i-1}
// + (A c_{i-1} - c_i) S^{-1} U_{i-1}^T (x_{k,i} = A x_{k,i-1} + w, conditioned on y_k), plus the smoothing
// term P^f_{i,l} W P^f_{i-1,l}^T (PLW = P^f_{i,l} W): Cov(x_{k,i}, x_{k,i-1} | y_{1:N}).
template <typename T, int NX, int NY>
SRTM_DEV void lag1_within(const Model<T, NX, NY>& M, const Window<T, NX, NY>& w, int i, const T (&A)[NX][NX],
                          const T (&Pprev)[NX][NX], const T (&Uprev)[NX][NY], const T (&PLW)[NX][NX],
                          const T (&PLprev)[NX][NX], T (&C)[NX][NX]) {
  T Dc[NX][NY], SU[NY][NX];
  {
    T cp[NX][NY], ci[NX][NY];
    load(cp, M.per_i(i - 1) + M.lay.o_ci);
    load(ci, M.per_i(i) + M.lay.o_ci);
    mm(A, cp, Dc);
#pragma unroll
    for (int r = 0; r < NX; ++r)
#pragma unroll
      for (int c = 0; c < NY; ++c) Dc[r][c] -= ci[r][c];
  }
#pragma unroll
  for (int r = 0; r < NY; ++r)
#pragma unroll
    for (int c = 0; c < NX; ++c) {
      T t = T(0);
#pragma unroll
      for (int q = 0; q < NY; ++q) t = my_fma(symget(w.Si, r, q), Uprev[c][q], t);
      SU[r][c] = t;
    }
  mm(A, Pprev, C);
#pragma unroll
  for (int r = 0; r < NX; ++r)
#pragma unroll
    for (int c = 0; c < NX; ++c) {
      T t = C[r][c];
#pragma unroll
      for (int q = 0; q < NY; ++q) t = my_fma(Dc[r][q], SU[q][c], t);
#pragma unroll
      for (int q = 0; q < NX; ++q) t = my_fma(PLW[r][q], PLprev[c][q], t);
      C[r][c] = t;
    }
}

// K8 (optional output): per tile, the lag-one smoothed cross-covariances of every fast step of
// its windows, Cs_fast[k][i-1] = Cov(x_{k,i}, x_{k,i-1} | y_{1:N}) with x_{k,0} = x_{k-1,l} and the prior
// state x_0 for the first window (Remark cross-covariances), from the same window quantities,
// carry and smoother correction (v, W) as the recovery; records staged and written as K7's.
template <typename T, int NX, int NY>
SRTM_DEV void lag1_body(const T* __restrict__ y, int64_t N, int L, const T* __restrict__ cst,
                        const T* __restrict__ carry, const T* __restrict__ sfx, const T* __restrict__ utree,
                        T* __restrict__ Cs_fast, int32_t* info, int64_t tile, int part, int nparts,
                        int nslow) {
  static_assert(TILE == 256, "one workgroup per tile");
  constexpr int NN = NX * NX;
  using Stg = OutStage<T, NX>;
  extern __shared__ char smraw[];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int64_t k = tile * TILE + tid;
  const int64_t w0 = tile * TILE + wv * 64;
  const Model<T, NX, NY> M{cst, make_const_layout(NX, NY, L)};
  const int nvalid = (int)((N - w0) < 64 ? ((N - w0) > 0 ? (N - w0) : 0) : 64);
  const Stg stg(smraw + (size_t)wv * Stg::BYTES);
  const bool valid = k < N;
  const int64_t kc = valid ? k : 0;
  T m[NX], P[NX][NX], yk[NY];
  const int nw = tile_windows(N, tile);
  const bool settled = tile_settled<T, NX>(utree, tile);
  int ibeg = 1, iend = L;  // this workgroup's fast steps
  {
    const StepShare<NX> share(L, part, nparts, nslow, settled);
    if (share.beg > L) return;
    ibeg = share.beg;
    iend = share.end;
  }
  const int64_t col = tile * (TILE * info_stride(NX)) + (valid ? tid : 0);  // the window's records
  const int64_t mcol = settled ? tile * (TILE * info_stride(NX)) : col;
  record_load(m, P, carry + col, carry + mcol, nw);
  gloadv(yk, y + kc * NY);
  Window<T, NX, NY> w;
  int flag = 0;
  if (!window_setup(M, L, m, P, yk, w) && valid) flag |= SRTM_INFO_INNOVATION_NOT_PD;
  T v[NX], W[NX][NX];
  const T zero[NX] = {};
  if (!info_correction<false>(M, L, w, zero, sfx + col, sfx + mcol, nw, v, W) && valid) flag |= SRTM_INFO_COMBINE_SINGULAR;
  T A[NX][NX];
  load(A, M.cst + M.lay.A);
  T Pprev[NX][NX], PLprev[NX][NX], Uprev[NX][NY];
  bool fin = true;
  auto seed = [&](int i) {  // what step i + 1 needs of step i
    T mf[NX];
    window_step<T, NX, NY, true>(M, w, i, mf, Pprev, PLprev);
    window_U(M, w, i, Uprev);
  };
  auto cross = [&](int i, T (&C)[NX][NX]) {  // step i's cross-covariance, from the state that seed or cross left
    T mf[NX], Pii[NX][NX], PiL[NX][NX], PLW[NX][NX];
    window_step<T, NX, NY, true>(M, w, i, mf, Pii, PiL);
    mm(PiL, W, PLW);
    if (i == 1) {  // across the window boundary, from the smoothed block of x_{k,1}
      T ms[NX], Ps[NX][NX], Qq[NX][NX], G[NX][NX], Pm[NX][NX], mb[NX];
#pragma unroll
      for (int r = 0; r < NX; ++r) {
        T t = mf[r];
#pragma unroll
        for (int q = 0; q < NX; ++q) t = my_fma(PiL[r][q], v[q], t);
        ms[r] = t;
#pragma unroll
        for (int c = r; c < NX; ++c) {
          T u = Pii[r][c];
#pragma unroll
          for (int q = 0; q < NX; ++q) u = my_fma(PLW[r][q], PiL[c][q], u);
          Ps[r][c] = u;
          Ps[c][r] = u;
        }
      }
      load(Qq, M.cst + M.lay.Q);
      if (!lag1_boundary(A, Qq, m, P, ms, Ps, G, Pm, mb, C) && valid) flag |= SRTM_INFO_PRED_SINGULAR;
    } else {
      lag1_within(M, w, i, A, Pprev, Uprev, PLW, PLprev, C);
    }
#pragma unroll
    for (int r = 0; r < NX; ++r)
#pragma unroll
      for (int c = 0; c < NX; ++c) fin = fin && isfinite(C[r][c]);
    window_U(M, w, i, Uprev);
#pragma unroll
    for (int r = 0; r < NX; ++r)
#pragma unroll
      for (int c = 0; c < NX; ++c) {
        Pprev[r][c] = Pii[r][c];
        PLprev[r][c] = PiL[r][c];
      }
  };
  if (settled) {  // a thread per fast step, then every wave writes the records to its 64 windows (Stream)
    constexpr int SC = 24, RB = NN * (int)sizeof(T);
    static_assert(SC * RB <= 64 * Stg::SBP, "the records fit one wave's staging");
#pragma unroll 1
    for (int i0 = ibeg; i0 <= iend; i0 += SC) {
      const int ns = iend - i0 + 1 < SC ? iend - i0 + 1 : SC;
      __syncthreads();  // the previous records are written
      if (tid < ns) {
        T C[NX][NX];
        if (i0 + tid > 1) seed(i0 + tid - 1);
        cross(i0 + tid, C);
        T* o = reinterpret_cast<T*>(smraw + tid * RB);
#pragma unroll
        for (int r = 0; r < NX; ++r)
#pragma unroll
          for (int c = 0; c < NX; ++c) o[r * NX + c] = C[r][c];
      }
      __syncthreads();
      Stream<RB> st(lane, ns, L);
#pragma unroll 1
      for (int j = 0; j < ns; ++j) st.put(smraw, reinterpret_cast<char*>(Cs_fast) + (w0 * L + (i0 - 1)) * RB);
    }
    if (!fin) flag |= SRTM_INFO_NONFINITE;
    if (flag && info) atomicOr(info, flag);
    return;
  }
  if (ibeg > 1) seed(ibeg - 1);
#pragma unroll 1
  for (int i = ibeg; i <= iend; ++i) {
    T C[NX][NX];
    cross(i, C);
    stg.put(lane, i - ibeg, zero, C);
    wave_sync();
    stg.flush(lane, nvalid, nullptr, Cs_fast, w0, L, i - ibeg, i, iend);
    wave_sync();
  }
  if (!fin && valid) flag |= SRTM_INFO_NONFINITE;
  if (flag && info) atomicOr(info, flag);
}

// ============================================================================ log-likelihood and gradient
// Marginal log-likelihood log p(y_{1:N}) = sum_k log N(y_k; C_bar m^f_{k-1,l}, S_k) (the IMKF
// prediction of y_k, eq. m-h-k-l), and its gradient with respect to F, Q and R by Fisher's
// identity: the gradient of log p(y | theta) is the expectation, under the smoothing
// distribution, of the gradient of the complete-data log-density
//   log p(x_0) + sum_t log N(x_t; F x_{t-1}, Q) + sum_k log N(y_k; (H/l) sum_i x_{k,i}, R).
// Written with the process noise w_t = x_t - F x_{t-1} and the measurement residual
// r_k = y_k - H xbar_k (xbar_k the window average):
//   dll/dF = Q^{-1} sum_t E[w_t x_{t-1}^T],
//   dll/dQ = 1/2 Q^{-1} sum_t (E[w_t w_t^T] - Q) Q^{-1},   dll/dR = 1/2 R^{-1} sum_k (E[r_k r_k^T] - R) R^{-1}
// (expectations under p(. | y_{1:N}); symmetric-matrix gradients for Q and R: dll = tr(G dQ)).
// The summands are formed per fast step directly in their centred form, from quantities that
// scale with Q and R, never as differences of second moments of the states: near the data's
// own parameters the sums nearly vanish, and differences of state moments would carry the
// rounding of the states into the gradient multiplied by the number of steps.
//
// Per window k, with the window prior (m, P) of x_{k,0} = x_{k-1,l}, S, e and U_i as in
// eq. update-fast, the noise w_i = x_{k,i} - F x_{k,i-1} of fast step i has
//   Cov(w_i, y_k | y_{1:k-1}) = b_i = c_i - F c_{i-1}   (c_0 = 0),
//   Cov(w_i, x_{k,l} | y_{1:k}) = K_i = Q (F^{l-i})^T - b_i S^{-1} U_l^T,
// and the future measurements reach the window only through x_{k,l} (the smoother correction
// v_k, W_k of eq. seq-smoothing-all), so under p(. | y_{1:N}):
//   E[w_i] = mu_i = b_i S^{-1} e + K_i v,   E[w_i w_i^T] - Q = -b_i S^{-1} b_i^T + K_i W K_i^T + mu_i mu_i^T,
//   E[w_i x_{k,i-1}^T] = -b_i S^{-1} U_{i-1}^T + K_i W P^f_{k,i-1,l}^T + mu_i m^s_{k,i-1}^T
// with U_0 = P C_bar^T, P^f_{k,0,l} = P F^{lT} - U_0 S^{-1} U_l^T and m^s_{k,i-1} = m^f_{k,i-1} + P^f_{k,i-1,l} v.
// The measurement residual: E[r_k] = R S^{-1} e - Z v and E[r_k r_k^T] - R = E[r_k] E[r_k]^T - R S^{-1} R
// + Z W Z^T with Z = R S^{-1} U_l^T.
// These statistics are computed in float64 for both element types, from the float64 copy of the
// model constants and the stored carry and smoother correction.
//
// Per-tile record (float64): ll, then (gradient) the tile sums of E[w w^T] - Q, E[w x^T] and
// E[r r^T] - R.
template <int NX, int NY>
struct StatLayout {
  static constexpr int NN = NX * NX;
  static constexpr int LL = 0, SW = 1, SWX = 1 + NN, SY = 1 + 2 * NN, SIZE = SY + NY * NY;
};

template <typename T, int N>
SRTM_DEV T det_small(const T (&a)[N][N]) {
  static_assert(N >= 1 && N <= 2, "det_small: N <= 2");
  if constexpr (N == 1)
    return a[0][0];
  else
    return a[0][0] * a[1][1] - a[0][1] * a[1][0];
}

template <typename T, int R, int C>
SRTM_DEV void gload_f64(double (&a)[R][C], const T* __restrict__ p) {
#pragma unroll
  for (int r = 0; r < R; ++r)
#pragma unroll
    for (int c = 0; c < C; ++c) a[r][c] = (double)gld(p + r * C + c);
}
template <typename T, int R>
SRTM_DEV void gloadv_f64(double (&a)[R], const T* __restrict__ p) {
#pragma unroll
  for (int r = 0; r < R; ++r) a[r] = (double)gld(p + r);
}

// Gradient statistics of window k (float64), added to Sw, Swx, Sy; the window's log-likelihood
// term in *ll. (m, P): its prior; yk: its measurement (y_k - mu_k with known inputs); col: its
// information record (columns col and mcol, element type T, in a tile of nw windows), or its smoother-correction record with the
// tile's incoming smoothed state `ti` (grad_by_elements); okc: whether the correction from it is usable; zL: its input
// response z_{k,l}; with known inputs Bm [nx][nu] and uk, the window's inputs [L][nu]. `tab`: LDS for the tables of
// up to RSTEPS fast steps, which all threads of the workgroup copy (stats_lds_bytes): as wave-uniform loads the
// six matrices of a step outgrow the scalar registers.
template <typename T, int NX, int NY>
SRTM_DEV bool grad_window(const Model<double, NX, NY>& M, int L, const double (&m)[NX], const double (&P)[NX][NX],
                          const double (&yk)[NY], const double (&R)[NY][NY], const T* __restrict__ col,
                          const T* __restrict__ mcol, int nw, const T* __restrict__ ti, const double (&zL)[NX], bool& okc, double& ll, double (&Sw)[NX][NX], double (&Swx)[NX][NX],
                          double (&Sy)[NY][NY], double* tab, const T* __restrict__ Bm = nullptr, const T* __restrict__ uk = nullptr,
                          int nu = 0) {
  Window<double, NX, NY> w;
  const bool ok = window_setup(M, L, m, P, yk, w);
  double e[NY];
  {
    double Cb[NY][NX];
    M.get(Cb, M.lay.Cbar);
    double quad = 0.0;
#pragma unroll
    for (int r = 0; r < NY; ++r) {
      double t = yk[r];
#pragma unroll
      for (int c = 0; c < NX; ++c) t = fma(-Cb[r][c], m[c], t);
      e[r] = t;
      quad += t * w.Se[r];
    }
    ll = -0.5 * (quad - log(det_small(w.Si)) + NY * 1.8378770664093453);  // log(2 pi)
  }
  double v[NX], W[NX][NX];
  if constexpr (grad_by_elements<T>()) {  // v = Et m_in + gt, W = Et P_in Et^T + St (smoother_part)
    constexpr int NN = NX * NX;
    okc = true;
    double Et[NX][NX], mi[NX], Pi[NX][NX], EP[NX][NX];
    gload_f64(Et, col);
    gloadv_f64(mi, ti);
    gload_f64(Pi, ti + NX);
#pragma unroll
    for (int r = 0; r < NX; ++r) {
      double t = (double)gld(col + NN + r);
#pragma unroll
      for (int q = 0; q < NX; ++q) t = fma(Et[r][q], mi[q], t);
      v[r] = t;
    }
    mm(Et, Pi, EP);
    int o = NN + NX;
#pragma unroll
    for (int r = 0; r < NX; ++r)
#pragma unroll
      for (int c = r; c < NX; ++c) {
        double t = (double)gld(col + o++);
#pragma unroll
        for (int q = 0; q < NX; ++q) t = fma(EP[r][q], Et[c][q], t);
        W[r][c] = t;
        W[c][r] = t;
      }
  } else {
    okc = info_correction<true>(M, L, w, zL, col, mcol, nw, v, W);
  }
  double A[NX][NX], Qm[NX][NX];
  M.get(A, M.lay.A);
  M.get(Qm, M.lay.Q);
  // step i-1 quantities: U_{i-1}, P^f_{k,i-1,l}, m^f_{k,i-1}, c_{i-1}; zin: input response z_{i-1}
  double Up[NX][NY], PLp[NX][NX], mfp[NX], cp[NX][NY], zin[NX];
#pragma unroll
  for (int r = 0; r < NX; ++r) {
    zin[r] = 0.0;
    mfp[r] = w.mp[r];
#pragma unroll
    for (int c = 0; c < NY; ++c) {
      Up[r][c] = w.V[r][c];
      cp[r][c] = 0.0;
    }
#pragma unroll
    for (int c = 0; c < NX; ++c) PLp[r][c] = w.Y1[r][c];
  }
#pragma unroll 1
  for (int i = 1; i <= L; ++i) {
    const int st = M.lay.per_i_stride, slot = (i - 1) % RSTEPS;
    double* tabA = tab + (L < RSTEPS ? L : RSTEPS) * st;  // A^{l-i} of the same steps
    if (slot == 0) {
      const int n = L - i + 1 < RSTEPS ? L - i + 1 : RSTEPS;
      const double* src = M.per_i(i);
      __syncthreads();  // the previous steps are done
      staged_copy<4, double>(n * st, threadIdx.x, TILE, [&](int q) { return gld(src + q); }, [&](int q, double x) { tab[q] = x; });
      staged_copy<4, double>(n * NX * NX, threadIdx.x, TILE,
                             [&](int q) {
                               const int back = L - i - q / (NX * NX);
                               return back > 0 ? gld(M.cst + M.per_i_off(back) + M.lay.o_Ai + q % (NX * NX)) : 0.0;
                             },
                             [&](int q, double x) { tabA[q] = x; });
      __syncthreads();
    }
    const double* ps = tab + slot * st;
    double ci[NX][NY], b[NX][NY], Kq[NX][NX];
    load(ci, ps + M.lay.o_ci);
#pragma unroll
    for (int r = 0; r < NX; ++r)
#pragma unroll
      for (int c = 0; c < NY; ++c) {
        double t = ci[r][c];
#pragma unroll
        for (int q = 0; q < NX; ++q) t = fma(-A[r][q], cp[q][c], t);
        b[r][c] = t;
      }
    // K_i = Q (A^{l-i})^T - b_i Y2 (Y2 = S^{-1} U_l^T)
    if (i < L) {
      double As[NX][NX];
      load(As, tabA + slot * NX * NX);
      mm_nt(Qm, As, Kq);
    } else {
#pragma unroll
      for (int r = 0; r < NX; ++r)
#pragma unroll
        for (int c = 0; c < NX; ++c) Kq[r][c] = Qm[r][c];
    }
#pragma unroll
    for (int r = 0; r < NX; ++r)
#pragma unroll
      for (int c = 0; c < NX; ++c) {
        double t = Kq[r][c];
#pragma unroll
        for (int q = 0; q < NY; ++q) t = fma(-b[r][q], w.Y2[q][c], t);
        Kq[r][c] = t;
      }
    double bS[NX][NY], mu[NX], KW[NX][NX], msp[NX];
#pragma unroll
    for (int r = 0; r < NX; ++r)
#pragma unroll
      for (int c = 0; c < NY; ++c) {
        double t = 0.0;
#pragma unroll
        for (int q = 0; q < NY; ++q) t = fma(b[r][q], symget(w.Si, q, c), t);
        bS[r][c] = t;
      }
    mm(Kq, W, KW);
#pragma unroll
    for (int r = 0; r < NX; ++r) {
      double t = 0.0, s2 = mfp[r];
#pragma unroll
      for (int q = 0; q < NY; ++q) t = fma(b[r][q], w.Se[q], t);
#pragma unroll
      for (int q = 0; q < NX; ++q) {
        t = fma(Kq[r][q], v[q], t);
        s2 = fma(PLp[r][q], v[q], s2);
      }
      mu[r] = t;
      msp[r] = s2;
    }
#pragma unroll
    for (int r = 0; r < NX; ++r)
#pragma unroll
      for (int c = 0; c < NX; ++c) {
        double sw = mu[r] * mu[c], sx = mu[r] * msp[c];
#pragma unroll
        for (int q = 0; q < NY; ++q) {
          sw = fma(-bS[r][q], b[c][q], sw);
          sx = fma(-bS[r][q], Up[c][q], sx);
        }
#pragma unroll
        for (int q = 0; q < NX; ++q) {
          sw = fma(KW[r][q], Kq[c][q], sw);
          sx = fma(KW[r][q], PLp[c][q], sx);
        }
        Sw[r][c] += sw;
        Swx[r][c] += sx;
      }
    // step i's own blocks for the next step; with known inputs the fast-step means also carry the
    // input response z_i = A z_{i-1} + B u_{k,i-1} (z_0 = 0), the noise statistics do not change
    if (i < L) {
      double Ai[NX][NX], Pii[NX][NX];
      load(Ai, ps + M.lay.o_Ai);
      step_blocks<true>(
          w, Ai, ci, [&](int r, int c) { return ps[M.lay.o_Qii + r * NX + c]; },
          [&](int r, int c) { return ps[M.lay.o_QiL + r * NX + c]; }, mfp, Pii, PLp);
      mm(Ai, w.V, Up);
#pragma unroll
      for (int r = 0; r < NX; ++r)
#pragma unroll
        for (int c = 0; c < NY; ++c) Up[r][c] += ci[r][c];
      if (uk) {
        double nz[NX];
#pragma unroll
        for (int r = 0; r < NX; ++r) {
          double t = 0.0;
#pragma unroll
          for (int j = 0; j < NU_MAX; ++j)
            if (j < nu) t = fma((double)gld(Bm + r * nu + j), (double)gld(uk + (i - 1) * nu + j), t);
#pragma unroll
          for (int q = 0; q < NX; ++q) t = fma(A[r][q], zin[q], t);
          nz[r] = t;
        }
#pragma unroll
        for (int r = 0; r < NX; ++r) {
          zin[r] = nz[r];
          mfp[r] += zin[r];
        }
      }
#pragma unroll
      for (int r = 0; r < NX; ++r)
#pragma unroll
        for (int c = 0; c < NY; ++c) cp[r][c] = ci[r][c];
    }
  }
  // measurement residual: E[r] = R S^{-1} e - Z v, E[r r^T] - R = E[r]E[r]^T - R S^{-1} R + Z W Z^T
  {
    double RSi[NY][NY], Z[NY][NX], d[NY], ZW[NY][NX], Si[NY][NY];
#pragma unroll
    for (int r = 0; r < NY; ++r)
#pragma unroll
      for (int c = 0; c < NY; ++c) Si[r][c] = symget(w.Si, r, c);
    mm(R, Si, RSi);
    mm(R, w.Y2, Z);
    mm(Z, W, ZW);
#pragma unroll
    for (int r = 0; r < NY; ++r) {
      double t = 0.0;
#pragma unroll
      for (int q = 0; q < NY; ++q) t = fma(RSi[r][q], e[q], t);
#pragma unroll
      for (int q = 0; q < NX; ++q) t = fma(-Z[r][q], v[q], t);
      d[r] = t;
    }
#pragma unroll
    for (int r = 0; r < NY; ++r)
#pragma unroll
      for (int c = 0; c < NY; ++c) {
        double t = d[r] * d[c];
#pragma unroll
        for (int q = 0; q < NY; ++q) t = fma(-RSi[r][q], R[q][c], t);
#pragma unroll
        for (int q = 0; q < NX; ++q) t = fma(ZW[r][q], Z[c][q], t);
        Sy[r][c] += t;
      }
  }
  return ok;
}

// Dynamic LDS of the statistics kernel with the gradient.
inline size_t stats_lds_bytes(int nx, int ny, int L) {
  return sizeof(double) * (size_t)(L < RSTEPS ? L : RSTEPS) * (make_const_layout(nx, ny, L).per_i_stride + nx * nx);
}

template <typename T, int NX, int NY, bool GRAD, bool INP>
SRTM_DEV void stats_body(const T* __restrict__ y, int64_t N, int L, const T* __restrict__ cst,
                         const double* __restrict__ cst64, InputView<T> in, const T* __restrict__ Rm,
                         const T* __restrict__ m0, const T* __restrict__ P0, const T* __restrict__ carry,
                         const T* __restrict__ sfx, const T* __restrict__ tin, const T* __restrict__ utree,
                         double* __restrict__ parts, int32_t* info, int64_t tile) {
  using SL = StatLayout<NX, NY>;
  constexpr int NC = SL::SIZE;
  __shared__ double red[TILE / 64][NC];
  extern __shared__ char smraw[];
  double* tab = reinterpret_cast<double*>(smraw);
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int64_t k = tile * TILE + tid;
  const bool valid = k < N;
  const int64_t kc = valid ? k : 0;
  const int nw = tile_windows(N, tile);
  const int64_t col = tile * (TILE * info_stride(NX)) + (valid ? tid : 0);  // the window's records
  const int64_t mcol = !(GRAD && grad_by_elements<T>()) && tile_settled<T, NX>(utree, tile)
                           ? tile * (TILE * info_stride(NX)) : col;
  double* part = parts + tile * SL::SIZE;
  int flag = 0;
  double ll = 0.0;
  double Sw[NX][NX], Swx[NX][NX], Sy[NY][NY];
#pragma unroll
  for (int r = 0; r < NX; ++r)
#pragma unroll
    for (int c = 0; c < NX; ++c) Sw[r][c] = Swx[r][c] = 0.0;
#pragma unroll
  for (int r = 0; r < NY; ++r)
#pragma unroll
    for (int c = 0; c < NY; ++c) Sy[r][c] = 0.0;
  if constexpr (GRAD) {
    const Model<double, NX, NY> M{cst64, make_const_layout(NX, NY, L)};
    double m[NX], P[NX][NX], yk[NY], R[NY][NY];
    if constexpr (!grad_by_elements<T>()) {
      record_load(m, P, carry + col, carry + mcol, nw);
    } else if (kc == 0) {
      gloadv_f64(m, m0);
      gload_f64(P, P0);
    } else {
      gloadv_f64(m, carry + (kc - 1) * (NX + NX * NX));
      gload_f64(P, carry + (kc - 1) * (NX + NX * NX) + NX);
    }
    double zL[NX];
#pragma unroll
    for (int r = 0; r < NX; ++r) zL[r] = 0.0;
    if constexpr (INP) {  // y_k - mu_k and z_{k,l} from the tile reductions' per-window record
      gloadv_f64(yk, in.rec + kc * (NY + NX));
      gloadv_f64(zL, in.rec + kc * (NY + NX) + NY);
    } else {
      gloadv_f64(yk, y + kc * NY);
    }
    gload_f64(R, Rm);
    bool okc = true;
    if (!grad_window<T, NX, NY>(M, L, m, P, yk, R, sfx + (grad_by_elements<T>() ? kc * sfx_stride(NX) : col), sfx + mcol, nw,
                                tin + tile * (NX + NX * NX), zL, okc, ll, Sw, Swx, Sy, tab,
                                INP ? in.B : nullptr, INP ? in.u + kc * L * in.nu : nullptr, INP ? in.nu : 0) &&
        valid)
      flag |= SRTM_INFO_INNOVATION_NOT_PD;
    if (!okc && valid) flag |= SRTM_INFO_COMBINE_SINGULAR;
  } else {
    const Model<T, NX, NY> M{cst, make_const_layout(NX, NY, L), in};
    T m[NX], P[NX][NX], yk[NY];
    record_load(m, P, carry + col, carry + mcol, nw);
    if constexpr (INP) {
      T zL[NX];
      window_meas<true>(M, y, kc, N, yk, zL);
    } else {
      gloadv(yk, y + kc * NY);
    }
    Window<T, NX, NY> w;
    if (!window_setup(M, L, m, P, yk, w) && valid) flag |= SRTM_INFO_INNOVATION_NOT_PD;
    T Cb[NY][NX];
    load(Cb, M.cst + M.lay.Cbar);
    double quad = 0.0;
#pragma unroll
    for (int r = 0; r < NY; ++r) {
      T t = yk[r];
#pragma unroll
      for (int c = 0; c < NX; ++c) t = my_fma(-Cb[r][c], m[c], t);
      quad += (double)t * (double)w.Se[r];
    }
    ll = -0.5 * (quad - log((double)det_small(w.Si)) + NY * 1.8378770664093453);  // log(2 pi)
  }
  // tile sums (fixed order: butterfly per wave, then waves 0..3)
  auto comp = [&](int c) -> double {
    if (!valid) return 0.0;
    if (c == SL::LL) return ll;
    if (c < SL::SWX) return Sw[(c - SL::SW) / NX][(c - SL::SW) % NX];
    if (c < SL::SY) return Swx[(c - SL::SWX) / NX][(c - SL::SWX) % NX];
    return Sy[(c - SL::SY) / NY][(c - SL::SY) % NY];
  };
  const int ncomp = GRAD ? NC : 1;
  if constexpr (GRAD) {
    double x[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) x[c] = comp(c);
    int start = 0, cnt = NC;
    wave_sums<NC, 32>(x, lane, start, cnt);
#pragma unroll
    for (int j = 0; j < (NC + 63) / 64; ++j)
      if (j < cnt) red[wv][start + j] = x[j];
  } else {
    const double s = wave_sum(comp(0));
    if (lane == 0) red[wv][0] = s;
  }
  __syncthreads();
  for (int c = tid; c < ncomp; c += blockDim.x) {
    double s = red[0][c];
    for (int q = 1; q < TILE / 64; ++q) s += red[q][c];
    part[c] = s;
  }
  if (flag && info) atomicOr(info, flag);
}

constexpr int SF_THREADS = 512;

// One workgroup per sequence: sums the tile records in a fixed order and forms the outputs
// dF = Q^{-1} Swx, dQ = 1/2 Q^{-1} Sw Q^{-1}, dR = 1/2 R^{-1} Sy R^{-1}.
template <typename T, int NX, int NY, bool GRAD>
SRTM_DEV void stats_final_body(int64_t nt, const T* __restrict__ Qm, const T* __restrict__ Rm,
                               const double* __restrict__ parts, T* __restrict__ ll_out, T* __restrict__ dF,
                               T* __restrict__ dQ, T* __restrict__ dR, int32_t* info) {
  using SL = StatLayout<NX, NY>;
  constexpr int NR = SL::SIZE, NW = SF_THREADS / 64;
  __shared__ double red[NW][NR];
  __shared__ double tot[NR];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int ncomp = GRAD ? NR : 1;
  // The log-likelihood alone: a thread per tile. With the gradient, lane c of a wave sums component c (and
  // c + 64 ..) of tiles wv, wv + NW, ... in order, eight records in flight. The waves' sums are added in
  // order. With a tile per thread and a tree over 256 threads for 16 components at a time the kernel took
  // 17 us for 64 tiles, almost all of it barriers and empty lanes.
  if constexpr (!GRAD) {
    double s = 0.0;
    for (int64_t t = tid; t < nt; t += SF_THREADS) s += gld(parts + t * SL::SIZE + SL::LL);
    s = wave_sum(s);
    if (lane == 0) red[wv][SL::LL] = s;
  } else {
    for (int c = lane; c < ncomp; c += 64) {
      double s = 0.0;
      for (int64_t t0 = wv; t0 < nt; t0 += 8 * NW) {
        double x[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) x[j] = t0 + j * NW < nt ? gld(parts + (t0 + j * NW) * SL::SIZE + c) : 0.0;
#pragma unroll
        for (int j = 0; j < 8; ++j) s += x[j];
      }
      red[wv][c] = s;
    }
  }
  __syncthreads();
  for (int c = tid; c < ncomp; c += SF_THREADS) {
    double s = red[0][c];
#pragma unroll
    for (int q = 1; q < NW; ++q) s += red[q][c];
    tot[c] = s;
  }
  __syncthreads();
  if (tid != 0) return;
  if (ll_out) ll_out[0] = (T)tot[SL::LL];
  if constexpr (GRAD) {
    double Q[NX][NX], R[NY][NY], Qi[NX][NX], Ri[NY][NY], Sw[NX][NX], Swx[NX][NX], Sy[NY][NY];
    for (int r = 0; r < NX; ++r)
      for (int c = 0; c < NX; ++c) {
        Q[r][c] = (double)Qm[r * NX + c];
        Sw[r][c] = tot[SL::SW + r * NX + c];
        Swx[r][c] = tot[SL::SWX + r * NX + c];
      }
    for (int r = 0; r < NY; ++r)
      for (int c = 0; c < NY; ++c) {
        R[r][c] = (double)Rm[r * NY + c];
        Sy[r][c] = tot[SL::SY + r * NY + c];
      }
    symmetrize(Q);
    symmetrize(R);
    symmetrize(Sw);
    symmetrize(Sy);
    int flag = 0;
    if (!spd_inv(Q, Qi)) flag |= SRTM_INFO_PRED_SINGULAR;
    if (!spd_inv(R, Ri)) flag |= SRTM_INFO_INNOVATION_NOT_PD;
    double tmp[NX][NX], G2[NX][NX];
    mm(Qi, Swx, tmp);
    for (int r = 0; r < NX; ++r)
      for (int c = 0; c < NX; ++c) dF[r * NX + c] = (T)tmp[r][c];
    mm(Qi, Sw, tmp);
    mm(tmp, Qi, G2);
    symmetrize(G2);
    for (int r = 0; r < NX; ++r)
      for (int c = 0; c < NX; ++c) dQ[r * NX + c] = (T)(0.5 * G2[r][c]);
    double RS[NY][NY], GR[NY][NY];
    mm(Ri, Sy, RS);
    mm(RS, Ri, GR);
    symmetrize(GR);
    for (int r = 0; r < NY; ++r)
      for (int c = 0; c < NY; ++c) dR[r * NY + c] = (T)(0.5 * GR[r][c]);
    if (flag && info) atomicOr(info, flag);
  }
}

// ============================================================================ kernels
// Every kernel takes the call's Batch. Kernels over sequences run one workgroup per sequence;
// kernels over tiles run one workgroup per tile of any sequence.
template <typename T, int NX, int NY>
struct Seq {  // one sequence's typed arrays and scan plan
  const T *F, *Q, *H, *R, *m0, *P0, *y;
  T *ms_fast, *Ps_fast, *ms_slow, *Ps_slow, *mf_fast, *Pf_fast, *mf_slow, *Pf_slow, *Cs_fast;
  T *cst, *ftagg, *ftst, *utree, *carry, *btagg, *btst, *sfx, *tvblk, *tvel;
  double *cst64, *hand, *stats, *tail, *lev64;
  int64_t N, tile0;
  int L;
  ScanPlan plan;
  bool smoother;
  int32_t* info;
  InputView<T> in;
};

template <typename T, int NX, int NY>
SRTM_DEV Seq<T, NX, NY> seq_view(const Batch& b, int s) {
  const SeqDesc d = b.table ? b.table[s] : b.one;
  Seq<T, NX, NY> q;
  q.F = as_global<T>(d.F);
  q.Q = as_global<T>(d.Q);
  q.H = as_global<T>(d.H);
  q.R = as_global<T>(d.R);
  q.m0 = as_global<T>(d.m0);
  q.P0 = as_global<T>(d.P0);
  q.y = as_global<T>(d.y);
  q.ms_fast = as_global<T>(d.ms_fast);
  q.Ps_fast = as_global<T>(d.Ps_fast);
  q.ms_slow = as_global<T>(d.ms_slow);
  q.Ps_slow = as_global<T>(d.Ps_slow);
  q.mf_fast = as_global<T>(d.mf_fast);
  q.Pf_fast = as_global<T>(d.Pf_fast);
  q.mf_slow = as_global<T>(d.mf_slow);
  q.Pf_slow = as_global<T>(d.Pf_slow);
  q.Cs_fast = as_global<T>(d.Cs_fast);
  q.N = d.N;
  q.tile0 = d.tile0;
  q.L = d.L;
  q.plan = make_scan_plan(d.N);
  const WorkLayout wl = make_work_layout(NX, NY, d.L, d.N, sizeof(T), d.smoother != 0, d.B != nullptr, d.tv != 0);
  char* base = as_global(b.ws) + d.ws_off;
  q.cst = reinterpret_cast<T*>(base + wl.consts);
  q.cst64 = reinterpret_cast<double*>(base + wl.consts64);
  q.hand = reinterpret_cast<double*>(base + wl.chain);
  q.ftagg = reinterpret_cast<T*>(base + wl.ftile_agg);
  q.ftst = reinterpret_cast<T*>(base + wl.ftile_state);
  q.utree = reinterpret_cast<T*>(base + wl.utree);
  q.carry = reinterpret_cast<T*>(base + wl.carry);
  q.btagg = reinterpret_cast<T*>(base + wl.btile_agg);
  q.btst = reinterpret_cast<T*>(base + wl.btile_state);
  q.sfx = reinterpret_cast<T*>(base + wl.sfx);
  q.tail = reinterpret_cast<double*>(base + wl.sfx + tail_info_off(d.N, NX, sizeof(T)));
  q.smoother = d.smoother != 0;
  q.lev64 = has_lev64<T, NX>(d.N) ? reinterpret_cast<double*>(base + wl.carry + lev64_off(d.N, NX, sizeof(T))) : nullptr;
  q.tvblk = reinterpret_cast<T*>(base + wl.tvblk);
  q.tvel = reinterpret_cast<T*>(base + wl.tvel);
  q.stats = reinterpret_cast<double*>(base + wl.stats);
  q.info = b.info ? b.info + s : nullptr;
  q.in = InputView<T>{as_global<T>(d.B), as_global<T>(d.u), q.H,
                      d.B ? reinterpret_cast<T*>(base + wl.inp) : nullptr, d.nu};
  return q;
}

SRTM_DEV int tile_sequence(const Batch& b, int64_t bid) { return b.tile_seq ? b.tile_seq[bid] : 0; }
SRTM_DEV int tile_sequence(const Batch& b) { return tile_sequence(b, blockIdx.x); }
// Tile of a sequence of nt tiles for its i-th workgroup, both ends first (0, nt - 1, 1, nt - 2, ...): the
// tiles that are not settled, next to the ends, take several times as long as the others and would
// otherwise be the launch's tail.
SRTM_DEV int64_t ends_first(int64_t i, int64_t nt) { return (i & 1) ? nt - 1 - (i >> 1) : i >> 1; }

// Stage bodies of the smoothing launches, for workgroup `bid` of the launch; the kernels below
// wrap them for one (nx, ny) pair, the mixed-pair kernels dispatch to them per workgroup.
template <typename T, int NX, int NY>
SRTM_DEV void kb_constants(const Batch& b, int64_t bid) {
  const Seq<T, NX, NY> q = seq_view<T, NX, NY>(b, (int)bid);
  constants_body<T, NX, NY>(q.F, q.Q, q.H, q.R, q.L, q.plan.nlev, q.cst, q.cst64, q.hand, q.lev64, q.info);
}

// Workgroups 0 .. nseq-1 continue the level chains of the sequences; the others reduce tile
// bid - nseq of the call.
template <typename T, int NX, int NY, bool INP, TreeForm FORM = tree_form<T, NX>()>
SRTM_DEV void kb_fwd_reduce(const Batch& b, int64_t bid, int nseq) {
  if (bid < nseq) {
    const Seq<T, NX, NY> q = seq_view<T, NX, NY>(b, (int)bid);
    chain_tail_body<T, NX, NY>(q.cst, q.hand, q.lev64, q.L, q.plan.nlev, q.info);
    return;
  }
  const int64_t t = bid - nseq;
  const Seq<T, NX, NY> q = seq_view<T, NX, NY>(b, tile_sequence(b, t));
  fwd_reduce_body<INP, FORM, T, NX, NY>(q.y, q.N, q.cst, q.L, q.in, q.ftagg, q.utree, t - q.tile0);
}

template <typename T, int NX, int NY, bool INP>
SRTM_DEV void kb_tile_tree(const Batch& b, int64_t bid, int nthr) {
  const Seq<T, NX, NY> q = seq_view<T, NX, NY>(b, (int)bid);
  tile_tree_body<INP, T, NX, NY>(q.y, q.N, q.plan.nlev, q.cst, q.lev64, q.L, q.in, q.ftagg, q.utree, q.ftst, q.tail, q.smoother,
                                 q.info, nthr);
}

// What the fold writes besides its records and the slow-rate filter covariances: the slow-rate filter means (where no
// smoothing recovery writes them), and the state after the last window (an output, or the only place where a failure
// there shows).
struct FoldOut {
  bool means, last;
};

template <typename T, int NX, int NY, bool SMOOTH, bool INP>
SRTM_DEV void kb_fold(const Batch& b, int64_t bid, FoldOut want) {
  Seq<T, NX, NY> q = seq_view<T, NX, NY>(b, tile_sequence(b, bid));
  if (!want.means) q.mf_slow = nullptr;
  fold_body<SMOOTH, INP, T, NX, NY>(q.y, q.N, q.L, q.plan.nlev, q.cst, q.lev64, q.in, q.m0, q.P0, q.ftagg, q.ftst, q.utree, q.tail,
                                    q.carry, q.mf_slow, q.Pf_slow, q.sfx, q.info, bid - q.tile0, want.last);
}

template <typename T, int NX, int NY>
SRTM_DEV void kb_fwd_tiles(const Batch& b, int64_t bid) {
  const Seq<T, NX, NY> q = seq_view<T, NX, NY>(b, (int)bid);
  fwd_tiles_body<T, NX, NY>(q.ftagg, q.plan.nt, q.plan.lchunk, q.plan.steps, q.plan.nlev, q.cst, q.L, q.m0, q.P0,
                            q.ftst, q.info);
}

template <typename T, int NX, int NY, bool INP>
SRTM_DEV void kb_fwd_bwd(const Batch& b, int64_t bid) {
  const Seq<T, NX, NY> q = seq_view<T, NX, NY>(b, tile_sequence(b, bid));
  fwd_bwd_body<INP, T, NX, NY>(q.y, q.N, q.L, q.cst, q.in, q.m0, q.P0, q.ftst, q.utree, q.carry, q.btagg, q.sfx, q.info, bid - q.tile0);
}

template <typename T, int NX, int NY>
SRTM_DEV void kb_bwd_tiles(const Batch& b, int64_t bid) {
  const Seq<T, NX, NY> q = seq_view<T, NX, NY>(b, (int)bid);
  bwd_tiles_body<T, NX, NY>(q.btagg, q.plan.nt, q.plan.lchunk, q.plan.steps, q.btst);
}

template <typename T, int NX, int NY>
SRTM_DEV void kb_tv_reduce(const Batch& b, int64_t bid) {
  const Seq<T, NX, NY> q = seq_view<T, NX, NY>(b, tile_sequence(b, bid));
  tv_reduce_body<T, NX, NY>(q.F, q.Q, q.H, q.R, q.y, q.N, q.L, q.tvblk, q.tvel, q.ftagg, q.info, bid - q.tile0);
}

template <typename T, int NX, int NY>
SRTM_DEV void kb_tv_tiles(const Batch& b, int64_t bid) {
  const Seq<T, NX, NY> q = seq_view<T, NX, NY>(b, (int)bid);
  tv_tiles_body<T, NX>(q.ftagg, q.plan.nt, q.plan.lchunk, q.plan.steps, q.m0, q.P0, q.ftst, q.info);
}

template <typename T, int NX, int NY, bool SMOOTH>
SRTM_DEV void kb_tv_fwd(const Batch& b, int64_t bid) {
  const Seq<T, NX, NY> q = seq_view<T, NX, NY>(b, tile_sequence(b, bid));
  tv_fwd_body<T, NX, NY, SMOOTH>(q.F, q.Q, q.H, q.y, q.N, q.L, q.tvblk, q.tvel, q.m0, q.P0, q.ftst, q.carry,
                                 q.mf_slow, q.Pf_slow, q.btagg, q.sfx, q.info, bid - q.tile0);
}

// MODE 1: filter outputs only; 2: smoother outputs; 3: both; 6: smoother outputs and slow filter means. Fast-rate outputs take all L
// steps; with only the slow smoothed state requested, step 1 suffices.
template <typename T, int NX, int NY, int MODE, bool INP, bool TV = false>
SRTM_DEV void kb_recover(const Batch& b, int64_t bid, Split sp) {
  int64_t i;
  int part, s;
  split_place(sp, bid, s, i, part);
  const bool extra = s >= 0;
  if (!extra) s = tile_sequence(b, i);
  const Seq<T, NX, NY> q = seq_view<T, NX, NY>(b, s);
  if (!extra) i -= q.tile0;
  const int nparts = i < END_TILES ? sp.ends : sp.all;
  if (i >= q.plan.nt || (!extra && part > 0 && nparts > sp.all)) return;
  const bool fast = (MODE & 1) || q.ms_fast || q.Ps_fast;
  if (!fast && !q.ms_slow && !q.Ps_slow) return;
  recover_body<T, NX, NY, MODE, INP, TV>(q.y, q.N, q.L, fast ? q.L : 1, TV ? q.tvblk : q.cst, q.in, q.F, q.Q, q.m0,
                                         q.P0, q.carry, q.sfx, q.btst, q.utree, q.mf_fast, q.Pf_fast, q.ms_fast, q.Ps_fast,
                                         q.ms_slow, q.Ps_slow, q.mf_slow, q.info, TV ? i : ends_first(i, q.plan.nt), part, sp.all, nparts);
}

template <typename T, int NX, int NY>
__global__ void __launch_bounds__(256) k_constants(Batch b) {
  kb_constants<T, NX, NY>(b, blockIdx.x);
}

template <typename T, int NX, int NY, bool INP, TreeForm FORM = tree_form<T, NX>()>
__global__ void __launch_bounds__(TILE) k_fwd_reduce(Batch b, int nseq) {
  kb_fwd_reduce<T, NX, NY, INP, FORM>(b, blockIdx.x, nseq);
}

template <typename T, int NX, int NY, bool INP>
__global__ void __launch_bounds__(TT) k_tile_tree(Batch b) {
  kb_tile_tree<T, NX, NY, INP>(b, blockIdx.x, TT);
}

// Workgroups a compute unit holds: with the rare refinement in its code the float32 fold would take 160 registers, 3 a
// unit, and 262144 windows at nx = 4 4 us more; its spills at 128 fall into that branch.
template <typename T, int NX, int NY, bool SMOOTH, bool INP>
__global__ void __launch_bounds__(TILE, NX > 4 && sizeof(T) == 8 ? 1 : NX <= 4 && sizeof(T) == 4 ? 4 : 2) k_fold(Batch b, FoldOut want) {
  kb_fold<T, NX, NY, SMOOTH, INP>(b, blockIdx.x, want);
}

template <typename T, int NX, int NY>
__global__ void __launch_bounds__(KS) k_fwd_tiles(Batch b) {
  kb_fwd_tiles<T, NX, NY>(b, blockIdx.x);
}

template <typename T, int NX, int NY, bool INP>
__global__ void __launch_bounds__(TILE) k_fwd_bwd(Batch b) {
  kb_fwd_bwd<T, NX, NY, INP>(b, blockIdx.x);
}

template <typename T, int NX, int NY>
__global__ void __launch_bounds__(KS) k_bwd_tiles(Batch b) {
  kb_bwd_tiles<T, NX, NY>(b, blockIdx.x);
}

// Per-window (time-varying) models: per-window constants and tile aggregates; the tile-level
// scan of whole elements; the fused per-tile forward (and smoother) pass.
template <typename T, int NX, int NY>
__global__ void __launch_bounds__(TILE) k_tv_reduce(Batch b) {
  kb_tv_reduce<T, NX, NY>(b, blockIdx.x);
}

template <typename T, int NX, int NY>
__global__ void __launch_bounds__(KS) k_tv_tiles(Batch b) {
  kb_tv_tiles<T, NX, NY>(b, blockIdx.x);
}

template <typename T, int NX, int NY, bool SMOOTH>
__global__ void __launch_bounds__(TILE) k_tv_fwd(Batch b) {
  kb_tv_fwd<T, NX, NY, SMOOTH>(b, blockIdx.x);
}

template <typename T, int NX, int NY, int MODE, bool INP, bool TV = false>
__global__ void __launch_bounds__(TILE, (recover_per_cu<T, NX, TV>())) k_recover(Batch b, Split sp) {
  kb_recover<T, NX, NY, MODE, INP, TV>(b, blockIdx.x, sp);
}

// The constants block without the scan levels (the sequential comparator needs no scan), and the
// sequential comparator itself: one lane per sequence.
template <typename T, int NX, int NY>
__global__ void __launch_bounds__(256) k_constants_seq(Batch b) {
  const Seq<T, NX, NY> q = seq_view<T, NX, NY>(b, blockIdx.x);
  constants_body<T, NX, NY>(q.F, q.Q, q.H, q.R, q.L, 0, q.cst, q.cst64, q.hand, nullptr, q.info);
}

template <typename T, int NX, int NY>
__global__ void __launch_bounds__(64) k_seq(Batch b, int nseq) {
  const int s = blockIdx.x * 64 + threadIdx.x;
  if (s >= nseq) return;
  const Seq<T, NX, NY> q = seq_view<T, NX, NY>(b, s);
  seq_body<T, NX, NY>(q.y, q.N, q.L, q.cst, q.m0, q.P0, q.carry, q.ms_fast, q.Ps_fast, q.ms_slow, q.Ps_slow, q.info);
}

template <typename T, int NX, int NY>
__global__ void __launch_bounds__(TILE) k_lag1(Batch b, Split sp) {
  const Seq<T, NX, NY> q = seq_view<T, NX, NY>(b, 0);  // one sequence; the parts of its end tiles first (kb_recover)
  if (!q.Cs_fast) return;
  int64_t i;
  int part, s;
  split_place(sp, blockIdx.x, s, i, part);
  const int nparts = i < END_TILES ? sp.ends : sp.all;
  if (i >= q.plan.nt || (s < 0 && part > 0 && nparts > sp.all)) return;
  lag1_body<T, NX, NY>(q.y, q.N, q.L, q.cst, q.carry, q.sfx, q.utree, q.Cs_fast, q.info, ends_first(i, q.plan.nt), part, sp.all, nparts);
}

template <typename T, int NX, int NY, bool GRAD, bool INP>
__global__ void __launch_bounds__(TILE) k_stats(Batch b) {
  const Seq<T, NX, NY> q = seq_view<T, NX, NY>(b, tile_sequence(b));
  stats_body<T, NX, NY, GRAD, INP>(q.y, q.N, q.L, q.cst, q.cst64, q.in, q.R, q.m0, q.P0, q.carry, q.sfx, q.btst, q.utree,
                                   q.stats, q.info, (int64_t)blockIdx.x - q.tile0);
}

// Outputs: the given arrays (one sequence), or else, per sequence of a batch, its four output
// slots (ms_fast, Ps_fast, ms_slow, Ps_slow) hold ll, dF, dQ and dR.
template <typename T, int NX, int NY, bool GRAD>
__global__ void __launch_bounds__(SF_THREADS) k_stats_final(Batch b, T* ll, T* dF, T* dQ, T* dR) {
  const Seq<T, NX, NY> q = seq_view<T, NX, NY>(b, blockIdx.x);
  const bool own = ll == nullptr;
  stats_final_body<T, NX, NY, GRAD>(q.plan.nt, q.Q, q.R, q.stats, own ? q.ms_fast : ll,
                                    own ? q.Ps_fast : dF, own ? q.ms_slow : dQ, own ? q.Ps_slow : dR, q.info);
}

// ============================================================================ launchers

struct Events {
  hipEvent_t const* ev;
  int n;
  int j;
  hipError_t pre(hipStream_t s) {
    if (!ev || 2 * j + 1 >= n) return hipSuccess;
    return hipEventRecord(ev[2 * j], s);
  }
  hipError_t post(hipStream_t s) {
    hipError_t e = hipSuccess;
    if (ev && 2 * j + 1 < n) e = hipEventRecord(ev[2 * j + 1], s);
    ++j;
    return e;
  }
};

#define SRTM_CHECK_LAUNCH()                    \
  do {                                         \
    hipError_t _e = hipGetLastError();         \
    if (_e != hipSuccess) return SRTM_E_HIP;   \
  } while (0)

// One launch that is a stage of its own. In a profiled call (per-stage events given) the stage's
// two events are taken by the dispatch itself (hipExtLaunchKernelGGL), so that they time the
// kernel alone rather than also the gap before it; otherwise a plain launch (calls recorded into a
// graph carry no events).
#define SRTM_STAGE(kernel, grid, block, lds, st, ...)                                               \
  do {                                                                                             \
    if (ev.ev && 2 * ev.j + 1 < ev.n) {                                                            \
      hipExtLaunchKernelGGL(kernel, grid, block, (std::uint32_t)(lds), st, ev.ev[2 * ev.j],         \
                            ev.ev[2 * ev.j + 1], 0u, __VA_ARGS__);                                 \
    } else {                                                                                       \
      hipLaunchKernelGGL(kernel, grid, block, lds, st, __VA_ARGS__);                               \
    }                                                                                              \
    ++ev.j;                                                                                        \
    SRTM_CHECK_LAUNCH();                                                                           \
  } while (0)

#define SRTM_EV(call)                          \
  do {                                         \
    if ((call) != hipSuccess) return SRTM_E_HIP; \
  } while (0)

constexpr size_t kMaxLdsBytes = 160 * 1024;  // LDS per workgroup on gfx950

// Dynamic LDS above 64 KiB must be allowed per kernel before launching.
inline bool allow_lds(const void* f, size_t bytes) {
  return bytes <= 65536 || hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes) == hipSuccess;
}

// Grid shape of one call: `nseq` sequences, `ntiles` tiles in all, the largest window length.
struct Launch {
  unsigned nseq;
  unsigned ntiles;
  int max_L;
};

// What follows the scans: the fast-rate recovery (modes 1-3, see k_recover), the
// log-likelihood alone (REC_LL, after the forward scan) or the log-likelihood and its gradient
// (REC_GRAD, after both scans); `lo` receives the latter two.
template <typename T>
struct LikOut {
  T *ll, *dF, *dQ, *dR;
};

// INP: the call has known inputs (every sequence of it).
template <typename T, int NX, int NY, bool INP>
srtm_status launch_all(const Batch& b, const Launch& g, bool smoother, int rec_mode, hipStream_t st, Events ev,
                       LikOut<T> lo = LikOut<T>{nullptr, nullptr, nullptr, nullptr}) {
  constexpr int NN = NX * NX;
  const size_t lds0 = constants_lds_bytes(NX, NY, g.max_L);
  if (!allow_lds((const void*)k_constants<T, NX, NY>, lds0)) return SRTM_E_HIP;
  SRTM_STAGE((k_constants<T, NX, NY>), dim3(g.nseq), dim3(256), lds0, st, b);

  constexpr size_t lds_red = fwd_reduce_lds_bytes<T, NX>();
  if (grad_by_elements<T>() && rec_mode == REC_GRAD) {
    SRTM_STAGE((k_fwd_reduce<T, NX, NY, INP, TREE_ROWS>), dim3(g.ntiles + g.nseq), dim3(TILE),
               lds_red, st, b, (int)g.nseq);
  } else {
    SRTM_STAGE((k_fwd_reduce<T, NX, NY, INP>), dim3(g.ntiles + g.nseq), dim3(TILE), lds_red, st, b, (int)g.nseq);
  }

  const int nlev_max = make_scan_plan((int64_t)g.ntiles * TILE).nlev;
  if constexpr (grad_by_elements<T>()) {
    if (rec_mode == REC_GRAD) {
      // slots, then the level records LOG_TILE .. nlev-1 of the longest sequence of the call
      const size_t lds_ft = sizeof(T) * ((size_t)KS * (NX + NN) +
                                         (size_t)(nlev_max - LOG_TILE) * make_const_layout(NX, NY, 1).lev_stride);
      const size_t lds_fb = sizeof(T) * (size_t)TILE * (2 * NN + NX > 4 * NX ? 2 * NN + NX : 4 * NX);
      const size_t lds_bk = sizeof(T) * (size_t)KS * (2 * NN + NX);
      if (!allow_lds((const void*)k_fwd_tiles<T, NX, NY>, lds_ft) ||
          !allow_lds((const void*)k_fwd_bwd<T, NX, NY, INP>, lds_fb) ||
          !allow_lds((const void*)k_bwd_tiles<T, NX, NY>, lds_bk))
        return SRTM_E_HIP;
      SRTM_STAGE((k_fwd_tiles<T, NX, NY>), dim3(g.nseq), dim3(KS), lds_ft, st, b);
      SRTM_STAGE((k_fwd_bwd<T, NX, NY, INP>), dim3(g.ntiles), dim3(TILE), lds_fb, st, b);
      hipLaunchKernelGGL((k_bwd_tiles<T, NX, NY>), dim3(g.nseq), dim3(KS), lds_bk, st, b);
      SRTM_CHECK_LAUNCH();
      hipLaunchKernelGGL((k_stats<T, NX, NY, true, INP>), dim3(g.ntiles), dim3(TILE), stats_lds_bytes(NX, NY, g.max_L), st, b);
      SRTM_CHECK_LAUNCH();
      hipLaunchKernelGGL((k_stats_final<T, NX, NY, true>), dim3(g.nseq), dim3(SF_THREADS), 0, st, b, lo.ll, lo.dF, lo.dQ,
                         lo.dR);
      SRTM_CHECK_LAUNCH();
      return SRTM_OK;
    }
  }
  // A call whose sequences are all of one tile has no tree above the tiles.
  if (g.ntiles > g.nseq) {
    const size_t lds_tt = tile_tree_lds_bytes<T, NX>(nlev_max);
    if (!allow_lds((const void*)k_tile_tree<T, NX, NY, INP>, lds_tt)) return SRTM_E_HIP;
    SRTM_STAGE((k_tile_tree<T, NX, NY, INP>), dim3(g.nseq), dim3(TT), lds_tt, st, b);
  } else {
    SRTM_EV(ev.pre(st));
    SRTM_EV(ev.post(st));
  }
  const size_t lds_fold = FoldLds<T, NX>(nlev_max).total;
  const Split sp = make_split<T, NX>(g.ntiles, g.nseq);
  const unsigned nrec = g.ntiles * sp.all + sp.extra;
  const FoldOut want{!(smoother && (rec_mode == 2 || rec_mode == 3)),
                     b.one.mf_slow || b.one.Pf_slow || rec_mode == REC_LL || rec_mode == REC_GRAD};

  // output staging, then the per-step tables of up to RSTEPS fast steps
  const size_t ptab = sizeof(T) * (size_t)(g.max_L < RSTEPS ? g.max_L : RSTEPS) *
                      make_const_layout(NX, NY, g.max_L).per_i_stride;
  const size_t lds_rec = (size_t)4 * OutStage<T, NX>::BYTES * ((rec_mode == 3) ? 2 : 1) + ptab;
  if (!smoother) {
    if (!allow_lds((const void*)k_fold<T, NX, NY, false, INP>, lds_fold)) return SRTM_E_HIP;
    SRTM_STAGE((k_fold<T, NX, NY, false, INP>), dim3(g.ntiles), dim3(TILE), lds_fold, st, b, want);
    if (rec_mode == 1) {
      if (!allow_lds((const void*)k_recover<T, NX, NY, 1, INP>, lds_rec)) return SRTM_E_HIP;
      SRTM_STAGE((k_recover<T, NX, NY, 1, INP>), dim3(nrec), dim3(TILE), lds_rec, st, b, sp);
    } else {
      SRTM_EV(ev.pre(st));
      if (rec_mode == REC_LL) {
        hipLaunchKernelGGL((k_stats<T, NX, NY, false, INP>), dim3(g.ntiles), dim3(TILE), 0, st, b);
        SRTM_CHECK_LAUNCH();
        hipLaunchKernelGGL((k_stats_final<T, NX, NY, false>), dim3(g.nseq), dim3(SF_THREADS), 0, st, b, lo.ll, lo.dF,
                           lo.dQ, lo.dR);
        SRTM_CHECK_LAUNCH();
      }
      SRTM_EV(ev.post(st));
    }
    return SRTM_OK;
  }

  if (!allow_lds((const void*)k_fold<T, NX, NY, true, INP>, lds_fold)) return SRTM_E_HIP;
  SRTM_STAGE((k_fold<T, NX, NY, true, INP>), dim3(g.ntiles), dim3(TILE), lds_fold, st, b, want);

  if (rec_mode == 2 && b.one.mf_slow) {
    if (!allow_lds((const void*)k_recover<T, NX, NY, 6, INP>, lds_rec)) return SRTM_E_HIP;
    SRTM_STAGE((k_recover<T, NX, NY, 6, INP>), dim3(nrec), dim3(TILE), lds_rec, st, b, sp);
  } else if (rec_mode == 2) {
    if (!allow_lds((const void*)k_recover<T, NX, NY, 2, INP>, lds_rec)) return SRTM_E_HIP;
    SRTM_STAGE((k_recover<T, NX, NY, 2, INP>), dim3(nrec), dim3(TILE), lds_rec, st, b, sp);
  } else if (rec_mode == 3 && lds_rec <= kMaxLdsBytes) {
    if (!allow_lds((const void*)k_recover<T, NX, NY, 3, INP>, lds_rec)) return SRTM_E_HIP;
    SRTM_STAGE((k_recover<T, NX, NY, 3, INP>), dim3(nrec), dim3(TILE), lds_rec, st, b, sp);
  } else {
    SRTM_EV(ev.pre(st));
    if (rec_mode == REC_GRAD) {
      hipLaunchKernelGGL((k_stats<T, NX, NY, true, INP>), dim3(g.ntiles), dim3(TILE), stats_lds_bytes(NX, NY, g.max_L), st, b);
      SRTM_CHECK_LAUNCH();
      hipLaunchKernelGGL((k_stats_final<T, NX, NY, true>), dim3(g.nseq), dim3(SF_THREADS), 0, st, b, lo.ll, lo.dF, lo.dQ,
                         lo.dR);
      SRTM_CHECK_LAUNCH();
    } else if (rec_mode == 3) {  // filter and smoother staging do not fit together: two passes
      const size_t lds1 = (size_t)4 * OutStage<T, NX>::BYTES + ptab;
      if (!allow_lds((const void*)k_recover<T, NX, NY, 1, INP>, lds1)) return SRTM_E_HIP;
      if (!allow_lds((const void*)k_recover<T, NX, NY, 6, INP>, lds1)) return SRTM_E_HIP;
      hipLaunchKernelGGL((k_recover<T, NX, NY, 1, INP>), dim3(nrec), dim3(TILE), lds1, st, b, sp);
      SRTM_CHECK_LAUNCH();
      hipLaunchKernelGGL((k_recover<T, NX, NY, 6, INP>), dim3(nrec), dim3(TILE), lds1, st, b, sp);
      SRTM_CHECK_LAUNCH();
    }
    SRTM_EV(ev.post(st));
  }
  return SRTM_OK;
}

// The sequential comparator (REC_SEQ): the constants, then one lane per sequence.
template <typename T, int NX, int NY>
srtm_status launch_seq(const Batch& b, const Launch& g, hipStream_t st) {
  const size_t lds0 = constants_lds_bytes(NX, NY, g.max_L);
  if (!allow_lds((const void*)k_constants_seq<T, NX, NY>, lds0)) return SRTM_E_HIP;
  hipLaunchKernelGGL((k_constants_seq<T, NX, NY>), dim3(g.nseq), dim3(256), lds0, st, b);
  SRTM_CHECK_LAUNCH();
  hipLaunchKernelGGL((k_seq<T, NX, NY>), dim3((g.nseq + 63) / 64), dim3(64), 0, st, b, (int)g.nseq);
  SRTM_CHECK_LAUNCH();
  return SRTM_OK;
}

// Per-window (time-varying) model, one sequence: 5 launches for the smoother (k_tv_reduce,
// k_tv_tiles, k_tv_fwd<1>, k_bwd_tiles, k_recover), 4 for the filter.
template <typename T, int NX, int NY>
srtm_status launch_tv(const Batch& b, const Launch& g, bool smoother, int rec_mode, hipStream_t st) {
  if constexpr (NX > TV_NX_MAX) {
    return SRTM_E_UNSUPPORTED;
  } else {
    constexpr int NN = NX * NX, FA = 3 * NN + 2 * NX;
    const size_t lds_el = sizeof(T) * (size_t)TILE * FA;  // a tile of whole elements
    if (!allow_lds((const void*)k_tv_reduce<T, NX, NY>, lds_el)) return SRTM_E_HIP;
    hipLaunchKernelGGL((k_tv_reduce<T, NX, NY>), dim3(g.ntiles), dim3(TILE), lds_el, st, b);
    SRTM_CHECK_LAUNCH();
    const size_t lds_ks = sizeof(T) * (size_t)KS * FA;
    if (!allow_lds((const void*)k_tv_tiles<T, NX, NY>, lds_ks)) return SRTM_E_HIP;
    hipLaunchKernelGGL((k_tv_tiles<T, NX, NY>), dim3(g.nseq), dim3(KS), lds_ks, st, b);
    SRTM_CHECK_LAUNCH();
    const size_t lds_rec = (size_t)4 * OutStage<T, NX>::BYTES + tv_model_lds_bytes<T, NX, NY>();
    if (!smoother) {
      if (!allow_lds((const void*)k_tv_fwd<T, NX, NY, false>, lds_el)) return SRTM_E_HIP;
      hipLaunchKernelGGL((k_tv_fwd<T, NX, NY, false>), dim3(g.ntiles), dim3(TILE), lds_el, st, b);
      SRTM_CHECK_LAUNCH();
      if (rec_mode == 1) {
        if (!allow_lds((const void*)k_recover<T, NX, NY, 1, false, true>, lds_rec)) return SRTM_E_HIP;
        hipLaunchKernelGGL((k_recover<T, NX, NY, 1, false, true>), dim3(g.ntiles), dim3(TILE), lds_rec, st, b, Split{0, 1, 1, 1});
        SRTM_CHECK_LAUNCH();
      }
      return SRTM_OK;
    }
    if (!allow_lds((const void*)k_tv_fwd<T, NX, NY, true>, lds_el)) return SRTM_E_HIP;
    hipLaunchKernelGGL((k_tv_fwd<T, NX, NY, true>), dim3(g.ntiles), dim3(TILE), lds_el, st, b);
    SRTM_CHECK_LAUNCH();
    const size_t lds_bk = sizeof(T) * (size_t)KS * (2 * NN + NX);
    if (!allow_lds((const void*)k_bwd_tiles<T, NX, NY>, lds_bk)) return SRTM_E_HIP;
    hipLaunchKernelGGL((k_bwd_tiles<T, NX, NY>), dim3(g.nseq), dim3(KS), lds_bk, st, b);
    SRTM_CHECK_LAUNCH();
    if (rec_mode == 2 || rec_mode == 3) {  // filter and smoother outputs: two recovery passes
      if (rec_mode == 3) {
        if (!allow_lds((const void*)k_recover<T, NX, NY, 1, false, true>, lds_rec)) return SRTM_E_HIP;
        hipLaunchKernelGGL((k_recover<T, NX, NY, 1, false, true>), dim3(g.ntiles), dim3(TILE), lds_rec, st, b, Split{0, 1, 1, 1});
        SRTM_CHECK_LAUNCH();
      }
      if (!allow_lds((const void*)k_recover<T, NX, NY, 2, false, true>, lds_rec)) return SRTM_E_HIP;
      hipLaunchKernelGGL((k_recover<T, NX, NY, 2, false, true>), dim3(g.ntiles), dim3(TILE), lds_rec, st, b, Split{0, 1, 1, 1});
      SRTM_CHECK_LAUNCH();
    }
    return SRTM_OK;
  }
}

// One sequence (srtm_filter / srtm_smooth).
template <typename T, int NX, int NY>
srtm_status run(const srtm_shape& sh, const Ptrs& p, bool smoother, hipStream_t st, Events ev, int lik_mode = 0,
                void* ll = nullptr, void* dF = nullptr, void* dQ = nullptr, void* dR = nullptr) {
  Batch b{};
  b.table = nullptr;
  b.tile_seq = nullptr;
  b.ws = static_cast<char*>(p.ws);
  b.info = p.info;
  SeqDesc& d = b.one;
  d.F = p.F; d.Q = p.Q; d.H = p.H; d.R = p.R; d.m0 = p.m0; d.P0 = p.P0; d.y = p.y;
  d.ms_fast = p.ms_fast; d.Ps_fast = p.Ps_fast; d.ms_slow = p.ms_slow; d.Ps_slow = p.Ps_slow;
  d.mf_fast = p.mf_fast; d.Pf_fast = p.Pf_fast; d.mf_slow = p.mf_slow; d.Pf_slow = p.Pf_slow;
  d.N = sh.N;
  d.tile0 = 0;
  d.ws_off = 0;
  d.L = sh.L;
  d.smoother = smoother ? 1 : 0;
  d.B = p.B;
  d.u = p.u;
  d.nu = p.B ? p.nu : 0;
  d.tv = p.tv ? 1 : 0;
  d.Cs_fast = p.Cs_fast;
  d.nx = NX;
  d.ny = NY;
  const Launch g{1u, (unsigned)((sh.N + TILE - 1) / TILE), (int)sh.L};
  const bool want_f = p.mf_fast || p.Pf_fast;
  const bool want_s = p.ms_fast || p.Ps_fast || p.ms_slow || p.Ps_slow;
  const int mode = lik_mode ? lik_mode : (smoother ? (want_f ? 3 : (want_s ? 2 : 0)) : (want_f ? 1 : 0));
  const LikOut<T> lo{static_cast<T*>(ll), static_cast<T*>(dF), static_cast<T*>(dQ), static_cast<T*>(dR)};
  if (lik_mode == REC_SEQ) {
    if (p.tv || p.B || p.Cs_fast || ev.ev || !smoother) return SRTM_E_UNSUPPORTED;
    return launch_seq<T, NX, NY>(b, g, st);
  }
  if (p.tv) {
    if (lik_mode || ev.ev) return SRTM_E_UNSUPPORTED;  // no log-likelihood or profiling form
    return launch_tv<T, NX, NY>(b, g, smoother, mode, st);
  }
  if (p.B) return launch_all<T, NX, NY, true>(b, g, smoother, mode, st, ev, lo);
  if (!p.Cs_fast) return launch_all<T, NX, NY, false>(b, g, smoother, mode, st, ev, lo);
  // lag-one cross-covariances: the smoother's launches, then one more pass over the tiles
  if (!smoother || lik_mode || ev.ev) return SRTM_E_UNSUPPORTED;
  const srtm_status s = launch_all<T, NX, NY, false>(b, g, smoother, mode, st, ev, lo);
  if (s != SRTM_OK) return s;
  const size_t lds = (size_t)4 * OutStage<T, NX>::BYTES;
  if (!allow_lds((const void*)k_lag1<T, NX, NY>, lds)) return SRTM_E_HIP;
  const Split sp = make_split<T, NX>(g.ntiles, 1);
  hipLaunchKernelGGL((k_lag1<T, NX, NY>), dim3(g.ntiles * sp.all + sp.extra), dim3(TILE), lds, st, b, sp);
  SRTM_CHECK_LAUNCH();
  return SRTM_OK;
}

// Many sequences (srtm_smooth_batch): `table` holds nseq descriptors followed by the sequence
// index of every tile, in device memory.
template <typename T, int NX, int NY>
srtm_status run_batch(const void* table, int nseq, int64_t ntiles, int max_L, void* ws, int32_t* info,
                      hipStream_t st, bool grad) {
  Batch b{};
  b.table = static_cast<const SeqDesc*>(table);
  b.tile_seq = reinterpret_cast<const int32_t*>(static_cast<const char*>(table) + batch_tile_map_offset(nseq));
  b.ws = static_cast<char*>(ws);
  b.info = info;
  const Launch g{(unsigned)nseq, (unsigned)ntiles, max_L};
  return launch_all<T, NX, NY, false>(b, g, true, grad ? REC_GRAD : 2, st, Events{nullptr, 0, 0});
}

}  // namespace srtm

#if defined(SRTM_MIXED_T)
// ---------------------------------------------------------------- mixed-pair launches
// One set of five launches (six with per-window models) for a batch whose sequences differ in (nx, ny) and kind (time-invariant
// model, with known inputs, or per-window model): every workgroup reads its sequence's descriptor
// and runs that pair's and kind's stage body. Each sequence gets exactly the per-pair kernels'
// arithmetic on the same tiles. This object is compiled once per element type (SRTM_MIXED_T).
namespace srtm {

template <typename T>
__global__ void __launch_bounds__(256) km_constants(Batch b) {
  const SeqDesc& d = b.table[blockIdx.x];
  if (d.tv) return;  // per-window models build their constants per tile in the next stage
#define SRTM_MX(a, c)                          \
  if (d.nx == a && d.ny == c) {                \
    kb_constants<T, a, c>(b, blockIdx.x);      \
    return;                                    \
  }
  SRTM_PAIRS(SRTM_MX)
#undef SRTM_MX
}

// Workgroups 0 .. nseq-1: level chains (time-invariant models); the rest: tile reductions.
template <typename T>
__global__ void __launch_bounds__(TILE) km_reduce(Batch b, int nseq) {
  const int64_t bid = blockIdx.x;
  const SeqDesc& d = b.table[bid < nseq ? (int)bid : tile_sequence(b, bid - nseq)];
#define SRTM_MX(a, c)                                                    \
  if (d.nx == a && d.ny == c) {                                          \
    if (d.tv) {                                                          \
      if constexpr (a <= TV_NX_MAX) {                                    \
        if (bid >= nseq) kb_tv_reduce<T, a, c>(b, bid - nseq);           \
      }                                                                  \
    } else if (d.B) {                                                    \
      kb_fwd_reduce<T, a, c, true>(b, bid, nseq);                        \
    } else {                                                             \
      kb_fwd_reduce<T, a, c, false>(b, bid, nseq);                       \
    }                                                                    \
    return;                                                              \
  }
  SRTM_PAIRS(SRTM_MX)
#undef SRTM_MX
}

template <typename T>
__global__ void __launch_bounds__(KS) km_tiles(Batch b) {
  const SeqDesc& d = b.table[blockIdx.x];
#define SRTM_MX(a, c)                                      \
  if (d.nx == a && d.ny == c) {                            \
    if (d.tv) {                                            \
      if constexpr (a <= TV_NX_MAX) kb_tv_tiles<T, a, c>(b, blockIdx.x); \
    } else if (d.B) {                                      \
      kb_tile_tree<T, a, c, true>(b, blockIdx.x, KS);      \
    } else {                                               \
      kb_tile_tree<T, a, c, false>(b, blockIdx.x, KS);     \
    }                                                      \
    return;                                                \
  }
  SRTM_PAIRS(SRTM_MX)
#undef SRTM_MX
}

template <typename T>
__global__ void __launch_bounds__(TILE) km_fold(Batch b) {
  const SeqDesc& d = b.table[tile_sequence(b)];
#define SRTM_MX(a, c)                                                    \
  if (d.nx == a && d.ny == c) {                                          \
    if (d.tv) {                                                          \
      if constexpr (a <= TV_NX_MAX) kb_tv_fwd<T, a, c, true>(b, blockIdx.x); \
    } else if (d.B) {                                                    \
      kb_fold<T, a, c, true, true>(b, blockIdx.x, FoldOut{false, false}); \
    } else {                                                             \
      kb_fold<T, a, c, true, false>(b, blockIdx.x, FoldOut{false, false}); \
    }                                                                    \
    return;                                                              \
  }
  SRTM_PAIRS(SRTM_MX)
#undef SRTM_MX
}

// Per-window models only: the tile-level reverse scan.
template <typename T>
__global__ void __launch_bounds__(KS) km_bwd_tiles(Batch b) {
  const SeqDesc& d = b.table[blockIdx.x];
  if (!d.tv) return;
#define SRTM_MX(a, c)                          \
  if (d.nx == a && d.ny == c) {                \
    if constexpr (a <= TV_NX_MAX) kb_bwd_tiles<T, a, c>(b, blockIdx.x); \
    return;                                    \
  }
  SRTM_PAIRS(SRTM_MX)
#undef SRTM_MX
}

template <typename T>
__global__ void __launch_bounds__(TILE) km_recover(Batch b, Split sp) {
  const SeqDesc& d = b.table[tile_sequence(b, blockIdx.x / (unsigned)sp.all)];
#define SRTM_MX(a, c)                                                           \
  if (d.nx == a && d.ny == c) {                                                 \
    if (d.tv) {                                                                 \
      if constexpr (a <= TV_NX_MAX)                                             \
        if (blockIdx.x % (unsigned)sp.all == 0)                                 \
          kb_recover<T, a, c, 2, false, true>(b, blockIdx.x / (unsigned)sp.all, Split{0, 1, 1, 1}); \
    } else if (d.B) {                                                           \
      kb_recover<T, a, c, 2, true>(b, blockIdx.x, sp);                          \
    } else {                                                                    \
      kb_recover<T, a, c, 2, false>(b, blockIdx.x, sp);                         \
    }                                                                           \
    return;                                                                     \
  }
  SRTM_PAIRS(SRTM_MX)
#undef SRTM_MX
}

// Dynamic LDS of the six stages for one sequence of pair (NX, NY): the launch takes the largest
// over the batch's sequences.
template <typename T, int NX, int NY>
void stage_lds(bool tv, int max_L, int nlev_max, size_t (&o)[6]) {
  constexpr int NN = NX * NX;
  auto up = [&](int j, size_t v) { o[j] = v > o[j] ? v : o[j]; };
  if (!tv) {
    up(0, constants_lds_bytes(NX, NY, max_L));
    up(1, fwd_reduce_lds_bytes<T, NX>());
    up(2, tile_tree_lds_bytes<T, NX>(nlev_max));
    up(3, FoldLds<T, NX>(nlev_max).total);
    up(5, (size_t)4 * OutStage<T, NX>::BYTES +
              sizeof(T) * (size_t)(max_L < RSTEPS ? max_L : RSTEPS) * make_const_layout(NX, NY, max_L).per_i_stride);
  } else {
    if constexpr (NX <= TV_NX_MAX) {
      constexpr int FA = 3 * NN + 2 * NX;
      up(1, sizeof(T) * (size_t)TILE * FA);
      up(2, sizeof(T) * (size_t)KS * FA);
      up(3, sizeof(T) * (size_t)TILE * FA);
      up(4, sizeof(T) * (size_t)KS * (2 * NN + NX));
      up(5, (size_t)4 * OutStage<T, NX>::BYTES + tv_model_lds_bytes<T, NX, NY>());
    }
  }
}

template <typename T>
srtm_status run_mixed(const SeqDesc* host, const void* table_dev, int nseq, int64_t ntiles, int max_L, void* ws,
                      int32_t* info, hipStream_t st) {
  Batch b{};
  b.table = static_cast<const SeqDesc*>(table_dev);
  b.tile_seq = reinterpret_cast<const int32_t*>(static_cast<const char*>(table_dev) + batch_tile_map_offset(nseq));
  b.ws = static_cast<char*>(ws);
  b.info = info;
  const int nlev_max = make_scan_plan(ntiles * TILE).nlev;
  size_t lds[6] = {0, 0, 0, 0, 0, 0};
  for (int s = 0; s < nseq; ++s) {
#define SRTM_MX(a, c) \
  if (host[s].nx == a && host[s].ny == c) stage_lds<T, a, c>(host[s].tv != 0, max_L, nlev_max, lds);
    SRTM_PAIRS(SRTM_MX)
#undef SRTM_MX
  }
  const void* fn[6] = {(const void*)km_constants<T>, (const void*)km_reduce<T>, (const void*)km_tiles<T>,
                       (const void*)km_fold<T>,      (const void*)km_bwd_tiles<T>, (const void*)km_recover<T>};
  for (int j = 0; j < 6; ++j)
    if (!allow_lds(fn[j], lds[j])) return SRTM_E_HIP;
  const unsigned ns = (unsigned)nseq, nt = (unsigned)ntiles;
  hipLaunchKernelGGL((km_constants<T>), dim3(ns), dim3(256), lds[0], st, b);
  SRTM_CHECK_LAUNCH();
  hipLaunchKernelGGL((km_reduce<T>), dim3(nt + ns), dim3(TILE), lds[1], st, b, nseq);
  SRTM_CHECK_LAUNCH();
  hipLaunchKernelGGL((km_tiles<T>), dim3(ns), dim3(KS), lds[2], st, b);
  SRTM_CHECK_LAUNCH();
  hipLaunchKernelGGL((km_fold<T>), dim3(nt), dim3(TILE), lds[3], st, b);
  SRTM_CHECK_LAUNCH();
  if (lds[4]) {  // per-window models among them
    hipLaunchKernelGGL((km_bwd_tiles<T>), dim3(ns), dim3(KS), lds[4], st, b);
    SRTM_CHECK_LAUNCH();
  }
  // The tiles of different pairs differ so much in time (nx = 6: 90 us, nx = 2: 10 us) that parts of all of them
  // fill the device better (178 tiles of 15 sequences: 94 us whole, 58 us in 4 parts, 62 us with those of nx <= 4
  // whole); with several tiles per compute unit they do that by themselves.
  const int parts = nt > 4 * CUS ? 1 : nt > 2 * CUS ? 2 : 4;
  const Split sp{0, parts, parts, 1};
  hipLaunchKernelGGL((km_recover<T>), dim3(nt * parts), dim3(TILE), lds[5], st, b, sp);
  SRTM_CHECK_LAUNCH();
  return SRTM_OK;
}

#define SRTM_MIXED_NAME2(t) run_mixed_##t
#define SRTM_MIXED_NAME(t) SRTM_MIXED_NAME2(t)
srtm_status SRTM_MIXED_NAME(SRTM_MIXED_T)(const SeqDesc* host, const void* table_dev, int nseq, int64_t ntiles,
                                          int max_L, void* ws, int32_t* info, hipStream_t st) {
  return run_mixed<SRTM_MIXED_T>(host, table_dev, nseq, ntiles, max_L, ws, info, st);
}

}  // namespace srtm
#else
// ---------------------------------------------------------------- this object's (nx, ny) pair
#if !defined(SRTM_NX) || !defined(SRTM_NY)
#error "srtm_kernels.hip is compiled once per (nx, ny) pair (SRTM_NX, SRTM_NY) or per element type (SRTM_MIXED_T)"
#endif
#define SRTM_NAME2(p, a, b) p##a##_##b
#define SRTM_NAME(p, a, b) SRTM_NAME2(p, a, b)

namespace srtm {
srtm_status SRTM_NAME(run_pair_, SRTM_NX, SRTM_NY)(int dtype, const srtm_shape& sh, const Ptrs& p, bool smoother,
                                                   hipStream_t st, hipEvent_t const* ev, int nev, int lik_mode,
                                                   void* ll, void* dF, void* dQ, void* dR) {
  const Events E{ev, nev, 0};
  if (dtype == SRTM_F64) return run<double, SRTM_NX, SRTM_NY>(sh, p, smoother, st, E, lik_mode, ll, dF, dQ, dR);
  return run<float, SRTM_NX, SRTM_NY>(sh, p, smoother, st, E, lik_mode, ll, dF, dQ, dR);
}

srtm_status SRTM_NAME(run_batch_pair_, SRTM_NX, SRTM_NY)(int dtype, const void* table, int nseq, int64_t ntiles,
                                                         int max_L, void* ws, int32_t* info, hipStream_t st,
                                                         bool grad) {
  if (dtype == SRTM_F64) return run_batch<double, SRTM_NX, SRTM_NY>(table, nseq, ntiles, max_L, ws, info, st, grad);
  return run_batch<float, SRTM_NX, SRTM_NY>(table, nseq, ntiles, max_L, ws, info, st, grad);
}
}  // namespace srtm
#endif  // SRTM_MIXED_T
