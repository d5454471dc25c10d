// The blocks of the TSQR tree (tsqr.hip) by 16-column panels: the factorization of a level's 256-row
// blocks and the formation of its part of Q.
//
// Panels P = 0 .. ceil(p/16)-1 (H_0 .. H_{p-1} = Q_0 Q_1 .., Q_P = I - V_P T_P V_P^T) are worked on in
// registers in the layout of v_mfma_f64_16x16x4's accumulators: lane l = 16 g + c holds column c of a
// panel and rows 16 I + 4 v + g (tile I = 0 .. 15, item v = 0 .. 3). That one layout serves
//   * the panel's reflector steps, where a column's values reach the other 15 columns of the lane
//     row by the DPP broadcast of v_fmac_f64;
//   * the matrix cores, as B operand of V^T A (4 rows per step = one register) and as
//     accumulator of A - V Z: the block never moves between layouts.
// LAPACK's Householder convention as in tsqr.hip, so R has the same row signs.
#include "lrp_kernels.h"

namespace lrp {

// cls[P]: the tile classes (bit k: tiles I with I mod 4 = k) in which the columns up to panel P can
// be nonzero. A block of stacked triangular factors has zeros below each factor's diagonal, which
// the reflectors keep, so at p_max = 64 panel P touches only P + 1 of the 4 classes.
struct PanelFactorArgs {
  const DevState* st;
  int ncols[2];
  const void* in[2];
  int in_f32;
  int64_t ldin;
  int64_t rows;
  int block_rows;
  int pmax;
  double* V[2];     // reflectors, block b at b block_rows pmax (layout: see store_reflectors)
  double* Rout[2];
  int64_t ldr;
  uint8_t cls[4];
};

struct PanelApplyArgs {
  const DevState* st;
  int ncols[2];
  const double* V[2];
  int64_t rows;
  int block_rows;
  int pmax;
  const double* T[2];  // parent pieces (rows b*pmax .. b*pmax+p of a matrix with ld ldt); null = identity
  int64_t ldt;
  double* Y[2];
  int64_t ldy;
  ApplySel sel;
  uint8_t cls[4];
};

constexpr int kWyThreads = 256;           // 4 waves, 16 columns each
constexpr int kPanel = 16;                // columns per panel
constexpr int kVLd = kPanel + 1;          // LDS row stride of a panel (odd: the transposed reads spread over the banks)

__device__ __forceinline__ wy4 mfma4(double a, double b, wy4 c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

// x of lane J of each 16-lane row, on all lanes of the row.
template <int J>
__device__ __forceinline__ double row_bcast(double x) {
  return __longlong_as_double(__builtin_amdgcn_mov_dpp(__double_as_longlong(x), 0x150 + J, 0xF, 0xF, false));
}

// sum_g' sel(g') x(16 g' + c) on every lane 16 g + c, sel the value of sel on lane row g' (the same
// on the row's lanes): the four lane rows are the inner dimension of the four 4 x 4 products of
// v_mfma_f64_4x4x4 (A lane l = row l % 4 of block l / 4 % 4, inner index l / 16; B lane l =
// column l % 16, inner index l / 16; result lane l = row l / 16, column l % 16). It takes 29
// cycles where two rounds of lane swaps and adds take 67.
__device__ __forceinline__ double rows_dot(double sel, double x) {
  return __builtin_amdgcn_mfma_f64_4x4x4f64(sel, x, 0.0, 0, 0, 0);
}

// d += bcast_J(a) b with bcast_J the value of lane J of the lane row, as one v_fmac_f64 with a DPP
// source (a broadcast move and an fma would take twice the issue slots). The instructions are
// written out because the compiler does not fold a 64-bit broadcast into the fma; each block
// starts with the two wait states that a DPP source needs after a VALU write, which the compiler's
// hazard handling does not add inside or before an asm block.
#define LRP_FMAC(D, A, B, N) "v_fmac_f64_dpp " D ", " A ", " B " row_newbcast:" N " row_mask:0xf bank_mask:0xf\n\t"
template <int J>
__device__ __forceinline__ void fmac1(double& d, double a, double b) {
  asm volatile("s_nop 1\n\t" LRP_FMAC("%0", "%1", "%2", "%c3") : "+v"(d) : "v"(a), "v"(b), "n"(J));
}
// d0, d1 += bcast_J(y) x over the 4 registers of a tile.
template <int J>
__device__ __forceinline__ void dot_tile(double& d0, double& d1, double y0, double y1, double y2, double y3,
                                         const double* x) {
  asm volatile("s_nop 1\n\t" LRP_FMAC("%0", "%2", "%6", "%c10") LRP_FMAC("%1", "%3", "%7", "%c10")
                   LRP_FMAC("%0", "%4", "%8", "%c10") LRP_FMAC("%1", "%5", "%9", "%c10")
               : "+v"(d0), "+v"(d1)
               : "v"(y0), "v"(y1), "v"(y2), "v"(y3), "v"(x[0]), "v"(x[1]), "v"(x[2]), "v"(x[3]), "n"(J));
}
template <int J>
__device__ __forceinline__ void dot_tile(double& d0, double& d1, const double* x) {
  dot_tile<J>(d0, d1, x[0], x[1], x[2], x[3], x);
}
// x += bcast_J(x) m over the 4 registers of a tile.
template <int J>
__device__ __forceinline__ void update_tile(double* x, double m) {
  asm volatile("s_nop 1\n\t" LRP_FMAC("%0", "%0", "%4", "%c5") LRP_FMAC("%1", "%1", "%4", "%c5")
                   LRP_FMAC("%2", "%2", "%4", "%c5") LRP_FMAC("%3", "%3", "%4", "%c5")
               : "+v"(x[0]), "+v"(x[1]), "+v"(x[2]), "+v"(x[3])
               : "v"(m), "n"(J));
}
// d0 + d1 += sum_{k < J} bcast_k(s) T[k].
template <int J>
__device__ __forceinline__ void t_column(double& d0, double& d1, double s, const double (&T)[16]) {
#define LRP_TCOL(STR)                                                                                        \
  asm volatile("s_nop 1\n\t" STR                                                                             \
               : "+v"(d0), "+v"(d1)                                                                          \
               : "v"(s), "v"(T[0]), "v"(T[1]), "v"(T[2]), "v"(T[3]), "v"(T[4]), "v"(T[5]), "v"(T[6]), "v"(T[7]), \
                 "v"(T[8]), "v"(T[9]), "v"(T[10]), "v"(T[11]), "v"(T[12]), "v"(T[13]), "v"(T[14]))
#define LRP_TC0 LRP_FMAC("%0", "%2", "%3", "0")
#define LRP_TC1 LRP_TC0 LRP_FMAC("%1", "%2", "%4", "1")
#define LRP_TC2 LRP_TC1 LRP_FMAC("%0", "%2", "%5", "2")
#define LRP_TC3 LRP_TC2 LRP_FMAC("%1", "%2", "%6", "3")
#define LRP_TC4 LRP_TC3 LRP_FMAC("%0", "%2", "%7", "4")
#define LRP_TC5 LRP_TC4 LRP_FMAC("%1", "%2", "%8", "5")
#define LRP_TC6 LRP_TC5 LRP_FMAC("%0", "%2", "%9", "6")
#define LRP_TC7 LRP_TC6 LRP_FMAC("%1", "%2", "%10", "7")
#define LRP_TC8 LRP_TC7 LRP_FMAC("%0", "%2", "%11", "8")
#define LRP_TC9 LRP_TC8 LRP_FMAC("%1", "%2", "%12", "9")
#define LRP_TC10 LRP_TC9 LRP_FMAC("%0", "%2", "%13", "10")
#define LRP_TC11 LRP_TC10 LRP_FMAC("%1", "%2", "%14", "11")
#define LRP_TC12 LRP_TC11 LRP_FMAC("%0", "%2", "%15", "12")
#define LRP_TC13 LRP_TC12 LRP_FMAC("%1", "%2", "%16", "13")
#define LRP_TC14 LRP_TC13 LRP_FMAC("%0", "%2", "%17", "14")
  if constexpr (J == 1) LRP_TCOL(LRP_TC0);
  else if constexpr (J == 2) LRP_TCOL(LRP_TC1);
  else if constexpr (J == 3) LRP_TCOL(LRP_TC2);
  else if constexpr (J == 4) LRP_TCOL(LRP_TC3);
  else if constexpr (J == 5) LRP_TCOL(LRP_TC4);
  else if constexpr (J == 6) LRP_TCOL(LRP_TC5);
  else if constexpr (J == 7) LRP_TCOL(LRP_TC6);
  else if constexpr (J == 8) LRP_TCOL(LRP_TC7);
  else if constexpr (J == 9) LRP_TCOL(LRP_TC8);
  else if constexpr (J == 10) LRP_TCOL(LRP_TC9);
  else if constexpr (J == 11) LRP_TCOL(LRP_TC10);
  else if constexpr (J == 12) LRP_TCOL(LRP_TC11);
  else if constexpr (J == 13) LRP_TCOL(LRP_TC12);
  else if constexpr (J == 14) LRP_TCOL(LRP_TC13);
  else if constexpr (J == 15) LRP_TCOL(LRP_TC14);
#undef LRP_TC0
#undef LRP_TC1
#undef LRP_TC2
#undef LRP_TC3
#undef LRP_TC4
#undef LRP_TC5
#undef LRP_TC6
#undef LRP_TC7
#undef LRP_TC8
#undef LRP_TC9
#undef LRP_TC10
#undef LRP_TC11
#undef LRP_TC12
#undef LRP_TC13
#undef LRP_TC14
#undef LRP_TCOL
}
// Per-column results of a panel, on every lane of the column (lanes c, 16 + c, ..) of every wave.
struct PanelCols {
  double u[16];  // after step J: u[J] = -tau_J v_J . x_c (see panel_step)
  double beta;   // R(c, c)
  double tau;    // 0 for H = I
  double r[4];   // R's diagonal tile (wave 0), above the diagonal
};

// LDS of the factorization. The waves' partial sums of a step are double-buffered, so that a step
// needs one barrier.
struct FactorShared {
  double V[4][64 * kVLd];            // per wave: its 64 rows of a panel, row-major (row stride kVLd)
  double W[4][3][4 * 64];            // per wave: its part of V^T A for the panels to the right
  double part[2][4][64];             // per wave and lane: dot products of a step
  double pivot[2][4][64];            // the pivot row's item (wave 0's counts)
  double T[kPanel * kVLd];           // T_P(i, j) at i kVLd + j
};

// Step J of a panel: the reflector of its column J and the update of the columns after it. Each
// wave holds 64 rows of the panel, x[4 s + v] (slots s = 0 .. 3 of 16 rows); the diagonal tile is
// slot 0 of wave 0, and the rows of the tile above the pivot are zero right of the diagonal (they
// have moved to pc.r). SLOTS is 1 where the other slots are zero, else 4: a build without branches
// per slot, since a taken branch costs a step as much (60 cycles) as the two sweeps over a slot.
//
// One reduction per step: with x_J the unscaled column, d_c = sum over the rows below the pivot
// of x_J x_c gives |x_tail|^2 on lane J and, once alpha - beta is known, u_c = v_J . x_c = d_c /
// (alpha - beta) + x_c(pivot): right of J the dot product of the update, left of J (whose
// registers hold finished reflectors) v_J . v_c, from which T follows. Every wave adds the four
// waves' parts in the same order and goes on by itself with the same bits. The update takes the
// scaled v_J (one extra product per register, 4 % of the time): of exactly proportional columns that are
// one large entry (the fibers of sine modes) a block then keeps nothing of that entry in a third to all
// of the columns and up to 1 eps in the others (the column kernels of tsqr.hip in none); the unscaled one
// always leaves some, unless the ratio is a power of two.
//
// With h = sqrt(alpha^2 + |x_tail|^2) and s = sign(alpha): beta = -s h, tau = (beta - alpha) /
// beta = 1 + |alpha| / h and 1 / (alpha - beta) = s / (|alpha| + h), so one reciprocal square root
// and one reciprocal give all of them.
template <int J, int SLOTS>
__device__ __forceinline__ void panel_step(double* x, int c, int g, int lane, bool top, FactorShared& sh,
                                           int w, PanelCols& pc) {
  constexpr int PV = J >> 2, PG = J & 3;  // the pivot row: item PV of lane row PG of wave 0
  asm volatile("" : "+v"(c), "+v"(g));    // lane masks are formed per step, not kept for all 16
  const int gp = top ? PG : -1;
  sh.pivot[J & 1][w][lane] = x[PV];
  double y = g == gp ? 0.0 : x[PV];
  double d0 = 0.0, d1 = 0.0;
  dot_tile<J>(d0, d1, PV == 0 ? y : x[0], PV == 1 ? y : x[1], PV == 2 ? y : x[2], PV == 3 ? y : x[3], x);
#pragma unroll
  for (int s = 1; s < SLOTS; ++s) dot_tile<J>(d0, d1, x + 4 * s);
  sh.part[J & 1][w][lane] = d0 + d1;
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
  const double p0 = sh.part[J & 1][0][lane], p1 = sh.part[J & 1][1][lane];
  const double p2 = sh.part[J & 1][2][lane], p3 = sh.part[J & 1][3][lane];
  const double pv = sh.pivot[J & 1][0][lane];
  const double d = rows_dot(1.0, (p0 + p2) + (p1 + p3));
  const double a = rows_dot(g == PG ? 1.0 : 0.0, pv);  // the pivot row's entry of every column, never -0
  const double alpha = row_bcast<J>(a), xn2 = row_bcast<J>(d);
  const double h2 = fma(alpha, alpha, xn2);
  double rh = rsq_nr(h2);
  // exponents outside 2^-960 .. 2^960 (uniform): the Newton steps would leave the number range
  if (__builtin_expect(__ballot((unsigned)(__double2hiint(h2) - ((1023 - 960) << 20)) > (unsigned)(1920 << 20)) != 0, 0)) {
    const bool big = h2 > 1.0;
    rh = rsq_nr(h2 * (big ? 0x1p-200 : 0x1p200)) * (big ? 0x1p-100 : 0x1p100);
    if (h2 == 0.0) rh = 0.0;
  }
  const double aa = fabs(alpha), h = h2 * rh;
  const bool none = xn2 == 0.0;  // nothing below the diagonal: H = I
  const double scale = none ? 0.0 : copysign(rcp_nr(aa + h), alpha);
  const double tau = none ? 0.0 : fma(aa, rh, 1.0);
  const double u = -tau * fma(scale, d, a);
  const double m = c > J ? u : 0.0;
  const double f = c == J ? scale : 1.0;
#pragma unroll
  for (int v = 0; v < 4; ++v) x[v] *= f;
#pragma unroll
  for (int e = 4; e < 4 * SLOTS; ++e) x[e] *= f;
  x[PV] = g == gp && c == J ? 1.0 : x[PV];
#pragma unroll
  for (int s = 0; s < SLOTS; ++s) update_tile<J>(x + 4 * s, m);
  const bool rrow = g == gp && c > J;  // row J of R
  pc.r[PV] = rrow ? x[PV] : pc.r[PV];
  x[PV] = rrow ? 0.0 : x[PV];
  pc.u[J] = u;
  pc.beta = c != J ? pc.beta : none ? alpha : -copysign(h, alpha);
  pc.tau = c == J ? tau : pc.tau;
}

template <int J, int SLOTS>
__device__ __forceinline__ void panel_steps(double* x, int cw, int c, int g, int lane, bool top, FactorShared& sh, int w,
                                            PanelCols& pc) {
  if constexpr (J < kPanel) {
    if (J < cw) panel_step<J, SLOTS>(x, c, g, lane, top, sh, w, pc);  // uniform
    panel_steps<J + 1, SLOTS>(x, cw, c, g, lane, top, sh, w, pc);
  }
}

// Row c of T_P in place of u: T(c, J) = sum_{k < J} T(c, k) u_k(J) for c < J (zero by itself for
// c > J), and T(J, J) = tau_J.
template <int J>
__device__ __forceinline__ void t_rows(PanelCols& pc, int c) {
  if constexpr (J < kPanel) {
    double t0 = c == J ? pc.tau : 0.0, t1 = 0.0;
    if constexpr (J > 0) t_column<J>(t0, t1, pc.u[J], pc.u);
    pc.u[J] = J > 1 ? t0 + t1 : t0;
    t_rows<J + 1>(pc, c);
  }
}

// Loads the wave's 64 rows of all columns (zeros outside the block and, unread, in the classes not
// in use). A lane reads one row, so that a load covers 64 consecutive rows of a column, and the
// values change to the tile layout through the wave's LDS st: a load in the tile layout touches 16
// cache lines (15000 cycles for a block of 64 columns where these take 7000, 20 bytes per cycle:
// what one CU's outstanding misses allow). FULL: the block has all 256 rows.
template <typename T, bool FULL>
__device__ __forceinline__ void load_block(const PanelFactorArgs& a, const T* X, int p, int nr, int w, int lane, double* st,
                                           double (&x)[4][16]) {
  const int c = lane & 15, g = lane >> 4;
  const int r = 64 * w + lane;
  T raw[4][kPanel];
#pragma unroll
  for (int q = 0; q < 4; ++q)
    if (kPanel * q < p) {  // uniform
#pragma unroll
      for (int k = 0; k < kPanel; ++k) raw[q][k] = T(0);
      const T* Xq = X + (int64_t)(kPanel * q) * a.ldin;
      if ((a.cls[q] >> g & 1) && (FULL || r < nr)) {
#pragma unroll
        for (int k = 0; k < kPanel; ++k) {
          raw[q][k] = Xq[(unsigned)r];
          Xq += kPanel * q + k < p - 1 ? a.ldin : 0;  // past the last column: that column again
        }
      }
    }
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    if (kPanel * q < p) {
#pragma unroll
      for (int k = 0; k < kPanel; ++k)
        st[lane * kVLd + k] = kPanel * (q + 1) <= p || kPanel * q + k < p ? (double)raw[q][k] : 0.0;
#pragma unroll
      for (int e = 0; e < 16; ++e) x[q][e] = st[(4 * e + g) * kVLd + c];
    } else {
#pragma unroll
      for (int e = 0; e < 16; ++e) x[q][e] = 0.0;
    }
  }
}

// V_P row-major: rows r < nr of the classes in use, cw columns, so that a wave's store is
// contiguous. In the diagonal tile (wave 0's slot 0, written by the caller) the entries on and above
// the diagonal (V's ones and zeros) carry T_P.
__device__ __forceinline__ void store_reflectors(const double* x, int sc, int P, int w, int c, int g, int lane, int cw,
                                                 int nr, bool top, double* V) {
  const bool full = cw == kPanel && nr == kTsqrRows;  // uniform, as the next ones
#pragma unroll
  for (int s = 0; s < 4; ++s)
    if ((sc >> s & 1) && !(top && s == 0)) {
      const int tile = 4 * w + ((s + P) & 3);
      if (full) {  // (16 tile + 4 v + g) 16 + c
        double* Vt = V + 256 * tile + lane;
#pragma unroll
        for (int v = 0; v < 4; ++v) Vt[64 * v] = x[4 * s + v];
      } else {
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int row = 16 * tile + 4 * v + g;
          if (c < cw && row < nr) V[row * cw + c] = x[4 * s + v];
        }
      }
    }
}

// One workgroup per 256-row block, wave w on rows 64w .. 64w+63 of all columns: x[q] holds panel
// P + q, slot s of it tile (s + P) mod 4 of the wave, so that one copy of the unrolled panel code
// serves every panel. After the steps of a panel each wave forms its part of W = V^T A for the
// panels to the right straight from registers, the parts are added through LDS, and each wave
// applies A - V (T^T W) to its rows; all four matrix cores work throughout.
__device__ __forceinline__ void factor_block(const PanelFactorArgs& a) {
  const int side = blockIdx.y;
  if (a.st && a.st->done) return;
  const int p = __builtin_amdgcn_readfirstlane(side_cols(a.st, a.ncols, side));
  const int64_t row0 = (int64_t)blockIdx.x * a.block_rows;
  const int nr = (int)min((int64_t)a.block_rows, a.rows - row0);
  if (p <= 0 || nr <= 0) return;
  const int t = threadIdx.x, lane = t & 63;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  __shared__ FactorShared sh;
  const int pt = (p + kPanel - 1) / kPanel;

  double x[4][16];
  if (a.in_f32) {
    const float* X = (const float*)a.in[side] + row0;
    if (nr == kTsqrRows)
      load_block<float, true>(a, X, p, nr, wave, lane, sh.V[wave], x);
    else
      load_block<float, false>(a, X, p, nr, wave, lane, sh.V[wave], x);
  } else {
    const double* X = (const double*)a.in[side] + row0;
    if (nr == kTsqrRows)
      load_block<double, true>(a, X, p, nr, wave, lane, sh.V[wave], x);
    else
      load_block<double, false>(a, X, p, nr, wave, lane, sh.V[wave], x);
  }
  for (int P = 0; P < pt; ++P) {
    // opaque copies: addresses are formed where they are used, not kept in registers over the loop
    int w = wave, c = lane & 15, g = lane >> 4;
    asm volatile("" : "+s"(w), "+v"(c), "+v"(g));
    const bool top = w == 0;  // uniform
    const int cw = min(kPanel, p - kPanel * P);
    const int cls = __builtin_amdgcn_readfirstlane(a.cls[P]);
    const int sc = ((cls >> P) | (cls << (4 - P))) & 15;  // slot classes
    double* Rc = a.Rout[side] + (int64_t)blockIdx.x * a.pmax + (int64_t)(kPanel * P + c) * a.ldr;
    PanelCols pc;
#pragma unroll
    for (int k = 0; k < kPanel; ++k) pc.u[k] = 0.0;  // columns past p stay zero
#pragma unroll
    for (int v = 0; v < 4; ++v) pc.r[v] = 0.0;
    pc.beta = 0.0;
    pc.tau = 0.0;
    // The matrix-core results in x are read by asm blocks from here on, which the compiler's wait
    // states do not cover.
#pragma unroll
    for (int s = 0; s < 4; ++s)
      asm volatile("" : "+v"(x[0][4 * s]), "+v"(x[0][4 * s + 1]), "+v"(x[0][4 * s + 2]), "+v"(x[0][4 * s + 3]));
    asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");
    // rows above the diagonal tile are final: R's, and zeros from here on
#pragma unroll
    for (int s = 1; s < 4; ++s)
      if (top && s + P >= 4) {  // uniform
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          if (c < cw) Rc[16 * (s + P - 4) + 4 * v + g] = x[0][4 * s + v];
          x[0][4 * s + v] = 0.0;
        }
      }
    if (sc == 1)
      panel_steps<0, 1>(x[0], cw, c, g, lane, top, sh, w, pc);
    else
      panel_steps<0, 4>(x[0], cw, c, g, lane, top, sh, w, pc);
    if (top) {  // R's diagonal
#pragma unroll
      for (int v = 0; v < 4; ++v) pc.r[v] = 4 * v + g == c ? pc.beta : pc.r[v];
    }
    const int right = pt - 1 - P;  // panels to the right
    double* vs = sh.V[w];
    wy4 W[3];
    if (right > 0) {
#pragma unroll
      for (int s = 0; s < 4; ++s)
        if (sc >> s & 1) {  // uniform
#pragma unroll
          for (int v = 0; v < 4; ++v) vs[(16 * s + 4 * v + g) * kVLd + c] = x[0][4 * s + v];
        }
#pragma unroll
      for (int q = 0; q < 3; ++q) {
        if (q < right) {  // uniform
          W[q] = wy4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
          for (int s = 0; s < 4; ++s)
            if (sc >> s & 1) {
#pragma unroll
              for (int v = 0; v < 4; ++v) W[q] = mfma4(x[0][4 * s + v], x[q + 1][4 * s + v], W[q]);
            }
#pragma unroll
          for (int v = 0; v < 4; ++v) sh.W[w][q][64 * v + lane] = W[q][v];
        }
      }
    }
    // While wave 3 forms T_P, the others write their reflectors out; it does so after the update.
    double* Vp = a.V[side] + row0 * a.pmax + (int64_t)kPanel * P * nr;
    if (w == 3) {
      t_rows<0>(pc, c);
      if (g == 0) {
#pragma unroll
        for (int k = 0; k < 16; ++k) sh.T[c * kVLd + k] = pc.u[k];
      }
    } else {
      store_reflectors(x[0], sc, P, w, c, g, lane, cw, nr, top, Vp);
    }
    __syncthreads();
    if (right > 0) {
      double vt[4][4];  // V(row c of slot s, 4 u + g)
#pragma unroll
      for (int s = 0; s < 4; ++s)
        if (sc >> s & 1) {
#pragma unroll
          for (int u = 0; u < 4; ++u) vt[s][u] = vs[(16 * s + c) * kVLd + 4 * u + g];
        }
#pragma unroll
      for (int q = 0; q < 3; ++q)
        if (q < right) {
#pragma unroll
          for (int v = 0; v < 4; ++v)
            W[q][v] = (sh.W[0][q][64 * v + lane] + sh.W[1][q][64 * v + lane]) +
                      (sh.W[2][q][64 * v + lane] + sh.W[3][q][64 * v + lane]);
          wy4 Z = {0.0, 0.0, 0.0, 0.0};  // -T^T W
#pragma unroll
          for (int u = 0; u < 4; ++u) Z = mfma4(-sh.T[(4 * u + g) * kVLd + c], W[q][u], Z);
#pragma unroll
          for (int s = 0; s < 4; ++s)
            if (sc >> s & 1) {
              double* xq = x[q + 1] + 4 * s;
              wy4 X4 = {xq[0], xq[1], xq[2], xq[3]};
#pragma unroll
              for (int u = 0; u < 4; ++u) X4 = mfma4(vt[s][u], Z[u], X4);
#pragma unroll
              for (int v = 0; v < 4; ++v) xq[v] = X4[v];
            }
        }
    }
    if (w == 3) store_reflectors(x[0], sc, P, w, c, g, lane, cw, nr, top, Vp);
    if (top && c < cw) {  // the diagonal tile and R's zeros below it
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int m = 4 * v + g, row = kPanel * P + m;
        if (row < a.pmax) Rc[row] = pc.r[v];
        if (row < nr) Vp[row * cw + c] = m <= c ? sh.T[m * kVLd + c] : x[0][v];
      }
      for (int r = kPanel * (P + 1) + g; r < a.pmax; r += 4) Rc[r] = 0.0;
    }
    // panel P + 1 takes the place of P, its diagonal tile slot 0's
    if (right > 0) {
#pragma unroll
      for (int q = 0; q < 3; ++q)
#pragma unroll
        for (int e = 0; e < 16; ++e) x[q][e] = x[q + 1][(e + 4) & 15];
    }
  }
}

// Bound by the issue of the steps' instructions: about 100 per step and wave, one per 6 to 7 cycles
// where a SIMD has a single wave, plus one LDS exchange and barrier (730 cycles with one slot in
// use, 970 with four). Two workgroups share a CU (70 KB of LDS, 256 registers) and fill each other's
// waits. Against the column kernel of tsqr.hip (a wave per 4 columns, two dependent reductions and
// a barrier per reflector): a level of few blocks 28 -> 20 us at p = 32, 40 -> 29 us at p = 45, 56 ->
// 41 us at p = 64; the leaves of n = 2^20 - 1 at p = 64 (4096 blocks) 943 -> 585 us.
template <class Src>
__global__ __launch_bounds__(kWyThreads) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_tsqr_panel_factor(Src in) {
  factor_block(kernel_args<PanelFactorArgs>(in));
}

// Q formation: Y = Q_0 Q_1 .. Q_{pt-1} [T_par; 0], the panels applied from the last to the first,
// Y <- Y - V_P (T_P (V_P^T Y)), on the FP64 matrix cores. Wave w holds columns 16w .. 16w+15 of Y
// in registers throughout and needs nothing of the other waves'; the panels are staged through two
// LDS buffers (the next one's loads in flight behind the products), one barrier per panel.
//
// Bound by the matrix cores where the chip is full (132 products of 16 x 16 x 4 per leaf panel and wave:
// 64 for V^T Y, 4 for T W, 64 for the update; 84 for the first panel applied, and fewer where tile
// classes are not in use; 72 cycles each) and by the chain of the panels where it is not. No triangular
// solve and no V^T V: the panels' T factors come from the factorization. Against the compact WY form of
// tsqr.hip: a level of few blocks 18 -> 13 us at p = 32, 26 -> 14 us at p = 45, 38 -> 20 us at p = 64; the
// leaves of n = 2^20 - 1 at p = 64 569 -> 405 us. Dealing rows instead of columns to the waves (the sums of
// V^T Y then cross the waves, two barriers per panel) was slower: 593 us.
//
// NT: the tiles that can hold rows of a block, 16 or, where a level is one short block, 4 or 8 (see
// tsqr_panel_apply).
template <class Src, int NT>
__global__ __launch_bounds__(kWyThreads) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_tsqr_panel_apply(Src in) {
  const PanelApplyArgs& a = kernel_args<PanelApplyArgs>(in);
  const int side = blockIdx.y;
  if (a.st && a.st->done) return;
  const int p = __builtin_amdgcn_readfirstlane(side_cols(a.st, a.ncols, side));
  const int block = apply_block(a.st, a.sel, side, a.block_rows);
  const int oc = apply_cols(a.st, a.sel, p);  // columns of T_par and of Y
  if (block < 0 || oc <= 0) return;
  const int64_t row0 = (int64_t)block * a.block_rows;
  const int nr = (int)min((int64_t)a.block_rows, a.rows - row0);
  if (p <= 0 || nr <= 0) return;
  const int t = threadIdx.x, lane = t & 63, c = lane & 15, g = lane >> 4;
  const int w = __builtin_amdgcn_readfirstlane(t >> 6);
  __shared__ double Vs[2][kTsqrRows * kVLd];
  __shared__ double Ts[2][kPanel * kVLd];
  const int pt = (p + kPanel - 1) / kPanel;
  const int col = kPanel * w + c;
  const double* Vb = a.V[side] + row0 * a.pmax;
  const int sr = t >> 4, scol = t & 15;  // staging: row sr of every tile, column scol

  // panel P of the reflectors as stored: item I is row 16 I + sr (tile I)
  double raw[NT];
  auto fetch = [&](int P) {
    const int cw = min(kPanel, p - kPanel * P);
    const double* V = Vb + (int64_t)kPanel * P * nr + min(scol, cw - 1);
    const int cls = __builtin_amdgcn_readfirstlane(a.cls[P]);
#pragma unroll
    for (int k = 0; k < 4; ++k)
      if (cls >> k & 1) {  // uniform
#pragma unroll
        for (int I = k; I < NT; I += 4) raw[I] = V[min(16 * I + sr, nr - 1) * cw];
      }
  };
  fetch(pt - 1);
  wy4 y[NT];
#pragma unroll
  for (int I = 0; I < NT; ++I) y[I] = wy4{0.0, 0.0, 0.0, 0.0};
  {
    const double* T = a.T[side];
    double tp[16];
#pragma unroll
    for (int e = 0; e < 16; ++e) tp[e] = 4 * e + g == col ? 1.0 : 0.0;
    if (T) {
      const double* Tc = T + (int64_t)block * a.pmax + (int64_t)min(col, oc - 1) * a.ldt;
#pragma unroll
      for (int e = 0; e < 16; ++e) tp[e] = Tc[min(4 * e + g, p - 1)];
    }
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      keep_loaded(tp[e]);
      y[e >> 2][e & 3] = (4 * e + g < p && col < oc) ? tp[e] : 0.0;
    }
  }
  for (int P = pt - 1; P >= 0; --P) {
    const int cw = min(kPanel, p - kPanel * P), cls = __builtin_amdgcn_readfirstlane(a.cls[P]);
    double* vs = Vs[P & 1] + sr * kVLd + scol;
    double* ts = Ts[P & 1];
#pragma unroll
    for (int k = 0; k < 4; ++k)
      if (cls >> k & 1) {
        // tile k: zeros above the diagonal tile; T_P on and above the diagonal
        keep_loaded(raw[k]);
        const double v0 = 16 * k + sr < nr && scol < cw ? raw[k] : 0.0;
        vs[16 * k * kVLd] = k < P ? 0.0 : k > P || sr > scol ? v0 : sr == scol ? 1.0 : 0.0;
        if (k == P) ts[sr * kVLd + scol] = sr <= scol ? v0 : 0.0;
#pragma unroll
        for (int I = k + 4; I < NT; I += 4) {
          keep_loaded(raw[I]);
          vs[16 * I * kVLd] = 16 * I + sr < nr && scol < cw ? raw[I] : 0.0;
        }
      }
    vs = Vs[P & 1];
    if (P > 0) fetch(P - 1);
    __syncthreads();
    if (kPanel * w < oc) {  // uniform
      // V_P^T Y; before the first panel Y is zero past the first 64 rows
      wy4 W = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int k = 0; k < 4; ++k)
        if (cls >> k & 1) {
#pragma unroll
          for (int I = k; I < NT; I += 4) {
            if (I >= 4 && P == pt - 1) break;  // uniform
#pragma unroll
            for (int v = 0; v < 4; ++v) W = mfma4(vs[(16 * I + 4 * v + g) * kVLd + c], y[I][v], W);
          }
        }
      wy4 Z = {0.0, 0.0, 0.0, 0.0};  // -T W
#pragma unroll
      for (int s = 0; s < 4; ++s) Z = mfma4(-ts[c * kVLd + 4 * s + g], W[s], Z);
#pragma unroll
      for (int k = 0; k < 4; ++k)
        if (cls >> k & 1) {
#pragma unroll
          for (int I = k; I < NT; I += 4)
#pragma unroll
            for (int s = 0; s < 4; ++s) y[I] = mfma4(vs[(16 * I + c) * kVLd + 4 * s + g], Z[s], y[I]);
        }
    }
  }
  // Out through LDS, so that a store covers 64 consecutive rows of a column (in the tile layout it
  // would touch 16 cache lines). The buffer is free: its panel was consumed before the last barrier.
  if (kPanel * w < oc) {
    double* st = Vs[1] + w * (kTsqrRows / 4) * kVLd;
    double* Yr = a.Y[side] + row0 + (int64_t)(kPanel * w) * a.ldy + lane;
    const int cols = min(kPanel, oc - kPanel * w);
#pragma unroll
    for (int b = 0; b < NT / 4; ++b) {
#pragma unroll
      for (int e = 0; e < 16; ++e) st[(4 * e + g) * kVLd + c] = y[4 * b + (e >> 2)][e & 3];
      double o[kPanel];
#pragma unroll
      for (int k = 0; k < kPanel; ++k) o[k] = st[lane * kVLd + k];
      if (64 * b + lane < nr) {
#pragma unroll
        for (int k = 0; k < kPanel; ++k)
          if (k < cols) Yr[64 * b + (int64_t)k * a.ldy] = o[k];  // uniform
      }
    }
  }
}

// Tile classes in use per panel (PanelFactorArgs::cls) at level L: all at the leaves; above, a tile of
// the stacked factors counts for panel P where one of its rows is row <= 16 P + 15 of its factor.
static void tile_classes(const TsqrPlan& p, int L, uint8_t (&cls)[4]) {
  for (int P = 0; P < 4; ++P) {
    cls[P] = L == 0 ? 15 : 0;
    for (int I = 0; L > 0 && 16 * I < p.lev[L].block_rows; ++I) {
      const int r = (16 * I) % p.pmax;  // the tile's first row within its factor
      if (r < kPanel * (P + 1) || r + 15 >= p.pmax) cls[P] |= (uint8_t)(1 << (I & 3));
    }
    cls[P] |= (uint8_t)(1 << P);  // the diagonal tile
  }
}

int tsqr_panel_factor(const TsqrPlan& p, int L, const TsqrIO& io, hipStream_t s) {
  const TsqrLevel& lv = p.lev[L];
  PanelFactorArgs f{};
  f.st = io.st;
  f.in_f32 = L == 0 ? io.x_f32 : 0;
  f.ldin = L == 0 ? io.ldx : (int64_t)p.lev[L - 1].nblocks * p.pmax;
  f.rows = lv.rows;
  f.block_rows = lv.block_rows;
  f.pmax = p.pmax;
  f.ldr = (int64_t)lv.nblocks * p.pmax;
  tile_classes(p, L, f.cls);
  for (int q = 0; q < 2; ++q) {
    f.ncols[q] = io.ncols[q];
    f.in[q] = L == 0 ? io.X[q] : p.lev[L - 1].Rout[q];
    f.V[q] = lv.V[q];
    f.Rout[q] = lv.Rout[q];
  }
  LRP_LAUNCH_G(K_TSQR_FACTOR, k_tsqr_panel_factor<PanelFactorArgs>, k_tsqr_panel_factor<GroupRef>,
               dim3(lv.nblocks, io.nsides), dim3(kWyThreads), 0, s, f);
  return launch_status();
}

int tsqr_panel_apply(const TsqrPlan& p, int L, const TsqrIO& io, const ApplyOut& o, hipStream_t s) {
  const TsqrLevel& lv = p.lev[L];
  PanelApplyArgs a{};
  a.st = io.st;
  a.rows = lv.rows;
  a.block_rows = lv.block_rows;
  a.pmax = p.pmax;
  a.ldt = o.ldt;
  a.ldy = o.ldy;
  a.sel = o.sel;
  tile_classes(p, L, a.cls);
  for (int q = 0; q < 2; ++q) {
    a.ncols[q] = io.ncols[q];
    a.V[q] = lv.V[q];
    a.T[q] = o.T[q];
    a.Y[q] = o.Y[q];
  }
  // A level of one block of at most 64 (128) rows, a small matrix or a tree's root, is a chain on its own
  // and need not multiply the tiles past its rows: 64 x 33 59 -> 49 us, 257 x 17 (its root of 34 rows) 61 ->
  // 56. The choice inside the kernel made it three times as long, and levels of more blocks, short last
  // one or not, 1 to 3 us slower each.
#define LRP_APPLY(NT)                                                                                           \
  LRP_LAUNCH_G(K_TSQR_APPLY, (k_tsqr_panel_apply<PanelApplyArgs, NT>), (k_tsqr_panel_apply<GroupRef, NT>),        \
               dim3(o.sel.pick ? p.pmax : lv.nblocks, io.nsides), dim3(kWyThreads), 0, s, a)
  if (lv.nblocks > 1 || lv.rows > 128)
    LRP_APPLY(16);
  else if (lv.rows > 64)
    LRP_APPLY(8);
  else
    LRP_APPLY(4);
#undef LRP_APPLY
  return launch_status();
}

}  // namespace lrp
