// Device code of the blocked Householder QR, shared by the chained single QR
// (qr.hip) and the batched step launches (batch.hip): register-block panel
// factorisation with the LAPACK dlarfg sign convention, block loads and
// stores, and the compact-WY block-reflector apply.
#pragma once

#include "common.h"

namespace sap {
namespace qr_dev {


constexpr int kPanelThreads = 512;
constexpr int kPanelWaves = kPanelThreads / kWave;

// Householder vector entry (implicit unit diagonal, zeros above) of panel
// column k at panel-relative row r; `y` is the stored value.
__device__ __forceinline__ double vval(int r, int k, double y) {
  return r > k ? y : (r == k ? 1.0 : 0.0);
}

// Sum over the 64 lanes of NV values per lane (NV a power of two, at most 64)
// by recursive halving: while more than one value is left a step exchanges
// half of them with the lane at distance 32, 16, 8, ... (v_permlane32_swap,
// v_permlane16_swap, then DPP moves within a row of 16), so NV totals cost
// NV - 1 + log2(64 / NV) additions instead of 6 NV.  On return v[0] of lane l
// is the total of value lane_value<NV>(l); the order of additions is fixed.
__device__ __forceinline__ void swap32(double a, double b, double &x, double &y) {
  const auto lo = __builtin_amdgcn_permlane32_swap(__double2loint(a), __double2loint(b), false, false);
  const auto hi = __builtin_amdgcn_permlane32_swap(__double2hiint(a), __double2hiint(b), false, false);
  x = __hiloint2double(hi[0], lo[0]);
  y = __hiloint2double(hi[1], lo[1]);
}
__device__ __forceinline__ void swap16(double a, double b, double &x, double &y) {
  const auto lo = __builtin_amdgcn_permlane16_swap(__double2loint(a), __double2loint(b), false, false);
  const auto hi = __builtin_amdgcn_permlane16_swap(__double2hiint(a), __double2hiint(b), false, false);
  x = __hiloint2double(hi[0], lo[0]);
  y = __hiloint2double(hi[1], lo[1]);
}
// One step within a row of 16 lanes: lanes with bit `BIT` clear keep a and
// take the partner's a, the others keep b; CTRL moves the partner's value.
template <int BIT, int CTRL>
__device__ __forceinline__ double halve_dpp(double a, double b) {
  const bool up = (threadIdx.x & BIT) != 0;
  return (up ? b : a) + dpp_mov<CTRL>(up ? a : b);
}
template <int NV, int C, int LEVEL>
__device__ __forceinline__ void reduce_level(double (&v)[NV]) {
  constexpr int H = C > 1 ? C / 2 : 1;
#pragma unroll
  for (int i = 0; i < H; ++i) {
    const double a = v[i], b = C > 1 ? v[i + H] : v[i];
    if constexpr (LEVEL == 32) {
      double x, y;
      swap32(a, b, x, y);
      v[i] = x + y;
    } else if constexpr (LEVEL == 16) {
      double x, y;
      swap16(a, b, x, y);
      v[i] = x + y;
    } else if constexpr (LEVEL == 8) {
      v[i] = C > 1 ? halve_dpp<8, 0x128>(a, b) : a + dpp_mov<0x128>(a);  // row_ror:8
    } else if constexpr (LEVEL == 4) {
      v[i] = C > 1 ? halve_dpp<4, 0x141>(a, b) : a + dpp_mov<0x141>(a);  // row_half_mirror
    } else if constexpr (LEVEL == 2) {
      v[i] = C > 1 ? halve_dpp<2, 0x4E>(a, b) : a + dpp_mov<0x4E>(a);  // quad_perm [2,3,0,1]
    } else {
      v[i] = C > 1 ? halve_dpp<1, 0xB1>(a, b) : a + dpp_mov<0xB1>(a);  // quad_perm [1,0,3,2]
    }
  }
  if constexpr (LEVEL > 1) reduce_level<NV, H, LEVEL / 2>(v);
}
template <int NV>
__device__ __forceinline__ void wave_reduce(double (&v)[NV]) {
  static_assert((NV & (NV - 1)) == 0 && NV >= 1 && NV <= 64, "a power of two");
  reduce_level<NV, NV, 32>(v);
}
// The value whose total wave_reduce leaves in lane l: the top log2(NV) bits of l.
template <int NV>
__device__ __forceinline__ int lane_value(int l) { return l / (kWave / NV); }

constexpr int pow2_at_least(int n) { return n <= 1 ? 1 : 2 * pow2_at_least((n + 1) / 2); }

// Shared state of the panel factorisation and the block-reflector apply (LDS).
// TH: threads of the workgroup (512 or 1024); thread t holds rows t + TH s.
template <int NB, int TH = kPanelThreads>
struct PanelShared {
  static constexpr int kGram = NB * (NB + 1) / 2;
  double red[TH / kWave][NB * NB];       // per-wave partials of W = V^T C
  double gred[TH / kWave][kGram];        // per-wave partials of the panel's Gram matrix
  double gtot[2][kGram];                 // their sum, and what it was rounded by
  double crow[2 * NB][NB];               // rows -NB..NB-1 of the panel before the last update
  double vrow[2 * NB][NB];               // those rows of the last update's reflectors
  double top[NB][NB];                    // rows 0..NB-1 of the panel, factored
  double U[NB][NB];                      // the rows below become (row) U
  double T[NB * NB];                     // the panel's T (column-major)
  double tauv[NB];
  int slow;                              // the Gram form was refused
  // column-by-column form
  double cred[2][TH / kWave][NB];        // per-wave partials of one panel column, by column parity
  double ctot[2][2 * NB];                // its totals (0..NB-1) and row J of the panel (NB..2NB-1)
  double G[NB][NB];                      // G[J][q] = v_q^T v_J (q < J), for T
};

// Thread t of a block holds rows t + TH s (s < S) of its columns; rows past the
// matrix's end are zero.  The NB rows from row0 (a multiple of NB, which
// divides 64) sit in one slot of one wave: calls f(slot, lr) in the threads
// that hold row0 + lr.
template <int S, int NB, int TH, typename F>
__device__ __forceinline__ void for_rows(int row0, F &&f) {
  static_assert(kWave % NB == 0, "the rows of a panel must not straddle two waves");
  const int t = threadIdx.x;
  const int s0 = row0 / TH, t0 = row0 % TH;
  if (__builtin_amdgcn_readfirstlane(t / kWave) != t0 / kWave) return;
#pragma unroll
  for (int s = 0; s < S; ++s)
    if (s == s0) {  // uniform
      const int lr = t - t0;
      if (lr >= 0 && lr < NB) f(s, lr);
    }
}

// A column of `rows` doubles as a buffer: loads past its end (and at kNoRow)
// return 0, stores there are dropped, so rows outside a range cost an offset
// select instead of a branch or a select per value.  AUX: cache policy of the
// access (kCoherent: through the coherence point shared by the XCDs, as the
// agent-scope atomics of trsv.h).
constexpr int kNoRow = static_cast<int>(0x80000000u);
constexpr int kCoherent = 16;  // sc1
__device__ __forceinline__ __amdgpu_buffer_rsrc_t column_buffer(const double *p, int rows) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<double *>(p), 0, rows * 8, 0x00020000);
}
template <int AUX>
__device__ __forceinline__ double load_row(__amdgpu_buffer_rsrc_t col, int off) {
  const auto v = __builtin_amdgcn_raw_buffer_load_b64(col, off, 0, AUX);
  return __hiloint2double(static_cast<int>(v[1]), static_cast<int>(v[0]));
}
template <int AUX>
__device__ __forceinline__ void store_row(__amdgpu_buffer_rsrc_t col, int off, double x) {
  typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
  const u32x2 v = {static_cast<unsigned>(__double2loint(x)), static_cast<unsigned>(__double2hiint(x))};
  __builtin_amdgcn_raw_buffer_store_b64(v, col, off, 0, AUX);
}

// Columns base + i ldy (i < NB; those past the nb there are repeat the last),
// rows [lo, rows); zero outside.  base is uniform.
template <int S, int NB, int TH, int AUX>
__device__ __forceinline__ void load_columns(const double *base, int64_t ldy, int rows, int nb, int lo,
                                             double (&X)[S][NB]) {
  __amdgpu_buffer_rsrc_t col[NB];
#pragma unroll
  for (int i = 0; i < NB; ++i) col[i] = column_buffer(base + static_cast<int64_t>(min(i, nb - 1)) * ldy, rows);
#pragma unroll
  for (int s = 0; s < S; ++s) {
    const int r = static_cast<int>(threadIdx.x) + TH * s;
    const int off = r >= lo ? r * 8 : kNoRow;
#pragma unroll
    for (int i = 0; i < NB; ++i) X[s][i] = load_row<AUX>(col[i], off);
  }
}
// Rows [lo, rows) of X to columns base + i ldy, i < nb.
template <int S, int NB, int TH, int AUX>
__device__ __forceinline__ void store_columns(double *base, int64_t ldy, int rows, int nb, int lo,
                                              const double (&X)[S][NB]) {
#pragma unroll
  for (int i = 0; i < NB; ++i) {
    if (i >= nb) continue;  // uniform
    const __amdgpu_buffer_rsrc_t col = column_buffer(base + static_cast<int64_t>(i) * ldy, rows);
#pragma unroll
    for (int s = 0; s < S; ++s) {
      const int r = static_cast<int>(threadIdx.x) + TH * s;
      store_row<AUX>(col, r >= lo ? r * 8 : kNoRow, X[s][i]);
    }
  }
}

// The reflectors of a panel from its stored columns, loaded from row0 on: unit
// diagonal and zeros above it in the panel's first NB rows.
template <int S, int NB, int TH>
__device__ __forceinline__ void unit_lower(double (&V)[S][NB], int row0) {
  for_rows<S, NB, TH>(row0, [&](int s, int lr) {
#pragma unroll
    for (int i = 0; i < NB; ++i) V[s][i] = vval(lr, i, V[s][i]);
  });
}

// Panel-relative rows: lr = t + TH s - roff (s < S); rows with lr < 0 lie above
// the panel (they belong to R) and only ride along.

// Column J of the panel: reflector, update of columns J+1.. of the panel,
// and what column J of T needs (tau_J, V_{<J}^T v_J, kept in LDS).  One batched
// workgroup reduction per column: with a = column J below the diagonal,
// alpha its diagonal entry and v = [1; a / (alpha - beta)], every quantity
// the column needs follows from a^T a and a^T (column x) for all x and from
// row J of the panel: v^T (column x) = P[J][x] + (a^T column x) / (alpha - beta).
// J is a template parameter so that every register index of the panel P is
// static (no scratch).
template <int S, int NB, int J, int TH>
__device__ __forceinline__ void panel_column(double (&P)[S][NB], PanelShared<NB, TH> &sh, int nb, int dr, int roff) {
  constexpr int B = J & 1;  // LDS buffers alternate between columns: one barrier fewer
  const int t = threadIdx.x;
  const int lane = t & (kWave - 1), wave = t / kWave;
  // Straight-line code: masks instead of per-row branches (the column is
  // latency-bound, and every branch costs exec-mask bookkeeping).
  double acc[NB];
#pragma unroll
  for (int x = 0; x < NB; ++x) acc[x] = 0.0;
#pragma unroll
  for (int s = 0; s < S; ++s) {
    const int lr = t + TH * s - roff;
    const double a = (lr > J && lr < dr) ? P[s][J] : 0.0;
#pragma unroll
    for (int x = 0; x < NB; ++x) acc[x] += a * P[s][x];
  }
  // row J of the panel is held by one thread: in its register row 0 where
  // J + roff < TH, else found by selects with static indices only
  if (J + roff < TH) {  // uniform
    if (J < dr && t == J + roff) {
#pragma unroll
      for (int x = 0; x < NB; ++x) sh.ctot[B][NB + x] = P[0][x];
    }
  } else {
    double rowv[NB];
    bool has_j = false;
#pragma unroll
    for (int x = 0; x < NB; ++x) rowv[x] = 0.0;
#pragma unroll
    for (int s = 0; s < S; ++s) {
      const int lr = t + TH * s - roff;
      const bool hit = lr == J && lr < dr;
      has_j = has_j || hit;
#pragma unroll
      for (int x = 0; x < NB; ++x) rowv[x] = hit ? P[s][x] : rowv[x];
    }
    if (has_j) {
#pragma unroll
      for (int x = 0; x < NB; ++x) sh.ctot[B][NB + x] = rowv[x];
    }
  }
#pragma unroll
  for (int x = 0; x < NB; ++x) acc[x] = wave_sum_u(acc[x]);
  if (lane == 0) {
#pragma unroll
    for (int x = 0; x < NB; ++x) sh.cred[B][wave][x] = acc[x];
  }
  __syncthreads();
  if (t < NB) {
    double s_ = 0.0;
    for (int w = 0; w < (TH / kWave); ++w) s_ += sh.cred[B][w][t];
    sh.ctot[B][t] = s_;
  }
  __syncthreads();
  const bool has_row = J < dr;  // uniform; a panel shorter than J+1 rows has no row J
  double tot[NB], row[NB];
#pragma unroll
  for (int x = 0; x < NB; ++x) {
    tot[x] = sh.ctot[B][x];
    row[x] = has_row ? sh.ctot[B][NB + x] : 0.0;
  }
  const double alpha = row[J];
  const double sq = tot[J];
  double tj, beta, scale;
  if (sq == 0.0) {
    tj = 0.0;
    beta = alpha;
    scale = 0.0;
  } else {
    const double nrm = sqrt(alpha * alpha + sq);
    beta = alpha >= 0.0 ? -nrm : nrm;
    tj = (beta - alpha) / beta;
    scale = 1.0 / (alpha - beta);
  }
  // dots[x] = v^T (column x): x > J weights the update of column x, x < J
  // gives V_{<J}^T v for the T factor
  double dots[NB], wgt[NB];
#pragma unroll
  for (int x = 0; x < NB; ++x) {
    dots[x] = x == J ? 0.0 : row[x] + scale * tot[x];
    wgt[x] = (x > J && x < nb) ? tj * dots[x] : 0.0;
  }
  // column J becomes v below the diagonal and beta on it; H_J = I - tj v v^T
  // is applied to the panel columns right of J (v = 0 outside the panel rows
  // from J on, where the subtraction leaves the value unchanged)
#pragma unroll
  for (int s = 0; s < S; ++s) {
    const int lr = t + TH * s - roff;
    const bool below = lr > J && lr < dr;
    const bool diag = lr == J;
    const double v = below ? P[s][J] * scale : (diag ? 1.0 : 0.0);
    P[s][J] = below ? v : (diag ? beta : P[s][J]);
#pragma unroll
    for (int x = J + 1; x < NB; ++x) P[s][x] -= wgt[x] * v;
  }
  // LDS only: a global store here would hold up the next column, since a
  // workgroup barrier waits for the wave's outstanding memory operations
  if (t == 0) {
    sh.tauv[J] = tj;
#pragma unroll
    for (int q = 0; q < J; ++q) sh.G[J][q] = dots[q];
  }
}

template <int S, int NB, int J, int TH>
__device__ __forceinline__ void panel_columns(double (&P)[S][NB], PanelShared<NB, TH> &sh, int nb, int dr, int roff) {
  if constexpr (J < NB) {
    if (J < nb) {  // nb is uniform: every thread reaches the same barriers
      panel_column<S, NB, J, TH>(P, sh, nb, dr, roff);
      panel_columns<S, NB, J + 1, TH>(P, sh, nb, dr, roff);
    }
  }
}

// The column-by-column form: one workgroup reduction per column.  Takes any
// panel.  Ends without a barrier.
template <int S, int NB, int TH>
__device__ __forceinline__ void factor_panel_columns(double (&P)[S][NB], PanelShared<NB, TH> &sh, int nb, int dr,
                                                     int roff) {
  const int t = threadIdx.x;
  if (t < NB * NB) sh.G[t / NB][t % NB] = 0.0;
  if (t < NB) sh.tauv[t] = 0.0;
  panel_columns<S, NB, 0, TH>(P, sh, nb, dr, roff);  // its first barrier orders the zeroing
  __syncthreads();
  if (t < NB) {
    const int l = t;
    double row[NB];
#pragma unroll
    for (int J = 0; J < NB; ++J) {
      double a = 0.0;
#pragma unroll
      for (int q = 0; q < J; ++q)
        if (q >= l) a += row[q] * sh.G[J][q];
      row[J] = J < l ? 0.0 : (J == l ? sh.tauv[J] : -sh.tauv[J] * a);
      sh.T[l + J * NB] = row[J];
    }
  }
}

// W2 = T^T V^T C for V held like C (zero outside the panel's rows) and T's
// element t in thread t of every wave's first NB*NB lanes: one reduction of
// NB*NB values per wave and a sum over the waves, which every wave takes by
// itself, so there is a single barrier.  Lane l (mod NB*NB) returns
// W2(l / NB, l % NB).  `sh.red` must not be in use: callers separate two
// products by a barrier.
template <int S, int NB, int TH>
__device__ __forceinline__ double wy_product(const double (&V)[S][NB], const double (&C)[S][NB], double tel,
                                             PanelShared<NB, TH> &sh) {
  constexpr int NW2 = NB * NB;
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  double acc[NW2];
#pragma unroll
  for (int s = 0; s < S; ++s)
#pragma unroll
    for (int i = 0; i < NB; ++i)
#pragma unroll
      for (int c = 0; c < NB; ++c) {
        const double a = V[s][i] * C[s][c];
        acc[i * NB + c] = s == 0 ? a : acc[i * NB + c] + a;
      }
  __builtin_amdgcn_sched_barrier(0);
  wave_reduce<NW2>(acc);
  if ((lane & (kWave / NW2 - 1)) == 0) sh.red[wave][lane_value<NW2>(lane)] = acc[0];
  __syncthreads();
  const int e = lane % NW2, ei = e / NB, ec = e % NB;
  double w = 0.0;
#pragma unroll
  for (int q = 0; q < TH / kWave; ++q) w += sh.red[q][e];
  double w2 = 0.0;  // sum_{l <= i} T(l, i) W(l, c)
#pragma unroll
  for (int l = 0; l < NB; ++l) {
    const double tl = __shfl(tel, l + ei * NB, kWave);
    const double wl = __shfl(w, l * NB + ec, kWave);
    w2 += l <= ei ? tl * wl : 0.0;
  }
  return w2;
}

// row <- row - v W2
template <int NB>
__device__ __forceinline__ void update_row(double (&c)[NB], const double (&v)[NB], const double (&W2)[NB][NB]) {
#pragma unroll
  for (int x = 0; x < NB; ++x) {
    double q = 0.0;
#pragma unroll
    for (int i = 0; i < NB; ++i) q += v[i] * W2[i][x];
    c[x] -= q;
  }
}

template <int NB>
__device__ __forceinline__ void spread_w2(double w2, double (&W2)[NB][NB]) {
#pragma unroll
  for (int i = 0; i < NB; ++i)
#pragma unroll
    for (int x = 0; x < NB; ++x) W2[i][x] = readlane(w2, i * NB + x);
}

// C <- (I - V T^T V^T) C.
template <int S, int NB, int TH>
__device__ __forceinline__ void apply_wy(const double (&V)[S][NB], double (&C)[S][NB], double tel,
                                         PanelShared<NB, TH> &sh) {
  double W2[NB][NB];
  spread_w2<NB>(wy_product<S, NB, TH>(V, C, tel, sh), W2);
#pragma unroll
  for (int s = 0; s < S; ++s) update_row<NB>(C[s], V[s], W2);
}

// sqrt(s) and 1 / sqrt(s) for normal s: the hardware estimate (2^-24) with one
// third-order step, the root corrected once more.
__device__ __forceinline__ void root(double s, double &r, double &inv) {
  const double y = __builtin_amdgcn_rsq(s);
  const double e = fma(-(s * y), y, 1.0);
  inv = fma(y * e, fma(0.375, e, 0.5), y);
  const double q = s * inv;
  r = fma(fma(-q, q, s), 0.5 * inv, q);
}
// 1 / a for normal a: the hardware estimate with two Newton steps.
__device__ __forceinline__ double reciprocal(double a) {
  double y = __builtin_amdgcn_rcp(a);
  y = fma(fma(-a, y, 1.0), y, y);
  return fma(fma(-a, y, 1.0), y, y);
}

// A column of the panel must keep at least this share of its squared norm on
// entry below the diagonal at its turn for the Gram form to take the panel
// (see the accuracy note at factor_update), and at least kGramTiny of it in
// absolute terms (the root's estimate is for normal numbers; an exactly zero
// column is taken).  A norm whose square overflows is refused too.
constexpr double kGramKeep = 0.75, kGramKeepTall = 0.65;
constexpr int kGramTall = 256;  // rows from which it is the smaller
// With fewer rows the ones that the update turns into R's take up to that much:
// such panels are factored column by column without asking (10 x 2: 25 -> 21 us).
constexpr int kGramRows = 64;
constexpr double kGramTiny = 1e-280;
constexpr double kGramHuge = 1e307;

// a + b = hi + lo exactly (Knuth's two-sum).
__device__ __forceinline__ void two_sum(double a, double b, double &hi, double &lo) {
  hi = a + b;
  const double bb = hi - a;
  lo = (a - (hi - bb)) + (b - bb);
}

// The Gram form's share of a panel that the previous panel's update has not
// reached yet: per-wave partials of G = C^T C (rows above that update are zero)
// and the rows roff - NB .. roff + NB-1 of the block (zero where there is
// none).  roff: the panel's first row; no barrier inside, one is needed before
// factor_update.
template <int S, int NB, int TH>
__device__ __forceinline__ void gram_prepare(const double (&C)[S][NB], PanelShared<NB, TH> &sh, int roff) {
  constexpr int NG = PanelShared<NB, TH>::kGram, NP = pow2_at_least(NG);
  const int t = threadIdx.x;
  const int lane = t & (kWave - 1), wave = t / kWave;
  double acc[NP];
#pragma unroll
  for (int v = NG; v < NP; ++v) acc[v] = 0.0;
#pragma unroll
  for (int s = 0; s < S; ++s) {
    int v = 0;
#pragma unroll
    for (int y = 0; y < NB; ++y)
#pragma unroll
      for (int x = 0; x <= y; ++x, ++v) {
        const double a = C[s][x] * C[s][y];
        acc[v] = s == 0 ? a : acc[v] + a;
      }
  }
  auto put = [&](int base) {
    return [&, base](int s, int lr) {
#pragma unroll
      for (int x = 0; x < NB; ++x) sh.crow[base + lr][x] = C[s][x];
    };
  };
  if (roff >= NB) for_rows<S, NB, TH>(roff - NB, put(0));
  else if (t < NB * NB) sh.crow[t / NB][t % NB] = 0.0;
  for_rows<S, NB, TH>(roff, put(NB));
  __builtin_amdgcn_sched_barrier(0);
  wave_reduce<NP>(acc);
  if ((lane & (kWave / NP - 1)) == 0 && lane_value<NP>(lane) < NG) sh.gred[wave][lane_value<NP>(lane)] = acc[0];
}

// G over the waves as an unevaluated sum, for factor_small (what the sum over the
// waves rounds off would be the same for all rows of a reflector).  By the first
// wave, after a barrier behind gram_prepare.
template <int NB, int TH>
__device__ __forceinline__ void gram_total(PanelShared<NB, TH> &sh) {
  constexpr int NG = PanelShared<NB, TH>::kGram, NW = TH / kWave;
  const int lane = static_cast<int>(threadIdx.x) & (kWave - 1), v = min(lane, NG - 1);
  double w[NW], lo = 0.0;
#pragma unroll
  for (int q = 0; q < NW; ++q) w[q] = sh.gred[q][v];
#pragma unroll
  for (int h = NW / 2; h >= 1; h /= 2)
#pragma unroll
    for (int q = 0; q < h; ++q) {
      double e;
      two_sum(w[q], w[q + h], w[q], e);
      lo += e;
    }
  if (lane < NG) {
    sh.gtot[0][lane] = w[0];
    sh.gtot[1][lane] = lo;
  }
  __builtin_amdgcn_sched_barrier(0);
}

// Row and column of element v of a packed upper triangle (columns in turn).
template <int NB>
struct PackedPairs {
  uint64_t xs = 0, ys = 0;
  constexpr PackedPairs() {
    int v = 0;
    for (int y = 0; y < NB; ++y)
      for (int x = 0; x <= y; ++x, ++v) {
        xs |= static_cast<uint64_t>(x) << (4 * v);
        ys |= static_cast<uint64_t>(y) << (4 * v);
      }
  }
};

// One wave: the panel's reflectors from G and its first rows (see
// factor_update).  w2 as wy_product returns it.  Fills sh.top, sh.U, sh.tauv,
// sh.T and sh.slow; the caller's barrier follows the first three.
template <int NB, int TH>
__device__ __forceinline__ void factor_small(PanelShared<NB, TH> &sh, int nb, double w2, double share, bool last) {
  constexpr int NG = PanelShared<NB, TH>::kGram;
  int lane = threadIdx.x & (kWave - 1);
  asm volatile("" : "+v"(lane));  // its LDS addresses are formed here, not kept through the chain's loop
  // G less the 2 NB rows that the update turns into rows of R and the panel's
  // own first rows: the rest of G does not change under the update (an
  // orthogonal transform of rows lo..hi).
  const int dr_ = (lane / NB) % (2 * NB), dx = lane % NB;
  double dv = sh.crow[dr_][dx];
  {
    double q = 0.0;
#pragma unroll
    for (int i = 0; i < NB; ++i) q += sh.vrow[dr_][i] * __shfl(w2, i * NB + dx, kWave);
    dv -= q;
  }
  if (lane < 2 * NB * NB) sh.crow[dr_][dx] = dv;
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
  __builtin_amdgcn_wave_barrier();
  const double keepl = sh.gtot[0][min(lane, NG - 1)];  // norms on entry (pairs x = y)
  double gs, gl;
  {
    static_assert(NG <= 16, "four bits a pair");
    constexpr PackedPairs<NB> pairs;
    const int v4 = 4 * min(lane, NG - 1);
    const int x = static_cast<int>(pairs.xs >> v4) & 15, y = static_cast<int>(pairs.ys >> v4) & 15;
    double rows = 0.0;
#pragma unroll
    for (int r = 0; r < 2 * NB; ++r) rows += sh.crow[r][x] * sh.crow[r][y];
    two_sum(keepl, -rows, gs, gl);
    gl += sh.gtot[1][min(lane, NG - 1)];
    if (x != y) {
      gs += gl;
      gl = 0.0;
    }
  }
  double g[NB][NB], D[NB][NB], a[NB][NB], U[NB][NB], vv[NB][NB], tj[NB], keep[NB];
  {
    int v = 0;
#pragma unroll
    for (int y = 0; y < NB; ++y)
#pragma unroll
      for (int x = 0; x <= y; ++x, ++v) {
        g[x][y] = readlane(gs, v);
        D[x][y] = x == y ? -readlane(gl, v) : 0.0;
        if (x == y) keep[x] = readlane(keepl, v);
      }
  }
#pragma unroll
  for (int r = 0; r < NB; ++r) {
    tj[r] = 0.0;
#pragma unroll
    for (int x = 0; x < NB; ++x) {
      a[r][x] = sh.crow[NB + r][x];
      U[r][x] = r == x ? 1.0 : 0.0;
      vv[r][x] = 0.0;
    }
  }
  bool bad = false;
  auto gg = [&](int x, int y) -> double & { return x <= y ? g[x][y] : g[y][x]; };
#pragma unroll
  for (int J = 0; J < NB; ++J) {
    if (J < nb) {  // uniform
      double tot[NB];
#pragma unroll
      for (int x = 0; x < NB; ++x) {
        double q = 0.0;
#pragma unroll
        for (int r = J + 1; r < NB; ++r) q += a[r][J] * a[r][x];
        if (x >= J) q -= D[J][x];
        tot[x] = gg(J, x) + q;
      }
      const double alpha = a[J][J], sq = tot[J];
      const bool zero = keep[J] == 0.0;
      // (NaN: refused)
      bad = bad || !(zero || (sq >= share * keep[J] && sq >= kGramTiny && keep[J] <= kGramHuge));
      double beta = alpha, scale = 0.0;
      if (!zero) {
        double nrm, inv;
        root(fma(alpha, alpha, sq), nrm, inv);
        beta = alpha >= 0.0 ? -nrm : nrm;
        // (beta - alpha) / beta of the rounded beta, which scale is taken from too
        const double num = nrm + fabs(alpha), quot = num * inv;
        tj[J] = fma(fma(-quot, nrm, num), inv, quot);
        scale = reciprocal(alpha - beta);
      }
      double cx[NB];
#pragma unroll
      for (int x = 0; x < NB; ++x) {
        const double dot = a[J][x] + scale * tot[x];
        if (x < J) vv[x][J] = dot;
        const double w = (x > J && x < nb) ? tj[J] * dot : 0.0;
        cx[x] = w * scale;
        if (x > J) {
          a[J][x] -= w;
#pragma unroll
          for (int r = J + 1; r < NB; ++r) a[r][x] -= cx[x] * a[r][J];
#pragma unroll
          for (int y = 0; y <= J; ++y) U[y][x] -= cx[x] * U[y][J];
        }
      }
#pragma unroll
      for (int r = J + 1; r < NB; ++r) a[r][J] *= scale;
      a[J][J] = beta;
#pragma unroll
      for (int y = 0; y <= J; ++y) U[y][J] *= scale;
      // G of the changed columns: hy = (column J)^T (new column y).  What the
      // steps take from G is summed by itself (D, from what G was rounded by) and
      // subtracted where G is used: G is rounded once, not at every step.
      double gJ[NB], hy[NB];
#pragma unroll
      for (int y = J; y < NB; ++y) gJ[y] = g[J][y] - D[J][y];
#pragma unroll
      for (int y = J + 1; y < NB; ++y) hy[y] = gJ[y] - cx[y] * gJ[J];
#pragma unroll
      for (int x = J + 1; x < NB; ++x) {
#pragma unroll
        for (int y = x; y < NB; ++y) D[x][y] += cx[x] * hy[y] + cx[y] * gJ[x];
#pragma unroll
        for (int q = 0; q < J; ++q) g[q][x] -= cx[x] * g[q][J];
      }
#pragma unroll
      for (int y = J + 1; y < NB; ++y) g[J][y] = scale * hy[y];
#pragma unroll
      for (int q = 0; q < J; ++q) g[q][J] *= scale;
    }
  }
  if (lane == 0) {
    sh.slow = bad ? 1 : 0;
#pragma unroll
    for (int r = 0; r < NB; ++r)
#pragma unroll
      for (int x = 0; x < NB; ++x) {
        sh.top[r][x] = a[r][x];
        if (r <= x) sh.U[r][x] = last ? U[r][x] : (r == x ? 1.0 : 0.0);
      }
#pragma unroll
    for (int x = 0; x < NB; ++x) sh.tauv[x] = tj[x];
  }
  __syncthreads();
  // T while the other waves already form their rows
  if (!bad && lane == 0) {
#pragma unroll
    for (int l = 0; l < NB; ++l) {
      double row[NB];
#pragma unroll
      for (int J = 0; J < NB; ++J) {
        double q = 0.0;
#pragma unroll
        for (int k = l; k < J; ++k) q += row[k] * vv[k][J];
        row[J] = J < l ? 0.0 : (J == l ? tj[J] : -tj[J] * q);
        sh.T[l + J * NB] = row[J];
      }
    }
  }
}

// T to store_t and tau, by the first wave, which wrote sh.T and sh.tauv (LDS
// operations of a wave are in order).
template <int NB, int TH, typename StoreT>
__device__ __forceinline__ void publish_small(PanelShared<NB, TH> &sh, int nb, int k0, double *__restrict__ tau,
                                              StoreT &&store_t) {
  if (__builtin_amdgcn_readfirstlane(threadIdx.x / kWave) != 0) return;
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
  __builtin_amdgcn_wave_barrier();
  int e = threadIdx.x;
  asm volatile("" : "+v"(e));  // (as factor_small's lane)
  if (e < NB * NB) store_t(e, sh.T[e]);
  if (e < nb) tau[k0 + e] = sh.tauv[e];
}

// The last update of a block, C <- (I - V T^T V^T) C, and the factorisation
// of the panel it becomes (columns k0 .. k0+nb-1, first row roff of the
// block's rows, the matrix ending at row hi); V and tel as for wy_product (V =
// 0 when there is no update, roff = 0).  gram_prepare, a barrier and gram_total precede it.
// The update's rows roff - NB .. roff-1 become rows of R: they go to
// put_r(row, column, value), row and column within the block, and are zero in
// C afterwards.  Writes tau and hands T to store_t(element, value) (column-
// major NB x NB, T(0:J, J) = -tau_J T(0:J, 0:J) V_{<J}^T v_J, T(J, J) = tau_J),
// both by the first wave.  Ends without a barrier.
//
// Gram form.  With the panel's rows [A1; A2] (A1 the first NB), its reflectors
// depend on A2 only through G = A2^T A2, so no column waits for a reduction of
// its own: the first wave runs the NB Householder steps on A1 and G (column x
// of A2 becomes column x minus a multiple of column J, and G is updated to
// match), accumulates the column operations in the upper triangular U, and
// every row below becomes (row) U, in the same sweep that applies the update.
// G itself is summed before the update's reflectors arrive (gram_prepare):
// the update is orthogonal, so G changes only by the rows it turns into R.
// A panel is bound by this dependent chain (one reduction, two barriers, NB
// roots and reciprocals, its rows' way in and out), not by its flops; qr.hip
// has its parts measured.
//
// Accuracy.  Each norm and product below the diagonal comes from G by
// subtraction; what a norm is off by, all rows of its reflector share.  The
// subtrahends are therefore summed by themselves, G's last sum keeps its
// rounding errors, and a panel with a column whose norm falls below 0.65 (0.75 with
// fewer than 256 rows) of the one that G was summed for (correlated columns, few
// rows, nothing below the diagonal, non-finite entries) is factored column by column.
// Against an 80-bit factorisation, over the error of the column-by-column form
// throughout (R and V; max ||(Q R - Y)_j|| / ||Y_j||; ||Q^T Q - I||): 0.85, 0.98, 0.95
// for 400 x 101 columns of norms 1 to 1e-4, and 0.97, 0.94, 0.94 for 800 x 201 with
// singular values that fall by eight decades in 1000; with G rounded at every step
// and a share of a quarter 1.31, 1.12, 1.36 for the first.  Where the shares
// lie: at 0.65 panels of 70 to 130 rows come out at up to 1.04, at 0.5 taller ones at
// 1.02 to 1.04; at 0.75 91 of the 251 panels of a 4000 x 1001 sketch of the
// second kind go column by column (2.9 ms), at 0.65 21 (2.26).
//
// warm: the panel has kGramRows rows, and gram_prepare and gram_total ran (without:
// the update alone, or with last the column-by-column form).  warm without last
// runs the factorisation's code too, with U the identity (left out for a panel
// that would be refused) and nothing stored.
template <int S, int NB, int TH, typename PutR, typename StoreT>
__device__ __forceinline__ void factor_update(double (&C)[S][NB], const double (&V)[S][NB], double tel,
                                              PanelShared<NB, TH> &sh, int nb, int hi, int roff, int k0,
                                              double *__restrict__ tau, bool warm, bool last, PutR &&put_r, StoreT &&store_t) {
  const int t = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(t / kWave);
  // the update's reflectors in the panel's first rows and the NB rows above
  auto put = [&](int base) {
    return [&, base](int s, int lr) {
#pragma unroll
      for (int i = 0; i < NB; ++i) sh.vrow[base + lr][i] = V[s][i];
    };
  };
  if (roff >= NB) for_rows<S, NB, TH>(roff - NB, put(0));
  else if (t < NB * NB) sh.vrow[t / NB][t % NB] = 0.0;
  for_rows<S, NB, TH>(roff, put(NB));
  const double w2 = wy_product<S, NB, TH>(V, C, tel, sh);
  __builtin_amdgcn_sched_barrier(0);
  if (warm) {
    if (wave == 0)
      factor_small<NB, TH>(sh, nb, w2, hi - roff >= kGramTall ? kGramKeepTall : kGramKeep, last);
    else
      __syncthreads();
  }
  __builtin_amdgcn_sched_barrier(0);
  double W2[NB][NB];
  spread_w2<NB>(w2, W2);
  // refused: a round that is not the last then leaves the panel as it is (the
  // identity would carry a non-finite column into the ones to its right)
  const bool gram = warm && __builtin_amdgcn_readfirstlane(sh.slow) == 0;
#pragma unroll
  for (int s = 0; s < S; ++s) update_row<NB>(C[s], V[s], W2);
  if (roff >= NB)
    for_rows<S, NB, TH>(roff - NB, [&](int s, int lr) {
#pragma unroll
      for (int x = 0; x < NB; ++x) {
        put_r(lr, x, C[s][x]);
        C[s][x] = 0.0;
      }
    });
  if (gram) {
    double U[NB][NB];
#pragma unroll
    for (int y = 0; y < NB; ++y)
#pragma unroll
      for (int x = y; x < NB; ++x) U[y][x] = sh.U[y][x];
#pragma unroll
    for (int s = 0; s < S; ++s)
#pragma unroll
      for (int x = NB - 1; x >= 0; --x) {
        double q = C[s][0] * U[0][x];
#pragma unroll
        for (int y = 1; y <= x; ++y) q += C[s][y] * U[y][x];
        C[s][x] = q;
      }
  }
  if (last && !gram) {
    __syncthreads();  // earlier users of the shared buffers are done
    factor_panel_columns<S, NB, TH>(C, sh, nb, hi - roff, roff);
  } else if (last) {
    for_rows<S, NB, TH>(roff, [&](int s, int lr) {
#pragma unroll
      for (int x = 0; x < NB; ++x) C[s][x] = sh.top[lr][x];
    });
  }
  if (last) publish_small<NB, TH>(sh, nb, k0, tau, store_t);
}

// A first panel of fewer than kGramRows rows: nothing to apply and no Gram form.
template <int S, int NB, int TH, typename StoreT>
__device__ __forceinline__ void factor_first_short(double (&C)[S][NB], PanelShared<NB, TH> &sh, int nb, int rows,
                                                   double *__restrict__ tau, StoreT &&store_t) {
  factor_panel_columns<S, NB, TH>(C, sh, nb, rows, 0);
  publish_small<NB, TH>(sh, nb, 0, tau, store_t);
}

}  // namespace qr_dev
}  // namespace sap
