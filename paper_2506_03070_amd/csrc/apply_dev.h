// Device code of the sketch apply's scatter form shared by the single and the
// batched launches: rows of A added into a strip of Y in LDS through a packed
// copy of the sketch.
#pragma once

#include "common.h"

namespace sap {
namespace apply_dev {

// Packed sketch rows (zeta = 8): eight 16-bit entries, the row of Y in bits
// 0-14 (d, the strip's spare row, for one outside [0, d)), bit 15 set for a
// negative sign.
constexpr int kPackMaxD = 32766;
__device__ __forceinline__ uint32_t pack_entry(int32_t r, int d, uint32_t pos) {
  return static_cast<uint32_t>(r >= 0 && r < d ? r : d) | ((pos ^ 1u) << 15);
}

// Adds the eight signed copies of v into column c of the strip acc (rows of W).
template <int W>
__device__ __forceinline__ void add_packed(double *acc, int c, uint4 e, double v) {
  const uint32_t word[4] = {e.x, e.y, e.z, e.w};
  const int lo = __double2loint(v), hi = __double2hiint(v);
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    const uint32_t h = (k & 1) ? word[k >> 1] >> 16 : word[k >> 1];
    const uint32_t neg = ((k & 1) ? word[k >> 1] : word[k >> 1] << 16) & 0x80000000u;
    atomicAdd(acc + (h & 0x7FFFu) * W + c, __hiloint2double(hi ^ static_cast<int>(neg), lo));
  }
}

// Rows of a batch per lane group; callers keep the bytes of a wave's batch, at
// most 64 kPackRows rows of A, below 2^31 (32-bit offsets).
constexpr int kPackRows = 8;

// Rows [i_begin, i_end) of A's columns col0 .. col0 + W-1 (those past the last
// repeat it; their sums are not stored) added into acc by a workgroup of
// `waves` waves.  The loads of a wave's next batch of rows are issued before
// the adds of the current one, and rows past the end come as zeros from the
// buffer's bounds: no branch and no select in the loop.  With int32 indices a
// batch is 88 registers, too many to hold two; a row's packed entries are 16
// bytes, and need no range check.  Cycles of a CU for 64 adds before and after,
// FP64 A: 15.4 -> 11.6 at 32 columns (400000 x 150, d = 600), 14.6 -> 10.1 at 16
// (200000 x 256, d = 1024), 15.1 -> 13.3 at 8 (300007 x 513, d = 2052), 20.0 ->
// 18.5 at 4 (65536 x 1000, d = 4000); the LDS adds alone take 9.5 without
// conflicts, which is what bounds it.
template <typename TA, int W>
__device__ __forceinline__ void add_rows_packed(double *acc, const TA *A, int64_t lda, int n, int col0,
                                                const uint4 *rows, int64_t i_begin, int64_t i_end, int waves) {
  constexpr int RPW = kWave / W, E = static_cast<int>(sizeof(TA));
  constexpr int U = E == 8 ? 6 : kPackRows;  // two batches within 128 registers
  const int lane = threadIdx.x & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int g = lane / W, c = lane % W;
  const int ld = static_cast<int>(lda) * E;
  const int a0 = g * ld + min(col0 + c, n - 1) * E;
  struct Batch {
    uint32_t a[U][E == 8 ? 2 : 1];
    uint4 e[U];
  };
  auto load = [&](int64_t base, Batch &b) {
    const int64_t left = min(i_end - base, static_cast<int64_t>(RPW * U));
    const auto ra = __builtin_amdgcn_make_buffer_rsrc(const_cast<TA *>(A + base * lda), 0,
                                                      static_cast<int>(((left - 1) * lda + n) * E), 0x00020000);
    const auto re = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint4 *>(rows + base), 0,
                                                      static_cast<int>(left * 16), 0x00020000);
    int at = a0;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if constexpr (E == 8) {
        const auto v = __builtin_amdgcn_raw_buffer_load_b64(ra, at, 0, 0);
        b.a[u][0] = v[0];
        b.a[u][1] = v[1];
      } else if constexpr (E == 4) {
        b.a[u][0] = __builtin_amdgcn_raw_buffer_load_b32(ra, at, 0, 0);
      } else {
        b.a[u][0] = __builtin_amdgcn_raw_buffer_load_b16(ra, at, 0, 0);
      }
      const auto e = __builtin_amdgcn_raw_buffer_load_b128(re, (g + u * RPW) * 16, 0, 0);
      b.e[u] = make_uint4(e[0], e[1], e[2], e[3]);
      at += RPW * ld;
    }
  };
  auto add = [&](const Batch &b) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      double v;
      if constexpr (E == 8) v = __hiloint2double(static_cast<int>(b.a[u][1]), static_cast<int>(b.a[u][0]));
      else if constexpr (E == 4) v = static_cast<double>(__uint_as_float(b.a[u][0]));
      else v = static_cast<double>(__uint_as_float(b.a[u][0] << 16));
      add_packed<W>(acc, c, b.e[u], v);
    }
  };
  const int64_t step = static_cast<int64_t>(waves) * RPW * U;
  int64_t base = i_begin + static_cast<int64_t>(wave) * RPW * U;
  if (base >= i_end) return;
  Batch b0, b1;
  load(base, b0);
  for (;;) {
    if (base + step < i_end) load(base + step, b1);
    add(b0);
    base += step;
    if (base >= i_end) return;
    if (base + step < i_end) load(base + step, b0);
    add(b1);
    base += step;
    if (base >= i_end) return;
  }
}

}  // namespace apply_dev
}  // namespace sap
