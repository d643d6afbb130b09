// Sketch apply Y = S [A b] on gfx950 (the sketching step of Alg. 1; the paper calls a
// library sparse-times-dense product, Sec. 3).
//
// Column j of S has zeta nonzeros, so row i of [A b] is added, with sign, into
// zeta rows of Y.  A is streamed from HBM once; Y (d x ncols, column-major)
// is cut into column strips, each owned by one workgroup for its whole life.
// Sums are FP64 whatever the types of A and Y.  Two forms:
//
// Scatter (apply_strip_kernel).  The strip Y[r_lo : r_lo + DR, c0 : c0 + W] sits
// in LDS, W the widest power of two (<= 32) with d * W doubles in 160 KB:
//   * W lanes serve one row of A: they load its W-element piece once and add
//     it into the zeta target rows with LDS atomics (ds_add_f64), so a wave
//     instruction serves 64 / W rows; the zeta row indices are read once per
//     row (same address for the W lanes: one broadcast);
//   * only when even W = 1 does not fit (d >= 20000) are the rows of Y split
//     into ranges, each range skipping the nonzeros outside it.
// It is bound by the LDS adds: 9.5 cycles a wave instruction without conflicts,
// 10.5 as run at W = 32, 18.5 at W = 4 (bank conflicts between the rows of an
// instruction), more below, where the lines of A count as well.
//
// Gather (apply_lists_kernel, apply_gather_kernel).  The strip (4 columns, or 2
// above 8192 rows) sits in registers, thread t holding rows t, t + 1024, ...;
// tiles of A's rows are staged in LDS and each thread reads the pieces that its
// rows take, from lists of the sketch sorted by target row within each tile
// (built once per apply, read by every strip).  A 16-byte LDS read serves two
// FP64 or four FP32 columns without an atomic, and the strip's width does not
// shrink with d.
//
// Common to both: the strips that share a cache line of A (consecutive strips)
// run on the same XCD, so a line fetched from HBM for one strip serves its
// neighbours from that XCD's L2; when strips alone do not fill the chip, the
// rows of A are split into slices whose partial strips a second kernel sums
// in a fixed order; the 1/sqrt(zeta) scale is applied once, after summation.
#include <hip/hip_bf16.h>

#include <algorithm>
#include <cmath>
#include <type_traits>

#include "apply_dev.h"
#include "common.h"

namespace sap {
namespace {

using namespace apply_dev;

constexpr int kApplyThreads = 1024;
constexpr int kApplyWaves = kApplyThreads / kWave;
constexpr size_t kApplyLdsBytes = 160000;  // gfx950: up to 160 KB of LDS per workgroup
constexpr int kXcds = 8;
constexpr int kUnroll = 8;                 // rows in flight per lane group
constexpr int kMaxW = 32;
constexpr int64_t kMinSliceRows = 4096;
constexpr int64_t kFineSliceRows = 512;

template <typename TA, typename T>
__device__ __forceinline__ T load_as(const TA *p) {
  if constexpr (std::is_same<TA, __hip_bfloat16>::value)
    return static_cast<T>(__bfloat162float(*p));
  else
    return static_cast<T>(*p);
}

// One work item = (strip, range, slice).
// FORM 2 (one range, zeta = 8, a packed copy of the sketch): add_rows_packed,
// but for the strip that holds b's column beside A's.
// FORM 1 (one range, zeta = 8, idx 16-byte aligned; where the copy does not pay
// or has no room in the workspace): per row two 16-byte index loads, every load of a batch
// of rows issued before any add, and no branches: a row past the slice end
// adds zeros, and an index outside [0, d) adds into a spare LDS row that is
// never written out.
// FORM 0: indices four at a time, those outside the range skipped.
// The strip fills the LDS, so a CU holds one workgroup (4 waves a SIMD);
// telling the compiler so lets it keep every load of a batch in flight
// instead of trading registers for an occupancy it never gets.
// The sums are FP64 for an FP32 Y too: ds_add_f32 takes 193 cycles a wave
// instruction on gfx950 in every access pattern, ds_add_f64 9.5 to 26
// (300007 x 513 FP32, d = 2052, FP32 Y: 12.1 ms with FP32 sums).
// run_if (nullable): the launch does nothing unless *run_if is set.
template <typename TA, typename TO, int W, int FORM>
__global__ __launch_bounds__(kApplyThreads) __attribute__((amdgpu_waves_per_eu(1, 4))) void apply_strip_kernel(
    const int32_t *__restrict__ idx, const uint4 *__restrict__ packed, const uint64_t *__restrict__ sign,
    int zeta, const TA *__restrict__ A,
    int64_t lda, const double *__restrict__ b, int64_t m, int n, int ncols, int d, int dr, int nstrips,
    int nranges, int nslices, int64_t rows_per_slice, TO *__restrict__ out, int64_t ldo, int64_t slice_stride,
    double h, int scale_now, const int *__restrict__ run_if) {
  extern __shared__ unsigned char lds_raw[];
  if (run_if && *run_if == 0) return;
  double *acc = reinterpret_cast<double *>(lds_raw);
  constexpr int RPW = kWave / W;  // rows per wave instruction

  // XCD-aware decode: workgroup IDs are dealt round-robin over the XCDs;
  // each XCD gets a contiguous block of work items, strip fastest.
  const int total = nstrips * nranges * nslices;
  const int per_xcd = (total + kXcds - 1) / kXcds;
  const int w = (blockIdx.x % kXcds) * per_xcd + blockIdx.x / kXcds;
  if (w >= total) return;
  const int strip = w % nstrips;
  const int range = (w / nstrips) % nranges;
  const int slice = w / (nstrips * nranges);
  const int c0 = strip * W;
  const int r_lo = range * dr;
  const int rows_here = min(dr, d - r_lo);

  for (int e = threadIdx.x; e < (rows_here + (FORM != 0 ? 1 : 0)) * W; e += kApplyThreads) acc[e] = 0.0;
  __syncthreads();

  const int64_t i_begin = static_cast<int64_t>(slice) * rows_per_slice;
  const int64_t i_end = min(m, i_begin + rows_per_slice);
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  const int g = lane / W, c = lane % W;
  const int col = c0 + c;
  const bool col_a = col < n;
  const bool col_b = (col == n) && (col < ncols);
  constexpr int64_t kStride = static_cast<int64_t>(kApplyWaves) * RPW * kUnroll;
  const bool packed_strip = FORM == 2 && (c0 + W <= n || ncols == n);  // uniform: no lane takes b
  if constexpr (FORM == 2) {
    if (packed_strip) add_rows_packed<TA, W>(acc, A, lda, n, c0, packed, i_begin, i_end, kApplyWaves);
  }
  for (int64_t base = i_begin + wave * (RPW * kUnroll) + g; base < i_end && !packed_strip; base += kStride) {
    if constexpr (FORM == 2) {
      double val[kUnroll];
      uint4 raw[kUnroll];
#pragma unroll
      for (int u = 0; u < kUnroll; ++u) {
        const int64_t i0 = base + u * RPW;
        const bool ok = i0 < i_end;
        const int64_t i = ok ? i0 : i_end - 1;
        double a = 0.0;
        if (col_a) a = load_as<TA, double>(A + i * lda + col);
        else if (col_b) a = b[i];
        val[u] = ok ? a : 0.0;
        raw[u] = packed[i];
      }
#pragma unroll
      for (int u = 0; u < kUnroll; ++u) add_packed<W>(acc, c, raw[u], val[u]);
    } else if constexpr (FORM == 1) {
      double val[kUnroll];
      uint32_t sg[kUnroll];
      int4 ix[kUnroll][2];
#pragma unroll
      for (int u = 0; u < kUnroll; ++u) {
        const int64_t i0 = base + u * RPW;
        const bool ok = i0 < i_end;
        const int64_t i = ok ? i0 : i_end - 1;
        double a = 0.0;
        if (col_a) a = load_as<TA, double>(A + i * lda + col);
        else if (col_b) a = b[i];
        val[u] = ok ? a : 0.0;
        sg[u] = static_cast<uint32_t>(sign[i]);
        const int4 *ip = reinterpret_cast<const int4 *>(idx + i * 8);
        ix[u][0] = ip[0];
        ix[u][1] = ip[1];
      }
#pragma unroll
      for (int u = 0; u < kUnroll; ++u) {
        const int rr[8] = {ix[u][0].x, ix[u][0].y, ix[u][0].z, ix[u][0].w,
                           ix[u][1].x, ix[u][1].y, ix[u][1].z, ix[u][1].w};
#pragma unroll
        for (int k = 0; k < 8; ++k) {
          const int r = static_cast<unsigned>(rr[k]) < static_cast<unsigned>(d) ? rr[k] : d;
          atomicAdd(acc + r * W + c, ((sg[u] >> k) & 1u) ? val[u] : -val[u]);
        }
      }
    } else {
#pragma unroll 2
      for (int u = 0; u < kUnroll; ++u) {
        const int64_t i = base + u * RPW;
        if (i >= i_end) break;
        double a = 0.0;
        if (col_a) a = load_as<TA, double>(A + i * lda + col);
        else if (col_b) a = b[i];
        const uint64_t sg = sign[i];
        const int32_t *ri = idx + i * zeta;
        for (int k0 = 0; k0 < zeta; k0 += 4) {
          int rr[4];
#pragma unroll
          for (int q = 0; q < 4; ++q) rr[q] = (k0 + q < zeta) ? ri[k0 + q] : -1;
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const int r = rr[q] - r_lo;
            if (rr[q] >= 0 && static_cast<unsigned>(r) < static_cast<unsigned>(rows_here))
              atomicAdd(acc + r * W + c, ((sg >> (k0 + q)) & 1ull) ? a : -a);
          }
        }
      }
    }
  }
  __syncthreads();

  const TO scale = scale_now ? static_cast<TO>(h) : TO(1);
  TO *dst = out + static_cast<int64_t>(slice) * slice_stride;
  for (int e = threadIdx.x; e < rows_here * W; e += kApplyThreads) {
    const int q = e / rows_here, r = e % rows_here;
    const int cc = c0 + q;
    if (cc < ncols) dst[(r_lo + r) + static_cast<int64_t>(cc) * ldo] = static_cast<TO>(acc[r * W + q]) * scale;
  }
}

// Y[r, c] = h * sum_s part[s][r + c*d], slices summed in ascending order.
// Does nothing when *run_if (nullable) differs from want.
template <typename TO>
__global__ __launch_bounds__(256) void apply_reduce_kernel(const TO *__restrict__ part, int nslices,
                                                           int64_t slice_stride, int d, int ncols,
                                                           TO *__restrict__ Y, int64_t ldy, double h,
                                                           const int *__restrict__ run_if, int want) {
  if (run_if && *run_if != want) return;
  const int64_t e = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
  if (e >= static_cast<int64_t>(d) * ncols) return;
  const int r = static_cast<int>(e % d);
  const int c = static_cast<int>(e / d);
  double s = 0.0;
  int k = 0;
  for (; k + 8 <= nslices; k += 8) {  // eight loads in flight, added in slice order
    TO v[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) v[q] = part[(k + q) * slice_stride + e];
#pragma unroll
    for (int q = 0; q < 8; ++q) s += v[q];
  }
  for (; k < nslices; ++k) s += part[k * slice_stride + e];
  Y[r + static_cast<int64_t>(c) * ldy] = static_cast<TO>(s) * static_cast<TO>(h);
}

// The packed copy (zeta = 8, d <= kPackMaxD), one row a thread.
__global__ __launch_bounds__(256) void pack_rows_kernel(const int32_t *__restrict__ idx,
                                                        const uint64_t *__restrict__ sign, int64_t m, int d,
                                                        uint4 *__restrict__ out, const int *__restrict__ run_if) {
  if (run_if && *run_if == 0) return;
  const int64_t i = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
  if (i >= m) return;
  const uint32_t s = static_cast<uint32_t>(sign[i]);
  uint32_t e[8];
#pragma unroll
  for (int k = 0; k < 8; ++k) e[k] = pack_entry(idx[i * 8 + k], d, (s >> k) & 1u);
  out[i] = make_uint4(e[0] | (e[1] << 16), e[2] | (e[3] << 16), e[4] | (e[5] << 16), e[6] | (e[7] << 16));
}

// What apply_workspace_bytes counts a packed copy for (a size that callers'
// limits are held against): this many bytes of strips re-reading 40 bytes a row.
constexpr double kCompactMinRereadBytes = 16e9;

// ---- gather form -------------------------------------------------------------
constexpr int kGatherWaves = kApplyWaves;
constexpr int kGatherTileBytes = 128 * 1024;
constexpr int kGatherMaxRows = 8192;  // rows of a tile: their pieces' places and the zero row's take 14 bits
constexpr int kSpareChunks = 8;       // past the lists: the gather reads up to three chunks ahead

// Element type of a staged tile, rows per tile.
template <typename TA>
using staged_t = typename std::conditional<std::is_same<TA, double>::value, double, float>::type;
constexpr int gather_rows(int esize, int w) {
  return kGatherTileBytes / (esize * w) < kGatherMaxRows ? kGatherTileBytes / (esize * w) : kGatherMaxRows;
}

// Lists.  The rows of Y come in groups of 64, group g = s * 16 + wave in slot s
// of a wave of the gather; a tile's groups are laid out wave by wave, so each
// wave reads its chunks in one run.  A chunk holds 4 entries for each of the 64
// rows (8 bytes a lane): the place of the row's piece (Piece, below) in bits 0-13,
// bit 15 set for a negative sign; a group has as many chunks as its longest row needs, the other
// rows' lists are filled up with the tile's zero row (index R).  One workgroup
// a tile: count, the chunk offsets, a run of chunks claimed from *cursor, the
// fill, then every entry placed at its rank.  A sketch whose rows are so
// unevenly hit that the lists pass `cap` chunks sets *flag: the gather then does
// nothing and the scatter form runs instead.
__global__ void apply_lists_reset_kernel(unsigned int *cursor, int *flag) {
  *cursor = 0;
  *flag = 0;
}

__global__ __launch_bounds__(kApplyThreads) void apply_lists_kernel(
    const int32_t *__restrict__ idx, const uint64_t *__restrict__ sign, int64_t m, int zeta, int d, int S, int R, int H,
    unsigned int cap, uint32_t *__restrict__ off, uint16_t *__restrict__ lists, unsigned int *cursor, int *flag) {
  extern __shared__ int lcount[];  // 64 * 16 * S row counts, then 16 * S + 1 offsets
  __shared__ unsigned int base_sh;
  const int groups = kGatherWaves * S;
  int *loff = lcount + groups * kWave;
  const int t = threadIdx.x;
  const int lane = t & (kWave - 1), wave = t / kWave;
  const int64_t i0 = static_cast<int64_t>(blockIdx.x) * R;
  const int rows = static_cast<int>(min<int64_t>(R, m - i0));
  const int count = rows * zeta;
  const int32_t *ti = idx + i0 * zeta;
  for (int e = t; e < groups * kWave; e += kApplyThreads) lcount[e] = 0;
  __syncthreads();
  for (int e = t; e < count; e += kApplyThreads) {
    const unsigned r = static_cast<unsigned>(ti[e]);
    if (r < static_cast<unsigned>(d)) atomicAdd(lcount + r, 1);
  }
  __syncthreads();
  for (int o = wave; o < groups; o += kGatherWaves) {  // group at place o: slot o % S of wave o / S
    const int g = (o % S) * kGatherWaves + o / S;
    int k = lcount[g * kWave + lane];
#pragma unroll
    for (int x = 32; x >= 1; x >>= 1) k = max(k, __shfl_xor(k, x, kWave));
    if (lane == 0) loff[o] = (k + 3) / 4;
  }
  __syncthreads();
  if (wave == 0) {  // exclusive scan of the chunk counts
    int run = 0;
    for (int o0 = 0; o0 < groups; o0 += kWave) {
      const int v = o0 + lane < groups ? loff[o0 + lane] : 0;
      int x = v;
#pragma unroll
      for (int k = 1; k < kWave; k <<= 1) {
        const int y = __shfl_up(x, k, kWave);
        if (lane >= k) x += y;
      }
      if (o0 + lane < groups) loff[o0 + lane] = run + x - v;
      run += __shfl(x, kWave - 1, kWave);
    }
    if (lane == 0) {
      loff[groups] = run;
      const unsigned base = atomicAdd(cursor, static_cast<unsigned>(run));
      const bool over = base > cap || static_cast<unsigned>(run) > cap - base;
      if (over) atomicOr(flag, 1);
      base_sh = over ? 0xFFFFFFFFu : base;
    }
  }
  __syncthreads();
  const unsigned base = base_sh;
  if (base == 0xFFFFFFFFu) return;  // uniform
  for (int o = t; o <= groups; o += kApplyThreads)
    off[static_cast<int64_t>(blockIdx.x) * (groups + 1) + o] = base + loff[o];
  const uint32_t pad = static_cast<uint32_t>(H * R) * 0x10001u;
  uint4 *fill = reinterpret_cast<uint4 *>(lists) + static_cast<int64_t>(base) * (kWave / 2);
  for (int e = t; e < loff[groups] * (kWave / 2); e += kApplyThreads) fill[e] = make_uint4(pad, pad, pad, pad);
  for (int e = t; e < groups * kWave; e += kApplyThreads) lcount[e] = 0;
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the fill is in place before any entry
  __syncthreads();
  for (int e = t; e < count; e += kApplyThreads) {
    const unsigned r = static_cast<unsigned>(ti[e]);
    if (r < static_cast<unsigned>(d)) {
      const int i = e / zeta, k = e - i * zeta;
      const int rank = atomicAdd(lcount + r, 1);
      const int g = static_cast<int>(r) / kWave;
      const int64_t chunk = static_cast<int64_t>(base) + loff[(g % kGatherWaves) * S + g / kGatherWaves] + (rank >> 2);
      const unsigned neg = ((sign[i0 + i] >> k) & 1ull) ? 0u : 0x8000u;
      const unsigned at = H == 2 ? 2u * i + (i & 1u) : static_cast<unsigned>(i);
      lists[(chunk * kWave + (r & (kWave - 1))) * 4 + (rank & 3)] = static_cast<uint16_t>(at | neg);
    }
  }
}

// A staged piece of a row (W elements, at most 32 bytes) in LDS, read as H parts
// of 16 (or one of 8) bytes.  A list entry's low 14 bits count parts: part 0 of
// row r sits at H r, of two parts at 2 r + (r & 1) with part 1 beside it (the
// index with its lowest bit flipped), so that one address serves both and the
// parts 0 of all rows spread over all banks.
template <typename TL, int W>
struct Piece {
  static constexpr int kPer = 16 / static_cast<int>(sizeof(TL)) < W ? 16 / static_cast<int>(sizeof(TL)) : W;
  static constexpr int H = W / kPer;
  static constexpr int kBytes = kPer * static_cast<int>(sizeof(TL));
  static_assert(H == 1 || H == 2, "one or two parts");
  typedef TL vec __attribute__((ext_vector_type(kPer)));
};

// One work item = (strip of W columns, slice of tiles).  Per tile: the pieces of
// its rows go from registers to LDS, then every thread sums its rows' lists
// while the next tile's loads go out one by one between the chunks: loads
// return in order, so a list asked for behind a whole tile would wait for all
// of it (that cost 1.65 ms of 4.3 at 2^20 x 1000, d = 4000).  Lists run three
// chunks ahead.  Bound by the lines that move from L2: a row's 16- or 32-byte
// piece takes a 128-byte line (2^19 x 1000 FP64: 1.3e8 of the 1.7e8 requests, 17 of 22
// GB, 1.67 ms; 1.18 of then 1.76 without the tile loads).  The LDS
// (active 73% of the kernel, 10 cycles an instruction, 59% of them bank conflicts) and
// the vector work (10 instructions an entry of 4 columns) come next; lists are about twice as long as their entries, since the
// 64 rows of a group wait for the longest.
template <typename TA, typename TO, int S, int W>
__global__ __launch_bounds__(kApplyThreads) __attribute__((amdgpu_waves_per_eu(4, 4))) void apply_gather_kernel(
    const uint32_t *__restrict__ off, const uint2 *__restrict__ lists, const int *__restrict__ flag,
    const TA *__restrict__ A, int64_t lda, int64_t m, int n, int d,
    int nstrips, int nslices, int ntiles, int tiles_per_slice, TO *__restrict__ out, int64_t ldo,
    int64_t slice_stride, double h, int scale_now) {
  using TL = staged_t<TA>;
  using P = Piece<TL, W>;
  constexpr int R = gather_rows(sizeof(TL), W);
  constexpr int kRowsPer = kApplyThreads / W;  // rows staged per step (even: a thread's rows have one parity)
  constexpr int PF = R / kRowsPer;
  constexpr int PS = (PF + S - 1) / S;         // next-tile loads per slot, in its first kSteps chunks
  constexpr int kSteps = 4;
  // with 64 registers of sums, fewer chunks ahead and fewer reads in flight
  constexpr int kRing = S * W >= 32 ? 2 : 3;
  constexpr int kAtOnce = (S * W >= 32 ? 2 : 4) / P::H;  // entries whose reads are in flight together
  extern __shared__ unsigned char lds_raw[];
  if (*flag != 0) return;
  const int total = nstrips * nslices;
  const int per_xcd = (total + kXcds - 1) / kXcds;
  const int item = (blockIdx.x % kXcds) * per_xcd + blockIdx.x / kXcds;
  if (item >= total) return;
  const int strip = item % nstrips, slice = item / nstrips;
  const int c0 = strip * W;
  const int t0 = slice * tiles_per_slice, t1 = min(ntiles, t0 + tiles_per_slice);
  const int t = threadIdx.x;
  const int lane = t & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(t / kWave);

  // staging: thread t takes column c0 + t % W of rows t / W, + kRowsPer, ...;
  // columns past the last repeat it (their sums are not stored).  A tile is a
  // buffer that ends with A's last row (rows past it read as zeros), so that an
  // element's address is one 32-bit addition.
  const int sc = t % W, sr = t / W;
  const int ld = static_cast<int>(lda) * static_cast<int>(sizeof(TA));
  const int at0 = sr * ld + min(c0 + sc, n - 1) * static_cast<int>(sizeof(TA));
  const int part = P::H * sr + ((sc / P::kPer) ^ (P::H == 2 ? (sr & 1) : 0));
  TL *put = reinterpret_cast<TL *>(lds_raw + part * P::kBytes) + sc % P::kPer;
  TL pf[PF];
  __amdgpu_buffer_rsrc_t tile;
  int at = at0;
  auto at_tile = [&](int tl) {
    at = at0;
    const int64_t i0 = static_cast<int64_t>(tl) * R;
    const int64_t bytes = ((min(m - i0, static_cast<int64_t>(R)) - 1) * lda + n) * static_cast<int64_t>(sizeof(TA));
    tile = __builtin_amdgcn_make_buffer_rsrc(const_cast<TA *>(A + i0 * lda), 0, static_cast<int>(bytes), 0x00020000);
  };
  auto load_row = [&](int q) {
    if constexpr (sizeof(TA) == 8) {
      const auto v = __builtin_amdgcn_raw_buffer_load_b64(tile, at, 0, 0);
      pf[q] = __hiloint2double(static_cast<int>(v[1]), static_cast<int>(v[0]));
    } else if constexpr (sizeof(TA) == 4) {
      pf[q] = __int_as_float(static_cast<int>(__builtin_amdgcn_raw_buffer_load_b32(tile, at, 0, 0)));
    } else {
      pf[q] = __int_as_float(static_cast<int>(__builtin_amdgcn_raw_buffer_load_b16(tile, at, 0, 0)) << 16);
    }
    at += kRowsPer * ld;
    asm volatile("" : "+v"(at));  // one running address, not PF of them kept for the whole kernel
  };
  if (t < W) reinterpret_cast<TL *>(lds_raw + static_cast<size_t>(R) * P::H * P::kBytes)[t] = TL(0);  // the zero row

  double acc[S][W];
#pragma unroll
  for (int s = 0; s < S; ++s)
#pragma unroll
    for (int w = 0; w < W; ++w) acc[s][w] = 0.0;
  at_tile(t0);
#pragma unroll
  for (int q = 0; q < PF; ++q) load_row(q);
  for (int tl = t0; tl < t1; ++tl) {
    // (the runs of chunks are followed by spare ones: reading ahead stays inside)
    const uint32_t *to = off + static_cast<int64_t>(tl) * (kGatherWaves * S + 1) + wave * S;
    const uint2 *lp = lists + static_cast<int64_t>(to[0]) * kWave;
    uint2 ring[kRing];
#pragma unroll
    for (int k = 0; k < kRing; ++k) ring[k] = lp[k * kWave + lane];
    __syncthreads();  // the previous tile's reads are done
#pragma unroll
    for (int q = 0; q < PF; ++q) put[q * kRowsPer * P::H * P::kPer] = pf[q];
    __syncthreads();
    at_tile(min(tl + 1, t1 - 1));  // (the last tile is loaded once more, not used)
#pragma unroll
    for (int s = 0; s < S; ++s) {
      int left = static_cast<int>(to[s + 1] - to[s]);
      auto sum_chunk = [&]() {
        const uint2 ch = ring[0];
#pragma unroll
        for (int k = 0; k + 1 < kRing; ++k) ring[k] = ring[k + 1];
        lp += kWave;
        ring[kRing - 1] = lp[(kRing - 1) * kWave + lane];
        constexpr int kShift = P::kBytes == 16 ? 4 : 3;
#pragma unroll
        for (int q0 = 0; q0 < 4; q0 += kAtOnce) {
          typename P::vec v[kAtOnce][P::H];
#pragma unroll
          for (int q = 0; q < kAtOnce; ++q) {
            const uint32_t e2 = q0 + q < 2 ? ch.x : ch.y;
            const uint32_t at = ((q0 + q) & 1) ? (e2 >> (16 - kShift)) & (0x3FFFu << kShift) : (e2 & 0x3FFFu) << kShift;
            v[q][0] = *reinterpret_cast<const typename P::vec *>(lds_raw + at);
            if constexpr (P::H == 2) v[q][1] = *reinterpret_cast<const typename P::vec *>(lds_raw + (at ^ 16u));
          }
#pragma unroll
          for (int q = 0; q < kAtOnce; ++q) {
            const uint32_t e2 = q0 + q < 2 ? ch.x : ch.y;
            const uint32_t neg = (((q0 + q) & 1) ? e2 : (e2 << 16)) & 0x80000000u;
            const double sgn = __hiloint2double(static_cast<int>(neg | 0x3FF00000u), 0);
#pragma unroll
            for (int hh = 0; hh < P::H; ++hh)
#pragma unroll
              for (int x = 0; x < P::kPer; ++x)
                acc[s][hh * P::kPer + x] = fma(static_cast<double>(v[q][hh][x]), sgn, acc[s][hh * P::kPer + x]);
          }
        }
      };
#pragma unroll
      for (int k = 0; k < kSteps; ++k) {
#pragma unroll
        for (int q = s * PS + k * PS / kSteps; q < s * PS + (k + 1) * PS / kSteps; ++q)
          if (q < PF) load_row(q);
        if (k < left) sum_chunk();
      }
      for (left -= kSteps; left > 0; --left) sum_chunk();
    }
  }
  const TO scale = scale_now ? static_cast<TO>(h) : TO(1);
  TO *dst = out + static_cast<int64_t>(slice) * slice_stride;
#pragma unroll
  for (int s = 0; s < S; ++s) {
    const int r = (s * kGatherWaves + wave) * kWave + lane;
    if (r >= d) continue;
#pragma unroll
    for (int w = 0; w < W; ++w)
      if (c0 + w < n) dst[r + static_cast<int64_t>(c0 + w) * ldo] = static_cast<TO>(acc[s][w]) * scale;
  }
}

// ---- plans --------------------------------------------------------------------
struct ApplyPlan {
  int w, dr, nstrips, nranges, nslices;
  int64_t rows_per_slice;
};

// Strip widths, and the slices every workspace has room for.
ApplyPlan make_plan(int num_cus, int64_t m, int d, int ncols, size_t esize) {
  ApplyPlan p{};
  // columns of a full-height strip (plus one spare row)
  const size_t fit = kApplyLdsBytes / (esize * (static_cast<size_t>(d) + 1));
  int w = 1;
  while (w * 2 <= kMaxW && static_cast<size_t>(w * 2) <= fit) w *= 2;
  // no wider than the matrix needs
  while (w > 1 && w / 2 >= ncols) w /= 2;
  p.w = w;
  if (fit >= 1) {
    p.nranges = 1;
    p.dr = d;
  } else {
    const int dr_max = static_cast<int>(kApplyLdsBytes / esize) - 1;  // plus the spare row
    p.nranges = (d + dr_max - 1) / dr_max;
    p.dr = (d + p.nranges - 1) / p.nranges;
  }
  p.nstrips = (ncols + w - 1) / w;
  // One resident workgroup per CU when the strip fills the LDS; split the
  // rows into slices when the strips alone leave CUs idle.
  const int items = p.nstrips * p.nranges;
  int ns = 1;
  if (items < num_cus) ns = (num_cus + items - 1) / items;
  const int64_t max_slices = std::max<int64_t>(1, m / kMinSliceRows);
  if (ns > max_slices) ns = static_cast<int>(max_slices);
  p.rows_per_slice = (m + ns - 1) / ns;
  p.nslices = static_cast<int>((m + p.rows_per_slice - 1) / p.rows_per_slice);
  if (p.nslices < 1) p.nslices = 1;
  return p;
}

// Time estimates (us) that the choices below compare; measured on one MI355X.
// Cycles of a CU for 64 adds in the scatter form, loads and bank conflicts
// included, with packed rows: 10.5 for W = 32 and 16, 13.5, 18.5 (d = 4000); for
// W = 2 (d = 8000) and 1 (12000) 25 and 33 while A stays in the 256 MB cache
// behind the XCDs (20000 rows of 1000 FP64) and 31 and 49 beyond (2^18 rows),
// where a 128-byte line moves for each 16 or 8 bytes; 3 more from the 32-bit
// indices, half as much again on the general path (zeta != 8).
double scatter_us(int num_cus, int zeta, const ApplyPlan &p, bool pack, bool near) {
  const double clk = ((p.w >= 16 ? 10.5 : p.w == 8 ? 13.5 : p.w == 4 ? 18.5 : p.w == 2 ? (near ? 25 : 31)
                                                                                       : (near ? 33 : 49)) *
                          (zeta == 8 && p.nranges == 1 ? 1.0 : 1.5) +
                      (pack ? 0 : 3)) *
                     p.nranges;
  const double items = static_cast<double>(p.nstrips) * p.nranges * p.nslices;
  const double rounds = std::ceil(items / num_cus);
  // with zeta = 8 whole batches of rows of the 16 waves, a short last one as long
  // as the others; the general path stops at the slice's last row
  const int64_t step = zeta == 8 && p.nranges == 1 ? static_cast<int64_t>(kApplyWaves) * (kWave / p.w) * kUnroll : 1;
  const double rows = static_cast<double>((p.rows_per_slice + step - 1) / step * step);
  const double strip = (rows * zeta * p.w / 64.0) * clk / 2400.0 / p.nranges;
  return rounds * (strip + 5.0);  // 5: the strip cleared and written out
}
// Partial strips written and read back at about 4 TB/s.
double parts_us(int nslices, int d, int ncols, size_t es) {
  return nslices > 1 ? 5.0 + 2.0 * nslices * static_cast<double>(d) * ncols * es / 4e6 : 0.0;
}

// The slices of p re-chosen, shorter ones too, by those estimates: 260 work
// items on 256 CUs take as long as 512 (300007 x 513, d = 2052), and 4 strips of
// 20000 rows in slices of 4096 keep 16 CUs busy (20000 x 100, d = 400: 114 us,
// 33 in slices of 512).
ApplyPlan fine_plan(int num_cus, int64_t m, int zeta, int d, int ncols, size_t es, const ApplyPlan &p, bool pack,
                    bool near) {
  ApplyPlan best = p;
  double best_us = scatter_us(num_cus, zeta, p, pack, near) + parts_us(p.nslices, d, ncols, es);
  const int most = static_cast<int>(std::min<int64_t>(64, (m + kFineSliceRows - 1) / kFineSliceRows));
  for (int ns = 1; ns <= most; ++ns) {
    ApplyPlan q = p;
    q.rows_per_slice = (m + ns - 1) / ns;
    q.nslices = static_cast<int>((m + q.rows_per_slice - 1) / q.rows_per_slice);
    const double us = scatter_us(num_cus, zeta, q, pack, near) + parts_us(q.nslices, d, ncols, es);
    if (us < 0.98 * best_us) {
      best_us = us;
      best = q;
    }
  }
  return best;
}

// Whether the strips read a packed copy: it saves about 3 cycles of a CU for 64
// adds (200000 x 257, d = 1024: 191 -> 141 us; 65536 x 501, d = 2600: 165 -> 142)
// and costs a launch and 56 bytes a row (20000 x 101, d = 400: 31 -> 33 us).
bool wants_pack(int num_cus, int64_t m, int zeta, int d, int64_t lda, const ApplyPlan &p) {
  if (zeta != 8 || p.nranges != 1 || d > kPackMaxD || lda >= (int64_t(1) << 31) / (8 * kWave * kPackRows)) return false;
  const double adds = static_cast<double>(m) * zeta * p.nstrips * p.w / 64.0;
  return adds / num_cus * 3.0 / 2400.0 > 4.0 + static_cast<double>(m) * 56.0 / 4e6;
}

size_t part_bytes(int nslices, int d, int ncols, size_t es) {
  return nslices > 1 ? static_cast<size_t>(nslices) * d * ncols * es + 256 : 0;
}

struct GatherPlan {
  bool use = false;
  int w = 0, s = 0;
  int rows = 0, ntiles = 0, nstrips = 0, nslices = 1, tiles_per_slice = 0;
  unsigned int cap = 0;  // chunks
  size_t bytes = 0;
  double us = 0.0;
};

// The gather form for A's n columns, if it is estimated to beat the scatter
// form's scatter: a step of the 16 waves, each through one chunk, takes about
// 0.74 us whatever the types (0.69 at d = 4000 FP64, 0.76 at d = 8192 FP32), the
// lists about 25 us and 1 ns an entry of a tile, b's column 25 us.  2^20 x 1000 FP64, d = 4000:
// 3.27 ms against 4.24; 2^18 x 2048 FP32, d = 8192: 1.75 against 3.6; 2^18 x 1000
// FP64, d = 8000: 0.92 against 1.64.  Below d = 2500 the scatter's strips are 8
// or more columns wide and the gather leaves waves without rows.
GatherPlan make_gather(int num_cus, int64_t m, int zeta, int d, int n, int64_t lda, sap_dtype a_type, size_t es_out,
                       double scatter) {
  GatherPlan g;
  const bool f64 = a_type == SAP_F64;
  if (d > 16384 || d < 2500) return g;
  g.w = d <= 8192 ? 4 : 2;
  g.s = d <= 3 * kApplyThreads ? 3 : d <= 4 * kApplyThreads ? 4 : d <= 8 * kApplyThreads ? 8 : 16;
  g.rows = gather_rows(f64 ? 8 : 4, g.w);
  // a tile is addressed with 32-bit byte offsets
  if (static_cast<double>(lda) * g.rows * (f64 ? 8 : a_type == SAP_F32 ? 4 : 2) >= 2147483648.0) return g;
  const int64_t ntiles = (m + g.rows - 1) / g.rows;
  if (ntiles > (1 << 20)) return g;
  g.ntiles = static_cast<int>(ntiles);
  g.nstrips = (n + g.w - 1) / g.w;
  // a bound on the mean longest list of a group of 64 rows (Poisson lengths)
  const double mu = static_cast<double>(std::min<int64_t>(m, g.rows)) * zeta / d;
  const double longest = mu + 2.7 * std::sqrt(mu) + 2.0;
  const int groups = (d + kWave - 1) / kWave;
  const double tile_us =
      ((groups + kGatherWaves - 1) / kGatherWaves) * ((mu + 2.55 * std::sqrt(mu) + 1.5) / 4.0) * 0.74 + 0.2;
  double best = 0.0;
  for (int k = 1; k <= 8 && k <= g.ntiles; ++k) {
    const int tps = (g.ntiles + k - 1) / k;
    const int ns = (g.ntiles + tps - 1) / tps;
    const double us = std::ceil(static_cast<double>(g.nstrips) * ns / num_cus) * tps * tile_us +
                      parts_us(ns, d, n, es_out);
    if (k == 1 || us < 0.98 * best) {
      best = us;
      g.nslices = ns;
      g.tiles_per_slice = tps;
    }
  }
  const double lists = 50.0 + std::ceil(static_cast<double>(g.ntiles) / num_cus) * g.rows * zeta * 1e-3;
  if (best + lists > 0.97 * scatter) return g;
  const double cap = static_cast<double>(g.ntiles) * groups * ((longest + 3.0) / 4.0) + 1024.0;
  if (cap > 2.0e9) return g;
  g.cap = static_cast<unsigned>(cap);
  g.bytes = 4 * 256 + static_cast<size_t>(g.ntiles) * (kGatherWaves * g.s + 1) * sizeof(uint32_t) +
            (static_cast<size_t>(g.cap) + kSpareChunks) * kWave * 8 + part_bytes(g.nslices, d, n, es_out);
  g.us = best + lists;
  g.use = true;
  return g;
}

// Everything an apply with room for it would do: the scatter form's plan for
// all columns; the gather's with the scatter plans of its fallback and of b.
struct FullPlan {
  ApplyPlan all, a, b;
  GatherPlan g;
  bool pack;
  size_t scatter_bytes, gather_bytes;
  double us;  // estimate of the form it picks
};
FullPlan full_plan(int num_cus, int64_t m, int zeta, int d, int n, int64_t lda, bool with_b, sap_dtype a_type,
                   size_t es, ApplyForm form) {
  FullPlan f;
  const int ncols = n + (with_b ? 1 : 0);
  const ApplyPlan p = make_plan(num_cus, m, d, ncols, sizeof(double));
  f.pack = wants_pack(num_cus, m, zeta, d, lda, p);
  const bool near = static_cast<double>(m) * lda * (a_type == SAP_F64 ? 8 : a_type == SAP_F32 ? 4 : 2) <= 256e6;
  f.all = fine_plan(num_cus, m, zeta, d, ncols, es, p, f.pack, near);
  const size_t copy = f.pack ? static_cast<size_t>(m) * 16 + 256 : 0;
  f.scatter_bytes = part_bytes(f.all.nslices, d, ncols, es) + copy + 1024;
  f.a = make_plan(num_cus, m, d, n, sizeof(double));
  f.b = fine_plan(num_cus, m, zeta, d, 1, es, make_plan(num_cus, m, d, 1, sizeof(double)), false, true);
  f.us = scatter_us(num_cus, zeta, f.all, f.pack, near) + parts_us(f.all.nslices, d, ncols, es);
  f.g = make_gather(num_cus, m, zeta, d, n, lda, a_type, es,
                    form == kApplyScatter ? 0.0 : form == kApplyGather ? INFINITY : f.us);
  if (f.g.use) f.us = f.g.us;
  f.gather_bytes = f.g.use ? f.g.bytes + part_bytes(f.a.nslices, d, n, es) + copy +
                                 (with_b ? part_bytes(f.b.nslices, d, 1, es) : 0) + 2048
                           : 0;
  return f;
}

template <typename TA, typename TO, int W>
void launch_strip(const ApplyPlan &p, dim3 grid, size_t lds, hipStream_t st, const sps_sketch *S, const TA *A,
                  int64_t lda, const double *b, int n, int ncols, TO *out, int64_t ldo, int64_t slice_stride,
                  double h, int scale_now, const uint4 *packed, const int *run_if) {
  const bool fast = S->zeta == 8 && p.nranges == 1 && (reinterpret_cast<uintptr_t>(S->idx) % 16 == 0);
#define SAP_STRIP(FORM)                                                                                           \
  apply_strip_kernel<TA, TO, W, FORM><<<grid, kApplyThreads, lds, st>>>(                                          \
      S->idx, packed, S->sign, S->zeta, A, lda, b, S->m, n, ncols, S->d, p.dr, p.nstrips, p.nranges, p.nslices,   \
      p.rows_per_slice, out, ldo, slice_stride, h, scale_now, run_if)
  if (packed != nullptr) SAP_STRIP(2);
  else if (fast) SAP_STRIP(1);
  else SAP_STRIP(0);
#undef SAP_STRIP
}

// The scatter form for columns 0 .. ncols-1 of [A b] into Y.
template <typename TA, typename TO>
sap_status scatter(sap_ctx *ctx, const sps_sketch *S, const TA *A, int64_t lda, const double *b, int n, int ncols,
                   const ApplyPlan &p, bool pack, TO *Y, int64_t ldy, Carve &cv, const int *run_if,
                   hipStream_t st) {
  const double h = 1.0 / std::sqrt(static_cast<double>(S->zeta));
  TO *out = Y;
  int64_t ldo = ldy, slice_stride = 0;
  int scale_now = 1;
  if (p.nslices > 1) {
    out = cv.take<TO>(static_cast<size_t>(p.nslices) * S->d * ncols);
    ldo = S->d;
    slice_stride = static_cast<int64_t>(S->d) * ncols;
    scale_now = 0;
  }
  const uint4 *packed = nullptr;
  if (pack) {
    uint4 *c = cv.take<uint4>(static_cast<size_t>(S->m));
    pack_rows_kernel<<<static_cast<unsigned>((S->m + 255) / 256), 256, 0, st>>>(S->idx, S->sign, S->m, S->d, c, run_if);
    SAP_HIP_TRY(hipGetLastError());
    packed = c;
  }
  const int total = p.nstrips * p.nranges * p.nslices;
  const int per_xcd = (total + kXcds - 1) / kXcds;
  const dim3 grid(static_cast<unsigned>(per_xcd * kXcds));
  const size_t lds = (static_cast<size_t>(p.dr) + 1) * p.w * sizeof(double);
#define SAP_STRIP_W(W) \
  launch_strip<TA, TO, W>(p, grid, lds, st, S, A, lda, b, n, ncols, out, ldo, slice_stride, h, scale_now, packed, run_if)
  switch (p.w) {
    case 1: SAP_STRIP_W(1); break;
    case 2: SAP_STRIP_W(2); break;
    case 4: SAP_STRIP_W(4); break;
    case 8: SAP_STRIP_W(8); break;
    case 16: SAP_STRIP_W(16); break;
    default: SAP_STRIP_W(32); break;
  }
#undef SAP_STRIP_W
  SAP_HIP_TRY(hipGetLastError());
  if (p.nslices > 1) {
    const int64_t tot = static_cast<int64_t>(S->d) * ncols;
    apply_reduce_kernel<TO><<<static_cast<unsigned>((tot + 255) / 256), 256, 0, st>>>(
        out, p.nslices, slice_stride, S->d, ncols, Y, ldy, h, run_if, 1);
    SAP_HIP_TRY(hipGetLastError());
  }
  return SAP_OK;
}

template <typename TA, typename TO>
sap_status gather(sap_ctx *ctx, const sps_sketch *S, const TA *A, int64_t lda, int n,
                  const GatherPlan &g, TO *Y, int64_t ldy, Carve &cv, int **flag_out, hipStream_t st) {
  const double h = 1.0 / std::sqrt(static_cast<double>(S->zeta));
  const int groups = kGatherWaves * g.s;
  int *flag = cv.take<int>(1);
  unsigned int *cursor = cv.take<unsigned int>(1);
  uint32_t *off = cv.take<uint32_t>(static_cast<size_t>(g.ntiles) * (groups + 1));
  uint16_t *lists = cv.take<uint16_t>((static_cast<size_t>(g.cap) + kSpareChunks) * kWave * 4);
  *flag_out = flag;
  TO *out = Y;
  int64_t ldo = ldy, slice_stride = 0;
  int scale_now = 1;
  if (g.nslices > 1) {
    out = cv.take<TO>(static_cast<size_t>(g.nslices) * S->d * n);
    ldo = S->d;
    slice_stride = static_cast<int64_t>(S->d) * n;
    scale_now = 0;
  }
  apply_lists_reset_kernel<<<1, 1, 0, st>>>(cursor, flag);
  apply_lists_kernel<<<g.ntiles, kApplyThreads, (static_cast<size_t>(groups) * kWave + groups + 1) * sizeof(int), st>>>(
      S->idx, S->sign, S->m, S->zeta, S->d, g.s, g.rows, g.w * static_cast<int>(sizeof(staged_t<TA>)) > 16 ? 2 : 1, g.cap, off, lists, cursor, flag);
  SAP_HIP_TRY(hipGetLastError());
  const int total = g.nstrips * g.nslices;
  const dim3 grid(static_cast<unsigned>((total + kXcds - 1) / kXcds * kXcds));
  const size_t lds = static_cast<size_t>(g.rows + 1) * g.w * sizeof(staged_t<TA>);
#define SAP_GATHER(SS, W)                                                                                        \
  apply_gather_kernel<TA, TO, SS, W><<<grid, kApplyThreads, lds, st>>>(                                           \
      off, reinterpret_cast<const uint2 *>(lists), flag, A, lda, S->m, n, S->d, g.nstrips, g.nslices,             \
      g.ntiles, g.tiles_per_slice, out, ldo, slice_stride, h, scale_now)
  switch (g.s) {
    case 3: SAP_GATHER(3, 4); break;
    case 4: SAP_GATHER(4, 4); break;
    case 8: SAP_GATHER(8, 4); break;
    default: SAP_GATHER(16, 2); break;
  }
#undef SAP_GATHER
  SAP_HIP_TRY(hipGetLastError());
  if (g.nslices > 1) {
    const int64_t tot = static_cast<int64_t>(S->d) * n;
    apply_reduce_kernel<TO><<<static_cast<unsigned>((tot + 255) / 256), 256, 0, st>>>(
        out, g.nslices, slice_stride, S->d, n, Y, ldy, h, flag, 0);
    SAP_HIP_TRY(hipGetLastError());
  }
  return SAP_OK;
}

template <typename TA, typename TO>
sap_status apply_typed(sap_ctx *ctx, const sps_sketch *S, const TA *A, int64_t lda, const double *b, int n,
                       sap_dtype a_type, TO *Y, int64_t ldy, void *work, size_t work_bytes, hipStream_t st,
                       ApplyForm form) {
  const int ncols = n + (b != nullptr ? 1 : 0);
  Carve cv(work);
  FullPlan f = full_plan(ctx->num_cus, S->m, S->zeta, S->d, n, lda, b != nullptr, a_type, sizeof(TO), form);
  if (f.g.use && f.gather_bytes <= work_bytes) {
    // A's columns by the gather (by the scatter form if the sketch is too
    // uneven for it), b's by the scatter form: one column
    int *flag = nullptr;
    sap_status s = gather<TA, TO>(ctx, S, A, lda, n, f.g, Y, ldy, cv, &flag, st);
    if (s != SAP_OK) return s;
    s = scatter<TA, TO>(ctx, S, A, lda, nullptr, n, n, f.a, f.pack, Y, ldy, cv, flag, st);
    if (s != SAP_OK || b == nullptr) return s;
    return scatter<TA, TO>(ctx, S, nullptr, 1, b, 0, 1, f.b, false, Y + static_cast<int64_t>(n) * ldy, ldy, cv,
                           nullptr, st);
  }
  if (f.scatter_bytes > work_bytes) {  // what apply_workspace_bytes counts
    f.all = make_plan(ctx->num_cus, S->m, S->d, ncols, sizeof(double));
    f.pack = f.pack && part_bytes(f.all.nslices, S->d, ncols, sizeof(TO)) + static_cast<size_t>(S->m) * 16 + 1280 <=
                           work_bytes;
  }
  return scatter<TA, TO>(ctx, S, A, lda, b, n, ncols, f.all, f.pack, Y, ldy, cv, nullptr, st);
}

}  // namespace

// Scratch of sps_apply_noalloc: a file-scope device array, one copy per GPU
// the library runs on, held until the process ends.  Host code never uses
// its name as an address (on the host it names a stand-in, not device
// memory): apply_scratch_init looks up this device's copy once and the
// context keeps that address.
static __device__ __align__(256) unsigned char g_apply_scratch[kNoAllocScratchBytes];

sap_status apply_scratch_init(sap_ctx *ctx) {
  void *p = nullptr;
  const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(g_apply_scratch));
  if (e != hipSuccess) return hip_fail(ctx, e, "hipGetSymbolAddress(apply scratch)");
  if (p == nullptr) return fail(ctx, SAP_EDEVICE, "apply scratch: no device address");
  ctx->apply_scratch = p;
  ctx->apply_scratch_bytes = kNoAllocScratchBytes;
  return SAP_OK;
}

// What every apply is given at least (and the size a caller's limits are held
// against): the scatter form's partial strips and packed copy.  An FP32 Y's
// FP64 sums make narrower strips and so never more slices than counted here.
size_t apply_workspace_bytes(sap_ctx *ctx, int64_t m, int zeta, int d, int ncols, sap_dtype y_type) {
  const size_t es = (y_type == SAP_F64) ? 8 : 4;
  const ApplyPlan p = make_plan(ctx->num_cus, m, d, ncols, es);
  size_t bytes = kApplyNoScratch;
  if (p.nslices > 1) bytes += static_cast<size_t>(p.nslices) * d * ncols * es;
  if (zeta == 8 && p.nranges == 1 && d <= 65535 &&
      static_cast<double>(p.nstrips) * static_cast<double>(m) * 40.0 >= kCompactMinRereadBytes)
    bytes += static_cast<size_t>(m) * 16 + 256;
  return bytes;
}

// What the gather form, finer slices and a packed copy use when they may; 0 for
// an apply that writes Y alone.
size_t apply_workspace_wanted(sap_ctx *ctx, int64_t m, int zeta, int d, int n, int64_t lda, bool with_b,
                              sap_dtype a_type, sap_dtype y_type, ApplyForm form) {
  const FullPlan f = full_plan(ctx->num_cus, m, zeta, d, n, lda, with_b, a_type, y_type == SAP_F64 ? 8 : 4, form);
  if (!f.g.use && !f.pack && f.all.nslices == 1) return 0;
  return (f.g.use ? f.gather_bytes : f.scatter_bytes) + 1024;
}

ApplyForm apply_form(sap_ctx *ctx, int64_t m, int zeta, int d, int n, int64_t lda, bool with_b, sap_dtype a_type,
                     sap_dtype y_type) {
  return full_plan(ctx->num_cus, m, zeta, d, n, lda, with_b, a_type, y_type == SAP_F64 ? 8 : 4, kApplyChoose).g.use
             ? kApplyGather
             : kApplyScatter;
}

double apply_estimate_us(sap_ctx *ctx, int64_t m, int zeta, int d, int n, int64_t lda, bool with_b, sap_dtype a_type,
                         sap_dtype y_type, ApplyForm form) {
  return full_plan(ctx->num_cus, m, zeta, d, n, lda, with_b, a_type, y_type == SAP_F64 ? 8 : 4, form).us;
}

sap_status launch_apply(sap_ctx *ctx, const sps_sketch *S, const void *A, int64_t lda,
                        sap_dtype a_type, const double *b, int n, void *Y, int64_t ldy,
                        sap_dtype y_type, void *work, size_t work_bytes, hipStream_t st, ApplyForm form) {
#define SAP_APPLY(TA, TO)                                                                                      \
  return apply_typed<TA, TO>(ctx, S, static_cast<const TA *>(A), lda, b, n, a_type, static_cast<TO *>(Y), ldy, \
                             work, work_bytes, st, form)
  if (y_type == SAP_F64) {
    switch (a_type) {
      case SAP_F64: SAP_APPLY(double, double);
      case SAP_F32: SAP_APPLY(float, double);
      case SAP_BF16: SAP_APPLY(__hip_bfloat16, double);
    }
  } else {
    switch (a_type) {
      case SAP_F64: SAP_APPLY(double, float);
      case SAP_F32: SAP_APPLY(float, float);
      case SAP_BF16: SAP_APPLY(__hip_bfloat16, float);
    }
  }
#undef SAP_APPLY
  return fail(ctx, SAP_EINVAL, "sps_apply: unsupported dtype combination");
}

}  // namespace sap

// For the tests: 2 if this apply runs the gather form where it has the scratch
// that it asks for, else 1.
extern "C" int sap_internal_apply_form(sap_ctx *ctx, int64_t m, int zeta, int d, int n, int64_t lda, int with_b,
                                       int a_type, int y_type) {
  return sap::apply_form(ctx, m, zeta, d, n, lda, with_b != 0, static_cast<sap_dtype>(a_type),
                         static_cast<sap_dtype>(y_type)) == sap::kApplyGather
             ? 2
             : 1;
}
