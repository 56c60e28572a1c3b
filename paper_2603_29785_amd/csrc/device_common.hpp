// Device-side row metadata, twiddle tables and launch geometry shared by the
// QTAM kernels (gfx950).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "fft_engine.hpp"

namespace qtam {

// ---------------------------------------------------------------------------
// Device-side tables
// ---------------------------------------------------------------------------
struct RowMeta {
  int s, lo, hi, off;   // centre bin, kept bin range, offset in the packed tables
};

// Envelope slot u of a row holds the kept bin c with (c - s) mod L = u (the
// roll of bin s to slot 0, Sec. III / App. A). The support holds at most L
// bins, so that bin is unique when it exists: c = lo + d with
// d = (u + s - lo) mod L, kept iff d <= hi - lo. Slot entries of a
// power-of-two L:
template <int L>
__device__ __forceinline__ int slot_entry(int u, const RowMeta& rm) {
  static_assert((L & (L - 1)) == 0, "power-of-two rows");
  return (u + rm.s - rm.lo) & (L - 1);
}

// A row is centred when its support lies inside s - L/2 .. s + L/2 - 1: the
// signed slot offset j (u, or u - L above L/2) then gives c = s + j directly.
// Every row whose window is narrower than the band is centred (its support
// is within s - h .. s + h and 2h + 1 <= L); a row of a regularised window
// keeps the whole band 0..N/2 and may not be.
__device__ __forceinline__ bool row_centred(const RowMeta& rm, int L) {
  return rm.lo >= rm.s - L / 2 && rm.hi < rm.s + L / 2;
}

// exp(-2 pi i m / N) for m in [0, N) as fine[m & (F-1)] * coarse[m >> log2 F]
template <typename C>
struct Twiddle2 {
  const C* fine;
  const C* coarse;
  int bits;
  __device__ __forceinline__ C operator()(int64_t m) const {
    const int64_t lo = m & ((int64_t(1) << bits) - 1);
    return c_mul(fine[lo], coarse[m >> bits]);
  }
};

// ---------------------------------------------------------------------------
// Launch geometry
// ---------------------------------------------------------------------------
template <typename T> constexpr int elems_per_thread() { return sizeof(T) == 4 ? 16 : 8; }

template <typename T, int L>
struct RowGeom {
  static constexpr int E0 = L < elems_per_thread<T>() ? L : elems_per_thread<T>();
  static constexpr int E = L / E0 > 1024 ? L / 1024 : E0;   // at most 1024 threads per transform
  static constexpr int TPR = L / E;
  static constexpr int G = TPR >= 256 ? 1 : 256 / TPR;   // transforms per workgroup
  static constexpr int NT = G * TPR;
};

// Envelope rows of the row kernels. WIDE: twice the values per thread (two
// groups of butterflies, exchanges in two rounds over half a region), so the
// 128 registers and the LDS of a CU hold twice the rows and more of them load,
// store or transform at any time. It takes enough rows to fill the chip twice
// over: with fewer, the one-group form has twice the waves per row. The
// butterflies are the same in both, and row_stats adds up in one order, so are
// all results, bit for bit.
// Measured (MI355X, forward / inverse rows, us, one group : two groups; few rows
// with products of twiddles in every pass):
//   FP32 N_out  4096, 65536 rows 501/573 : 477/561;   2048 rows 21/24 : 22/24
//   FP32 N_out  8192, 16384 rows 332/373 : 284/320;    512 rows 16/19 : 17/18
//   FP32 N_out 16384,  8192 rows 388/438 : 314/356;    256 rows 20/20 : 21/21
//   FP64 N_out  4096, 16384 rows 281/315 : 234/279;    512 rows 15/15 : 16/16
//   FP64 N_out  8192,  8192 rows 385/412 : 323/361;    256 rows 20/18 : 20/20
// (At its 128 registers k_inv_rows<double, 4096>, k_fwd_rows<float, 2048> and the
// FP32 dense rows spill 8 to 24 bytes a lane in this form, and gain all the same.)
template <typename T, int L> constexpr bool wide_rows() {
  return sizeof(T) == 4 ? L >= 2048 && L <= 16384 : L >= 1024 && L <= 8192;
}
// Envelope bytes of a launch from which rows take the two-group form: 64 MB
// where one group leaves at most two rows per CU (rows of 64 KB and more), 256
// MB where it leaves four (both forms within 3% of each other in between).
constexpr int64_t wide_from_bytes(int64_t row_bytes) {
  return row_bytes >= 65536 ? int64_t(64) << 20 : int64_t(256) << 20;
}
template <typename T, int L, bool WIDE = false>
struct RowsGeom {
  static constexpr int E = WIDE ? 2 * elems_per_thread<T>() : RowGeom<T, L>::E;
  static constexpr int RM = WIDE ? elems_per_thread<T>() : (E < 16 ? E : 16);
  static constexpr int TPR = L / E;
  static constexpr int G = TPR >= 256 ? 1 : 256 / TPR;
  static constexpr int NT = G * TPR;
  static constexpr int LDS = WIDE ? lds_size(L / 2) : fft_lds_elems<T, L>();
  template <int S, int TW = TW_MIXED> using Fft = BlockFft<T, L, E, S, TW, RM, WIDE>;
};

// Columns per workgroup of the four-step passes: C * L values fill at most
// 64 KiB of LDS, at least 4 columns for 32/64-byte contiguous runs.
// EP > 0 sets the values per thread (the second four-step pass of the
// spectrum and synthesis transforms runs faster with 8 in FP32: twice the
// waves per workgroup for its LDS-staged rows).
template <typename T, int L, int EP = 0, int CW = 0>
struct ColGeom {
  static constexpr int E0 = EP > 0 ? EP : elems_per_thread<T>();
  static constexpr int E = L < E0 ? L : E0;
  static constexpr int TPR = L / E;
  static constexpr int CAP = (65536 / (2 * int(sizeof(T)))) / L;
  // CW > 0 asks for CW columns where their LDS (with its padding) fits in
  // 144 KiB and CW * TPR threads make one workgroup
  static constexpr bool WIDE = CW > 0 && CW * (L + L / 32) * 2 * int(sizeof(T)) <= 147456 && CW * TPR <= 1024;
  static constexpr int CC = WIDE ? CW : (CAP >= 16 ? 16 : (CAP >= 4 ? CAP : 4));
  static constexpr int NT = CC * TPR;
};

// Workgroups go round-robin over the 8 XCDs, each with its own L2. Where R
// sibling workgroups share cache lines (decimated reads, interleaved writes),
// workgroup b of units * R takes sibling s of unit v such that the siblings
// of a unit are a multiple of 8 apart: one XCD, at nearly the same time, so
// its L2 joins their parts of a line.
template <int R>
__device__ __forceinline__ void sibling_block(int64_t b, int64_t units, int64_t& v, int& s) {
  const int64_t v0 = b / (8 * R) * 8, m = units - v0 < 8 ? units - v0 : 8, k = b - v0 * R;
  v = v0 + k % m;
  s = static_cast<int>(k / m);
}

}  // namespace qtam
