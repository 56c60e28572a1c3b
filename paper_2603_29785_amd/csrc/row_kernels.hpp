// Row kernels: the fused forward rows (gather x window, baseband placement,
// N_out-point inverse FFT; Sec. III, App. A and C demodulation) and the
// inverse rows (N_out-point FFT, kept slots x dual weights; Sec. III inverse,
// App. C re-modulation), their chirp-z forms for N_out that are not powers of
// two, their four-step forms for rows longer than one workgroup, and the
// dense-tile and single-tile kernels.
#pragma once

#include "device_common.hpp"
#include "mask_kernels.hpp"

namespace qtam {

// Dense tiles: row k of segment s is the N-point inverse transform of its
// packed kept entries at their bins lo..hi (zeros elsewhere), N = R * Md.
// Decimated by R: T[n1 + R n2] = IDFT_Md(A_n1)[n2], A_n1[k] = sum over the
// bins c = k mod Md of Z[c] e^{+2 pi i n1 c / N} (one bin, or a few where the
// support is wider than Md). The values k = index(i), i < E, of sibling n1 of
// a row, straight from its packed entries: r a resource over the len of them
// (the entry of bin c at c - lo; beyond it reads 0), the same for the wave.
template <typename T, int E, typename Index>
__device__ __forceinline__ void dense_values(typename Complex<T>::type (&v)[E], Index&& index, rsrc_t r, int64_t md,
                                             int n1, int lo, int len, int64_t n,
                                             const Twiddle2<typename Complex<T>::type>& tw2) {
  using C = typename Complex<T>::type;
  const unsigned nn = static_cast<unsigned>(n);
  auto root = [&](unsigned d) {   // e^{+2 pi i n1 (lo + d) / N}; n1 (lo + d) < 4 N
    unsigned m = static_cast<unsigned>(n1) * (static_cast<unsigned>(lo) + d);
    if (m >= 2 * nn) m -= 2 * nn;
    if (m >= nn) m -= nn;
    return c_conj(tw2(m));
  };
#pragma unroll
  for (int i = 0; i < E; ++i)
    v[i] = bload<C>(r, (static_cast<unsigned>(index(i) - lo) & static_cast<unsigned>(md - 1)) * sizeof(C));
  if (n1 > 0) {
#pragma unroll
    for (int i = 0; i < E; ++i)
      v[i] = c_mul(v[i], root(static_cast<unsigned>(index(i) - lo) & static_cast<unsigned>(md - 1)));
  }
  for (int more = static_cast<int>(md); more < len; more += static_cast<int>(md)) {   // supports wider than Md
#pragma unroll
    for (int i = 0; i < E; ++i) {
      const unsigned d = (static_cast<unsigned>(index(i) - lo) & static_cast<unsigned>(md - 1)) + more;
      if (d < static_cast<unsigned>(len)) {
        const C z = bload<C>(r, d * static_cast<unsigned>(sizeof(C)));
        v[i] = c_add(v[i], n1 > 0 ? c_mul(z, root(d)) : z);
      }
    }
  }
}

// Md in one workgroup: packed entries to the finished tile, one launch. The R
// siblings of a row write its interleaved values from one XCD. Bound by the
// write of the tiles. Measured on MI355X, FP32, 16 x 24576 samples, 62 rows
// (R = 3, 195 MB of tiles), forward + dense: 306 us with placing, radix pass,
// transforms and permutation as passes of their own, 123 us with this kernel;
// 16 x 16384 samples (R = 1) 126 to 78 us, and to 68 us in the two-group form
// (wide_from_bytes); with R = 3 that form has more rows between the parts of a
// line and is slower (162 us), so siblings keep one group.
template <typename T, int L, int R, bool WIDE = false>
__global__ __launch_bounds__((RowsGeom<T, L, WIDE>::NT), (WIDE ? 4 : 1)) void k_dense_rows(
    const typename Complex<T>::type* __restrict__ Sbuf, typename Complex<T>::type* __restrict__ D,
    const RowMeta* __restrict__ rows, int nrows, int64_t count, int64_t sum_len,
    const typename Complex<T>::type* __restrict__ tw, Twiddle2<typename Complex<T>::type> tw2) {
  using C = typename Complex<T>::type;
  using Geo = RowsGeom<T, L, WIDE>;
  using F = typename Geo::template Fft<+1, TW_POW>;
  __shared__ C lds[Geo::G * Geo::LDS];
  const int t = threadIdx.x, g = t / Geo::TPR, tl = t % Geo::TPR;
  int64_t u = blockIdx.x;
  int n1 = 0;
  if constexpr (R > 1) sibling_block<R>(blockIdx.x, gridDim.x / R, u, n1);
  int gr = static_cast<int>(u) * Geo::G + g;
  if constexpr (Geo::TPR >= 64) gr = __builtin_amdgcn_readfirstlane(gr);
  const bool ok = gr < count;
  const int seg = ok ? gr / nrows : 0;
  const RowMeta rm = rows[ok ? gr - seg * nrows : 0];
  const int len = ok ? rm.hi - rm.lo + 1 : 0;
  const C* src = Sbuf + int64_t(seg) * sum_len + rm.off;
  C v[Geo::E];
  if constexpr (Geo::TPR >= 64) {
    dense_values<T>(v, [&](int i) { return tl + F::in_off(i); }, make_rsrc(src, static_cast<uint32_t>(len * sizeof(C))),
                    L, n1, rm.lo, len, int64_t(R) * L, tw2);
  } else {   // several rows per wave
#pragma unroll
    for (int i = 0; i < Geo::E; ++i) {
      v[i] = C{0, 0};
      for (int d = (tl + F::in_off(i) - rm.lo) & (L - 1); d < len; d += L) {
        const C z = src[d];
        v[i] = c_add(v[i], n1 > 0 ? c_mul(z, c_conj(tw2(n1 * (rm.lo + d) % (R * L)))) : z);
      }
    }
  }
  F::run(v, lds + g * Geo::LDS, tl, F::twiddles(tw));
  if (!ok) return;
  C* dst = D + int64_t(gr) * (R * L) + n1 + R * tl;
#pragma unroll
  for (int i = 0; i < Geo::E; ++i) dst[R * F::out_off(i)] = v[i];
}

// Md = L1 * L2 in two passes: this column pass (as k_fft_cols over the values
// above, into the workspace), then k_fft_rows_t, which writes the interleaved
// tile. blockIdx.y = row * R + n1. Measured, 64 rows, FP32, forward + dense:
// 4 x 131072 samples (R = 1) 396 to 300 us, 4 x 98304 (R = 3) 433 to 255 us.
// (4096-point columns of R = 3, 5, from 2^24-point rows on, spill 248 bytes a
// lane; two rows of 3 2^24 samples 3.6 to 2.2 ms.)
template <typename T, int L2, int R>
__global__ __launch_bounds__((ColGeom<T, L2>::NT)) void k_dense_cols(
    const typename Complex<T>::type* __restrict__ Sbuf, typename Complex<T>::type* __restrict__ A,
    const RowMeta* __restrict__ rows, int nrows, int64_t sum_len, int64_t md, int64_t l1,
    const typename Complex<T>::type* __restrict__ tw, Twiddle2<typename Complex<T>::type> tw2) {
  using C = typename Complex<T>::type;
  using Geo = ColGeom<T, L2>;
  using F = BlockFft<T, L2, Geo::E, +1>;
  __shared__ C lds[Geo::CC * lds_size(L2)];
  const int t = threadIdx.x, cc = t % Geo::CC, tl = t / Geo::CC;
  const int64_t c1 = int64_t(blockIdx.x) * Geo::CC + cc;
  const int64_t gr = blockIdx.y / R;
  const int n1 = blockIdx.y % R;
  const int64_t seg = gr / nrows;
  const RowMeta rm = rows[gr - seg * nrows];
  const int len = rm.hi - rm.lo + 1;
  C v[Geo::E];
  dense_values<T>(v, [&](int i) { return static_cast<int>(c1 + l1 * F::in_index(tl, i)); },
                  make_rsrc(Sbuf + seg * sum_len + rm.off, static_cast<uint32_t>(len * sizeof(C))), md, n1, rm.lo, len,
                  R * md, tw2);
  F::run(v, lds + cc * lds_size(L2), tl, F::twiddles(tw));
  C* dst = A + int64_t(blockIdx.y) * md + c1;
#pragma unroll
  for (int i = 0; i < Geo::E; ++i) {
    const int64_t k2 = F::out_index(tl, i);
    dst[l1 * k2] = c_mul(v[i], c_conj(tw2(R * c1 * k2)));   // exp(+2 pi i c1 k2 / Md)
  }
}

// Single-tile recovery: row `row` of each segment, its N_out-point forward
// transform, every slot that holds a kept bin c (slot_entry) times the tile
// table (sqrt(N/N_out) / W / N) into Sx[seg][c]. One segment per row group.
template <typename T, int L>
__global__ __launch_bounds__((RowGeom<T, L>::NT)) void k_tile_rows(
    const typename Complex<T>::type* __restrict__ Y, typename Complex<T>::type* __restrict__ Sx,
    const RowMeta* __restrict__ rows, const T* __restrict__ tab, int R, int row, int segs, int half,
    const typename Complex<T>::type* __restrict__ tw) {
  using C = typename Complex<T>::type;
  using Geo = RowGeom<T, L>;
  using F = BlockFft<T, L, Geo::E, -1, TW_MIXED>;
  __shared__ C lds[Geo::G * fft_lds_elems<T, L>()];
  const int t = threadIdx.x, g = t / Geo::TPR, tl = t % Geo::TPR;
  const int seg = static_cast<int>(blockIdx.x) * Geo::G + g;
  const bool ok = seg < segs;
  const rsrc_t ry = make_rsrc(Y + (int64_t(ok ? seg : 0) * R + row) * L, ok ? static_cast<uint32_t>(L * sizeof(C)) : 0u);
  C v[Geo::E];
#pragma unroll
  for (int i = 0; i < Geo::E; ++i) v[i] = bload<C>(ry, static_cast<uint32_t>(tl + F::in_off(i)) * sizeof(C));
  F::run(v, lds + g * fft_lds_elems<T, L>(), tl, F::twiddles(tw));
  if (!ok) return;
  const RowMeta rm = rows[row];
  C* dst = Sx + int64_t(seg) * (half + 1);
#pragma unroll
  for (int i = 0; i < Geo::E; ++i) {
    const int d = slot_entry<L>(tl + F::out_off(i), rm);
    if (d <= rm.hi - rm.lo) {
      const T w = tab[rm.off + d];
      dst[rm.lo + d] = C{v[i].x * w, v[i].y * w};
    }
  }
}

// Workgroups are dispatched round-robin over the 8 XCDs (workgroup i runs on
// XCD i mod 8) and roughly in index order. Renumbering them so that XCD x
// takes the x-th eighth of the units makes the workgroups resident on one XCD
// at a time work on neighbouring rows, whose spectrum that XCD's L2 holds.
__device__ __forceinline__ int xcd_major_block(int nblocks) {
  const int b = blockIdx.x;
  if (nblocks & 7) return b;
  return (b & 7) * (nblocks >> 3) + (b >> 3);
}

// Fused forward rows: the windowed spectrum bins of a row are dropped at
// their baseband slots (c - s_k) mod N_out (roll to baseband, crop, zero pad),
// the N_out-point inverse FFT runs in registers and LDS, and the envelope row
// is stored. One unit of G consecutive rows per workgroup.
// Cache policy of the envelope stores: Y is written once and not read again
// by the forward, so streaming it past the L2 keeps the spectrum and the plan
// tables, which every row re-reads, resident there (measured: the forward
// rows kernel of the batched workload drops from 0.70 to 0.50 ms). Loads of
// Y by the inverse keep the default policy (streaming them measured no gain
// and slowed the overlap-add that follows).
constexpr int kYStore = kCacheNT;
constexpr int kYLoad = kCacheDefault;
// The packed kept slots are read once, by the overlap-add after the whole
// inverse-rows launch: streamed as well (measured 1-3% on both kernels).
constexpr int kSStore = kCacheNT;

// Hides a value's derivation from the optimiser (an empty asm that keeps it
// in a VGPR), so per-element offsets stay one add from a precomputed base
// instead of being refolded into an add and a shift per resource.
__device__ __forceinline__ void opaque(unsigned& v) { asm volatile("" : "+v"(v)); }
__device__ __forceinline__ int opaque_copy(int v) {
  asm volatile("" : "+v"(v));
  return v;
}

// Row statistics (sum and max of |Y|^2 over the row) of the E values each of
// a row's TPR threads holds. Lanes of one row inside a wave combine by an xor
// butterfly (every lane ends with the same bits); rows spanning several waves
// then add the per-wave results in wave order through `part` (LDS the
// transform no longer reads, H * NT / 64 elements). Every thread of the block
// must call it.
// H = 2: two-group rows. Registers come in runs of RL values (last radix), run
// q at tl + q TPR, and a thread of the one-group form holds every second run:
// those of parity h belong to its thread tl + h TPR. The sums are kept apart
// by parity and combined in the waves and the wave order of the one-group
// form, so a row's statistics have the same bits in both.
template <typename T, int E, int TPR, int NT, int H, int RL>
__device__ __forceinline__ void row_stats(const typename Complex<T>::type (&v)[E], int tl, bool ok,
                                          typename Complex<T>::type* __restrict__ dst,
                                          typename Complex<T>::type* __restrict__ part) {
  using C = typename Complex<T>::type;
  static_assert(H == 1 || (TPR >= 64 && E % (2 * RL) == 0), "whole waves and runs in pairs");
  constexpr int W = TPR < 64 ? TPR : 64;     // lanes of a row within one wave
  constexpr int WPR = TPR > 64 ? TPR / 64 : 1;
  T e[H] = {}, m[H] = {};
#pragma unroll
  for (int i = 0; i < E; ++i) {
    const int h = (i / RL) % H;
    const T a = v[i].x * v[i].x + v[i].y * v[i].y;
    e[h] += a;
    m[h] = fmax(m[h], a);
  }
#pragma unroll
  for (int h = 0; h < H; ++h) {
#pragma unroll
    for (int o = 1; o < W; o <<= 1) {
      e[h] += __shfl_xor(e[h], o, W);
      m[h] = fmax(m[h], __shfl_xor(m[h], o, W));
    }
  }
  if constexpr (WPR == 1) {
    if (ok && tl == 0) *dst = H == 1 ? C{e[0], m[0]} : C{e[0] + e[H - 1], fmax(m[0], m[H - 1])};
  } else {
    const int wave = threadIdx.x >> 6, w = tl >> 6;
    if ((threadIdx.x & 63) == 0) {
#pragma unroll
      for (int h = 0; h < H; ++h) part[H * (wave - w) + h * WPR + w] = C{e[h], m[h]};
    }
    __syncthreads();
    if (ok && tl == 0) {
      const C* pr = part + H * wave;
      C r = pr[0];
#pragma unroll
      for (int i = 1; i < H * WPR; ++i) {
        r.x += pr[i].x;
        r.y = fmax(r.y, pr[i].y);
      }
      *dst = r;
    }
  }
}

// Sum of one value per thread over each row of the block, in a fixed order:
// an xor butterfly over a row's lanes within a wave, then (rows spanning
// several waves) the per-wave sums in wave order through `part` (LDS the
// transform no longer reads, NT/64 elements). Every thread of the block must
// call it.
template <typename T, int TPR, int NT>
__device__ __forceinline__ void row_sum(T s, int tl, bool ok, T* __restrict__ dst, T* __restrict__ part) {
  constexpr int W = TPR < 64 ? TPR : 64;
  constexpr int WPR = TPR > 64 ? TPR / 64 : 1;
#pragma unroll
  for (int o = 1; o < W; o <<= 1) s += __shfl_xor(s, o, W);
  if constexpr (WPR == 1) {
    if (ok && tl == 0) *dst = s;
  } else {
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = s;
    __syncthreads();
    if (ok && tl == 0) {
      const T* pr = part + (threadIdx.x >> 6);
      T r = pr[0];
#pragma unroll
      for (int w = 1; w < WPR; ++w) r += pr[w];
      *dst = r;
    }
  }
}

// When a wave holds one row (TPR >= 64) and the row touches neither DC nor
// Nyquist, buffer resources scoped to the row's kept support do the cropping:
// slots outside it fall outside the resources and read 0, with no test.
// Otherwise each slot is tested; ANALYTIC then computes the bisquare weight
// scale_k (1 - (j/h_k)^2)^2 instead of reading the table.
// MBWD (the inverse adjoint of a masked inverse): the transform's output is
// the gradient G with respect to the masked envelope Y' = g_k m Y; the kernel
// reads Y (mY, same layout as the output) and stores dL/dY instead, and the
// row's sum of m Re(conj(Y) G) goes to mpart[row] (the gain gradient's share).
template <typename T, int L, bool ANALYTIC, bool STATS, bool MBWD = false, bool WIDE = false>
__global__ __launch_bounds__((RowsGeom<T, L, WIDE>::NT), (WIDE ? 4 : 1)) void k_fwd_rows(
    const typename Complex<T>::type* __restrict__ spec, typename Complex<T>::type* __restrict__ Y,
    const RowMeta* __restrict__ rows, const typename Complex<T>::type* __restrict__ roww,
    const T* __restrict__ tab, int R, int total, int half, int sum_len, int64_t spec_elems,
    const typename Complex<T>::type* __restrict__ tw, int nblocks, typename Complex<T>::type* __restrict__ stats,
    const typename Complex<T>::type* __restrict__ mY, const T* __restrict__ mgain, const T* __restrict__ mlam,
    T* __restrict__ mpart) {
  using C = typename Complex<T>::type;
  using Geo = RowsGeom<T, L, WIDE>;
  using F = typename Geo::template Fft<+1>;
  constexpr bool kWaveRow = Geo::TPR >= 64;   // every lane of a wave is on the same row
  __shared__ C lds[Geo::G * Geo::LDS];
  const int t = threadIdx.x, g = t / Geo::TPR, tl = t % Geo::TPR;
  const int u = xcd_major_block(nblocks);
  int gr = u * Geo::G + g;
  if constexpr (kWaveRow) gr = __builtin_amdgcn_readfirstlane(gr);
  const bool ok = gr < total;
  const int seg = ok ? gr / R : 0;
  const int row = ok ? gr - seg * R : 0;
  const RowMeta rm = rows[row];
  const bool centred = row_centred(rm, L);
  C v[Geo::E];
  if (kWaveRow && rm.lo > 0 && rm.hi < half && centred) {
    const int len = rm.hi - rm.lo + 1;
    const rsrc_t rz = make_rsrc(spec + int64_t(seg) * half + rm.lo, ok ? static_cast<uint32_t>(len * sizeof(C)) : 0u);
    const rsrc_t rt = make_rsrc(tab + rm.off, ok ? static_cast<uint32_t>(len * sizeof(T)) : 0u);
    const int db = rm.s - rm.lo + tl;   // kept-bin index d = c - lo of the slot with offset 0
    // byte offsets of d in both resources, advanced by constants (negative d
    // wraps beyond the resource and reads 0)
    unsigned bx = static_cast<unsigned>(db) * static_cast<unsigned>(sizeof(C));
    unsigned bw = static_cast<unsigned>(db) * static_cast<unsigned>(sizeof(T));
    opaque(bx);
    opaque(bw);
#pragma unroll
    for (int i = 0; i < Geo::E; ++i) {
      const int off = F::in_off(i);
      const unsigned j = static_cast<unsigned>(off < L / 2 ? off : off - L);
      const C x = bload<C>(rz, bx + j * static_cast<unsigned>(sizeof(C)));
      const T w = bload<T>(rt, bw + j * static_cast<unsigned>(sizeof(T)));
      v[i] = C{x.x * w, x.y * w};
    }
  } else {
    const rsrc_t rz = make_rsrc(spec, static_cast<uint32_t>(spec_elems * sizeof(C)));
    const rsrc_t rt = make_rsrc(tab, static_cast<uint32_t>(sum_len * sizeof(T)));

    const unsigned zb = static_cast<unsigned>(seg) * static_cast<unsigned>(half);
    const int last = rm.hi - rm.lo;
    // X[c] of the slots holding a kept bin c = lo + d; other slots get an
    // offset beyond the buffer and read 0 without touching memory
#pragma unroll
    for (int i = 0; i < Geo::E; ++i) {
      const int d = slot_entry<L>(tl + F::in_off(i), rm);
      const int c = rm.lo + d;
      const bool in = ok && d <= last;
      const unsigned vo = in ? (zb + static_cast<unsigned>(c == half ? 0 : c)) * static_cast<unsigned>(sizeof(C))
                             : 0xFFFFFFFFu;
      v[i] = bload<C>(rz, vo);
    }
    C sw{0, 0};
    if constexpr (ANALYTIC) sw = roww[row];   // (scale_k, 1/h_k)
#pragma unroll
    for (int i = 0; i < Geo::E; ++i) {
      const int d = slot_entry<L>(tl + F::in_off(i), rm);
      const int c = rm.lo + d;
      const int j = c - rm.s;
      C val = v[i];
      if (c == 0) val.y = 0;               // slot 0 of the spectrum holds (X[0], X[N/2])
      if (c == half) val = C{val.y, 0};
      T w;
      if constexpr (ANALYTIC) {
        const T x = static_cast<T>(j) * sw.y;
        const T b = (T(1) - x) * (T(1) + x);
        w = sw.x * b * b;
      } else {
        const bool in = ok && d <= last;
        w = bload<T>(rt, static_cast<uint32_t>(in ? rm.off + d : 0) * sizeof(T));
      }
      v[i] = C{val.x * w, val.y * w};
    }
  }
  // Inputs of a centred row outside its kept offsets [jlo, jhi] are zero; when every
  // lane of this wave has zeros in first-pass inputs 1..14 (or 2..13) the
  // first pass skips them (same results, fewer operations).
  int nz = 0;
  if constexpr (kWaveRow && F::R0 == 16) {
    const int jlo = rm.lo - rm.s, jhi = rm.hi - rm.s;
    const int t0 = __builtin_amdgcn_readfirstlane(tl) & ~63;
    // input r of group q of lane tl sits at slot tl + q TPR + r Q
    constexpr int Q = L / 16, TOP = 63 + (Geo::E / 16 - 1) * Geo::TPR;
    auto zero = [&](int a, int b) { return t0 + a * Q > jhi && t0 + TOP + b * Q < L + jlo; };
    nz = !centred ? 0 : (zero(1, 14) ? 2 : (zero(2, 13) ? 4 : 0));
  }
  F::run(v, lds + g * Geo::LDS, tl, F::twiddles(tw), nz);
  const int64_t r0 = int64_t(u) * Geo::G;
  const int64_t nrow = total - r0 < Geo::G ? total - r0 : Geo::G;
  const rsrc_t ry = make_rsrc(Y + r0 * L, static_cast<uint32_t>(nrow * L * sizeof(C)));
  const uint32_t vb = static_cast<uint32_t>(g * L + tl) * sizeof(C);
  if constexpr (MBWD) {
    const rsrc_t rm = make_rsrc(mY + r0 * L, static_cast<uint32_t>(nrow * L * sizeof(C)));
    const T gk = ok ? mgain[row] : T(0), lk = ok ? mlam[row] : T(0);
    T acc = 0;
#pragma unroll
    for (int i = 0; i < Geo::E; ++i) {
      const C yv = bload<C>(rm, vb, F::out_off(i) * sizeof(C));
      v[i] = MaskMath<T>::grad(yv, v[i], gk, lk, acc);
    }
#pragma unroll
    for (int i = 0; i < Geo::E; ++i) bstore<C, kYStore>(ry, v[i], vb, F::out_off(i) * sizeof(C));
    row_sum<T, Geo::TPR, Geo::NT>(acc, tl, ok, mpart + gr, reinterpret_cast<T*>(lds));
  } else {
#pragma unroll
    for (int i = 0; i < Geo::E; ++i) bstore<C, kYStore>(ry, v[i], vb, F::out_off(i) * sizeof(C));
    if constexpr (STATS) row_stats<T, Geo::E, Geo::TPR, Geo::NT, WIDE ? 2 : 1, F::RL>(v, tl, ok, stats + gr, lds);
  }
}

// Inverse rows: N_out-point FFT of each envelope row; the kept slots times the
// table go to the packed per-segment buffer Sbuf[seg * sum_len + off + c - lo].
// With one row per wave, resources scoped to the row's packed entries drop
// the other slots' stores without a test.
// MASK (a masked inverse): each loaded value y becomes g_k max(0, 1 -
// lambda_k / |y|) y (the mask of the denoiser) before the transform.
template <typename T, int L, bool MASK = false, bool WIDE = false>
__global__ __launch_bounds__((RowsGeom<T, L, WIDE>::NT), (WIDE ? 4 : 1)) void k_inv_rows(
    const typename Complex<T>::type* __restrict__ Y, typename Complex<T>::type* __restrict__ Sbuf,
    const RowMeta* __restrict__ rows, const T* __restrict__ tab, int R, int total, int sum_len, int segs,
    const typename Complex<T>::type* __restrict__ tw, const T* __restrict__ mgain, const T* __restrict__ mlam) {
  using C = typename Complex<T>::type;
  using Geo = RowsGeom<T, L, WIDE>;
  using F = typename Geo::template Fft<-1>;
  constexpr bool kWaveRow = Geo::TPR >= 64;
  __shared__ C lds[Geo::G * Geo::LDS];
  const int t = threadIdx.x, g = t / Geo::TPR, tl = t % Geo::TPR;
  const int64_t r0 = int64_t(blockIdx.x) * Geo::G;
  const int64_t nrow = total - r0 < Geo::G ? total - r0 : Geo::G;
  const rsrc_t ry = make_rsrc(Y + r0 * L, static_cast<uint32_t>(nrow * L * sizeof(C)));
  const uint32_t vb = static_cast<uint32_t>(g * L + tl) * sizeof(C);
  C v[Geo::E];
#pragma unroll
  for (int i = 0; i < Geo::E; ++i) v[i] = bload<C, kYLoad>(ry, vb, F::in_off(i) * sizeof(C));
  if constexpr (MASK) {
    int gm = static_cast<int>(r0) + g;
    if constexpr (kWaveRow) gm = __builtin_amdgcn_readfirstlane(gm);
    const int km = gm < total ? gm % R : 0;
    const T gk = mgain[km], lk = mlam[km];
#pragma unroll
    for (int i = 0; i < Geo::E; ++i) v[i] = MaskMath<T>::apply(v[i], gk, lk);
  }
  if constexpr (kWaveRow) {
    // the row's weights are requested before the transform, so their latency
    // hides behind it; rows past the end get empty resources
    const int gr = __builtin_amdgcn_readfirstlane(static_cast<int>(r0) + g);
    const bool ok = gr < total;
    const int seg = ok ? gr / R : 0;
    const RowMeta rm = rows[ok ? gr - seg * R : 0];
    const int len = ok ? rm.hi - rm.lo + 1 : 0;
    const int db = rm.s - rm.lo + tl;   // d = c - lo for the slot u = tl + off
    const rsrc_t rs = make_rsrc(Sbuf + int64_t(seg) * sum_len + rm.off, static_cast<uint32_t>(len * sizeof(C)));
    const rsrc_t rt = make_rsrc(tab + rm.off, static_cast<uint32_t>(len * sizeof(T)));
    const bool centred = row_centred(rm, L);
    unsigned bs = static_cast<unsigned>(db) * static_cast<unsigned>(sizeof(C));
    unsigned bw = static_cast<unsigned>(db) * static_cast<unsigned>(sizeof(T));
    opaque(bs);
    opaque(bw);
    // (rows of two groups per thread load them after the transform: registers)
    constexpr bool kEarly = !WIDE && Geo::E <= 16;
    T w[kEarly ? Geo::E : 1];
    if constexpr (kEarly) {
#pragma unroll
      for (int i = 0; i < Geo::E; ++i) {
        const int off = F::out_off(i);
        const unsigned j = static_cast<unsigned>(off < L / 2 ? off : off - L);
        w[i] = bload<T>(rt, bw + j * static_cast<unsigned>(sizeof(T)));
      }
    }
    F::run(v, lds + g * Geo::LDS, tl, F::twiddles(tw));
    if (!centred) {
      // a row of a regularised window: slot entries taken modulo L (the
      // early weights above are not used)
#pragma unroll
      for (int i = 0; i < Geo::E; ++i) {
        const unsigned d = static_cast<unsigned>(slot_entry<L>(tl + F::out_off(i), rm));
        const T wi = bload<T>(rt, d * static_cast<unsigned>(sizeof(T)));
        bstore<C, kSStore>(rs, C{v[i].x * wi, v[i].y * wi}, d * static_cast<unsigned>(sizeof(C)));
      }
      return;
    }
#pragma unroll
    for (int i = 0; i < Geo::E; ++i) {
      const int off = F::out_off(i);
      const unsigned j = static_cast<unsigned>(off < L / 2 ? off : off - L);
      T wi;
      if constexpr (kEarly) wi = w[i];
      else wi = bload<T>(rt, bw + j * static_cast<unsigned>(sizeof(T)));
      bstore<C, kSStore>(rs, C{v[i].x * wi, v[i].y * wi}, bs + j * static_cast<unsigned>(sizeof(C)));
    }
  } else {
    F::run(v, lds + g * Geo::LDS, tl, F::twiddles(tw));
    const int gr = static_cast<int>(r0) + g;
    if (gr >= total) return;
    const int seg = gr / R;
    const RowMeta rm = rows[gr - seg * R];
    const int len = rm.hi - rm.lo + 1;
    const rsrc_t rs = make_rsrc(Sbuf, static_cast<uint32_t>(int64_t(segs) * sum_len * sizeof(C)));
    const rsrc_t rt = make_rsrc(tab, static_cast<uint32_t>(sum_len * sizeof(T)));
    const unsigned sb = static_cast<unsigned>(seg) * static_cast<unsigned>(sum_len) + static_cast<unsigned>(rm.off);
#pragma unroll
    for (int i = 0; i < Geo::E; ++i) {
      const int d = slot_entry<L>(tl + F::out_off(i), rm);
      if (d < len) {
        const T w = bload<T>(rt, (rm.off + d) * sizeof(T));
        bstore<C, kSStore>(rs, C{v[i].x * w, v[i].y * w}, (sb + d) * sizeof(C));
      }
    }
  }
}

// Envelope lengths M = N_out that are not powers of two (the paper's minimal
// N_out, say): each row's length-M DFT by Bluestein's chirp-z identity,
//   sum_u g[u] e^{S 2 pi i u m / M} = a[m] sum_u (g[u] a[u]) b[m - u],
//   a[v] = e^{S pi i v^2 / M}, b[v] = conj(a[v]),
// the convolution as a cyclic one of power-of-two length L >= 2M - 1: a
// forward FFT, a product with Bhat = FFT_L(b wrapped) / L, an inverse FFT.
// Tables (FP64-built): chirp a[0..M) and Bhat[0..L) of the transform's sign.
template <typename T, int L, typename C, int E>
__device__ __forceinline__ void chirp_convolve(C (&v)[E], C* lds, int tl, const C* __restrict__ bhat,
                                               const C* __restrict__ tw) {
  using Geo = RowGeom<T, L>;
  static_assert(Geo::E == E, "row geometry");
  using F = BlockFft<T, L, Geo::E, -1>;
  using Fi = BlockFft<T, L, Geo::E, +1>;
  F::run(v, lds, tl, F::twiddles(tw));
#pragma unroll
  for (int i = 0; i < Geo::E; ++i) v[i] = c_mul(v[i], bhat[tl + F::out_off(i)]);
  // back to the input order of the second transform
#pragma unroll
  for (int i = 0; i < Geo::E; ++i) lds[lds_pad(tl + F::out_off(i))] = v[i];
  __syncthreads();
#pragma unroll
  for (int i = 0; i < Geo::E; ++i) v[i] = lds[lds_pad(tl + Fi::in_off(i))];
  __syncthreads();
  Fi::run(v, lds, tl, Fi::twiddles(tw));
}

// Forward rows, M not a power of two: gather the kept bins of each row at
// their slots (c - s) mod M times the forward table and the chirp, then
// Bluestein (sign +) and the output chirp; outputs m < M are stored.
template <typename T, int L>
__global__ __launch_bounds__((RowGeom<T, L>::NT)) void k_fwd_rows_bs(
    const typename Complex<T>::type* __restrict__ spec, typename Complex<T>::type* __restrict__ Y,
    const RowMeta* __restrict__ rows, const T* __restrict__ tab, int R, int total, int half, int sum_len,
    int64_t spec_elems, int M, const typename Complex<T>::type* __restrict__ chirp,
    const typename Complex<T>::type* __restrict__ bhat, const typename Complex<T>::type* __restrict__ tw) {
  using C = typename Complex<T>::type;
  using Geo = RowGeom<T, L>;
  using F = BlockFft<T, L, Geo::E, -1>;
  using Fi = BlockFft<T, L, Geo::E, +1>;
  __shared__ C lds[Geo::G * lds_size(L)];
  const int t = threadIdx.x, g = t / Geo::TPR, tl = t % Geo::TPR;
  const int gr = static_cast<int>(blockIdx.x) * Geo::G + g;
  const bool ok = gr < total;
  const int seg = ok ? gr / R : 0;
  const RowMeta rm = rows[ok ? gr - seg * R : 0];
  const rsrc_t rz = make_rsrc(spec, static_cast<uint32_t>(spec_elems * sizeof(C)));
  const rsrc_t rt = make_rsrc(tab, static_cast<uint32_t>(sum_len * sizeof(T)));
  const unsigned zb = static_cast<unsigned>(seg) * static_cast<unsigned>(half);
  // slot u holds the kept bin c = lo + d, d = (u + s - lo) mod M, if d <= hi - lo
  int sh = (rm.s - rm.lo) % M;
  if (sh < 0) sh += M;
  C v[Geo::E];
#pragma unroll
  for (int i = 0; i < Geo::E; ++i) {
    const int u = tl + F::in_off(i);                 // Bluestein slot; < M holds data
    const int d = u + sh < M ? u + sh : u + sh - M;
    const int c = rm.lo + d;
    const bool in = ok && u < M && d <= rm.hi - rm.lo;
    const unsigned vo = in ? (zb + static_cast<unsigned>(c == half ? 0 : c)) * static_cast<unsigned>(sizeof(C))
                           : 0xFFFFFFFFu;
    C x = bload<C>(rz, vo);
    if (c == 0) x.y = 0;
    if (c == half) x = C{x.y, 0};
    const T w = bload<T>(rt, static_cast<uint32_t>(in ? rm.off + d : 0) * sizeof(T));
    const C a = chirp[u < M ? u : 0];   // x is 0 outside the support
    v[i] = c_mul(C{x.x * w, x.y * w}, a);
  }
  chirp_convolve<T, L>(v, lds + g * lds_size(L), tl, bhat, tw);
  if (!ok) return;
  C* yrow = Y + int64_t(gr) * M;
#pragma unroll
  for (int i = 0; i < Geo::E; ++i) {
    const int m = tl + Fi::out_off(i);
    if (m < M) yrow[m] = c_mul(v[i], chirp[m]);
  }
}

// Inverse rows, M not a power of two: Bluestein (sign -) over each envelope
// row, then the kept slots times the table into the packed buffer.
template <typename T, int L>
__global__ __launch_bounds__((RowGeom<T, L>::NT)) void k_inv_rows_bs(
    const typename Complex<T>::type* __restrict__ Y, typename Complex<T>::type* __restrict__ Sbuf,
    const RowMeta* __restrict__ rows, const T* __restrict__ tab, int R, int total, int sum_len, int M,
    const typename Complex<T>::type* __restrict__ chirp, const typename Complex<T>::type* __restrict__ bhat,
    const typename Complex<T>::type* __restrict__ tw) {
  using C = typename Complex<T>::type;
  using Geo = RowGeom<T, L>;
  using F = BlockFft<T, L, Geo::E, -1>;
  using Fi = BlockFft<T, L, Geo::E, +1>;
  __shared__ C lds[Geo::G * lds_size(L)];
  const int t = threadIdx.x, g = t / Geo::TPR, tl = t % Geo::TPR;
  const int gr = static_cast<int>(blockIdx.x) * Geo::G + g;
  const bool ok = gr < total;
  const C* yrow = Y + int64_t(ok ? gr : 0) * M;
  C v[Geo::E];
#pragma unroll
  for (int i = 0; i < Geo::E; ++i) {
    const int u = tl + F::in_off(i);
    const bool in = ok && u < M;
    const int uc = in ? u : 0;
    const C z = c_mul(yrow[uc], c_conj(chirp[uc]));
    v[i] = in ? z : C{0, 0};
  }
  chirp_convolve<T, L>(v, lds + g * lds_size(L), tl, bhat, tw);
  if (!ok) return;
  const int seg = gr / R;
  const RowMeta rm = rows[gr - seg * R];
  C* srow = Sbuf + int64_t(seg) * sum_len + rm.off;
  int sh = (rm.s - rm.lo) % M;   // slot u holds kept entry d = (u + s - lo) mod M
  if (sh < 0) sh += M;
#pragma unroll
  for (int i = 0; i < Geo::E; ++i) {
    const int u = tl + Fi::out_off(i);
    if (u >= M) continue;
    const int d = u + sh < M ? u + sh : u + sh - M;
    if (d > rm.hi - rm.lo) continue;
    const C z = c_mul(v[i], c_conj(chirp[u]));
    const T w = tab[rm.off + d];
    srow[d] = C{z.x * w, z.y * w};
  }
}

// Envelope lengths M = N_out that are not powers of two, plain windows: the
// same identity by overlap-save. Row k has inputs only at the offsets j in
// [jlo, jhi] = [lo - s, hi - s] of its support, so
//   Y[m] = a[m] sum_j (g[j] a[j]) conj(a[m - j])
// needs the chirp at lags m - j only. The outputs are taken in blocks: block i
// holds the lags V_i .. V_i + L - 1, V_i = -JP + i B (JP, JN the largest
// positive and negative offsets of any row, B = L - JP - JN), and one cyclic
// convolution of length L with them gives every m with V_i + jhi <= m <
// V_i + L + jlo, which is block i of this row up to where block i + 1 starts.
// The transform of the inputs is shared by a row's blocks: 1 + blocks
// transforms of length L per row, where one convolution over all outputs
// takes two of length >= 2 M - 1. A row of narrow support needs fewer blocks.
// The inverse is its transpose: the blocks' transforms times conj(Bhat_i) add
// up in registers, then one inverse transform. Bhat_i = FFT_L(conj a[V_i + t])
// / L, t = 0 .. L - 1, built in FP64. The transform's rounding spreads over all
// L outputs of a convolution whether a block stores them or not, so lags that
// no stored output needs are zero (they only add to outputs that are dropped),
// and Bhat takes out the mean gain of the two transforms (transform_gain).
// Errors against extended precision, 62 rows of 24576 samples, forward /
// inverse, M = 1028 .. 26591: FP32 2.2-2.5e-7 / 2.3-2.6e-7 (2.7-2.9e-7 /
// 2.8-3.1e-7 without the two, 2.5-3.1e-7 / 2.6-3.3e-7 by one convolution),
// FP64 5.5-6.6e-16 / 6.0-6.7e-16 (7.8-8.5e-16 / 7.9-8.5e-16 with angles rounded
// to double, 7.4-8.3e-16 / 9.0-11e-16 by one convolution).
// The output registers of a transform hold the same indices as the input
// registers of the next one in another order (both sets are the multiples of
// TPR), so no exchange stands between the two.
// What bounds it: vector ALU issue and the latency between its transforms
// (registers and LDS, packed FP32 off), as in the other row kernels; four
// waves per SIMD, so the table loads of a block's transforms are kept from
// being hoisted out of the block loop (they would take 64 registers and spill).
// Measured on MI355X, FP32, 62 rows of 24576-sample segments: forward + inverse
// of 128 segments with N_out = 12289 (support 1537) 11.45 ms by length-32768
// transforms through memory, 0.74 ms here (L = 4096, 4 or 5 blocks); forward of
// 1024 segments with N_out = 1028 (support 1027) 0.87 ms by one length-4096
// convolution per row, 0.47 ms here (L = 2048, one block for rows of at most
// 507 bins a side, else two). Rows whose convolution over all outputs is
// shorter than one per wave (1024 values FP32, 512 FP64) keep that form: here
// 8700 rows of 109 values, forward + inverse, took 69 us against 51.
struct OsPlan {
  int M, JP, B;          // N_out, largest positive offset, block step
  int nmax;              // blocks of the table Bhat
  const int* blocks;     // [R] blocks needed by the rows of a workgroup that starts at this row
};

// Input register of F2 that holds the index of output register i of F1.
template <typename F1, typename F2, int E>
constexpr int os_in_reg(int i) {
  for (int k = 0; k < E; ++k)
    if (F2::in_off(k) == F1::out_off(i)) return k;
  return -1;
}

// ONE: a workgroup per row and block (blockIdx.y), for few rows.
template <typename T, int L, bool ONE>
__global__ __launch_bounds__((RowGeom<T, L>::NT), (ONE ? 1 : 4)) void k_fwd_rows_os(
    const typename Complex<T>::type* __restrict__ spec, typename Complex<T>::type* __restrict__ Y,
    const RowMeta* __restrict__ rows, const typename Complex<T>::type* __restrict__ tab, int R, int total, int half, OsPlan os,
    const typename Complex<T>::type* __restrict__ chirp, const typename Complex<T>::type* __restrict__ bhat,
    const typename Complex<T>::type* __restrict__ tw, int nblocks) {
  using C = typename Complex<T>::type;
  using Geo = RowGeom<T, L>;
  using F = BlockFft<T, L, Geo::E, -1>;
  using Fi = BlockFft<T, L, Geo::E, +1>;
  static_assert(Geo::TPR >= 64, "a wave holds one row");
  __shared__ C lds[Geo::G * lds_size(L)];
  const int t = threadIdx.x, g = t / Geo::TPR, tl = t % Geo::TPR;
  C* reg = lds + g * lds_size(L);
  const int u = xcd_major_block(nblocks);
  int gr = u * Geo::G + g;
  gr = __builtin_amdgcn_readfirstlane(gr);
  const bool ok = gr < total;
  const int seg = ok ? gr / R : 0;
  const RowMeta rm = rows[ok ? gr - seg * R : 0];
  const int len = ok ? rm.hi - rm.lo + 1 : 0;
  const int jlo = rm.lo - rm.s, jhi = rm.hi - rm.s;
  const int nb = __builtin_amdgcn_readfirstlane(os.blocks[(u * Geo::G) % R]);
  if (static_cast<int>(blockIdx.y) >= nb) return;
  const rsrc_t rc = make_rsrc(chirp, static_cast<uint32_t>(os.M * sizeof(C)));
  C v[Geo::E];
  {
    // kept bins c = s + j at slot j mod L (j the signed slot), times the table
    // (window and chirp); slots outside the support read 0
    const C* Z = spec + int64_t(seg) * half;
    const C z0 = Z[0];   // (X[0], X[N/2])
    // (the entries below Nyquist; kept in a scalar register, else every load
    // of the gather becomes a loop over lanes that waits for it)
    const int zlen = __builtin_amdgcn_readfirstlane(ok && rm.hi == half ? len - 1 : len);
    const rsrc_t rz = make_rsrc(Z + rm.lo, static_cast<uint32_t>(zlen * sizeof(C)));
    const rsrc_t rt = make_rsrc(tab + rm.off, static_cast<uint32_t>(len * sizeof(C)));
    unsigned bx = static_cast<unsigned>(tl - jlo) * static_cast<unsigned>(sizeof(C));   // d = c - lo of offset 0
    opaque(bx);
#pragma unroll
    for (int i = 0; i < Geo::E; ++i) {
      const int off = F::in_off(i);
      const unsigned j = static_cast<unsigned>(off < L / 2 ? off : off - L) * static_cast<unsigned>(sizeof(C));
      v[i] = c_mul(bload<C>(rz, bx + j), bload<C>(rt, bx + j));
    }
    if (rm.lo == 0 || rm.hi == half) {
#pragma unroll
      for (int i = 0; i < Geo::E; ++i) {
        const int off = F::in_off(i);
        const int c = rm.s + tl + (off < L / 2 ? off : off - L);
        const bool dc = c == 0 && rm.lo == 0, ny = c == half && rm.hi == half;
        if (ok && (dc || ny)) {
          const C w = tab[rm.off + (c - rm.lo)];
          const T x = dc ? z0.x : z0.y;
          v[i] = C{x * w.x, x * w.y};
        }
      }
    }
  }
  int nz = 0;
  if constexpr (F::R0 == 16 && Geo::E == 16) {
    const int t0 = __builtin_amdgcn_readfirstlane(tl) & ~63;
    constexpr int Q = L / 16;   // input i of lane tl sits at slot tl + i Q
    auto zero = [&](int a, int b) { return t0 + a * Q > jhi && t0 + 63 + b * Q < L + jlo; };
    nz = zero(1, 14) ? 2 : (zero(2, 13) ? 4 : 0);
  }
  F::run(v, reg, tl, F::twiddles(tw), nz);
  C* yrow = Y + int64_t(ok ? gr : 0) * os.M;
  const rsrc_t rb = make_rsrc(bhat, static_cast<uint32_t>(os.nmax * L * int(sizeof(C))));
  // all blocks of the rows, or (few rows: the input transform repeated instead
  // of a workgroup's blocks in series) the one of blockIdx.y
  const int b0 = ONE ? static_cast<int>(blockIdx.y) : 0, b1 = ONE ? b0 + 1 : nb;
  int done = b0 == 0 ? 0 : (b0 - 1) * os.B - os.JP + L + jlo;   // outputs stored by the blocks before
  for (int b = b0; b < b1; ++b) {
    const int tb = ONE ? tl : opaque_copy(tl);   // keeps the transform's table loads in the loop (registers)
    C z[Geo::E];
#pragma unroll
    for (int i = 0; i < Geo::E; ++i) {
      constexpr auto in_reg = os_in_reg<F, Fi, Geo::E>;
      z[in_reg(i)] = c_mul(v[i], bload<C>(rb, static_cast<uint32_t>(tl) * sizeof(C),
                                          static_cast<uint32_t>(b * L + F::out_off(i)) * sizeof(C)));
    }
    Fi::run(z, reg, tb, Fi::twiddles(tw));
    const int V = b * os.B - os.JP;
    const int end = V + L + jlo < os.M ? V + L + jlo : os.M;
    if (ok && end > done) {
      // outputs done .. end - 1, at t = m - V
      unsigned bc = static_cast<unsigned>(V + tl) * static_cast<unsigned>(sizeof(C));
      unsigned bs = static_cast<unsigned>(V + tl - done) * static_cast<unsigned>(sizeof(C));
      opaque(bc);
      opaque(bs);
      const rsrc_t ry = make_rsrc(yrow + done, static_cast<uint32_t>((end - done) * sizeof(C)));
#pragma unroll
      for (int i = 0; i < Geo::E; ++i) {
        const unsigned o = static_cast<unsigned>(Fi::out_off(i)) * static_cast<unsigned>(sizeof(C));
        bstore<C, kYStore>(ry, c_mul(z[i], bload<C>(rc, bc + o)), bs + o);
      }
      done = end;
    }
  }
}

// PB > 1: one row per workgroup, whose PB thread groups transform PB blocks
// side by side; then each group adds up the blocks for its share of the
// registers, in the order of the blocks, so the bits are those of one group
// after the other. For launches of at most a row per CU, which otherwise wait
// for one block after the other, and for transforms of at most 128 threads: a
// group of 256 has a wave on every SIMD of its CU already, and four of them
// there take as long as four in turn (62 rows of 12289 values, L = 4096: 26 us
// in turn, 31 us side by side). Inverse rows in turn : side by side (: by one
// convolution): FP32 8 rows of 3535 values 22 : 14 (: 15) us, 16 rows of 1537
// values 14 : 11.3 (: 10.5) us, 8 rows of 2501 values 21 : 11 (: 15) us, in FP64
// 25 : 13 (: 20) us.
template <typename T, int L> constexpr int os_side_by_side() { return RowGeom<T, L>::TPR <= 128 ? 4 : 1; }

template <typename T, int L, int PB>
__global__ __launch_bounds__((PB > 1 ? PB * RowGeom<T, L>::TPR : RowGeom<T, L>::NT),
                             (PB > 1 ? (PB * RowGeom<T, L>::TPR + 255) / 256 : 4)) void k_inv_rows_os(
    const typename Complex<T>::type* __restrict__ Y, typename Complex<T>::type* __restrict__ Sbuf,
    const RowMeta* __restrict__ rows, const typename Complex<T>::type* __restrict__ tab, int R, int total, int sum_len, OsPlan os,
    const typename Complex<T>::type* __restrict__ chirp, const typename Complex<T>::type* __restrict__ bhat,
    const typename Complex<T>::type* __restrict__ tw) {
  using C = typename Complex<T>::type;
  using Geo = RowGeom<T, L>;
  using F = BlockFft<T, L, Geo::E, -1>;
  using Fi = BlockFft<T, L, Geo::E, +1>;
  static_assert(Geo::TPR >= 64, "a wave holds one row");
  constexpr int G = PB > 1 ? 1 : Geo::G;   // rows of a workgroup
  __shared__ C lds[G * PB * lds_size(L)];
  const int t = threadIdx.x, g = t / Geo::TPR, tl = t % Geo::TPR;
  const int pb = PB > 1 ? __builtin_amdgcn_readfirstlane(g) : 0;
  C* reg = lds + g * lds_size(L);
  const int u = static_cast<int>(blockIdx.x);
  int gr = u * G + (PB > 1 ? 0 : g);
  gr = __builtin_amdgcn_readfirstlane(gr);
  const bool ok = gr < total;
  const int seg = ok ? gr / R : 0;
  const RowMeta rm = rows[ok ? gr - seg * R : 0];
  const int len = ok ? rm.hi - rm.lo + 1 : 0;
  const int jlo = rm.lo - rm.s;
  const int nb = __builtin_amdgcn_readfirstlane(os.blocks[(u * G) % R]);
  const rsrc_t rc = make_rsrc(chirp, static_cast<uint32_t>(os.M * sizeof(C)));
  const rsrc_t rb = make_rsrc(bhat, static_cast<uint32_t>(os.nmax * L * int(sizeof(C))));
  const C* yrow = Y + int64_t(ok ? gr : 0) * os.M;
  auto end_of = [&](int b) {   // inputs of the blocks up to b
    const int e = b * os.B - os.JP + L + jlo;
    return e < os.M ? e : os.M;
  };
  constexpr int S = Geo::E / PB;   // registers that a group adds up: pb S .. pb S + S - 1
  C acc[S];
#pragma unroll
  for (int j = 0; j < S; ++j) acc[j] = C{0, 0};
  auto off_of = [&](int j) {   // F::out_off(pb S + j)
    const int i = pb * S + j;
    return i / F::RL * Geo::TPR + i % F::RL * (L / F::RL);
  };
  auto table = [&](int b, int j) {
    return bload<C>(rb, static_cast<uint32_t>(tl) * sizeof(C), static_cast<uint32_t>(b * L + off_of(j)) * sizeof(C));
  };
  auto add = [&](int j, C x, C bh) {
    const C h = c_conj(bh);
    acc[j] = C{fmadd(x.x, h.x, fmadd(-x.y, h.y, acc[j].x)), fmadd(x.x, h.y, fmadd(x.y, h.x, acc[j].y))};
  };
  for (int b0 = 0; b0 < nb; b0 += PB) {
    const int b = b0 + pb;
    const int done = b == 0 ? 0 : end_of(b - 1), end = ok && b < nb ? end_of(b) : done;
    const int V = b * os.B - os.JP;
    unsigned bc = static_cast<unsigned>(V + tl) * static_cast<unsigned>(sizeof(C));
    unsigned by = static_cast<unsigned>(V + tl - done) * static_cast<unsigned>(sizeof(C));
    opaque(bc);
    opaque(by);
    const rsrc_t ry = make_rsrc(yrow + done, static_cast<uint32_t>((end - done) * sizeof(C)));
    C v[Geo::E];
#pragma unroll
    for (int i = 0; i < Geo::E; ++i) {
      const unsigned o = static_cast<unsigned>(F::in_off(i)) * static_cast<unsigned>(sizeof(C));
      v[i] = c_mul(bload<C>(ry, by + o), c_conj(bload<C>(rc, bc + o)));
    }
    F::run(v, reg, opaque_copy(tl), F::twiddles(tw));   // (table loads stay in the loop: registers)
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (PB == 1) {
#pragma unroll
      for (int j = 0; j < S; ++j) add(j, v[j], table(b, j));
    } else {
#pragma unroll
      for (int i = 0; i < Geo::E; ++i) reg[lds_pad(tl + F::out_off(i))] = v[i];
      C h[PB][S];
#pragma unroll
      for (int q = 0; q < PB; ++q) {
#pragma unroll
        for (int j = 0; j < S; ++j) h[q][j] = table(b0 + q < nb ? b0 + q : b0, j);
      }
      __syncthreads();
#pragma unroll
      for (int q = 0; q < PB; ++q) {
        if (b0 + q < nb) {
#pragma unroll
          for (int j = 0; j < S; ++j) add(j, lds[q * lds_size(L) + lds_pad(tl + off_of(j))], h[q][j]);
        }
      }
      __syncthreads();
    }
  }
  C z[Geo::E];
  if constexpr (PB == 1) {
#pragma unroll
    for (int i = 0; i < Geo::E; ++i) {
      constexpr auto in_reg = os_in_reg<F, Fi, Geo::E>;
      z[in_reg(i)] = acc[i];
    }
  } else {
#pragma unroll
    for (int j = 0; j < S; ++j) lds[lds_pad(tl + off_of(j))] = acc[j];
    __syncthreads();
#pragma unroll
    for (int i = 0; i < Geo::E; ++i) z[i] = lds[lds_pad(tl + Fi::in_off(i))];
    __syncthreads();
  }
  Fi::run(z, reg, tl, Fi::twiddles(tw));
  if (!ok || pb > 0) return;
  // slot j mod L holds the kept entry d = j - jlo; the table holds its
  // conjugate chirp too
  const rsrc_t rs = make_rsrc(Sbuf + int64_t(seg) * sum_len + rm.off, static_cast<uint32_t>(len * sizeof(C)));
  const rsrc_t rt = make_rsrc(tab + rm.off, static_cast<uint32_t>(len * sizeof(C)));
  unsigned bs = static_cast<unsigned>(tl - jlo) * static_cast<unsigned>(sizeof(C));
  opaque(bs);
#pragma unroll
  for (int i = 0; i < Geo::E; ++i) {
    const int off = Fi::out_off(i);
    const unsigned j = static_cast<unsigned>(off < L / 2 ? off : off - L) * static_cast<unsigned>(sizeof(C));
    bstore<C>(rs, c_mul(z[i], bload<C>(rt, bs + j)), bs + j);
  }
}

// Chirp-z rows whose convolution length L exceeds one workgroup's transform:
// the products before and after the length-L cyclic convolution run as
// element passes around four-step transforms through the workspace (rows of
// L values, row gr = seg * R + k). Same identity and tables as above.
// Forward, before: B[gr][u] = X[c] F_k[c] a[u] for the kept bin c of slot
// u < M (slot_entry modulo M), 0 for the other u < L.
template <typename T>
__global__ __launch_bounds__(256) void k_bs_fwd_prep(const typename Complex<T>::type* __restrict__ spec,
                                                     typename Complex<T>::type* __restrict__ B,
                                                     const RowMeta* __restrict__ rows, const T* __restrict__ tab,
                                                     int R, int half, int M, int64_t L,
                                                     const typename Complex<T>::type* __restrict__ chirp) {
  using C = typename Complex<T>::type;
  const int64_t u = int64_t(blockIdx.x) * 256 + threadIdx.x;
  if (u >= L) return;
  const int64_t gr = blockIdx.y;
  const int64_t seg = gr / R;
  const RowMeta rm = rows[gr - seg * R];
  C val{0, 0};
  if (u < M) {
    int sh = (rm.s - rm.lo) % M;
    if (sh < 0) sh += M;
    const int d = static_cast<int>(u) + sh < M ? static_cast<int>(u) + sh : static_cast<int>(u) + sh - M;
    if (d <= rm.hi - rm.lo) {
      const int c = rm.lo + d;
      C x = spec[seg * half + (c == half ? 0 : c)];
      if (c == 0) x.y = 0;                     // slot 0 of the spectrum holds (X[0], X[N/2])
      if (c == half) x = C{x.y, 0};
      const T w = tab[rm.off + d];
      val = c_mul(C{x.x * w, x.y * w}, chirp[u]);
    }
  }
  B[gr * L + u] = val;
}

// Inverse, before: B[gr][u] = Y[gr][u] conj(a[u]) for u < M, 0 for u < L.
template <typename T>
__global__ __launch_bounds__(256) void k_bs_inv_prep(const typename Complex<T>::type* __restrict__ Y,
                                                     typename Complex<T>::type* __restrict__ B, int M, int64_t L,
                                                     const typename Complex<T>::type* __restrict__ chirp) {
  using C = typename Complex<T>::type;
  const int64_t u = int64_t(blockIdx.x) * 256 + threadIdx.x;
  if (u >= L) return;
  const int64_t gr = blockIdx.y;
  B[gr * L + u] = u < M ? c_mul(Y[gr * M + u], c_conj(chirp[u])) : C{0, 0};
}

// The spectrum of the convolution: B[gr][k] *= Bhat[k] (Bhat holds the 1/L).
template <typename T>
__global__ __launch_bounds__(256) void k_bs_mul(typename Complex<T>::type* __restrict__ B, int64_t L,
                                                const typename Complex<T>::type* __restrict__ bhat) {
  const int64_t k = int64_t(blockIdx.x) * 256 + threadIdx.x;
  if (k >= L) return;
  const int64_t i = int64_t(blockIdx.y) * L + k;
  B[i] = c_mul(B[i], bhat[k]);
}

// Forward, after: Y[gr][m] = B[gr][m] a[m], m < M.
template <typename T>
__global__ __launch_bounds__(256) void k_bs_fwd_post(const typename Complex<T>::type* __restrict__ B,
                                                     typename Complex<T>::type* __restrict__ Y, int M, int64_t L,
                                                     const typename Complex<T>::type* __restrict__ chirp) {
  const int64_t m = int64_t(blockIdx.x) * 256 + threadIdx.x;
  if (m >= M) return;
  const int64_t gr = blockIdx.y;
  Y[gr * M + m] = c_mul(B[gr * L + m], chirp[m]);
}

// Inverse, after: the kept slots u < M times conj(a[u]) and the table into
// the packed buffer Sbuf[seg * sum_len + off + d].
template <typename T>
__global__ __launch_bounds__(256) void k_bs_inv_post(const typename Complex<T>::type* __restrict__ B,
                                                     typename Complex<T>::type* __restrict__ Sbuf,
                                                     const RowMeta* __restrict__ rows, const T* __restrict__ tab,
                                                     int R, int64_t sum_len, int M, int64_t L,
                                                     const typename Complex<T>::type* __restrict__ chirp) {
  using C = typename Complex<T>::type;
  const int u = static_cast<int>(blockIdx.x) * 256 + static_cast<int>(threadIdx.x);
  if (u >= M) return;
  const int64_t gr = blockIdx.y;
  const int64_t seg = gr / R;
  const RowMeta rm = rows[gr - seg * R];
  int sh = (rm.s - rm.lo) % M;
  if (sh < 0) sh += M;
  const int d = u + sh < M ? u + sh : u + sh - M;
  if (d > rm.hi - rm.lo) return;
  const C z = c_mul(B[gr * L + u], c_conj(chirp[u]));
  const T w = tab[rm.off + d];
  Sbuf[seg * sum_len + rm.off + d] = C{z.x * w, z.y * w};
}

// Rows longer than one workgroup's LDS transform (four-step over the
// workspace, N_out = L1 * L2, slot u = n1 + L1 n2, output m = k2 + L2 k1).
// Forward, first pass: for every row, column n1 gathers its L2 slots from the
// spectrum (windowed, zero outside the kept support), runs the length-L2
// inverse FFT, multiplies by exp(+2 pi i n1 k2 / N_out) and stores A[n1 + L1 k2]
// of the row. The second pass is k_fft_rows_t over the rows (lengths L1).
template <typename T, int L2>
__global__ __launch_bounds__((ColGeom<T, L2>::NT)) void k_fwd_rows_cols(
    const typename Complex<T>::type* __restrict__ spec, typename Complex<T>::type* __restrict__ A,
    const RowMeta* __restrict__ rows, const T* __restrict__ tab, int R, int half, int64_t n_out, int64_t l1,
    const typename Complex<T>::type* __restrict__ tw, Twiddle2<typename Complex<T>::type> tw2) {
  using C = typename Complex<T>::type;
  using Geo = ColGeom<T, L2>;
  using F = BlockFft<T, L2, Geo::E, +1>;
  __shared__ C lds[Geo::CC * lds_size(L2)];
  const int t = threadIdx.x, cc = t % Geo::CC, tl = t / Geo::CC;
  const int64_t n1 = int64_t(blockIdx.x) * Geo::CC + cc;
  const int64_t gr = blockIdx.y;               // row of the chunk
  const int64_t seg = gr / R;
  const RowMeta rm = rows[int(gr - seg * R)];
  const C* Z = spec + seg * half;
  C v[Geo::E];
#pragma unroll
  for (int i = 0; i < Geo::E; ++i) {
    const int64_t u = n1 + l1 * F::in_index(tl, i);
    const int64_t c = rm.lo + ((u + rm.s - rm.lo) & (n_out - 1));   // kept bin of slot u, if <= hi
    C val{0, 0};
    if (c <= rm.hi) {
      val = Z[c == half ? 0 : c];
      if (c == 0) val.y = 0;                  // slot 0 holds (X[0], X[N/2])
      if (c == half) val = C{val.y, 0};
      const T w = tab[rm.off + (c - rm.lo)];
      val = C{val.x * w, val.y * w};
    }
    v[i] = val;
  }
  F::run(v, lds + cc * lds_size(L2), tl, F::twiddles(tw));
  C* dst = A + gr * n_out + n1;
#pragma unroll
  for (int i = 0; i < Geo::E; ++i) {
    const int64_t k2 = F::out_index(tl, i);
    C w = tw2(n1 * k2);
    w.y = -w.y;                               // exp(+2 pi i n1 k2 / N_out)
    dst[l1 * k2] = c_mul(v[i], w);
  }
}

// Inverse, second pass over long rows: length-L1 FFTs along the rows k2 of
// the intermediate (CC rows per workgroup, staged through LDS), then the kept
// output slots m = k2 + L2 k1 times the table go to the packed buffer.
template <typename T, int L1>
__global__ __launch_bounds__((ColGeom<T, L1>::NT)) void k_inv_rows_rowst(
    const typename Complex<T>::type* __restrict__ A, typename Complex<T>::type* __restrict__ Sbuf,
    const RowMeta* __restrict__ rows, const T* __restrict__ tab, int R, int64_t sum_len, int64_t n_out,
    int64_t l2, const typename Complex<T>::type* __restrict__ tw) {
  using C = typename Complex<T>::type;
  using Geo = ColGeom<T, L1>;
  using F = BlockFft<T, L1, Geo::E, -1>;
  __shared__ C lds[Geo::CC * lds_size(L1)];
  const int t = threadIdx.x;
  const int64_t gr = blockIdx.y;
  const int64_t k2_0 = int64_t(blockIdx.x) * Geo::CC;
  const C* src = A + gr * n_out + k2_0 * L1;
  for (int i = t; i < Geo::CC * L1; i += Geo::NT) lds[(i / L1) * lds_size(L1) + lds_pad(i % L1)] = src[i];
  __syncthreads();
  const int cc = t % Geo::CC, tl = t / Geo::CC;
  C* reg = lds + cc * lds_size(L1);
  C v[Geo::E];
#pragma unroll
  for (int i = 0; i < Geo::E; ++i) v[i] = reg[lds_pad(F::in_index(tl, i))];
  __syncthreads();
  F::run(v, reg, tl, F::twiddles(tw));
  const int64_t seg = gr / R;
  const RowMeta rm = rows[int(gr - seg * R)];
  C* dst = Sbuf + seg * sum_len + rm.off - rm.lo;
  const T* tb = tab + rm.off - rm.lo;
#pragma unroll
  for (int i = 0; i < Geo::E; ++i) {
    const int64_t m = k2_0 + cc + l2 * F::out_index(tl, i);
    const int64_t c = rm.lo + ((m + rm.s - rm.lo) & (n_out - 1));   // kept bin of slot m, if <= hi
    if (c <= rm.hi) {
      const T w = tb[c];
      dst[c] = C{v[i].x * w, v[i].y * w};
    }
  }
}

// Single-tile recovery on rows longer than one workgroup: the second pass of
// the row's N_out-point forward transform (after k_fft_cols over row `row` of
// each segment, intermediate rows of stride a_stride), then the kept slots
// times the tile table into Sx[seg][c], as k_tile_rows does.
template <typename T, int L1>
__global__ __launch_bounds__((ColGeom<T, L1>::NT)) void k_tile_rows_rowst(
    const typename Complex<T>::type* __restrict__ A, typename Complex<T>::type* __restrict__ Sx,
    const RowMeta* __restrict__ rows, const T* __restrict__ tab, int row, int half, int64_t a_stride,
    int64_t n_out, int64_t l2, const typename Complex<T>::type* __restrict__ tw) {
  using C = typename Complex<T>::type;
  using Geo = ColGeom<T, L1>;
  using F = BlockFft<T, L1, Geo::E, -1>;
  __shared__ C lds[Geo::CC * lds_size(L1)];
  const int t = threadIdx.x;
  const int64_t seg = blockIdx.y;
  const int64_t k2_0 = int64_t(blockIdx.x) * Geo::CC;
  const C* src = A + seg * a_stride + k2_0 * L1;
  for (int i = t; i < Geo::CC * L1; i += Geo::NT) lds[(i / L1) * lds_size(L1) + lds_pad(i % L1)] = src[i];
  __syncthreads();
  const int cc = t % Geo::CC, tl = t / Geo::CC;
  C* reg = lds + cc * lds_size(L1);
  C v[Geo::E];
#pragma unroll
  for (int i = 0; i < Geo::E; ++i) v[i] = reg[lds_pad(F::in_index(tl, i))];
  __syncthreads();
  F::run(v, reg, tl, F::twiddles(tw));
  const RowMeta rm = rows[row];
  C* dst = Sx + seg * (half + 1);
  const T* tb = tab + rm.off - rm.lo;
#pragma unroll
  for (int i = 0; i < Geo::E; ++i) {
    const int64_t m = k2_0 + cc + l2 * F::out_index(tl, i);
    const int64_t c = rm.lo + ((m + rm.s - rm.lo) & (n_out - 1));   // kept bin of slot m, if <= hi
    if (c <= rm.hi) {
      const T w = tb[c];
      dst[c] = C{v[i].x * w, v[i].y * w};
    }
  }
}

}  // namespace qtam
