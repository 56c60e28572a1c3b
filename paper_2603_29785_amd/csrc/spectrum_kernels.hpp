// Spectrum and synthesis kernels: the N/2-point complex transforms of the
// packed real signal (one pass, or the two passes of the four-step
// factorisation N/2 = N1 * N2), the real-signal twist, and the decimation by
// 3 or 5 around power-of-two transforms (App. A RFFT; App. C DFT convention).
#pragma once

#include "device_common.hpp"

namespace qtam {

// Batched contiguous complex FFTs of length L: transform t reads
// in[t*stride + n] and writes out[t*stride + k]. A chunk holds count
// transforms; every buffer of it is below 2 GiB.
// RIN = r > 1: transform t = seg * r + n1 reads the decimated signal
// in[seg * r * L + n1 + r n] (its r siblings read the same lines); ROUT = r:
// it writes out[seg * r * L + n1 + r k]. stride = L then.
template <typename T, int L, int S, int RIN = 1, int ROUT = 1>
__global__ __launch_bounds__((RowGeom<T, L>::NT)) void k_fft_rows(
    const typename Complex<T>::type* __restrict__ in, typename Complex<T>::type* __restrict__ out,
    int64_t count, int64_t stride, const typename Complex<T>::type* __restrict__ tw) {
  using C = typename Complex<T>::type;
  using Geo = RowGeom<T, L>;
  using F = BlockFft<T, L, Geo::E, S>;
  static_assert((RIN == 1 && ROUT == 1) || Geo::G == 1, "decimated rows: one transform per workgroup");
  __shared__ C lds[Geo::G * lds_size(L)];
  const int t = threadIdx.x, g = t / Geo::TPR, tl = t % Geo::TPR;
  int64_t tr0 = int64_t(blockIdx.x) * Geo::G;
  if constexpr (RIN * ROUT > 1) {
    int64_t v;
    int s;
    sibling_block<RIN * ROUT>(tr0, count / (RIN * ROUT), v, s);
    tr0 = v * (RIN * ROUT) + s;
  }
  const int64_t nt = count - tr0 < Geo::G ? count - tr0 : Geo::G;   // transforms of this block
  const uint32_t bytes = static_cast<uint32_t>((nt - 1) * stride + L) * sizeof(C);
  // lanes of transforms past the end fall outside [0, bytes): loads give 0
  const rsrc_t rin = RIN > 1 ? make_rsrc(in + tr0 / RIN * (RIN * L) + tr0 % RIN, (RIN * (L - 1) + 1) * sizeof(C))
                             : make_rsrc(in + tr0 * stride, bytes);
  const rsrc_t rout = ROUT > 1 ? make_rsrc(out + tr0 / ROUT * (ROUT * L) + tr0 % ROUT, (ROUT * (L - 1) + 1) * sizeof(C))
                               : make_rsrc(out + tr0 * stride, bytes);
  const uint32_t vb = static_cast<uint32_t>(g * stride + tl) * sizeof(C);
  C v[Geo::E];
#pragma unroll
  for (int i = 0; i < Geo::E; ++i) v[i] = bload<C>(rin, vb * RIN, F::in_off(i) * RIN * sizeof(C));
  F::run(v, lds + g * lds_size(L), tl, F::twiddles(tw));
  if (g < nt) {
#pragma unroll
    for (int i = 0; i < Geo::E; ++i) bstore<C>(rout, v[i], vb * ROUT, F::out_off(i) * ROUT * sizeof(C));
  }
}

// Four-step, first pass: length-N2 FFTs down the columns n1 of the N1 x N2
// view (element stride N1), times exp(S 2 pi i n1 k2 / M), written back in
// place-order. CC adjacent columns per workgroup, column index fastest
// across threads so every access is a contiguous run of CC values.
// RIN = r > 1: blockIdx.y = seg * r + n1d reads the decimated signal
// in[seg * r * seg_stride + n1d + r n] (runs at stride r; the siblings n1d
// read the same lines, from the cache).
template <typename T, int L, int S, int CW = 0, int RIN = 1>
__global__ __launch_bounds__((ColGeom<T, L, 0, CW>::NT)) void k_fft_cols(
    const typename Complex<T>::type* __restrict__ in, typename Complex<T>::type* __restrict__ out,
    int64_t n1_count, int64_t seg_stride, const typename Complex<T>::type* __restrict__ tw,
    Twiddle2<typename Complex<T>::type> tw2, int tw_mul) {
  using C = typename Complex<T>::type;
  using Geo = ColGeom<T, L, 0, CW>;
  using F = BlockFft<T, L, Geo::E, S>;
  __shared__ C lds[Geo::CC * lds_size(L)];
  const int t = threadIdx.x, c = t % Geo::CC, tl = t / Geo::CC;
  int64_t bx = blockIdx.x, by = blockIdx.y;   // column tile, transform
  int sib = 0;
  if constexpr (RIN > 1) {
    int64_t v;
    sibling_block<RIN>(by * gridDim.x + bx, int64_t(gridDim.x) * (gridDim.y / RIN), v, sib);
    bx = v % gridDim.x;
    by = v / gridDim.x * RIN + sib;
  }
  const int64_t n1 = bx * Geo::CC + c;
  const int64_t base = by * seg_stride + n1;
  const int64_t bin = RIN > 1 ? (by - sib) * seg_stride + sib + RIN * n1 : base;
  C v[Geo::E];
#pragma unroll
  for (int i = 0; i < Geo::E; ++i) v[i] = in[bin + RIN * n1_count * F::in_index(tl, i)];
  F::run(v, lds + c * lds_size(L), tl, F::twiddles(tw));
#pragma unroll
  for (int i = 0; i < Geo::E; ++i) {
    const int64_t k2 = F::out_index(tl, i);
    // exp(-2 pi i n1 k2 / M), M = N1 N2, from the table of exp(-2 pi i m / (tw_mul M))
    C w = tw2(tw_mul * n1 * k2);
    if constexpr (S > 0) w.y = -w.y;
    out[base + n1_count * k2] = c_mul(v[i], w);
  }
}

// Four-step, second pass: length-N1 FFTs along the contiguous rows k2 of the
// intermediate; CC rows per workgroup are staged through LDS with a linear
// (coalesced) load, results go to Z[k2 + N2 k1] in runs of CC values.
// ROUT = r > 1: blockIdx.y = seg * r + n1d writes the interleaved signal
// out[seg * r * seg_stride + n1d + r n] (the siblings fill the same lines).
template <typename T, int L, int S, int EP = 0, int CW = 0, int ROUT = 1>
__global__ __launch_bounds__((ColGeom<T, L, EP, CW>::NT)) void k_fft_rows_t(
    const typename Complex<T>::type* __restrict__ in, typename Complex<T>::type* __restrict__ out,
    int64_t n2_count, int64_t seg_stride, const typename Complex<T>::type* __restrict__ tw) {
  using C = typename Complex<T>::type;
  using Geo = ColGeom<T, L, EP, CW>;
  using F = BlockFft<T, L, Geo::E, S>;
  __shared__ C lds[Geo::CC * lds_size(L)];
  const int t = threadIdx.x;
  int64_t bx = blockIdx.x, by = blockIdx.y;   // row tile, transform
  int sib = 0;
  if constexpr (ROUT > 1) {
    int64_t v;
    sibling_block<ROUT>(by * gridDim.x + bx, int64_t(gridDim.x) * (gridDim.y / ROUT), v, sib);
    bx = v % gridDim.x;
    by = v / gridDim.x * ROUT + sib;
  }
  const int64_t k2_0 = bx * Geo::CC;
  const C* src = in + by * seg_stride + k2_0 * L;
  for (int i = t; i < Geo::CC * L; i += Geo::NT) lds[(i / L) * lds_size(L) + lds_pad(i % L)] = src[i];
  __syncthreads();
  const int c = t % Geo::CC, tl = t / Geo::CC;
  C* reg = lds + c * lds_size(L);
  C v[Geo::E];
#pragma unroll
  for (int i = 0; i < Geo::E; ++i) v[i] = reg[lds_pad(F::in_index(tl, i))];
  __syncthreads();
  F::run(v, reg, tl, F::twiddles(tw));
  C* dst = out + (by - sib) * seg_stride + sib + ROUT * (k2_0 + c);
#pragma unroll
  for (int i = 0; i < Geo::E; ++i) dst[ROUT * n2_count * F::out_index(tl, i)] = v[i];
}

// Four-step second pass fused with the real-signal twist (combine_twist below): the
// output of row k2 at k1 (bin m = k2 + N2 k1 of Z) meets its mirror
// N/2 - m in row N2 - k2 at N1 - 1 - k1 (row 0: itself at N1 - k1 mod N1), so
// a workgroup takes mirrored row pairs: H = CC/2 rows j H + c and their
// mirrors N2 - j H - c (workgroup 0: rows 0 .. H-1, N2/2 and N2-H+1 .. N2-1,
// rows 0 and N2/2 being their own mirrors). After the row transforms the
// values go through LDS to the thread that twists each bin.
template <typename T, int L, int EP = 0, int CW = 0>
__global__ __launch_bounds__((ColGeom<T, L, EP, CW>::NT)) void k_spec_rows_twist(
    const typename Complex<T>::type* __restrict__ in, typename Complex<T>::type* __restrict__ out, int64_t n2,
    int64_t seg_stride, const typename Complex<T>::type* __restrict__ tw, Twiddle2<typename Complex<T>::type> tw2) {
  using C = typename Complex<T>::type;
  using Geo = ColGeom<T, L, EP, CW>;
  using F = BlockFft<T, L, Geo::E, -1>;
  constexpr int CC = Geo::CC, H = CC / 2;
  static_assert(CC % 2 == 0, "paired rows");
  __shared__ C lds[CC * lds_size(L)];
  const int t = threadIdx.x;
  const int64_t j = blockIdx.x;
  auto row_of = [&](int c) -> int64_t {
    if (j == 0) return c < H ? c : (c == H ? n2 / 2 : n2 - (c - H));
    return c < H ? j * H + c : n2 - (j * H + (c - H));
  };
  const C* src = in + int64_t(blockIdx.y) * seg_stride;
  for (int i = t; i < CC * L; i += Geo::NT) {
    const int c = i / L;
    lds[c * lds_size(L) + lds_pad(i % L)] = src[row_of(c) * L + (i % L)];
  }
  __syncthreads();
  const int c = t % CC, tl = t / CC;
  C* reg = lds + c * lds_size(L);
  C v[Geo::E];
#pragma unroll
  for (int i = 0; i < Geo::E; ++i) v[i] = reg[lds_pad(F::in_index(tl, i))];
  __syncthreads();
  F::run(v, reg, tl, F::twiddles(tw));
  // every transform's output into its own LDS column, then the twist
#pragma unroll
  for (int i = 0; i < Geo::E; ++i) reg[lds_pad(F::out_index(tl, i))] = v[i];
  __syncthreads();
  const int64_t r = row_of(c);
  const int pc = (j == 0 && (c == 0 || c == H)) ? c : (c < H ? c + H : c - H);
  const C* preg = lds + pc * lds_size(L);
  C* dst = out + int64_t(blockIdx.y) * seg_stride;
  const T hh = T(0.5);
#pragma unroll
  for (int i = 0; i < Geo::E; ++i) {
    const int k1 = F::out_index(tl, i);
    const int64_t m = r + n2 * k1;
    const C zp = v[i];
    if (m == 0) {   // X[0] and X[N/2] share slot 0
      dst[0] = C{zp.x + zp.y, zp.x - zp.y};
      continue;
    }
    const int k1m = r == 0 ? (L - k1) & (L - 1) : L - 1 - k1;
    const C zq = preg[lds_pad(k1m)];
    const C w = tw2(m);                          // e^{-2 pi i m / N}
    const C a = c_add(zp, c_conj(zq)), b = c_sub(zp, c_conj(zq));
    const C xp = c_add(a, c_mul_si<-1>(c_mul(w, b)));
    dst[m] = C{xp.x * hh, xp.y * hh};
  }
}

// Segment lengths with N/2 = r * M2, r in {3, 5}, M2 a power of two: the
// half-size transform splits into r interleaved length-M2 transforms
// (decimation by r) and one radix-r combination.
//   forward:  Zp[n1][n2] = z[n1 + r n2];  F_n1 = DFT_M2(Zp[n1]);
//             Z[k2 + M2 k1] = sum_n1 e^{-2 pi i n1 k1 / r} e^{-2 pi i n1 k2 / (N/2)} F_n1[k2]
//   inverse:  A_n1[k2] = e^{+2 pi i n1 k2 / (N/2)} sum_k1 Z[k2 + M2 k1] e^{+2 pi i n1 k1 / r};
//             z[n1 + r n2] = IDFT_M2(A_n1)[n2]
// The first transform pass reads the decimated signal in place and the last
// synthesis pass writes the interleaved one, so no pass only permutes;
// k_radix does the combination of the synthesis, k_radix_twist that of the
// analysis with the real-signal twist, and where a segment fits one workgroup
// k_spec_seg / k_syn_seg do all of it.

// cos / sin of 2 pi k / R for R = 1, 3, 5
template <typename T, int R>
__device__ __forceinline__ typename Complex<T>::type root_r(int k) {
  using C = typename Complex<T>::type;
  if constexpr (R == 1) {
    return C{1, 0};
  } else if constexpr (R == 3) {
    constexpr T c1 = static_cast<T>(-0.5), s1 = static_cast<T>(0.86602540378443864676);
    return k == 0 ? C{1, 0} : (k == 1 ? C{c1, s1} : C{c1, -s1});
  } else {
    constexpr T c1 = static_cast<T>(0.30901699437494742410), s1 = static_cast<T>(0.95105651629515357212);
    constexpr T c2 = static_cast<T>(-0.80901699437494742410), s2 = static_cast<T>(0.58778525229247312917);
    return k == 0 ? C{1, 0} : k == 1 ? C{c1, s1} : k == 2 ? C{c2, s2} : k == 3 ? C{c2, -s2} : C{c1, -s1};
  }
}

// b = radix-R DFT of a, kernel exp(S 2 pi i n k / R)
template <typename T, int R, int S>
__device__ __forceinline__ void dft_r(const typename Complex<T>::type (&a)[R], typename Complex<T>::type (&b)[R]) {
  using C = typename Complex<T>::type;
#pragma unroll
  for (int k = 0; k < R; ++k) {
    C acc = a[0];
#pragma unroll
    for (int n = 1; n < R; ++n) {
      const C w = root_r<T, R>((n * k) % R);
      acc = c_add(acc, c_mul(a[n], S > 0 ? w : c_conj(w)));
    }
    b[k] = acc;
  }
}

// Radix-R combination of a synthesis: the spectrum Z to the decimated rows
// A_n1, in rows of m2.
template <typename T, int R>
__global__ __launch_bounds__(256) void k_radix(const typename Complex<T>::type* __restrict__ in,
                                               typename Complex<T>::type* __restrict__ out, int64_t m2,
                                               Twiddle2<typename Complex<T>::type> tw2) {
  using C = typename Complex<T>::type;
  const int64_t k2 = int64_t(blockIdx.x) * 256 + threadIdx.x;
  if (k2 >= m2) return;
  const int64_t base = int64_t(blockIdx.y) * R * m2;
  C a[R], b[R];
#pragma unroll
  for (int k1 = 0; k1 < R; ++k1) a[k1] = in[base + k2 + m2 * k1];
  dft_r<T, R, +1>(a, b);
#pragma unroll
  for (int n1 = 0; n1 < R; ++n1)
    out[base + n1 * m2 + k2] = n1 == 0 ? b[0] : c_mul(b[n1], c_conj(tw2(2 * n1 * k2)));
}

// Real-signal spectrum from the N/2-point transform Z of the even/odd pairs
// of a segment: for c in [0, N/2]
//   X[c] = (Z[c] + Z*[N/2-c])/2 - (i/2) e^{-2 pi i c/N} (Z[c] - Z*[N/2-c])
// (indices of Z mod N/2); the real X[0] and X[N/2] share slot 0 as
// (X[0], X[N/2]). Here the bins c = k2 + M2 k1 of one k2 in [0, M2/2] and
// their mirrors N/2 - c (k2' = M2 - k2, k1' = R - 1 - k1; at k2 = 0 the
// mirrors are k1' = R - k1 mod R of the same k2), from the decimated
// transforms' values a[n1] at k2 and b[n1] at (M2 - k2) mod M2, each already
// times its e^{-2 pi i n1 k / (N/2)}.
template <typename T, int R>
__device__ __forceinline__ void combine_twist(const typename Complex<T>::type (&a)[R],
                                              const typename Complex<T>::type (&b)[R], int k2, int m2,
                                              typename Complex<T>::type* __restrict__ out,
                                              const Twiddle2<typename Complex<T>::type>& tw2) {
  using C = typename Complex<T>::type;
  const T h = T(0.5);
  C z[R], y[R];
  dft_r<T, R, -1>(a, z);
  const bool own = k2 == 0 || 2 * k2 == m2;   // the mirrors are bins of this k2
  if (!own) dft_r<T, R, -1>(b, y);
#pragma unroll
  for (int k1 = 0; k1 < R; ++k1) {
    const int c = k2 + m2 * k1;
    if (c == 0) {
      out[0] = C{z[0].x + z[0].y, z[0].x - z[0].y};
      continue;
    }
    const C zp = z[k1];
    const C zq = !own ? y[R - 1 - k1] : k2 == 0 ? z[(R - k1) % R] : z[R - 1 - k1];
    const C w = tw2(c);                           // e^{-2 pi i c/N}; at the mirror it is -conj(w)
    const C s = c_add(zp, c_conj(zq)), d = c_sub(zp, c_conj(zq));
    const C x = c_add(s, c_mul_si<-1>(c_mul(w, d)));
    out[c] = C{x.x * h, x.y * h};
    if (!own) {
      const C s2 = c_add(zq, c_conj(zp)), d2 = c_sub(zq, c_conj(zp));
      const C x2 = c_sub(s2, c_mul_si<-1>(c_mul(c_conj(w), d2)));
      out[R * m2 - c] = C{x2.x * h, x2.y * h};
    }
  }
}

// Radix-R combination of the decimated transforms F (rows of m2 per segment)
// and the real-signal twist in one pass over memory.
template <typename T, int R>
__global__ __launch_bounds__(256) void k_radix_twist(const typename Complex<T>::type* __restrict__ in,
                                                     typename Complex<T>::type* __restrict__ out, int64_t m2,
                                                     Twiddle2<typename Complex<T>::type> tw2) {
  using C = typename Complex<T>::type;
  const int64_t k2 = int64_t(blockIdx.x) * 256 + threadIdx.x;
  if (k2 > m2 / 2) return;
  const int64_t q2 = k2 == 0 ? 0 : m2 - k2;
  const int64_t base = int64_t(blockIdx.y) * R * m2;
  C a[R], b[R];
#pragma unroll
  for (int n1 = 0; n1 < R; ++n1) {
    a[n1] = in[base + n1 * m2 + k2];
    b[n1] = in[base + n1 * m2 + q2];
    if (n1 > 0) {
      a[n1] = c_mul(a[n1], tw2(2 * n1 * k2));
      b[n1] = c_mul(b[n1], tw2(2 * n1 * q2));
    }
  }
  combine_twist<T, R>(a, b, static_cast<int>(k2), static_cast<int>(m2), out + base, tw2);
}

// Segments whose N/2 = R * M2 complex values fit the LDS of a workgroup: the
// whole spectrum (decimated read, R transforms of length M2 side by side,
// combination, real-signal twist) and the whole synthesis transform (its
// mirror image) in one launch each, with no pass over memory but the read of
// the signal and the write of the spectrum. G segments per workgroup while
// their threads make at most 256. Bound by memory at many segments and by one
// transform's latency at few. Measured on MI355X, FP32: spectra of 1024 x
// 24576 samples (R = 3) 148 us as permutation, transforms, combination and
// twist, 78 us here; one 16384-sample segment forward + inverse (R = 1) 35.9
// to 32.3 us. Segments above one workgroup, without the permutation passes
// (256 x 49152 samples, forward + inverse with 16 rows): 229 to 184 us.
template <typename T, int M2, int R>
struct SegGeom {
  static constexpr int E = RowGeom<T, M2>::E;
  static constexpr int TPR = M2 / E;          // threads of one length-M2 transform
  static constexpr int TS = R * TPR;          // threads of one segment
  static constexpr int G = TS >= 256 ? 1 : 256 / TS;
  static constexpr int NT = G * TS;
  static constexpr size_t LDS = size_t(G) * R * lds_size(M2) * 2 * sizeof(T);
  static constexpr bool FITS = LDS <= 160u * 1024u && NT <= 1024;
};

template <typename T, int M2, int R>
__global__ __launch_bounds__((SegGeom<T, M2, R>::NT)) void k_spec_seg(
    const typename Complex<T>::type* __restrict__ in, typename Complex<T>::type* __restrict__ out, int64_t segs,
    const typename Complex<T>::type* __restrict__ tw, Twiddle2<typename Complex<T>::type> tw2) {
  using C = typename Complex<T>::type;
  using Geo = SegGeom<T, M2, R>;
  using F = BlockFft<T, M2, Geo::E, -1>;
  __shared__ C lds[Geo::G * R * lds_size(M2)];
  const int t = threadIdx.x, q = t / Geo::TPR, tl = t % Geo::TPR;   // q = g * R + n1
  const int g = t / Geo::TS, n1 = q % R;
  const int64_t s0 = int64_t(blockIdx.x) * Geo::G;
  const int64_t ns = segs - s0 < Geo::G ? segs - s0 : Geo::G;
  // lanes of segments past the end fall outside the resource: loads give 0
  const rsrc_t rin = make_rsrc(in + s0 * R * M2, static_cast<uint32_t>(ns * R * M2) * sizeof(C));
  const uint32_t vb = static_cast<uint32_t>(g * R * M2 + n1 + R * tl) * sizeof(C);
  C v[Geo::E];
#pragma unroll
  for (int i = 0; i < Geo::E; ++i) v[i] = bload<C>(rin, vb, R * F::in_off(i) * sizeof(C));
  C* reg = lds + q * lds_size(M2);
  F::run(v, reg, tl, F::twiddles(tw));
#pragma unroll
  for (int i = 0; i < Geo::E; ++i) {
    const int k2 = tl + F::out_off(i);
    if (R > 1 && n1 > 0) v[i] = c_mul(v[i], tw2(2 * n1 * k2));
    reg[lds_pad(k2)] = v[i];
  }
  __syncthreads();
  if (g >= ns) return;
  const C* rows = lds + g * R * lds_size(M2);
  C* dst = out + (s0 + g) * (R * M2);
  // unrolled, so that the twiddle loads of all rounds are in flight at once
  constexpr int ROUNDS = (M2 / 2 + Geo::TS) / Geo::TS;
#pragma unroll
  for (int i = 0; i < ROUNDS; ++i) {
    const int k2 = t - g * Geo::TS + i * Geo::TS;
    if (i == ROUNDS - 1 && k2 > M2 / 2) break;
    C a[R], b[R];
#pragma unroll
    for (int n = 0; n < R; ++n) {
      a[n] = rows[n * lds_size(M2) + lds_pad(k2)];
      b[n] = rows[n * lds_size(M2) + lds_pad((M2 - k2) & (M2 - 1))];
    }
    combine_twist<T, R>(a, b, k2, M2, dst, tw2);
  }
}

template <typename T, int M2, int R>
__global__ __launch_bounds__((SegGeom<T, M2, R>::NT)) void k_syn_seg(
    const typename Complex<T>::type* __restrict__ in, typename Complex<T>::type* __restrict__ out, int64_t segs,
    const typename Complex<T>::type* __restrict__ tw, Twiddle2<typename Complex<T>::type> tw2) {
  using C = typename Complex<T>::type;
  using Geo = SegGeom<T, M2, R>;
  using F = BlockFft<T, M2, Geo::E, +1>;
  __shared__ C lds[Geo::G * R * lds_size(M2)];
  const int t = threadIdx.x, q = t / Geo::TPR, tl = t % Geo::TPR;
  const int g = t / Geo::TS, ts = t - g * Geo::TS;
  const int64_t seg = int64_t(blockIdx.x) * Geo::G + g;
  const bool ok = seg < segs;
  C* rows = lds + g * R * lds_size(M2);
  const C* src = in + (ok ? seg : 0) * (R * M2);
  for (int k2 = ts; k2 < M2; k2 += Geo::TS) {
    C a[R], b[R];
#pragma unroll
    for (int k1 = 0; k1 < R; ++k1) a[k1] = src[k2 + M2 * k1];
    dft_r<T, R, +1>(a, b);
#pragma unroll
    for (int n = 0; n < R; ++n)
      rows[n * lds_size(M2) + lds_pad(k2)] = n == 0 ? b[0] : c_mul(b[n], c_conj(tw2(2 * n * k2)));
  }
  __syncthreads();
  C* reg = lds + q * lds_size(M2);
  C v[Geo::E];
#pragma unroll
  for (int i = 0; i < Geo::E; ++i) v[i] = reg[lds_pad(tl + F::in_off(i))];
  __syncthreads();
  F::run(v, reg, tl, F::twiddles(tw));
#pragma unroll
  for (int i = 0; i < Geo::E; ++i) reg[lds_pad(tl + F::out_off(i))] = v[i];
  __syncthreads();
  if (!ok) return;
  C* dst = out + seg * (R * M2);
  for (int i = ts; i < R * M2; i += Geo::TS) dst[i] = rows[(i % R) * lds_size(M2) + lds_pad(i / R)];
}

// The synthesis transform of a few segments as R sibling workgroups each: one
// decimated row n1 straight from the spectrum (every sibling reads all of it),
// its transform, and the interleaved store, the same operations as above. A
// workgroup that holds a segment of more than 512 threads has three or more
// waves on a SIMD and is bound by its CU's vector ALU; the siblings take R CUs.
// Whole inverse in a graph, 16 to 32 rows, one workgroup : siblings, us:
// FP32 24576 samples, 1 / 4 / 32 / 84 segments  20.1 / 20.7 / 25.8 / 36.4 : 18.7 / 19.4 / 24.5 / 37.1
// FP64 12288 samples                            17.9 / 18.8 / 24.3 / 33.6 : 15.7 / 16.6 / 22.1 / 32.5
// FP32 20480 samples (R = 5, rows of two waves) 19.8 / 20.5 / 25.1 / 34.2 : 20.2 / 20.9 / 25.2 / 35.0
// (with separate radix, transform and permutation passes 18.4 / 19.2 / 26.3 /
// 41.1, 17.0 / 17.8 / 25.2 / 39.2 and 18.0 / 18.9 / 25.8 / 39.1).
template <typename T, int M2, int R>
constexpr bool syn_siblings() { return R > 1 && SegGeom<T, M2, R>::TS > 512 && !(sizeof(T) == 4 && R == 5); }

template <typename T, int M2, int R>
__global__ __launch_bounds__((RowGeom<T, M2>::TPR), 1) void k_syn_siblings(
    const typename Complex<T>::type* __restrict__ in, typename Complex<T>::type* __restrict__ out, int64_t segs,
    const typename Complex<T>::type* __restrict__ tw, Twiddle2<typename Complex<T>::type> tw2) {
  using C = typename Complex<T>::type;
  using Geo = RowGeom<T, M2>;
  using F = BlockFft<T, M2, Geo::E, +1>;
  __shared__ C lds[lds_size(M2)];
  const int tl = threadIdx.x;
  int64_t seg;
  int n1;
  sibling_block<R>(blockIdx.x, segs, seg, n1);
  const C* src = in + seg * (R * M2);
  // every load in flight before the first is used
  C a[Geo::E][R], wf[Geo::E], wc[Geo::E], v[Geo::E];
#pragma unroll
  for (int i = 0; i < Geo::E; ++i) {
    const int k2 = tl + F::in_off(i), m = 2 * n1 * k2;
#pragma unroll
    for (int k1 = 0; k1 < R; ++k1) a[i][k1] = src[k2 + M2 * k1];
    wf[i] = tw2.fine[m & ((1 << tw2.bits) - 1)];
    wc[i] = tw2.coarse[m >> tw2.bits];
  }
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int i = 0; i < Geo::E; ++i) {
    v[i] = a[i][0];
#pragma unroll
    for (int k1 = 1; k1 < R; ++k1) v[i] = c_add(v[i], c_mul(a[i][k1], root_r<T, R>(n1 * k1 % R)));
    if (n1 > 0) v[i] = c_mul(v[i], c_conj(c_mul(wf[i], wc[i])));
  }
  F::run(v, lds, tl, F::twiddles(tw));
  C* dst = out + seg * (R * M2) + n1;
#pragma unroll
  for (int i = 0; i < Geo::E; ++i) dst[R * (tl + F::out_off(i))] = v[i];
}

}  // namespace qtam
