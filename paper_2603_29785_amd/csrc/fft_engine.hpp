// Block-level Stockham FFT engine for gfx950.
//
// A transform of length L (a power of two) is processed by TPR = L/E threads,
// each holding E complex values in registers. Every pass applies radix-R
// butterflies (R = min(E, 16), the last pass possibly smaller; with E = 32 a
// thread holds two groups) to values held in registers; between passes the
// values are exchanged through an LDS region of the transform (in two rounds
// over half of it when the whole would not fit). First-pass inputs and last-pass outputs are addressed so that
// consecutive threads touch consecutive elements: kernels feed the engine
// straight from global memory and store its results straight back, coalesced.
//
// Layout of the registers of thread tl (tl in [0, TPR)):
//   before the first pass: v[q*R0 + r] = a[tl + q*TPR + r*(L/R0)]
//   after the last pass:   v[q*RL + r] = A[tl + q*TPR + r*(L/RL)]
// Twiddles: every pass after the first (stride NS, radix R) needs
// w^r, w = exp(-2 pi i k / (NS R)), r in [1, R), for its k = j mod NS, from a
// per-pass table built on the host in FP64, in blocks [s*NS + k], so the
// threads of a wave, which hold consecutive k, read consecutive entries.
// TW_POW stores only the base powers w^1, w^2, w^4, w^8 (those below R); the
// other powers are products of at most three of them: four loads instead of
// fifteen per radix-16 pass keep the twiddle traffic small next to the data
// streamed through the caches, where the table is long. TW_MIXED (the envelope
// rows) stores every power for passes of stride at most kFullStride, a table
// of a few KiB that stays in the L1 cache: each twiddle is then rounded once.
// With products in that pass too a row's FP32 error is 5 to 7% larger and its
// systematic part, a scale below 1, 34 to 52% (rel-L2 of 512 / 2048 / 4096
// points 1.12e-7 / 1.26e-7 / 1.35e-7 against 1.04e-7 / 1.19e-7 / 1.29e-7). As
// fifteen 8-byte loads it costs 3 to 10% of the rows (4096 values 498/577 us
// forward / inverse against 486/542), as eight 16-byte loads (FP32, tw_pairs)
// next to nothing: 472/561.
// Direction S = -1 computes sum_n a_n e^{-2 pi i nk/L}, S = +1 the
// unnormalised inverse kernel e^{+2 pi i nk/L} (conjugated twiddles).
// Arithmetic: twiddles and rotations are applied inside the butterflies' fused
// multiply-adds and LDS offsets are one address plus constants; against
// rounding each product first and one address per element this takes 733
// vector instructions in the 4096-point inverse rows kernel where it took 896,
// with slightly smaller errors. It bought 1 to 2.5% (256 x 131072 samples,
// three Q: 3.91 to 3.85 ms; 32 x 2^21: 4.25 to 4.16 ms): these kernels wait
// for memory and barriers as much as for the vector ALU.
#pragma once

#include <hip/hip_runtime.h>

#include "gmem.hpp"

namespace qtam {

template <typename T> struct Complex;
template <> struct Complex<float> { using type = float2; };
template <> struct Complex<double> { using type = double2; };

template <typename C> __device__ __forceinline__ C c_add(C a, C b) { return C{a.x + b.x, a.y + b.y}; }
template <typename C> __device__ __forceinline__ C c_sub(C a, C b) { return C{a.x - b.x, a.y - b.y}; }
template <typename C> __device__ __forceinline__ C c_conj(C a) { return C{a.x, -a.y}; }
// Fused multiply-add with the product and the addend chosen here, not by the
// compiler: every kernel instantiation then rounds the same way, so variants
// of one kernel (with or without row statistics, say) write identical bits.
__device__ __forceinline__ float fmadd(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__device__ __forceinline__ double fmadd(double a, double b, double c) { return __builtin_fma(a, b, c); }

template <typename C> __device__ __forceinline__ C c_mul(C a, C b) {
  return C{fmadd(a.x, b.x, -(a.y * b.y)), fmadd(a.x, b.y, a.y * b.x)};
}
// a * (S i): S = +1 multiplies by i, S = -1 by -i
template <int S, typename C> __device__ __forceinline__ C c_mul_si(C a) {
  if constexpr (S > 0) return C{-a.y, a.x};
  else return C{a.y, -a.x};
}

// acc + s v and acc + s (S i) v with a real scale s
template <typename C, typename T> __device__ __forceinline__ C c_fma_s(C acc, C v, T s) {
  return C{fmadd(v.x, s, acc.x), fmadd(v.y, s, acc.y)};
}
template <int S, typename C, typename T> __device__ __forceinline__ C c_fma_si(C acc, C v, T s) {
  constexpr T g = static_cast<T>(S);
  return C{fmadd(v.y, -g * s, acc.x), fmadd(v.x, g * s, acc.y)};
}
// acc + a w, and 2 q - t (t = q + p gives q - p: two fused multiply-adds for
// the second output of a butterfly whose product p was never formed)
template <typename C> __device__ __forceinline__ C c_fma(C acc, C a, C w) {
  return C{fmadd(a.x, w.x, fmadd(-a.y, w.y, acc.x)), fmadd(a.x, w.y, fmadd(a.y, w.x, acc.y))};
}
template <typename C> __device__ __forceinline__ C c_twice_minus(C q, C t) {
  using T = decltype(q.x);
  return C{fmadd(T(2), q.x, -t.x), fmadd(T(2), q.y, -t.y)};
}

// Rotations by exp(S 2 pi i k / 16) up to a real scale that the following
// butterfly applies in its fused multiply-adds: k = 2 and 6 with scale
// sqrt(1/2) (c_rot45, c_rot135), k = 1 with scale cos(pi/8) (c_rot22), k = 3
// with the same scale (c_rot67), k = 9 with its negative.
struct Root16 {
  static constexpr double c1 = 0.92387953251128675613;   // cos(pi/8)
  static constexpr double t1 = 0.41421356237309504880;   // tan(pi/8)
  static constexpr double r2 = 0.70710678118654752440;   // sqrt(1/2)
};
template <int S, typename C> __device__ __forceinline__ C c_rot45(C a) {
  if constexpr (S > 0) return C{a.x - a.y, a.y + a.x};
  else return C{a.x + a.y, a.y - a.x};
}
template <int S, typename C> __device__ __forceinline__ C c_rot135(C a) {
  if constexpr (S > 0) return C{-a.x - a.y, a.x - a.y};
  else return C{a.y - a.x, -a.x - a.y};
}
template <int S, typename C> __device__ __forceinline__ C c_rot22(C a) {
  using T = decltype(a.x);
  constexpr T t = static_cast<T>(S * Root16::t1);
  return C{fmadd(a.y, -t, a.x), fmadd(a.x, t, a.y)};
}
template <int S, typename C> __device__ __forceinline__ C c_rot67(C a) {
  using T = decltype(a.x);
  constexpr T t = static_cast<T>(Root16::t1);
  if constexpr (S > 0) return C{fmadd(a.x, t, -a.y), fmadd(a.y, t, a.x)};
  else return C{fmadd(a.x, t, a.y), fmadd(a.y, t, -a.x)};
}

template <int S, typename C>
__device__ __forceinline__ void dft2(C& a0, C& a1) {
  const C t = a0;
  a0 = c_add(t, a1);
  a1 = c_sub(t, a1);
}

template <int S, typename C>
__device__ __forceinline__ void dft4(C& a0, C& a1, C& a2, C& a3) {
  const C t0 = c_add(a0, a2), t1 = c_sub(a0, a2);
  const C t2 = c_add(a1, a3), t3 = c_mul_si<S>(c_sub(a1, a3));
  a0 = c_add(t0, t2);
  a2 = c_sub(t0, t2);
  a1 = c_add(t1, t3);
  a3 = c_sub(t1, t3);
}

// Length-4 DFT whose inputs 1..3 (or 0..3) still take their twiddles: the
// products go into the butterflies' fused multiply-adds, 24 (28) operations
// where multiplying first takes 28 (32).
template <int S, bool FIRST, typename C>
__device__ __forceinline__ void dft4_tw(C& a0, C& a1, C& a2, C& a3, C w0, C w1, C w2, C w3) {
  if constexpr (FIRST) a0 = c_mul(a0, w0);
  const C t0 = c_fma(a0, a2, w2), t1 = c_twice_minus(a0, t0);
  const C q = c_mul(a1, w1);
  const C t2 = c_fma(q, a3, w3), t3 = c_mul_si<S>(c_twice_minus(q, t2));
  a0 = c_add(t0, t2);
  a2 = c_sub(t0, t2);
  a1 = c_add(t1, t3);
  a3 = c_sub(t1, t3);
}

// Second half of a radix-16 DFT split as n = 4 n1 + n2: group n2's output
// k1 sits at a[4 k1 + n2]; twiddles exp(S 2 pi i n2 k1 / 16), then the outer
// length-4 DFTs over the groups, results in natural order. The rotations keep
// their scales for the last additions (80 operations; 96 when each product is
// rounded first).
template <int S, typename C>
__device__ __forceinline__ void dft16_outer(C* a) {
  using T = decltype(a[0].x);
  constexpr T c1 = static_cast<T>(Root16::c1), r2 = static_cast<T>(Root16::r2);
  C y[16];
  auto last = [&](int k1, C t0, C t1, C t2, C t3, T s) {   // t2, t3 up to the scale s
    y[k1] = c_fma_s(t0, t2, s);
    y[k1 + 8] = c_fma_s(t0, t2, -s);
    y[k1 + 4] = c_fma_si<S>(t1, t3, s);
    y[k1 + 12] = c_fma_si<S>(t1, t3, -s);
  };
  {
    C b0 = a[0], b1 = a[1], b2 = a[2], b3 = a[3];
    dft4<S>(b0, b1, b2, b3);
    y[0] = b0;
    y[4] = b1;
    y[8] = b2;
    y[12] = b3;
  }
  {
    const C u = c_rot45<S>(a[6]), p1 = c_rot22<S>(a[5]), p3 = c_rot67<S>(a[7]);
    last(1, c_fma_s(a[4], u, r2), c_fma_s(a[4], u, -r2), c_add(p1, p3), c_sub(p1, p3), c1);
  }
  {
    const C b2 = c_mul_si<S>(a[10]), u1 = c_rot45<S>(a[9]), u3 = c_rot135<S>(a[11]);
    last(2, c_add(a[8], b2), c_sub(a[8], b2), c_add(u1, u3), c_sub(u1, u3), r2);
  }
  {
    const C u = c_rot135<S>(a[14]), p1 = c_rot67<S>(a[13]), p3 = c_rot22<S>(a[15]);   // p3 with scale -c1
    last(3, c_fma_s(a[12], u, r2), c_fma_s(a[12], u, -r2), c_sub(p1, p3), c_add(p1, p3), c1);
  }
#pragma unroll
  for (int i = 0; i < 16; ++i) a[i] = y[i];
}

// Radix-16 DFT of inputs known to be zero except a[0], a[1], a[14], a[15]
// (NZ = 4) or a[0], a[15] (NZ = 2): the operations of dft_small<S, 16> on the
// non-zero terms only, in the same order, so the results are the same bits
// (up to the sign of zeros). Each inner length-4 DFT then has one non-zero
// input: at n1 = 0 it copies it to all four outputs; at n1 = 3 the outputs
// are x, S i (-x), -x, -(S i (-x)).
template <int S, int NZ, typename C>
__device__ __forceinline__ void dft16_sparse(C* a) {
  static_assert(NZ == 2 || NZ == 4, "two or four non-zero inputs");
  auto from_first = [&](int n2) {   // group n2 with its only input at n1 = 0
    a[n2 + 4] = a[n2];
    a[n2 + 8] = a[n2];
    a[n2 + 12] = a[n2];
  };
  auto from_last = [&](int n2) {    // group n2 with its only input at n1 = 3
    const C x = a[n2 + 12];
    const C r = c_mul_si<S>(C{-x.x, -x.y});
    a[n2] = x;
    a[n2 + 4] = r;
    a[n2 + 8] = C{-x.x, -x.y};
    a[n2 + 12] = C{-r.x, -r.y};
  };
  from_first(0);
  from_last(3);
  if constexpr (NZ == 4) {
    from_first(1);
    from_last(2);
    dft16_outer<S>(a);
  } else {
    // groups 1 and 2 are zero: each outer length-4 DFT sees (b0, 0, 0, b3)
    using T = decltype(a[0].x);
    constexpr T c1 = static_cast<T>(Root16::c1), r2 = static_cast<T>(Root16::r2);
    C y[16];
    auto last = [&](int k1, C b0, C p, T s) {   // b3 times its root = s p
      y[k1] = c_fma_s(b0, p, s);
      y[k1 + 8] = c_fma_s(b0, p, -s);
      y[k1 + 4] = c_fma_si<S>(b0, p, -s);
      y[k1 + 12] = c_fma_si<S>(b0, p, s);
    };
    last(0, a[0], a[3], T(1));
    last(1, a[4], c_rot67<S>(a[7]), c1);
    last(2, a[8], c_rot135<S>(a[11]), r2);
    last(3, a[12], c_rot22<S>(a[15]), -c1);
#pragma unroll
    for (int i = 0; i < 16; ++i) a[i] = y[i];
  }
}

// Second half of a radix-8 DFT split as n = 2 n1 + n2: group n2's output k1
// sits at a[2 k1 + n2].
template <int S, typename C>
__device__ __forceinline__ void dft8_outer(C* a) {
  using T = decltype(a[0].x);
  constexpr T r2 = static_cast<T>(Root16::r2);
  const C u1 = c_rot45<S>(a[3]), u2 = c_mul_si<S>(a[5]), u3 = c_rot135<S>(a[7]);
  const C y[8] = {c_add(a[0], a[1]),     c_fma_s(a[2], u1, r2),  c_add(a[4], u2), c_fma_s(a[6], u3, r2),
                  c_sub(a[0], a[1]),     c_fma_s(a[2], u1, -r2), c_sub(a[4], u2), c_fma_s(a[6], u3, -r2)};
#pragma unroll
  for (int i = 0; i < 8; ++i) a[i] = y[i];
}

// In-register DFT of R values in natural order (R in 1, 2, 4, 8, 16).
// R = 8 and 16 split as n = 4 n1 + n2 ... : inner radix-4 DFTs over strided
// groups, twiddles exp(S 2 pi i n2 k1 / R), outer DFTs over the groups.
template <int S, int R, typename C>
__device__ __forceinline__ void dft_small(C* a) {
  if constexpr (R == 1) {
  } else if constexpr (R == 2) {
    dft2<S>(a[0], a[1]);
  } else if constexpr (R == 4) {
    dft4<S>(a[0], a[1], a[2], a[3]);
  } else if constexpr (R == 8) {
    // n = 2 n1 + n2, k = k1 + 4 k2
    dft4<S>(a[0], a[2], a[4], a[6]);
    dft4<S>(a[1], a[3], a[5], a[7]);
    dft8_outer<S>(a);
  } else if constexpr (R == 16) {
    // n = 4 n1 + n2: group n2 holds a[n2], a[4+n2], a[8+n2], a[12+n2]
    dft4<S>(a[0], a[4], a[8], a[12]);
    dft4<S>(a[1], a[5], a[9], a[13]);
    dft4<S>(a[2], a[6], a[10], a[14]);
    dft4<S>(a[3], a[7], a[11], a[15]);
    dft16_outer<S>(a);
  }
}

// The same of a[r] w[r] (w[0] is 1 and not read).
template <int S, int R, typename C>
__device__ __forceinline__ void dft_small_tw(C* a, const C* w) {
  if constexpr (R == 2) {
    const C t = c_fma(a[0], a[1], w[1]);
    a[1] = c_twice_minus(a[0], t);
    a[0] = t;
  } else if constexpr (R == 4) {
    dft4_tw<S, false>(a[0], a[1], a[2], a[3], C{}, w[1], w[2], w[3]);
  } else if constexpr (R == 8) {
    dft4_tw<S, false>(a[0], a[2], a[4], a[6], C{}, w[2], w[4], w[6]);
    dft4_tw<S, true>(a[1], a[3], a[5], a[7], w[1], w[3], w[5], w[7]);
    dft8_outer<S>(a);
  } else {
    static_assert(R == 16, "radices 2, 4, 8, 16");
    dft4_tw<S, false>(a[0], a[4], a[8], a[12], C{}, w[4], w[8], w[12]);
    dft4_tw<S, true>(a[1], a[5], a[9], a[13], w[1], w[5], w[9], w[13]);
    dft4_tw<S, true>(a[2], a[6], a[10], a[14], w[2], w[6], w[10], w[14]);
    dft4_tw<S, true>(a[3], a[7], a[11], a[15], w[3], w[7], w[11], w[15]);
    dft16_outer<S>(a);
  }
}

// LDS index with one pad element every 32, which spreads power-of-two strides
// over the banks; the map is affine inside each run of 32, so exchanges keep
// constant instruction offsets.
__device__ __forceinline__ int lds_pad(int i) { return i + (i >> 5); }
constexpr int lds_size(int l) { return l + l / 32 + 1; }
// lds_pad(i + c) for a c that shares no bit with i: lds_pad(i) plus a constant
constexpr int lds_step(int c) { return c + (c >> 5); }

// Twiddle tables of the passes (see above).
enum TwiddleMode { TW_POW = 0, TW_MIXED = 1 };
constexpr int kFullStride = 16;
constexpr bool tw_full_pass(int mode, int ns) { return mode == TW_MIXED && ns <= kFullStride; }
// FP32 tables hold the powers of such a pass as pairs (w^r, w^(r+1)), r odd, in
// blocks [r/2 * NS + k]: 16 bytes a load, eight loads instead of fifteen.
template <typename T> constexpr bool tw_pairs() { return sizeof(T) == 4; }

// LDS a transform of length L needs: the padded exchange region, or half of
// it when the whole one would not fit the 160 KiB of a workgroup (the
// exchanges then go in two rounds, one per half of the destination indices).
template <typename T, int L>
constexpr bool fft_split() {
  return size_t(lds_size(L)) * sizeof(typename Complex<T>::type) > 160u * 1024u;
}
template <typename T, int L>
constexpr int fft_lds_elems() {
  return fft_split<T, L>() ? lds_size(L / 2) : lds_size(L);
}

// RM: largest butterfly; E = 2 RM holds two groups. HALF: the exchanges in two
// rounds over half the region although the whole would fit (so that more rows
// are resident on a CU).
template <typename T, int L, int E, int S, int TW = TW_POW, int RM = (E < 16 ? E : 16), bool HALF = false>
struct BlockFft {
  using C = typename Complex<T>::type;
  static_assert((L & (L - 1)) == 0 && (E & (E - 1)) == 0 && E <= L && E <= 2 * RM, "pow2 sizes");
  static constexpr int TPR = L / E;
  static constexpr int RMAX = RM;
  static constexpr int radix(int ns) { return (L / ns >= RMAX) ? RMAX : L / ns; }
  static constexpr bool SPLIT = HALF || fft_split<T, L>();
  static constexpr int WN = E > RMAX ? RMAX : E;   // twiddle registers: one group at a time when E > RMAX
  static constexpr int last_ns() {
    int ns = 1;
    while (ns * radix(ns) < L) ns *= radix(ns);
    return ns;
  }
  static constexpr int R0 = radix(1);
  static constexpr int RL = radix(last_ns());
  // number of stored powers of the radix-r pass of stride ns: w^(2^s) < r, or
  // all w^s, s < r (FP32: in pairs, one more)
  static constexpr int slots(int r, int ns) {
    return tw_full_pass(TW, ns) ? (tw_pairs<T>() ? r : r - 1) : r >= 16 ? 4 : r >= 8 ? 3 : r >= 4 ? 2 : r >= 2 ? 1 : 0;
  }
  // start of the twiddle block of the pass with stride ns
  static constexpr int tw_offset(int ns) {
    int off = 0, n = 1;
    while (n < ns) {
      if (n > 1) off += slots(radix(n), n) * n;
      n *= radix(n);
    }
    return off;
  }
  static constexpr int tw_size() { return tw_offset(L); }
  // registers of a radix-R2 pass whose input index lies below L/2
  static constexpr int lower_reads(int r2) {
    int n = 0;
    for (int q = 0; q < E / r2; ++q)
      for (int r = 0; r < r2; ++r) n += (q * TPR + r * (L / r2) < L / 2) ? 1 : 0;
    return n;
  }

  __device__ static __forceinline__ int in_index(int tl, int i) {
    return tl + (i / R0) * TPR + (i % R0) * (L / R0);
  }
  __device__ static __forceinline__ int out_index(int tl, int i) {
    return tl + (i / RL) * TPR + (i % RL) * (L / RL);
  }

  // Twiddles of the pass with stride NS for this thread: w[q*R + r], r >= 1,
  // read, or formed from the base powers w^1, w^2, w^4, w^8 (groups q0 .. q1-1, stored from
  // w[0] on when only one group is held at a time).
  template <int NS>
  __device__ static __forceinline__ void load_twiddles(C (&w)[WN], int tl, rsrc_t tw, int q0 = 0,
                                                       int q1 = E / radix(NS)) {
    constexpr int R = radix(NS);
#pragma unroll
    for (int q = q0; q < q1; ++q) {
      const uint32_t k = static_cast<uint32_t>((tl + q * TPR) & (NS - 1));
      if constexpr (tw_full_pass(TW, NS) && tw_pairs<T>()) {
#pragma unroll
        for (int r = 1; r < R; r += 2) {
          const float4 p = bload<float4>(tw, k * 2 * sizeof(C), (tw_offset(NS) + (r - 1) * NS) * sizeof(C));
          w[(q - q0) * R + r] = C{p.x, p.y};
          if (r + 1 < R) w[(q - q0) * R + r + 1] = C{p.z, p.w};
        }
      } else if constexpr (tw_full_pass(TW, NS)) {
#pragma unroll
        for (int r = 1; r < R; ++r)
          w[(q - q0) * R + r] = bload<C>(tw, k * sizeof(C), (tw_offset(NS) + (r - 1) * NS) * sizeof(C));
      } else {
        C a[16];
#pragma unroll
        for (int sl = 0; sl < slots(R, NS); ++sl)
          a[1 << sl] = bload<C>(tw, k * sizeof(C), (tw_offset(NS) + sl * NS) * sizeof(C));
        if constexpr (R > 2) a[3] = c_mul(a[2], a[1]);
        if constexpr (R > 4) {
          a[5] = c_mul(a[4], a[1]);
          a[6] = c_mul(a[4], a[2]);
          a[7] = c_mul(a[4], a[3]);
        }
        if constexpr (R > 8) {
#pragma unroll
          for (int r = 9; r < 16; ++r) a[r] = c_mul(a[8], a[r - 8]);
        }
#pragma unroll
        for (int r = 1; r < R; ++r) w[(q - q0) * R + r] = a[r];
      }
    }
  }

  // One radix-R pass on registers: for NS > 1 its twiddles are read and
  // applied, then the butterflies; unless it was the last pass the values
  // are exchanged through LDS into the next pass's order.
  template <int NS>
  __device__ static __forceinline__ void pass(C (&v)[E], C (&w)[WN], C* lds, int tl, rsrc_t tw, int nz) {
    constexpr int R = radix(NS);
    constexpr bool kAll = WN == E;   // all groups' twiddles at once, else one group at a time
    if constexpr (NS > 1 && kAll) load_twiddles<NS>(w, tl, tw);
#pragma unroll
    for (int q = 0; q < E / R; ++q) {
      if constexpr (NS > 1) {
        if constexpr (!kAll) load_twiddles<NS>(w, tl, tw, q, q + 1);
        C t[R];
#pragma unroll
        for (int r = 1; r < R; ++r) {
          t[r] = w[(kAll ? q * R : 0) + r];
          if constexpr (S > 0) t[r].y = -t[r].y;
        }
        dft_small_tw<S, R>(&v[q * R], t);
      } else if constexpr (R == 16) {
        if (nz == 2) dft16_sparse<S, 2>(&v[q * R]);
        else if (nz == 4) dft16_sparse<S, 4>(&v[q * R]);
        else dft_small<S, R>(&v[q * R]);
      } else {
        dft_small<S, R>(&v[q * R]);
      }
    }
    if constexpr (NS * R < L) {
      constexpr int NS2 = NS * R;
      constexpr int R2 = radix(NS2);
      if constexpr (!SPLIT) {
#pragma unroll
        for (int q = 0; q < E / R; ++q) {
          const int j = tl + q * TPR;
          const int k = j & (NS - 1);
          const int base = lds_pad((j - k) * R + k);   // no bit of r NS set
#pragma unroll
          for (int r = 0; r < R; ++r) lds[base + lds_step(r * NS)] = v[q * R + r];
        }
        __syncthreads();
#pragma unroll
        for (int q = 0; q < E / R2; ++q) {
          const int j = lds_pad(tl) + lds_step(q * TPR);   // tl < TPR, tl + q TPR < L / R2
#pragma unroll
          for (int r = 0; r < R2; ++r) v[q * R2 + r] = lds[j + lds_step(r * (L / R2))];
        }
        __syncthreads();
      } else {
        // The LDS region holds half of the indices. With two register groups
        // per pass (E = 2R) and NS dividing TPR, group 0 holds exactly the
        // values bound for indices below L/2 and group 1 the others, and a
        // value bound for register (q, r) of the next pass comes from below
        // L/2 iff q TPR + r L/R2 < L/2 (tl < TPR; both terms are multiples of
        // TPR). Round 0 moves the lower half (into tmp, since the registers it
        // fills may still hold group-1 values), round 1 the upper half.
        static_assert(E / R == 2 && TPR % NS == 0 && lower_reads(R2) == E / 2, "split exchange layout");
        constexpr int H = L / 2;
        C tmp[E / 2];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          {
            const int j = tl + h * TPR;
            const int k = j & (NS - 1);
            const int base = lds_pad((j - k) * R + k - h * H);
#pragma unroll
            for (int r = 0; r < R; ++r) lds[base + lds_step(r * NS)] = v[h * R + r];
          }
          __syncthreads();
          int n = 0;
#pragma unroll
          for (int q = 0; q < E / R2; ++q) {
#pragma unroll
            for (int r = 0; r < R2; ++r) {
              const int off = q * TPR + r * (L / R2);   // compile-time after unrolling
              if ((off < H) == (h == 0)) {
                const C x = lds[lds_pad(tl) + lds_step(off - h * H)];
                if (h == 0) tmp[n++] = x;
                else v[q * R2 + r] = x;
              }
            }
          }
          __syncthreads();
        }
        int n = 0;
#pragma unroll
        for (int q = 0; q < E / R2; ++q) {
#pragma unroll
          for (int r = 0; r < R2; ++r) {
            if (q * TPR + r * (L / R2) < H) v[q * R2 + r] = tmp[n++];
          }
        }
      }
      pass<NS2>(v, w, lds, tl, tw, 0);
    }
  }

  // Every thread of the workgroup must call run (it contains barriers).
  // tw: buffer resource over the per-pass twiddle table of this (L, E).
  // nz = 2 or 4 (wave-uniform) when the first pass is radix 16 and each of
  // the wave's first-pass groups is zero except v[0] and v[15] (2), or except
  // v[0], v[1], v[14], v[15] (4): that pass then skips the zero terms, with
  // the same results; any other value runs the full transform.
  __device__ static __forceinline__ void run(C (&v)[E], C* lds, int tl, rsrc_t tw, int nz = 0) {
    C w[WN];
    pass<1>(v, w, lds, tl, tw, nz);
  }
  // offsets of register element i from the thread's own index tl
  static constexpr int in_off(int i) { return (i / R0) * TPR + (i % R0) * (L / R0); }
  static constexpr int out_off(int i) { return (i / RL) * TPR + (i % RL) * (L / RL); }
  __device__ static __forceinline__ rsrc_t twiddles(const C* tw) {
    return make_rsrc(tw, static_cast<uint32_t>((tw_size() > 0 ? tw_size() : 1) * sizeof(C)));
  }
};

}  // namespace qtam
