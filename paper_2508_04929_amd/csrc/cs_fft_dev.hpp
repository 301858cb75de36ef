// Device code of the FFT passes: Stockham transforms of compile-time length
// whose butterflies (up to 16 points) live in registers.
//
// A transform of length L = R0 R1 R2 runs as one pass per factor; between two
// passes the values cross LDS once.  A team of TS threads shares a transform;
// in a pass of radix R thread t takes the butterflies j = t, t + TS, ...
// < L / R: inputs j + i L / R, outputs (j / Ns) Ns R + j % Ns + i Ns (i < R, Ns
// the product of the earlier radices).  The last pass has Ns = L / R, so it
// leaves the outputs where a first pass of the same radix wants its inputs: a
// transform back, with the radices in reverse order, starts from the same
// registers.  HBM-bound at large batches: for 256 images of 128^2 the CTF column
// pass takes 13 us (34 MB, 2.6 TB/s) and the loss row pass 18 us; with radices of
// 4 and less at run-time strides, one LDS round trip and barrier each, and
// columns read in 32-byte pieces they took 34 and 34 us.  An axis of a 256^3
// volume: 24 and 41 us (z, y; 135 MB) against 85.
#pragma once

#include "cs_internal.hpp"

namespace cs {

// Radices and team size of each supported length (even, prime factors 2 and
// 3, up to 512): two passes where factors up to 16 allow, three otherwise.
template <int R0_, int R1_, int R2_, int TS_>
struct FftRadices {
  static constexpr int R0 = R0_, R1 = R1_, R2 = R2_, L = R0_ * R1_ * R2_, TS = TS_;
  typedef FftRadices<R1_ == 1 ? R0_ : R2_ == 1 ? R1_ : R2_, R1_ == 1 ? 1 : R2_ == 1 ? R0_ : R1_,
                     R2_ == 1 ? 1 : R0_, TS_> Reverse;
};

#define CS_FFT_LENGTHS(X)                                                          \
  X(2, 2, 1, 1, 1) X(4, 2, 2, 1, 2) X(6, 3, 2, 1, 3) X(8, 4, 2, 1, 2)              \
  X(12, 4, 3, 1, 4) X(16, 4, 4, 1, 4) X(18, 6, 3, 1, 6) X(24, 6, 4, 1, 6)          \
  X(32, 8, 4, 1, 8) X(36, 6, 6, 1, 6) X(48, 8, 6, 1, 8) X(54, 9, 6, 1, 9)          \
  X(64, 8, 8, 1, 8) X(72, 9, 8, 1, 9) X(96, 12, 8, 1, 12) X(108, 12, 9, 1, 12)     \
  X(128, 16, 8, 1, 8) X(144, 12, 12, 1, 12) X(162, 9, 9, 2, 18)                   \
  X(192, 16, 12, 1, 16) X(216, 9, 8, 3, 27) X(256, 16, 16, 1, 16)                  \
  X(288, 8, 6, 6, 48) X(324, 9, 6, 6, 54) X(384, 8, 8, 6, 64) X(432, 9, 8, 6, 72)  \
  X(486, 9, 9, 6, 81) X(512, 8, 8, 8, 64)

__device__ __forceinline__ float2 cmul(float2 a, float2 b) {
  return make_float2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
__device__ __forceinline__ float2 cadd(float2 a, float2 b) { return make_float2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ float2 csub(float2 a, float2 b) { return make_float2(a.x - b.x, a.y - b.y); }
// a times -i (forward) or +i (inverse)
template <bool INV>
__device__ __forceinline__ float2 crot(float2 a) {
  return INV ? make_float2(-a.y, a.x) : make_float2(a.y, -a.x);
}

// exp(-+ 2 pi i k / n) for the points inside a butterfly (n = 6, 8, 9, 12, 16)
template <bool INV>
__device__ __forceinline__ float2 cunit(int k, int n) {
  constexpr float c9[9] = {1.f, 0.76604444311897804f, 0.17364817766693035f, -0.5f, -0.93969262078590838f,
                           -0.93969262078590838f, -0.5f, 0.17364817766693035f, 0.76604444311897804f};
  constexpr float s9[9] = {0.f, 0.64278760968653933f, 0.98480775301220806f, 0.86602540378443865f,
                           0.34202014332566873f, -0.34202014332566873f, -0.86602540378443865f,
                           -0.98480775301220806f, -0.64278760968653933f};
  constexpr float c16[16] = {1.f, 0.92387953251128674f, 0.70710678118654752f, 0.38268343236508977f,
                             0.f, -0.38268343236508977f, -0.70710678118654752f, -0.92387953251128674f,
                             -1.f, -0.92387953251128674f, -0.70710678118654752f, -0.38268343236508977f,
                             0.f, 0.38268343236508977f, 0.70710678118654752f, 0.92387953251128674f};
  constexpr float c12[12] = {1.f, 0.86602540378443865f, 0.5f, 0.f, -0.5f, -0.86602540378443865f,
                             -1.f, -0.86602540378443865f, -0.5f, 0.f, 0.5f, 0.86602540378443865f};
  float c, s;
  if (n == 9) {
    c = c9[k % 9];
    s = s9[k % 9];
  } else if (n == 12 || n == 6) {
    const int q = k * (12 / n) % 12;
    c = c12[q];
    s = c12[(q + 9) % 12];
  } else {
    const int q = k * (16 / n) % 16;
    c = c16[q];
    s = c16[(q + 12) % 16];
  }
  return make_float2(c, INV ? s : -s);
}

// R-point transforms in registers, outputs in natural order.
template <int R, bool INV>
__device__ __forceinline__ void dft(float2 *v) {
  if constexpr (R == 2) {
    const float2 a = v[0];
    v[0] = cadd(a, v[1]);
    v[1] = csub(a, v[1]);
  } else if constexpr (R == 3) {
    const float c3 = 0.86602540378443865f;  // sqrt(3) / 2
    const float2 s = cadd(v[1], v[2]), d = crot<INV>(csub(v[1], v[2]));
    const float2 m = make_float2(v[0].x - 0.5f * s.x, v[0].y - 0.5f * s.y);
    v[0] = cadd(v[0], s);
    v[1] = make_float2(m.x + c3 * d.x, m.y + c3 * d.y);
    v[2] = make_float2(m.x - c3 * d.x, m.y - c3 * d.y);
  } else if constexpr (R == 4) {
    const float2 a0 = cadd(v[0], v[2]), a1 = csub(v[0], v[2]);
    const float2 a2 = cadd(v[1], v[3]), a3 = crot<INV>(csub(v[1], v[3]));
    v[0] = cadd(a0, a2);
    v[1] = cadd(a1, a3);
    v[2] = csub(a0, a2);
    v[3] = csub(a1, a3);
  } else {
    // R = A B: B transforms of A points over stride B, twiddles, A of B points
    constexpr int A = R == 9 || R == 6 ? 3 : 4, B = R / A;
    float2 u[B][A];
#pragma unroll
    for (int b = 0; b < B; ++b) {
#pragma unroll
      for (int a = 0; a < A; ++a) u[b][a] = v[b + B * a];
      dft<A, INV>(u[b]);
#pragma unroll
      for (int a = 1; a < A; ++a)
        if (b) u[b][a] = 4 * a * b == R ? crot<INV>(u[b][a]) : cmul(u[b][a], cunit<INV>(a * b, R));
    }
#pragma unroll
    for (int a = 0; a < A; ++a) {
      float2 w[B];
#pragma unroll
      for (int b = 0; b < B; ++b) w[b] = u[b][a];
      dft<B, INV>(w);
#pragma unroll
      for (int b = 0; b < B; ++b) v[a + A * b] = w[b];
    }
  }
}

// The values of a pass of radix R that a thread holds: v[m][i] of butterfly
// j = t + m TS.
template <class P, int R>
struct FftVals {
  static constexpr int kJ = P::L / R, kN = (kJ + P::TS - 1) / P::TS;
  float2 v[kN][R];
  template <class F>
  __device__ __forceinline__ void inputs(int t, F f) {  // v = f(j + i L / R)
#pragma unroll
    for (int m = 0; m < kN; ++m) {
      const int j = t + m * P::TS;
      const bool in = kJ % P::TS == 0 || j < kJ;
#pragma unroll
      for (int i = 0; i < R; ++i) v[m][i] = in ? f(j + i * kJ) : make_float2(0.f, 0.f);
    }
  }
  template <int Ns, class F>
  __device__ __forceinline__ void outputs(int t, F f) {  // f(output index, value)
#pragma unroll
    for (int m = 0; m < kN; ++m) {
      const int j = t + m * P::TS;
      if (kJ % P::TS != 0 && j >= kJ) continue;
      const int base = (j / Ns) * Ns * R + j % Ns;
#pragma unroll
      for (int i = 0; i < R; ++i) f(base + i * Ns, v[m][i]);
    }
  }
  // twiddles after earlier passes of Ns points (tw[k] = exp(-2 pi i k / L)) ...
  struct Twiddles {
    float2 w[kN][R];
  };
  template <int Ns>
  static __device__ __forceinline__ Twiddles twiddles(int t, const float2 *tw) {
    Twiddles w;
#pragma unroll
    for (int m = 0; m < kN; ++m) {
      const int j = t + m * P::TS;
      const int k = (kJ % P::TS == 0 || j < kJ) ? j % Ns : 0;
#pragma unroll
      for (int i = 1; i < R; ++i) w.w[m][i] = tw[i * k * (P::L / (Ns * R))];
    }
    return w;
  }
  template <bool INV>
  __device__ __forceinline__ void twist(const Twiddles &w) {
#pragma unroll
    for (int m = 0; m < kN; ++m)
#pragma unroll
      for (int i = 1; i < R; ++i)
        v[m][i] = cmul(v[m][i], INV ? make_float2(w.w[m][i].x, -w.w[m][i].y) : w.w[m][i]);
  }
  // ... and the butterflies
  template <bool INV>
  __device__ __forceinline__ void butterflies() {
#pragma unroll
    for (int m = 0; m < kN; ++m) dft<R, INV>(v[m]);
  }
};

// Place of value q of a transform in LDS: one more every R0, so that the
// writes of a first pass (stride R0) spread over the banks.
template <class P>
__device__ __forceinline__ int fft_place(int q) {
  return q + q / P::R0;
}
template <class P>
constexpr int fft_places() {
  return P::L + (P::L + P::R0 - 1) / P::R0;
}

template <class P>
struct FftLast {
  static constexpr int R = P::R1 == 1 ? P::R0 : P::R2 == 1 ? P::R1 : P::R2;
  typedef FftVals<P, R> Vals;
};

// From the first pass's inputs to the last pass's values (outputs k + i L / R,
// R the last radix).  at(q): the LDS slot of value q of this transform.  The
// slots must be free; every thread of the block calls this.
template <class P, bool INV, class At>
__device__ __forceinline__ typename FftLast<P>::Vals fft_run(FftVals<P, P::R0> &a, int t, const float2 *tw,
                                                            At at) {
  if constexpr (P::R1 == 1) {
    a.template butterflies<INV>();
    return a;
  } else {
    // the twiddles are requested before the barriers that their use follows
    const auto wb = FftVals<P, P::R1>::template twiddles<P::R0>(t, tw);
    a.template butterflies<INV>();
    a.template outputs<1>(t, [&](int q, float2 z) { at(q) = z; });
    __syncthreads();
    FftVals<P, P::R1> b;
    b.inputs(t, [&](int q) { return at(q); });
    b.template twist<INV>(wb);
    if constexpr (P::R2 == 1) {
      b.template butterflies<INV>();
      return b;
    } else {
      const auto wc = FftVals<P, P::R2>::template twiddles<P::R0 * P::R1>(t, tw);
      b.template butterflies<INV>();
      __syncthreads();
      b.template outputs<P::R0>(t, [&](int q, float2 z) { at(q) = z; });
      __syncthreads();
      FftVals<P, P::R2> c;
      c.inputs(t, [&](int q) { return at(q); });
      c.template twist<INV>(wc);
      c.template butterflies<INV>();
      return c;
    }
  }
}

// The same values as the first pass of the transform in reverse order.
template <class P>
__device__ __forceinline__ FftVals<typename P::Reverse, P::Reverse::R0> fft_turn(
    const typename FftLast<P>::Vals &r) {
  typedef FftVals<typename P::Reverse, P::Reverse::R0> V;
  static_assert(P::Reverse::R0 == FftLast<P>::R, "same layout");
  V a;
#pragma unroll
  for (int m = 0; m < V::kN; ++m)
#pragma unroll
    for (int i = 0; i < P::Reverse::R0; ++i) a.v[m][i] = r.v[m][i];
  return a;
}

// LDS values that a transform (and its way back) needs.
template <class P>
constexpr int fft_slots() {
  return fft_places<P>() > fft_places<typename P::Reverse>() ? fft_places<P>()
                                                             : fft_places<typename P::Reverse>();
}

}  // namespace cs
