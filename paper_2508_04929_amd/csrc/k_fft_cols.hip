// FFT passes over columns (axes that are not contiguous): the CTF application,
// the Fourier shift, and the y and z axes of a volume.
//
// A block takes CPW adjacent columns, thread c + CPW t being thread t of column
// c's team: a wave reads and writes CPW x 8 consecutive bytes of a row (whole
// 128-byte lines at 16), and so it does in LDS.  The transform, the multiplier
// and the transform back stay in registers but for one or two crossings of LDS
// each way.
#include <algorithm>

#include "cs_fft_dev.hpp"

namespace cs {

// Column group of this block: the grid is (column groups, images) and the
// XCD-aware order keeps an image's adjacent column groups on one XCD.
__device__ __forceinline__ void cols_block(int &b, int &group) {
  const int j = xcd_work(blockIdx.x + gridDim.x * blockIdx.y, gridDim.x * gridDim.y);
  b = j / gridDim.x;
  group = j % gridDim.x;
}

// Columns kx of an array [L][stride], `n` of them: inputs of a forward transform.
template <class P, int CPW>
struct ColTeam {
  int c, t, kx;
  bool valid;
  __device__ ColTeam(int group, int n) {
    c = threadIdx.x % CPW;
    t = threadIdx.x / CPW;
    kx = group * CPW + c;
    valid = kx < n;
  }
  __device__ typename FftLast<P>::Vals forward(const float2 *col, size_t stride, const float2 *tw,
                                               float2 *lds) const {
    FftVals<P, P::R0> a;
    a.inputs(t, [&](int q) { return valid ? col[(size_t)q * stride] : make_float2(0.f, 0.f); });
    return fft_run<P, false>(a, t, tw, [&](int q) -> float2 & { return lds[fft_place<P>(q) * CPW + c]; });
  }
  // times mul(index, value) and back, in place
  template <class Mul>
  __device__ void apply(float2 *col, size_t stride, const float2 *tw, float2 *lds, const Mul &mul) const {
    typedef typename P::Reverse Rev;
    auto z = forward(col, stride, tw, lds);
    if (valid) {
#pragma unroll
      for (int m = 0; m < z.kN; ++m) {
        const int j = t + m * P::TS;
        if (z.kJ % P::TS != 0 && j >= z.kJ) continue;
#pragma unroll
        for (int i = 0; i < FftLast<P>::R; ++i) z.v[m][i] = mul(j + i * z.kJ, z.v[m][i]);
      }
    }
    __syncthreads();
    FftVals<Rev, Rev::R0> a = fft_turn<P>(z);
    auto o = fft_run<Rev, true>(a, t, tw, [&](int q) -> float2 & { return lds[fft_place<Rev>(q) * CPW + c]; });
    if (valid)
      o.template outputs<P::L / FftLast<Rev>::R>(t, [&](int q, float2 v) { col[(size_t)q * stride] = v; });
  }
};

// times the table H^ / D^2 (Eq. 14)
template <class P, int CPW>
__global__ void __launch_bounds__(CPW * P::TS)
k_cols_ctf(float2 *spec, const float2 *tw, const float *table) {
  extern __shared__ float2 lds[];
  constexpr int L = P::L, Dh = L / 2 + 1;
  int b, group;
  cols_block(b, group);
  const ColTeam<P, CPW> w(group, Dh);
  const float *hcol = table + (size_t)b * L * Dh + w.kx;
  w.apply(spec + (size_t)b * L * Dh + w.kx, Dh, tw, lds, [&](int ky, float2 z) {
    const float h = hcol[(size_t)ky * Dh];
    return make_float2(z.x * h, z.y * h);
  });
}

// Translation of image b by (a_c, a_r) = (sign t_x / p, -sign t_y / p)
// columns / rows (the row axis is y-flipped, Eq. 13): times
// exp(-2 pi i (kx a_c + ky a_r) / L) / L^2 with signed frequency indices,
// made Hermitian on the Nyquist lines of even L (the real part of the
// complex inverse transform): cos(pi a) there in place of the exponential,
// cos(pi (a_c + a_r)) at the corner.  Turns in FP64, one FP32 sincos.
template <class P, int CPW>
__global__ void __launch_bounds__(CPW * P::TS)
k_cols_shift(float2 *spec, const float2 *tw, const float *shift, float inv_pixel, float sign) {
  extern __shared__ float2 lds[];
  constexpr int L = P::L, Dh = L / 2 + 1;
  int b, group;
  cols_block(b, group);
  const ColTeam<P, CPW> w(group, Dh);
  const int kx = w.kx;
  const double ac = (double)(sign * shift[2 * b] * inv_pixel);
  const double ar = -(double)(sign * shift[2 * b + 1] * inv_pixel);
  const bool even = (L % 2) == 0;
  const int half = L / 2;
  const float norm = 1.f / ((float)L * (float)L);
  // the cosines of the Nyquist lines, once per thread: a copy of that code per
  // value kept small launches waiting for instructions (one image of 256 x 256
  // 20.9 us, now 17.0; 64 images 46.8 and 40.6)
  const bool nx = even && kx == half;
  const double amp_x = nx ? cos(M_PI * ac) : 1.0;              // rows but the Nyquist one
  const double amp_y = cos(nx ? M_PI * (ac + ar) : M_PI * ar);  // the Nyquist row
  w.apply(spec + (size_t)b * L * Dh + kx, Dh, tw, lds, [&](int ky, float2 z) {
    const bool ny = even && ky == half;
    const int fy = ky < (L + 1) / 2 ? ky : ky - L;
    const double amp = ny ? amp_y : amp_x;
    const double turns = nx && ny ? 0.0
                         : nx     ? -(double)fy * ar / L
                         : ny     ? -(double)kx * ac / L
                                  : -((double)kx * ac + (double)fy * ar) / L;
    const float red = (float)((turns - rint(turns)) * (2.0 * M_PI));
    float sn, cs;
    sincosf(red, &sn, &cs);
    const float m = (float)amp * norm;
    const float re = cs * m, im = sn * m;
    return make_float2(z.x * re - z.y * im, z.x * im + z.y * re);
  });
}

// Forward transform along the middle axis of data[outer][L][inner]
// (complex, in place), outer index = blockIdx.y: the y and z passes of the 3-D
// transform of a volume.
template <class P, int CPW>
__global__ void __launch_bounds__(CPW * P::TS)
k_axis(float2 *data, const float2 *tw, int inner) {
  extern __shared__ float2 lds[];
  const ColTeam<P, CPW> w(blockIdx.x, inner);
  float2 *col = data + (size_t)blockIdx.y * P::L * inner + w.kx;
  auto z = w.forward(col, inner, tw, lds);
  if (w.valid)
    z.template outputs<P::L / FftLast<P>::R>(w.t, [&](int q, float2 v) { col[(size_t)q * inner] = v; });
}

// Columns per block: 16 (a 128-byte line) up to 256 points, 8 above, 4 where
// the launch asks for small blocks.
constexpr int wide_cols(int L) { return L <= 256 ? 16 : 8; }

#define X(N, A, B, C, T) \
  case N: return narrow ? &k_cols_ctf<FftRadices<A, B, C, T>, 4> : &k_cols_ctf<FftRadices<A, B, C, T>, wide_cols(N)>;
ColsCtfFn fft_cols_ctf(int L, bool narrow) {
  switch (L) { CS_FFT_LENGTHS(X) }
  return nullptr;
}
#undef X
#define X(N, A, B, C, T) \
  case N: return narrow ? &k_cols_shift<FftRadices<A, B, C, T>, 4> : &k_cols_shift<FftRadices<A, B, C, T>, wide_cols(N)>;
ColsShiftFn fft_cols_shift(int L, bool narrow) {
  switch (L) { CS_FFT_LENGTHS(X) }
  return nullptr;
}
#undef X
#define X(N, A, B, C, T) \
  case N: return &k_axis<FftRadices<A, B, C, T>, wide_cols(N)>;
AxisFn fft_axis(int L) {
  switch (L) { CS_FFT_LENGTHS(X) }
  return nullptr;
}
#undef X
FftLaunch fft_rows_launch(int L, int64_t B) {
  // teams of 256 threads' worth of row pairs per block, of 64 where a small
  // batch would fill fewer than two blocks per CU
  const FftShape s = fft_shape(L);
  int teams = std::max(1, 256 / s.ts);
  if ((int64_t)((L / 2 + teams - 1) / teams) * B < 512) teams = std::max(1, 64 / s.ts);
  return FftLaunch{dim3((L / 2 + teams - 1) / teams, (unsigned)B), dim3(teams * s.ts),
                   (size_t)teams * s.slots * sizeof(float2), false};
}

FftLaunch fft_cols_launch(int L, int64_t columns, int64_t B, bool may_narrow) {
  const FftShape s = fft_shape(L);
  int cpw = wide_cols(L);
  const bool narrow = may_narrow && (columns + cpw - 1) / cpw * B < 256;
  if (narrow) cpw = 4;
  return FftLaunch{dim3((unsigned)((columns + cpw - 1) / cpw), (unsigned)B), dim3(cpw * s.ts),
                   (size_t)cpw * s.slots * sizeof(float2), narrow};
}

}  // namespace cs
