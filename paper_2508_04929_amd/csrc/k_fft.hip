// Fourier-space CTF application, loss and adjoint (App. A.2, Eq. 14; Sec. 3.3.5).
//
// X = F^-1(H^ . F(Q)) is computed as
//   rows:     real FFT of every row (two rows packed as one complex FFT)
//   columns:  for each of the D/2+1 half-spectrum columns: FFT over rows,
//             times H^ (real) and the 1/D^2 normalisation, inverse FFT over
//             rows
//   rows:     inverse real FFT of every row (two rows packed again)
// with twiddles from an FP64-accurate table (k_twiddles).  Because H^ is real
// and even, the same column pass is its own adjoint, so the loss gradient
// G_Q = F^-1(H^ . F(G_X)) reuses the three passes; the row pass between the
// two applications fuses the inverse rows of X, the residual X - Y, the
// squared-error partial sums and the forward rows of G_X.  The transforms
// themselves are those of cs_fft_dev.hpp; the passes over rows are here, those
// over columns in k_fft_cols.hip.
#include "cs_ctf_dev.hpp"
#include "cs_fft_dev.hpp"

namespace cs {

FftShape fft_shape(int L) {
  FftShape s;
  switch (L) {
#define X(N, A, B, C, T)                                \
  case N:                                               \
    s.ts = T;                                           \
    s.slots = fft_slots<FftRadices<A, B, C, T>>();      \
    break;
    CS_FFT_LENGTHS(X)
#undef X
  }
  return s;
}

// Twiddle table of one transform length: tw[k] = exp(-2 pi i k / L),
// evaluated in FP64 and rounded once to FP32.
__global__ void __launch_bounds__(256) k_twiddles(int L, float2 *tw) {
  const int k = blockIdx.x * 256 + threadIdx.x;
  if (k >= L) return;
  double sn, cn;
  sincospi(2.0 * (double)k / (double)L, &sn, &cn);
  tw[k] = make_float2((float)cn, (float)-sn);
}

// ---------------------------------------------------------------------------
// Row kernels: one team of TS threads per row pair, blockDim.x / TS teams per
// block (the host picks fewer for small batches).
// ---------------------------------------------------------------------------
template <class P>
struct RowTeam {
  int t, pr;          // thread of the team, row pair
  bool valid;
  float2 *slot;       // the team's LDS
  __device__ RowTeam(float2 *lds) {
    const int team = threadIdx.x / P::TS;
    t = threadIdx.x - team * P::TS;
    pr = blockIdx.x * (blockDim.x / P::TS) + team;
    valid = pr < P::L / 2;
    slot = lds + team * fft_slots<P>();
  }
  template <class Q>
  __device__ float2 &at(int q) const { return slot[fft_place<Q>(q)]; }
};

// Spectra of the two rows from the transform Z of row a + i row b,
//   A = (Z + conj(Zm)) / 2,  B = (Z - conj(Zm)) / (2i),  Zm = Z[L - k].
template <class P>
__device__ __forceinline__ void split_store(const typename FftLast<P>::Vals &z, const RowTeam<P> &w,
                                            float2 *sa, float2 *sb, float2 *slot) {
  constexpr int L = P::L;
  __syncthreads();
  const_cast<typename FftLast<P>::Vals &>(z).template outputs<L / FftLast<P>::R>(
      w.t, [&](int q, float2 v) { slot[q] = v; });
  __syncthreads();
  if (!w.valid) return;
  for (int k = w.t; k <= L / 2; k += P::TS) {
    const float2 Z = slot[k], Zm = slot[k ? L - k : 0];
    const float dx = Z.x - Zm.x, dy = Z.y + Zm.y;
    sa[k] = make_float2(0.5f * (Z.x + Zm.x), 0.5f * (Z.y - Zm.y));
    sb[k] = make_float2(0.5f * dy, -0.5f * dx);
  }
}

// Value q of the Hermitian-packed spectrum A + i B of two rows.
template <int L>
__device__ __forceinline__ float2 packed(const float2 *sa, const float2 *sb, int q) {
  const bool up = q > L / 2;
  const int k = up ? L - q : q;
  float2 A = sa[k], B = sb[k];
  if (q == 0 || q == L / 2) A.y = B.y = 0.f;
  if (up) {
    A.y = -A.y;
    B.y = -B.y;
  }
  return make_float2(A.x - B.y, A.y + B.x);
}

// spec[b][r][0..D/2] = rFFT(src[b][r][:]) for every row
template <class P>
__global__ void __launch_bounds__(256)
k_rows_fwd(const float *src, const float2 *tw, float2 *spec) {
  extern __shared__ float2 lds[];
  constexpr int L = P::L, Dh = L / 2 + 1;
  const RowTeam<P> w(lds);
  const float *ra = src + ((size_t)blockIdx.y * L + 2 * w.pr) * L;
  FftVals<P, P::R0> a;
  a.inputs(w.t, [&](int q) { return w.valid ? make_float2(ra[q], ra[L + q]) : make_float2(0.f, 0.f); });
  const auto z = fft_run<P, false>(a, w.t, tw, [&](int q) -> float2 & { return w.template at<P>(q); });
  float2 *sa = spec + ((size_t)blockIdx.y * L + 2 * w.pr) * Dh;
  split_store<P>(z, w, sa, sa + Dh, w.slot);
}

template <class P>
__global__ void __launch_bounds__(256)
k_rows_inv(const float2 *spec, const float2 *tw, float *dst) {
  extern __shared__ float2 lds[];
  constexpr int L = P::L, Dh = L / 2 + 1;
  const RowTeam<P> w(lds);
  const float2 *sa = spec + ((size_t)blockIdx.y * L + 2 * w.pr) * Dh;
  FftVals<P, P::R0> a;
  a.inputs(w.t, [&](int q) { return w.valid ? packed<L>(sa, sa + Dh, q) : make_float2(0.f, 0.f); });
  auto z = fft_run<P, true>(a, w.t, tw, [&](int q) -> float2 & { return w.template at<P>(q); });
  if (!w.valid) return;
  float *ra = dst + ((size_t)blockIdx.y * L + 2 * w.pr) * L;
  z.template outputs<L / FftLast<P>::R>(w.t, [&](int q, float2 v) {
    ra[q] = v.x;
    ra[L + q] = v.y;
  });
}

// Fused: inverse rows of X, optional X output, residual R = X - Y, partial
// sums of R^2 per row pair, G_X = grad_scale * R and (when the adjoint follows)
// the forward rows of G_X written back into spec.
template <class P>
__global__ void __launch_bounds__(256)
k_rows_inv_loss(float2 *spec, const float2 *tw, const float *obs, float *images_out,
                float grad_scale, int adjoint, float *loss_part) {
  extern __shared__ float2 lds[];
  __shared__ double red[256];
  constexpr int L = P::L, Dh = L / 2 + 1;
  typedef typename P::Reverse Rev;
  const RowTeam<P> w(lds);
  float2 *sa = spec + ((size_t)blockIdx.y * L + 2 * w.pr) * Dh;
  const size_t row0 = ((size_t)blockIdx.y * L + 2 * w.pr) * L;
  FftVals<P, P::R0> a;
  a.inputs(w.t, [&](int q) { return w.valid ? packed<L>(sa, sa + Dh, q) : make_float2(0.f, 0.f); });
  // observed values of this thread, requested with the inputs
  typename FftLast<P>::Vals y;
  y.inputs(w.t, [&](int q) {
    return w.valid ? make_float2(obs[row0 + q], obs[row0 + L + q]) : make_float2(0.f, 0.f);
  });
  auto z = fft_run<P, true>(a, w.t, tw, [&](int q) -> float2 & { return w.template at<P>(q); });
  if (images_out && w.valid)
    z.template outputs<L / FftLast<P>::R>(w.t, [&](int q, float2 v) {
      images_out[row0 + q] = v.x;
      images_out[row0 + L + q] = v.y;
    });
  // (squares and sums in FP64: a team's values are one chain of L additions)
  double acc = 0.0;
#pragma unroll
  for (int m = 0; m < z.kN; ++m)
#pragma unroll
    for (int i = 0; i < FftLast<P>::R; ++i) {
      const float ra = z.v[m][i].x - y.v[m][i].x, rb = z.v[m][i].y - y.v[m][i].y;
      if (z.kJ % P::TS == 0 || w.t + m * P::TS < z.kJ) acc += (double)ra * ra + (double)rb * rb;
      z.v[m][i] = make_float2(grad_scale * ra, grad_scale * rb);
    }
  red[threadIdx.x] = acc;
  __syncthreads();
  if (w.t == 0 && w.valid) {
    for (int k = 1; k < P::TS; ++k) acc += red[threadIdx.x + k];
    loss_part[(size_t)blockIdx.y * (L / 2) + w.pr] = (float)acc;
  }
  if (!adjoint) return;
  FftVals<Rev, Rev::R0> g = fft_turn<P>(z);
  const auto s = fft_run<Rev, false>(g, w.t, tw, [&](int q) -> float2 & { return w.template at<Rev>(q); });
  RowTeam<Rev> wr(lds);
  split_store<Rev>(s, wr, sa, sa + Dh, w.slot);
}

#define X(N, A, B, C, T) \
  case N: return &k_rows_fwd<FftRadices<A, B, C, T>>;
RowsFwdFn fft_rows_fwd(int L) {
  switch (L) { CS_FFT_LENGTHS(X) }
  return nullptr;
}
#undef X
#define X(N, A, B, C, T) \
  case N: return &k_rows_inv<FftRadices<A, B, C, T>>;
RowsInvFn fft_rows_inv(int L) {
  switch (L) { CS_FFT_LENGTHS(X) }
  return nullptr;
}
#undef X
#define X(N, A, B, C, T) \
  case N: return &k_rows_inv_loss<FftRadices<A, B, C, T>>;
RowsInvLossFn fft_rows_inv_loss(int L) {
  switch (L) { CS_FFT_LENGTHS(X) }
  return nullptr;
}
#undef X

// H^ / D^2 on the half-spectrum grid [B][D][D/2+1], once per call.
__global__ void __launch_bounds__(256)
k_ctf_table(int L, float pixel, CtfDev ctf, int B, float *table) {
  // grid rows walk the images (b = blockIdx.y, blockIdx.y + gridDim.y, ...);
  // a thread fills entries blockIdx.x * 256 + threadIdx.x + k * gridDim.x *
  // 256 of an image with its constants (defocus, astigmatism angle, phase,
  // frequency step) evaluated once
  const int Dh = L / 2 + 1;
  const int per = L * Dh;
  const float norm = 1.f / ((float)L * (float)L);
  const CtfGrid g = ctf_grid(L, pixel, ctf);
  for (int b = blockIdx.y; b < B; b += gridDim.y) {
    float *row = table + (size_t)b * per;
    if (!ctf.enabled) {
      for (int r = blockIdx.x * 256 + threadIdx.x; r < per; r += gridDim.x * 256) row[r] = norm;
      continue;
    }
    const CtfParticle q = ctf_particle(ctf, b);
    for (int r = blockIdx.x * 256 + threadIdx.x; r < per; r += gridDim.x * 256) {
      const int ky = r / Dh, kx = r % Dh;
      row[r] = ctf_value(ky, kx, L, g, ctf, q) * norm;
    }
  }
}

// loss[b] = scale * sum of the row-pair partials of image b (one block per
// image, FP64 sums), then loss[B] = the total in image order.
__global__ void __launch_bounds__(256)
k_loss_reduce(const float *loss_part, int B, int parts, float scale, float *loss) {
  __shared__ double red[4];
  const int b = blockIdx.x;
  double s = 0.0;
  for (int k = threadIdx.x; k < parts; k += 256) s += (double)loss_part[(size_t)b * parts + k];
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
  __syncthreads();
  if (threadIdx.x == 0) {
    const float v = (float)(scale * (red[0] + red[1] + red[2] + red[3]));
    loss[b] = v;
    if (B == 1) loss[1] = v;  // the total of one image (k_loss_total is skipped)
  }
}

// Both in one block, for few partials: a wave per image, then the total.
__global__ void __launch_bounds__(1024)
k_loss_small(const float *loss_part, int B, int parts, float scale, float *loss) {
  __shared__ double red[16];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  double tot = 0.0;
  for (int b = wv; b < B; b += 16) {
    double s = 0.0;
    for (int k = lane; k < parts; k += 64) s += (double)loss_part[(size_t)b * parts + k];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
    const float v = (float)(scale * s);
    if (lane == 0) loss[b] = v;
    tot += (double)v;
  }
  if (lane == 0) red[wv] = tot;
  __syncthreads();
  if (threadIdx.x == 0) {
    double s = 0.0;
    for (int w = 0; w < 16; ++w) s += red[w];
    loss[B] = (float)s;
  }
}

__global__ void __launch_bounds__(256) k_loss_total(float *loss, int B) {
  __shared__ double red[4];
  double s = 0.0;
  for (int b = threadIdx.x; b < B; b += 256) s += (double)loss[b];
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
  __syncthreads();
  if (threadIdx.x == 0) loss[B] = (float)(red[0] + red[1] + red[2] + red[3]);
}

// No-CTF residual (X = Q): loss partials per row, optional X output and
// G_Q = grad_scale (X - Y) written in place over Q.
__global__ void __launch_bounds__(256)
k_residual(float *Q, const float *obs, float *images_out, int B, int D, float grad_scale,
           float *loss_part) {
  const int row = blockIdx.x, b = blockIdx.y;
  const size_t o = ((size_t)b * D + row) * D;
  float acc = 0.f;
  for (int j = threadIdx.x; j < D; j += 256) {
    const float x = Q[o + j];
    if (images_out) images_out[o + j] = x;
    const float r = x - obs[o + j];
    acc += r * r;
    Q[o + j] = grad_scale * r;
  }
  __shared__ float red[4];
#pragma unroll
  for (int s = 32; s > 0; s >>= 1) acc += __shfl_xor(acc, s, 64);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = acc;
  __syncthreads();
  if (threadIdx.x == 0) loss_part[(size_t)b * D + row] = red[0] + red[1] + red[2] + red[3];
}


}  // namespace cs
