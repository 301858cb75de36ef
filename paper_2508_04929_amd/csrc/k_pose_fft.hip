// The FFT passes of pose scoring (banks, and particles at sides other than 128).
//
// Their results are rounded to bfloat16 operands, and the best of thousands of
// scores is a whole number: a transform that rounds differently in FP32 moves
// some of those roundings and, rarely, a winner.  These kernels therefore keep
// the arithmetic that existing banks and searches have (Stockham passes of
// radix 4, 2 and 3 in this order, one LDS round trip each); everything whose
// results are FP32 numbers uses cs_fft_dev.hpp, at about half the time per
// pass.
#include "cs_fft_dev.hpp"
#include "cs_pose.hpp"

namespace cs {

// One Stockham transform of length P.L by a team of `ts` threads (thread
// index t within the team).  x holds the input, y is scratch; returns the
// buffer that holds the result.  Every thread of the block must call it
// (it synchronises the block after every stage).
__device__ float2 *fft_team(float2 *x, float2 *y, const FftPlan &P, const float2 *tw, int t,
                            int ts, bool inverse) {
  const int L = P.L;
  int Ns = 1;
  const float sg = inverse ? 1.f : -1.f;  // sign of the exponent
  for (int st = 0; st < P.nst; ++st) {
    const int R = P.radix[st];
    const int LR = L / R;
    const int tws = L / (Ns * R);
    for (int j = t; j < LR; j += ts) {
      const int k = j % Ns;
      const int base = (j / Ns) * Ns * R + k;
      if (R == 4) {
        float2 v0 = x[j], v1 = x[j + LR], v2 = x[j + 2 * LR], v3 = x[j + 3 * LR];
        if (k) {
          float2 w1 = tw[k * tws], w2 = tw[2 * k * tws], w3 = tw[3 * k * tws];
          if (inverse) { w1.y = -w1.y; w2.y = -w2.y; w3.y = -w3.y; }
          v1 = cmul(v1, w1); v2 = cmul(v2, w2); v3 = cmul(v3, w3);
        }
        const float2 a0 = make_float2(v0.x + v2.x, v0.y + v2.y);
        const float2 a1 = make_float2(v0.x - v2.x, v0.y - v2.y);
        const float2 a2 = make_float2(v1.x + v3.x, v1.y + v3.y);
        const float2 a3 = make_float2(v1.x - v3.x, v1.y - v3.y);
        // y1 = a1 + sg*i*a3, y3 = a1 - sg*i*a3
        y[base] = make_float2(a0.x + a2.x, a0.y + a2.y);
        y[base + Ns] = make_float2(a1.x - sg * a3.y, a1.y + sg * a3.x);
        y[base + 2 * Ns] = make_float2(a0.x - a2.x, a0.y - a2.y);
        y[base + 3 * Ns] = make_float2(a1.x + sg * a3.y, a1.y - sg * a3.x);
      } else if (R == 2) {
        float2 v0 = x[j], v1 = x[j + LR];
        if (k) {
          float2 w1 = tw[k * tws];
          if (inverse) w1.y = -w1.y;
          v1 = cmul(v1, w1);
        }
        y[base] = make_float2(v0.x + v1.x, v0.y + v1.y);
        y[base + Ns] = make_float2(v0.x - v1.x, v0.y - v1.y);
      } else {  // R == 3
        float2 v0 = x[j], v1 = x[j + LR], v2 = x[j + 2 * LR];
        if (k) {
          float2 w1 = tw[k * tws], w2 = tw[2 * k * tws];
          if (inverse) { w1.y = -w1.y; w2.y = -w2.y; }
          v1 = cmul(v1, w1); v2 = cmul(v2, w2);
        }
        const float c3 = 0.86602540378443864676f;  // sqrt(3)/2
        const float2 t1 = make_float2(v1.x + v2.x, v1.y + v2.y);
        const float2 t2 = make_float2(v1.x - v2.x, v1.y - v2.y);
        const float2 m = make_float2(v0.x - 0.5f * t1.x, v0.y - 0.5f * t1.y);
        // y1 = m + sg*i*c3*t2, y2 = m - sg*i*c3*t2
        y[base] = make_float2(v0.x + t1.x, v0.y + t1.y);
        y[base + Ns] = make_float2(m.x - sg * c3 * t2.y, m.y + sg * c3 * t2.x);
        y[base + 2 * Ns] = make_float2(m.x + sg * c3 * t2.y, m.y - sg * c3 * t2.x);
      }
    }
    __syncthreads();
    float2 *tmp = x; x = y; y = tmp;
    Ns *= R;
  }
  return x;
}

// Row kernels: one team of 64 threads per row pair, four teams per block.

// ---------------------------------------------------------------------------
// Forward row pass: spec[b][r][0..D/2] = rFFT(src[b][r][:]) for every row.
// ---------------------------------------------------------------------------
__device__ __forceinline__ void split_store(const float2 *res, int L, int t, float2 *spec_a,
                                            float2 *spec_b, bool valid) {
  for (int k = t; k <= L / 2; k += 64) {
    const float2 Z = res[k];
    const float2 Zm = res[(L - k) % L];
    // A = (Z + conj(Zm)) / 2,  B = (Z - conj(Zm)) / (2i)
    const float dx = Z.x - Zm.x, dy = Z.y + Zm.y;
    if (valid) {
      spec_a[k] = make_float2(0.5f * (Z.x + Zm.x), 0.5f * (Z.y - Zm.y));
      spec_b[k] = make_float2(0.5f * dy, -0.5f * dx);
    }
  }
}

__global__ void __launch_bounds__(256)
k_pose_fft_rows_fwd(const float *src, FftPlan P, const float2 *tw, int B, float2 *spec) {
  extern __shared__ float2 lds[];
  const int L = P.L, Dh = L / 2 + 1;
  const int teams = blockDim.x >> 6, team = threadIdx.x >> 6, t = threadIdx.x & 63;
  const int pr = blockIdx.x * teams + team;  // row pair
  const int b = blockIdx.y;
  const bool valid = pr < L / 2;
  float2 *x = lds + team * 2 * L, *y = x + L;
  float2 *twl = lds + teams * 2 * L;
  for (int k = threadIdx.x; k < L; k += blockDim.x) twl[k] = tw[k];
  const float *ra = src + ((size_t)b * L + 2 * pr) * L;
  for (int j = t; j < L; j += 64) x[j] = valid ? make_float2(ra[j], ra[L + j]) : make_float2(0.f, 0.f);
  __syncthreads();
  const float2 *res = fft_team(x, y, P, twl, t, 64, false);
  float2 *sa = spec + ((size_t)b * L + 2 * pr) * Dh;
  split_store(res, L, t, sa, sa + Dh, valid);
}

// ---------------------------------------------------------------------------
// Column pass: for cpw adjacent half-spectrum columns per block, FFT over
// rows, times a multiplier mul(ky, kx, z) of image blockIdx.y, inverse FFT
// over rows, in place.
// ---------------------------------------------------------------------------
// Image and column group of this block: the grid is (column groups, images)
// and the XCD-aware order keeps an image's adjacent column groups (whose
// rows share cache lines) on one XCD.
__device__ __forceinline__ void cols_block(int &b, int &group) {
  const int j = xcd_work(blockIdx.x + gridDim.x * blockIdx.y, gridDim.x * gridDim.y);
  b = j / gridDim.x;
  group = j % gridDim.x;
}

template <class Mul>
__device__ __forceinline__ void fft_cols_apply(float2 *spec, const FftPlan &P, const float2 *tw,
                                               int cpw, int b, int group, const Mul &mul) {
  extern __shared__ float2 lds[];
  const int L = P.L, Dh = L / 2 + 1;
  const int kx0 = group * cpw;
  const int ts = 256 / cpw;
  const int team = threadIdx.x / ts, t = threadIdx.x % ts;
  float2 *img = spec + (size_t)b * L * Dh;
  float2 *twl = lds + (size_t)cpw * 2 * L;
  for (int k = threadIdx.x; k < L; k += 256) twl[k] = tw[k];
  // coalesced load: consecutive threads take consecutive columns of a row
  for (int q = threadIdx.x; q < cpw * L; q += 256) {
    const int c = q % cpw, r = q / cpw;
    const int kx = kx0 + c;
    lds[c * 2 * L + r] = (kx < Dh) ? img[(size_t)r * Dh + kx] : make_float2(0.f, 0.f);
  }
  __syncthreads();
  float2 *x = lds + team * 2 * L, *y = x + L;
  float2 *res = fft_team(x, y, P, twl, t, ts, false);
  const int kx = kx0 + team;
  for (int ky = t; ky < L; ky += ts) res[ky] = (kx < Dh) ? mul(ky, kx, res[ky]) : make_float2(0.f, 0.f);
  __syncthreads();
  float2 *other = (res == x) ? y : x;
  float2 *out = fft_team(res, other, P, twl, t, ts, true);
  // every team's result sits in the same half of its buffer pair
  const int oofs = (int)(out - (lds + team * 2 * L));
  for (int q = threadIdx.x; q < cpw * L; q += 256) {
    const int c = q % cpw, r = q / cpw;
    const int kc = kx0 + c;
    if (kc < Dh) img[(size_t)r * Dh + kc] = lds[c * 2 * L + oofs + r];
  }
}

// times the table H^ / D^2 (Eq. 14)
__global__ void __launch_bounds__(256)
k_pose_fft_cols_ctf(float2 *spec, FftPlan P, const float2 *tw, int B, int cpw, const float *table) {
  const int L = P.L, Dh = L / 2 + 1;
  int b, group;
  cols_block(b, group);
  const float *hcol = table + (size_t)b * L * Dh;
  fft_cols_apply(spec, P, tw, cpw, b, group, [&](int ky, int kx, float2 z) {
    const float h = hcol[(size_t)ky * Dh + kx];
    return make_float2(z.x * h, z.y * h);
  });
}

// Hermitian-packed inverse of two half-spectrum rows into one complex row.
__device__ __forceinline__ void pack_inverse(const float2 *sa, const float2 *sb, int L, int t,
                                             float2 *x, bool valid) {
  const int half = L / 2;
  for (int k = t; k < L; k += 64) {
    float2 A, Bv;
    if (!valid) {
      A = Bv = make_float2(0.f, 0.f);
    } else if (k <= half) {
      A = sa[k];
      Bv = sb[k];
      if (k == 0 || (k == half && (L % 2 == 0))) { A.y = 0.f; Bv.y = 0.f; }
    } else {
      A = sa[L - k];
      Bv = sb[L - k];
      A.y = -A.y;
      Bv.y = -Bv.y;
    }
    x[k] = make_float2(A.x - Bv.y, A.y + Bv.x);  // A + i B
  }
}

__global__ void __launch_bounds__(256)
k_pose_fft_rows_inv(const float2 *spec, FftPlan P, const float2 *tw, int B, float *dst) {
  extern __shared__ float2 lds[];
  const int L = P.L, Dh = L / 2 + 1;
  const int teams = blockDim.x >> 6, team = threadIdx.x >> 6, t = threadIdx.x & 63;
  const int pr = blockIdx.x * teams + team;
  const int b = blockIdx.y;
  const bool valid = pr < L / 2;
  float2 *x = lds + team * 2 * L, *y = x + L;
  float2 *twl = lds + teams * 2 * L;
  for (int k = threadIdx.x; k < L; k += blockDim.x) twl[k] = tw[k];
  const float2 *sa = spec + ((size_t)b * L + 2 * pr) * Dh;
  pack_inverse(sa, sa + Dh, L, t, x, valid);
  __syncthreads();
  const float2 *res = fft_team(x, y, P, twl, t, 64, true);
  if (valid) {
    float *ra = dst + ((size_t)b * L + 2 * pr) * L;
    for (int j = t; j < L; j += 64) {
      const float2 z = res[j];
      ra[j] = z.x;
      ra[L + j] = z.y;
    }
  }
}

// ---------------------------------------------------------------------------
// Column pass for power spectra: for cpw adjacent half-spectrum columns per
// block, forward FFT over rows and |.|^2 stored as bfloat16 (nearest even)
// at out[b * ld + ky * (D/2+1) + kx].
// ---------------------------------------------------------------------------
__device__ __forceinline__ unsigned short f2bf_rne(float x) {
  unsigned u = __float_as_uint(x);
  if ((u & 0x7fffffffu) > 0x7f800000u) return (unsigned short)((u >> 16) | 0x40u);
  u += 0x7fffu + ((u >> 16) & 1u);
  return (unsigned short)(u >> 16);
}

__global__ void __launch_bounds__(256)
k_pose_fft_cols_power(const float2 *spec, FftPlan P, const float2 *tw, int B, int cpw,
                 unsigned short *out, size_t ld) {
  extern __shared__ float2 lds[];
  const int L = P.L, Dh = L / 2 + 1;
  const int b = blockIdx.y;
  const int kx0 = blockIdx.x * cpw;
  const int ts = 256 / cpw;
  const int team = threadIdx.x / ts, t = threadIdx.x % ts;
  const float2 *img = spec + (size_t)b * L * Dh;
  float2 *twl = lds + (size_t)cpw * 2 * L;
  for (int k = threadIdx.x; k < L; k += 256) twl[k] = tw[k];
  for (int q = threadIdx.x; q < cpw * L; q += 256) {
    const int c = q % cpw, r = q / cpw;
    const int kx = kx0 + c;
    lds[c * 2 * L + r] = (kx < Dh) ? img[(size_t)r * Dh + kx] : make_float2(0.f, 0.f);
  }
  __syncthreads();
  float2 *x = lds + team * 2 * L, *y = x + L;
  const float2 *res = fft_team(x, y, P, twl, t, ts, false);
  const int kx = kx0 + team;
  if (kx < Dh) {
    unsigned short *o = out + (size_t)b * ld + kx;
    for (int ky = t; ky < L; ky += ts) {
      const float2 z = res[ky];
      o[(size_t)ky * Dh] = f2bf_rne(z.x * z.x + z.y * z.y);
    }
  }
}

}  // namespace cs
