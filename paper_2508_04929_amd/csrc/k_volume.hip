// Voxelisation of the mixture and Fourier shell correlation.
//
// The reconstruction is a Gaussian mixture; the overview of Sec. 3 reads
// the final volume out by voxelising it, and Sec. 4 compares volumes by the
// Fourier shell correlation of Eq. 10 with the 0.143 threshold.
//
// Voxelisation: voxel (iz, iy, ix) sits at ((ix - c0) p, (iy - c0) p,
// (iz - c0) p) and holds sum_n A_n (2 pi)^-3/2 det(Sigma_n)^-1/2
// exp(-q_n / 2) over the Gaussians with q_n <= q_cut.  Bricks of 8^3 voxels:
// every Gaussian is listed under the bricks its q <= q_cut box touches
// (counting sort); a block evaluates one brick against its list, one wave
// per 4^3 sub-cube, each Gaussian only where a conservative bound of its
// form over the sub-cube is within the cut.  Each voxel's sum is kept as a 64-bit fixed-point integer
// (scale 2^e with the bound sum_n |w_n| < 2^61 / scale), so the result does
// not depend on the order of the list: it is reproducible bit for bit.
//
// FSC: the 3-D real DFT is the renderer's row pass (real rows along x, two
// per complex transform) over the D slices, then the same Stockham
// transform along y and along z (k_axis); shell sums of
// Re(Fa conj Fb), |Fa|^2, |Fb|^2 (weight 2 off the kx = 0 and Nyquist
// planes) are again exact 64-bit fixed-point sums, scaled by Parseval's
// bound D^3 max(sum Va^2, sum Vb^2) on every shell sum.
#include "cs_volume.hpp"

namespace cs {

constexpr int kBrick = 8;

__device__ __forceinline__ int clampi(float x, int lo, int hi) {
  x = fminf(fmaxf(x, (float)lo), (float)hi);
  return (int)x;
}

// Per Gaussian: mean and weight, inverse covariance (FP64 adjugate) and the
// brick range of its q <= q_cut box; per block the sum of |w| (fixed-order
// tree, FP64) for the fixed-point scale.
__global__ void __launch_bounds__(256)
k_vox_prep(const float4 *gc, VoxGeom V, float4 *rec, int4 *box, double *wpart) {
  __shared__ double red[256];
  const int n = blockIdx.x * 256 + threadIdx.x;
  double aw = 0.0;
  if (n < V.N) {
    const float4 g0 = gc[3 * n], g1 = gc[3 * n + 1], g2 = gc[3 * n + 2];
    const double sxx = g1.x, sxy = g1.y, sxz = g1.z, syy = g1.w, syz = g2.x, szz = g2.y;
    const double cxx = syy * szz - syz * syz, cxy = sxz * syz - sxy * szz, cxz = sxy * syz - sxz * syy;
    const double cyy = sxx * szz - sxz * sxz, cyz = sxy * sxz - sxx * syz, czz = sxx * syy - sxy * sxy;
    const double det = fmax(sxx * cxx + sxy * cxy + sxz * cxz, 1e-30);
    const float w = (float)((double)g0.w * 0.063493635934240969 / sqrt(det));  // (2 pi)^-3/2
    aw = fabs((double)w);
    // quadratic form scaled by log2(e) / 2, cross terms doubled, so that
    // exp(-q / 2) = 2^-(x^T B x) with B = (log2(e) / 2) Sigma^-1
    const double f = 0.72134752044448170 / det;  // log2(e) / 2 / det
    rec[3 * n] = make_float4(g0.x, g0.y, g0.z, w);
    rec[3 * n + 1] = make_float4((float)(cxx * f), (float)(2.0 * cxy * f), (float)(2.0 * cxz * f),
                                 (float)(cyy * f));
    rec[3 * n + 2] = make_float4((float)(2.0 * cyz * f), (float)(czz * f), 0.f, 0.f);
    // axis-aligned box of the ellipsoid q <= q_cut: half extents sqrt(q_cut S_ii)
    const float mu[3] = {g0.x, g0.y, g0.z};
    const float hh[3] = {sqrtf(V.q_cut * g1.x), sqrtf(V.q_cut * g1.w), sqrtf(V.q_cut * g2.y)};
    const float ip = 1.f / V.pixel;
    int lo[3], hi[3];
    bool empty = false;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      const float a = ceilf((mu[k] - hh[k]) * ip + (float)V.c0);
      const float b = floorf((mu[k] + hh[k]) * ip + (float)V.c0);
      empty |= !(a <= b) || b < 0.f || a > (float)(V.D - 1);
      lo[k] = clampi(a, 0, V.D - 1) / kBrick;
      hi[k] = clampi(b, 0, V.D - 1) / kBrick;
    }
    box[n] = empty ? make_int4(0, 0, 0, 0)
                   : make_int4(lo[0] | (hi[0] << 16), lo[1] | (hi[1] << 16), lo[2] | (hi[2] << 16), 1);
  }
  red[threadIdx.x] = aw;
  __syncthreads();
  for (int h = 128; h > 0; h >>= 1) {
    if ((int)threadIdx.x < h) red[threadIdx.x] += red[threadIdx.x + h];
    __syncthreads();
  }
  if (threadIdx.x == 0) wpart[blockIdx.x] = red[0];
}

// A box of bricks, or of the cells that it meets, or its part inside a cell.
struct Box {
  int x0, y0, z0, nx, ny, m;
  // [lo >> sh, hi >> sh] of the box clipped to [c, c + n) on every axis
  __device__ Box(int4 b, int sh, int cx = 0, int cy = 0, int cz = 0, int n = 1 << 20) {
    x0 = max((b.x & 0xffff) >> sh, cx);
    y0 = max((b.y & 0xffff) >> sh, cy);
    z0 = max((b.z & 0xffff) >> sh, cz);
    nx = min(b.x >> (16 + sh), cx + n - 1) - x0 + 1;
    ny = min(b.y >> (16 + sh), cy + n - 1) - y0 + 1;
    m = b.w ? nx * ny * (min(b.z >> (16 + sh), cz + n - 1) - z0 + 1) : 0;
  }
  __device__ int3 at(int l) const {  // entry l, x fastest
    const int r = l / nx, z = r / ny;
    return make_int3(x0 + l - r * nx, y0 + r - z * ny, z0 + z);
  }
};

// The lists are built in two levels: Gaussians under cells of 2^3 bricks (4^3 in
// volumes above 256^3), then each cell's Gaussians under its bricks.  Both levels
// count in LDS, and a block adds to memory once per cell that it met.  With a memory
// atomic per (brick, Gaussian) pair the 200000 Gaussians of 14 bricks each in a 256^3
// volume took 107 us to count, 57 to scan over 32768 bricks and 98 to list, bound by
// those atomics; the two levels take 22 + 6 + 21 + 27 us.

// Gaussians and (brick, Gaussian) pairs of every cell; 8 lanes to a Gaussian.
// The lists are indexed with 32 bits, so the totals are kept in 64: where they do
// not fit, the counts may have wrapped and nothing may be listed.
__global__ void __launch_bounds__(1024)
k_vox_count(const int4 *box, VoxGeom V, int2 *count, unsigned long long *total) {
  extern __shared__ int2 hist[];  // [nc^3]
  __shared__ unsigned long long sum[2];
  const int ncell = V.nc * V.nc * V.nc;
  if (threadIdx.x < 2) sum[threadIdx.x] = 0ull;
  for (int i = threadIdx.x; i < ncell; i += 1024) hist[i] = make_int2(0, 0);
  __syncthreads();
  const int n1 = min(V.N, (int)(blockIdx.x + 1) * V.per);
  for (int n = blockIdx.x * V.per + threadIdx.x / 8; n < n1; n += 128) {
    const int4 b = box[n];
    const Box cells(b, V.cs);
    for (int l = threadIdx.x % 8; l < cells.m; l += 8) {
      const int3 c = cells.at(l);
      int2 *h = &hist[(c.z * V.nc + c.y) * V.nc + c.x];
      atomicAdd(&h->x, 1);
      atomicAdd(&h->y, Box(b, 0, c.x << V.cs, c.y << V.cs, c.z << V.cs, 1 << V.cs).m);
    }
  }
  __syncthreads();
  unsigned long long cells = 0ull, pairs = 0ull;
  for (int i = threadIdx.x; i < ncell; i += 1024)
    if (hist[i].x) {
      atomicAdd(&count[i].x, hist[i].x);
      atomicAdd(&count[i].y, hist[i].y);
      cells += hist[i].x;
      pairs += hist[i].y;
    }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    cells += __shfl_xor(cells, o, 64);
    pairs += __shfl_xor(pairs, o, 64);
  }
  if ((threadIdx.x & 63) == 0) {
    atomicAdd(&sum[0], cells);
    atomicAdd(&sum[1], pairs);
  }
  __syncthreads();
  if (threadIdx.x < 2) atomicAdd(&total[threadIdx.x], sum[threadIdx.x]);
}

// Exclusive scans of the cell counts (one block) and the fixed-point scale of
// the voxel sums from the bound sum_n |w_n| (k_vox_prep's per-block partials
// added in a fixed order, FP64).
__global__ void __launch_bounds__(1024)
k_vox_scan(const int2 *count, int ncell, const double *wpart, int nwp, int2 *off, double *scale) {
  __shared__ int2 wave[16];
  __shared__ double wsum[1024];
  const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
  double ws = 0.0;
  for (int i = t; i < nwp; i += 1024) ws += wpart[i];
  wsum[t] = ws;
  // at most 4096 cells, four adjacent ones per thread
  int2 v[4], s = make_int2(0, 0);
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    v[u] = 4 * t + u < ncell ? count[4 * t + u] : make_int2(0, 0);
    s = make_int2(s.x + v[u].x, s.y + v[u].y);
  }
  int2 x = s;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int2 y = make_int2(__shfl_up(x.x, o, 64), __shfl_up(x.y, o, 64));
    if (lane >= o) x = make_int2(x.x + y.x, x.y + y.y);
  }
  if (lane == 63) wave[wv] = x;
  __syncthreads();
  int2 at = make_int2(x.x - s.x, x.y - s.y), all = make_int2(0, 0);
#pragma unroll
  for (int w = 0; w < 16; ++w) {
    const int2 y = wave[w];
    if (w < wv) at = make_int2(at.x + y.x, at.y + y.y);
    all = make_int2(all.x + y.x, all.y + y.y);
  }
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    if (4 * t + u < ncell) off[4 * t + u] = at;
    at = make_int2(at.x + v[u].x, at.y + v[u].y);
  }
  for (int h = 512; h > 0; h >>= 1) {
    if (t < h) wsum[t] += wsum[t + h];
    __syncthreads();
  }
  if (t == 0) {
    off[ncell] = all;
    const double total = wsum[0] > 0.0 ? wsum[0] : 1.0;
    int e;
    frexp(total, &e);  // total < 2^e
    *scale = ldexp(1.0, 61 - e);
  }
}

// Cell lists: the counts of k_vox_count once more, a place in the list per cell
// that the block met, then its Gaussians in any order.
__global__ void __launch_bounds__(1024)
k_vox_fill(const int4 *box, VoxGeom V, const int2 *off, int *cursor, int *cell_list) {
  extern __shared__ int place[];  // [nc^3]
  const int ncell = V.nc * V.nc * V.nc;
  for (int i = threadIdx.x; i < ncell; i += 1024) place[i] = 0;
  __syncthreads();
  const int n0 = blockIdx.x * V.per + threadIdx.x / 8, n1 = min(V.N, (int)(blockIdx.x + 1) * V.per);
  for (int n = n0; n < n1; n += 128) {
    const Box cells(box[n], V.cs);
    for (int l = threadIdx.x % 8; l < cells.m; l += 8) {
      const int3 c = cells.at(l);
      atomicAdd(&place[(c.z * V.nc + c.y) * V.nc + c.x], 1);
    }
  }
  __syncthreads();
  for (int i = threadIdx.x; i < ncell; i += 1024)
    if (place[i]) place[i] = off[i].x + atomicAdd(&cursor[i], place[i]);
  __syncthreads();
  for (int n = n0; n < n1; n += 128) {
    const Box cells(box[n], V.cs);
    for (int l = threadIdx.x % 8; l < cells.m; l += 8) {
      const int3 c = cells.at(l);
      cell_list[atomicAdd(&place[(c.z * V.nc + c.y) * V.nc + c.x], 1)] = n;
    }
  }
}

// Brick lists of one cell per block: start and length of every brick's list, then
// the lists.  A thread per Gaussian; the place in a brick's list comes from the
// ballot of the wave's Gaussians that touch the brick (counters in LDS, 8 or 64
// for all threads, took 97 us for the mixture above; now 27 us).
template <int CS>
__global__ void __launch_bounds__(512)
k_vox_cell(const int4 *box, VoxGeom V, const int2 *off, const int *cell_list, int2 *range, int *list) {
  constexpr int kSide = 1 << CS, kBricks = 1 << 3 * CS;
  __shared__ int at[8][kBricks];  // per wave: its count, then its place in the lists
  const int k = blockIdx.x, t = threadIdx.x, lane = t & 63, wv = t >> 6;
  const int cx = k % V.nc << CS, cy = k / V.nc % V.nc << CS, cz = k / (V.nc * V.nc) << CS;
  const int2 b0 = off[k];
  const int cnt = off[k + 1].x - b0.x;
  // bricks of a Gaussian along an axis as bits; none: past the list's end
  auto bits = [&](int lohi, int c) {
    const int lo = max((lohi & 0xffff) - c, 0), hi = min((lohi >> 16) - c, kSide - 1);
    return (2u << hi) - (1u << lo);
  };
  auto touched = [&](int e, int &n, unsigned m[3]) {
    m[0] = m[1] = m[2] = 0u;
    if (e >= cnt) return;
    n = cell_list[b0.x + e];
    const int4 b = box[n];
    m[0] = bits(b.x, cx);
    m[1] = bits(b.y, cy);
    m[2] = bits(b.z, cz);
  };
  auto hit = [&](const unsigned m[3], int q) {
    return (m[0] >> (q & (kSide - 1)) & m[1] >> (q >> CS & (kSide - 1)) & m[2] >> (q >> 2 * CS) & 1u) != 0u;
  };
  int mine = 0;  // the wave's count of brick `lane`
  for (int e0 = wv * 64; e0 < cnt; e0 += 512) {
    int n = 0;
    unsigned m[3];
    touched(e0 + lane, n, m);
#pragma unroll
    for (int q = 0; q < kBricks; ++q) {
      const int c = __popcll(__ballot(hit(m, q)));
      if (lane == q) mine += c;
    }
  }
  if (lane < kBricks) at[wv][lane] = mine;
  __syncthreads();
  if (wv == 0) {
    int c = 0;
    if (lane < kBricks)
      for (int w = 0; w < 8; ++w) c += at[w][lane];
    int x = c;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int y = __shfl_up(x, o, 64);
      if (lane >= o) x += y;
    }
    if (lane < kBricks) {
      const int bx = cx + (lane & (kSide - 1)), by = cy + (lane >> CS & (kSide - 1)), bz = cz + (lane >> 2 * CS);
      int first = b0.y + x - c;
      if (bx < V.nb && by < V.nb && bz < V.nb) range[(bz * V.nb + by) * V.nb + bx] = make_int2(first, c);
      for (int w = 0; w < 8; ++w) {
        const int y = at[w][lane];
        at[w][lane] = first;
        first += y;
      }
    }
  }
  __syncthreads();
  mine = lane < kBricks ? at[wv][lane] : 0;
  const unsigned long long below = (1ull << lane) - 1ull;
  for (int e0 = wv * 64; e0 < cnt; e0 += 512) {
    int n = 0;
    unsigned m[3];
    touched(e0 + lane, n, m);
#pragma unroll
    for (int q = 0; q < kBricks; ++q) {
      const bool in = hit(m, q);
      const unsigned long long w = __ballot(in);
      const int first = __builtin_amdgcn_readlane(mine, q);
      if (in) list[first + __popcll(w & below)] = n;
      if (lane == q) mine += __popcll(w);
    }
  }
}
template __global__ void k_vox_cell<1>(const int4 *, VoxGeom, const int2 *, const int *, int2 *, int *);
template __global__ void k_vox_cell<2>(const int4 *, VoxGeom, const int2 *, const int *, int2 *, int *);

// Lower bound of the scaled form over the voxel centres of a 4^3 sub-cube,
// minus a rounding margin: with c the centre of the sub-cube, h = 1.5 p the
// largest offset of a voxel centre from it along each axis and P the
// (positive semi-definite) form, q(c + d) = q(c) + 2 d.P(c - mu) + d.P d
// >= q(c) - h sum_k |2 (P(c - mu))_k|.  The margin T / 1024, with
// T = sum_ij |P_ij| (|c_i - mu_i| + h)(|c_j - mu_j| + h) bounding every term
// of q over the sub-cube, exceeds by far the rounding of both this bound and
// the per-voxel evaluation (positions included), so a sub-cube whose bound
// exceeds the cut holds no voxel that the per-voxel test would keep.
__device__ __forceinline__ float subcube_bound(float4 a, float4 B, float4 C, float cx, float cy,
                                               float cz, float h) {
  const float dx = cx - a.x, dy = cy - a.y, dz = cz - a.z;
  const float q = fmaf(dz, fmaf(C.y, dz, fmaf(B.z, dx, C.x * dy)),
                       fmaf(fmaf(B.x, dx, B.y * dy), dx, B.w * dy * dy));
  const float gx = fmaf(2.f * B.x, dx, fmaf(B.y, dy, B.z * dz));
  const float gy = fmaf(B.y, dx, fmaf(2.f * B.w, dy, C.x * dz));
  const float gz = fmaf(B.z, dx, fmaf(C.x, dy, 2.f * C.y * dz));
  const float ax = fabsf(dx) + h, ay = fabsf(dy) + h, az = fabsf(dz) + h;
  const float T = fabsf(B.x) * ax * ax + fabsf(B.w) * ay * ay + fabsf(C.y) * az * az +
                  ax * (fabsf(B.y) * ay + fabsf(B.z) * az) + fabsf(C.x) * ay * az;
  return q - h * (fabsf(gx) + fabsf(gy) + fabsf(gz)) - T * (1.f / 1024.f);
}

// One Gaussian's term at one voxel: the scaled form (mean in a; form in B, C),
// the cut and the magnitude |w| 2^-q as an integer in units of 2^-k, truncated
// (below 2^61), for a.w = |w| 2^k.  Branch-free: y = |w| 2^(k - q),
// its part above 2^32 is trunc(y 2^-32) and the rest, y - hi 2^32, is exact too
// (the bits of y below 2^32), so both convert exactly.  A function of the Gaussian
// and the voxel alone, so the voxel sums do not depend on the order of their
// terms.
__device__ __forceinline__ unsigned long long vox_term(float4 a, float4 B, float2 C, float px, float py,
                                                       float pz, float qc) {
  const float dx = px - a.x, dy = py - a.y;
  const float cxy = fmaf(fmaf(B.x, dx, B.y * dy), dx, B.w * dy * dy);
  const float fz = fmaf(B.z, dx, C.x * dy);
  const float dz = pz - a.z;
  const float q = fmaf(dz, fmaf(C.y, dz, fz), cxy);
  const float e = a.w * __builtin_amdgcn_exp2f(-q);
  const float y = q <= qc ? e : 0.f;
  const float hi = truncf(y * 0x1p-32f);
  const float lo = fmaf(hi, -0x1p32f, y);
  return ((unsigned long long)(unsigned)hi << 32) | (unsigned long long)(unsigned)lo;
}

// One 4^3 sub-cube of a brick per wave (a workgroup of 64), one voxel per
// lane.  The eight sub-cubes of brick k are the workgroups
// 64 (k / 8) + 8 s + k % 8, s = 0 .. 7: workgroups are dealt to the eight
// XCDs in turn, so all eight land on the XCD of k % 8 and share its L2 for
// the brick's list and records.  The wave takes the list 64 Gaussians at a
// time: each lane loads one record and tests it against the sub-cube, the kept
// ones are staged in LDS, scaled, and the wave evaluates them one ballot bit at a
// time (two per pass).  The per-voxel arithmetic (form, cut, exp2, fixed point) is
// the same for every kept Gaussian whatever the order, and the sums are integers,
// so the result is that of evaluating every listed Gaussian at every voxel of the
// brick.
//
// VALU-bound: some 30 waves' terms per Gaussian of sd 1 voxel, 26 instructions
// each.  With the sign and the scale applied per voxel (38) the 200000 Gaussians
// above took 427 us; now 328.  Slower: the records through scalar loads (540 us,
// their cache's misses), and sums in LDS by the Gaussians' own columns (64-bit LDS
// atomics take four cycles per lane: 1.9 ms).
__global__ void __launch_bounds__(64)
k_vox_eval(const float4 *__restrict__ rec, const int *__restrict__ list,
           const int2 *__restrict__ range, VoxGeom V, const double *__restrict__ scale, float *__restrict__ vol) {
  __shared__ float4 sa[64], sb[64];
  __shared__ float2 sc[64];
  const int b = blockIdx.x;
  const int k = (b >> 6) * 8 + (b & 7), s = (b >> 3) & 7;
  if (k >= V.nb * V.nb * V.nb) return;
  const int bx = k % V.nb, by = (k / V.nb) % V.nb, bz = k / (V.nb * V.nb);
  const int lane = threadIdx.x;
  const int sx = bx * kBrick + 4 * (s & 1), sy = by * kBrick + 4 * ((s >> 1) & 1),
            sz = bz * kBrick + 4 * (s >> 2);
  const int ix = sx + (lane & 3), iy = sy + ((lane >> 2) & 3), iz = sz + (lane >> 4);
  const float px = (float)(ix - V.c0) * V.pixel, py = (float)(iy - V.c0) * V.pixel;
  const float pz = (float)(iz - V.c0) * V.pixel;
  const float h = 1.5f * V.pixel;
  const float cx = ((float)(sx - V.c0) + 1.5f) * V.pixel, cy = ((float)(sy - V.c0) + 1.5f) * V.pixel,
              cz = ((float)(sz - V.c0) + 1.5f) * V.pixel;
  const double S = *scale;
  int k2;
  frexp(S, &k2);
  const int kk = k2 - 1;                    // S = 2^(k2 - 1)
  const float qc = V.q_cut * 0.72134752f;   // the cut in the scaled form
  unsigned long long acc0 = 0, acc1 = 0;
  const int b0 = range[k].x, cnt = range[k].y;
  for (int c = 0; c < cnt; c += 64) {
    bool keep = false, neg = false;
    if (c + lane < cnt) {
      const int n = list[b0 + c + lane];
      const float4 a = rec[3 * n], B = rec[3 * n + 1], C = rec[3 * n + 2];
      keep = subcube_bound(a, B, C, cx, cy, cz, h) <= qc;
      neg = a.w < 0.f;
      sa[lane] = make_float4(a.x, a.y, a.z, ldexpf(fabsf(a.w), kk));
      sb[lane] = B;
      sc[lane] = make_float2(C.x, C.y);
    }
    __syncthreads();
    unsigned long long bits = __ballot(keep);
    const unsigned long long minus = __ballot(neg);
    if ((bits & minus) == 0ull) {
      while (bits) {  // two kept Gaussians per pass: independent chains
        const int j0 = __builtin_ctzll(bits);
        bits &= bits - 1ull;
        const bool two = bits != 0ull;
        const int j1 = two ? __builtin_ctzll(bits) : j0;
        bits &= bits - 1ull;
        acc0 += vox_term(sa[j0], sb[j0], sc[j0], px, py, pz, qc);
        const unsigned long long t1 = vox_term(sa[j1], sb[j1], sc[j1], px, py, pz, qc);
        if (two) acc1 += t1;
      }
    } else {
      for (; bits; bits &= bits - 1ull) {
        const int j = __builtin_ctzll(bits);
        const unsigned long long t0 = vox_term(sa[j], sb[j], sc[j], px, py, pz, qc);
        acc0 += minus >> j & 1ull ? 0ull - t0 : t0;
      }
    }
    __syncthreads();
  }
  vol[((int64_t)iz * V.D + iy) * V.D + ix] = (float)((double)(long long)(acc0 + acc1) / S);
}

// ---------------------------------------------------------------------------
// FSC
// ---------------------------------------------------------------------------

// Sum of squares of each volume in FP64: a fixed grid of kEnergyBlocks
// blocks, each over a fixed strided subset, so the summation order (and the
// scale below) does not depend on the device or on timing.
__global__ void __launch_bounds__(256)
k_fsc_energy_part(const float *va, const float *vb, int64_t n, double *part) {
  __shared__ double r[2][256];
  const int t = threadIdx.x;
  double a = 0.0, b = 0.0;
  const int64_t stride = (int64_t)kEnergyBlocks * 256;
  int64_t i = (int64_t)blockIdx.x * 256 + t;
  for (; i + 3 * stride < n; i += 4 * stride) {  // four independent loads in flight
    const float a0 = va[i], a1 = va[i + stride], a2 = va[i + 2 * stride], a3 = va[i + 3 * stride];
    const float b0 = vb[i], b1 = vb[i + stride], b2 = vb[i + 2 * stride], b3 = vb[i + 3 * stride];
    a += (double)a0 * a0 + (double)a1 * a1 + (double)a2 * a2 + (double)a3 * a3;
    b += (double)b0 * b0 + (double)b1 * b1 + (double)b2 * b2 + (double)b3 * b3;
  }
  for (; i < n; i += stride) {
    a += (double)va[i] * va[i];
    b += (double)vb[i] * vb[i];
  }
  r[0][t] = a;
  r[1][t] = b;
  __syncthreads();
  for (int h = 128; h > 0; h >>= 1) {
    if (t < h) {
      r[0][t] += r[0][t + h];
      r[1][t] += r[1][t + h];
    }
    __syncthreads();
  }
  if (t == 0) {
    part[blockIdx.x] = r[0][0];
    part[kEnergyBlocks + blockIdx.x] = r[1][0];
  }
}

// Total of the block sums (fixed tree) and the shell scale from it.
__global__ void __launch_bounds__(kEnergyBlocks)
k_fsc_energy_scale(const double *part, int D, double *scale) {
  __shared__ double r[2][kEnergyBlocks];
  const int t = threadIdx.x;
  r[0][t] = part[t];
  r[1][t] = part[kEnergyBlocks + t];
  __syncthreads();
  for (int h = kEnergyBlocks / 2; h > 0; h >>= 1) {
    if (t < h) {
      r[0][t] += r[0][t + h];
      r[1][t] += r[1][t + h];
    }
    __syncthreads();
  }
  if (t == 0) {
    // every shell sum is at most D^3 max(sum Va^2, sum Vb^2) (Parseval)
    double bound = (double)D * D * D * fmax(r[0][0], r[1][0]);
    if (!(bound > 0.0)) bound = 1.0;
    int e;
    frexp(bound, &e);
    *scale = ldexp(1.0, 61 - e);
  }
}

// Shell sums over the half spectrum [kz][ky][kx] (kx = 0 .. D/2).  A thread adds
// the up to four values (+-ky, +-kz) of a shell before it adds to LDS, where a
// sum has kShellCopies places in different banks: neighbouring lanes share
// shells.  One block per CU: each adds all its shells to memory, and 2048 blocks
// queued up there (256^3, 135 MB: 54 us, now 28).
__global__ void __launch_bounds__(1024)
k_fsc_shells(const float2 *fa, const float2 *fb, int D, const double *scale,
             unsigned long long *sums) {
  extern __shared__ unsigned long long ls[];  // [3][ns][kShellCopies]
  const int ns = D / 2 + 1, Dh = D / 2 + 1;
  for (int i = threadIdx.x; i < 3 * ns * kShellCopies; i += 1024) ls[i] = 0ull;
  __syncthreads();
  const double S = *scale;
  const unsigned total = (unsigned)Dh * Dh * Dh;
  for (unsigned i = blockIdx.x * 1024 + threadIdx.x; i < total; i += gridDim.x * 1024) {
    const unsigned r = i / (unsigned)Dh;
    const int kx = (int)(i - r * Dh), fz = (int)(r / (unsigned)Dh), fy = (int)r - fz * Dh;
    // (exact: the root of an integer below 2^18 stays 2^-12 away from a half)
    const int s = (int)rintf(sqrtf((float)(kx * kx + fy * fy + fz * fz)));
    if (s > D / 2) continue;
    const double w = (kx == 0 || kx == D / 2) ? 1.0 : 2.0;
    long long num = 0, da = 0, db = 0;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      if ((u & 1 && (fy == 0 || fy == D / 2)) || (u & 2 && (fz == 0 || fz == D / 2))) continue;
      const int64_t at = ((int64_t)(u & 2 ? D - fz : fz) * D + (u & 1 ? D - fy : fy)) * Dh + kx;
      const float2 a = fa[at], b = fb[at];
      num += __double2ll_rn(w * ((double)a.x * b.x + (double)a.y * b.y) * S);
      da += __double2ll_rn(w * ((double)a.x * a.x + (double)a.y * a.y) * S);
      db += __double2ll_rn(w * ((double)b.x * b.x + (double)b.y * b.y) * S);
    }
    unsigned long long *l = ls + s * kShellCopies + threadIdx.x % kShellCopies;
    atomicAdd(l, (unsigned long long)num);
    atomicAdd(l + ns * kShellCopies, (unsigned long long)da);
    atomicAdd(l + 2 * ns * kShellCopies, (unsigned long long)db);
  }
  __syncthreads();
  for (int i = threadIdx.x; i < 3 * ns; i += 1024) {
    unsigned long long v = 0ull;
    for (int c = 0; c < kShellCopies; ++c) v += ls[i * kShellCopies + c];
    if (v) atomicAdd(&sums[i], v);
  }
}

__global__ void __launch_bounds__(256)
k_fsc_final(const unsigned long long *sums, int ns, const double *scale, float *fsc) {
  const int s = blockIdx.x * 256 + threadIdx.x;
  if (s >= ns) return;
  const double S = *scale;
  const double num = (double)(long long)sums[s] / S;
  const double da = (double)(long long)sums[ns + s] / S, db = (double)(long long)sums[2 * ns + s] / S;
  const double den = sqrt(da * db);
  fsc[s] = den > 0.0 ? (float)(num / den) : 0.f;
}

// Resolution read-out of an FSC curve: the first shell k >= 1 whose
// correlation is below the threshold (the last shell, D/2, when none is),
// and D p / k in Angstrom.  One wave: a ballot over the shells in order.
__global__ void __launch_bounds__(64)
k_fsc_resolution(const float *fsc, int ns, int D, float pixel, float threshold, int *shell,
                 float *resolution) {
  int first = ns - 1;
  for (int base = 1; base < ns; base += 64) {
    const int k = base + (int)threadIdx.x;
    const unsigned long long below = __ballot(k < ns && fsc[k] < threshold);
    if (below) {
      first = base + __ffsll((long long)below) - 1;
      break;
    }
  }
  if (threadIdx.x == 0) {
    if (shell) *shell = first;
    if (resolution) *resolution = (float)((double)D * (double)pixel / (double)first);
  }
}

__global__ void __launch_bounds__(256) k_fill_u64z(unsigned long long *p, int n) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i < n) p[i] = 0ull;
}

__global__ void __launch_bounds__(256) k_fill_i32z(int *p, int n) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i < n) p[i] = 0;
}

}  // namespace cs
