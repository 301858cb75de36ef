// Forward and adjoint splat kernels (Alg. 2 SumSplats and its backward).
//
// Work decomposition: every visible (image, Gaussian) record belongs to one
// owner tile (T x T pixels); its whole truncated footprint lies inside the
// tile's canvas, the tile plus a halo on every side.  A work item is a chunk
// of at most `budget` records of one owner tile.  Inside an item each lane
// owns one Gaussian and walks its exact footprint row by row: the row span
// comes from the q_cut ellipse, and along a row the Gaussian obeys the
// two-multiply recurrence
//     e(j+1) = e(j) r(j),   r(j+1) = r(j) K,   K = exp(-a)
// (a is the pixel-unit conic's xx entry), so no transcendental is evaluated
// per pixel.  The forward accumulates into an LDS canvas in 32-bit fixed
// point with integer LDS atomics (LDS float atomics are ~30x slower on
// gfx950; integer addition also makes the sum order-independent, matching
// the order-free additive splat of Sec. 3.3.4).  The fixed-point scale of
// an item is the largest power of two with scale * sum|w| <= 2^30, so no
// pixel can overflow.  The backward reads G_Q from an LDS copy of the
// canvas region and accumulates the six pixel moments per Gaussian in
// registers, so no per-pixel state is stored between the passes.
#include "cs_internal.hpp"

namespace cs {

// Hardware exp2/sqrt (v_exp_f32 / v_sqrt_f32, about 1 ulp; results below
// 2^-126 flush to zero, far under the 1e-6 truncation of every term).
__device__ __forceinline__ float hexp2(float x) { return __builtin_amdgcn_exp2f(x); }
__device__ __forceinline__ float hsqrt(float x) { return __builtin_amdgcn_sqrtf(x); }

// Exact column span of the row at vertical offset di = i - v for the
// ellipse q <= q_cut, clipped to [clo, chi]: first column j0 and length L
// (false for an empty row).  aqk = al * qk.  The span ends are converted to
// integers before clamping (finite here: al > 0 and the record fits its
// canvas).
__device__ __forceinline__ bool row_span(float u, float di, float al, float be, float det_s,
                                         float inv_al, float aqk, int clo, int chi, int &j0,
                                         int &L) {
  const float disc = aqk - det_s * di * di;
  if (!(disc >= 0.f)) return false;
  const float h = hsqrt(disc) * inv_al;
  const float cen = u - be * di * inv_al;
  j0 = max((int)ceilf(cen - h), clo);
  L = min((int)floorf(cen + h), chi) - j0 + 1;
  return L > 0;
}

// Row of flat index x in rows of length n: x / n through a float reciprocal
// (exact while x < 2^20 and n <= 1024: the quotient (x + 1/2) / n stays at
// least 1 / (2 n) away from an integer, far above the rounding error).
__device__ __forceinline__ int row_of(int x, float inv_n) {
  return (int)(((float)x + 0.5f) * inv_n);
}

// Work items in turn: the first problem's first gridDim.x items go to the blocks
// by their index, the rest through the counter.  A block of a small call takes
// its one item without a round trip to the counter, which every block of the
// launch would queue up for twice.  A block barrier lies between the last next()
// of one problem and the first of the next one: only then has every wave read the
// slot that the first thread is about to overwrite.
struct ItemQueue {
  int *counter, *slot;
  int nitems, first, base;
  __device__ ItemQueue(int *counter, int *slot, int nitems, int p)
      : counter(counter), slot(slot), nitems(nitems), first(p == 0 ? (int)blockIdx.x : -1),
        base(p == 0 ? (int)gridDim.x : 0) {}
  __device__ int next() {  // nitems or more: none left
    if (first >= 0) {
      const int it = first;
      first = -1;
      return it;
    }
    if (base >= nitems) return nitems;
    if (threadIdx.x == 0) *slot = base + atomicAdd(counter, 1);
    __syncthreads();
    return *slot;
  }
};

// ---------------------------------------------------------------------------
// Dealing records to lanes.  Every lane walks its own Gaussian, so at a step
// the lanes of a wave touch canvas words around their own centres; words of
// equal address mod 64 fall into one LDS bank and serialise.  With rows of
// S words, a lane's word at row i, column j sits in bank (S i + j) mod 64;
// as all lanes step rows and columns together, the bank of lane l is
// key_l + w_l + (a common offset), where key_l = (S i0_l + floor(u_l)) mod 64
// (its first row and centre column) and w_l in {0, 1} the rounding of its
// span start.  A chunk of kDealChunk records is therefore put in an order in
// which every 64 consecutive records carry distinct keys, the first 32 even
// keys and the last 32 odd keys: records are grouped by key, and round r
// takes the r-th record of every group in the order 0, 2, ..., 62, 1, 3,
// ..., 63 (a record's place is the size of the earlier rounds plus the
// non-empty groups before its own in its round).  Within a half-wave the keys
// then differ by at least 2, so the span-start rounding cannot make two lanes
// meet.  The order only changes which lane takes which record: every result
// is the same.  Groups of more than kDealRounds records keep the list order.
// Dealing costs a pass over the chunk's records and pays where footprints
// are wide (many steps per record); it is the launch option lane_order = 1,
// chosen per problem by the autotuner.
// ---------------------------------------------------------------------------
constexpr int kDealChunk = 512;
constexpr int kDealRounds = 32;

struct DealLds {
  unsigned long long M[kDealRounds];  // round r: groups with more than r records
  int R[kDealRounds];                 // records in rounds before r
  int cnt[64];
  unsigned short perm[kDealChunk];    // place -> record (within the chunk)
  int ok;
};

__device__ __forceinline__ void deal(const float4 *list, size_t base, int n, int S, int R0, int C0,
                                     DealLds &d) {
  const int t = threadIdx.x;
  if (t < 64) d.cnt[t] = 0;
  __syncthreads();
  constexpr int kPer = kDealChunk / kBlock;
  int key[kPer], rows[kPer];
  float u[kPer];
#pragma unroll
  for (int j = 0; j < kPer; ++j) {  // (past the end: the last record, unused)
    const size_t g = base + min(t + j * kBlock, n - 1);
    u[j] = list[2 * g].x;
    rows[j] = __float_as_int(list[2 * g + 1].w);
  }
#pragma unroll
  for (int j = 0; j < kPer; ++j) {
    const int g = t + j * kBlock;
    key[j] = -1;
    if (g < n) {
      const int k = (S * ((rows[j] & 0xffff) - R0) + (int)floorf(u[j]) - C0) & 63;
      const int grp = (k >> 1) | ((k & 1) << 5);  // even keys first, then odd
      key[j] = (atomicAdd(&d.cnt[grp], 1) << 6) | grp;
    }
  }
  __syncthreads();
  if (t < 64) {  // one wave lays out the rounds
    const int c = d.cnt[t];
    int mx = c;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) mx = max(mx, __shfl_xor(mx, o, 64));
    const bool ok = mx <= kDealRounds;
    if (ok) {
      int run = 0;
      for (int r = 0; r < mx; ++r) {
        const unsigned long long m = __ballot(c > r);
        if (t == 0) {
          d.M[r] = m;
          d.R[r] = run;
        }
        run += __popcll(m);
      }
    }
    if (t == 0) d.ok = ok;
  }
  __syncthreads();
  const bool ok = d.ok;
#pragma unroll
  for (int j = 0; j < kPer; ++j) {
    if (key[j] < 0) continue;
    const int g = t + j * kBlock;
    int pos = g;
    if (ok) {
      const int r = key[j] >> 6, grp = key[j] & 63;
      pos = d.R[r] + __popcll(d.M[r] & ((1ull << grp) - 1ull));
    }
    d.perm[pos] = (unsigned short)g;
  }
  __syncthreads();
}

// ---------------------------------------------------------------------------
// Sorting records by footprint shape.  A wave steps as many rows as its
// tallest footprint and, per row, as many pixel groups as its widest active
// span, so where footprint sizes spread (anisotropic Gaussians with
// log-normal scales) most lanes idle for most steps.  Launch option
// lane_order = 2 orders each chunk of kSortChunk records by (row count,
// width class) with a counting sort in LDS: the row count is the record's
// row range clipped to the canvas (capped at 31), the width class the
// widest span, 2 sqrt(qk / a) at the centre row, in steps of four pixels
// (capped at 7).  The order among equal keys follows the LDS atomics and
// is not fixed, which is harmless: as with the dealt order, only the lane
// that walks a record changes, never its arithmetic, and the forward sums
// are order-free integers, so every result is the same.
//
// Forward, an item keeps its list order from the first chunk on of which more than
// an eighth is as tall as the canvas: sorted, the lanes of a wave would all start
// on its first row and add to the same addresses (rendering 37 images of 24 x 24,
// 20000 Gaussians of sd 3 pixels, 915 us sorted and 796 in list order; 16 images of
// 32 x 32, 66000, 1151 and 954; of sd 1 pixel 142 and 174).  At a sixteenth those
// of sd 1 pixel in 16 x 16 would lose 6 %.  The adjoint adds to no shared pixels
// and gains from the sort there, too.
// ---------------------------------------------------------------------------
constexpr int kSortChunk = 1024;
constexpr int kSortKeys = 256;  // 32 row counts x 8 width classes
static_assert(kSortKeys == kBlock, "one key counter per thread");

struct SortLds {
  int start[kSortKeys];
  int wsum[kBlock / 64];
  int full;  // records as tall as the canvas
  unsigned short perm[kSortChunk];  // place -> record (within the chunk)
};

union OrderLds {
  DealLds deal;
  SortLds sort;
};

template <bool kForward>
__device__ __forceinline__ bool size_sort(const float4 *list, size_t base, int n, int rlo, int rhi,
                                          float qk, SortLds &d) {
  const int t = threadIdx.x;
  d.start[t] = 0;
  if (t == 0) d.full = 0;
  __syncthreads();
  constexpr int kPer = kSortChunk / kBlock;
  int key[kPer], rows[kPer];
  float al[kPer];
  int full = 0;
#pragma unroll
  for (int j = 0; j < kPer; ++j) {  // (past the end: the last record, unused)
    const size_t g = base + min(t + j * kBlock, n - 1);
    al[j] = list[2 * g].z;
    rows[j] = __float_as_int(list[2 * g + 1].w);
  }
#pragma unroll
  for (int j = 0; j < kPer; ++j) {
    const int g = t + j * kBlock;
    key[j] = -1;
    if (g < n) {
      const int nr = min(rows[j] >> 16, rhi) - max(rows[j] & 0xffff, rlo) + 1;
      full += nr > rhi - rlo;
      const int wc = (int)fminf(2.f * hsqrt(qk * __builtin_amdgcn_rcpf(al[j])), 64.f) >> 2;
      const int k = min(max(nr, 0), 31) * 8 + min(wc, 7);
      key[j] = (atomicAdd(&d.start[k], 1) << 8) | k;
    }
  }
  if (kForward) {
    if (full) atomicAdd(&d.full, full);
    __syncthreads();
    if (8 * d.full > n) return false;
  } else {
    __syncthreads();
  }
  // exclusive scan of the key counts: wave scans, then the wave totals
  const int c = d.start[t];
  int x = c;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int y = __shfl_up(x, o, 64);
    if ((t & 63) >= o) x += y;
  }
  if ((t & 63) == 63) d.wsum[t >> 6] = x;
  __syncthreads();
  int off = x - c;
  for (int w = 0; w < (t >> 6); ++w) off += d.wsum[w];
  d.start[t] = off;
  __syncthreads();
#pragma unroll
  for (int j = 0; j < kPer; ++j)
    if (key[j] >= 0) d.perm[d.start[key[j] & 255] + (key[j] >> 8)] = (unsigned short)(t + j * kBlock);
  __syncthreads();
  return true;
}

// Records per ordered chunk for an item of w records, by lane_order.
__device__ __forceinline__ int chunk_len(const Geom &G, int w) {
  return G.deal == 1 ? kDealChunk : G.deal == 2 ? kSortChunk : w;
}

// Orders one chunk of records as the launch option lane_order asks and
// returns the place -> record map (null: list order).  Block-wide: every
// thread of the block calls it.
template <bool kForward>
__device__ __forceinline__ const unsigned short *order_records(const float4 *list, size_t base,
                                                               int n, const Geom &G, int R0, int C0,
                                                               int rlo, int rhi, OrderLds &o) {
  if (G.deal == 1) {
    deal(list, base, n, G.S, R0, C0, o.deal);
    return o.deal.perm;
  }
  if (G.deal == 2) {
    return size_sort<kForward>(list, base, n, rlo, rhi, G.qk, o.sort) ? o.sort.perm : nullptr;
  }
  return nullptr;
}

// Place in the order of a thread's record k: each wave takes 64 / RS adjacent
// places of every block-wide group, the waves in turn forwards and backwards, so
// that in the order by footprint none has the larger ones every time (they meet at
// a barrier after the chunk).  With the orders' keys read together before their LDS
// atomics (a chunk was four round trips one after another) this took the loss and
// gradient of 256 images of 128 x 128 from 789 to 771 us (773 without the turns)
// and the uneven batch of eight mixtures from 7655 to 7486 us.
template <int RS>
__device__ __forceinline__ int place(int k) {
  const int wv = threadIdx.x >> 6, lane = threadIdx.x & 63;
  return (k * (kBlock / 64) + (k & 1 ? kBlock / 64 - 1 - wv : wv)) * (64 / RS) + lane / RS;
}

// A thread's first record in list order, requested with the work item where
// several lanes share one (small calls, whose items are one pass of the block):
// its round trip runs beside the item's other loads.
template <int RS>
struct FirstRecord {
  size_t rec;
  float4 r0, r1;
  __device__ FirstRecord(const float4 *list, const int4 &itm) {
    if (RS == 1) return;
    rec = 2 * ((size_t)itm.z + min((int)threadIdx.x / RS, itm.w - 1));
    r0 = list[rec];
    r1 = list[rec + 1];
  }
  __device__ void get(const float4 *list, size_t at, float4 &a, float4 &b) {
    if (RS > 1 && at == rec) {
      a = r0;
      b = r1;
    } else {
      a = list[at];
      b = list[at + 1];
    }
  }
};

// ---------------------------------------------------------------------------
// Forward: partial canvas of one work item.  RS adjacent lanes share a record,
// taking every RS-th of its rows: 1 where there are records enough to fill the
// chip, 4 for smaller calls, whose time is one wave's walk over its tallest
// footprint (one image of 1000 Gaussians: 24 -> 9.5 us with tiles of 32 beside;
// eight lanes gave no more).  The sums are integers, so the lanes' order is free.
// ---------------------------------------------------------------------------
template <int RS>
__global__ void __launch_bounds__(kBlock) k_splat_fwd_rs(MultiProb MP) {
  extern __shared__ int4 smem4[];     // 16-byte aligned dynamic LDS
  int *icanvas = (int *)smem4;        // C rows of stride S (fixed point)
  __shared__ int slot;
  __shared__ float wsum[kBlock / 64];
  __shared__ OrderLds ol;
  // drain the problems' queues in order: blocks that find one exhausted move on
  for (int p = 0; p < MP.count; ++p) {
  if (p > 0) __syncthreads();  // the slot has been read
  const Geom G = MP.p[p].G;
  const float4 *list = MP.p[p].list;
  const int4 *items = MP.p[p].items;
  float *partials = MP.p[p].partials;
  const int nitems = *MP.p[p].n_items;
  ItemQueue queue(MP.p[p].queue, &slot, nitems, p);
  const int CS = G.C * G.S;
  for (;;) {
    const int it = queue.next();
    if (it >= nitems) break;
    for (int i = threadIdx.x; i < CS / 4; i += kBlock) smem4[i] = make_int4(0, 0, 0, 0);
    for (int i = (CS & ~3) + threadIdx.x; i < CS; i += kBlock) icanvas[i] = 0;
    const int4 itm = items[it];
    FirstRecord<RS> fr(list, itm);
    // fixed-point scale: 2^e with 2^e * sum|w| <= 2^30 (the item's |w| are
    // contiguous beside the list, summed in a fixed order)
    const float *wa = MP.p[p].wabs + itm.z;
    float aw = 0.f;
    // four loads in flight per thread, added in the same order as one at a time
    int g = threadIdx.x;
    for (; g + 3 * kBlock < itm.w; g += 4 * kBlock) {
      const float a0 = wa[g], a1 = wa[g + kBlock], a2 = wa[g + 2 * kBlock], a3 = wa[g + 3 * kBlock];
      aw += a0;
      aw += a1;
      aw += a2;
      aw += a3;
    }
    for (; g < itm.w; g += kBlock) aw += wa[g];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) aw += __shfl_xor(aw, o, 64);
    if ((threadIdx.x & 63) == 0) wsum[threadIdx.x >> 6] = aw;
    __syncthreads();
    const float tot = wsum[0] + wsum[1] + wsum[2] + wsum[3];
    int ex = 0;
    if (tot > 0.f && isfinite(tot)) {
      frexpf(tot, &ex);          // tot in [2^(ex-1), 2^ex)
      ex = min(max(30 - ex, -126), 126);  // 2^ex * tot < 2^30 (unless clamped)
    }
    const float scale = ldexpf(1.f, ex), inv_scale = ldexpf(1.f, -ex);
    const int ty = itm.y / G.ntx, tx = itm.y % G.ntx;
    const int R0 = ty * G.T - G.halo, C0 = tx * G.T - G.halo;
    const int rlo = max(R0, 0), rhi = min(R0 + G.C - 1, G.D - 1);
    const int clo = max(C0, 0), chi = min(C0 + G.C - 1, G.D - 1);
    __syncthreads();  // canvas cleared
    const int chunk = chunk_len(G, itm.w);
    for (int c0 = 0, nc; c0 < itm.w; c0 += nc) {
    nc = min(chunk, itm.w - c0);
    const unsigned short *perm =
        order_records<true>(list, (size_t)itm.z + c0, nc, G, R0, C0, rlo, rhi, ol);
    if (!perm) nc = itm.w - c0;  // the rest in list order, too
    for (int k = 0; k * (kBlock / RS) < nc; ++k) {
      const int s = place<RS>(k);
      if (s >= nc) continue;
      const size_t rec = 2 * ((size_t)itm.z + c0 + (perm ? perm[s] : s));
      float4 r0, r1;
      fr.get(list, rec, r0, r1);
      const float u = r0.x, v = r0.y, al = r0.z, be = r0.w, ga = r1.x, w = r1.y * scale;
      const int rows = __float_as_int(r1.w);
      const int i0 = max(rows & 0xffff, rlo) + (int)threadIdx.x % RS, i1 = min(rows >> 16, rhi);
      const float det_s = al * ga - be * be;
      const float inv_al = 1.f / al;
      const float aqk = al * G.qk;
      const float K = hexp2(-2.f * al);
      float fi = (float)i0;
      int rowo = (i0 - R0) * G.S - C0;  // canvas offset of (row i, column 0)
      for (int i = i0; i <= i1; i += RS, fi += (float)RS, rowo += RS * G.S) {
        const float di = fi - v;
        int j0, L;
        if (!row_span(u, di, al, be, det_s, inv_al, aqk, clo, chi, j0, L)) continue;
        const float dj = (float)j0 - u;
        float e = w * hexp2(-(al * dj * dj + 2.f * be * dj * di + ga * di * di));
        float r = hexp2(-(al * (2.f * dj + 1.f) + 2.f * be * di));
        int *px = icanvas + rowo + j0;
        const int L4 = L & ~3;
        for (int k = 0; k < L4; k += 4) {
          const int v0 = __float2int_rn(e); e *= r; r *= K;
          const int v1 = __float2int_rn(e); e *= r; r *= K;
          const int v2 = __float2int_rn(e); e *= r; r *= K;
          const int v3 = __float2int_rn(e); e *= r; r *= K;
          atomicAdd(px + k, v0);
          atomicAdd(px + k + 1, v1);
          atomicAdd(px + k + 2, v2);
          atomicAdd(px + k + 3, v3);
        }
        if (L4 < L) {  // 1 to 3 trailing pixels
          const int v0 = __float2int_rn(e); e *= r; r *= K;
          const int v1 = __float2int_rn(e); e *= r;
          const int v2 = __float2int_rn(e);
          atomicAdd(px + L4, v0);
          if (L4 + 1 < L) atomicAdd(px + L4 + 1, v1);
          if (L4 + 2 < L) atomicAdd(px + L4 + 2, v2);
        }
      }
    }
    __syncthreads();  // the next chunk rewrites the order
    }
    float *out = partials + (size_t)it * G.C * G.C;
    const float inv_c = 1.f / (float)G.C;
    for (int i = threadIdx.x; i < G.C * G.C; i += kBlock) {
      const int r = row_of(i, inv_c), c = i - r * G.C;
      out[i] = (float)icanvas[r * G.S + c] * inv_scale;
    }
    __syncthreads();
  }
  }
}

// ---------------------------------------------------------------------------
// Wide Gaussians (footprint larger than the canvas): exp per pixel of their
// pixel box.
// ---------------------------------------------------------------------------
__device__ __forceinline__ void wide_box(const float4 r0, const float4 r1, const Geom &G,
                                         int &i0, int &i1, int &j0, int &j1) {
  const int rows = __float_as_int(r1.w);
  i0 = rows & 0xffff;
  i1 = rows >> 16;
  const float det_s = r0.z * r1.x - r0.w * r0.w;
  const float hx = sqrtf(G.qk * r1.x / det_s);
  j0 = clamp_px(ceilf(r0.x - hx), 0, G.D);
  j1 = clamp_px(floorf(r0.x + hx), -1, G.D - 1);
}

// ---------------------------------------------------------------------------
// Q for one (image, tile): every pixel sums, in a fixed order, the partial
// canvases of the owner tiles whose canvas covers it (its own tile and the
// neighbours whose halo reaches it).  When tile, halo and D are multiples
// of 4, a thread takes four adjacent pixels of a row (16-byte loads) and
// keeps four items in flight.  The image's wide records follow: those whose box
// meets the block's rows are gathered in LDS, in list order, and every pixel
// sums their terms in FP64 in that order before adding them to Q.  That replaces
// a kernel per record with a 64-bit atomic per pixel and two passes over the
// images: 16 images of 256 x 256 with 20000 records of sd 13 pixels each took
// 50 ms for loss and gradient, now 21 ms, and calls without wide records three
// launches fewer.
//
// S threads share a pixel group, each taking every S-th item and record, and
// their sums are added in order: 1 where the tiles alone fill the chip, 4 for
// calls of few images, whose time is one thread's walk over its items, 16 or 64
// where those few images have many Gaussians, whose wide records would otherwise
// be a few blocks' work (one image of 100 x 100, 500000 Gaussians of sd 3.5 pixels:
// 8.0 ms with 4 threads, 2.6 ms with 16).
// ---------------------------------------------------------------------------
__device__ __forceinline__ float4 f4add(float4 a, float4 b) {
  return make_float4(a.x + b.x, a.y + b.y, a.z + b.z, a.w + b.w);
}

template <int S>
__global__ void __launch_bounds__(kBlock)
k_canvas_reduce_s(const float *partials, const int *item_off, const int *n_items, const int *off,
                  const int *count, const float4 *list, Geom G, float *Q) {
  constexpr int kPix = kBlock / S;  // pixel groups per block and pass
  // XCD-aware order: a work index runs over the z-split parts of a tile,
  // then the tiles of an image, so the blocks that read one canvas (its own
  // and its neighbours' halos) meet in one XCD's L2
  const int zsplit = gridDim.z;
  const int j = xcd_work(blockIdx.x + gridDim.x * (blockIdx.y + gridDim.y * blockIdx.z),
                         gridDim.x * gridDim.y * zsplit);
  const int zz = j % zsplit, t = (j / zsplit) % gridDim.x, b = j / (zsplit * gridDim.x);
  const int ty = t / G.ntx, tx = t % G.ntx;
  // item ranges of the 3 x 3 owner tiles around this one (empty outside the
  // image), read once per block rather than per pixel and neighbour
  __shared__ int2 range[9];
  __shared__ float4 wrec[kBlock][2];
  __shared__ int kept[kBlock / 64];
  __shared__ float4 facc[S > 1 ? kBlock : 1];
  __shared__ double4 dacc[S > 1 ? kBlock : 1];
  const int n_wide = n_items[1] > 0 ? count[b * G.K + G.ntiles] : 0;
  if (threadIdx.x < 9) {
    const int sy = ty + threadIdx.x / 3 - 1, sx = tx + threadIdx.x % 3 - 1;
    int2 r = make_int2(0, 0);
    if (sy >= 0 && sy < G.ntx && sx >= 0 && sx < G.ntx) {
      const int e = b * G.K + sy * G.ntx + sx;
      r = make_int2(item_off[e], item_off[e + 1]);
    }
    range[threadIdx.x] = r;
  }
  __syncthreads();
  const int r_lo = ty * G.T, r_hi = min(r_lo + G.T, G.D);
  const int c_lo = tx * G.T, c_hi = min(c_lo + G.T, G.D);
  const int wdt = c_hi - c_lo;
  float *img = Q + (size_t)b * G.D * G.D;
  const size_t CC = (size_t)G.C * G.C;
  const bool vec = (G.T % 4 == 0) && (G.halo % 4 == 0) && (G.D % 4 == 0);
  const int px_per = vec ? 4 : 1;
  const int wq = wdt / px_per;
  const int nq = (r_hi - r_lo) * wq;
  const int part = S > 1 ? threadIdx.x / kPix : 0;
  for (int q0 = zz * kPix; q0 < nq; q0 += kPix * zsplit) {
    const int q = q0 + threadIdx.x % kPix;
    const bool live = q < nq;
    if (S == 1 && n_wide == 0 && !live) continue;
    const int i = r_lo + q / wq, j = c_lo + px_per * (q % wq);
    float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
    int phase = 0;  // items of the ranges before, modulo S
    for (int dy = live ? -1 : 2; dy <= 1; ++dy) {
      const int sy = ty + dy;
      if (sy < 0 || sy >= G.ntx) continue;
      const int ri = i - (sy * G.T - G.halo);
      if (ri < 0 || ri >= G.C) continue;
      for (int dx = -1; dx <= 1; ++dx) {
        const int sx = tx + dx;
        if (sx < 0 || sx >= G.ntx) continue;
        const int cj = j - (sx * G.T - G.halo);
        if (cj < 0 || cj >= G.C) continue;
        const int2 r = range[3 * (dy + 1) + dx + 1];
        const int it0 = r.x + (S > 1 ? (part - phase) & (S - 1) : 0), it1 = r.y;
        if (S > 1) phase = (phase + r.y - r.x) & (S - 1);
        const float *base = partials + (size_t)ri * G.C + cj;
        if (vec) {
          int it = it0;
          for (; it + 3 * S < it1; it += 4 * S) {
            const float4 a0 = *(const float4 *)(base + (size_t)it * CC);
            const float4 a1 = *(const float4 *)(base + (size_t)(it + S) * CC);
            const float4 a2 = *(const float4 *)(base + (size_t)(it + 2 * S) * CC);
            const float4 a3 = *(const float4 *)(base + (size_t)(it + 3 * S) * CC);
            acc = f4add(acc, f4add(f4add(a0, a1), f4add(a2, a3)));
          }
          for (; it < it1; it += S) acc = f4add(acc, *(const float4 *)(base + (size_t)it * CC));
        } else {
          for (int it = it0; it < it1; it += S) acc.x += base[(size_t)it * CC];
        }
      }
    }
    if (n_wide > 0) {
      const float4 *wl = list + 2 * (size_t)off[b * G.K + G.ntiles];
      const int ra = r_lo + q0 / wq, rb = min(r_lo + (q0 + kPix - 1) / wq, r_hi - 1);
      double wide[4] = {0.0, 0.0, 0.0, 0.0};
      for (int c0 = 0; c0 < n_wide; c0 += kBlock) {
        const int k = c0 + threadIdx.x;
        float4 r0 = make_float4(0, 0, 0, 0), r1 = r0;
        bool keep = false;
        if (k < n_wide) {
          r0 = wl[2 * (size_t)k];
          r1 = wl[2 * (size_t)k + 1];
          int i0, i1, j0, j1;
          wide_box(r0, r1, G, i0, i1, j0, j1);
          keep = i0 <= rb && i1 >= ra && j0 < c_hi && j1 >= c_lo;
          r1.z = __int_as_float(j0 | (j1 << 16));
        }
        const unsigned long long bits = __ballot(keep);
        const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
        if (lane == 0) kept[wv] = __popcll(bits);
        __syncthreads();
        int at = __popcll(bits & ((1ull << lane) - 1ull)), total = 0;
        for (int w = 0; w < kBlock / 64; ++w) {
          at += w < wv ? kept[w] : 0;
          total += kept[w];
        }
        if (keep) {
          wrec[at][0] = r0;
          wrec[at][1] = r1;
        }
        __syncthreads();
#pragma unroll 2
        for (int m = part; m < total; m += S) {
          const float4 a = wrec[m][0], c = wrec[m][1];
          const int rows = __float_as_int(c.w), cols = __float_as_int(c.z);
          const bool in = i >= (rows & 0xffff) && i <= (rows >> 16);
          const float di = (float)i - a.y;
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            if (e >= px_per) break;
            const float dj = (float)(j + e) - a.x;
            const float qq = a.z * dj * dj + 2.f * a.w * dj * di + c.x * di * di;
            const bool on = in && j + e >= (cols & 0xffff) && j + e <= (cols >> 16) && qq <= G.qk;
            wide[e] += on ? (double)(c.y * hexp2(-qq)) : 0.0;
          }
        }
        __syncthreads();
      }
      if (S > 1) {
        dacc[threadIdx.x] = make_double4(wide[0], wide[1], wide[2], wide[3]);
        __syncthreads();
        if (part == 0)
          for (int p = 1; p < S; ++p) {
            const double4 d = dacc[threadIdx.x + p * kPix];
            wide[0] += d.x;
            wide[1] += d.y;
            wide[2] += d.z;
            wide[3] += d.w;
          }
      }
      if (part == 0) {
        acc.x += (float)wide[0];
        acc.y += (float)wide[1];
        acc.z += (float)wide[2];
        acc.w += (float)wide[3];
      }
    }
    if (S > 1) {
      facc[threadIdx.x] = acc;
      __syncthreads();
      if (part == 0)
        for (int p = 1; p < S; ++p) acc = f4add(acc, facc[threadIdx.x + p * kPix]);
      __syncthreads();
    }
    if (!live || part) continue;
    float *o = img + (size_t)i * G.D + j;
    if (vec) {
      *(float4 *)o = acc;
    } else {
      o[0] = acc.x;
    }
  }
}
template __global__ void k_canvas_reduce_s<1>(const float *, const int *, const int *, const int *, const int *,
                                              const float4 *, Geom, float *);
template __global__ void k_canvas_reduce_s<4>(const float *, const int *, const int *, const int *, const int *,
                                              const float4 *, Geom, float *);
template __global__ void k_canvas_reduce_s<16>(const float *, const int *, const int *, const int *, const int *,
                                               const float4 *, Geom, float *);
template __global__ void k_canvas_reduce_s<64>(const float *, const int *, const int *, const int *, const int *,
                                               const float4 *, Geom, float *);

// ---------------------------------------------------------------------------
// Wide records k = part, part + parts, ... of one image in the adjoint, W waves
// to a record (1, or all four of the block): per-lane moments over its pixel box,
// then a fixed-order sum.  A block per record spends its time in the two barriers
// where records are small (8 images of 128 x 128, 2000 records each: 1.95 ms for
// loss and gradient with it and a division per pixel, 0.85 ms with a wave per
// record and the split sums of k_canvas_reduce), a wave per record leaves waves
// idle where they are few (50 records over one image of 512 x 512, adjoint: 733 us,
// with a block each 188).  A lane adds runs of eight pixels before it adds them to
// its sums, which keeps its chain of additions short in large images, and requests
// a pixel one step ahead; unrolled loops took more registers than the rest of the
// kernel leaves at seven waves per SIMD (training step of 64 images of 256 x 256
// 2,610 us with 88, 2,585 with 69).
// ---------------------------------------------------------------------------
template <int W>
__device__ __forceinline__ void wide_moments(const float4 *list, int start, int cnt, int part, int parts,
                                             const Geom &G, int b, const float *GQ, float *mom,
                                             float (*red)[6]) {
  constexpr int kStep = 64 * W;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, first = threadIdx.x % kStep;
  const float *img = GQ + (size_t)b * G.D * G.D;
  for (int k = part; k < cnt; k += parts) {
    const float4 r0 = list[2 * (size_t)(start + k)], r1 = list[2 * (size_t)(start + k) + 1];
    int i0, i1, j0, j1;
    wide_box(r0, r1, G, i0, i1, j0, j1);
    float m[6] = {0, 0, 0, 0, 0, 0};
    if (i1 >= i0 && j1 >= j0) {
      const int wdt = j1 - j0 + 1, npx = (i1 - i0 + 1) * wdt;
      // (row, column) of this lane's first pixel and of a step of kStep pixels
      int i = i0 + first / wdt, j = j0 + first % wdt;
      const int si = kStep / wdt, sj = kStep % wdt;
      float s[6] = {0, 0, 0, 0, 0, 0};
      float g = img[min(i, i1) * G.D + j];
#pragma unroll 1
      for (int q = first, k = 1; q < npx; q += kStep, ++k) {
        const float dj = (float)j - r0.x, di = (float)i - r0.y, now = g;
        i += si;
        j += sj;
        if (j > j1) {
          j -= wdt;
          ++i;
        }
        g = img[min(i, i1) * G.D + j];  // the next pixel's (past the end: one of the last row, unused)
        const float qq = r0.z * dj * dj + 2.f * r0.w * dj * di + r1.x * di * di;
        const float t = qq <= G.qk ? now * hexp2(-qq) : 0.f;
        s[0] += t; s[1] += t * dj; s[2] += t * di;
        s[3] += t * dj * dj; s[4] += t * dj * di; s[5] += t * di * di;
        if (k % 8 == 0) {
#pragma unroll
          for (int c = 0; c < 6; ++c) {
            m[c] += s[c];
            s[c] = 0.f;
          }
        }
      }
#pragma unroll
      for (int c = 0; c < 6; ++c) m[c] += s[c];
    }
#pragma unroll
    for (int c = 0; c < 6; ++c)
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) m[c] += __shfl_xor(m[c], o, 64);
    float *o = mom + ((size_t)b * G.N + __float_as_int(r1.z)) * 6;
    if (W == 1) {
      if (lane == 0) {
#pragma unroll
        for (int c = 0; c < 6; ++c) o[c] = m[c];
      }
    } else {
      if (lane == 0) {
#pragma unroll
        for (int c = 0; c < 6; ++c) red[wv][c] = m[c];
      }
      __syncthreads();
      if (threadIdx.x < 6) {
        const int c = threadIdx.x;
        o[c] = (red[0][c] + red[1][c]) + (red[2][c] + red[3][c]);
      }
      __syncthreads();
    }
  }
}

// ---------------------------------------------------------------------------
// Backward: six pixel moments per (image, Gaussian) of one work item,
//   m = sum G_Q e (1, dj, di, dj^2, dj di, di^2),  e = exp(-q/2),
// with dj = j - u, di = i - v (pixels).  Written to mom[(b N + n) 6 + k].
// ---------------------------------------------------------------------------
template <int RS>
__global__ void __launch_bounds__(kBlock) k_splat_bwd_rs(MultiProb MP) {
  extern __shared__ float gq[];  // C rows of stride S
  __shared__ int slot;
  __shared__ float wred[kBlock / 64][6];
  __shared__ OrderLds ol;
  for (int p = 0; p < MP.count; ++p) {
  if (p > 0) __syncthreads();  // the slot has been read
  const Geom G = MP.p[p].G;
  const float4 *list = MP.p[p].list;
  const int4 *items = MP.p[p].items;
  const float *GQ = MP.p[p].GQ;
  float *mom = MP.p[p].mom;
  const int nitems = *MP.p[p].n_items;
  ItemQueue queue(MP.p[p].queue + 1, &slot, nitems, p);
  for (;;) {
    const int it = queue.next();
    if (it >= nitems) break;
    const int4 itm = items[it];
    FirstRecord<RS> fr(list, itm);
    const int b = itm.x;
    const int ty = itm.y / G.ntx, tx = itm.y % G.ntx;
    const int R0 = ty * G.T - G.halo, C0 = tx * G.T - G.halo;
    const int rlo = max(R0, 0), rhi = min(R0 + G.C - 1, G.D - 1);
    const int clo = max(C0, 0), chi = min(C0 + G.C - 1, G.D - 1);
    const float *src = GQ + (size_t)b * G.D * G.D;
    const float inv_s = 1.f / (float)G.S;
    // G_Q of the canvas region into LDS (zero outside the image and in the
    // row padding): four unconditional loads in flight per thread (outside
    // the image they read the image's first value, then dropped)
    const int CS = G.C * G.S;
    for (int q0 = threadIdx.x; q0 < CS; q0 += 4 * kBlock) {
      float v[4];
      bool ok[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int q = q0 + u * kBlock;
        const int r = row_of(q, inv_s), c = q - r * G.S;
        const int i = R0 + r, j = C0 + c;
        ok[u] = q < CS && c < G.C && i >= 0 && i < G.D && j >= 0 && j < G.D;
        v[u] = src[ok[u] ? (size_t)i * G.D + j : 0];
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int q = q0 + u * kBlock;
        if (q < CS) gq[q] = ok[u] ? v[u] : 0.f;
      }
    }
    __syncthreads();
    const int chunk = chunk_len(G, itm.w);
    for (int c0 = 0; c0 < itm.w; c0 += chunk) {
    const int nc = min(chunk, itm.w - c0);
    const unsigned short *perm =
        order_records<false>(list, (size_t)itm.z + c0, nc, G, R0, C0, rlo, rhi, ol);
    for (int k = 0; k * (kBlock / RS) < nc; ++k) {
      const int s = place<RS>(k);
      if (s >= nc) continue;
      const size_t rec = 2 * ((size_t)itm.z + c0 + (perm ? perm[s] : s));
      float4 r0, r1;
      fr.get(list, rec, r0, r1);
      const float u = r0.x, v = r0.y, al = r0.z, be = r0.w, ga = r1.x;
      const int n = __float_as_int(r1.z);
      const int rows = __float_as_int(r1.w);
      const int i0 = max(rows & 0xffff, rlo) + (int)threadIdx.x % RS, i1 = min(rows >> 16, rhi);
      const float det_s = al * ga - be * be;
      const float inv_al = 1.f / al;
      const float aqk = al * G.qk;
      const float K = hexp2(-2.f * al);
      float m0 = 0.f, m1 = 0.f, m2 = 0.f, m3 = 0.f, m4 = 0.f, m5 = 0.f;
      float fi = (float)i0;
      int rowo = (i0 - R0) * G.S - C0;  // canvas offset of (row i, column 0)
      for (int i = i0; i <= i1; i += RS, fi += (float)RS, rowo += RS * G.S) {
        const float di = fi - v;
        int j0, L;
        if (!row_span(u, di, al, be, det_s, inv_al, aqk, clo, chi, j0, L)) continue;
        const float dj = (float)j0 - u;
        float e = hexp2(-(al * dj * dj + 2.f * be * dj * di + ga * di * di));
        float r = hexp2(-(al * (2.f * dj + 1.f) + 2.f * be * di));
        const float *px = gq + rowo + j0;
        // Prefix-sum moments over t_k = G_Q e, k = 0 .. M-1 (M steps, t_k = 0
        // for k >= L):
        //   a0 = sum t_k, a1 = sum t_k (M-k), a2 = sum t_k (M-k)(M-k+1)/2
        float a0 = 0.f, a1 = 0.f, a2 = 0.f;
        const int L4 = L & ~3;
        for (int k = 0; k < L4; k += 4) {
          const float g0 = px[k], g1 = px[k + 1], g2 = px[k + 2], g3 = px[k + 3];
          float t = g0 * e; e *= r; r *= K;
          a0 += t; a1 += a0; a2 += a1;
          t = g1 * e; e *= r; r *= K;
          a0 += t; a1 += a0; a2 += a1;
          t = g2 * e; e *= r; r *= K;
          a0 += t; a1 += a0; a2 += a1;
          t = g3 * e; e *= r; r *= K;
          a0 += t; a1 += a0; a2 += a1;
        }
        int M = L4;
        if (L4 < L) {
          // 1 to 3 trailing pixels as three steps with G_Q = 0 past the span.
          // The three reads are unconditional: the span ends at column C - 1
          // at most, so they reach column C + 1 at most, inside the row of
          // stride C + 4.
          const float g0 = px[L4], h1 = px[L4 + 1], h2 = px[L4 + 2];
          const float g1 = L4 + 1 < L ? h1 : 0.f;
          const float g2 = L4 + 2 < L ? h2 : 0.f;
          float t = g0 * e; e *= r; r *= K;
          a0 += t; a1 += a0; a2 += a1;
          t = g1 * e; e *= r;
          a0 += t; a1 += a0; a2 += a1;
          t = g2 * e;
          a0 += t; a1 += a0; a2 += a1;
          M = L4 + 3;
        }
        // sum t dj = c a0 - a1, sum t dj^2 = c^2 a0 - 2 c a1 + 2 a2 - a1, c = dj0 + M
        const float c = dj + (float)M;
        const float sdj = c * a0 - a1;
        const float sdj2 = c * (c * a0 - 2.f * a1) + 2.f * a2 - a1;
        m0 += a0;
        m1 += sdj;
        m2 += a0 * di;
        m3 += sdj2;
        m4 += sdj * di;
        m5 += a0 * di * di;
      }
#pragma unroll
      for (int o = 1; o < RS; o <<= 1) {  // the lanes of a record, in a fixed tree
        m0 += __shfl_xor(m0, o, 64);
        m1 += __shfl_xor(m1, o, 64);
        m2 += __shfl_xor(m2, o, 64);
        m3 += __shfl_xor(m3, o, 64);
        m4 += __shfl_xor(m4, o, 64);
        m5 += __shfl_xor(m5, o, 64);
      }
      if (RS > 1 && threadIdx.x % RS) continue;
      float *o = mom + ((size_t)b * G.N + n) * 6;
      o[0] = m0; o[1] = m1; o[2] = m2; o[3] = m3; o[4] = m4; o[5] = m5;
    }
    __syncthreads();  // the next chunk rewrites the order
    }
  }
  // wide records: unit (image, part) after unit; a block to a record where each
  // part has three at most, else a wave (200 records in each of 4 images of 256 x
  // 256, 128 parts: 217 us by waves, 107 by blocks; at four of a part's the waves
  // are all busy)
  if (MP.p[p].n_items[1] > 0) {
    const int parts = G.wide_parts, units = G.B * parts;
    for (int un = blockIdx.x; un < units; un += gridDim.x) {
      const int wb = un / parts, part = un % parts, e = wb * G.K + G.ntiles;
      const int start = MP.p[p].off[e], cnt = MP.p[p].count[e];
      if (cnt <= 3 * parts)
        wide_moments<4>(list, start, cnt, part, parts, G, wb, GQ, mom, wred);
      else
        wide_moments<1>(list, start, cnt, part * 4 + (threadIdx.x >> 6), parts * 4, G, wb, GQ, mom, wred);
    }
  }
  }
}
template __global__ void k_splat_fwd_rs<1>(MultiProb MP);
template __global__ void k_splat_bwd_rs<1>(MultiProb MP);
template __global__ void k_splat_fwd_rs<4>(MultiProb MP);
template __global__ void k_splat_bwd_rs<4>(MultiProb MP);

}  // namespace cs
