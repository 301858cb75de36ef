// Host side of the voxelisation and FSC entry points (cs_voxelize, cs_fsc).
#include <algorithm>

#include "../../include/cryosplat.h"
#include "cs_host.hpp"
#include "cs_volume.hpp"

using namespace cs;

namespace {

constexpr float kDefaultQCutVol = 27.631021115928547f;  // 2 ln 1e6, as the renderer

size_t al256v(size_t x) { return (x + 255) & ~size_t(255); }
unsigned cdivv(int64_t a, int64_t b) { return (unsigned)((a + b - 1) / b); }

}  // namespace

extern "C" {

int cs_voxelize(cs_ctx *ctx, const cs_gaussians *g, int32_t D, float pixel, float q_cut,
                float *vol, void *stream) {
  if (!ctx) return CS_ERR_INVALID_ARG;
  if (!g || !vol) return fail(ctx, CS_ERR_INVALID_ARG, "null gaussians or volume");
  if (g->n < 0) return fail(ctx, CS_ERR_INVALID_ARG, "negative Gaussian count");
  if (g->n > 0 && (!g->means || !g->log_scales || !g->quats || !g->amps))
    return fail(ctx, CS_ERR_INVALID_ARG, "null Gaussian parameter array");
  if (g->scale_act != 0 && g->scale_act != 1) return fail(ctx, CS_ERR_INVALID_ARG, "bad scale_act");
  if (g->amp_act != 0 && g->amp_act != 1) return fail(ctx, CS_ERR_INVALID_ARG, "bad amp_act");
  if (D < 8 || D % 8 != 0 || D > 512) return fail(ctx, CS_ERR_UNSUPPORTED, "D must be a multiple of 8 in [8, 512]");
  if (!(pixel > 0.f)) return fail(ctx, CS_ERR_INVALID_ARG, "voxel size must be positive");
  HIPCHK(hipSetDevice(ctx->device));
  hipStream_t st = (hipStream_t)stream;
  const int N = (int)g->n, nb = D / 8, nbr = nb * nb * nb;
  const int csh = nb <= 32 ? 1 : 2, nc = (nb + (1 << csh) - 1) >> csh, ncell = nc * nc * nc;
  // blocks of the counting kernels: at most one per CU, as each adds every cell it met
  const int per = (int)std::max<int64_t>(128, cdivv(N, 256));
  const VoxGeom V{N, D, D / 2, nb, csh, nc, per, pixel, q_cut > 0.f ? q_cut : kDefaultQCutVol};
  const size_t o_gc = 0, o_rec = o_gc + al256v((size_t)N * 48 + 16);
  const size_t o_box = o_rec + al256v((size_t)N * 48 + 16);
  const size_t o_tot = o_box + al256v((size_t)N * 16 + 16);  // totals and counts, cleared together
  const size_t o_cnt = o_tot + 16;
  const size_t o_cur = o_cnt + (size_t)ncell * 8;  // cleared with the counts
  const size_t o_off = al256v(o_cur + (size_t)ncell * 4);
  const size_t o_rng = o_off + al256v((size_t)(ncell + 1) * 8);
  const size_t o_scale = o_rng + al256v((size_t)nbr * 8);
  const int nwp = (int)cdivv(N, 256);  // blocks of k_vox_prep: partial sums of |w|
  const size_t o_wp = o_scale + 256;
  const size_t o_list = o_wp + al256v((size_t)nwp * 8 + 8);
  int rc = grow(ctx, &ctx->vol, &ctx->vol_bytes, o_list + 256);
  if (rc) return rc;
  // per-Gaussian records, brick counts and offsets, fixed-point scale
  auto prepare = [&]() -> int {
    char *w = (char *)ctx->vol;
    float4 *gc = (float4 *)(w + o_gc), *rec = (float4 *)(w + o_rec);
    TLAUNCH(k_fill_i32z, dim3(cdivv(3 * ncell + 4, 256)), dim3(256), 0, st, (int *)(w + o_tot), 3 * ncell + 4);
    if (N > 0) {
      Geom G{};
      G.N = N;
      G.scale_act = g->scale_act;
      G.amp_act = g->amp_act;
      TLAUNCH(k_build, dim3(cdivv(N, kBlock)), dim3(kBlock), 0, st, gauss_dev(*g), G, gc);
      TLAUNCH(k_vox_prep, dim3(nwp), dim3(256), 0, st, (const float4 *)gc, V, rec,
              (int4 *)(w + o_box), (double *)(w + o_wp));
      TLAUNCH(k_vox_count, dim3(cdivv(N, per)), dim3(1024), (size_t)ncell * 8, st,
              (const int4 *)(w + o_box), V, (int2 *)(w + o_cnt), (unsigned long long *)(w + o_tot));
    }
    TLAUNCH(k_vox_scan, dim3(1), dim3(1024), 0, st, (const int2 *)(w + o_cnt), ncell,
            (const double *)(w + o_wp), N > 0 ? nwp : 0, (int2 *)(w + o_off), (double *)(w + o_scale));
    return CS_OK;
  };
  rc = prepare();
  if (rc) return rc;
  // the list lengths are known only now: read them back (this call synchronises)
  struct {
    unsigned long long x, y;
  } total;
  HIPCHK(hipMemcpyAsync(&total, (char *)ctx->vol + o_tot, sizeof(total), hipMemcpyDeviceToHost, st));
  HIPCHK(hipStreamSynchronize(st));
  if (total.x > INT32_MAX || total.y > INT32_MAX)
    return fail(ctx, CS_ERR_UNSUPPORTED, "too many (brick, Gaussian) pairs");
  const size_t o_cells = o_list + al256v((size_t)total.y * 4 + 4);
  const size_t need = o_cells + al256v((size_t)total.x * 4 + 4);
  if (need > ctx->vol_bytes) {
    // a larger scratch does not keep its contents: prepare again (same values)
    rc = grow(ctx, &ctx->vol, &ctx->vol_bytes, need);
    if (rc) return rc;
    rc = prepare();
    if (rc) return rc;
  }
  char *w = (char *)ctx->vol;
  const float4 *rec = (const float4 *)(w + o_rec);
  const int2 *off = (const int2 *)(w + o_off);
  const double *scale = (const double *)(w + o_scale);
  int *list = (int *)(w + o_list), *cells = (int *)(w + o_cells);
  int2 *range = (int2 *)(w + o_rng);
  if (N > 0 && total.x > 0)
    TLAUNCH(k_vox_fill, dim3(cdivv(N, per)), dim3(1024), (size_t)ncell * 4, st, (const int4 *)(w + o_box), V,
            off, (int *)(w + o_cur), cells);
  typedef void (*CellFn)(const int4 *, VoxGeom, const int2 *, const int *, int2 *, int *);
  const CellFn k_vox_cell = csh == 1 ? &cs::k_vox_cell<1> : &cs::k_vox_cell<2>;
  TLAUNCH(k_vox_cell, dim3(ncell), dim3(512), 0, st, (const int4 *)(w + o_box), V, off, (const int *)cells,
          range, list);
  // one 64-lane workgroup per 4^3 sub-cube, eight per brick (XCD-aware order)
  TLAUNCH(k_vox_eval, dim3(cdivv(nbr, 8) * 64), dim3(64), 0, st, rec, (const int *)list, (const int2 *)range, V,
          scale, vol);
  return CS_OK;
}

int cs_fsc(cs_ctx *ctx, const float *vol_a, const float *vol_b, int32_t D, float *fsc,
           void *stream) {
  if (!ctx) return CS_ERR_INVALID_ARG;
  if (!vol_a || !vol_b || !fsc) return fail(ctx, CS_ERR_INVALID_ARG, "null volume or output");
  if (!fft_length(D))
    return fail(ctx, CS_ERR_UNSUPPORTED, "D must be even with prime factors 2 and 3 (<= 512)");
  HIPCHK(hipSetDevice(ctx->device));
  hipStream_t st = (hipStream_t)stream;
  const float2 *tw = nullptr;
  int rc = get_twiddles(ctx, D, &tw);
  if (rc) return rc;
  const int Dh = D / 2 + 1, ns = D / 2 + 1;
  const size_t spec = (size_t)D * D * Dh * 8;
  const size_t o_a = 0, o_b = al256v(spec), o_scale = o_b + al256v(spec), o_sums = o_scale + 256;
  const size_t o_part = o_sums + al256v((size_t)3 * ns * 8);
  rc = grow(ctx, &ctx->vol, &ctx->vol_bytes, o_part + (size_t)2 * kEnergyBlocks * 8);
  if (rc) return rc;
  char *w = (char *)ctx->vol;
  float2 *fa = (float2 *)(w + o_a), *fb = (float2 *)(w + o_b);
  double *scale = (double *)(w + o_scale);
  unsigned long long *sums = (unsigned long long *)(w + o_sums);
  double *part = (double *)(w + o_part);
  TLAUNCH(k_fsc_energy_part, dim3(kEnergyBlocks), dim3(256), 0, st, vol_a, vol_b,
          (int64_t)D * D * D, part);
  TLAUNCH(k_fsc_energy_scale, dim3(1), dim3(kEnergyBlocks), 0, st, (const double *)part, D, scale);
  const RowsFwdFn k_fft_rows_fwd = fft_rows_fwd(D);
  const AxisFn k_fft_axis = fft_axis(D);
  const FftLaunch rx = fft_rows_launch(D, D), ry = fft_cols_launch(D, Dh, D, false);
  const FftLaunch rz = fft_cols_launch(D, (int64_t)D * Dh, 1, false);
  for (int v = 0; v < 2; ++v) {
    const float *src = v ? vol_b : vol_a;
    float2 *F = v ? fb : fa;
    TLAUNCH(k_fft_rows_fwd, rx.grid, rx.block, rx.lds, st, src, tw, F);       // x (real rows)
    TLAUNCH(k_fft_axis, ry.grid, ry.block, ry.lds, st, F, tw, Dh);            // y
    TLAUNCH(k_fft_axis, rz.grid, rz.block, rz.lds, st, F, tw, D * Dh);        // z
  }
  TLAUNCH(k_fill_u64z, dim3(cdivv(3 * ns, 256)), dim3(256), 0, st, sums, 3 * ns);
  const unsigned blocks = std::min<unsigned>(256, cdivv((int64_t)Dh * Dh * Dh, 1024));
  TLAUNCH(k_fsc_shells, dim3(blocks), dim3(1024), (size_t)3 * ns * 8 * kShellCopies, st, (const float2 *)fa,
          (const float2 *)fb, D, (const double *)scale, sums);
  TLAUNCH(k_fsc_final, dim3(cdivv(ns, 256)), dim3(256), 0, st, (const unsigned long long *)sums, ns,
          (const double *)scale, fsc);
  return CS_OK;
}

int cs_fsc_resolution(cs_ctx *ctx, const float *fsc, int32_t D, float pixel, float threshold,
                      int32_t *shell, float *resolution, void *stream) {
  if (!ctx) return CS_ERR_INVALID_ARG;
  if (!fsc || (!shell && !resolution)) return fail(ctx, CS_ERR_INVALID_ARG, "null curve or outputs");
  if (D < 2 || D % 2 != 0 || D > 512) return fail(ctx, CS_ERR_UNSUPPORTED, "D must be even, at most 512");
  if (!(pixel > 0.f)) return fail(ctx, CS_ERR_INVALID_ARG, "voxel size must be positive");
  if (!(threshold == threshold)) return fail(ctx, CS_ERR_INVALID_ARG, "threshold is NaN");
  HIPCHK(hipSetDevice(ctx->device));
  TLAUNCH(k_fsc_resolution, dim3(1), dim3(64), 0, (hipStream_t)stream, fsc, D / 2 + 1, D, pixel,
          threshold, (int *)shell, resolution);
  return CS_OK;
}

}  // extern "C"
