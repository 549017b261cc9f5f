// Plain advection entry points: one box, one launch per pass.
// The kernels are thin wrappers around the shared sweep bodies: every sweep
// is a PLIC pass over the mixed cells and one streaming pass over all tracers.
#include "advect_kernels.hpp"

using namespace advect;

namespace {

constexpr int kXWaves = 8;  // wavefronts per workgroup of the x-sweep: a 512-cell row per workgroup

__global__ __launch_bounds__(256) void k_scan_mixed(const double *__restrict__ c, int64_t total,
                                                    uint32_t *__restrict__ list, int *__restrict__ counts,
                                                    int64_t nregions, int rsize) {
  scan_body(c, total, list, counts, nregions, rsize, ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6);
}

template <int D>
__global__ __launch_bounds__(256) void k_plic(const double *__restrict__ cin, const double *__restrict__ s,
                                              const uint32_t *__restrict__ list, const int *__restrict__ counts,
                                              int64_t nregions, int rsize, double *__restrict__ fmix, int nx, int ny,
                                              int nz, Divisors dv) {
  plic_body<D>(cin, s, list, counts, nregions, rsize, fmix, nx, ny, nz, dv, (int64_t)blockIdx.x * kPlicRegions);
}

// One streaming pass over every tracer: ngrp groups of GM or GM - 1, group k
// filling list regions k * gstride onwards. D = 0 with rows above a list
// region's cells: kXWaves wavefronts per workgroup share segment ends.
template <int D, int GM>
__global__ __launch_bounds__(D == 0 ? 64 * kXWaves : 256) void k_stream(
    const double *__restrict__ cin, double *__restrict__ cout, const double *__restrict__ s,
    const double *__restrict__ fmix, uint64_t *__restrict__ ccbits, int cc, int ntr, int nx, int ny, int nz,
    int words, int chunk, uint32_t *__restrict__ list_next, int *__restrict__ counts_next, int rsize, int ngrp,
    int64_t gstride, FastDiv fnx) {
  const GroupTile g = group_tile(((int)blockIdx.z * gridDim.y + blockIdx.y) * gridDim.x + blockIdx.x, gridDim.x,
                                 gridDim.y, gridDim.z / ngrp, ngrp, D == 1);
  stream_group<D, GM, kXWaves>(cin, cout, s, fmix, ccbits, cc, ntr, nx, ny, nz, words, chunk, list_next,
                           counts_next, g.grp * gstride, rsize, g, gridDim.x, gridDim.y, fnx);
}

// The sweeps in the flat layout.
template <int D, int GM>
__global__ __launch_bounds__(256) void k_stream_flat(const double *__restrict__ cin, double *__restrict__ cout,
                                                     const double *__restrict__ s, const double *__restrict__ fmix,
                                                     uint64_t *__restrict__ ccbits, int cc, int ntr, int nx, int ny,
                                                     int nz, int words, int chunk, uint32_t *__restrict__ list_next,
                                                     int *__restrict__ counts_next, int rsize, int ngrp,
                                                     int64_t gstride, FastDiv fnx) {
  const GroupTile g = group_tile(((int)blockIdx.z * gridDim.y + blockIdx.y) * gridDim.x + blockIdx.x, gridDim.x,
                                 gridDim.y, gridDim.z / ngrp, ngrp, D == 1);
  stream_group<D, GM, kFlat>(cin, cout, s, fmix, ccbits, cc, ntr, nx, ny, nz, words, chunk, list_next, counts_next,
                             g.grp * gstride, rsize, g, gridDim.x, gridDim.y, fnx);
}

// The x-sweep marching along whole rows (4 wavefronts per workgroup).
template <int GM>
__global__ __launch_bounds__(256) void k_stream_rows(const double *__restrict__ cin, double *__restrict__ cout,
                                                     const double *__restrict__ s, const double *__restrict__ fmix,
                                                     uint64_t *__restrict__ ccbits, int cc, int ntr, int nx,
                                                     int ny, int nz, int words, int chunk,
                                                     uint32_t *__restrict__ list_next, int *__restrict__ counts_next,
                                                     int rsize, int ngrp, int64_t gstride, FastDiv fnx) {
  const GroupTile g = group_tile(((int)blockIdx.z * gridDim.y + blockIdx.y) * gridDim.x + blockIdx.x, gridDim.x,
                                 gridDim.y, gridDim.z / ngrp, ngrp, false);
  stream_group<0, GM, 0>(cin, cout, s, fmix, ccbits, cc, ntr, nx, ny, nz, words, chunk, list_next, counts_next,
                     g.grp * gstride, rsize, g, gridDim.x, gridDim.y, fnx);
}

// Per-block maximum of |s| over the three arrays and a non-finite flag.
__global__ __launch_bounds__(256) void k_courant_max(const double *__restrict__ sx, const double *__restrict__ sy,
                                                     const double *__restrict__ sz, int64_t n, double *__restrict__ out) {
  __shared__ double red[256];
  double m = 0.0;
  for (int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; q < n; q += (int64_t)gridDim.x * blockDim.x) {
    double a = fabs(sx[q]), b = fabs(sy[q]), c = fabs(sz[q]);
    if (!(a <= 1e300) || !(b <= 1e300) || !(c <= 1e300)) m = INFINITY;  // NaN or inf
    else m = fmax(m, fmax(a, fmax(b, c)));
  }
  red[threadIdx.x] = m;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) red[threadIdx.x] = fmax(red[threadIdx.x], red[threadIdx.x + w]);
    __syncthreads();
  }
  if (threadIdx.x == 0) out[blockIdx.x] = red[0];
}

}  // namespace

struct SweepBuffers {
  double *fmix;
  uint64_t *bits;
  uint32_t *list[2];
  int *counts[2];
  int64_t nregions[2];  // regions filled into each list
  int stride[2];        // entries per region of each list
  int rsize;            // entries per region a streaming pass fills
};

// Workgroup layout of the x-sweep: whole-row wavefronts (0) when a row has at
// most `chunk` segments (so a wavefront's cells fit its list region), else
// kXWaves wavefronts sharing segment ends through LDS.
static inline int x_wpb(int words, int chunk) { return words <= chunk ? 0 : kXWaves; }

// Marching chunk of the streaming passes: the longest that still gives every
// sweep kWaves wavefronts (a long chunk re-reads fewer rows at its ends; a
// wavefront's march is a serial chain of dependent positions, so a grid of
// few wavefronts takes the chain's time however little it has to do). Never
// below a row's segments, so that the x-sweep keeps whole-row wavefronts where
// it has them at the longest chunk. One step, chunk 32 everywhere against this
// rule (the scan below included): 64^3 x 2 184.7 -> 60 us (chunk 4),
// 134x129x141 x 7 716 -> 546 us, 200x180x210 x 4 747 -> 700 us; kWaves 4096
// leaves the second at 667, 16384 and 32768 are within 2% of 8192 on all.
static int pick_chunk(int nx, int ny, int nz, int ntr) {
  const int words = (nx + 63) / 64;
  const bool flat = flat_rows(nx, ny, nz);
  int chunk = kMaxChunk;
  while (chunk > 4 && (flat || words <= chunk / 2)) {
    int64_t least = INT64_MAX;
    for (int d = 0; d < 3; ++d) {
      const int64_t w = stream_waves(d, nx, ny, nz, chunk, d == 0 ? x_wpb(words, chunk) : 4, flat) *
                        num_groups(ntr);
      least = w < least ? w : least;
    }
    if (least >= kWaves) break;
    chunk /= 2;
  }
  return chunk;
}
// Tracer-cells per wavefront of the initial scan, by the same rule.
static int scan_span(int64_t total) {
  int span = region_size(kMaxChunk);
  while (span > 64 * kScanBatch && total / span < kWaves) span /= 2;
  return span;
}

template <int D, int GM>
static void launch_stream(dim3 grid, bool flat, const FastDiv &fnx, hipStream_t stream, const double *cin, double *cout,
                          const double *s, SweepBuffers &sb, int cc, int nx, int ny, int nz, int ntr, int words,
                          int chunk, int nxt, int64_t per) {
  const int ngrp = num_groups(ntr);
  if (flat)
    hipLaunchKernelGGL((k_stream_flat<D, GM>), grid, dim3(256), 0, stream, cin, cout, s, sb.fmix, sb.bits, cc, ntr, nx,
                       ny, nz, words, chunk, sb.list[nxt], sb.counts[nxt], sb.rsize, ngrp, per, fnx);
  else if (D == 0 && x_wpb(words, chunk) == 0)
    hipLaunchKernelGGL((k_stream_rows<GM>), grid, dim3(256), 0, stream, cin, cout, s, sb.fmix, sb.bits, cc, ntr, nx,
                       ny, nz, words, chunk, sb.list[nxt], sb.counts[nxt], sb.rsize, ngrp, per, fnx);
  else
    hipLaunchKernelGGL((k_stream<D, GM>), grid, dim3(D == 0 ? 64 * kXWaves : 256), 0, stream, cin, cout, s, sb.fmix,
                       sb.bits, cc, ntr, nx, ny, nz, words, chunk, sb.list[nxt], sb.counts[nxt], sb.rsize, ngrp,
                       per, fnx);
}

template <int D>
static void launch_sweep_axis(vofmt_ctx *ctx, const double *cin, double *cout, const double *s, SweepBuffers &sb,
                              int cc, int cur, int nx, int ny, int nz, int ntr, int words, int chunk,
                              hipStream_t stream) {
  const int nxt = cur ^ 1;
  const int64_t nreg = sb.nregions[cur];
  Divisors dv;
  dv.n3 = make_fastdiv((uint32_t)((int64_t)nx * ny * nz));
  dv.nx = make_fastdiv((uint32_t)nx);
  dv.ny = make_fastdiv((uint32_t)ny);
  static const char *plic_names[3] = {"k_plic<0>", "k_plic<1>", "k_plic<2>"};
  static const char *stream_names[3] = {"k_stream<0>", "k_stream<1>", "k_stream<2>"};
  int rec = prof_begin(ctx, plic_names[D], stream);
  hipLaunchKernelGGL((k_plic<D>), dim3(ceil_div(nreg, kPlicRegions)), dim3(64 * kPlicRegions), 0, stream, cin, s,
                     sb.list[cur], sb.counts[cur], nreg, sb.stride[cur], sb.fmix, nx, ny, nz, dv);
  prof_end(ctx, rec, stream);
  const int wpb = (D == 0) ? x_wpb(words, chunk) : 4;
  const bool flat = flat_rows(nx, ny, nz);
  const int64_t per = stream_waves(D, nx, ny, nz, chunk, wpb, flat);
  const Tiles tg = stream_tiles(D, nx, ny, nz, chunk, wpb, flat);
  const dim3 grid(tg.gx, tg.gy, tg.gz * num_groups(ntr));
  static_assert(kMaxGroup == 4, "streaming passes are instantiated for groups of at most 4");
  rec = prof_begin(ctx, stream_names[D], stream);
  auto launch = [&](auto GM) {
    launch_stream<D, decltype(GM)::value>(grid, flat, dv.nx, stream, cin, cout, s, sb, cc, nx, ny, nz, ntr, words,
                                          chunk, nxt, per);
  };
  switch (largest_group(ntr)) {
    case 4: launch(std::integral_constant<int, 4>{}); break;
    case 3: launch(std::integral_constant<int, 3>{}); break;
    case 2: launch(std::integral_constant<int, 2>{}); break;
    default: launch(std::integral_constant<int, 1>{}); break;
  }
  prof_end(ctx, rec, stream);
  sb.nregions[nxt] = num_groups(ntr) * per;
  sb.stride[nxt] = sb.rsize;
}

static int launch_sweep(vofmt_ctx *ctx, int d, const double *cin, double *cout, const double *s, SweepBuffers &sb,
                        int cc, int cur, int nx, int ny, int nz, int ntr, int words, int chunk, hipStream_t stream) {
  if (d == 0) launch_sweep_axis<0>(ctx, cin, cout, s, sb, cc, cur, nx, ny, nz, ntr, words, chunk, stream);
  else if (d == 1) launch_sweep_axis<1>(ctx, cin, cout, s, sb, cc, cur, nx, ny, nz, ntr, words, chunk, stream);
  else launch_sweep_axis<2>(ctx, cin, cout, s, sb, cc, cur, nx, ny, nz, ntr, words, chunk, stream);
  return (int)hipGetLastError();
}

extern "C" int vofmt_advect(vofmt_ctx *ctx, int32_t nx, int32_t ny, int32_t nz, int32_t ntracers, double *c,
                            const double *sx, const double *sy, const double *sz, int64_t step0, int32_t nsteps,
                            hipStream_t stream) {
  if (!ctx) return VOFMT_E_ARG;
  if (nx < 1 || ny < 1 || nz < 1 || ntracers < 0 || nsteps < 0 || step0 < 0)
    return set_err(ctx, VOFMT_E_ARG, "vofmt_advect: bad sizes (nx=%d ny=%d nz=%d ntracers=%d nsteps=%d step0=%lld)",
                   nx, ny, nz, ntracers, nsteps, (long long)step0);
  if (ntracers == 0 || nsteps == 0) return VOFMT_OK;
  if (!c || !sx || !sy || !sz) return set_err(ctx, VOFMT_E_ARG, "vofmt_advect: null pointer");
  if (ny > 65535 || ceil_div(nz, 4) > 65535 || ceil_div(ny, kMaxChunk) > 65535 || ceil_div(nz, kMaxChunk) > 65535)
    return set_err(ctx, VOFMT_E_ARG, "vofmt_advect: grid too large");
  VOFMT_HIP(ctx, hipSetDevice(ctx->device));
  const int64_t n3 = (int64_t)nx * ny * nz;
  if ((int64_t)ntracers * n3 >= ((int64_t)1 << 32))
    return set_err(ctx, VOFMT_E_ARG, "vofmt_advect: ntracers * cells must stay below 2^32");
  const double *s3[3] = {sx, sy, sz};
  const int words = (int)ceil_div(nx, 64);
  const size_t field_bytes = sizeof(double) * (size_t)n3 * ntracers;
  double *tmp = (double *)scratch(ctx, SLOT_PINGPONG, field_bytes);
  double *fmix = (double *)scratch(ctx, SLOT_FMIX, field_bytes);
  uint64_t *bits = (uint64_t *)scratch(ctx, SLOT_CCBITS, sizeof(uint64_t) * (size_t)ntracers * nz * ny * words);
  // list regions: enough for the largest sweep launch set and for the initial scan
  const int chunk = pick_chunk(nx, ny, nz, ntracers);
  const int rsize = region_size(chunk);
  const int64_t total = (int64_t)ntracers * n3;
  const int span = scan_span(total);
  const int64_t scanreg = (total + span - 1) / span;
  int64_t maxreg = max_regions(nx, ny, nz, ntracers, chunk, x_wpb(words, chunk), flat_rows(nx, ny, nz));
  if (maxreg * rsize < scanreg * span) maxreg = (scanreg * span + rsize - 1) / rsize;
  const int64_t maxcnt = maxreg > scanreg ? maxreg : scanreg;
  uint32_t *lists = (uint32_t *)scratch(ctx, SLOT_MIXLIST, sizeof(uint32_t) * 2 * (size_t)maxreg * rsize);
  int *counts = (int *)scratch(ctx, SLOT_COUNTS, sizeof(int) * 2 * (size_t)maxcnt);
  if (!tmp || !fmix || !bits || !lists || !counts) return VOFMT_E_NOMEM;
  SweepBuffers sb;
  sb.fmix = fmix;
  sb.bits = bits;
  sb.list[0] = lists;
  sb.list[1] = lists + (size_t)maxreg * rsize;
  sb.counts[0] = counts;
  sb.counts[1] = counts + maxcnt;
  sb.nregions[0] = scanreg;
  sb.nregions[1] = 0;
  sb.stride[0] = span;
  sb.stride[1] = rsize;
  sb.rsize = rsize;
  // mixed cells of the input field
  const int rec = prof_begin(ctx, "k_scan_mixed", stream);
  hipLaunchKernelGGL(k_scan_mixed, dim3(ceil_div(scanreg, 4)), dim3(256), 0, stream, c, total, sb.list[0],
                     sb.counts[0], scanreg, span);
  prof_end(ctx, rec, stream);
  VOFMT_HIP(ctx, hipGetLastError());
  int cur_list = 0;
  // The last sweep has to write c. With an odd number of sweeps the first
  // three go c -> tmp -> third -> c, the others c -> tmp -> c; without memory
  // for the third copy the result is copied back instead (one step of
  // 134x129x141 x 7: 497 -> 445 us without that copy).
  double *third =
      nsteps % 2 == 1 ? (double *)third_copy(ctx, field_bytes, stream) : nullptr;
  double *cur = c, *nxt = tmp;
  for (int32_t st = 0; st < nsteps; ++st) {
    const int64_t g = step0 + st;
    for (int r = 0; r < 3; ++r) {
      const int d = (int)((g + r) % 3);
      int rc = launch_sweep(ctx, d, cur, nxt, s3[d], sb, cc_mode(g, r), cur_list, nx, ny, nz, ntracers, words, chunk,
                            stream);
      if (rc) return hip_check(ctx, (hipError_t)rc, "sweep launch");
      cur_list ^= 1;
      double *t = cur;
      cur = nxt;
      nxt = t;
      if (third && st == 0) nxt = r == 0 ? third : (r == 1 ? c : tmp);
    }
  }
  if (cur != c)
    VOFMT_HIP(ctx, hipMemcpyAsync(c, cur, sizeof(double) * (size_t)n3 * ntracers, hipMemcpyDeviceToDevice, stream));
  return VOFMT_OK;
}

extern "C" int vofmt_check_courant(vofmt_ctx *ctx, int32_t nx, int32_t ny, int32_t nz, const double *sx,
                                   const double *sy, const double *sz, double *smax_host, hipStream_t stream) {
  if (!ctx) return VOFMT_E_ARG;
  if (nx < 1 || ny < 1 || nz < 1 || !sx || !sy || !sz || !smax_host)
    return set_err(ctx, VOFMT_E_ARG, "vofmt_check_courant: bad arguments");
  VOFMT_HIP(ctx, hipSetDevice(ctx->device));
  const int nblk = 1024;
  double *part = (double *)scratch(ctx, SLOT_MISC, sizeof(double) * nblk);
  double *h = (double *)host_scratch(ctx, sizeof(double) * nblk);
  if (!part || !h) return VOFMT_E_NOMEM;
  const int64_t n = (int64_t)nx * ny * nz;
  hipLaunchKernelGGL(k_courant_max, dim3(nblk), dim3(256), 0, stream, sx, sy, sz, n, part);
  VOFMT_HIP(ctx, hipGetLastError());
  VOFMT_HIP(ctx, hipMemcpyAsync(h, part, sizeof(double) * nblk, hipMemcpyDeviceToHost, stream));
  VOFMT_HIP(ctx, hipStreamSynchronize(stream));
  double m = 0.0;
  for (int b = 0; b < nblk; ++b) m = fmax(m, h[b]);
  *smax_host = m;
  if (!(m <= 1e300)) return set_err(ctx, VOFMT_E_NONFINITE, "vofmt_check_courant: non-finite face velocity");
  if (m > 0.5) return set_err(ctx, VOFMT_E_CFL, "vofmt_check_courant: max |s| = %g exceeds 0.5", m);
  return VOFMT_OK;
}
