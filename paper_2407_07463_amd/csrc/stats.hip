// Nearest-particle statistics (section "Nearest particle statistics").
//
// For every drop i the minimum-image vectors to all other drops are formed
// exactly as in the definition (per axis: subtract L if r > L/2, add L if
// r <= -L/2; d2 = (rx^2 + ry^2) + rz^2); the nearest set is every j with d2
// equal to the minimum, with tie weight h = 1/N_i (eq. 4). Each nearest pair
// is binned in (r, theta) (eqs. 8 and 10) with integer weights 720720/N_i,
// accumulated by 64-bit integer atomics (order-independent, exact), and
// contributes h r and h r r^T to the moments M (eq. 11) and R (eq. 14).
// Per-drop moment contributions are summed in a fixed tree order, so every
// output is reproducible bit for bit.
#include <mutex>

#include "common.hpp"

namespace {

constexpr int kBlock = 256;
constexpr uint64_t kFixedOne = 720720ull;  // lcm(1..16)
constexpr int32_t kMaxSlices = 64;          // candidate slices of the nearest search

struct Box {
  double L[3];
};

// (d - L, d + L or d + 0, which is d up to the sign of a zero)
__device__ __forceinline__ double min_image(double d, double L) {
  return d + (d > 0.5 * L ? -L : (d <= -0.5 * L ? L : 0.0));
}

// The same up to its sign, which its square does not see: |d|, or L - |d| (of any
// sign for points outside the box) where that is smaller, that is beyond L / 2.
__device__ __forceinline__ double image_distance(double d, double L) { return fmin(fabs(d), L - fabs(d)); }

// Candidate slices: the j range is cut into `ns` slices of `len` indices
// (a multiple of kBlock); workgroup (ib, s) scans slice s for the kBlock
// drops of block ib and keeps, per drop, the slice's smallest d2, the first j
// attaining it and how many j attain it. The candidates' loop has no branch: it
// is a chain of dependent selects that unrolled bodies overlap. Few drops are bound
// by that chain, many by its instructions, whence the image's distance by a minimum
// (the whole call for 100, 5000 and 100000 drops: a branch per axis and comparison 66, 133 and 8800 us,
// the image by two selects 42, 91 and 10100, so 40, 79 and 6380).
__global__ __launch_bounds__(kBlock) void k_nearest_slice(const double *__restrict__ xyz, int32_t n, Box box,
                                                          int32_t len, double *__restrict__ sbest,
                                                          int32_t *__restrict__ sbj, int32_t *__restrict__ sties) {
  __shared__ double sx[kBlock], sy[kBlock], sz[kBlock];
  const int32_t i = blockIdx.x * kBlock + threadIdx.x;
  const int32_t s = blockIdx.y;
  double xi = 0, yi = 0, zi = 0;
  if (i < n) {
    xi = xyz[3 * (int64_t)i];
    yi = xyz[3 * (int64_t)i + 1];
    zi = xyz[3 * (int64_t)i + 2];
  }
  double best = INFINITY;
  int32_t bj = -1, ties = 0;
  const int32_t jbeg = s * len;
  const int32_t jend = (n - jbeg < len) ? n : jbeg + len;
  for (int32_t j0 = jbeg; j0 < jend; j0 += kBlock) {
    const int32_t jj = j0 + threadIdx.x;
    __syncthreads();
    if (jj < jend) {
      sx[threadIdx.x] = xyz[3 * (int64_t)jj];
      sy[threadIdx.x] = xyz[3 * (int64_t)jj + 1];
      sz[threadIdx.x] = xyz[3 * (int64_t)jj + 2];
    }
    __syncthreads();
    const int32_t m = (jend - j0 < kBlock) ? jend - j0 : kBlock;
    if (i < n) {
#pragma unroll 4
      for (int k = 0; k < m; ++k) {
        const int32_t j = j0 + k;
        const double rx = image_distance(sx[k] - xi, box.L[0]);
        const double ry = image_distance(sy[k] - yi, box.L[1]);
        const double rz = image_distance(sz[k] - zi, box.L[2]);
        const double d2 = (rx * rx + ry * ry) + rz * rz;
        const bool less = (d2 < best) & (j != i), equal = (d2 == best) & (j != i);
        ties = less ? 1 : ties + (equal ? 1 : 0);
        bj = less ? j : bj;
        best = less ? d2 : best;
      }
    }
  }
  if (i < n) {
    const int64_t o = (int64_t)s * n + i;
    sbest[o] = best;
    sbj[o] = bj;
    sties[o] = ties;
  }
}

// Slices combined in increasing order: the minimum over slices, the first j
// of the first slice that attains it, and the tie counts of every slice that
// attains it, which is exactly what one scan over all j in order yields.
__global__ __launch_bounds__(kBlock) void k_nearest_combine(int32_t n, int32_t ns, const double *__restrict__ sbest,
                                                            const int32_t *__restrict__ sbj,
                                                            const int32_t *__restrict__ sties,
                                                            int32_t *__restrict__ nn_index,
                                                            int32_t *__restrict__ nn_ties,
                                                            double *__restrict__ best_d2) {
  const int32_t i = blockIdx.x * kBlock + threadIdx.x;
  if (i >= n) return;
  double best = INFINITY;
  int32_t bj = -1, ties = 0;
  for (int32_t s = 0; s < ns; ++s) {
    const int64_t o = (int64_t)s * n + i;
    const double d2 = sbest[o];
    if (d2 < best) {
      best = d2;
      bj = sbj[o];
      ties = sties[o];
    } else if (d2 == best && sties[o] > 0) {
      ties += sties[o];
    }
  }
  nn_index[i] = bj;
  nn_ties[i] = ties;
  best_d2[i] = best;
}

// The last e of lo .. hi with holds(e), where holds is true up to some e and
// false after it; lo - 1 if there is none.
template <class F>
__device__ __forceinline__ int last_of(int lo, int hi, F holds) {
  int below = lo - 1, above = hi + 1;  // true (or before the range), false (or after it)
  while (above - below > 1) {
    const int mid = (below + above) >> 1;
    if (holds(mid)) below = mid;
    else above = mid;
  }
  return below;
}

// Bin the nearest pairs of drop i and write its moment contributions
// part[12*i ..]: sum_j h r (3) and sum_j h r r^T (9), j ascending.
__global__ __launch_bounds__(kBlock) void k_pairs(const double *__restrict__ xyz, int32_t n, Box box, int vaxis,
                                                  int nr, int nth, const double *__restrict__ edges,
                                                  const int32_t *__restrict__ nn_index,
                                                  const int32_t *__restrict__ nn_ties,
                                                  const double *__restrict__ best_d2, uint64_t *__restrict__ hist,
                                                  double *__restrict__ part) {
  const int32_t i = blockIdx.x * kBlock + threadIdx.x;
  if (i >= n) return;
  const double *r2e = edges;           // nr + 1
  const double *ce = edges + nr + 1;   // nth + 1
  const double xi = xyz[3 * (int64_t)i], yi = xyz[3 * (int64_t)i + 1], zi = xyz[3 * (int64_t)i + 2];
  const double best = best_d2[i];
  const int ties = nn_ties[i];
  const double h = 1.0 / (double)ties;
  const uint64_t wfix = kFixedOne / (uint64_t)ties;
  double sm[3] = {0, 0, 0}, sr[9] = {0, 0, 0, 0, 0, 0, 0, 0, 0};
  // No j before the first nearest index attains the minimum, and the scan
  // ends once all `ties` nearest drops are found: the same j, in the same
  // order, as a scan over every j.
  int found = 0;
  const int32_t jfirst = nn_index[i] < 0 ? 0 : nn_index[i];
  for (int32_t j = jfirst; j < n && found < ties; ++j) {
    if (j == i) continue;
    double r[3];
    r[0] = min_image(xyz[3 * (int64_t)j] - xi, box.L[0]);
    r[1] = min_image(xyz[3 * (int64_t)j + 1] - yi, box.L[1]);
    r[2] = min_image(xyz[3 * (int64_t)j + 2] - zi, box.L[2]);
    const double d2 = (r[0] * r[0] + r[1] * r[1]) + r[2] * r[2];
    if (d2 != best) continue;
    ++found;
    // k: the last edge at or below d2. m: the last interior edge with
    // rv |rv| <= (c |c|) d2. The edges are strictly ordered, so both hold for the
    // edges up to theirs; for a d2 that is not finite every edge is looked at.
    int k = -1, m = 0;
    const double rv = (vaxis == 0) ? r[0] : ((vaxis == 1) ? r[1] : r[2]);
    auto polar = [&](int e) {
      const double c = ce[e];
      return rv * fabs(rv) <= (c * fabs(c)) * d2;
    };
    if (d2 < INFINITY) {
      k = last_of(0, nr, [&](int e) { return r2e[e] <= d2; });
      m = last_of(1, nth - 1, polar);
    } else {
      for (int e = 0; e <= nr; ++e)
        if (r2e[e] <= d2) k = e;
      for (int e = 1; e < nth; ++e)
        if (polar(e)) m = e;
    }
    if (k < 0 || k >= nr) atomicAdd((unsigned long long *)&hist[(int64_t)nr * nth], (unsigned long long)wfix);
    else atomicAdd((unsigned long long *)&hist[(int64_t)k * nth + m], (unsigned long long)wfix);
    for (int a = 0; a < 3; ++a) {
      sm[a] += h * r[a];
      for (int b = 0; b < 3; ++b) sr[3 * a + b] += h * (r[a] * r[b]);
    }
  }
  double *o = part + 12 * (int64_t)i;
  for (int a = 0; a < 3; ++a) o[a] = sm[a];
  for (int a = 0; a < 9; ++a) o[3 + a] = sr[a];
}

// Fixed-order reduction of the per-drop contributions (one workgroup), then
// the deviatoric part A = R - (tr R / 3) delta of the second moment.
__global__ __launch_bounds__(kBlock) void k_moments(const double *__restrict__ part, int32_t n, double *__restrict__ M,
                                                    double *__restrict__ R, double *__restrict__ A) {
  __shared__ double red[12][kBlock];
  double acc[12];
  for (int a = 0; a < 12; ++a) acc[a] = 0.0;
#pragma unroll 4
  for (int32_t i = threadIdx.x; i < n; i += kBlock)
#pragma unroll
    for (int a = 0; a < 12; ++a) acc[a] += part[12 * (int64_t)i + a];
  // the tree that adds thread t + w to thread t for w = 128, 64, .. 1: its first
  // two levels by the wavefront that owns the value, the others inside it
#pragma unroll
  for (int a = 0; a < 12; ++a) red[a][threadIdx.x] = acc[a];
  __syncthreads();
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  static_assert(kBlock == 256, "two levels across four wavefronts");
  for (int a = wv; a < 12; a += kBlock / 64) {
    double v = (red[a][lane] + red[a][lane + 128]) + (red[a][lane + 64] + red[a][lane + 192]);
    for (int w = 32; w > 0; w >>= 1) v += __shfl_down(v, w, 64);
    if (lane == 0) red[a][0] = v;  // (read by this wavefront alone before)
  }
  __syncthreads();
  if (threadIdx.x < 3) M[threadIdx.x] = red[threadIdx.x][0] / (double)n;
  if (threadIdx.x < 9) R[threadIdx.x] = red[3 + threadIdx.x][0] / (double)n;
  if (A != nullptr && threadIdx.x < 9) {
    const double r0 = red[3][0] / (double)n, r4 = red[7][0] / (double)n, r8 = red[11][0] / (double)n;
    const double tr = (r0 + r4) + r8;
    const double rv = red[3 + threadIdx.x][0] / (double)n;
    A[threadIdx.x] = (threadIdx.x % 4 == 0) ? rv - tr / 3.0 : rv;
  }
}

// Densities of the nearest-pair vector at the bin centres from an
// accumulated histogram (eqs. 8 and 10): P(r, theta) = E_km / (E 2 pi r^2
// sin(theta) dr dtheta) and P_r(r) = sum_m E_km / (E 4 pi r^2 dr), E the
// events in units of 1/720720. One thread per bin, then one per radial bin for
// its row sum; edges[0..nr] are the radii, edges[nr+1..] the polar angles.
__global__ __launch_bounds__(kBlock) void k_pair_pdfs(int32_t nr, int32_t nth, const double *__restrict__ edges,
                                                      const uint64_t *__restrict__ hist, int64_t events,
                                                      double *__restrict__ P, double *__restrict__ Pr) {
  const int64_t q = (int64_t)blockIdx.x * kBlock + threadIdx.x, bins = (int64_t)nr * nth;
  if (q >= bins + nr) return;
  const double pi = 3.14159265358979323846;
  const double *re = edges, *te = edges + nr + 1;
  const double E = (double)events * 720720.0;
  const int32_t k = (int32_t)(q < bins ? q / nth : q - bins);
  const double rc = 0.5 * (re[k] + re[k + 1]);
  const double dr = re[k + 1] - re[k];
  if (q < bins) {
    const int32_t m = (int32_t)(q - (int64_t)k * nth);
    const double tc = 0.5 * (te[m] + te[m + 1]);
    const double dth = te[m + 1] - te[m];
    P[q] = (double)hist[q] / (E * (2.0 * pi * (rc * rc) * sin(tc) * dr * dth));
    return;
  }
  uint64_t row = 0;
#pragma unroll 8
  for (int32_t m = 0; m < nth; ++m) row += hist[(int64_t)k * nth + m];
  Pr[k] = (double)row / (E * (4.0 * pi * (rc * rc) * dr));
}

// Bin edges as a kernel argument: no staging buffer and no copy.
constexpr int32_t kMaxEdgeArgs = 384;
struct EdgeTable {
  double e[kMaxEdgeArgs];
};
static_assert(sizeof(EdgeTable) <= 3072, "kernel argument size");

// The first launch of a call: the histogram cleared (n entries) and the edges
// (ne of them, 0 where they were copied) stored.
__global__ __launch_bounds__(kBlock) void k_begin(EdgeTable t, int32_t ne, double *__restrict__ edges,
                                                  uint64_t *__restrict__ hist, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (i < n) hist[i] = 0;
  if (i < ne) edges[i] = t.e[i];
}

}  // namespace

// Argument checks shared by both entry points (host data only).
static int check_stats_args(vofmt_ctx *ctx, const char *fn, int32_t n, const double *xyz, const double *box,
                            int32_t vertical_axis, int32_t nr, int32_t ntheta, const double *r2_edges,
                            const double *cos_edges, int32_t *nn_index, int32_t *nn_ties, uint64_t *hist_fixed,
                            double *M, double *R) {
  if (n < 2 || vertical_axis < 0 || vertical_axis > 2 || nr < 1 || ntheta < 1)
    return set_err(ctx, VOFMT_E_ARG, "%s: bad sizes (n=%d nr=%d ntheta=%d axis=%d)", fn, n, nr, ntheta,
                   vertical_axis);
  if (!xyz || !box || !r2_edges || !cos_edges || !nn_index || !nn_ties || !hist_fixed || !M || !R)
    return set_err(ctx, VOFMT_E_ARG, "%s: null pointer", fn);
  for (int a = 0; a < 3; ++a)
    if (!(box[a] > 0.0)) return set_err(ctx, VOFMT_E_ARG, "%s: box must be positive", fn);
  for (int e = 0; e < nr; ++e)
    if (!(r2_edges[e] < r2_edges[e + 1])) return set_err(ctx, VOFMT_E_ARG, "%s: r2_edges must increase", fn);
  for (int e = 0; e < ntheta; ++e)
    if (!(cos_edges[e] > cos_edges[e + 1])) return set_err(ctx, VOFMT_E_ARG, "%s: cos_edges must decrease", fn);
  return VOFMT_OK;
}

// Candidate slices of the nearest search: at most kMaxSlices slices, each a
// whole number of kBlock indices.
struct SliceShape {
  int32_t nblk, len, ns;
};
static SliceShape slice_shape(int32_t n) {
  SliceShape sh;
  sh.nblk = (int32_t)ceil_div(n, kBlock);
  const int32_t per = (int32_t)ceil_div(sh.nblk, kMaxSlices);
  sh.len = per * kBlock;
  sh.ns = (int32_t)ceil_div(n, sh.len);
  return sh;
}

// Edges first [0 .. n0] and second [0 .. n1] on the device: as a kernel argument
// where they fit (ne > 0; k_begin stores them), else copied through the pinned
// staging buffer `stage` (which must stay as it is until the stream has run).
struct Edges {
  EdgeTable t;
  int32_t ne;
};
static hipError_t put_edges(Edges &ed, const double *first, int32_t n0, const double *second, int32_t n1,
                            double *stage, double *dedge, hipStream_t stream) {
  const int64_t all = (int64_t)n0 + n1 + 2;
  ed.ne = all <= kMaxEdgeArgs ? (int32_t)all : 0;
  double *to = ed.ne > 0 ? ed.t.e : stage;
  for (int e = 0; e <= n0; ++e) to[e] = first[e];
  for (int e = 0; e <= n1; ++e) to[n0 + 1 + e] = second[e];
  if (ed.ne > 0) {
    for (int e = ed.ne; e < kMaxEdgeArgs; ++e) ed.t.e[e] = 0.0;
    return hipSuccess;
  }
  return hipMemcpyAsync(dedge, stage, sizeof(double) * (size_t)all, hipMemcpyHostToDevice, stream);
}

// The kernels of one call, on device buffers: dedge (where the edges are or go),
// best [n], part [12 n], sl (ns * n * 16 bytes).
static void launch_stats(const Edges &ed, int32_t n, const double *xyz, const double *box, int32_t vertical_axis, int32_t nr,
                         int32_t ntheta, double *dedge, double *best, double *part, char *sl,
                         int32_t *nn_index, int32_t *nn_ties, uint64_t *hist_fixed, double *M, double *R, double *A,
                         hipStream_t stream) {
  const SliceShape sh = slice_shape(n);
  double *sbest = (double *)sl;
  int32_t *sbj = (int32_t *)(sbest + (size_t)sh.ns * n);
  int32_t *sties = sbj + (size_t)sh.ns * n;
  Box b;
  for (int a = 0; a < 3; ++a) b.L[a] = box[a];
  const int64_t nh = (int64_t)nr * ntheta + 1;
  hipLaunchKernelGGL(k_begin, dim3(ceil_div(nh > ed.ne ? nh : ed.ne, kBlock)), dim3(kBlock), 0, stream, ed.t, ed.ne,
                     dedge, hist_fixed, nh);
  hipLaunchKernelGGL(k_nearest_slice, dim3(sh.nblk, sh.ns), dim3(kBlock), 0, stream, xyz, n, b, sh.len, sbest, sbj,
                     sties);
  hipLaunchKernelGGL(k_nearest_combine, dim3(sh.nblk), dim3(kBlock), 0, stream, n, sh.ns, sbest, sbj, sties,
                     nn_index, nn_ties, best);
  hipLaunchKernelGGL(k_pairs, dim3(ceil_div(n, kBlock)), dim3(kBlock), 0, stream, xyz, n, b, vertical_axis, nr,
                     ntheta, dedge, nn_index, nn_ties, best, hist_fixed, part);
  hipLaunchKernelGGL(k_moments, dim3(1), dim3(kBlock), 0, stream, part, n, M, R, A);
}

extern "C" int vofmt_nearest_pair_stats(vofmt_ctx *ctx, int32_t n, const double *xyz, const double *box,
                                        int32_t vertical_axis, int32_t nr, int32_t ntheta, const double *r2_edges,
                                        const double *cos_edges, int32_t *nn_index, int32_t *nn_ties,
                                        uint64_t *hist_fixed, double *M, double *R, double *A,
                                        hipStream_t stream) {
  if (!ctx) return VOFMT_E_ARG;
  int rc = check_stats_args(ctx, "vofmt_nearest_pair_stats", n, xyz, box, vertical_axis, nr, ntheta, r2_edges,
                            cos_edges, nn_index, nn_ties, hist_fixed, M, R);
  if (rc) return rc;
  VOFMT_HIP(ctx, hipSetDevice(ctx->device));
  const size_t nedge = (size_t)nr + 1 + (size_t)ntheta + 1;
  const SliceShape sh = slice_shape(n);
  double *dedge = (double *)scratch(ctx, SLOT_MISC, sizeof(double) * nedge);
  double *best = (double *)scratch(ctx, SLOT_MISC2, sizeof(double) * (size_t)n);
  double *part = (double *)scratch(ctx, SLOT_MISC3, sizeof(double) * 12 * (size_t)n);
  char *sl = (char *)scratch(ctx, SLOT_LABEL_A, (sizeof(double) + 2 * sizeof(int32_t)) * (size_t)sh.ns * n);
  double *hstage = (double *)host_scratch(ctx, sizeof(double) * nedge);
  if (!dedge || !best || !part || !sl || !hstage) return VOFMT_E_NOMEM;
  Edges ed;
  VOFMT_HIP(ctx, put_edges(ed, r2_edges, nr, cos_edges, ntheta, hstage, dedge, stream));
  launch_stats(ed, n, xyz, box, vertical_axis, nr, ntheta, dedge, best, part, sl, nn_index, nn_ties, hist_fixed, M, R,
               A, stream);
  VOFMT_HIP(ctx, hipGetLastError());
  VOFMT_HIP(ctx, hipStreamSynchronize(stream));
  return VOFMT_OK;
}

// ---------------------------------------------------------------- no-allocation variant
//
// vofmt_nearest_pair_stats_noalloc runs the same kernels on a fixed device
// array of this file instead of context scratch, and takes the bin edges as a
// kernel argument instead of through pinned host staging, so it allocates
// nothing and does not synchronise. Limits: n <= kNoAllocMaxDrops,
// nr + ntheta + 2 <= kNoAllocMaxEdges. Every call on a device shares the
// device's copy of the array: calls that overlap on one device race.
constexpr int32_t kNoAllocMaxDrops = 8192;
constexpr int32_t kNoAllocMaxEdges = kMaxEdgeArgs;
constexpr size_t kNoAllocOffBest = 256 * ((sizeof(double) * kNoAllocMaxEdges + 255) / 256);
constexpr size_t kNoAllocOffPart = kNoAllocOffBest + sizeof(double) * kNoAllocMaxDrops;
constexpr size_t kNoAllocOffSlices = kNoAllocOffPart + 12 * sizeof(double) * kNoAllocMaxDrops;
// slices of the largest call: at most ceil(8192 / kBlock) = 32 of one kBlock each
constexpr size_t kNoAllocSliceBytes = (sizeof(double) + 2 * sizeof(int32_t)) * 32 * (size_t)kNoAllocMaxDrops;
constexpr size_t kNoAllocBytes = kNoAllocOffSlices + kNoAllocSliceBytes;  // 4.8 MiB
static_assert(kNoAllocOffPart % 256 == 0 && kNoAllocOffSlices % 256 == 0, "aligned parts");
static_assert(kNoAllocMaxDrops / kBlock <= kMaxSlices, "one slice per block at the largest size");

static __device__ __align__(256) unsigned char noalloc_scratch[kNoAllocBytes];

constexpr int kNoAllocMaxDevices = 64;
static void *g_noalloc_ptr[kNoAllocMaxDevices] = {};
static std::mutex g_noalloc_mu;

// Device address of this device's copy of noalloc_scratch, looked up once per
// device with that device current (called by vofmt_create). The host-side
// name of the array is not a device address and is never passed to a kernel.
hipError_t noalloc_setup(int device) {
  if (device < 0 || device >= kNoAllocMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_noalloc_mu);
  if (g_noalloc_ptr[device]) return hipSuccess;
  void *p = nullptr;
  const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(noalloc_scratch));
  if (e != hipSuccess) return e;
  g_noalloc_ptr[device] = p;
  return hipSuccess;
}

extern "C" int vofmt_nearest_pair_stats_noalloc(vofmt_ctx *ctx, int32_t n, const double *xyz, const double *box,
                                                int32_t vertical_axis, int32_t nr, int32_t ntheta,
                                                const double *r2_edges, const double *cos_edges, int32_t *nn_index,
                                                int32_t *nn_ties, uint64_t *hist_fixed, double *M, double *R,
                                                double *A, hipStream_t stream) {
  if (!ctx) return VOFMT_E_ARG;
  const char *fn = "vofmt_nearest_pair_stats_noalloc";
  int rc = check_stats_args(ctx, fn, n, xyz, box, vertical_axis, nr, ntheta, r2_edges, cos_edges, nn_index, nn_ties,
                            hist_fixed, M, R);
  if (rc) return rc;
  if (n > kNoAllocMaxDrops)
    return set_err(ctx, VOFMT_E_ARG, "%s: n=%d drops exceeds the fixed scratch limit of %d", fn, n,
                   kNoAllocMaxDrops);
  if ((int64_t)nr + ntheta + 2 > kNoAllocMaxEdges)
    return set_err(ctx, VOFMT_E_ARG, "%s: nr + ntheta + 2 = %lld edges exceeds the limit of %d", fn,
                   (long long)nr + ntheta + 2, kNoAllocMaxEdges);
  const SliceShape sh = slice_shape(n);
  if ((size_t)sh.ns * n * (sizeof(double) + 2 * sizeof(int32_t)) > kNoAllocSliceBytes)
    return set_err(ctx, VOFMT_E_ARG, "%s: slice table exceeds the fixed scratch", fn);
  if (ctx->device < 0 || ctx->device >= kNoAllocMaxDevices || !g_noalloc_ptr[ctx->device])
    return set_err(ctx, VOFMT_E_HIP, "%s: the fixed scratch of device %d has no address", fn, ctx->device);
  VOFMT_HIP(ctx, hipSetDevice(ctx->device));
  char *base = (char *)g_noalloc_ptr[ctx->device];
  double *dedge = (double *)base;
  double *best = (double *)(base + kNoAllocOffBest);
  double *part = (double *)(base + kNoAllocOffPart);
  char *sl = base + kNoAllocOffSlices;
  Edges ed;
  VOFMT_HIP(ctx, put_edges(ed, r2_edges, nr, cos_edges, ntheta, nullptr, dedge, stream));
  launch_stats(ed, n, xyz, box, vertical_axis, nr, ntheta, dedge, best, part, sl, nn_index, nn_ties, hist_fixed, M, R,
               A, stream);
  VOFMT_HIP(ctx, hipGetLastError());
  return VOFMT_OK;
}

extern "C" int vofmt_pair_pdfs(vofmt_ctx *ctx, int32_t nr, int32_t ntheta, const double *r_edges,
                               const double *theta_edges, const uint64_t *hist_fixed, int64_t events, double *P,
                               double *Pr, hipStream_t stream) {
  if (!ctx) return VOFMT_E_ARG;
  if (nr < 1 || ntheta < 1 || events < 1)
    return set_err(ctx, VOFMT_E_ARG, "vofmt_pair_pdfs: bad sizes (nr=%d ntheta=%d events=%lld)", nr, ntheta,
                   (long long)events);
  if (!r_edges || !theta_edges || !hist_fixed || !P || !Pr)
    return set_err(ctx, VOFMT_E_ARG, "vofmt_pair_pdfs: null pointer");
  if (!(r_edges[0] >= 0.0) || !(theta_edges[0] >= 0.0) || !(theta_edges[ntheta] <= 3.14159265358979323846))
    return set_err(ctx, VOFMT_E_ARG, "vofmt_pair_pdfs: edges outside r >= 0, 0 <= theta <= pi");
  for (int e = 0; e < nr; ++e)
    if (!(r_edges[e] < r_edges[e + 1])) return set_err(ctx, VOFMT_E_ARG, "vofmt_pair_pdfs: r_edges must increase");
  for (int e = 0; e < ntheta; ++e)
    if (!(theta_edges[e] < theta_edges[e + 1]))
      return set_err(ctx, VOFMT_E_ARG, "vofmt_pair_pdfs: theta_edges must increase");
  VOFMT_HIP(ctx, hipSetDevice(ctx->device));
  const size_t nedge = (size_t)nr + 1 + (size_t)ntheta + 1;
  double *dedge = (double *)scratch(ctx, SLOT_MISC, sizeof(double) * nedge);
  double *hstage = (double *)host_scratch(ctx, sizeof(double) * nedge);
  if (!dedge || !hstage) return VOFMT_E_NOMEM;
  Edges ed;
  VOFMT_HIP(ctx, put_edges(ed, r_edges, nr, theta_edges, ntheta, hstage, dedge, stream));
  if (ed.ne > 0)
    hipLaunchKernelGGL(k_begin, dim3(ceil_div(ed.ne, kBlock)), dim3(kBlock), 0, stream, ed.t, ed.ne, dedge,
                       (uint64_t *)nullptr, (int64_t)0);
  hipLaunchKernelGGL(k_pair_pdfs, dim3(ceil_div((int64_t)nr * ntheta + nr, kBlock)), dim3(kBlock), 0, stream, nr, ntheta, dedge, hist_fixed,
                     events, P, Pr);
  VOFMT_HIP(ctx, hipGetLastError());
  VOFMT_HIP(ctx, hipStreamSynchronize(stream));
  return VOFMT_OK;
}
