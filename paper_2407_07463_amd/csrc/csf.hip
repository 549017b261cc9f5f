// Multi-tracer surface-tension force on the cell faces.
//
// The force is the sum over the tracers of gamma kappa_i grad C_i, each
// curvature computed as for a single tracer (section "The no-coalescence.h
// algorithm"), here in the balanced-force face-centred form (Popinet 2018,
// referred to in section "Numerical method"): on the lower d-face of cell p,
// between m = p - e_d and p,
//   F_d[p] = gamma * sum_i phi_i (C_i[p] - C_i[m]),
// phi_i the mean of kappa_i[p] and kappa_i[m] where both are defined, the
// defined one where one is, no contribution where neither is or where C_i
// does not jump. Undefined curvature is NaN. The tracers are summed in
// increasing order, then scaled by gamma.
//
// One pass streams every tracer's C and kappa once: a wavefront holds 64
// consecutive cells of a row, a workgroup eight rows, and each thread marches
// along z keeping the previous plane's C and kappa of its tracers in registers.
// The x and y neighbours come from the workgroup's own rows through LDS; the
// row below the tile and the column before it are loaded once by threads
// spread over the workgroup.
#include <cmath>

#include "common.hpp"

namespace {

constexpr int kTX = 64, kTY = 8;
constexpr int kMaxGroup = 8;  // one wavefront per tracer loads the row below the tile
constexpr int kStage = 4;     // tracers exchanged through LDS per barrier
static_assert(kMaxGroup <= kTY, "a tracer's row below the tile is loaded by the wavefront of its number");

// Branch-free (selects only), so that every load of a plane is issued before
// the first use.
__device__ __forceinline__ double face_term(double cp, double cm, double kp, double km) {
  const double d = cp - cm;
  const bool hp = kp == kp, hm = km == km;  // defined: not NaN
  const double phi = hp ? (hm ? (kp + km) * 0.5 : kp) : km;
  return (d == 0.0 || !(hp || hm)) ? 0.0 : phi * d;
}

// The double `bytes` after p, for a p that is the same in all lanes: kept in
// scalar registers, so that an access needs one vector register of address.
typedef __attribute__((address_space(1))) double gdouble;
__device__ __forceinline__ gdouble &at_uniform(const double *p, unsigned bytes) {
  const unsigned long long b = (unsigned long long)p;
  const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)b), hi = __builtin_amdgcn_readfirstlane((unsigned)(b >> 32));
  typedef __attribute__((address_space(1))) char gchar;
  return *(gdouble *)((gchar *)(((unsigned long long)hi << 32) | lo) + bytes);
}

// Lane l's value in every lane (l the same in all of them).
__device__ __forceinline__ double lane_value(double v, int l) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_readlane((int)b, l), hi = __builtin_amdgcn_readlane((int)(b >> 32), l);
  return __longlong_as_double(((long long)hi << 32) | (long long)(unsigned)lo);
}

// Tracers [t0, t0 + G): the running sums start from 0 (first group) or from
// the partial sums stored by the previous group, and the last group stores
// gamma times the sums. Every thread takes part in every barrier; threads
// without a cell load a clamped cell and store nothing.
//
// Bound by HBM as long as loads stay in flight: a tracer's next plane is loaded
// as soon as its faces of this plane are summed, into the registers of the
// plane below, and the row and column of the halo by threads spread over the
// workgroup (2 G + 3 loads a thread and plane). With every thread loading its
// neighbours itself and using them in the plane they were issued in, a
// wavefront waited out a latency per plane: 748 us at 256^3 x 8 and 5.51 ms at
// 512^3 x 8 (3.7 TB/s of the method's bytes), 531 us and 4.20 ms so (4.9 TB/s).
// kStage tracers per barrier in two alternating buffers (74 KB) leave two
// workgroups a CU; 2 tracers per barrier measured the same.
template <int G>
__global__ __launch_bounds__(kTX *kTY, 4) void k_csf(const double *__restrict__ c, const double *__restrict__ kap,
                                                     int nx, int ny, int nz, int zc, int t0, double gamma, int first,
                                                     int last, double *__restrict__ fx, double *__restrict__ fy,
                                                     double *__restrict__ fz) {
  constexpr int A = G > 0 ? G : 1;
  // [buffer][tracer of the stage][C, kappa][row below the tile, its rows][x]
  __shared__ double buf[2][A < kStage ? A : kStage][2][kTY + 1][kTX];
  // XCD-aware tile order: workgroups are dealt to the 8 XCDs in turn, so the
  // hardware id is mapped to a tile index that gives each XCD a contiguous
  // run of tiles; neighbouring tiles (whose rows are each other's halo) then
  // share an L2.
  const unsigned nwg = gridDim.x, id = blockIdx.x;
  const unsigned per = nwg / 8, rem = nwg % 8, xk8 = id % 8;
  const unsigned L = xk8 * per + (xk8 < rem ? xk8 : rem) + id / 8;
  const unsigned tx = (nx + kTX - 1) / kTX, ty = (ny + kTY - 1) / kTY;
  // (divisions run in vector registers: back to scalar ones, and everything derived from them)
  const int bx = __builtin_amdgcn_readfirstlane((int)(L % tx)), by = __builtin_amdgcn_readfirstlane((int)((L / tx) % ty)),
            bz = __builtin_amdgcn_readfirstlane((int)(L / (tx * ty)));
  const int lane = threadIdx.x & (kTX - 1), w = __builtin_amdgcn_readfirstlane(threadIdx.x / kTX);
  const int x = bx * kTX + lane;
  const int y = by * kTY + w;
  const bool act = x < nx && y < ny;
  const int xc = x < nx ? x : nx - 1, yc = y < ny ? y : ny - 1;  // clamped cell of an inactive thread
  const int z0 = bz * zc;
  const int z1 = z0 + zc < nz ? z0 + zc : nz;
  const int64_t n3 = (int64_t)nx * ny * nz, plane = (int64_t)nx * ny;
  const double *ct = c + (int64_t)t0 * n3;
  const double *kt = kap + (int64_t)t0 * n3;
  // in a plane, all but the lane's part the same over the wavefront: this row,
  // the row below the tile, the cell before the tile in this row
  const int64_t own = (int64_t)yc * nx + (int64_t)bx * kTX;
  const int64_t below = (int64_t)(by == 0 ? ny - 1 : by * kTY - 1) * nx + (int64_t)bx * kTX;
  const int64_t before = (int64_t)yc * nx + (bx == 0 ? nx - 1 : bx * kTX - 1);
  const unsigned at = (unsigned)(xc - bx * kTX) * (unsigned)sizeof(double);
  const bool edge_y = w < G, edge_x = lane < 2 * G;
  // lane 2g of the column's loads holds C of tracer g, lane 2g + 1 its kappa
  const double *col = ((lane & 1) ? kt : ct) + (edge_x ? lane >> 1 : 0) * n3 + before;
  const double *row_c = ct + (edge_y ? w : 0) * n3 + below, *row_k = kt + (edge_y ? w : 0) * n3 + below;
  // One plane's values each: a tracer's entry of the plane below takes the next
  // plane's value as soon as its faces are summed, then the two change places.
  double ca[A], ka[A], cb[A], kb[A];
  double yc_n = 0.0, yk_n = 0.0, x_n = 0.0;  // halo of the plane that comes next
  auto load = [&](int z, int g, double *cv, double *kv) {
    const int64_t q = g * n3 + z * plane + own;
    cv[g] = at_uniform(ct + q, at);
    kv[g] = at_uniform(kt + q, at);
  };
  auto load_row = [&](int z) {
    if (edge_y) {
      yc_n = at_uniform(row_c + z * plane, at);
      yk_n = at_uniform(row_k + z * plane, at);
    }
  };
  auto load_column = [&](int z) {
    if (edge_x) x_n = col[z * plane];
  };
#pragma unroll
  for (int g = 0; g < G; ++g) load(z0 == 0 ? nz - 1 : z0 - 1, g, ca, ka);
#pragma unroll
  for (int g = 0; g < G; ++g) load(z0, g, cb, kb);
  load_row(z0);
  load_column(z0);
  int b = 0;
  auto sum_plane = [&](int z, double *cp, double *kp, double *cz, double *kz) {
    double *const px = fx + (z * plane + own), *const py = fy + (z * plane + own), *const pz = fz + (z * plane + own);
    double sx = 0.0, sy = 0.0, sz = 0.0;
    if (!first && act) {
      sx = at_uniform(px, at);
      sy = at_uniform(py, at);
      sz = at_uniform(pz, at);
    }
    const double x_p = x_n;
    const int zn = z + 1 < z1 ? z + 1 : z;  // (the last plane again, unused: no branch around the loads)
    load_column(zn);
#pragma unroll
    for (int g0 = 0; g0 < G; g0 += kStage) {
#pragma unroll
      for (int g = g0; g < g0 + kStage && g < G; ++g) {
        buf[b][g - g0][0][w + 1][lane] = cp[g];
        buf[b][g - g0][1][w + 1][lane] = kp[g];
      }
      if (w >= g0 && w < g0 + kStage && w < G) {
        buf[b][w - g0][0][0][lane] = yc_n;
        buf[b][w - g0][1][0][lane] = yk_n;
        load_row(zn);
      }
      __syncthreads();
#pragma unroll
      for (int g = g0; g < g0 + kStage && g < G; ++g) {
        const auto &bc = buf[b][g - g0][0], &bk = buf[b][g - g0][1];
        const int lm = lane == 0 ? 0 : lane - 1;
        const double cl = bc[w + 1][lm], kl = bk[w + 1][lm];
        const double c0 = lane_value(x_p, 2 * g), k0 = lane_value(x_p, 2 * g + 1);
        sx += face_term(cp[g], lane == 0 ? c0 : cl, kp[g], lane == 0 ? k0 : kl);
        sy += face_term(cp[g], bc[w][lane], kp[g], bk[w][lane]);
        sz += face_term(cp[g], cz[g], kp[g], kz[g]);
        load(zn, g, cz, kz);
        // tracer by tracer, not sunk to the stores (every tracer's values would stay live until there)
        asm volatile("" : "+v"(sx), "+v"(sy), "+v"(sz));
        __builtin_amdgcn_sched_barrier(0);
      }
      // (the other buffer next: its readers are all past this barrier)
      b ^= 1;
    }
    if (last) {
      sx = gamma * sx;
      sy = gamma * sy;
      sz = gamma * sz;
    }
    if (act) {
      __builtin_nontemporal_store(sx, &at_uniform(px, at));
      __builtin_nontemporal_store(sy, &at_uniform(py, at));
      __builtin_nontemporal_store(sz, &at_uniform(pz, at));
    }
  };
  for (int z = z0; z < z1; z += 2) {
    sum_plane(z, cb, kb, ca, ka);
    if (z + 1 < z1) sum_plane(z + 1, ca, ka, cb, kb);
  }
}

template <int G>
void launch_csf(dim3 grid, hipStream_t stream, const double *c, const double *kap, int nx, int ny, int nz, int zc,
                int t0, double gamma, int first, int last, double *fx, double *fy, double *fz) {
  hipLaunchKernelGGL(k_csf<G>, grid, dim3(kTX * kTY), 0, stream, c, kap, nx, ny, nz, zc, t0, gamma, first, last, fx,
                     fy, fz);
}

// Planes per workgroup: 32 (33 planes read for 32 written), fewer while the
// grid has less than two rounds of workgroups at two a CU. 16 against 32:
// 557 and 531 us at 256^3 x 8; 64 is slower again (4.38 and 4.20 ms at 512^3 x 8).
int planes_per_group(int nx, int ny, int nz) {
  int zc = 32;
  while (zc > 2 && (int64_t)ceil_div(nx, kTX) * ceil_div(ny, kTY) * ceil_div(nz, zc) < 1024) zc /= 2;
  return zc;
}

}  // namespace

extern "C" int vofmt_csf_force(vofmt_ctx *ctx, int32_t nx, int32_t ny, int32_t nz, int32_t ntracers,
                               const double *c, const double *kappa, double gamma, double *fx, double *fy, double *fz,
                               hipStream_t stream) {
  if (!ctx) return VOFMT_E_ARG;
  if (nx < 1 || ny < 1 || nz < 1 || ntracers < 0) return set_err(ctx, VOFMT_E_ARG, "vofmt_csf_force: bad sizes");
  if (!std::isfinite(gamma)) return set_err(ctx, VOFMT_E_ARG, "vofmt_csf_force: gamma is not finite");
  if (!fx || !fy || !fz || (ntracers > 0 && (!c || !kappa)))
    return set_err(ctx, VOFMT_E_ARG, "vofmt_csf_force: null pointer");
  VOFMT_HIP(ctx, hipSetDevice(ctx->device));
  const int zc = planes_per_group(nx, ny, nz);
  const int64_t tiles = (int64_t)ceil_div(nx, kTX) * ceil_div(ny, kTY) * ceil_div(nz, zc);
  if (tiles > INT32_MAX) return set_err(ctx, VOFMT_E_ARG, "vofmt_csf_force: grid too large");
  const dim3 grid((unsigned)tiles);
  if (ntracers == 0) {  // no interface: zero force
    launch_csf<0>(grid, stream, c, kappa, nx, ny, nz, zc, 0, gamma, 1, 1, fx, fy, fz);
    return hip_check(ctx, hipGetLastError(), "k_csf");
  }
  // the fewest groups of at most kMaxGroup tracers, of even sizes: every group
  // after the first reads and writes the partial sums again
  const int ngrp = (ntracers + kMaxGroup - 1) / kMaxGroup;
  for (int k = 0, t0 = 0; k < ngrp; ++k) {
    const int g = ntracers / ngrp + (k < ntracers % ngrp ? 1 : 0);
    const int first = t0 == 0, last = t0 + g == ntracers;
    auto go = [&](auto launch) {
      launch(grid, stream, c, kappa, nx, ny, nz, zc, t0, gamma, first, last, fx, fy, fz);
    };
    switch (g) {
      case 8: go(launch_csf<8>); break;
      case 7: go(launch_csf<7>); break;
      case 6: go(launch_csf<6>); break;
      case 5: go(launch_csf<5>); break;
      case 4: go(launch_csf<4>); break;
      case 3: go(launch_csf<3>); break;
      case 2: go(launch_csf<2>); break;
      default: go(launch_csf<1>); break;
    }
    VOFMT_HIP(ctx, hipGetLastError());
    t0 += g;
  }
  return VOFMT_OK;
}
