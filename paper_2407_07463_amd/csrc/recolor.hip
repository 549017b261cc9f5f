// Reassignment of drops in near contact to other tracers: Steps 1-4 of
// section "The no-coalescence.h algorithm".
//
// Reading: drops are the (tracer, label) pairs; two distinct drops are
// neighbours when occupied cells of each lie at a periodic offset o with
// |o|^2 < (1 + gap)^2 (o = 0 included across tracers); neighbours in the
// same tracer conflict; drops are visited in ascending (tracer, label) and a
// drop whose current tracer is held by an earlier neighbour moves to the
// smallest tracer none of its neighbours holds, or to a new one.
//
// GPU scheme:
//   1. own[p]: global id of the only drop occupying cell p, -1 if none,
//      -2 if several (drops of different tracers overlapping);
//   2. the boundary cells of the drops scan the offsets of the ball and set
//      the bits of each pair of neighbouring drops in a D x D adjacency bitmap
//      (atomicOr in both directions; its content is independent of thread
//      order): tile by tile in LDS where the ball reaches 4 cells or less,
//      from an ordered list of those cells beyond that;
//   3. the bitmap is turned into sorted neighbour lists (CSR);
//   4. the greedy pass: in rounds by one workgroup, or by one wavefront when a
//      drop needs a new tracer;
//   5. the host reads back the tracer count (capacity check), then every
//      cell clears its moved-out values and adds them to the new fields.
//
// Stencil mode (vofmt_recolor_tracers_stencil): the neighbour relation of
// step 2 is the paper's criterion read literally. Within a tracer, two drops
// are neighbours when an empty cell (label 0) has one of them and the other
// at opposite offsets +o, -o of the 5x5x5 stencil (Steps 1-3): one thread per
// 64-cell row segment tests the 62 opposite pairs on occupancy bits of the 25
// neighbouring rows, and one wavefront takes each segment that has a pair and
// compares the labels. Across tracers, drops are neighbours ("in contact",
// Step 4) when cells of the two lie within 4 cells along every axis (the
// stencil's reach), found by the scan of step 2 over the half 9x9x9 cube,
// pairs within one tracer skipped.
#include <algorithm>
#include <cstring>

#include "common.hpp"
#include "compact.hpp"

namespace {

constexpr int kBlock = 256;
constexpr int kMaxTracers = 64;    // tracers are bits of a 64-bit mask
constexpr int kMaxDrops = 32768;   // the adjacency bitmap is D^2 bits
constexpr int kChunk = 4096;       // neighbour ids staged in LDS per chunk

struct TracerOffsets {
  int32_t off[kMaxTracers + 1];  // first global drop id of each tracer
};

// Owners are 16-bit: at most kMaxDrops ids, -1 and -2.
typedef int16_t owner_t;
static_assert(kMaxDrops - 1 <= INT16_MAX, "drop ids fit 16 bits");

__device__ __forceinline__ void add_owner(int32_t &o, int32_t l, int t, const TracerOffsets &to) {
  if (l > 0 && to.off[t] + l <= to.off[t + 1]) o = (o == -1) ? to.off[t] + l - 1 : -2;
}

__global__ __launch_bounds__(kBlock) void k_owner(const int32_t *__restrict__ lab, int64_t n3, int ntr,
                                                  TracerOffsets to, owner_t *__restrict__ own) {
  const int64_t p = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (p >= n3) return;
  int32_t o = -1;
  for (int t = 0; t < ntr; ++t) add_owner(o, lab[(int64_t)t * n3 + p], t, to);
  own[p] = (owner_t)o;
}

// The same for 4 consecutive cells per thread with 16-byte label loads
// (labels 16-byte aligned and n3 a multiple of 4).
__global__ __launch_bounds__(kBlock) void k_owner4(const int4 *__restrict__ lab, int64_t n4, int ntr,
                                                   TracerOffsets to, short4 *__restrict__ own) {
  const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (i >= n4) return;
  int32_t o[4] = {-1, -1, -1, -1};
  for (int t = 0; t < ntr; ++t) {
    const int4 l4 = lab[(int64_t)t * n4 + i];
    const int32_t l[4] = {l4.x, l4.y, l4.z, l4.w};
#pragma unroll
    for (int k = 0; k < 4; ++k) add_owner(o[k], l[k], t, to);
  }
  own[i] = make_short4((short)o[0], (short)o[1], (short)o[2], (short)o[3]);
}

// v in (-n, 2n): one conditional add or subtract instead of a modulo
__device__ __forceinline__ int wrap_near(int v, int n) { return v < 0 ? v + n : (v >= n ? v - n : v); }

// The pair (a, b) in both directions.
__device__ __forceinline__ void set_edge(uint32_t *adj, int64_t words, int32_t a, int32_t b) {
  uint32_t *w = adj + (int64_t)a * words + (b >> 5);
  const uint32_t bit = 1u << (b & 31);
  if (*w & bit) return;  // (whoever sets it sets the other direction too)
  atomicOr(w, bit);
  atomicOr(adj + (int64_t)b * words + (a >> 5), 1u << (a & 31));
}

// Calls f(id) for every drop occupying cell p (for cells shared by several drops).
template <class F>
__device__ __forceinline__ void for_drops_at(const int32_t *__restrict__ lab, int64_t n3, int ntr,
                                             const TracerOffsets &to, int64_t p, F f) {
  for (int t = 0; t < ntr; ++t) {
    const int32_t l = lab[(int64_t)t * n3 + p];
    if (l > 0 && to.off[t] + l <= to.off[t + 1]) f(to.off[t] + l - 1);
  }
}

__device__ __forceinline__ void edges_of(const owner_t *__restrict__ own, const int32_t *__restrict__ lab, int nx,
                                         int ny, int nz, int ntr, const TracerOffsets &to,
                                         const int4 *__restrict__ offs, int noffs, int small_offsets,
                                         uint32_t *__restrict__ adj, int64_t words, int64_t n3, const FastDiv &fnx,
                                         const FastDiv &fny, const int32_t *__restrict__ cross_T0, int64_t p) {
  // cross_T0 != null: only drops of different tracers (initial tracer per drop) are related
  auto set_edge = [&](uint32_t *adj_, int64_t words_, int32_t u, int32_t v) {
    if (cross_T0 != nullptr && cross_T0[u] == cross_T0[v]) return;
    ::set_edge(adj_, words_, u, v);
  };
  const int32_t a = own[p];
  const uint32_t r = fast_div((uint32_t)p, fnx), zz = fast_div(r, fny);  // cells < 2^31
  const int x = (int)((uint32_t)p - r * (uint32_t)nx), y = (int)(r - zz * (uint32_t)ny), z = (int)zz;
  if (a == -2) {
    // drops sharing this very cell are neighbours (offset 0 across tracers)
    for_drops_at(lab, n3, ntr, to, p, [&](int32_t u) {
      for_drops_at(lab, n3, ntr, to, p, [&](int32_t v) {
        if (u != v) set_edge(adj, words, u, v);
      });
    });
  }
  // Of a shared cell's drops only those look further that have a boundary here
  // (bits of their tracers): see the choice of cells below, drop by drop.
  uint64_t mine = 0;
  if (a == -2) {
    const int64_t plane = (int64_t)ny * nx, yr = (int64_t)y * nx, zr = z * plane;
    const int64_t xm = zr + yr + wrap_dec(x, nx), xp = zr + yr + wrap_inc(x, nx);
    const int64_t ym = zr + (int64_t)wrap_dec(y, ny) * nx + x, yp = zr + (int64_t)wrap_inc(y, ny) * nx + x;
    const int64_t zm = wrap_dec(z, nz) * plane + yr + x, zp = wrap_inc(z, nz) * plane + yr + x;
    for (int t = 0; t < ntr; ++t) {
      const int32_t *lt = lab + (int64_t)t * n3;
      const int32_t l = lt[p];
      const bool inside = lt[xm] == l && lt[xp] == l && lt[ym] == l && lt[yp] == l && lt[zm] == l && lt[zp] == l;
      if (l > 0 && to.off[t] + l <= to.off[t + 1] && !inside) mine |= 1ull << t;
    }
    if (mine == 0ull) return;
  }
  // The owners of kBatch offsets are loaded together (past the last offset
  // every lane loads its own cell and ignores it); a drop just paired with
  // this cell's drop is not paired again (a boundary cell sees a neighbouring
  // drop through many offsets).
  constexpr int kBatch = 8;
  int32_t last_b = -1;
  for (int k0 = 0; k0 < noffs; k0 += kBatch) {
    int32_t bs[kBatch];
    int64_t qs[kBatch];
#pragma unroll
    for (int j = 0; j < kBatch; ++j) {
      const int k = k0 + j < noffs ? k0 + j : 0;
      const int4 o = offs[k];
      const int64_t q = small_offsets ? ((int64_t)wrap_near(z + o.z, nz) * ny + wrap_near(y + o.y, ny)) * nx +
                                            wrap_near(x + o.x, nx)
                                      : ((int64_t)wrap_any(z + o.z, nz) * ny + wrap_any(y + o.y, ny)) * nx +
                                            wrap_any(x + o.x, nx);
      qs[j] = (k0 + j < noffs) ? q : p;
      bs[j] = own[qs[j]];
    }
#pragma unroll
    for (int j = 0; j < kBatch; ++j) {
      if (k0 + j >= noffs) break;
      const int64_t q = qs[j];
      const int32_t b = bs[j];
      if (b == -1) continue;
      if (a >= 0 && b >= 0) {
        if (a != b && b != last_b) {
          set_edge(adj, words, a, b);
          last_b = b;
        }
        continue;
      }
      // a shared cell on either side: every drop of p with every drop of q
      auto with_q = [&](int32_t u) {
        if (b >= 0) {
          if (u != b) set_edge(adj, words, u, b);
        } else {
          for_drops_at(lab, n3, ntr, to, q, [&](int32_t v) {
            if (u != v) set_edge(adj, words, u, v);
          });
        }
      };
      if (a >= 0) with_q(a);
      else
        for (int t = 0; t < ntr; ++t)
          if ((mine >> t) & 1ull) with_q(to.off[t] + lab[(int64_t)t * n3 + p] - 1);
    }
  }
}


// Cells that can find a pair: shared cells, and cells of one drop with a
// six-neighbour not owned by that drop. An interior cell finds no pair that
// a boundary cell of its drop does not: a lattice path from it towards any
// other drop's cell, one axis step at a time, only gets closer and leaves the
// drop through a boundary cell.
// The owner array (-1 empty, -2 shared, else the drop) of every cell gives
// the predicate: a shared cell, or a cell of one drop with a six-neighbour
// not owned by it. Block counts (kBlock cells) and one bit per cell, for
// compact::k_write_ordered_bits: lane l of a wavefront holds cell p (64
// consecutive cells), its x neighbours come from the lanes beside it, and
// only a row's end cells and the wavefront's edge lanes load theirs. The y
// and z neighbours are loaded for cells of one drop only.
__global__ __launch_bounds__(kBlock) void k_pair_source_counts(const owner_t *__restrict__ own, int nx, int ny,
                                                               int nz, FastDiv fnx, FastDiv fny, int64_t n,
                                                               int32_t *__restrict__ bc, uint64_t *__restrict__ bits) {
  const int64_t p = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  const int lane = threadIdx.x & 63;
  const bool in = p < n;
  const int64_t pc = in ? p : n - 1;  // (a lane past the end shadows the last cell)
  const int32_t a = own[pc];
  const uint32_t r = fast_div((uint32_t)pc, fnx), zz = fast_div(r, fny);
  const int x = (int)((uint32_t)pc - r * (uint32_t)nx), y = (int)(r - zz * (uint32_t)ny), z = (int)zz;
  const int64_t row = (int64_t)r * nx;
  // x neighbours: from the lanes beside, unless across the wavefront's edge or the row's end
  int32_t am = __shfl_up(a, 1, 64), ap = __shfl_down(a, 1, 64);
  const bool load_m = lane == 0 || x == 0, load_p = lane == 63 || x == nx - 1;
  if (a >= 0 && load_m) am = own[row + wrap_dec(x, nx)];
  if (a >= 0 && load_p) ap = own[row + wrap_inc(x, nx)];
  bool hit = false;
  if (a == -2) {
    hit = true;
  } else if (a >= 0) {
    const int64_t plane = (int64_t)ny * nx, zr = (int64_t)z * plane;
    const int32_t ym = own[zr + (int64_t)wrap_dec(y, ny) * nx + x], yp = own[zr + (int64_t)wrap_inc(y, ny) * nx + x];
    const int32_t zm = own[(int64_t)wrap_dec(z, nz) * plane + (int64_t)y * nx + x];
    const int32_t zp = own[(int64_t)wrap_inc(z, nz) * plane + (int64_t)y * nx + x];
    hit = !(am == a && ap == a && ym == a && yp == a && zm == a && zp == a);
  }
  hit = hit && in;
  __shared__ int wc[kBlock / 64];
  const uint64_t mask = __ballot(hit);
  if (lane == 0) {
    wc[threadIdx.x >> 6] = (int)__popcll(mask);
    if (in) bits[p >> 6] = mask;  // (a wavefront wholly past n has no word)
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    int t = 0;
    for (int w = 0; w < kBlock / 64; ++w) t += wc[w];
    bc[blockIdx.x] = t;
  }
}

// Near-contact pairs seen from the listed cells (persistent grid).
__global__ __launch_bounds__(kBlock) void k_edges(const owner_t *__restrict__ own, const int32_t *__restrict__ lab,
                                                  int nx, int ny, int nz, int ntr, TracerOffsets to,
                                                  const int4 *__restrict__ offs, int noffs, int small_offsets,
                                                  const int32_t *__restrict__ list, const int32_t *__restrict__ count,
                                                  uint32_t *__restrict__ adj, int64_t words, FastDiv fnx,
                                                  FastDiv fny, const int32_t *__restrict__ cross_T0) {
  const int64_t n3 = (int64_t)nx * ny * nz;
  const int nlist = *count;
  for (int qi = blockIdx.x * kBlock + threadIdx.x; qi < nlist; qi += gridDim.x * kBlock) {
    const int64_t p = list[qi];
    edges_of(own, lab, nx, ny, nz, ntr, to, offs, noffs, small_offsets, adj, words, n3, fnx, fny, cross_T0, p);
  }
}

// Owners and occupancy of one 64-cell row segment per wavefront, for every
// tracer from one read of its labels: bit l of word occ[t][z][y][w] is
// (label > 0) of cell x = 64 w + l (0 beyond the row). nseg1: words per tracer.
constexpr int kOccBatch = 4;  // tracers whose labels are in flight together
__global__ __launch_bounds__(kBlock) void k_owner_occ(const int32_t *__restrict__ lab, int nx, int64_t nseg1,
                                                      int64_t n3, int words, FastDiv fw, int ntr, TracerOffsets to,
                                                      owner_t *__restrict__ own, uint64_t *__restrict__ occ) {
  const int64_t seg = ((int64_t)blockIdx.x * kBlock + threadIdx.x) >> 6;
  const int lane = threadIdx.x & 63;
  if (seg >= nseg1) return;  // whole wavefront
  const uint32_t row = fast_div((uint32_t)seg, fw);
  const int x = 64 * (int)((uint32_t)seg - row * (uint32_t)words) + lane;
  const int64_t p = (int64_t)row * nx + x;
  const bool in = x < nx;
  int32_t o = -1;
  for (int t0 = 0; t0 < ntr; t0 += kOccBatch) {
    int32_t l[kOccBatch];
#pragma unroll
    for (int k = 0; k < kOccBatch; ++k) l[k] = (in && t0 + k < ntr) ? lab[(int64_t)(t0 + k) * n3 + p] : 0;
#pragma unroll
    for (int k = 0; k < kOccBatch; ++k) {
      if (t0 + k >= ntr) break;
      add_owner(o, l[k], t0 + k, to);
      const uint64_t b = __ballot(l[k] > 0);
      if (lane == 0) occ[(int64_t)(t0 + k) * nseg1 + seg] = b;
    }
  }
  if (in) own[p] = (owner_t)o;
}

// Bit m of v (m < 16) to bit 4m.
__device__ __forceinline__ uint64_t spread4(uint64_t v) {
  v &= 0xFFFFull;
  v = (v | (v << 24)) & 0x000000FF000000FFull;
  v = (v | (v << 12)) & 0x000F000F000F000Full;
  v = (v | (v << 6)) & 0x0303030303030303ull;
  v = (v | (v << 3)) & 0x1111111111111111ull;
  return v;
}

// The same when rows hold a multiple of 256 cells: one wavefront per four
// segments of a row, each lane loading four labels of a tracer at once (cells
// 4l .. 4l+3 of the 256); ballot k holds component k of every lane, and the
// word of segment j interleaves 16 bits of each ballot. One read of the labels
// for owners and words: 104 + 108 us as two passes at 256^3 x 8, 112 us so.
__global__ __launch_bounds__(kBlock) void k_owner_occ4(const int4 *__restrict__ lab4, int64_t ngroups, int ntr,
                                                       TracerOffsets to, short4 *__restrict__ own,
                                                       uint64_t *__restrict__ occ) {
  const int64_t g = ((int64_t)blockIdx.x * kBlock + threadIdx.x) >> 6;
  const int lane = threadIdx.x & 63;
  if (g >= ngroups) return;  // whole wavefront
  int32_t o[4] = {-1, -1, -1, -1};
  for (int t0 = 0; t0 < ntr; t0 += kOccBatch) {
    int4 v[kOccBatch];
#pragma unroll
    for (int k = 0; k < kOccBatch; ++k)  // segments 4g .. 4g+3 are cells 256g .. 256g+255 of a field
      v[k] = lab4[((int64_t)(t0 + k < ntr ? t0 + k : t0) * ngroups + g) * 64 + lane];
#pragma unroll
    for (int k = 0; k < kOccBatch; ++k) {
      const int t = t0 + k;
      if (t >= ntr) break;
      add_owner(o[0], v[k].x, t, to);
      add_owner(o[1], v[k].y, t, to);
      add_owner(o[2], v[k].z, t, to);
      add_owner(o[3], v[k].w, t, to);
      const uint64_t b0 = __ballot(v[k].x > 0), b1 = __ballot(v[k].y > 0), b2 = __ballot(v[k].z > 0),
                     b3 = __ballot(v[k].w > 0);
      if (lane < 4) {
        const int sh = 16 * lane;
        occ[4 * ((int64_t)t * ngroups + g) + lane] =
            spread4(b0 >> sh) | (spread4(b1 >> sh) << 1) | (spread4(b2 >> sh) << 2) | (spread4(b3 >> sh) << 3);
      }
    }
  }
  own[g * 64 + lane] = make_short4((short)o[0], (short)o[1], (short)o[2], (short)o[3]);
}

// Bits of cells xs, xs+1, ..., xs+63 (periodic in x, xs any integer) of one
// row of occupancy words. Windows inside the row take two aligned words; the
// rest (the row's ends, rows shorter than 64 cells) assemble the bits piece by
// piece.
__device__ __forceinline__ uint64_t row_window(const uint64_t *__restrict__ rw, int nx, int xs) {
  if (xs >= 0 && xs + 64 <= nx) {
    const int w = xs >> 6, b = xs & 63;
    return b == 0 ? rw[w] : ((rw[w] >> b) | (rw[w + 1] << (64 - b)));
  }
  int x = wrap_any(xs, nx);
  uint64_t res = 0;
  int got = 0;
  while (got < 64) {
    const int b = x & 63;
    int take = 64 - b;
    if (take > nx - x) take = nx - x;
    if (take > 64 - got) take = 64 - got;
    uint64_t chunk = rw[x >> 6] >> b;
    if (take < 64) chunk &= (1ull << take) - 1ull;
    res |= chunk << got;
    got += take;
    x += take;
    if (x == nx) x = 0;
  }
  return res;
}

// One of each opposite pair of offsets o of the 5x5x5 stencil (o > 0 in
// (z, y, x) order): 62 pairs, as (ox, oy, oz) in -2..2.
struct StencilPairs {
  int8_t o[62][3];
};
static StencilPairs make_stencil_pairs() {
  StencilPairs sp{};
  int k = 0;
  for (int oz = -2; oz <= 2; ++oz)
    for (int oy = -2; oy <= 2; ++oy)
      for (int ox = -2; ox <= 2; ++ox)
        if (oz > 0 || (oz == 0 && (oy > 0 || (oy == 0 && ox > 0)))) {
          sp.o[k][0] = (int8_t)ox;
          sp.o[k][1] = (int8_t)oy;
          sp.o[k][2] = (int8_t)oz;
          ++k;
        }
  return sp;
}

// (t, row of the tracer, y, z, word) of segment seg of all tracers: segment
// counts stay below 2^31, so the divisions are 32-bit multiply-shifts.
struct SegAt {
  int t, w, y, z;
  int64_t r;
};
__device__ __forceinline__ SegAt seg_at(uint32_t seg, int words, int64_t rows, int ny, const FastDiv &fw,
                                        const FastDiv &frows, const FastDiv &fny) {
  SegAt s;
  const uint32_t tr = fast_div(seg, fw);
  s.w = (int)(seg - tr * (uint32_t)words);
  const uint32_t t32 = fast_div(tr, frows);
  s.t = (int)t32;
  s.r = (int64_t)(tr - t32 * (uint32_t)rows);
  const uint32_t z32 = fast_div((uint32_t)s.r, fny);
  s.z = (int)z32;
  s.y = (int)((uint32_t)s.r - z32 * (uint32_t)ny);
  return s;
}

// offsets reach 2 cells: one conditional wrap when the axis has 3 cells or more
__device__ __forceinline__ int wrap2(int v, int n) {
  return n >= 3 ? (v < 0 ? v + n : (v >= n ? v - n : v)) : wrap_any(v, n);
}

// Steps 1-3 find a pair around an empty cell p (label 0) when p + o and p - o
// are occupied for one of the 62 opposite offset pairs. One thread per row
// segment tests all pairs for its 64 cells on occupancy bits: for each of the
// 12 opposite row pairs (and the cell's own row) the row's 64 cells shifted by
// -2 .. 2, and the AND of opposite shifts with the empty cells. A drop of
// convex shape has no such cell (the midpoint of a point in p + o and one in
// p - o lies in p), so few segments are left; their indices are appended to
// `list` in any order. One wavefront per segment instead, a lane per pair,
// spent a wavefront's whole pass on every segment: 642 us at 256^3 x 8, 4.64
// ms at 512^3 x 8, against 95 us and 0.70 ms for this pass and the
// listed segments together.
//
// A row's window needs the two cells before and after its 64. FAST: rows of 3
// cells or more whose last segment holds at least 2 (nx % 64 != 1): they are the
// top and bottom bits of the words beside it (at a row's ends, of its other
// end), and every shifted half is one funnel shift.
template <bool FAST>
__global__ __launch_bounds__(kBlock) void k_stencil_segments(const uint64_t *__restrict__ occ, int nx, int ny, int nz,
                                                             int words, int64_t nseg, FastDiv fw, FastDiv frows,
                                                             FastDiv fny, int32_t *__restrict__ list,
                                                             uint32_t *__restrict__ count) {
  const int64_t seg = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  const int64_t rows = (int64_t)nz * ny;
  uint64_t any = 0;
  if (seg < nseg) {
    const SegAt s = seg_at((uint32_t)seg, words, rows, ny, fw, frows, fny);
    const uint64_t *occ_t = occ + (int64_t)s.t * rows * words;
    const int x0 = 64 * s.w;
    const bool end = s.w == words - 1;
    const int nlast = nx - 64 * (words - 1), nvalid = end ? nlast : 64;
    const uint64_t valid = nvalid == 64 ? ~0ull : ((1ull << nvalid) - 1ull);
    const int ip = s.w > 0 ? s.w - 1 : words - 1;  // the words before and after, around the row
    const int in = end ? 0 : s.w + 1;
    const int shp = s.w > 0 ? 0 : 64 - nlast;      // brings the cell before x0 to bit 63
    const int shn = 64 - nvalid;                   // and the cell after the 64 to bit 0
    // the 64 cells from x0 + d, d = -2 .. 2, of a row, as halves
    struct Shifts {
      uint32_t lo[5], hi[5];
    };
    auto shifts = [&](int dy, int dz) -> Shifts {
      const uint64_t *rw = occ_t + (uint32_t)((wrap2(s.z + dz, nz) * ny + wrap2(s.y + dy, ny)) * words);
      Shifts o;
      if constexpr (FAST) {
        const uint64_t nw = rw[in], w0 = rw[s.w];
        const uint32_t before = (uint32_t)((rw[ip] << shp) >> 32), after = (uint32_t)(nw >> shn);
        const uint64_t w = shn > 0 ? w0 | (nw << nvalid) : w0;
        const uint32_t l = (uint32_t)w, h = (uint32_t)(w >> 32);
        o.lo[0] = __builtin_amdgcn_alignbit(l, before, 30);
        o.hi[0] = __builtin_amdgcn_alignbit(h, l, 30);
        o.lo[1] = __builtin_amdgcn_alignbit(l, before, 31);
        o.hi[1] = __builtin_amdgcn_alignbit(h, l, 31);
        o.lo[2] = l;
        o.hi[2] = h;
        o.lo[3] = __builtin_amdgcn_alignbit(h, l, 1);
        o.hi[3] = __builtin_amdgcn_alignbit(after, h, 1);
        o.lo[4] = __builtin_amdgcn_alignbit(h, l, 2);
        o.hi[4] = __builtin_amdgcn_alignbit(after, h, 2);
      } else {
        for (int d = 0; d < 5; ++d) {
          const uint64_t v = row_window(rw, nx, x0 + d - 2);
          o.lo[d] = (uint32_t)v;
          o.hi[d] = (uint32_t)(v >> 32);
        }
      }
      return o;
    };
    const Shifts c = shifts(0, 0);
    uint32_t lo = (c.lo[0] & c.lo[4]) | (c.lo[1] & c.lo[3]), hi = (c.hi[0] & c.hi[4]) | (c.hi[1] & c.hi[3]);
#pragma unroll
    for (int k = 0; k < 12; ++k) {
      const int dz = k < 2 ? 0 : (k < 7 ? 1 : 2), dy = k < 2 ? k + 1 : (k < 7 ? k - 4 : k - 9);
      const Shifts a = shifts(dy, dz), b = shifts(-dy, -dz);
#pragma unroll
      for (int d = 0; d < 5; ++d) {
        lo |= a.lo[d] & b.lo[4 - d];
        hi |= a.hi[d] & b.hi[4 - d];
      }
    }
    any = (((uint64_t)hi << 32) | lo) & ~(((uint64_t)c.hi[2] << 32) | c.lo[2]) & valid;
  }
  const uint64_t mask = __ballot(any != 0ull);
  if (mask == 0ull) return;  // whole wavefront
  const int lane = threadIdx.x & 63;
  uint32_t base = 0;
  if (lane == 0) base = atomicAdd(count, (uint32_t)__popcll(mask));
  base = (uint32_t)__builtin_amdgcn_readfirstlane((int)base);
  if (any != 0ull) list[base + (uint32_t)__popcll(mask & ((1ull << lane) - 1ull))] = (int32_t)seg;
}

// The pairs of the listed segments (persistent grid, one wavefront per
// segment). Lane k < 62 takes the opposite pair k of the stencil, offsets +o
// and -o, and forms from three 64-bit windows of occupancy bits the cells whose
// centre is empty and whose cells at +o and -o are both occupied; for each such
// cell it loads the two labels and records the two drops as neighbours when
// they differ (Step 3).
__global__ __launch_bounds__(kBlock) void k_stencil_edges(const int32_t *__restrict__ lab,
                                                          const uint64_t *__restrict__ occ, int nx, int ny, int nz,
                                                          int words, TracerOffsets to, StencilPairs sp,
                                                          uint32_t *__restrict__ adj, int64_t awords, FastDiv fw,
                                                          FastDiv frows, FastDiv fny, const int32_t *__restrict__ list,
                                                          const uint32_t *__restrict__ count) {
  const int lane = threadIdx.x & 63;
  const int64_t rows = (int64_t)nz * ny;
  const uint32_t nlist = *count;
  for (uint32_t q = (blockIdx.x * kBlock + threadIdx.x) >> 6; q < nlist; q += gridDim.x * (kBlock / 64)) {
  const SegAt sg = seg_at((uint32_t)list[q], words, rows, ny, fw, frows, fny);
  const int t = sg.t, w = sg.w, y = sg.y, z = sg.z;
  const int64_t r = sg.r;
  const uint64_t *occ_t = occ + (int64_t)t * rows * words;
  const int x0 = 64 * w;
  const int nvalid = nx - x0 < 64 ? nx - x0 : 64;
  const uint64_t valid = nvalid == 64 ? ~0ull : ((1ull << nvalid) - 1ull);
  const uint64_t empty = ~occ_t[r * words + w] & valid;  // bit i: cell x0 + i has no drop of tracer t
  uint64_t cand = 0;
  int ox = 0, oy = 0, oz = 0;
  if (lane < 62) {
    ox = sp.o[lane][0];
    oy = sp.o[lane][1];
    oz = sp.o[lane][2];
    const uint64_t *rp = occ_t + ((int64_t)wrap2(z + oz, nz) * ny + wrap2(y + oy, ny)) * words;
    const uint64_t *rm = occ_t + ((int64_t)wrap2(z - oz, nz) * ny + wrap2(y - oy, ny)) * words;
    // bit i: cell x0 + i + ox of the row at +o, cell x0 + i - ox of the row at -o
    cand = row_window(rp, nx, x0 + ox) & row_window(rm, nx, x0 - ox) & empty;
  }
  const int64_t rowp = ((int64_t)t * nz + wrap2(z + oz, nz)) * ny + wrap2(y + oy, ny);
  const int64_t rowm = ((int64_t)t * nz + wrap2(z - oz, nz)) * ny + wrap2(y - oy, ny);
  const int64_t qc = (((int64_t)t * nz + z) * ny + y) * nx + x0;  // a cell of the segment (x0 < nx)
  // The labels of up to kBatch cells are loaded together (every lane loads,
  // from the segment's first cell when it has no cell left, and selects
  // afterwards); a pair of drops just recorded by this lane is not recorded
  // again (the cells of a gap between two drops mostly see the same pair).
  constexpr int kBatch = 8;
  int32_t last_a = 0, last_b = 0;
  while (cand) {
    int32_t la[kBatch], lb[kBatch];
    bool has[kBatch];
#pragma unroll
    for (int u = 0; u < kBatch; ++u) {
      has[u] = cand != 0ull;
      const int i = has[u] ? __ffsll((unsigned long long)cand) - 1 : 0;
      cand &= cand - 1;
      const int x = x0 + i;
      const int64_t qp = rowp * nx + wrap2(x + ox, nx), qm = rowm * nx + wrap2(x - ox, nx);
      la[u] = lab[has[u] ? qp : qc];
      lb[u] = lab[has[u] ? qm : qc];
    }
#pragma unroll
    for (int u = 0; u < kBatch; ++u) {
      const int32_t a = la[u], b = lb[u];
      if (has[u] && a != b && a > 0 && b > 0 && to.off[t] + a <= to.off[t + 1] && to.off[t] + b <= to.off[t + 1] &&
          !(a == last_a && b == last_b)) {
        const int32_t ga = to.off[t] + a - 1, gb = to.off[t] + b - 1;
        set_edge(adj, awords, ga, gb);
        last_a = a;
        last_b = b;
      }
    }
  }
  }
}

// Near-contact pairs, tile by tile: a workgroup takes 64 x 8 x 8 cells and
// holds their owners in LDS with the halo that a half ball of reach R needs (R
// cells along x and y on both sides, R above and one below along z). The
// tile's boundary cells (a shared cell, or a cell of one drop with a
// six-neighbour not owned by it: an interior cell finds no pair that a boundary
// cell of its drop does not, since a lattice path from it towards any other
// drop's cell, one axis step at a time, only gets closer and leaves the drop
// through a boundary cell) are compacted into an LDS list, so that full
// wavefronts scan the offsets, and every owner they look at is an LDS read.
// From a list of those cells in memory (counted, scanned, written, then
// scattered 4-byte loads, one cache line per lane) the same pairs took 1.60 ms
// at 512^3 x 8 drops with the 40 offsets of the distance 1.5 and 0.39 ms so;
// the 364 offsets of the stencil mode 4.9 ms, and 1.06 ms so. Most boundary
// cells have no other drop near: those whose reach, taken as whole groups of 4
// cells along x and the whole y-range, holds one drop are not listed (0.39 ->
// 0.33 and 1.06 -> 0.90 ms).
// cross_T0 != null: only drops of different tracers (initial tracer per drop)
// are related.
constexpr int kTileX = 64, kTileY = 8, kTileZ = 8;
constexpr int kMaxTileReach = 4;
constexpr int kHaloX = 4;  // cells of x-halo held, whatever the reach: the tile's rows stay 8-byte aligned
constexpr int kPairCache = 256;
// The half ball as rows of cells along x: row k covers x + lo .. x + hi at the
// LDS offset `base` of its (dy, dz), offsets first .. first + hi - lo of the ball's.
constexpr int kMaxTileRows = (kMaxTileReach + 1) * (2 * kMaxTileReach + 1);
struct TileRows {
  int n, all;
  int16_t base[kMaxTileRows], first[kMaxTileRows];
  int8_t lo[kMaxTileRows], hi[kMaxTileRows];
};
template <int R>
struct TileDims {
  static constexpr int LX = kTileX + 2 * kHaloX, LY = kTileY + 2 * R, LZ = kTileZ + R + 1;
};
typedef uint16_t owner2 __attribute__((ext_vector_type(2)));
typedef int16_t sowner2 __attribute__((ext_vector_type(2)));
// Smallest and largest drop of a group of cells, in the low and the high half:
// minima of the unsigned values, in which cells of no or of several drops are the
// largest, and maxima of the signed, in which they are the smallest.
constexpr uint32_t kNoDrops = 0xFFFFFFFFu;
__device__ __forceinline__ uint32_t low_high(uint32_t u, uint32_t v) {
  const uint32_t lo = (u & 0xFFFFu) < (v & 0xFFFFu) ? u & 0xFFFFu : v & 0xFFFFu;
  const int32_t hu = (int32_t)u >> 16, hv = (int32_t)v >> 16;
  return lo | ((uint32_t)(hu > hv ? hu : hv) << 16);
}

// split workgroups take a tile together, each with its owners in LDS and the
// boundary cells of every split-th group of 16 rows: up to kSplitTiles of them,
// two a CU (two fields of 64^3, 64 tiles, a tenth of the cells shared, gap 3.5
// and stencil 1.20 and 1.55 ms without the split, 0.49 and 0.64 so; 18 separate
// drops 149 -> 133 and 184 -> 166 us).
constexpr int64_t kSplitTiles = 512;
template <int R>
__global__ __launch_bounds__(kBlock) void k_tile_edges(const owner_t *__restrict__ own,
                                                       const int32_t *__restrict__ lab, int nx, int ny, int nz,
                                                       int ntr, TracerOffsets to, TileRows rows,
                                                       int tx, int ty, int split, uint32_t *__restrict__ adj,
                                                       int64_t words, const int32_t *__restrict__ cross_T0) {
  constexpr int LX = TileDims<R>::LX, LY = TileDims<R>::LY, LZ = TileDims<R>::LZ;
  constexpr int kWaves = kBlock / 64, kRows = LY * LZ;
  constexpr int ND = R + 1;  // pairs of cells that cover 2 R + 1 cells from either parity
  // (8 entries behind the last row: a window's superset may end there)
  __shared__ __attribute__((aligned(16))) owner_t tile[LX * kRows + 8];
  // cells of one drop from the front, shared cells from the back
  constexpr int kCellsOfTile = kTileX * kTileY * kTileZ;
  __shared__ uint16_t list[kCellsOfTile];
  __shared__ uint32_t known[kPairCache];  // pairs already in the bitmap
  __shared__ int nlist, nshared;
  // smallest and largest drop: of 4 cells along x and all y of a plane, and of
  // what the half balls of 4 of the tile's cells in a plane can reach
  constexpr int kGroupsX = LX / 4, kOwnX = kTileX / 4;
  // In their place then the half ball's offsets, for the shared cells: (ox, oy, oz)
  // + 8 in 4 bits each, the LDS offset above (four workgroups of R = 4 a CU, not three).
  constexpr int kBall = ((2 * R + 1) * (2 * R + 1) * (2 * R + 1) - 1) / 2, kReach = kGroupsX * LZ + kOwnX * kTileZ;
  __shared__ uint32_t small[kBall > kReach ? kBall : kReach];
  uint32_t *const of_group = small, *const in_reach = small + kGroupsX * LZ, *const ball = small;
  static_assert(kGroupsX * LZ <= kBlock && kOwnX * kTileZ <= kBlock && kMaxTileReach <= 4, "a thread each, x-reach of one group");
  // each XCD takes a contiguous run of tiles, so that a tile's halo is in its L2
  const unsigned nwg = gridDim.x, per = nwg / 8, rem = nwg % 8, k8 = blockIdx.x % 8;
  const unsigned W = k8 * per + (k8 < rem ? k8 : rem) + blockIdx.x / 8, L = W / split;
  const int part = (int)(W % split);
  const int x0 = (int)(L % tx) * kTileX, y0 = (int)((L / tx) % ty) * kTileY, z0 = (int)(L / ((unsigned)tx * ty)) * kTileZ;
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // Cells before the tile's row (y0 - R + ly, z0 - 1 + lz): at_y[ly] + at_z[lz],
  // -1 for a row R or more past the grid's end, nobody's neighbour here.
  __shared__ int32_t at_y[LY], at_z[LZ];
  if (threadIdx.x == 0) nlist = nshared = 0;
  if (threadIdx.x < kPairCache) known[threadIdx.x] = ~0u;
  if (threadIdx.x < 8) tile[LX * kRows + threadIdx.x] = (owner_t)-1;
  if (threadIdx.x < LY) {
    const int y = y0 - R + (int)threadIdx.x;
    at_y[threadIdx.x] = y < ny + R ? wrap_near(y, ny) * nx : -1;
  } else if (threadIdx.x >= 64 && threadIdx.x < 64 + LZ) {
    const int z = z0 - 1 + (int)threadIdx.x - 64;
    at_z[threadIdx.x - 64] = z < nz + R ? wrap_near(z, nz) * (ny * nx) : -1;
  }
  __syncthreads();
  if (nx % 4 == 0) {
    // groups of 4 cells, 8 bytes, that never straddle a row's end: a thread
    // keeps its group of the row and takes every kStep-th row
    constexpr int kGroups = LX / 4, kStep = kBlock / kGroups, kInFlight = 5;
    const int r1 = threadIdx.x / kGroups, g = threadIdx.x % kGroups;
    const int xg = x0 - kHaloX + 4 * g;
    const bool mine = r1 < kStep && xg < nx + kHaloX;
    const owner_t *src = own + wrap_near(xg, nx);
    for (int r0 = r1; r0 < kRows; r0 += kStep * kInFlight) {
      uint2 v[kInFlight];
#pragma unroll
      for (int k = 0; k < kInFlight; ++k) {
        const int r = r0 + k * kStep;
        v[k] = make_uint2(~0u, ~0u);
        if (r < kRows && mine) {
          const int oy = at_y[r % LY], oz = at_z[r / LY];
          if (oy >= 0 && oz >= 0) v[k] = *(const uint2 *)(src + (uint32_t)(oy + oz));
        }
      }
#pragma unroll
      for (int k = 0; k < kInFlight; ++k)
        if (r0 + k * kStep < kRows && r1 < kStep) *(uint2 *)(tile + (r0 + k * kStep) * LX + 4 * g) = v[k];
    }
  } else {
    auto owner_at = [&](int r, int i) -> owner_t {
      const int x = x0 - kHaloX + i, oy = at_y[r % LY], oz = at_z[r / LY];
      return (x < nx + kHaloX && oy >= 0 && oz >= 0) ? own[(uint32_t)(oy + oz + wrap_near(x, nx))] : (owner_t)-1;
    };
    // 64 cells of a row per wavefront, then the last 8 of the rows
    constexpr int kInFlight = 13;
    for (int r0 = wv; r0 < kRows; r0 += kWaves * kInFlight) {
      owner_t v[kInFlight];
#pragma unroll
      for (int k = 0; k < kInFlight; ++k) v[k] = r0 + k * kWaves < kRows ? owner_at(r0 + k * kWaves, lane) : (owner_t)-1;
#pragma unroll
      for (int k = 0; k < kInFlight; ++k)
        if (r0 + k * kWaves < kRows) tile[(r0 + k * kWaves) * LX + lane] = v[k];
    }
    for (int e = threadIdx.x; e < kRows * 8; e += kBlock) tile[(e >> 3) * LX + 64 + (e & 7)] = owner_at(e >> 3, 64 + (e & 7));
  }
  __syncthreads();
  if (threadIdx.x < kGroupsX * LZ) {
    const int g = threadIdx.x % kGroupsX, lz = threadIdx.x / kGroupsX;
    owner2 lo = (uint16_t)0xFFFF;
    sowner2 hi = (int16_t)-1;
    for (int ly = 0; ly < LY; ++ly) {
      const uint2 w = *(const uint2 *)(tile + (lz * LY + ly) * LX + 4 * g);
      lo = __builtin_elementwise_min(lo, __builtin_elementwise_min(__builtin_bit_cast(owner2, w.x), __builtin_bit_cast(owner2, w.y)));
      hi = __builtin_elementwise_max(hi, __builtin_elementwise_max(__builtin_bit_cast(sowner2, w.x), __builtin_bit_cast(sowner2, w.y)));
    }
    of_group[threadIdx.x] = low_high((uint32_t)lo.x | ((uint32_t)(uint16_t)hi.x << 16), (uint32_t)lo.y | ((uint32_t)(uint16_t)hi.y << 16));
  }
  __syncthreads();
  if (threadIdx.x < kOwnX * kTileZ) {
    const int g = threadIdx.x % kOwnX + kHaloX / 4, dz = threadIdx.x / kOwnX;
    uint32_t m = kNoDrops;
#pragma unroll
    for (int oz = 0; oz <= R; ++oz)
#pragma unroll
      for (int og = -1; og <= 1; ++og) m = low_high(m, of_group[(dz + 1 + oz) * kGroupsX + g + og]);
    in_reach[threadIdx.x] = m;
  }
  __syncthreads();
  // boundary cells: 4 consecutive cells per lane, 4 rows per wavefront; not
  // those that reach no drop but their own
  for (int r0 = 4 * (wv + kWaves * part); r0 < kTileY * kTileZ; r0 += 4 * kWaves * split) {
    const int r = r0 + (lane >> 4), dy = r % kTileY, dz = r / kTileY;
    const int xl = 4 * (lane & 15), i = ((dz + 1) * LY + dy + R) * LX + kHaloX + xl;
    auto four = [&](int at) { return *(const uint64_t *)(tile + at); };
    const uint64_t c = four(i);
    // fields that differ from a neighbour's along x, y or z
    const uint64_t d = (c ^ ((c << 16) | (uint16_t)tile[i - 1])) | (c ^ ((c >> 16) | ((uint64_t)(uint16_t)tile[i + 4] << 48))) |
                       (c ^ four(i - LX)) | (c ^ four(i + LX)) | (c ^ four(i - LX * LY)) | (c ^ four(i + LX * LY));
    const bool in = y0 + dy < ny && z0 + dz < nz;
    const uint32_t reached = in_reach[dz * kOwnX + (lane & 15)];
    const bool others = (reached & 0xFFFFu) != reached >> 16;
    uint64_t mask[4];
    int total = 0, at = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int32_t a = (int16_t)(c >> (16 * k));
      const bool cell = in && x0 + xl + k < nx;
      if (cell && a == -2) list[kCellsOfTile - 1 - atomicAdd(&nshared, 1)] = (uint16_t)(i + k);
      mask[k] = __ballot(others && cell && a >= 0 && ((d >> (16 * k)) & 0xFFFFull) != 0ull);
      total += (int)__popcll(mask[k]);
    }
    if (total == 0) continue;  // whole wavefront
    if (lane == 0) at = atomicAdd(&nlist, total);
    at = __builtin_amdgcn_readfirstlane(at);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int e = at + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(mask[k] >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask[k], 0u));
      if ((mask[k] >> lane) & 1ull) list[e] = (uint16_t)(i + k);
      at += (int)__popcll(mask[k]);
    }
  }
  __syncthreads();
  const int n = nlist;
  const int64_t n3 = (int64_t)nx * ny * nz;
  auto edge = [&](int32_t u, int32_t v) {
    if (u == v) return;
    const uint32_t key = (uint32_t)u * kMaxDrops + (uint32_t)v;
    uint32_t *slot = &known[((uint32_t)u * 31u + (uint32_t)v) % kPairCache];
    if (*slot == key) return;
    *slot = key;
    if (cross_T0 != nullptr && cross_T0[u] == cross_T0[v]) return;
    set_edge(adj, words, u, v);
  };
  // A row is looked at cell by cell only where some cell of it (or of the one
  // beside it that the pairs of cells include) holds one drop, not this cell's
  // and not the one just paired (a boundary cell sees a neighbouring drop
  // through many offsets). Shared cells are left to the loop below.
  for (int q = threadIdx.x; q < n; q += kBlock) {
    const int i = list[q];
    const int32_t a = tile[i];
    int32_t last = a;
    const owner2 none = (uint16_t)0xFFFF, several = (uint16_t)0xFFFE, mine = (uint16_t)a;
    for (int k = 0; k < rows.n; ++k) {
      const int at = i + rows.base[k];
      const int s0 = (at + rows.lo[k]) & ~1;
      const owner2 before = (uint16_t)last;
      owner2 m = 0;
#pragma unroll
      for (int j = 0; j < ND; ++j) {
        const owner2 w = *(const owner2 *)(tile + s0 + 2 * j);
        // 0 for -1 and -2 (the two largest), for a and for last
        m |= __builtin_elementwise_min(__builtin_elementwise_min((owner2)(w ^ mine), (owner2)(w ^ before)),
                                       __builtin_elementwise_min((owner2)(w ^ none), (owner2)(w ^ several)));
      }
      if (__builtin_bit_cast(uint32_t, m) == 0u) continue;
      for (int dx = rows.lo[k]; dx <= rows.hi[k]; ++dx) {
        const int32_t b = tile[at + dx];
        if (b < 0 || b == a || b == last) continue;
        edge(a, b);
        last = b;
      }
    }
  }
  // Shared cells, a wavefront each: the drops sharing one are neighbours (offset 0
  // across tracers), and those that have a boundary there (a six-neighbour without
  // the drop; the argument above holds for each drop) look through the ball, a lane
  // per offset of its forward half and of the opposite one. The cells of one drop
  // above do not look at shared ones, so these look at cells of one drop on both
  // sides, and at shared cells forwards. Every tracer's labels there are read once
  // for all the drops of this cell.
  // (Four fields of 192^3 whose drops overlap, the whole call with gap 1.5, gap 3.5
  // and the stencil: every drop of the cell through the whole cube around it, shared
  // cells both ways and their labels once per drop, 10.8, 59.5 and 65.2 ms; 3.3, 5.7
  // and 7.4 so; from the list in memory, a thread per cell, 4.7, 15.7 and 33.8.)
  if (nshared == 0) return;  // (uniform over the workgroup)
  constexpr int kTurns = (kBall + 63) / 64, kLabels = 4;  // offsets a lane; tracers whose labels are in flight together
  if (threadIdx.x < rows.n) {
    const int base = rows.base[threadIdx.x], lo = rows.lo[threadIdx.x], first = rows.first[threadIdx.x];
    const int row = base / LX, oz = (row + R) / LY, oy = row - oz * LY;  // (base = LX (LY oz + oy))
    for (int dx = lo; dx <= rows.hi[threadIdx.x]; ++dx)
      ball[first + dx - lo] = ((uint32_t)(base + dx) << 16) | (uint32_t)((oz + 8) << 8 | (oy + 8) << 4 | (dx + 8));
  }
  __syncthreads();
  for (int q = wv; q < nshared; q += kWaves) {
    const int i = list[kCellsOfTile - 1 - q], r = i / LX;
    const int x = x0 - kHaloX + i % LX, y = y0 - R + r % LY, z = z0 - 1 + r / LY;
    auto cell_at = [&](int ox, int oy, int oz) {
      return ((int64_t)wrap_near(z + oz, nz) * ny + wrap_near(y + oy, ny)) * nx + wrap_near(x + ox, nx);
    };
    int32_t here = -1;  // lane t: the drop of tracer t here (at most 64 tracers)
    bool boundary = false;
    if (lane < ntr) {
      const int32_t *l = lab + (int64_t)lane * n3;
      const int32_t l0 = l[cell_at(0, 0, 0)];
      const int32_t xm = l[cell_at(-1, 0, 0)], xp = l[cell_at(1, 0, 0)], ym = l[cell_at(0, -1, 0)],
                    yp = l[cell_at(0, 1, 0)], zm = l[cell_at(0, 0, -1)], zp = l[cell_at(0, 0, 1)];
      if (l0 > 0 && to.off[lane] + l0 <= to.off[lane + 1]) here = to.off[lane] + l0 - 1;
      boundary = here >= 0 && !(xm == l0 && xp == l0 && ym == l0 && yp == l0 && zm == l0 && zp == l0);
    }
    for (uint64_t left = __ballot(here >= 0); left; left &= left - 1) {
      const int32_t u = __builtin_amdgcn_readlane(here, (int)__builtin_ctzll(left));
      if (here > u) edge(u, here);
    }
    const uint64_t drops = __ballot(boundary);
    if (drops == 0ull || rows.all == 0) continue;  // whole wavefront
    auto pairs_with = [&](int32_t v) {
      for (uint64_t left = drops; left; left &= left - 1)
        edge(__builtin_amdgcn_readlane(here, (int)__builtin_ctzll(left)), v);
    };
    // (every lane loads, from a valid slot when it has no offset or no shared cell there)
    int32_t f[kTurns], g[kTurns], at[kTurns];
    bool shared = false;
#pragma unroll
    for (int j = 0; j < kTurns; ++j) {
      const bool in = lane + 64 * j < rows.all;
      const uint32_t o = ball[in ? lane + 64 * j : 0];
      const int ox = (int)(o & 15u) - 8, oy = (int)(o >> 4 & 15u) - 8, oz = (int)(o >> 8 & 15u) - 8;
      f[j] = tile[i + ((int32_t)o >> 16)];
      g[j] = own[cell_at(-ox, -oy, -oz)];
      if (!in) f[j] = g[j] = -1;
      at[j] = f[j] == -2 ? (int32_t)cell_at(ox, oy, oz) : (int32_t)cell_at(0, 0, 0);
      shared = shared || f[j] == -2;
    }
#pragma unroll
    for (int j = 0; j < kTurns; ++j) {
      if (f[j] >= 0) pairs_with(f[j]);
      if (g[j] >= 0) pairs_with(g[j]);
    }
    if (__ballot(shared) == 0ull) continue;  // whole wavefront
    for (int t0 = 0; t0 < ntr; t0 += kLabels) {
      int32_t l[kTurns][kLabels];
#pragma unroll
      for (int j = 0; j < kTurns; ++j)
#pragma unroll
        for (int k = 0; k < kLabels; ++k) l[j][k] = lab[(int64_t)(t0 + k < ntr ? t0 + k : t0) * n3 + at[j]];
#pragma unroll
      for (int j = 0; j < kTurns; ++j)
#pragma unroll
        for (int k = 0; k < kLabels; ++k) {
          const int t = t0 + k;
          if (t < ntr && f[j] == -2 && l[j][k] > 0 && to.off[t] + l[j][k] <= to.off[t + 1]) pairs_with(to.off[t] + l[j][k] - 1);
        }
    }
  }
}

__global__ void k_fill_u32(uint32_t *p, int64_t n, uint32_t v) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    p[i] = v;
}

__global__ void k_fill_f64(double *p, int64_t n, double v) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    p[i] = v;
}

// Degree of every drop: one wavefront per drop, its row of the bitmap read in
// order (a thread per drop, rows apart, took 33 us at 5508 drops, 5 so).
__global__ __launch_bounds__(kBlock) void k_degree(const uint32_t *__restrict__ adj, int32_t D, int64_t words,
                                                   int32_t *__restrict__ deg) {
  const int32_t g = (int32_t)(((int64_t)blockIdx.x * kBlock + threadIdx.x) >> 6);
  const int lane = threadIdx.x & 63;
  if (g >= D) return;  // whole wavefront
  int s = 0;
  for (int64_t w = lane; w < words; w += 64) s += __popc(adj[(int64_t)g * words + w]);
#pragma unroll
  for (int k = 32; k > 0; k >>= 1) s += __shfl_xor(s, k, 64);
  if (lane == 0) deg[g] = s;
}

// Exclusive scan of D degrees (single workgroup) into rowptr[0..D].
__global__ __launch_bounds__(1024) void k_scan_deg(const int32_t *__restrict__ deg, int32_t D,
                                                   int32_t *__restrict__ rowptr) {
  __shared__ int64_t part[1024];
  const int t = threadIdx.x;
  const int64_t per = ((int64_t)D + 1023) / 1024;
  const int64_t lo = t * per, hi = (lo + per < D) ? lo + per : D;
  int64_t s = 0;
  for (int64_t i = lo; i < hi; ++i) s += deg[i];
  part[t] = s;
  __syncthreads();
  for (int off = 1; off < 1024; off <<= 1) {
    int64_t add = (t >= off) ? part[t - off] : 0;
    __syncthreads();
    part[t] += add;
    __syncthreads();
  }
  int64_t run = (t == 0) ? 0 : part[t - 1];
  for (int64_t i = lo; i < hi; ++i) {
    rowptr[i] = (int32_t)run;
    run += deg[i];
  }
  if (t == 1023) rowptr[D] = (int32_t)part[1023];
}

// The neighbours of every drop in ascending order, one wavefront per drop: 64
// words a round, each lane's offset from the words before it.
__global__ __launch_bounds__(kBlock) void k_csr_fill(const uint32_t *__restrict__ adj, int32_t D, int64_t words,
                                                     const int32_t *__restrict__ rowptr, int32_t cap,
                                                     int32_t *__restrict__ nbr) {
  if (rowptr[D] > cap) return;  // (k_greedy_rounds tells)
  const int32_t g = (int32_t)(((int64_t)blockIdx.x * kBlock + threadIdx.x) >> 6);
  const int lane = threadIdx.x & 63;
  if (g >= D) return;  // whole wavefront
  int32_t e0 = rowptr[g];
  for (int64_t w0 = 0; w0 < words; w0 += 64) {
    const int64_t w = w0 + lane;
    uint32_t bits = w < words ? adj[(int64_t)g * words + w] : 0u;
    const int mine = __popc(bits);
    int upto = mine;  // of the lanes up to this one
#pragma unroll
    for (int k = 1; k < 64; k <<= 1) {
      const int below = __shfl_up(upto, k, 64);
      if (lane >= k) upto += below;
    }
    int32_t e = e0 + upto - mine;
    while (bits) {
      const int b = __ffs(bits) - 1;
      bits &= bits - 1;
      nbr[e++] = (int32_t)(w * 32 + b);
    }
    e0 += __shfl(upto, 63, 64);
  }
}

// The greedy pass, one wavefront. T0: initial tracer per drop. Outputs
// new_tracer, and res[0] = tracers after, res[1] = moved drops, res[2] = 1 on
// capacity overflow (then new_tracer is meaningless and nothing is moved).
__global__ __launch_bounds__(64) void k_greedy(const int32_t *__restrict__ rowptr, const int32_t *__restrict__ nbr,
                                               const int32_t *__restrict__ T0, int32_t D, int ntr, int max_tracers,
                                               int32_t *__restrict__ new_tracer, int32_t *__restrict__ res) {
  __shared__ int8_t T[kMaxDrops];
  __shared__ int32_t stage[kChunk];
  const int lane = threadIdx.x;
  for (int32_t g = lane; g < D; g += 64) T[g] = (int8_t)T0[g];
  __syncthreads();
  int N = ntr;
  int32_t moved = 0;
  int overflow = 0;
  int32_t base = 0;  // first neighbour index staged
  int32_t staged_end = 0;
  for (int32_t g = 0; g < D && !overflow; ++g) {
    const int32_t e0 = rowptr[g], e1 = rowptr[g + 1];
    const int tg = T[g];
    bool conflict = false;
    uint64_t used = 0;
    for (int32_t e = e0; e < e1; e += 64) {
      // make sure [e, min(e+64, e1)) is staged
      if (e + 64 > staged_end && staged_end < e1) {
        __syncthreads();
        base = e;
        staged_end = (base + kChunk < rowptr[D]) ? base + kChunk : rowptr[D];
        for (int32_t k = lane; k < staged_end - base; k += 64) stage[k] = nbr[base + k];
        __syncthreads();
      }
      const int32_t idx = e + lane;
      bool c = false;
      uint64_t u = 0;
      if (idx < e1) {
        const int32_t h = stage[idx - base];
        const int th = T[h];
        c = (h < g) && (th == tg);
        u = 1ull << th;
      }
      conflict = conflict || (__ballot(c) != 0ull);
      // OR-reduction of the tracer masks across the wavefront
#pragma unroll
      for (int s = 32; s > 0; s >>= 1) u |= __shfl_xor(u, s, 64);
      used |= u;
    }
    if (!conflict) continue;
    uint64_t avail = ~used & ~(1ull << tg);
    if (N < 64) avail &= (1ull << N) - 1;
    int n;
    if (avail) {
      n = __ffsll((unsigned long long)avail) - 1;
    } else {
      if (N + 1 > max_tracers) {
        overflow = 1;
        break;
      }
      n = N++;
    }
    __syncthreads();
    if (lane == 0) T[g] = (int8_t)n;
    ++moved;
    __syncthreads();
  }
  __syncthreads();
  for (int32_t g = lane; g < D; g += 64) new_tracer[g] = T[g];
  if (lane == 0) {
    res[0] = N;
    res[1] = moved;
    res[2] = overflow;
  }
}

// The same greedy pass decided in rounds by one workgroup. A drop's decision
// reads the final tracers of its earlier neighbours and the initial tracers
// of its later ones (a later neighbour cannot be decided before it), and the
// number of tracers in use, which changes only when a drop needs a new
// tracer. With no new tracer, a drop can be decided as soon as all its
// earlier neighbours are, and the result is the sequential pass's: each round
// decides every such drop (the smallest undecided drop always is one, so the
// rounds end), then applies the decisions. If some drop needs a new tracer,
// res[3] = 1 and the caller runs the sequential pass instead; if the neighbour
// list was too short, res[3] = 2 and res[4] its length.
__global__ __launch_bounds__(1024) void k_greedy_rounds(const int32_t *__restrict__ rowptr,
                                                        const int32_t *__restrict__ nbr,
                                                        const int32_t *__restrict__ T0, int32_t D, int ntr,
                                                        int32_t cap, int32_t *__restrict__ new_tracer,
                                                        int32_t *__restrict__ res) {
  if (rowptr[D] > cap) {  // (uniform) more neighbours than the list holds: nothing decided
    if (threadIdx.x == 0) {
      res[3] = 2;
      res[4] = rowptr[D];
    }
    return;
  }
  __shared__ int8_t T[kMaxDrops];
  __shared__ int8_t dec[kMaxDrops];  // this round's decisions, -1 for none
  __shared__ uint32_t done[kMaxDrops / 32];
  __shared__ int s_changed, s_moved, s_new;
  const int tid = threadIdx.x;
  for (int32_t g = tid; g < D; g += 1024) {
    T[g] = (int8_t)T0[g];
    dec[g] = -1;
  }
  for (int32_t i = tid; i < kMaxDrops / 32; i += 1024) done[i] = 0u;
  if (tid == 0) {
    s_moved = 0;
    s_new = 0;
  }
  const uint64_t inuse = (ntr < 64) ? ((1ull << ntr) - 1) : ~0ull;
  while (true) {
    __syncthreads();
    if (tid == 0) s_changed = 0;
    __syncthreads();
    for (int32_t g = tid; g < D; g += 1024) {
      if ((done[g >> 5] >> (g & 31)) & 1u) continue;
      const int tg = T[g];
      bool ready = true, conflict = false;
      uint64_t used = 0;
      for (int32_t e = rowptr[g]; e < rowptr[g + 1]; ++e) {
        const int32_t h = nbr[e];
        if (h < g && !((done[h >> 5] >> (h & 31)) & 1u)) {
          ready = false;
          break;
        }
        const int th = T[h];
        conflict = conflict || (h < g && th == tg);
        used |= 1ull << th;
      }
      if (!ready) continue;
      int n = tg;
      if (conflict) {
        const uint64_t avail = ~used & ~(1ull << tg) & inuse;
        if (avail) n = __ffsll((unsigned long long)avail) - 1;
        else s_new = 1;
        atomicAdd(&s_moved, 1);
      }
      dec[g] = (int8_t)n;
      s_changed = 1;
    }
    __syncthreads();
    if (!s_changed || s_new) break;  // uniform: read after the barrier
    for (int32_t g = tid; g < D; g += 1024)
      if (dec[g] >= 0) {
        T[g] = dec[g];
        dec[g] = -1;
        atomicOr(&done[g >> 5], 1u << (g & 31));
      }
  }
  for (int32_t g = tid; g < D; g += 1024) new_tracer[g] = T[g];
  if (tid == 0) {
    res[0] = ntr;
    res[1] = s_moved;
    res[2] = 0;
    res[3] = s_new;
  }
}

__global__ void k_initial_tracers(int32_t *T0, int32_t D, int ntr, TracerOffsets to) {
  const int32_t g = blockIdx.x * blockDim.x + threadIdx.x;
  if (g >= D) return;
  int t = 0;
  while (t + 1 < ntr && to.off[t + 1] <= g) ++t;
  T0[g] = t;
}

// Move the cells of every moved drop: first clear every moved-out value of
// the cell, then add each to its new field.
// Moves the cells of every drop whose tracer changes: the old field is
// cleared first, then the values are added to the new fields. A cell owned by
// one drop (own >= 0, tracer T0[own]) needs only the owner array; cells
// shared by several drops read every tracer's labels.
__global__ __launch_bounds__(kBlock) void k_move(double *__restrict__ c, const int32_t *__restrict__ lab, int64_t n3,
                                                 int ntr, TracerOffsets to, const owner_t *__restrict__ own,
                                                 const int32_t *__restrict__ T0, const int32_t *__restrict__ newt) {
  const int64_t p = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (p >= n3) return;
  const int32_t o = own[p];
  if (o == -1) return;
  if (o >= 0) {
    const int t = T0[o], n = newt[o];
    if (n == t) return;
    double *src = c + (int64_t)t * n3 + p, *dst = c + (int64_t)n * n3 + p;
    const double v = *src;
    *src = 0.0;
    *dst = *dst + v;
    return;
  }
  int cnt = 0;
  for (int t = 0; t < ntr; ++t) {
    const int32_t l = lab[(int64_t)t * n3 + p];
    if (l > 0 && to.off[t] + l <= to.off[t + 1] && newt[to.off[t] + l - 1] != t) ++cnt;
  }
  if (cnt == 0) return;
  double vals[kMaxTracers];
  int dst[kMaxTracers];
  int k = 0;
  for (int t = 0; t < ntr; ++t) {
    const int32_t l = lab[(int64_t)t * n3 + p];
    if (l <= 0 || to.off[t] + l > to.off[t + 1]) continue;
    const int n = newt[to.off[t] + l - 1];
    if (n == t) continue;
    vals[k] = c[(int64_t)t * n3 + p];
    dst[k] = n;
    c[(int64_t)t * n3 + p] = 0.0;
    ++k;
  }
  for (int u = 0; u < k; ++u) {
    double *q = c + (int64_t)dst[u] * n3 + p;
    *q = *q + vals[u];
  }
}

// Sum of the retired tracers' fields for the compaction: workgroup b sums
// cells [b*chunk, (b+1)*chunk) of the concatenation of the retired fields
// (strided per thread, then a fixed tree); k_sum_parts adds the parts in
// order. Reproducible bit for bit.
constexpr int kSumBlock = 256;
__global__ __launch_bounds__(kSumBlock) void k_sum_retired(const double *__restrict__ c, const int32_t *__restrict__ which,
                                                          int nret, int64_t n3, int64_t chunk,
                                                          double *__restrict__ part) {
  const int64_t total = (int64_t)nret * n3;
  const int64_t q0 = (int64_t)blockIdx.x * chunk;
  const int64_t q1 = q0 + chunk < total ? q0 + chunk : total;
  double acc = 0.0;
  int64_t r = (q0 + threadIdx.x) / n3, rend = (r + 1) * n3;  // field of q, and where it ends
  for (int64_t q = q0 + threadIdx.x; q < q1; q += kSumBlock) {
    while (q >= rend) {  // (a field holds at least one cell: n3 >= 1)
      ++r;
      rend += n3;
    }
    acc += c[(int64_t)which[r] * n3 + (q - (rend - n3))];
  }
  __shared__ double red[kSumBlock];
  red[threadIdx.x] = acc;
  __syncthreads();
  for (int w = kSumBlock / 2; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) part[blockIdx.x] = red[0];
}
__global__ void k_sum_parts(const double *__restrict__ part, int n, double *__restrict__ out) {
  if (threadIdx.x != 0 || blockIdx.x != 0) return;
  double s = 0.0;
  for (int i = 0; i < n; ++i) s += part[i];
  *out = s;
}

}  // namespace

// Both recolouring modes: stencil == 0 relates drops within the distance
// threshold gap_cells, stencil != 0 by the literal 5x5x5 criterion (gap_cells
// unused). `fn` names the entry point in error messages.
static int recolor_impl(vofmt_ctx *ctx, const char *fn, int stencil, int32_t nx, int32_t ny, int32_t nz,
                        int32_t *ntracers_host, int32_t max_tracers, double *c, const int32_t *labels,
                        const int32_t *ndrops_host, double gap_cells, int32_t *new_tracer, int32_t *nmoved_host,
                        hipStream_t stream) {
  if (!ctx) return VOFMT_E_ARG;
  if (!ntracers_host || !nmoved_host || !ndrops_host) return set_err(ctx, VOFMT_E_ARG, "%s: null host pointer", fn);
  const int ntr = *ntracers_host;
  if (nx < 1 || ny < 1 || nz < 1 || ntr < 0 || ntr > max_tracers || max_tracers > kMaxTracers ||
      (!stencil && (!(gap_cells >= 0.0) || gap_cells > 64.0)))
    return set_err(ctx, VOFMT_E_ARG, "%s: bad arguments (ntracers=%d max_tracers=%d (<= %d) gap=%g)", fn, ntr,
                   max_tracers, kMaxTracers, gap_cells);
  *nmoved_host = 0;
  if (ntr == 0) return VOFMT_OK;
  if (!c || !labels) return set_err(ctx, VOFMT_E_ARG, "%s: null pointer", fn);
  TracerOffsets to;
  to.off[0] = 0;
  int64_t D = 0;
  for (int t = 0; t < ntr; ++t) {
    if (ndrops_host[t] < 0) return set_err(ctx, VOFMT_E_ARG, "%s: negative drop count", fn);
    D += ndrops_host[t];
    to.off[t + 1] = (int32_t)D;
  }
  for (int t = ntr + 1; t <= kMaxTracers; ++t) to.off[t] = (int32_t)D;
  if (D == 0) return VOFMT_OK;
  if (D > kMaxDrops) return set_err(ctx, VOFMT_E_ARG, "%s: more than %d drops", fn, kMaxDrops);
  if (!new_tracer) return set_err(ctx, VOFMT_E_ARG, "%s: null new_tracer", fn);
  const int64_t n3 = (int64_t)nx * ny * nz;
  if (n3 >= INT32_MAX) return set_err(ctx, VOFMT_E_ARG, "%s: more than 2^31-1 cells per field", fn);
  VOFMT_HIP(ctx, hipSetDevice(ctx->device));
  // Offsets scanned from the listed cells, one of each opposite pair (o > 0
  // in (z, y, x) order): a pair of drops is found from one side only, and
  // set_edge records it in both directions.
  // - distance mode: the half ball |o|^2 < (1+gap)^2. Every pair is still
  //   found: the two cells of the pair at the smallest offset are both listed
  //   (a cell whose six neighbours all held its drop would have a neighbour
  //   closer to the other drop), so the listed cell from which that offset
  //   points forward finds it;
  // - stencil mode (contacts across tracers): the half cube max|o_a| <= 4.
  //   A pair of cells at the smallest (max|o_a|, sum|o_a|) is listed on both
  //   sides: an axis step from an interior cell towards the other drop
  //   lowers the sum and does not raise the maximum.
  const int R = stencil ? 4 : (int)floor(1.0 + gap_cells);
  const double lim = stencil ? 1e300 : (1.0 + gap_cells) * (1.0 + gap_cells);
  std::vector<int4> hoffs;
  for (int oz = -R; oz <= R; ++oz)
    for (int oy = -R; oy <= R; ++oy)
      for (int ox = -R; ox <= R; ++ox) {
        const double o2 = (double)(ox * ox + oy * oy + oz * oz);
        if (o2 == 0.0 || !(o2 < lim)) continue;
        if (!(oz > 0 || (oz == 0 && (oy > 0 || (oy == 0 && ox > 0))))) continue;
        hoffs.push_back(make_int4(ox, oy, oz, 0));
      }
  const int noffs = (int)hoffs.size();
  // Tiles in LDS up to the reach that fits them (kMaxTileReach), where every
  // axis is longer than the tile's halo (an owner then wraps at most once);
  // the ordered list of boundary cells for the rest.
  const int Rt = R <= 2 ? 2 : kMaxTileReach;
  const bool tiled = R <= kMaxTileReach && kHaloX < nx && Rt < ny && Rt < nz;
  const int64_t words = (D + 31) / 32;
  owner_t *own = (owner_t *)scratch(ctx, SLOT_LABEL_B, sizeof(owner_t) * (size_t)n3);
  // the bitmap, then the number of listed row segments (stencil mode)
  uint32_t *adj = (uint32_t *)scratch(ctx, SLOT_LABEL_A, sizeof(uint32_t) * (size_t)(D * words + 1));
  uint32_t *nsegs = adj + D * words;
  int32_t *small = (int32_t *)scratch(ctx, SLOT_LABEL_C, sizeof(int32_t) * (size_t)(4 * D + 16));
  int32_t *hres = (int32_t *)host_scratch(ctx, 256 + sizeof(int4) * (size_t)noffs);
  if (!own || !adj || !small || !hres) return VOFMT_E_NOMEM;
  int32_t *deg = small, *rowptr = small + D, *T0 = small + 2 * D + 1;
  int32_t *nbr = nullptr;
  int cus = 0;
  if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, ctx->device) != hipSuccess || cus < 1)
    cus = 256;
  const unsigned nbc = ceil_div(n3, kBlock);
  hipLaunchKernelGGL(k_fill_u32, dim3(1024), dim3(256), 0, stream, adj, D * words + 1, 0u);
  // initial tracer of every drop (the stencil mode's cross-tracer filter reads it)
  hipLaunchKernelGGL(k_initial_tracers, dim3(ceil_div(D, 256)), dim3(256), 0, stream, T0, (int32_t)D, ntr, to);
  if (stencil) {
    // owners and occupancy bits per row segment, then Steps 1-3 within every tracer on the bits
    const int xw = (int)ceil_div(nx, 64);
    const int64_t rows = (int64_t)nz * ny;
    const int64_t nseg1 = rows * xw, nseg = ntr * nseg1;
    if ((nseg * 64 + kBlock - 1) / kBlock > INT32_MAX || nseg >= INT32_MAX)
      return set_err(ctx, VOFMT_E_ARG, "%s: grid too large", fn);
    uint64_t *occ = (uint64_t *)scratch(ctx, SLOT_OCC, sizeof(uint64_t) * (size_t)nseg);
    int32_t *seglist = (int32_t *)scratch(ctx, SLOT_OCC_LIST, sizeof(int32_t) * (size_t)nseg);
    if (!occ || !seglist) return VOFMT_E_NOMEM;
    const FastDiv fw = make_fastdiv((uint32_t)xw), frows = make_fastdiv((uint32_t)rows),
                  fny = make_fastdiv((uint32_t)ny);
    const unsigned nblk = ceil_div(nseg1, kBlock / 64);
    if (nx % 256 == 0 && ((uintptr_t)labels & 15) == 0)
      hipLaunchKernelGGL(k_owner_occ4, dim3(ceil_div(nseg1 / 4, kBlock / 64)), dim3(kBlock), 0, stream,
                         (const int4 *)labels, nseg1 / 4, ntr, to, (short4 *)own, occ);
    else
      hipLaunchKernelGGL(k_owner_occ, dim3(nblk), dim3(kBlock), 0, stream, labels, nx, nseg1, n3, xw, fw, ntr, to,
                         own, occ);
    const unsigned nblk_s = ceil_div(nseg, kBlock);
    if (nx >= 3 && nx % 64 != 1)
      hipLaunchKernelGGL((k_stencil_segments<true>), dim3(nblk_s), dim3(kBlock), 0, stream, occ, nx, ny, nz, xw, nseg,
                         fw, frows, fny, seglist, nsegs);
    else
      hipLaunchKernelGGL((k_stencil_segments<false>), dim3(nblk_s), dim3(kBlock), 0, stream, occ, nx, ny, nz, xw,
                         nseg, fw, frows, fny, seglist, nsegs);
    hipLaunchKernelGGL(k_stencil_edges, dim3(8 * cus), dim3(kBlock), 0, stream, labels, occ, nx, ny, nz, xw, to,
                       make_stencil_pairs(), adj, words, fw, frows, fny, seglist, nsegs);
  } else if (n3 % 4 == 0 && ((uintptr_t)labels & 15) == 0) {
    hipLaunchKernelGGL(k_owner4, dim3(ceil_div(n3 / 4, kBlock)), dim3(kBlock), 0, stream, (const int4 *)labels,
                       n3 / 4, ntr, to, (short4 *)own);
  } else {
    hipLaunchKernelGGL(k_owner, dim3(nbc), dim3(kBlock), 0, stream, labels, n3, ntr, to, own);
  }
  if (tiled) {
    const int LX = TileDims<2>::LX, LY = kTileY + 2 * Rt;
    TileRows lo{};  // hoffs is in (z, y, x) order: a row's offsets are consecutive
    for (const int4 &o : hoffs) {
      const int16_t base = (int16_t)((o.z * LY + o.y) * LX);
      if (lo.n == 0 || lo.base[lo.n - 1] != base) {
        lo.base[lo.n] = base;
        lo.first[lo.n] = (int16_t)lo.all;
        lo.lo[lo.n++] = (int8_t)o.x;
      }
      ++lo.all;
      lo.hi[lo.n - 1] = (int8_t)o.x;
    }
    const int tx = (int)ceil_div(nx, kTileX), ty = (int)ceil_div(ny, kTileY);
    const int64_t tiles = (int64_t)tx * ty * ceil_div(nz, kTileZ);
    int split = 1;
    while (split < kTileY * kTileZ / (4 * (kBlock / 64)) && 2 * split * tiles <= kSplitTiles) split *= 2;
    const int32_t *cross = stencil ? (const int32_t *)T0 : nullptr;
    if (Rt == 2)
      hipLaunchKernelGGL((k_tile_edges<2>), dim3((unsigned)(tiles * split)), dim3(kBlock), 0, stream, own, labels, nx,
                         ny, nz, ntr, to, lo, tx, ty, split, adj, words, cross);
    else
      hipLaunchKernelGGL((k_tile_edges<kMaxTileReach>), dim3((unsigned)(tiles * split)), dim3(kBlock), 0, stream, own,
                         labels, nx, ny, nz, ntr, to, lo, tx, ty, split, adj, words, cross);
  } else {
    // the cells that can see a pair, in order, then the pairs they see
    const int64_t lt = compact::list_tiles_if(n3);
    int4 *doffs = (int4 *)scratch(ctx, SLOT_MISC2, sizeof(int4) * (size_t)(noffs > 0 ? noffs : 1));
    int32_t *srcs = (int32_t *)scratch(ctx, SLOT_RECOLOR_LIST, sizeof(int32_t) * (size_t)n3);
    int32_t *bc = (int32_t *)scratch(ctx, SLOT_MISC, sizeof(int32_t) * (size_t)nbc);
    int32_t *tot = (int32_t *)scratch(ctx, SLOT_CURV_COUNT, sizeof(int32_t) * (size_t)(lt + 2));
    uint64_t *pbits = (uint64_t *)scratch(ctx, SLOT_CURV_HF, sizeof(uint64_t) * (size_t)((n3 + 63) / 64));
    if (!doffs || !srcs || !bc || !tot || !pbits) return VOFMT_E_NOMEM;
    // pinned staging: results in the first 256 bytes, offsets after them
    if (noffs > 0) {
      memcpy(hres + 64, hoffs.data(), sizeof(int4) * noffs);
      VOFMT_HIP(ctx, hipMemcpyAsync(doffs, hres + 64, sizeof(int4) * noffs, hipMemcpyHostToDevice, stream));
    }
    const int small_offsets = (R < nx && R < ny && R < nz) ? 1 : 0;
    // the ordered list of those cells: counts and bits, the tiled scan, the list from the bits
    const int64_t nb = (n3 + kBlock - 1) / kBlock, nt = (nb + compact::kTile - 1) / compact::kTile;
    static_assert(kBlock == compact::kBlock, "block counts and the tiled scan share the block size");
    hipLaunchKernelGGL(k_pair_source_counts, dim3((unsigned)nb), dim3(kBlock), 0, stream, own, nx, ny, nz,
                       make_fastdiv((uint32_t)nx), make_fastdiv((uint32_t)ny), n3, bc, pbits);
    hipLaunchKernelGGL(compact::k_scan_tile, dim3((unsigned)nt), dim3(compact::kTile), 0, stream, bc, nb, tot,
                       (int64_t)0, (int64_t)0);
    hipLaunchKernelGGL(compact::k_scan_totals, dim3(1), dim3(compact::kTile), 0, stream, tot, nt, (int64_t)0);
    hipLaunchKernelGGL(compact::k_write_ordered_bits, dim3((unsigned)((nb + kBlock / 64 - 1) / (kBlock / 64))),
                       dim3(kBlock), 0, stream, n3, pbits, bc, tot, srcs);
    hipLaunchKernelGGL(k_edges, dim3(8 * cus), dim3(kBlock), 0, stream, own, labels, nx, ny, nz, ntr, to, doffs,
                       noffs, small_offsets, srcs, tot + lt, adj, words, make_fastdiv((uint32_t)nx),
                       make_fastdiv((uint32_t)ny), stencil ? (const int32_t *)T0 : nullptr);
  }
  hipLaunchKernelGGL(k_degree, dim3(ceil_div(D, kBlock / 64)), dim3(kBlock), 0, stream, adj, (int32_t)D, words, deg);
  hipLaunchKernelGGL(k_scan_deg, dim3(1), dim3(1024), 0, stream, deg, (int32_t)D, rowptr);
  // The neighbour list has room for 32 per drop, or what an earlier call needed;
  // the kernels check, and a longer list is filled again. Results go to pinned
  // memory.
  int32_t cap = (int32_t)std::min<int64_t>(INT32_MAX, std::max<int64_t>(32 * D, (int64_t)(ctx->cap[SLOT_MISC3] / sizeof(int32_t))));
  while (true) {
    nbr = (int32_t *)scratch(ctx, SLOT_MISC3, sizeof(int32_t) * (size_t)cap);
    if (!nbr) return VOFMT_E_NOMEM;
    hipLaunchKernelGGL(k_csr_fill, dim3(ceil_div(D, kBlock / 64)), dim3(kBlock), 0, stream, adj, (int32_t)D, words,
                       rowptr, cap, nbr);
    hipLaunchKernelGGL(k_greedy_rounds, dim3(1), dim3(1024), 0, stream, rowptr, nbr, T0, (int32_t)D, ntr, cap,
                       new_tracer, hres);
    VOFMT_HIP(ctx, hipGetLastError());
    VOFMT_HIP(ctx, hipStreamSynchronize(stream));
    if (hres[3] != 2) break;
    cap = hres[4];
  }
  if (hres[3]) {  // a drop needs a new tracer: the sequential pass
    hipLaunchKernelGGL(k_greedy, dim3(1), dim3(64), 0, stream, rowptr, nbr, T0, (int32_t)D, ntr, max_tracers,
                       new_tracer, hres);
    VOFMT_HIP(ctx, hipGetLastError());
    VOFMT_HIP(ctx, hipStreamSynchronize(stream));
  }
  const int Nnew = hres[0], moved = hres[1], overflow = hres[2];
  if (overflow) return set_err(ctx, VOFMT_E_CAPACITY, "%s: more than max_tracers=%d tracers needed", fn, max_tracers);
  if (moved > 0) {
    if (Nnew > ntr)
      hipLaunchKernelGGL(k_fill_f64, dim3(1024), dim3(256), 0, stream, c + (int64_t)ntr * n3,
                         (int64_t)(Nnew - ntr) * n3, 0.0);
    hipLaunchKernelGGL(k_move, dim3(nbc), dim3(kBlock), 0, stream, c, labels, n3, ntr, to, own, T0, new_tracer);
    VOFMT_HIP(ctx, hipGetLastError());
  }
  *ntracers_host = Nnew;
  *nmoved_host = moved;
  return VOFMT_OK;
}

extern "C" int vofmt_recolor_tracers(vofmt_ctx *ctx, int32_t nx, int32_t ny, int32_t nz, int32_t *ntracers_host,
                                     int32_t max_tracers, double *c, const int32_t *labels, const int32_t *ndrops_host,
                                     double gap_cells, int32_t *new_tracer, int32_t *nmoved_host, hipStream_t stream) {
  return recolor_impl(ctx, "vofmt_recolor_tracers", 0, nx, ny, nz, ntracers_host, max_tracers, c, labels,
                      ndrops_host, gap_cells, new_tracer, nmoved_host, stream);
}

extern "C" int vofmt_recolor_tracers_stencil(vofmt_ctx *ctx, int32_t nx, int32_t ny, int32_t nz,
                                             int32_t *ntracers_host, int32_t max_tracers, double *c,
                                             const int32_t *labels, const int32_t *ndrops_host, int32_t *new_tracer,
                                             int32_t *nmoved_host, hipStream_t stream) {
  return recolor_impl(ctx, "vofmt_recolor_tracers_stencil", 1, nx, ny, nz, ntracers_host, max_tracers, c, labels,
                      ndrops_host, 0.0, new_tracer, nmoved_host, stream);
}

extern "C" int vofmt_compact_tracers(vofmt_ctx *ctx, int32_t nx, int32_t ny, int32_t nz, int32_t *ntracers_host,
                                     double *c, const int32_t *ndrops_host, int32_t *new_index_host,
                                     double *discarded_host, hipStream_t stream) {
  if (!ctx) return VOFMT_E_ARG;
  if (nx < 1 || ny < 1 || nz < 1 || !ntracers_host || *ntracers_host < 0)
    return set_err(ctx, VOFMT_E_ARG, "vofmt_compact_tracers: bad sizes");
  const int ntr = *ntracers_host;
  if (ntr > 0 && (!c || !ndrops_host || !new_index_host || !discarded_host))
    return set_err(ctx, VOFMT_E_ARG, "vofmt_compact_tracers: null pointer");
  if (discarded_host) *discarded_host = 0.0;
  if (ntr == 0) return VOFMT_OK;
  const int64_t n3 = (int64_t)nx * ny * nz;
  std::vector<int32_t> retired;
  int k = 0;
  for (int t = 0; t < ntr; ++t) {
    if (ndrops_host[t] < 0) return set_err(ctx, VOFMT_E_ARG, "vofmt_compact_tracers: negative drop count");
    if (ndrops_host[t] > 0) new_index_host[t] = k++;
    else {
      new_index_host[t] = -1;
      retired.push_back(t);
    }
  }
  if (retired.empty()) return VOFMT_OK;
  VOFMT_HIP(ctx, hipSetDevice(ctx->device));
  // the discarded volume, before any field moves
  const int nret = (int)retired.size();
  const int64_t total = (int64_t)nret * n3;
  const int64_t chunk = (int64_t)kSumBlock * 64;
  const int64_t nparts = (total + chunk - 1) / chunk;
  if (nparts > INT32_MAX) return set_err(ctx, VOFMT_E_ARG, "vofmt_compact_tracers: fields too large");
  int32_t *which = (int32_t *)scratch(ctx, SLOT_MISC, sizeof(int32_t) * (size_t)nret);
  double *part = (double *)scratch(ctx, SLOT_MISC2, sizeof(double) * ((size_t)nparts + 1));
  double *hres = (double *)host_scratch(ctx, sizeof(double));
  if (!which || !part || !hres) return VOFMT_E_NOMEM;
  VOFMT_HIP(ctx, hipMemcpyAsync(which, retired.data(), sizeof(int32_t) * (size_t)nret, hipMemcpyHostToDevice,
                                stream));
  hipLaunchKernelGGL(k_sum_retired, dim3((unsigned)nparts), dim3(kSumBlock), 0, stream, c, which, nret, n3, chunk,
                     part);
  hipLaunchKernelGGL(k_sum_parts, dim3(1), dim3(64), 0, stream, part, (int)nparts, part + nparts);
  VOFMT_HIP(ctx, hipGetLastError());
  VOFMT_HIP(ctx, hipMemcpyAsync(hres, part + nparts, sizeof(double), hipMemcpyDeviceToHost, stream));
  // kept fields move down in increasing order (each to a slot already read or retired)
  for (int t = 0; t < ntr; ++t) {
    const int d = new_index_host[t];
    if (d >= 0 && d != t)
      VOFMT_HIP(ctx, hipMemcpyAsync(c + (int64_t)d * n3, c + (int64_t)t * n3, sizeof(double) * (size_t)n3,
                                    hipMemcpyDeviceToDevice, stream));
  }
  hipLaunchKernelGGL(k_fill_f64, dim3(1024), dim3(256), 0, stream, c + (int64_t)k * n3, (int64_t)(ntr - k) * n3,
                     0.0);
  VOFMT_HIP(ctx, hipGetLastError());
  VOFMT_HIP(ctx, hipStreamSynchronize(stream));
  *discarded_host = *hres;
  *ntracers_host = k;
  return VOFMT_OK;
}
