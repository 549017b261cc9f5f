// Lists of the interface (mixed) cells of one field in increasing cell order:
// block counts (with one bit per cell), a tiled scan, then a second pass that
// writes the list from the bits. No
// atomics, so the order is fixed. A cell is an interface cell when its value
// lies more than 1e-12 inside (0, 1); round-off residues of pure cells are not.
#pragma once

#include "common.hpp"

namespace compact {
namespace {  // each translation unit gets its own kernels

constexpr int kBlock = 256;
constexpr int kTile = 1024;  // entries per scan tile

constexpr double kResidue = 1e-12;
__device__ __forceinline__ bool is_mixed(double v) { return v > kResidue && v < 1.0 - kResidue; }

// The mixed-cell list takes blocks of kCells cells, a wavefront kWave
// consecutive ones of them as kListWords 64-cell words: few, long-lived
// workgroups (blocks of 2048 cells: the counting pass 231 us over a 512^3 field,
// 193 us so).
constexpr int kListWords = 32;
constexpr int kWave = 64 * kListWords;
constexpr int64_t kCells = (int64_t)kWave * (kBlock / 64);

// Mixed cells per block of kCells cells, and the mixed-cell bits: word
// p / 64 of `bits` for cells p .. p + 63.
__global__ __launch_bounds__(kBlock) void k_block_counts(const double *__restrict__ c, int64_t n3,
                                                         int32_t *__restrict__ bc, uint64_t *__restrict__ bits) {
  constexpr int kInFlight = 16;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int64_t pw = blockIdx.x * kCells + (int64_t)w * kWave;  // the wavefront's first cell
  uint32_t lo = 0, hi = 0;                                      // lane j: word j
  int n = 0;                                                    // wavefront-uniform
#pragma unroll
  for (int j0 = 0; j0 < kListWords; j0 += kInFlight) {
    double v[kInFlight];
#pragma unroll
    for (int j = 0; j < kInFlight; ++j) {
      const int64_t p = pw + 64 * (j0 + j) + lane;
      v[j] = p < n3 ? c[p] : 0.0;  // (0: not mixed)
    }
#pragma unroll
    for (int j = 0; j < kInFlight; ++j) {
      const uint64_t mk = __ballot(is_mixed(v[j]));
      n += (int)__popcll(mk);
      if (lane == j0 + j) {
        lo = (uint32_t)mk;
        hi = (uint32_t)(mk >> 32);
      }
    }
  }
  if (lane < kListWords && pw + 64 * lane < n3) bits[(pw >> 6) + lane] = ((uint64_t)hi << 32) | lo;
  __shared__ int wc[kBlock / 64];
  if (lane == 0) wc[w] = n;
  __syncthreads();
  if (threadIdx.x == 0) {
    int t = 0;
    for (int k = 0; k < kBlock / 64; ++k) t += wc[k];
    bc[blockIdx.x] = t;
  }
}

// Exclusive scan of one tile of kTile entries in place; the tile total goes to tot[tile].
// Batches of arrays along blockIdx.y: array b starts at v + b * vstride, its totals at
// tot + b * tstride.
__global__ __launch_bounds__(kTile) void k_scan_tile(int32_t *__restrict__ v, int64_t n, int32_t *__restrict__ tot,
                                                     int64_t vstride, int64_t tstride) {
  v += blockIdx.y * vstride;
  tot += blockIdx.y * tstride;
  __shared__ int32_t s[kTile];
  const int64_t i = (int64_t)blockIdx.x * kTile + threadIdx.x;
  const int32_t x = (i < n) ? v[i] : 0;
  s[threadIdx.x] = x;
  __syncthreads();
  for (int off = 1; off < kTile; off <<= 1) {
    const int32_t add = (threadIdx.x >= (unsigned)off) ? s[threadIdx.x - off] : 0;
    __syncthreads();
    s[threadIdx.x] += add;
    __syncthreads();
  }
  if (i < n) v[i] = s[threadIdx.x] - x;
  if (threadIdx.x == kTile - 1) tot[blockIdx.x] = s[kTile - 1];
}

// Exclusive scan of the tile totals (one workgroup, any length); the grand
// total goes to tot[ntiles]. Batches along blockIdx.y as in k_scan_tile.
__global__ __launch_bounds__(kTile) void k_scan_totals(int32_t *__restrict__ tot, int64_t ntiles, int64_t tstride) {
  tot += blockIdx.y * tstride;
  __shared__ int32_t s[kTile];
  __shared__ int32_t carry;
  if (threadIdx.x == 0) carry = 0;
  __syncthreads();
  for (int64_t base = 0; base < ntiles; base += kTile) {
    const int64_t i = base + threadIdx.x;
    const int32_t x = (i < ntiles) ? tot[i] : 0;
    s[threadIdx.x] = x;
    __syncthreads();
    for (int off = 1; off < kTile; off <<= 1) {
      const int32_t add = (threadIdx.x >= (unsigned)off) ? s[threadIdx.x - off] : 0;
      __syncthreads();
      s[threadIdx.x] += add;
      __syncthreads();
    }
    if (i < ntiles) tot[i] = carry + s[threadIdx.x] - x;
    __syncthreads();
    if (threadIdx.x == 0) carry += s[kTile - 1];
    __syncthreads();
  }
  if (threadIdx.x == 0) tot[ntiles] = carry;
}

// Ordered list: block b writes its mixed cells from the bits of the counting
// pass (the field is not read again), after the entries of the blocks before
// it: bc[b] plus the totals of the tiles before its own, or (SCANNED false) the
// sum of the counts before bc[b]. The last block stores the list's length in
// *length. With
// kappa/status given, every cell first gets NaN / 0 (the listed cells are
// written later, by the list's readers): 16 bytes a lane and not kept in the
// caches (272 us with a store of 8 and one of 1 byte a lane over a 512^3 field,
// 238 us so).
template <bool SCANNED>
__global__ __launch_bounds__(kBlock) void k_write_ordered(const uint64_t *__restrict__ bits, int64_t n3,
                                                          const int32_t *__restrict__ bc,
                                                          const int32_t *__restrict__ tot,
                                                          int32_t *__restrict__ length, int32_t *__restrict__ list,
                                                          double *__restrict__ kappa, uint8_t *__restrict__ status) {
  typedef double double2u __attribute__((ext_vector_type(2), aligned(8)));
  typedef uint32_t uint4u __attribute__((ext_vector_type(4), aligned(1)));
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int64_t pw = blockIdx.x * kCells + (int64_t)w * kWave;
  uint64_t word = (lane < kListWords && pw + 64 * lane < n3) ? bits[(pw >> 6) + lane] : 0ull;
  if (kappa) {
    const double nan = __builtin_nan("");
    if (pw + kWave <= n3) {
#pragma unroll
      for (int j = 0; j < kWave / 128; ++j)
        __builtin_nontemporal_store((double2u){nan, nan}, (double2u *)(kappa + pw + 128 * j + 2 * lane));
#pragma unroll
      for (int j = 0; j < kWave / 1024; ++j)
        __builtin_nontemporal_store((uint4u){0u, 0u, 0u, 0u}, (uint4u *)(status + pw + 1024 * j + 16 * lane));
    } else {
      for (int64_t p = pw + lane; p < n3; p += 64) {
        kappa[p] = nan;
        status[p] = 0;
      }
    }
  }
  // entries of the words before this lane's, of the wavefronts and of the tiles before
  const int mine = (int)__popcll(word);
  int upto = mine;
#pragma unroll
  for (int k = 1; k < 64; k <<= 1) {
    const int below = __shfl_up(upto, k, 64);
    if (lane >= k) upto += below;
  }
  __shared__ int wc[kBlock / 64], before[kBlock / 64];
  if (lane == 63) wc[w] = upto;
  const int32_t *v = SCANNED ? tot : bc;
  int part = 0;
  for (int64_t k = threadIdx.x; k < (SCANNED ? blockIdx.x / kTile : blockIdx.x); k += kBlock) part += v[k];
#pragma unroll
  for (int k = 32; k > 0; k >>= 1) part += __shfl_xor(part, k, 64);
  if (lane == 0) before[w] = part;
  __syncthreads();
  int run = SCANNED ? bc[blockIdx.x] : 0;
  for (int k = 0; k < kBlock / 64; ++k) run += before[k] + (k < w ? wc[k] : 0);
  if (blockIdx.x == gridDim.x - 1 && w == kBlock / 64 - 1 && lane == 63) *length = run + upto;
  run += upto - mine;
  while (word) {
    list[run++] = (int32_t)(pw + 64 * lane) + (int32_t)__builtin_ctzll(word);
    word &= word - 1;
  }
}

// The ordered list of the mixed cells of c into `list` (capacity n3), its
// length into *length (device or pinned host memory). bc: ceil(n3 / kBlock) ints of
// scratch; tot: list_tiles(n3) ints; bits: ceil(n3 / 64) words of scratch.
inline void launch_ordered_list(const double *c, int64_t n3, int32_t *bc, int32_t *tot, int32_t *list, double *kappa,
                                uint8_t *status, uint64_t *bits, int32_t *length, hipStream_t stream) {
  const int64_t nb = (n3 + kCells - 1) / kCells;
  const int64_t ntiles = (nb + kTile - 1) / kTile;
  hipLaunchKernelGGL(k_block_counts, dim3((unsigned)nb), dim3(kBlock), 0, stream, c, n3, bc, bits);
  // up to kDirect blocks (33M cells) each sums the counts before its own: the
  // scan is one more launch of about 5 us (64^3: 41 -> 38 us for the call; 256^3 and
  // 318^3, 2048 and 3926 blocks: 141 -> 139 and 259 -> 257)
  constexpr int64_t kDirect = 4096;
  if (nb <= kDirect) {
    hipLaunchKernelGGL(k_write_ordered<false>, dim3((unsigned)nb), dim3(kBlock), 0, stream, bits, n3, bc, tot, length,
                       list, kappa, status);
    return;
  }
  hipLaunchKernelGGL(k_scan_tile, dim3((unsigned)ntiles), dim3(kTile), 0, stream, bc, nb, tot, (int64_t)0, (int64_t)0);
  hipLaunchKernelGGL(k_write_ordered<true>, dim3((unsigned)nb), dim3(kBlock), 0, stream, bits, n3, bc, tot, length,
                     list, kappa, status);
}

// Scan tiles of the mixed-cell list of n3 cells.
inline int64_t list_tiles(int64_t n3) { return ((n3 + kCells - 1) / kCells + kTile - 1) / kTile; }
// Scan tiles of a predicate list of n cells (one block count per kBlock cells).
inline int64_t list_tiles_if(int64_t n) { return ((n + kBlock - 1) / kBlock + kTile - 1) / kTile; }

// Ordered lists of the cells p < n of a predicate whose counting pass stores
// it as one bit per cell (one 64-bit word per wavefront of cells) and one
// count per kBlock cells: the writing pass reads the bits.
// One wavefront per block of kBlock cells (its kBlock / 64 words), four
// blocks per workgroup: word j's set bits are written in round j, after the
// block's offset and the bits of its earlier words.
__global__ __launch_bounds__(kBlock) void k_write_ordered_bits(int64_t n, const uint64_t *__restrict__ bits,
                                                               const int32_t *__restrict__ bc,
                                                               const int32_t *__restrict__ tot,
                                                               int32_t *__restrict__ list) {
  constexpr int kWords = kBlock / 64;
  const int lane = threadIdx.x & 63;
  const int64_t b = (int64_t)blockIdx.x * (kBlock / 64) + (threadIdx.x >> 6);  // this wavefront's block
  const int64_t nb = (n + kBlock - 1) / kBlock;
  if (b >= nb) return;  // whole wavefront
  const int64_t c0 = b * kBlock;
  uint64_t wm[kWords];
#pragma unroll
  for (int j = 0; j < kWords; ++j) wm[j] = (c0 + 64 * j < n) ? bits[(c0 >> 6) + j] : 0ull;
  int idx = bc[b] + tot[b / kTile];
  const uint64_t below = (1ull << lane) - 1;
#pragma unroll
  for (int j = 0; j < kWords; ++j) {
    if ((wm[j] >> lane) & 1ull) list[idx + (int)__popcll(wm[j] & below)] = (int32_t)(c0 + 64 * j + lane);
    idx += (int)__popcll(wm[j]);
  }
}

}  // namespace
}  // namespace compact
