// LBVH construction over Gaussians on gfx950 (Sec. IV-A: one leaf per Gaussian holding
// its world->unit-sphere transform; the baseline's 20-triangle proxy mesh per Gaussian).
//
// Pipeline, all on one stream, no host synchronisation:
//   bounds of the centroids (two-stage min/max, exact)
//   63-bit Morton codes (binary32 quantisation with fp contraction off, so the codes are
//     an exact integer function of the inputs)
//   stable LSD radix sort of the codes with their positions, 8 passes of 8 bits
//   leaf records and leaf boxes in sorted order, and the boxes of 2, 4, 8, ... leaves
//   radix tree over the sorted (code, position) keys (Karras 2012, one thread per node, which
//   also forms its box: exact min/max), with the subtrees of the next step and a subtree cut
//   kept for the trace's per-tile cost estimates
//   treelet restructuring by surface-area cost (5-leaf treelets, one workgroup per subtree
//     of at most 256 leaves; beyond a million leaves three passes over the subtrees and
//     one over the nodes above them), unless the plain radix tree is asked for
//   collapse to four-wide quantised node records, laid out in subtree blocks
#include <hip/hip_runtime.h>

#include <algorithm>
#include <map>
#include <mutex>
#include <cmath>
#include <type_traits>

#include "camera.h"
#include "grtx_internal.h"

namespace grtx {
namespace {

constexpr int kBlock = 256;

// ------------------------------------------------------------------ centroid bounds

// (It also clears what later kernels count in: the density grid and a few counters.)
__global__ void __launch_bounds__(kBlock) k_bounds_partial(const float* __restrict__ pts, int64_t n,
                                                           float* __restrict__ partial, uint4* __restrict__ grid,
                                                           uint32_t* __restrict__ counters, int n_counters) {
  for (int i = blockIdx.x * kBlock + threadIdx.x; i < kDensityCells / 4; i += gridDim.x * kBlock)
    grid[i] = make_uint4(0u, 0u, 0u, 0u);
  if (blockIdx.x == 0 && (int)threadIdx.x < n_counters) counters[threadIdx.x] = 0u;
  float lo[3] = {INFINITY, INFINITY, INFINITY}, hi[3] = {-INFINITY, -INFINITY, -INFINITY};
  for (int64_t i = blockIdx.x * (int64_t)kBlock + threadIdx.x; i < n; i += (int64_t)gridDim.x * kBlock) {
    for (int a = 0; a < 3; ++a) {
      float v = pts[3 * i + a];
      lo[a] = fminf(lo[a], v);
      hi[a] = fmaxf(hi[a], v);
    }
  }
  __shared__ float s[6][kBlock];
  for (int a = 0; a < 3; ++a) {
    s[a][threadIdx.x] = lo[a];
    s[3 + a][threadIdx.x] = hi[a];
  }
  __syncthreads();
  for (int w = kBlock / 2; w > 0; w >>= 1) {
    if (threadIdx.x < w)
      for (int a = 0; a < 3; ++a) {
        s[a][threadIdx.x] = fminf(s[a][threadIdx.x], s[a][threadIdx.x + w]);
        s[3 + a][threadIdx.x] = fmaxf(s[3 + a][threadIdx.x], s[3 + a][threadIdx.x + w]);
      }
    __syncthreads();
  }
  if (threadIdx.x < 6) partial[blockIdx.x * 6 + threadIdx.x] = s[threadIdx.x][0];
}

// The workgroups' bounds into one (out: lo xyz, hi xyz, for the whole workgroup).
__device__ __forceinline__ void final_bounds(const float* __restrict__ partial, int nparts, float (*s)[kBlock],
                                             float out[6]) {
  float v[6] = {INFINITY, INFINITY, INFINITY, -INFINITY, -INFINITY, -INFINITY};
  for (int i = threadIdx.x; i < nparts; i += kBlock)
    for (int a = 0; a < 3; ++a) {
      v[a] = fminf(v[a], partial[i * 6 + a]);
      v[3 + a] = fmaxf(v[3 + a], partial[i * 6 + 3 + a]);
    }
  // a wave by shuffles, then the waves' by everyone
#pragma unroll
  for (int w = 32; w > 0; w >>= 1)
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      v[a] = fminf(v[a], __shfl_xor(v[a], w));
      v[3 + a] = fmaxf(v[3 + a], __shfl_xor(v[3 + a], w));
    }
  if ((threadIdx.x & 63) == 0)
    for (int a = 0; a < 6; ++a) s[a][threadIdx.x >> 6] = v[a];
  __syncthreads();
  for (int a = 0; a < 6; ++a) {
    out[a] = s[a][0];
    for (int w = 1; w < kBlock / 64; ++w) out[a] = a < 3 ? fminf(out[a], s[a][w]) : fmaxf(out[a], s[a][w]);
  }
}

// ------------------------------------------------------------------ Morton codes

__device__ __forceinline__ uint64_t spread3(uint32_t v) {
  uint64_t x = v & 0x1FFFFFu;
  x = (x | (x << 32)) & 0x1F00000000FFFFull;
  x = (x | (x << 16)) & 0x1F0000FF0000FFull;
  x = (x | (x << 8)) & 0x100F00F00F00F00Full;
  x = (x | (x << 4)) & 0x10C30C30C30C30C3ull;
  x = (x | (x << 2)) & 0x1249249249249249ull;
  return x;
}

__device__ __forceinline__ uint32_t quantise(float v, float lo, float scale) {
#pragma clang fp contract(off)
  float rel = v - lo;
  float pos = rel * scale;
  float fl = floorf(pos);
  return fl <= 0.f ? 0u : (fl >= 2097151.f ? 2097151u : (uint32_t)fl);
}

// (Every workgroup forms the bounds from the partial ones, 256 of them or fewer, rather than
// wait for a launch that does it once; the first writes them for the kernels that follow.)
__global__ void __launch_bounds__(kBlock) k_morton(const float* __restrict__ pts, int64_t n,
                                                   const float* __restrict__ partial, int nparts,
                                                   float* __restrict__ bounds, float* __restrict__ dbox,
                                                   uint64_t* __restrict__ codes) {
#pragma clang fp contract(off)
  __shared__ float s[6][kBlock];
  float box[6];
  final_bounds(partial, nparts, s, box);
  if (blockIdx.x == 0 && threadIdx.x < 6) bounds[threadIdx.x] = dbox[threadIdx.x] = box[threadIdx.x];
  for (int64_t i = blockIdx.x * (int64_t)kBlock + threadIdx.x; i < n; i += (int64_t)gridDim.x * kBlock) {
    uint32_t q[3];
    for (int a = 0; a < 3; ++a) {
      float lo = box[a], hi = box[3 + a];
      float ext = hi - lo;
      float scale = ext > 0.f ? 2097152.f / ext : 0.f;  // correctly rounded division
      q[a] = quantise(pts[3 * i + a], lo, scale);
    }
    codes[i] = (spread3(q[0]) << 2) | (spread3(q[1]) << 1) | spread3(q[2]);
  }
}

// ------------------------------------------------------------------ radix sort (stable LSD)

// Keys per thread: 16 for large sorts; 4 up to kRadixSmall keys, so that a sort of a few
// hundred thousand keys still spreads over ~100 workgroups instead of ~25.
constexpr int kRadixItems = 16;
constexpr int kRadixItemsSmall = 4;
constexpr int64_t kRadixSmall = (int64_t)256 * kBlock * kRadixItemsSmall;
// Up to this many workgroups, each scatter workgroup derives its own offsets from the
// histogram table (a digit's counts over all workgroups), so no scan launch is needed.
constexpr int kRadixFusedBlocks = 256;

// A sort whose number of keys only the device knows gets a sixteenth of the workgroups that its
// bound would need (a ray lists far fewer hits than its list holds), within these limits; each
// takes as many consecutive tiles as the true number asks for. With a workgroup per tile of the
// bound, the table of counts itself (33 MB for 512x512 rays x 512 hits) took most of the time:
// 240 us a pass for 10.7M keys, 109 us now.
constexpr int kRadixDeviceBlocks = 1024;

// Tiles that each of `nblocks` workgroups takes.
__device__ __forceinline__ int64_t radix_tiles(int64_t n, int64_t tile, int nblocks) {
  return max((int64_t)1, (n + tile * nblocks - 1) / (tile * nblocks));
}

// `n_dev` (may be null) holds the number of keys on the device when the host knows only a
// bound `n` (workgroups past the count see no keys).
template <class K, int BITS>
__global__ void __launch_bounds__(kBlock) k_radix_hist(const K* __restrict__ keys, int64_t n, int shift, int items,
                                                       uint32_t* __restrict__ hist, int nblocks, bool fused,
                                                       const uint32_t* __restrict__ n_dev, uint32_t* __restrict__ rows,
                                                       int n_rows) {
  if (n_dev) n = min(n, (int64_t)*n_dev);
  constexpr int kBins = 1 << BITS;
  __shared__ uint32_t s_cnt[kBins];
  for (int d = threadIdx.x; d < kBins; d += kBlock) s_cnt[d] = 0;
  __syncthreads();
  const int64_t span = radix_tiles(n, (int64_t)kBlock * items, nblocks) * kBlock * items;
  const int64_t base = (int64_t)blockIdx.x * span;
  const int64_t end = min(n, base + span);
  for (int64_t i0 = base + threadIdx.x; i0 < end; i0 += kBlock * kRadixItems) {
    K key[kRadixItems];  // (all loads in flight together)
#pragma unroll
    for (int r = 0; r < kRadixItems; ++r) key[r] = i0 + r * kBlock < end ? keys[i0 + r * kBlock] : (K)0;
#pragma unroll
    for (int r = 0; r < kRadixItems; ++r)
      if (i0 + r * kBlock < end) atomicAdd(&s_cnt[(uint32_t)(key[r] >> shift) & (kBins - 1u)], 1u);
  }
  __syncthreads();
  // digit-major ([digit][workgroup]) for the scan; workgroup-major rows for the fused scatter
  // (and this workgroup's rows of the later passes cleared, which the scatters count in)
  for (int p = 0; p < n_rows; ++p)
    for (int d = threadIdx.x; d < kBins; d += kBlock) rows[((size_t)p * nblocks + blockIdx.x) * kBins + d] = 0u;
  for (int d = threadIdx.x; d < kBins; d += kBlock)
    hist[fused ? (size_t)blockIdx.x * kBins + d : (size_t)d * nblocks + blockIdx.x] = s_cnt[d];
}

// Exclusive scan of `n` uint32 in chunks of kScanChunk.
constexpr int kScanItems = 16;
constexpr int kScanChunk = kBlock * kScanItems;

__device__ uint32_t block_exclusive_scan(uint32_t v, uint32_t* s_tmp, uint32_t* total) {
  // A wave by shuffles, then the waves' sums (in s_tmp) by everyone: two barriers.
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  uint32_t incl = v;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const uint32_t x = __shfl_up(incl, off);
    incl += lane >= off ? x : 0u;
  }
  if (lane == 63) s_tmp[wave] = incl;
  __syncthreads();
  uint32_t before = 0, all = 0;
#pragma unroll
  for (int w = 0; w < kBlock / 64; ++w) {
    const uint32_t x = s_tmp[w];
    before += w < wave ? x : 0u;
    all += x;
  }
  *total = all;
  __syncthreads();
  return before + incl - v;
}

__global__ void __launch_bounds__(kBlock) k_scan_reduce(const uint32_t* __restrict__ in, int64_t n,
                                                        uint32_t* __restrict__ partial) {
  __shared__ uint32_t s[kBlock];
  int64_t base = (int64_t)blockIdx.x * kScanChunk + (int64_t)threadIdx.x * kScanItems;
  uint32_t acc = 0;
  for (int j = 0; j < kScanItems; ++j)
    if (base + j < n) acc += in[base + j];
  s[threadIdx.x] = acc;
  __syncthreads();
  for (int w = kBlock / 2; w > 0; w >>= 1) {
    if (threadIdx.x < w) s[threadIdx.x] += s[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) partial[blockIdx.x] = s[0];
}

// One block: exclusive scan of up to kScanChunk partials in place.
__global__ void __launch_bounds__(kBlock) k_scan_partials(uint32_t* __restrict__ partial, int n) {
  __shared__ uint32_t s[kBlock];
  uint32_t v[kScanItems];
  uint32_t acc = 0;
  for (int j = 0; j < kScanItems; ++j) {
    int i = threadIdx.x * kScanItems + j;
    v[j] = i < n ? partial[i] : 0u;
    acc += v[j];
  }
  uint32_t tot;
  uint32_t run = block_exclusive_scan(acc, s, &tot);
  for (int j = 0; j < kScanItems; ++j) {
    int i = threadIdx.x * kScanItems + j;
    if (i < n) partial[i] = run;
    run += v[j];
  }
}

__global__ void __launch_bounds__(kBlock) k_scan_down(const uint32_t* __restrict__ in, int64_t n,
                                                      const uint32_t* __restrict__ partial,
                                                      uint32_t* __restrict__ out) {
  __shared__ uint32_t s[kBlock];
  int64_t base = (int64_t)blockIdx.x * kScanChunk + (int64_t)threadIdx.x * kScanItems;
  uint32_t v[kScanItems];
  uint32_t acc = 0;
  for (int j = 0; j < kScanItems; ++j) {
    v[j] = base + j < n ? in[base + j] : 0u;
    acc += v[j];
  }
  uint32_t tot;
  uint32_t run = block_exclusive_scan(acc, s, &tot) + (partial ? partial[blockIdx.x] : 0u);
  for (int j = 0; j < kScanItems; ++j) {
    if (base + j < n) out[base + j] = run;
    run += v[j];
  }
}

// Exclusive scan of up to a few chunks in one workgroup, chunk after chunk with a running
// carry: one launch where the three-kernel scan would spend two more on a tiny partial pass.
constexpr int kScanLoopChunks = 8;
__global__ void __launch_bounds__(kBlock) k_scan_loop(const uint32_t* __restrict__ in, int64_t n,
                                                      uint32_t* __restrict__ out) {
  __shared__ uint32_t s[kBlock];
  uint32_t carry = 0;
  for (int64_t c0 = 0; c0 < n; c0 += kScanChunk) {
    const int64_t base = c0 + (int64_t)threadIdx.x * kScanItems;
    uint32_t v[kScanItems];
    uint32_t acc = 0;
    for (int j = 0; j < kScanItems; ++j) {
      v[j] = base + j < n ? in[base + j] : 0u;
      acc += v[j];
    }
    uint32_t tot;
    uint32_t run = block_exclusive_scan(acc, s, &tot) + carry;
    for (int j = 0; j < kScanItems; ++j) {
      if (base + j < n) out[base + j] = run;
      run += v[j];
    }
    carry += tot;
    __syncthreads();
  }
}

// `offsets` is either the scanned histogram table ([digit][workgroup], exclusive), or, with
// `fused`, the raw counts in workgroup-major rows: then thread d adds digit d's counts of the
// workgroups before this one, and a block scan over the 256 digit totals gives the digit's
// start. A wave takes ITEMS x 64 consecutive keys and ranks them against its own counters, with
// no barrier between rounds; then the waves' counts are added up once. Bound by latency at 100k
// keys (10 us a pass), by memory at 3M (28 us for 72 MB; 53 before, with four barriers a round
// and the keys written where they stood; 61 without the barriers but not through LDS).
template <class K, int ITEMS, int BITS>
__global__ void __launch_bounds__(kBlock) k_radix_scatter(const K* __restrict__ keys_in,
                                                          const uint32_t* __restrict__ vals_in, int64_t n, int shift,
                                                          const uint32_t* __restrict__ offsets, int nblocks, bool fused,
                                                          K* __restrict__ keys_out, uint32_t* __restrict__ vals_out,
                                                          const uint32_t* __restrict__ n_dev,
                                                          uint32_t* __restrict__ next_hist) {
  if (n_dev) n = min(n, (int64_t)*n_dev);
  constexpr int kTile = kBlock * ITEMS;
  const int64_t span = radix_tiles(n, kTile, nblocks) * kTile;
  const int64_t begin = (int64_t)blockIdx.x * span;
  if (begin >= n) return;  // the whole workgroup is past the keys
  constexpr int kBins = 1 << BITS;
  constexpr int kOwn = kBins / kBlock;  // a thread's digits: kOwn of them from kOwn * threadIdx.x on
  __shared__ uint32_t s_cnt[kBlock / 64][kBins];
  __shared__ uint32_t s_tmp[kBins];
  __shared__ K s_key[ITEMS == kRadixItems ? kTile : 1];
  __shared__ uint32_t s_val[ITEMS == kRadixItems ? kTile : 1];
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  const uint64_t lt_mask = lane ? (~0ull >> (64 - lane)) : 0ull;
  const int d0 = kOwn * threadIdx.x;
  uint32_t off[kOwn];
  if (fused) {
    // (32 rows' loads in flight together: the rows come from beyond this XCD's L2)
    uint32_t before[kOwn] = {}, total[kOwn] = {};
    auto rows = [&](int b, auto some) __attribute__((always_inline)) {
      constexpr int N = decltype(some)::value;
      uint32_t c[N][kOwn];
#pragma unroll
      for (int u = 0; u < N; ++u)
#pragma unroll
        for (int d = 0; d < kOwn; ++d) c[u][d] = offsets[(size_t)(b + u) * kBins + d0 + d];
#pragma unroll
      for (int u = 0; u < N; ++u)
#pragma unroll
        for (int d = 0; d < kOwn; ++d) {
          total[d] += c[u][d];
          before[d] += b + u < (int)blockIdx.x ? c[u][d] : 0u;
        }
    };
    int b = 0;
    for (; b + 32 <= nblocks; b += 32) rows(b, std::integral_constant<int, 32>());
    for (; b + 8 <= nblocks; b += 8) rows(b, std::integral_constant<int, 8>());
    for (; b < nblocks; ++b) rows(b, std::integral_constant<int, 1>());
    uint32_t all, sum = 0;
#pragma unroll
    for (int d = 0; d < kOwn; ++d) sum += total[d];
    uint32_t at = block_exclusive_scan(sum, s_tmp, &all);
#pragma unroll
    for (int d = 0; d < kOwn; ++d) {
      off[d] = at + before[d];
      at += total[d];
    }
  } else {
#pragma unroll
    for (int d = 0; d < kOwn; ++d) off[d] = offsets[(size_t)(d0 + d) * nblocks + blockIdx.x];
  }
  const int64_t stop = min(n, begin + span);
  for (int64_t tile = begin; tile < stop; tile += kTile) {
    const int64_t first = tile + wave * (64 * ITEMS) + lane;
    K key[ITEMS];
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) key[r] = first + r * 64 < n ? keys_in[first + r * 64] : (K)0;
    uint32_t val[ITEMS];
#pragma unroll
    for (int r = 0; r < ITEMS; ++r)
      val[r] = !vals_in ? (uint32_t)(first + r * 64) : first + r * 64 < n ? vals_in[first + r * 64] : 0u;
    for (int w = 0; w < kBlock / 64; ++w)
#pragma unroll
      for (int d = 0; d < kOwn; ++d) s_cnt[w][d0 + d] = 0u;
    __syncthreads();
    uint32_t rank[ITEMS];
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) {
      const bool valid = first + r * 64 < n;
      const uint32_t digit = (uint32_t)(key[r] >> shift) & (kBins - 1u);
      uint64_t peers = __ballot(valid);
#pragma unroll
      for (int b = 0; b < BITS; ++b) {
        const bool bit = (digit >> b) & 1u;
        const uint64_t m = __ballot(valid && bit);
        peers &= bit ? m : ~m;
      }
      const uint32_t in_round = (uint32_t)__popcll(peers & lt_mask);
      const uint32_t before = s_cnt[wave][digit];
      rank[r] = before + in_round;
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
      if (valid && in_round == 0) s_cnt[wave][digit] = before + (uint32_t)__popcll(peers);
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
    }
    __syncthreads();
    uint32_t mine[kOwn], sum = 0;
#pragma unroll
    for (int d = 0; d < kOwn; ++d) {
      mine[d] = 0;
#pragma unroll
      for (int w = 0; w < kBlock / 64; ++w) mine[d] += s_cnt[w][d0 + d];
      sum += mine[d];
    }
    if constexpr (ITEMS == kRadixItems) {
      // large sorts go through LDS in their new order, so that runs of a digit are written
      // together
      uint32_t all;
      uint32_t at = block_exclusive_scan(sum, s_tmp, &all);
#pragma unroll
      for (int d = 0; d < kOwn; ++d) {
        s_tmp[d0 + d] = off[d] - at;  // from a place here to its place in the result
#pragma unroll
        for (int w = 0; w < kBlock / 64; ++w) {
          const uint32_t c = s_cnt[w][d0 + d];
          s_cnt[w][d0 + d] = at;
          at += c;
        }
      }
      __syncthreads();
#pragma unroll
      for (int r = 0; r < ITEMS; ++r)
        if (first + r * 64 < n) {
          const uint32_t i = s_cnt[wave][(uint32_t)(key[r] >> shift) & (kBins - 1u)] + rank[r];
          s_key[i] = key[r];
          s_val[i] = val[r];
        }
      __syncthreads();
#pragma unroll
      for (int r = 0; r < ITEMS; ++r) {
        const uint32_t i = (uint32_t)(r * kBlock) + threadIdx.x;
        if (i < all) {
          const K k = s_key[i];
          const uint32_t pos = s_tmp[(uint32_t)(k >> shift) & (kBins - 1u)] + i;
          keys_out[pos] = k;
          vals_out[pos] = s_val[i];
        }
      }
    } else {
#pragma unroll
      for (int d = 0; d < kOwn; ++d) {
        uint32_t at = off[d];
#pragma unroll
        for (int w = 0; w < kBlock / 64; ++w) {
          const uint32_t c = s_cnt[w][d0 + d];
          s_cnt[w][d0 + d] = at;
          at += c;
        }
      }
      __syncthreads();
#pragma unroll
      for (int r = 0; r < ITEMS; ++r) {
        if (first + r * 64 < n) {
          const uint32_t pos = s_cnt[wave][(uint32_t)(key[r] >> shift) & (kBins - 1u)] + rank[r];
          keys_out[pos] = key[r];
          vals_out[pos] = val[r];
          // counted for the next pass, in the row of the workgroup that will read the key
          // (these sorts have a workgroup for each tile)
          if (next_hist)
            atomicAdd(next_hist + (size_t)(pos / (uint32_t)kTile) * kBins + ((uint32_t)(key[r] >> (shift + BITS)) & (kBins - 1u)), 1u);
        }
      }
    }
#pragma unroll
    for (int d = 0; d < kOwn; ++d) off[d] += mine[d];
    if (tile + kTile < stop) __syncthreads();
  }
}

// ------------------------------------------------------------------ radix tree (Karras)

__device__ __forceinline__ int prefix_len(const uint64_t* __restrict__ codes, int64_t n, int64_t i, int64_t j) {
  if (j < 0 || j >= n) return -1;
  uint64_t a = codes[i], b = codes[j];
  if (a != b) return __clzll(a ^ b);
  return 64 + __clz((uint32_t)i ^ (uint32_t)j);
}

// ------------------------------------------------------------------ leaves

struct GaussIn {
  const float* means;
  const float* scales;
  const float* quats;
  const float* opac;
};

__device__ __forceinline__ void quat_rot(const float* q4, float R[3][3]) {
  float w = q4[0], x = q4[1], y = q4[2], z = q4[3];
  float inv = rsqrtf(w * w + x * x + y * y + z * z);
  w *= inv; x *= inv; y *= inv; z *= inv;
  R[0][0] = 1.f - 2.f * (y * y + z * z); R[0][1] = 2.f * (x * y - w * z);       R[0][2] = 2.f * (x * z + w * y);
  R[1][0] = 2.f * (x * y + w * z);       R[1][1] = 1.f - 2.f * (x * x + z * z); R[1][2] = 2.f * (y * z - w * x);
  R[2][0] = 2.f * (x * z - w * y);       R[2][1] = 2.f * (y * z + w * x);       R[2][2] = 1.f - 2.f * (x * x + y * y);
}

// Relative padding of the leaf boxes: the box must contain the bounding ellipsoid as the
// leaf test sees it in binary32 (rounding of R, rho and of the transformed ray).
constexpr float kBoxPad = 1.0f + 1.0f / 128.0f;

struct GaussGeom {
  float R[3][3];
  float s[3];
  float rho;
  float o;
  bool active;
};

__device__ __forceinline__ GaussGeom gauss_geom(const GaussIn& g, int64_t i, float alpha_min) {
  GaussGeom G;
  quat_rot(g.quats + 4 * i, G.R);
  for (int a = 0; a < 3; ++a) G.s[a] = g.scales[3 * i + a];
  G.o = g.opac[i];
  G.active = G.o > alpha_min && G.s[0] > 0.f && G.s[1] > 0.f && G.s[2] > 0.f;
  G.rho = G.active ? sqrtf(2.f * logf(G.o / alpha_min)) : 0.f;
  return G;
}

// Box of the bounding ellipsoid scaled by `scale` about mu (1 for the sphere leaf; the
// icosahedron's circumradius over its inradius for the icosahedron instance leaf, whose
// mesh lies inside that scaled ellipsoid).
__device__ __forceinline__ void gauss_box(const GaussIn& g, int64_t i, const GaussGeom& G, float scale, float lo[3],
                                          float hi[3]) {
  for (int j = 0; j < 3; ++j) {
    float m = g.means[3 * i + j];
    float h = 0.f;
    if (G.active) {
      float v = 0.f;
      for (int k = 0; k < 3; ++k) v += G.R[j][k] * G.R[j][k] * G.s[k] * G.s[k];
      h = G.rho * sqrtf(v) * (kBoxPad * scale);
    }
    lo[j] = m - h;
    hi[j] = m + h;
  }
}

// Counts a wave's leaves (in sorted order, so that neighbours mostly share a cell) in the
// density grid over `bounds`: one atomic per run of equal cells. Every lane of the wave calls it;
// `in`: the lane has a leaf.
__device__ __forceinline__ void count_density(bool in, float x, float y, float z, const float* __restrict__ bounds,
                                              uint32_t* __restrict__ grid) {
  const int cell = in ? density_cell(x, y, z, bounds) : -1;
  const int lane = threadIdx.x & 63;
  const int before = __shfl_up(cell, 1);
  const bool head = in && (lane == 0 || before != cell);
  const uint64_t heads = __ballot(head), live = __ballot(in);
  if (head) {
    const uint64_t later = lane == 63 ? 0ull : heads >> (lane + 1) << (lane + 1);
    const int end = later ? __ffsll((unsigned long long)later) - 1 : __popcll(live);
    atomicAdd(grid + cell, (uint32_t)(end - lane));
  }
}

// Sphere leaves: instance record and box for sorted position p.
__global__ void __launch_bounds__(kBlock) k_sphere_leaves(GaussIn g, const uint32_t* __restrict__ perm, int64_t n,
                                                          float alpha_min, float box_scale, float4* __restrict__ inst,
                                                          float* __restrict__ boxes, const float* __restrict__ bounds,
                                                          uint32_t* __restrict__ grid) {
  int64_t p = blockIdx.x * (int64_t)kBlock + threadIdx.x;
  const uint32_t i = p < n ? perm[p] : 0u;
  count_density(p < n, g.means[3 * (int64_t)i], g.means[3 * (int64_t)i + 1], g.means[3 * (int64_t)i + 2], bounds, grid);
  if (p >= n) return;
  GaussGeom G = gauss_geom(g, i, alpha_min);
  float4 r[4];
  float* rr = reinterpret_cast<float*>(r);
  for (int a = 0; a < 3; ++a) {
    // row a of A = column a of R / (rho s_a)
    float sc = G.active ? 1.f / (G.rho * G.s[a]) : 0.f;
    rr[4 * a + 0] = G.R[0][a] * sc;
    rr[4 * a + 1] = G.R[1][a] * sc;
    rr[4 * a + 2] = G.R[2][a] * sc;
    rr[4 * a + 3] = g.means[3 * i + a];
  }
  rr[12] = G.o;
  rr[13] = G.active ? log2f(G.o / alpha_min) : 0.f;
  rr[14] = __uint_as_float(i);
  rr[15] = __uint_as_float(G.active ? 1u : 0u);
  for (int q = 0; q < 4; ++q) inst[4 * p + q] = r[q];
  float lo[3], hi[3];
  gauss_box(g, i, G, box_scale, lo, hi);
  float* bx = boxes + ((n - 1) + p) * 6;
  for (int a = 0; a < 3; ++a) {
    bx[a] = lo[a];
    bx[3 + a] = hi[a];
  }
}

// ------------------------------------------------------------------ proxy mesh (baseline)

// Regular icosahedron of inradius 1 (its faces touch the unit sphere from outside):
// vertices and outward-wound faces, derived on the host from the definition.
struct Ico {
  float v[12][3];
  unsigned char f[20][3];
};

// Instance record in Gaussian order (used by the proxy BVH's blending).
__device__ __forceinline__ void write_instance(const GaussIn& g, uint32_t i, const GaussGeom& G, float alpha_min,
                                               float4* __restrict__ dst) {
  float r[16];
  for (int a = 0; a < 3; ++a) {
    float sc = G.active ? 1.f / (G.rho * G.s[a]) : 0.f;
    r[4 * a + 0] = G.R[0][a] * sc;
    r[4 * a + 1] = G.R[1][a] * sc;
    r[4 * a + 2] = G.R[2][a] * sc;
    r[4 * a + 3] = g.means[3 * i + a];
  }
  r[12] = G.o;
  r[13] = G.active ? log2f(G.o / alpha_min) : 0.f;
  r[14] = __uint_as_float(i);
  r[15] = __uint_as_float(G.active ? 1u : 0u);
  for (int q = 0; q < 4; ++q) dst[q] = make_float4(r[4 * q], r[4 * q + 1], r[4 * q + 2], r[4 * q + 3]);
}

// Relative and absolute padding of a triangle's box: the binary32 hit distance of a ray
// crossing the triangle must stay inside the box's slab interval.
constexpr float kTriPadRel = 1.0f / 1024.0f;
constexpr float kTriPadAbs = 1.0f / 131072.0f;

// One thread per Gaussian: instance record (Gaussian order), 20 world triangles
// mu + R diag(rho s) v_ico with their boxes and box centres (triangle order 20 g + face).
__global__ void __launch_bounds__(kBlock) k_proxy_setup(GaussIn g, int64_t n, float alpha_min, Ico ico,
                                                        float4* __restrict__ inst, float4* __restrict__ tri,
                                                        float* __restrict__ tbox, float* __restrict__ cent) {
  int64_t i = blockIdx.x * (int64_t)kBlock + threadIdx.x;
  if (i >= n) return;
  GaussGeom G = gauss_geom(g, i, alpha_min);
  write_instance(g, (uint32_t)i, G, alpha_min, inst + 4 * i);
  float w[12][3];
  for (int v = 0; v < 12; ++v)
    for (int a = 0; a < 3; ++a) {
      float acc = 0.f;
      for (int k = 0; k < 3; ++k) acc += G.R[a][k] * (G.rho * G.s[k] * ico.v[v][k]);
      w[v][a] = g.means[3 * i + a] + acc;  // inactive: rho = 0, a point at mu
    }
  for (int f = 0; f < 20; ++f) {
    const int64_t t = 20 * i + f;
    const float* A = w[ico.f[f][0]];
    const float* B = w[ico.f[f][1]];
    const float* C = w[ico.f[f][2]];
    tri[3 * t + 0] = make_float4(A[0], A[1], A[2], __uint_as_float((uint32_t)i));
    tri[3 * t + 1] = make_float4(B[0], B[1], B[2], 0.f);
    tri[3 * t + 2] = make_float4(C[0], C[1], C[2], 0.f);
    for (int a = 0; a < 3; ++a) {
      float lo = fminf(A[a], fminf(B[a], C[a]));
      float hi = fmaxf(A[a], fmaxf(B[a], C[a]));
      float pad = (hi - lo) * kTriPadRel + (fabsf(lo) + fabsf(hi)) * kTriPadAbs;
      tbox[6 * t + a] = lo - pad;
      tbox[6 * t + 3 + a] = hi + pad;
      cent[3 * t + a] = 0.5f * (lo + hi);
    }
  }
}

// Gather triangle records and boxes into sorted-leaf order.
__global__ void __launch_bounds__(kBlock) k_proxy_leaves(const uint32_t* __restrict__ perm, int64_t m,
                                                         const float4* __restrict__ tri_in,
                                                         const float* __restrict__ box_in,
                                                         float4* __restrict__ tri_out, float* __restrict__ boxes,
                                                         const float* __restrict__ cent, const float* __restrict__ bounds,
                                                         uint32_t* __restrict__ grid) {
  int64_t p = blockIdx.x * (int64_t)kBlock + threadIdx.x;
  const uint32_t t = p < m ? perm[p] : 0u;
  count_density(p < m, cent[3 * (int64_t)t], cent[3 * (int64_t)t + 1], cent[3 * (int64_t)t + 2], bounds, grid);
  if (p >= m) return;
  for (int q = 0; q < 3; ++q) tri_out[3 * p + q] = tri_in[3 * (int64_t)t + q];
  float* bx = boxes + ((m - 1) + p) * 6;
  for (int a = 0; a < 6; ++a) bx[a] = box_in[6 * (int64_t)t + a];
}

// ------------------------------------------------------------------ boxes of leaf ranges
// Every internal node of the radix tree covers a run of sorted leaves, so its box needs no
// bottom-up pass over the tree: unions of 2, 4, 8, ... consecutive leaves (aligned; the last of
// each level may be short) are formed eight levels per launch, and a node takes its run as at
// most two of them per level. The unions are exact minima and maxima, so the boxes are those of
// any other order. (At 100k leaves the two launches and the node's look-ups replace 17 + 39 us
// of bottom-up refit; at 3M 577 + 103 us.)
constexpr int kBoxLevels = 32;
struct BoxLevels {
  const float* leaves;      // level 0
  float* up;                // the levels above, one after the other
  int64_t at[kBoxLevels];   // first entry of each level in `up`
  int64_t size[kBoxLevels];
  int count;                // levels, the leaves' included
};

__device__ __forceinline__ const float* level_box(const BoxLevels& B, int level, int64_t i) {
  return level == 0 ? B.leaves + 6 * i : B.up + 6 * (B.at[level] + i);
}

__device__ __forceinline__ void join_box(float (&b)[6], const float* __restrict__ v) {
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    b[a] = fminf(b[a], v[a]);
    b[3 + a] = fmaxf(b[3 + a], v[3 + a]);
  }
}

// Levels from+1 .. from+8 over 256 entries of level `from` per workgroup.
__global__ void __launch_bounds__(kBlock) k_box_levels(BoxLevels B, int from) {
  __shared__ float s_box[kBlock][6];
  const int t = threadIdx.x;
  int64_t i = blockIdx.x * (int64_t)kBlock + t;
  if (i < B.size[from]) {
    const float* v = level_box(B, from, i);
    for (int a = 0; a < 6; ++a) s_box[t][a] = v[a];
  }
  for (int k = 1; k <= 8 && from + k < B.count; ++k) {
    __syncthreads();
    const int64_t j = (blockIdx.x * (int64_t)kBlock >> k) + t;
    float b[6];
    const bool mine = t < (kBlock >> k) && j < B.size[from + k];
    if (mine) {
      for (int a = 0; a < 6; ++a) b[a] = s_box[2 * t][a];
      if (2 * j + 1 < B.size[from + k - 1]) join_box(b, s_box[2 * t + 1]);
      float* dst = B.up + 6 * (B.at[from + k] + j);
      for (int a = 0; a < 6; ++a) dst[a] = b[a];
    }
    __syncthreads();
    if (mine)
      for (int a = 0; a < 6; ++a) s_box[t][a] = b[a];
  }
}

// Box of the leaves lo..hi.
__device__ __forceinline__ void run_box(const BoxLevels& B, uint32_t lo, uint32_t hi, float (&b)[6]) {
  for (int a = 0; a < 3; ++a) b[a] = INFINITY, b[3 + a] = -INFINITY;
  uint32_t l = lo, r = hi + 1u;
  for (int level = 0; l < r; ++level) {
    if (l & 1u) join_box(b, level_box(B, level, l++));
    if (r & 1u) join_box(b, level_box(B, level, --r));
    l >>= 1;
    r >>= 1;
  }
}

// ------------------------------------------------------------------ the radix tree (Karras)
// One thread per internal node: its range of sorted leaves, its children, its box and leaf
// count. A node of more than `ns` leaves lists its children of at most that many as subtrees of
// the restructuring pass, and one of more than `cut` leaves its children of at most that many
// for the trace's per-tile cost estimates (lo, leaf count) (hi, 0), up to kCutCap; 0: neither.
// The lists' order follows the threads' and nothing depends on it. With `depth` the kernel
// does its work only where the restructured tree measured there is deeper than max_depth: it
// puts the plain tree back (and clears the heights that are then measured again).
struct TopologyOut {
  uint32_t* child;
  uint32_t* parent;
  uint2* range;
  uint32_t* count;
  float* boxes;
  uint32_t* roots;
  uint32_t* n_roots;
  float4* cut;
  uint32_t* n_cut;
  uint32_t* heights;  // cleared, or null
};

__device__ __forceinline__ uint32_t list_place(bool want, uint32_t* counter) {
  const uint64_t m = __ballot(want);
  if (!m) return 0u;
  const int lane = threadIdx.x & 63, leader = __ffsll((unsigned long long)m) - 1;
  uint32_t base = 0u;
  if (lane == leader) base = atomicAdd(counter, (uint32_t)__popcll(m));
  return __shfl(base, leader) + (uint32_t)__popcll(m & ((1ull << lane) - 1ull));
}

__global__ void __launch_bounds__(kBlock) k_topology(const uint64_t* __restrict__ codes, int64_t n, BoxLevels B,
                                                     TopologyOut O, uint32_t ns, uint32_t cut,
                                                     const uint32_t* __restrict__ depth, int max_depth) {
  if (depth && *depth <= (uint32_t)max_depth) return;
  const int64_t i = blockIdx.x * (int64_t)kBlock + threadIdx.x;
  const bool mine = i < n - 1;
  int64_t gamma = 0, lo = 0, hi = 0;
  if (mine) {
    const int d = prefix_len(codes, n, i, i + 1) - prefix_len(codes, n, i, i - 1) > 0 ? 1 : -1;
    const int dmin = prefix_len(codes, n, i, i - d);
    int64_t lmax = 2;
    while (prefix_len(codes, n, i, i + lmax * d) > dmin) lmax <<= 1;
    int64_t l = 0;
    for (int64_t t = lmax >> 1; t >= 1; t >>= 1)
      if (prefix_len(codes, n, i, i + (l + t) * d) > dmin) l += t;
    const int64_t j = i + l * d;
    const int dnode = prefix_len(codes, n, i, j);
    int64_t s = 0;
    int64_t t = l;
    do {
      t = (t + 1) >> 1;
      if (prefix_len(codes, n, i, i + (s + t) * d) > dnode) s += t;
    } while (t > 1);
    gamma = i + s * d + (d < 0 ? -1 : 0);
    lo = i < j ? i : j;
    hi = i < j ? j : i;
    const uint32_t left = lo == gamma ? kLeafFlag | (uint32_t)gamma : (uint32_t)gamma;
    const uint32_t right = hi == gamma + 1 ? kLeafFlag | (uint32_t)(gamma + 1) : (uint32_t)(gamma + 1);
    O.parent[lo == gamma ? (n - 1) + gamma : gamma] = (uint32_t)i;
    O.parent[hi == gamma + 1 ? (n - 1) + gamma + 1 : gamma + 1] = (uint32_t)i;
    O.child[2 * i] = left;
    O.child[2 * i + 1] = right;
    O.range[i] = make_uint2((uint32_t)lo, (uint32_t)hi);
    O.count[i] = (uint32_t)(hi - lo + 1);  // leaves below the node
    if (i == 0) O.parent[0] = kNoParent;
    if (O.heights) O.heights[i] = 0u;
    float b[6];
    run_box(B, (uint32_t)lo, (uint32_t)hi, b);
    for (int a = 0; a < 6; ++a) O.boxes[6 * i + a] = b[a];
  }
  const uint32_t own = mine ? (uint32_t)(hi - lo + 1) : 0u;
  if (ns) {
    const bool whole = mine && i == 0 && own <= ns;
    const uint32_t at = list_place(whole, O.n_roots);
    if (whole) O.roots[at] = 0u;
  }
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    const int64_t a = k == 0 ? lo : gamma + 1, e = k == 0 ? gamma : hi;
    const uint32_t cnt = (uint32_t)(e - a + 1);
    if (ns) {
      const bool sub = own > ns && cnt <= ns;
      const uint32_t at = list_place(sub, O.n_roots);
      if (sub) O.roots[at] = cnt == 1u ? (uint32_t)(n - 1 + a) : (uint32_t)(k == 0 ? gamma : gamma + 1);
    }
    if (cut) {
      const bool piece = own > cut && cnt <= cut;
      const uint32_t at = list_place(piece, O.n_cut);
      if (piece && at < (uint32_t)kCutCap) {
        float b[6];
        run_box(B, (uint32_t)a, (uint32_t)e, b);
        O.cut[2 * (int64_t)at] = make_float4(b[0], b[1], b[2], (float)cnt);
        O.cut[2 * (int64_t)at + 1] = make_float4(b[3], b[4], b[5], 0.f);
      }
    }
  }
}

__device__ __forceinline__ void child_box(const float* boxes, int64_t n, uint32_t c, float b[6]) {
  const int64_t idx = (c & kLeafFlag) ? (n - 1) + (c & ~kLeafFlag) : c;
#pragma unroll
  for (int a = 0; a < 6; ++a) b[a] = boxes[idx * 6 + a];
}

// The largest subtree that one wave lays out (see the record layout below).
constexpr int64_t kLayoutLeaves = 128;
constexpr int kLayoutBlock = 1024;

// Four-wide node records (layout in grtx_internal.h), written once every box is final, and for
// the nodes above kLayoutLeaves leaves their entries' leaf counts.
__global__ void __launch_bounds__(kBlock) k_wide(int64_t n, const uint32_t* __restrict__ child,
                                                 const float* __restrict__ boxes, const uint32_t* __restrict__ count,
                                                 float4* __restrict__ nodes, uint4* __restrict__ counts) {
  const int64_t i = blockIdx.x * (int64_t)kBlock + threadIdx.x;
  if (i >= n - 1) return;
  // Start from the two children and open the internal entry of largest surface area
  // until there are four entries or none is internal (greedy collapse; every internal
  // node has a record, so a record may list nodes from any depth below it).
  uint32_t ref[4] = {child[2 * i], child[2 * i + 1], kNoChild, kNoChild};
  int cnt = 2;
  while (cnt < 4) {
    int best = -1;
    float best_area = -1.f;
    for (int j = 0; j < cnt; ++j) {
      if (ref[j] & kLeafFlag) continue;
      const float* bb = boxes + 6 * (int64_t)ref[j];
      const float ex = bb[3] - bb[0], ey = bb[4] - bb[1], ez = bb[5] - bb[2];
      const float area = ex * ey + ey * ez + ez * ex;
      if (area > best_area) {
        best_area = area;
        best = j;
      }
    }
    if (best < 0) break;
    const uint32_t c = ref[best];
    ref[best] = child[2 * (int64_t)c];
    ref[cnt++] = child[2 * (int64_t)c + 1];
  }
  const float* own = boxes + 6 * i;  // the union of the children's boxes
  float org[3], step[3];
  uint32_t wlo[3] = {0u, 0u, 0u}, whi[3] = {0u, 0u, 0u};
  for (int a = 0; a < 3; ++a) {
    org[a] = own[a];
    const double ext = (double)own[3 + a] - (double)own[a];
    int e = -126;
    if (ext > 0.0) {
      (void)frexp(ext / 254.0, &e);  // ext / 254 <= 2^e
      e = e < -126 ? -126 : e;
    }
    step[a] = ldexpf(1.0f, e);
  }
  for (int j = 0; j < cnt; ++j) {
    float b[6];
    child_box(boxes, n, ref[j], b);
    for (int a = 0; a < 3; ++a) {
      const double s = (double)step[a];
      double ql = floor(((double)b[a] - (double)org[a]) / s);
      double qh = ceil(((double)b[3 + a] - (double)org[a]) / s);
      ql = ql < 0.0 ? 0.0 : ql > 255.0 ? 255.0 : ql;
      qh = qh < 0.0 ? 0.0 : qh > 255.0 ? 255.0 : qh;
      wlo[a] |= (uint32_t)ql << (8 * j);
      whi[a] |= (uint32_t)qh << (8 * j);
    }
  }
  if (count[i] > (uint32_t)kLayoutLeaves) {
    uint32_t c[4];
    for (int j = 0; j < 4; ++j) c[j] = ref[j] != kNoChild && !(ref[j] & kLeafFlag) ? count[ref[j]] : 0u;
    counts[i] = make_uint4(c[0], c[1], c[2], c[3]);
  }
  float4* r = nodes + (int64_t)kNodeF4 * i;
  r[0] = make_float4(org[0], org[1], org[2], step[0]);
  r[1] = make_float4(step[1], step[2], __uint_as_float(ref[0]), __uint_as_float(ref[1]));
  r[2] = make_float4(__uint_as_float(ref[2]), __uint_as_float(ref[3]), __uint_as_float(wlo[0]),
                     __uint_as_float(wlo[1]));
  r[3] = make_float4(__uint_as_float(wlo[2]), __uint_as_float(whi[0]), __uint_as_float(whi[1]),
                     __uint_as_float(whi[2]));
}

// ------------------------------------------------------------------ record layout
// Only the records that the traversal can reach are kept, about a third of the radix
// tree's internal nodes: the root's, and recursively those its entries list (a record's
// opened entries are interior to it). They are laid out breadth first: the records of
// nodes above kLayoutLeaves leaves by one workgroup, level by level, from position 0;
// each node of at most kLayoutLeaves leaves that such a record lists starts a task, a
// block of (leaves - 1) positions (the most records its subtree can have) reserved after
// the first `top_cap` positions, which one wave fills breadth first. So the records a
// ray meets near each other lie near each other, and the lines fetched hold live records
// only. `qold` maps each position of the top levels to the radix-tree node whose record it
// holds.
// Reserve and record a task for internal node c (leaf count cnt); returns its position.
__device__ __forceinline__ uint32_t new_task(uint32_t c, uint32_t cnt, uint32_t top_cap, uint32_t* task_cursor,
                                             uint32_t* n_tasks, uint2* tasks) {
  const uint32_t start = top_cap + atomicAdd(task_cursor, cnt - 1u);
  tasks[atomicAdd(n_tasks, 1u)] = make_uint2(c, start);
  return start;
}

// Root entry: the root's box and reference (internal node 0, or leaf 0 for one leaf); and the
// final depth and kind of the tree: out[0] = depth, out[1] = 1 if a restructured tree was
// kept. `tree` is the restructured tree's depth (null: none was made), `plain` the plain one's
// where it counts (null: a single leaf).
struct FinishArgs {
  const float* box;
  uint32_t ref;
  float* roots;
  const uint32_t* tree;
  int max_depth;
  const uint32_t* plain;
  uint32_t* out;
};
__device__ __forceinline__ void finish_tree(const FinishArgs& F) {
  if (threadIdx.x < 6) F.roots[threadIdx.x] = F.box[threadIdx.x];
  if (threadIdx.x == 6) F.roots[6] = __uint_as_float(F.ref);
  if (threadIdx.x == 7) {
    F.roots[7] = 0.f;
    const bool kept = F.tree && *F.tree <= (uint32_t)F.max_depth;
    const uint32_t d = kept ? *F.tree : F.plain ? *F.plain : 0u;
    F.out[0] = d;
    F.out[1] = kept ? 1u : 0u;
  }
}
// (for a single leaf; trees with nodes are finished by their layout)
__global__ void k_finish(FinishArgs F) { finish_tree(F); }

// The top levels (one workgroup; its counters live in LDS until the end). Root = radix-tree
// node 0 at position 0; with at most kLayoutLeaves leaves in all, the root itself is the
// only task (top_cap = 0). A level costs the latency of its loads: the record and its entries'
// counts are read together, and the positions' nodes pass through LDS while they fit there, so
// that the barrier need not wait for stores to memory (100k leaves: 52 us with the counts read after
// the records and the nodes in memory, 43 us so;
// 3M: 425 and 298).
constexpr uint32_t kLayoutHeld = 8192;  // positions whose nodes LDS holds
__global__ void __launch_bounds__(kLayoutBlock) k_layout_top(int64_t m, const float4* __restrict__ wide,
                                                             const uint4* __restrict__ counts, uint32_t top_cap,
                                                             float4* __restrict__ nodes, uint32_t* __restrict__ qold,
                                                             uint2* __restrict__ tasks, uint32_t* __restrict__ ctr,
                                                             FinishArgs F) {
  finish_tree(F);
  __shared__ uint32_t s_next, s_cursor, s_tasks;
  __shared__ uint32_t s_old[kLayoutHeld];
  if (m <= kLayoutLeaves) {
    if (threadIdx.x == 0) {
      ctr[0] = (uint32_t)(m - 1);
      ctr[1] = 1u;
      tasks[0] = make_uint2(0u, 0u);
    }
    return;
  }
  if (threadIdx.x == 0) {
    s_cursor = 0u;
    s_tasks = 0u;
    s_old[0] = 0u;
    s_next = 1u;
  }
  __syncthreads();
  uint32_t begin = 0, end = 1;
  while (begin < end) {
    for (uint32_t q = begin + threadIdx.x; q < end; q += kLayoutBlock) {
      const uint32_t old = q < kLayoutHeld ? s_old[q] : qold[q];
      const float4* src = wide + (int64_t)kNodeF4 * old;
      const uint4 c4 = counts[old];
      float4 q0 = src[0], q1 = src[1], q2 = src[2], q3 = src[3];
      uint32_t r[4] = {__float_as_uint(q1.z), __float_as_uint(q1.w), __float_as_uint(q2.x), __float_as_uint(q2.y)};
      const uint32_t cnt[4] = {c4.x, c4.y, c4.z, c4.w};
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        if (r[j] == kNoChild || (r[j] & kLeafFlag)) continue;
        if (cnt[j] > (uint32_t)kLayoutLeaves) {
          const uint32_t pos = atomicAdd(&s_next, 1u);
          if (pos < kLayoutHeld) s_old[pos] = r[j];
          else qold[pos] = r[j];
          r[j] = pos;
        } else {
          r[j] = new_task(r[j], cnt[j], top_cap, &s_cursor, &s_tasks, tasks);
        }
      }
      q1.z = __uint_as_float(r[0]);
      q1.w = __uint_as_float(r[1]);
      q2.x = __uint_as_float(r[2]);
      q2.y = __uint_as_float(r[3]);
      float4* dst = nodes + (int64_t)kNodeF4 * q;
      dst[0] = q0;
      dst[1] = q1;
      dst[2] = q2;
      dst[3] = q3;
    }
    // (a barrier for LDS alone while every position read next is held there)
    auto meet = [&]() {
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
      __builtin_amdgcn_s_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
    };
    meet();
    begin = end;
    end = s_next;
    if (end <= kLayoutHeld) meet();
    else __syncthreads();
  }
  if (threadIdx.x == 0) {
    ctr[0] = s_cursor;
    ctr[1] = s_tasks;
  }
}

// The tasks: one wave fills a block breadth first, a level at a time. The records of one
// level belong to disjoint subtrees of two leaves or more, so a block of at most
// kLayoutLeaves leaves has at most kLayoutLeaves / 2 = 64 records per level: one per lane.
// Each lane places its record, its internal entries taking the next positions in lane and
// entry order (the order a sequential breadth-first fill gives), and passes their
// radix-tree nodes through LDS to the lanes that place them on the next level.
static_assert(kLayoutLeaves / 2 <= 64, "a level of a layout block must fit one wave");
__global__ void __launch_bounds__(kBlock) k_layout_tasks(const float4* __restrict__ wide, const uint2* __restrict__ tasks,
                                                         const uint32_t* __restrict__ ctr, float4* __restrict__ nodes) {
  __shared__ uint32_t s_next[kBlock / 64][64];
  const uint32_t n = ctr[1];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const uint64_t below = lane ? ~0ull >> (64 - lane) : 0ull;
  for (uint32_t t = blockIdx.x * (kBlock / 64) + w; t < n; t += gridDim.x * (kBlock / 64)) {
    const uint2 task = tasks[t];
    uint32_t begin = task.y, width = 1, old = task.x;
    while (width > 0) {
      const bool mine = (uint32_t)lane < width;
      float4 q0{}, q1{}, q2{}, q3{};
      if (mine) {
        const float4* src = wide + (int64_t)kNodeF4 * old;
        q0 = src[0];
        q1 = src[1];
        q2 = src[2];
        q3 = src[3];
      }
      uint32_t r[4] = {__float_as_uint(q1.z), __float_as_uint(q1.w), __float_as_uint(q2.x), __float_as_uint(q2.y)};
      bool in[4];
      uint32_t below_n = 0, total = 0;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        in[j] = mine && r[j] != kNoChild && !(r[j] & kLeafFlag);
        const uint64_t m = __ballot(in[j]);
        below_n += (uint32_t)__popcll(m & below);
        total += (uint32_t)__popcll(m);
      }
      const uint32_t nbeg = begin + width;
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // last level's reads of s_next are done
      if (mine) {
        uint32_t k = below_n;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          if (in[j]) {
            s_next[w][k] = r[j];
            r[j] = nbeg + k;
            ++k;
          }
        }
        q1.z = __uint_as_float(r[0]);
        q1.w = __uint_as_float(r[1]);
        q2.x = __uint_as_float(r[2]);
        q2.y = __uint_as_float(r[3]);
        float4* dst = nodes + (int64_t)kNodeF4 * (begin + (uint32_t)lane);
        dst[0] = q0;
        dst[1] = q1;
        dst[2] = q2;
        dst[3] = q3;
      }
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // this level's writes to s_next are done
      width = total < 64u ? total : 64u;  // (total <= 64 by the bound above)
      old = (uint32_t)lane < width ? s_next[w][lane] : 0u;
      begin = nbeg;
    }
  }
}

// ------------------------------------------------------------------ pinhole rays

__global__ void __launch_bounds__(kBlock) k_pinhole(CameraFrame cf, int W, int H, float* __restrict__ origins,
                                                    float* __restrict__ dirs) {
  int64_t i = blockIdx.x * (int64_t)kBlock + threadIdx.x;
  if (i >= (int64_t)W * H) return;
  int y = (int)(i / W), x = (int)(i - (int64_t)y * W);
  float dx, dy, dz;
  pinhole_dir(cf.fwd[0], cf.fwd[1], cf.fwd[2], cf.right[0], cf.right[1], cf.right[2], cf.up[0], cf.up[1], cf.up[2], x, y,
              W, H, &dx, &dy, &dz);
  origins[3 * i + 0] = cf.eye[0];
  origins[3 * i + 1] = cf.eye[1];
  origins[3 * i + 2] = cf.eye[2];
  dirs[3 * i + 0] = dx;
  dirs[3 * i + 1] = dy;
  dirs[3 * i + 2] = dz;
}

__global__ void __launch_bounds__(kBlock) k_fill_u32(uint32_t* p, int64_t n, uint32_t v) {
  int64_t i = blockIdx.x * (int64_t)kBlock + threadIdx.x;
  if (i < n) p[i] = v;
}

inline unsigned grid_for(int64_t n) { return (unsigned)std::max<int64_t>(1, (n + kBlock - 1) / kBlock); }



// Sorts keys by `passes` digits: *kres and *vres receive the arrays that hold the sorted keys and the
// positions they came from (after an even number of passes `keys` and `vals`, else the temporaries).
template <class K, int BITS>
grtx_status radix_sort(K* keys, uint32_t* vals, K* tkeys, uint32_t* tvals, int64_t n, Scratch& sc, hipStream_t s,
                       int passes, const uint32_t* n_dev, K** kres, uint32_t** vres) {
  const int items = n <= kRadixSmall ? kRadixItemsSmall : kRadixItems;
  const int64_t tile = (int64_t)kBlock * items;
  const int64_t tiles = (n + tile - 1) / tile;
  if (tiles > (int64_t)kScanChunk * kScanChunk / 256) {  // (the table of eight-bit digits must fit a scan)
    set_error("radix sort: %lld keys exceed the supported size", (long long)n);
    return GRTX_ERR_INVALID_ARG;
  }
  int nblocks = (int)tiles;
  if (n_dev && nblocks > kRadixFusedBlocks)
    nblocks = std::max(kRadixFusedBlocks, std::min(kRadixDeviceBlocks, nblocks / 16));
  const bool fused = nblocks <= kRadixFusedBlocks;
  int64_t hn = (int64_t)nblocks << BITS;
  uint32_t *hist = nullptr, *offs = nullptr, *part = nullptr;
  int nparts = (int)((hn + kScanChunk - 1) / kScanChunk);
  GRTX_TRY(sc.get(&hist, hn));
  GRTX_TRY(sc.get(&offs, hn));
  GRTX_TRY(sc.get(&part, nparts));
  K* kin = keys;
  uint32_t* vin = vals;
  K* kout = tkeys;
  uint32_t* vout = tvals;
  // Small fused sorts count the next pass's digits in the scatter (rows of their own per pass,
  // cleared by the counting kernel), so that only the first pass has a counting kernel: 12 against 14 us a pass at 100k
  // keys; at a million the atomics cost more than the kernel (51 against 38 us).
  uint32_t* rows = nullptr;
  const bool counts_next = fused && items == kRadixItemsSmall && passes > 1;
  if (counts_next) {
    GRTX_TRY(sc.get(&rows, hn * (passes - 1)));
  }
  for (int pass = 0; pass < passes; ++pass) {
    int shift = BITS * pass;
    if (!counts_next || pass == 0)
      hipLaunchKernelGGL((k_radix_hist<K, BITS>), dim3(nblocks), dim3(kBlock), 0, s, kin, n, shift, items, hist, nblocks, fused,
                         n_dev, rows, counts_next ? passes - 1 : 0);
    if (fused) {
      // the scatter turns the counts into offsets itself
    } else {
      hipLaunchKernelGGL(k_scan_reduce, dim3(nparts), dim3(kBlock), 0, s, hist, hn, part);
      hipLaunchKernelGGL(k_scan_partials, dim3(1), dim3(kBlock), 0, s, part, nparts);
      hipLaunchKernelGGL(k_scan_down, dim3(nparts), dim3(kBlock), 0, s, hist, hn, part, offs);
    }
    const uint32_t* counts = !fused ? offs : !counts_next || pass == 0 ? hist : rows + hn * (pass - 1);
    const uint32_t* from = pass == 0 ? nullptr : vin;  // (at first a key's value is its position)
    if (items == kRadixItemsSmall)
      hipLaunchKernelGGL((k_radix_scatter<K, kRadixItemsSmall, BITS>), dim3(nblocks), dim3(kBlock), 0, s, kin, from, n, shift,
                         counts, nblocks, fused, kout, vout, n_dev,
                         counts_next && pass + 1 < passes ? rows + hn * pass : nullptr);
    else
      hipLaunchKernelGGL((k_radix_scatter<K, kRadixItems, BITS>), dim3(nblocks), dim3(kBlock), 0, s, kin, from, n, shift,
                         counts, nblocks, fused, kout, vout, n_dev, (uint32_t*)nullptr);
    GRTX_LAUNCH_CHECK();
    std::swap(kin, kout);
    std::swap(vin, vout);
  }
  *kres = kin;
  *vres = vin;
  return GRTX_OK;
}

// ------------------------------------------------------------------ treelet restructuring
// One bottom-up pass over the radix tree that rebuilds, at every internal node, the
// treelet of the node and its largest descendants (up to kTreeletLeaves treelet leaves,
// opened by largest surface area) into the binary topology of least surface-area cost,
// found by dynamic programming over the subsets of the treelet leaves (restructuring after
// Karras and Aila's treelet optimisation). Leaves keep their sorted positions, so the
// leaf order of the instances and every traced result are unchanged; only internal nodes
// are rewired, each keeping its index. A node comes after both of its subtrees: inside a subtree
// the nodes are taken by height, and above the subtrees by the second of the two threads that
// reach a node from its children.
constexpr int kTreeletLeaves = 5;
constexpr float kCostNode = 1.2f;  // surface-area cost of visiting an internal node
constexpr float kCostLeaf = 1.f;   // ... of testing a leaf

// Half the surface area of a box, and that of a set of treelet leaves. They differ in which
// product is rounded by itself; each is written out, so that a tree is the same whatever kernel
// builds it.
__device__ __forceinline__ float half_area(const float* __restrict__ b) {
  const float ex = fmaxf(b[3] - b[0], 0.f), ey = fmaxf(b[4] - b[1], 0.f), ez = fmaxf(b[5] - b[2], 0.f);
  return fmaf(ez, ex, fmaf(ex, ey, ey * ez));
}
__device__ __forceinline__ float set_area(const float* __restrict__ b) {
  const float ex = fmaxf(b[3] - b[0], 0.f), ey = fmaxf(b[4] - b[1], 0.f), ez = fmaxf(b[5] - b[2], 0.f);
  return fmaf(ez, ex, fmaf(ey, ez, ex * ey));
}

__device__ __forceinline__ uint32_t node_of(uint32_t c, int64_t nint) {
  return (c & kLeafFlag) ? (uint32_t)(nint + (c & ~kLeafFlag)) : c;
}
__device__ __forceinline__ uint32_t ref_of(uint32_t u, int64_t nint) {
  return (int64_t)u >= nint ? kLeafFlag | (uint32_t)(u - nint) : u;
}

// The nodes above the subtrees take a thread each (k_treelet_top). Its work arrays of the subset
// dynamic programme live in LDS, entry-major ([entry][thread]), so that lanes index them
// independently; NS threads per workgroup.
constexpr int kSets = 1 << kTreeletLeaves;
template <int NS>
struct TreeletLds {
  float copt[kSets][NS];
  uint8_t split[kSets][NS];
  int stack_set[kTreeletLeaves][NS];
  uint32_t stack_node[kTreeletLeaves][NS];
};
// Subtree size of the per-subtree pass: 256 leaves, 128 above a million leaves. Smaller
// subtrees give shorter bottom-up chains and twice the workgroups per CU, but leave more nodes
// above them untouched where no second pass runs (100k: 0.7% more node visits per ray).
inline int subtree_leaves(int64_t m) { return m > ((int64_t)1 << 20) ? 128 : 256; }
// Per-subtree passes: one, three above a million leaves. Each further pass rebuilds the
// treelets the previous one left, and skips treelet roots of fewer than kLaterPassLeaves
// leaves (doubled per pass), where little is left to gain (after Karras and Aila's
// repeated passes with a growing minimum). The rule was set when a lane traced a ray: three
// passes at 3M leaves then took 5% off the trace for 2 ms of build. With sixteen lanes per ray,
// one pass against three: at 3M the build 3.8 and 6.3 ms, a 1920x1080 frame 18.0 and 19.8, 2M
// incoherent rays 45.6 and 44.3; at 1M the build 1.45 and 2.5 ms, 524,287 rays 6.85 and 6.74; at
// 100k 0.43 and 0.58 ms, the frame 2.71 and 2.69.
inline int treelet_passes(int64_t m) { return m > ((int64_t)1 << 20) ? 3 : 1; }
constexpr uint32_t kLaterPassLeaves = 4;

// Subset dynamic programme over NL treelet leaves, unrolled at compile time so that every
// subset and split index is a constant (the costs stay in registers); the chosen splits and
// costs then go to the thread's LDS column for the rebuild.
template <int NL, class Lds>
__device__ __forceinline__ void treelet_dp(const float (&lb)[kTreeletLeaves][6], const float (&lcost)[kTreeletLeaves],
                                           Lds& L, int tid) {
  float copt[1 << NL];
#pragma unroll
  for (int S = 1; S < (1 << NL); ++S) {
    if ((S & (S - 1)) == 0) {
      copt[S] = lcost[__builtin_ctz(S)];
      L.copt[S][tid] = copt[S];
      continue;
    }
    float b[6] = {INFINITY, INFINITY, INFINITY, -INFINITY, -INFINITY, -INFINITY};
#pragma unroll
    for (int q = 0; q < NL; ++q)
      if (S >> q & 1) {
#pragma unroll
        for (int a = 0; a < 3; ++a) {
          b[a] = fminf(b[a], lb[q][a]);
          b[3 + a] = fmaxf(b[3 + a], lb[q][3 + a]);
        }
      }
    float best = INFINITY;
    int bp = S & -S;  // (a split also where no cost is finite: boxes of infinite Gaussians)
#pragma unroll
    for (int P = 1; P < S; ++P) {
      if ((P & S) != P || !(P & S & -S)) continue;  // each split once: the part holding the lowest leaf
      const float c = copt[P] + copt[S ^ P];
      if (c < best) {
        best = c;
        bp = P;
      }
    }
    copt[S] = kCostNode * set_area(b) + best;
    L.copt[S][tid] = copt[S];
    L.split[S][tid] = (uint8_t)bp;
  }
}

template <class Lds>
__device__ __forceinline__ void restructure(uint32_t p, int64_t nint, uint32_t* __restrict__ child, uint32_t* __restrict__ parent,
                            float* __restrict__ boxes, float* __restrict__ cost, uint32_t* __restrict__ count,
                            Lds& L, int tid) {
  // treelet leaves (registers, constant indices only) and its internal nodes
  uint32_t leaf[kTreeletLeaves], inner[kTreeletLeaves - 1];
  float larea[kTreeletLeaves];
#pragma unroll
  for (int q = 0; q < kTreeletLeaves; ++q) {
    leaf[q] = 0u;
    larea[q] = -1.f;
  }
#pragma unroll
  for (int q = 0; q < kTreeletLeaves - 1; ++q) inner[q] = p;
  int nl = 2;
  leaf[0] = node_of(child[2 * (int64_t)p], nint);
  leaf[1] = node_of(child[2 * (int64_t)p + 1], nint);
  larea[0] = half_area(boxes + 6 * (int64_t)leaf[0]);
  larea[1] = half_area(boxes + 6 * (int64_t)leaf[1]);
#pragma unroll
  for (int step = 0; step < kTreeletLeaves - 2; ++step) {
    // open the internal treelet leaf of largest surface area
    int best = -1;
    float ba = -1.f;
#pragma unroll
    for (int q = 0; q < kTreeletLeaves; ++q)
      if (q < nl && (int64_t)leaf[q] < nint && larea[q] > ba) {
        ba = larea[q];
        best = q;
      }
    if (best < 0) break;
    uint32_t x = 0u;
#pragma unroll
    for (int q = 0; q < kTreeletLeaves; ++q)
      if (q == best) x = leaf[q];
    inner[step + 1] = x;
    const uint32_t c0 = node_of(child[2 * (int64_t)x], nint), c1 = node_of(child[2 * (int64_t)x + 1], nint);
    const float a0 = half_area(boxes + 6 * (int64_t)c0), a1 = half_area(boxes + 6 * (int64_t)c1);
#pragma unroll
    for (int q = 0; q < kTreeletLeaves; ++q) {
      if (q == best) {
        leaf[q] = c0;
        larea[q] = a0;
      }
      if (q == nl) {
        leaf[q] = c1;
        larea[q] = a1;
      }
    }
    ++nl;
  }
  // the treelet leaves' boxes, counts and costs, read once
  float lb[kTreeletLeaves][6];
  uint32_t lcnt[kTreeletLeaves];
  float lcost[kTreeletLeaves];
#pragma unroll
  for (int q = 0; q < kTreeletLeaves; ++q) {
    if (q < nl) {
      const float* bq = boxes + 6 * (int64_t)leaf[q];
#pragma unroll
      for (int a = 0; a < 6; ++a) lb[q][a] = bq[a];
      lcnt[q] = (int64_t)leaf[q] >= nint ? 1u : count[leaf[q]];
      lcost[q] = cost[leaf[q]];
    } else {
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        lb[q][a] = INFINITY;
        lb[q][3 + a] = -INFINITY;
      }
      lcnt[q] = 0u;
      lcost[q] = 0.f;
    }
  }
  auto set_box = [&](int S, float b[6]) __attribute__((always_inline)) {
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      b[a] = INFINITY;
      b[3 + a] = -INFINITY;
    }
#pragma unroll
    for (int q = 0; q < kTreeletLeaves; ++q)
      if (S >> q & 1) {
#pragma unroll
        for (int a = 0; a < 3; ++a) {
          b[a] = fminf(b[a], lb[q][a]);
          b[3 + a] = fmaxf(b[3 + a], lb[q][3 + a]);
        }
      }
  };
  // optimal cost of every subset of the treelet leaves and the split that reaches it
  const int full = (1 << nl) - 1;
  if (nl == kTreeletLeaves) treelet_dp<kTreeletLeaves>(lb, lcost, L, tid);
  else if (nl == 4) treelet_dp<4>(lb, lcost, L, tid);
  else if (nl == 3) treelet_dp<3>(lb, lcost, L, tid);
  else treelet_dp<2>(lb, lcost, L, tid);
  // rebuild top-down, reusing the treelet's internal nodes (p stays the root)
  int sp = 0, next = 1;
  L.stack_set[0][tid] = full;
  L.stack_node[0][tid] = p;
  sp = 1;
  while (sp > 0) {
    --sp;
    const int S = L.stack_set[sp][tid];
    const uint32_t node = L.stack_node[sp][tid];
    const int P = L.split[S][tid];
    for (int k = 0; k < 2; ++k) {
      const int X = k == 0 ? P : S ^ P;
      uint32_t c = 0u;
      if ((X & (X - 1)) == 0) {
#pragma unroll
        for (int q = 0; q < kTreeletLeaves; ++q)
          if (X == (1 << q)) c = leaf[q];
      } else {
#pragma unroll
        for (int q = 1; q < kTreeletLeaves - 1; ++q)
          if (q == next) c = inner[q];
        ++next;
        L.stack_set[sp][tid] = X;
        L.stack_node[sp][tid] = c;
        ++sp;
      }
      child[2 * (int64_t)node + k] = ref_of(c, nint);
      parent[c] = node;
    }
    float b[6];
    set_box(S, b);
    uint32_t cnt = 0;
#pragma unroll
    for (int q = 0; q < kTreeletLeaves; ++q)
      if (S >> q & 1) cnt += lcnt[q];
    float* nb = boxes + 6 * (int64_t)node;
#pragma unroll
    for (int a = 0; a < 6; ++a) nb[a] = b[a];
    cost[node] = L.copt[S][tid];
    count[node] = cnt;
  }
}

// The passes run per subtree of at most NS leaves whose parent has more (the nodes above keep
// the radix tree's topology): one workgroup takes a subtree, whose leaves are a contiguous run
// [lo, hi] of sorted positions. An internal node of the radix tree is numbered after one end of
// its range, a right child (and the root) after its first leaf, a left child after its last: the
// subtree's internal nodes are the indices lo..hi-1 where its root is lo, and lo+1..hi where it
// is hi. Restructuring only permutes them. The whole subtree sits in LDS for all of its passes. A pass takes the nodes
// by height, lowest first (what a node's treelet holds was taken at a lower height), each by a
// team of sixteen lanes that share out the subsets of the treelet's leaves; nodes that keep
// their children take one lane.
// What bounds it is the chain of heights, some 15 to 20 treelets one after the other: 3 to 4 us
// each, where one lane per treelet with its data in global memory took 8 (100k leaves: 130 to
// 78 us), and above a million leaves the vector units' issue (3M leaves, three passes: 5.42 to
// 3.5 ms). The trees are the same.
constexpr int kTeam = 16;
constexpr uint16_t kNoLocal = 0xFFFFu;
template <int NS>
struct SubtreeLds {
  // internal nodes 0..n-2, then leaves n-1..2n-2
  float box[2 * NS - 1][6];
  float area[2 * NS - 1];
  float cost[2 * NS - 1];
  uint16_t count[2 * NS - 1];
  uint16_t kid[NS - 1][2];
  uint16_t par[2 * NS - 1];
  uint16_t list[NS - 1];           // internal nodes by height
  uint32_t height[NS - 1];
  uint32_t first[NS + 1];          // places of each height in `list`
  uint32_t max_height;
  struct Team {
    float cost[kSets];
    uint16_t leaf[8];              // the treelet's leaves
    uint8_t node[kSets];           // which of its nodes stands for the subset once rebuilt
    uint8_t split[kSets];
  } team[NS / kTeam];
};
static_assert(kTreeletLeaves == 5, "a team holds the ten pairs, ten triples, five quads and the full set's fifteen splits");

__device__ __forceinline__ void lds_order() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// Rebuilds the treelet of node p, by the sixteen lanes tl = 0..15 of one team. A lane holds one
// pair, one triple and one quad of the treelet's leaves, so that every size takes one round of
// LDS reads; the full set takes one split per lane.
template <int NS>
__device__ __forceinline__ void team_restructure(SubtreeLds<NS>& L, typename SubtreeLds<NS>::Team& W, int n, uint32_t p,
                                                 int tl) {
  // treelet leaves and the nodes between them, the same in every lane
  uint32_t leaf[kTreeletLeaves], inner[kTreeletLeaves - 1];
  float larea[kTreeletLeaves];
#pragma unroll
  for (int q = 0; q < kTreeletLeaves; ++q) leaf[q] = 0u, larea[q] = -1.f;
#pragma unroll
  for (int q = 0; q < kTreeletLeaves - 1; ++q) inner[q] = p;
  int nl = 2;
  leaf[0] = L.kid[p][0];
  leaf[1] = L.kid[p][1];
  larea[0] = L.area[leaf[0]];
  larea[1] = L.area[leaf[1]];
#pragma unroll
  for (int step = 0; step < kTreeletLeaves - 2; ++step) {
    // open the internal treelet leaf of largest surface area
    int best = -1;
    float ba = -1.f;
    uint32_t x = 0u;
#pragma unroll
    for (int q = 0; q < step + 2; ++q)
      if (leaf[q] < (uint32_t)(n - 1) && larea[q] > ba) {
        ba = larea[q];
        best = q;
        x = leaf[q];
      }
    if (best < 0) break;
    inner[step + 1] = x;
    const uint32_t c0 = L.kid[x][0], c1 = L.kid[x][1];
    const float a0 = L.area[c0];
#pragma unroll
    for (int q = 0; q < step + 2; ++q)
      if (q == best) leaf[q] = c0, larea[q] = a0;
    leaf[step + 2] = c1;
    larea[step + 2] = L.area[c1];
    ++nl;
  }
  const uint32_t full = (1u << nl) - 1u;
  if (tl < kTreeletLeaves) {
    uint32_t mine = leaf[0];
#pragma unroll
    for (int q = 1; q < kTreeletLeaves; ++q)
      if (q == tl) mine = leaf[q];
    W.leaf[tl] = (uint16_t)mine;
    W.cost[1 << tl] = L.cost[mine];
  }
  // this lane's subsets of two, three and four leaves (five bits each; none: beyond `full`)
  constexpr uint64_t kPairs = 3ull | 5ull << 5 | 6ull << 10 | 9ull << 15 | 10ull << 20 | 12ull << 25 | 17ull << 30 |
                              18ull << 35 | 20ull << 40 | 24ull << 45;
  constexpr uint64_t kTriples = 7ull | 11ull << 5 | 13ull << 10 | 14ull << 15 | 19ull << 20 | 21ull << 25 | 22ull << 30 |
                                25ull << 35 | 26ull << 40 | 28ull << 45;
  constexpr uint32_t kQuads = 15u | 23u << 5 | 27u << 10 | 29u << 15 | 30u << 20;
  const uint32_t set[3] = {tl < 10 ? (uint32_t)(kPairs >> (5 * tl)) & 31u : 32u,
                           tl < 10 ? (uint32_t)(kTriples >> (5 * tl)) & 31u : 32u,
                           tl < 5 ? (kQuads >> (5 * tl)) & 31u : 32u};
  lds_order();
  float box[3][6], area[3];
  uint32_t cnt[3];
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    cnt[k] = 0u;
    area[k] = 0.f;
    if (set[k] <= full) {
      W.node[set[k]] = 0xFFu;
      uint32_t rest = set[k];
#pragma unroll
      for (int i = 0; i < k + 2; ++i) {
        const uint32_t v = W.leaf[__ffs((int)rest) - 1];
        rest &= rest - 1u;
        const float* bv = L.box[v];
        cnt[k] += L.count[v];
#pragma unroll
        for (int a = 0; a < 3; ++a) {
          box[k][a] = i == 0 ? bv[a] : fminf(box[k][a], bv[a]);
          box[k][3 + a] = i == 0 ? bv[3 + a] : fmaxf(box[k][3 + a], bv[3 + a]);
        }
      }
      area[k] = set_area(box[k]);
    }
  }
  // optimal cost of every subset and the split that reaches it: a split is the part that holds
  // the lowest leaf; in ascending order the first of the cheapest is taken
  float own[3] = {0.f, 0.f, 0.f};
  auto better = [](float c, uint32_t P, float& best, uint32_t& bp) __attribute__((always_inline)) {
    if (c < best) best = c, bp = P;
  };
  if (set[0] <= full) {
    const uint32_t S = set[0], lo = S & (0u - S);
    own[0] = kCostNode * area[0] + (W.cost[lo] + W.cost[S ^ lo]);
    W.cost[S] = own[0];
    W.split[S] = (uint8_t)lo;
  }
  lds_order();
  if (set[1] <= full) {
    const uint32_t S = set[1], x = S & (0u - S), yz = S ^ x, y = yz & (0u - yz), z = yz ^ y;
    const float cx = W.cost[x], cy = W.cost[y], cz = W.cost[z], cyz = W.cost[yz], cxy = W.cost[x | y],
                cxz = W.cost[x | z];
    float best = INFINITY;
    uint32_t bp = x;
    better(cx + cyz, x, best, bp);
    better(cxy + cz, x | y, best, bp);
    better(cxz + cy, x | z, best, bp);
    own[1] = kCostNode * area[1] + best;
    W.cost[S] = own[1];
    W.split[S] = (uint8_t)bp;
  }
  lds_order();
  if (set[2] <= full) {
    const uint32_t S = set[2], x = S & (0u - S), r1 = S ^ x, y = r1 & (0u - r1), r2 = r1 ^ y, z = r2 & (0u - r2),
                   w = r2 ^ z;
    const float c1 = W.cost[x] + W.cost[r1], c2 = W.cost[x | y] + W.cost[r2], c3 = W.cost[x | z] + W.cost[y | w],
                c4 = W.cost[x | y | z] + W.cost[w], c5 = W.cost[x | w] + W.cost[y | z],
                c6 = W.cost[x | y | w] + W.cost[z], c7 = W.cost[x | z | w] + W.cost[y];
    float best = INFINITY;
    uint32_t bp = x;
    better(c1, x, best, bp);
    better(c2, x | y, best, bp);
    better(c3, x | z, best, bp);
    better(c4, x | y | z, best, bp);
    better(c5, x | w, best, bp);
    better(c6, x | y | w, best, bp);
    better(c7, x | z | w, best, bp);
    own[2] = kCostNode * area[2] + best;
    W.cost[S] = own[2];
    W.split[S] = (uint8_t)bp;
  }
  lds_order();
  uint32_t full_split = 0u;
  if (nl == kTreeletLeaves) {
    const uint32_t q = 2u * (uint32_t)tl;
    const float c = tl < 15 ? W.cost[1u | q] + W.cost[30u ^ q] : INFINITY;
    float least = c;
#pragma unroll
    for (int off = 8; off > 0; off >>= 1) least = fminf(least, __shfl_xor(least, off));
    // (of the fifteen splits; where no cost is a number, the first)
    const uint32_t eq = (uint32_t)(__ballot(c == least) >> (threadIdx.x & 48)) & 0x7FFFu;
    full_split = 1u | 2u * (uint32_t)(eq ? __ffs((int)eq) - 1 : 0);
    if (tl == 0) L.cost[p] = kCostNode * set_area(L.box[p]) + least;
  }
  // rebuild top-down, reusing the treelet's internal nodes (p stays the root); the subsets still
  // to be split are stacked in one register, eight bits each: the subset and its node's number
  if (tl == 0) {
    uint32_t stack = full | 0x80u, next = 1u;  // (the top byte's bit 7 marks an entry)
    while (stack) {
      const uint32_t S = stack & 31u, me = stack >> 5 & 3u;
      stack >>= 8;
      const uint32_t P = S == 31u ? full_split : W.split[S];
      uint32_t node = p;
#pragma unroll
      for (int q = 1; q < kTreeletLeaves - 1; ++q)
        if ((uint32_t)q == me) node = inner[q];
      if (S != 31u) W.node[S] = (uint8_t)me;
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        const uint32_t X = k == 0 ? P : S ^ P;
        uint32_t c;
        if ((X & (X - 1u)) == 0u) {
          c = leaf[0];
#pragma unroll
          for (int q = 1; q < kTreeletLeaves; ++q)
            if (X == (1u << q)) c = leaf[q];
        } else {
          c = inner[1];
#pragma unroll
          for (int q = 2; q < kTreeletLeaves - 1; ++q)
            if ((uint32_t)q == next) c = inner[q];
          stack = stack << 8 | (X | next << 5 | 0x80u);
          ++next;
        }
        L.kid[node][k] = (uint16_t)c;
      }
    }
  }
  lds_order();
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const uint32_t me = set[k] <= full ? W.node[set[k]] : 0xFFu;
    if (me != 0xFFu) {
      uint32_t node = p;
#pragma unroll
      for (int q = 1; q < kTreeletLeaves - 1; ++q)
        if ((uint32_t)q == me) node = inner[q];
#pragma unroll
      for (int a = 0; a < 6; ++a) L.box[node][a] = box[k][a];
      L.area[node] = half_area(box[k]);
      L.cost[node] = own[k];
      L.count[node] = (uint16_t)cnt[k];
    }
  }
  lds_order();
}

template <int NS>
__global__ void __launch_bounds__(NS) k_treelet(int64_t m, const uint32_t* __restrict__ roots,
                                                const uint32_t* __restrict__ n_roots, const uint2* __restrict__ range,
                                                uint32_t* __restrict__ child, uint32_t* __restrict__ parent,
                                                float* __restrict__ boxes, float* __restrict__ cost,
                                                uint32_t* __restrict__ count, int passes, uint32_t* depth) {
  __shared__ SubtreeLds<NS> L;
  const int64_t nint = m - 1;
  const uint32_t nr = *n_roots;
  const int tid = threadIdx.x, tl = tid & (kTeam - 1), team = tid / kTeam;
  for (uint32_t item = blockIdx.x; item < nr; item += gridDim.x) {
    const uint32_t r = roots[item];
    const bool inner_root = (int64_t)r < nint;
    const int64_t lo = inner_root ? (int64_t)range[r].x : (int64_t)r - nint;
    const int n = inner_root ? (int)(range[r].y - range[r].x + 1u) : 1;
    const int64_t first = (int64_t)r == lo ? lo : lo + 1;  // internal node 0 of the subtree
    __syncthreads();  // (the subtree before this one is written back)
    if (tid < n) {
      const int64_t u = nint + lo + tid;
      const int v = n - 1 + tid;
      float b[6];
#pragma unroll
      for (int a = 0; a < 6; ++a) L.box[v][a] = b[a] = boxes[6 * u + a];
      L.area[v] = half_area(b);
      L.cost[v] = kCostLeaf * L.area[v];
      L.count[v] = 1;
      if (cost) cost[u] = L.cost[v];
    }
    if (tid < n - 1) {
      const int64_t u = first + tid;
      float b[6];
#pragma unroll
      for (int a = 0; a < 6; ++a) L.box[tid][a] = b[a] = boxes[6 * u + a];
      L.area[tid] = half_area(b);
      L.count[tid] = (uint16_t)count[u];
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        const uint32_t c = child[2 * u + k];
        L.kid[tid][k] = (uint16_t)((c & kLeafFlag) ? (int64_t)(c & ~kLeafFlag) - lo + n - 1 : (int64_t)c - first);
      }
    }
    __syncthreads();
    // the depth of the whole tree: this subtree's height below the nodes above it
    auto measure = [&](uint32_t h) __attribute__((always_inline)) {
      for (uint32_t q = parent[r]; q != kNoParent; q = parent[q]) ++h;
      atomicMax(depth, h);
    };
    if (n < 3) {
      if (n == 2 && tid == 0 && cost)  // (summed as the last pass below does)
        cost[first] = passes > 1 ? kCostNode * L.area[0] + L.cost[1] + L.cost[2]
                                 : kCostNode * set_area(L.box[0]) + (L.cost[1] + L.cost[2]);
      if (tid == 0 && depth) measure((uint32_t)n - 1u);
      continue;
    }
    const uint32_t root = (uint32_t)((int64_t)r - first);
    // heights: internal nodes on the longest path down from each node, itself included
    auto find_heights = [&]() __attribute__((always_inline)) {
      if (tid < n - 1) {
        L.par[L.kid[tid][0]] = (uint16_t)tid;
        L.par[L.kid[tid][1]] = (uint16_t)tid;
        L.height[tid] = 0u;
      }
      __syncthreads();
      if (tid == 0) L.par[root] = kNoLocal;
      __syncthreads();
      if (tid < n) {
        uint32_t q = L.par[n - 1 + tid], d = 1u;
        while (q != kNoLocal && atomicMax(&L.height[q], d) < d) {
          ++d;
          q = L.par[q];
        }
      }
      __syncthreads();
    };
    for (int pass = 0; pass < passes; ++pass) {
      const uint32_t min_leaves = pass == 0 ? 0u : kLaterPassLeaves << (pass - 1);
      // the nodes listed by height
      for (int i = tid; i < NS + 1; i += NS) L.first[i] = 0u;
      find_heights();
      if (tid < n - 1) {
        atomicAdd(&L.first[L.height[tid]], 1u);
        if (tid == (int)root) L.max_height = L.height[tid];
      }
      __syncthreads();
      const uint32_t top = L.max_height;
      if (tid == 0) {
        uint32_t run = 0u;
        for (uint32_t h = 1u; h <= top; ++h) {
          const uint32_t c = L.first[h];
          L.first[h] = run;
          run += c;
        }
      }
      __syncthreads();
      if (tid < n - 1) L.list[atomicAdd(&L.first[L.height[tid]], 1u)] = (uint16_t)tid;
      __syncthreads();
      // (first[h] is now the end of height h, so the start of height h + 1)
      for (uint32_t h = 1u; h <= top; ++h) {
        const uint32_t beg = h == 1u ? 0u : L.first[h - 1], end = L.first[h];
        for (uint32_t i = beg + (uint32_t)tid; i < end; i += NS) {
          const uint32_t p = L.list[i];
          const float c0 = L.cost[L.kid[p][0]], c1 = L.cost[L.kid[p][1]];
          if (min_leaves != 0u && L.count[p] < min_leaves) L.cost[p] = kCostNode * L.area[p] + c0 + c1;
          else if (L.count[p] == 2u) L.cost[p] = kCostNode * set_area(L.box[p]) + (c0 + c1);
        }
        for (uint32_t i = beg + (uint32_t)team; i < end; i += NS / kTeam) {
          const uint32_t p = L.list[i];
          const uint32_t c = L.count[p];
          if (c > 2u && c >= min_leaves) team_restructure<NS>(L, L.team[team], n, p, tl);
        }
        __syncthreads();
      }
    }
    if (tid < n - 1) {
      const int64_t u = first + tid;
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        const uint32_t c = L.kid[tid][k];
        const bool is_leaf = c >= (uint32_t)(n - 1);
        child[2 * u + k] = is_leaf ? kLeafFlag | (uint32_t)(lo + c - (uint32_t)(n - 1)) : (uint32_t)(first + c);
        parent[is_leaf ? nint + lo + c - (uint32_t)(n - 1) : first + c] = (uint32_t)u;
      }
#pragma unroll
      for (int a = 0; a < 6; ++a) boxes[6 * u + a] = L.box[tid][a];
      count[u] = L.count[tid];
      if (cost) cost[u] = L.cost[tid];
    }
    if (depth) {
      find_heights();
      if (tid == 0) measure(L.height[root]);
    }
  }
}

// The nodes above the subtrees, in a second pass for trees of more than kTopPassLeaves
// leaves (below that the top part is a few hundred nodes and the pass costs more than it
// saves): a thread per subtree root walks up, the second arrival at a node restructures
// it. Threads of different workgroups hand over here, so the counters are agent-scope
// atomics in global memory.
constexpr int64_t kTopPassLeaves = (int64_t)1 << 20;
template <int NS>
__global__ void __launch_bounds__(NS) k_treelet_top(int64_t m, const uint32_t* __restrict__ roots,
                                                                const uint32_t* __restrict__ n_roots,
                                                                uint32_t* child, uint32_t* parent, float* boxes,
                                                                float* cost, uint32_t* count,
                                                                uint32_t* arrivals) {
  __shared__ TreeletLds<NS> L;
  const int tid = threadIdx.x;
  const int64_t k = blockIdx.x * (int64_t)NS + tid;
  if (k >= (int64_t)*n_roots) return;
  const int64_t nint = m - 1;
  uint32_t p = parent[roots[k]];
  while (p != kNoParent) {
    if (__hip_atomic_fetch_add(arrivals + p, 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT) == 0u) return;
    restructure(p, nint, child, parent, boxes, cost, count, L, tid);
    p = parent[p];
  }
}


// ------------------------------------------------------------------ tree depth
// Depth of the tree in internal nodes on the longest root-to-leaf path, which bounds the
// trace's traversal stack (a four-wide record leaves at most three entries pending per
// level). One thread per leaf climbs towards the root carrying the number of internal
// nodes below it on its path and raises the per-node maximum `h`; it stops where a path at
// least as long has already been recorded, so most climbs end after a few steps. The
// root is node 0. A climb longer than `cap` stops there and records cap + 1 at the root
// (the tree is then too deep whatever its exact depth). With `depth` it runs only where that
// is beyond max_depth. (Up to 2^20 leaves the restructuring pass measures its tree itself.)
__global__ void __launch_bounds__(kBlock) k_tree_height(int64_t m, const uint32_t* __restrict__ parent,
                                                        uint32_t* __restrict__ h, int cap,
                                                        const uint32_t* __restrict__ depth, int max_depth) {
  if (depth && *depth <= (uint32_t)max_depth) return;
  const int64_t i = blockIdx.x * (int64_t)kBlock + threadIdx.x;
  if (i >= m) return;
  uint32_t p = parent[(m - 1) + i];
  uint32_t d = 1;
  while (p != kNoParent) {
    if (d > (uint32_t)cap) {
      atomicMax(h, (uint32_t)cap + 1u);
      return;
    }
    if (atomicMax(h + p, d) >= d) return;
    ++d;
    p = parent[p];
  }
}

}  // namespace

// Build over `n` points (centroids) whose leaf boxes/records are produced by `leaves`.
// Icosahedron of inradius 1, from its definition: the 12 points (0,+-1,+-phi) and their
// cyclic permutations; faces are the vertex triples at mutual distance 2 (the edge), wound
// so that (B-A) x (C-A) points away from the centre; scaled so face planes are at distance 1.
static Ico make_icosahedron() {
  const double phi = 0.5 * (1.0 + std::sqrt(5.0));
  double v[12][3];
  int nv = 0;
  for (int sa = -1; sa <= 1; sa += 2)
    for (int sb = -1; sb <= 1; sb += 2) {
      const double p[3] = {0.0, (double)sa, sb * phi};
      for (int rot = 0; rot < 3; ++rot) {
        for (int a = 0; a < 3; ++a) v[nv][a] = p[(a + 3 - rot) % 3];
        ++nv;
      }
    }
  Ico ico{};
  int nf = 0;
  double inr = 0.0;
  for (int i = 0; i < 12; ++i)
    for (int j = i + 1; j < 12; ++j)
      for (int k = j + 1; k < 12; ++k) {
        auto d2 = [&](int x, int y) {
          double s2 = 0.0;
          for (int a = 0; a < 3; ++a) s2 += (v[x][a] - v[y][a]) * (v[x][a] - v[y][a]);
          return s2;
        };
        if (std::fabs(d2(i, j) - 4.0) > 1e-9 || std::fabs(d2(j, k) - 4.0) > 1e-9 || std::fabs(d2(i, k) - 4.0) > 1e-9)
          continue;
        double e1[3], e2[3], nrm[3], cen = 0.0;
        for (int a = 0; a < 3; ++a) {
          e1[a] = v[j][a] - v[i][a];
          e2[a] = v[k][a] - v[i][a];
        }
        nrm[0] = e1[1] * e2[2] - e1[2] * e2[1];
        nrm[1] = e1[2] * e2[0] - e1[0] * e2[2];
        nrm[2] = e1[0] * e2[1] - e1[1] * e2[0];
        for (int a = 0; a < 3; ++a) cen += nrm[a] * v[i][a];
        bool out = cen > 0.0;
        ico.f[nf][0] = (unsigned char)i;
        ico.f[nf][1] = (unsigned char)(out ? j : k);
        ico.f[nf][2] = (unsigned char)(out ? k : j);
        double nl = std::sqrt(nrm[0] * nrm[0] + nrm[1] * nrm[1] + nrm[2] * nrm[2]);
        inr = std::fabs(cen) / nl;
        ++nf;
      }
  for (int i = 0; i < 12; ++i)
    for (int a = 0; a < 3; ++a) ico.v[i][a] = (float)(v[i][a] / inr);
  return ico;
}

struct ScratchArena {
  char* base = nullptr;
  size_t cap = 0;
  size_t top = 0;      // bytes handed out from the arena
  size_t logical = 0;  // bytes handed out in total, overflow included
  size_t high = 0;     // largest `logical` seen
  int depth = 0;       // live Scratch objects
};

namespace {
std::mutex g_arena_lock;
std::map<std::pair<int, hipStream_t>, ScratchArena> g_arenas;
}  // namespace

Scratch::Scratch(hipStream_t s) : s_(s) {
  int dev = 0;
  (void)hipGetDevice(&dev);
  {
    std::lock_guard<std::mutex> g(g_arena_lock);
    arena_ = &g_arenas[{dev, s}];
  }
  mark_ = arena_->top;
  logical_mark_ = arena_->logical;
  ++arena_->depth;
}

grtx_status Scratch::raw(void** p, size_t bytes) {
  bytes = (bytes + 255) & ~(size_t)255;
  ScratchArena& a = *arena_;
  a.logical += bytes;
  a.high = std::max(a.high, a.logical);
  if (a.base && a.top + bytes <= a.cap) {
    *p = a.base + a.top;
    a.top += bytes;
    return GRTX_OK;
  }
  void* q = nullptr;
  GRTX_HIP(hipMallocAsync(&q, bytes, s_));
  extra_.push_back(q);
  *p = q;
  return GRTX_OK;
}

Scratch::~Scratch() {
  for (void* q : extra_) (void)hipFreeAsync(q, s_);
  ScratchArena& a = *arena_;
  a.top = mark_;
  a.logical = logical_mark_;
  if (--a.depth == 0 && a.high > a.cap) {
    if (a.base) (void)hipFreeAsync(a.base, s_);
    a.base = nullptr;
    a.cap = 0;
    const size_t want = a.high + a.high / 4;
    void* q = nullptr;
    if (hipMallocAsync(&q, want, s_) == hipSuccess) {
      a.base = static_cast<char*>(q);
      a.cap = want;
    } else {
      (void)hipGetLastError();
    }
  }
}

grtx_status build_bvh(const grtx_gaussians* g, grtx_bvh_kind kind, float alpha_min, bool restructure_tree,
                      int max_depth, hipStream_t s, Bvh* b) {
  b->kind = kind;
  b->n_gauss = g->count;
  b->sh_degree = g->sh_degree;
  b->alpha_min = alpha_min;
  b->opacities = g->opacities;
  b->sh = g->sh;
  b->build_stream = s;
  GRTX_HIP(hipGetDevice(&b->device));
  const bool proxy = kind == GRTX_BVH_PROXY20;
  const int64_t n = g->count;
  const int64_t m = proxy ? 20 * n : n;  // leaves
  b->n_leaves = m;
  if (n == 0) return GRTX_OK;
  GaussIn gi{g->means, g->scales, g->quats, g->opacities};
  const int64_t nint = m - 1;
  // node record positions: the top levels in [0, top_cap), then one block per subtree task
  // (a tree's nodes above kLayoutLeaves leaves can number up to m - 1 when it is lopsided)
  const int64_t top_cap = m > kLayoutLeaves ? m : 0;
  const int64_t node_slots = nint > 0 ? top_cap + m : 0;
  if (node_slots >= (int64_t)kLeafFlag) {
    set_error("build: %lld leaves exceed the node positions a record reference can hold", (long long)m);
    return GRTX_ERR_INVALID_ARG;
  }
  b->node_slots = node_slots;
  // every array the handle owns in one allocation (each hipMalloc costs host time per frame)
  auto layout = [&](auto&& put) {
    put(&b->codes, m);
    put(&b->perm, m);
    put(&b->child, 2 * std::max<int64_t>(nint, 1));
    put(&b->parent, 2 * m - 1);
    put(&b->boxes, 6 * (2 * m - 1));
    put(&b->nodes, kNodeF4 * std::max<int64_t>(node_slots, 1));
    put(&b->inst, 4 * n);
    if (proxy) put(&b->tris, 3 * m);
    put(&b->roots, 8);
    put(&b->cut, 2 * (int64_t)kCutCap);
    put(&b->depth, 4);  // depth and kind, then the cut's length and a counter of the build's
    put(&b->density, kDensityCells);
    put(&b->dbox, 6);
  };
  size_t total = 0;
  layout([&](auto** p, int64_t count) {
    total = (total + 255) & ~(size_t)255;
    total += (size_t)std::max<int64_t>(count, 1) * sizeof(**p);
  });
  void* block = nullptr;
  GRTX_HIP(hipMalloc(&block, total));
  b->allocations.push_back(block);
  b->bytes += total;
  size_t off = 0;
  layout([&](auto** p, int64_t count) {
    off = (off + 255) & ~(size_t)255;
    *p = reinterpret_cast<std::remove_reference_t<decltype(*p)>>(static_cast<char*>(block) + off);
    off += (size_t)std::max<int64_t>(count, 1) * sizeof(**p);
  });
  b->n_cut = b->depth + 2;
  b->root_box = b->boxes;  // node 0: the root, or the only leaf when m == 1

  Scratch sc(s);
  float *partial = nullptr, *bounds = nullptr, *cent = nullptr, *tbox = nullptr;
  float4* ttmp = nullptr;
  uint64_t* tkeys = nullptr;
  uint32_t* tvals = nullptr;
  int nparts = (int)std::min<int64_t>(256, (m + kBlock - 1) / kBlock);
  FinishArgs fin{b->root_box, m == 1 ? kLeafFlag : 0u, b->roots, nullptr, max_depth, nullptr, b->depth};
  GRTX_TRY(sc.get(&partial, 6 * nparts));
  GRTX_TRY(sc.get(&bounds, 6));
  GRTX_TRY(sc.get(&tkeys, m));
  GRTX_TRY(sc.get(&tvals, m));
  uint2* range = nullptr;
  uint32_t* count = nullptr;  // leaves below each internal node
  GRTX_TRY(sc.get(&range, std::max<int64_t>(nint, 1)));
  GRTX_TRY(sc.get(&count, std::max<int64_t>(nint, 1)));
  // cleared with the first kernel: the tree's depth (two words), the cut's length, and the
  // number of subtrees the restructuring pass takes
  uint32_t* const counters = b->depth;
  uint32_t* const n_roots = b->depth + 3;
  const float* points = g->means;
  if (proxy) {
    GRTX_TRY(sc.get(&cent, 3 * m));
    GRTX_TRY(sc.get(&tbox, 6 * m));
    GRTX_TRY(sc.get(&ttmp, 3 * m));
    static const Ico ico = make_icosahedron();
    hipLaunchKernelGGL(k_proxy_setup, dim3(grid_for(n)), dim3(kBlock), 0, s, gi, n, alpha_min, ico, b->inst, ttmp,
                       tbox, cent);
    points = cent;
  }
  hipLaunchKernelGGL(k_bounds_partial, dim3(nparts), dim3(kBlock), 0, s, points, m, partial,
                     reinterpret_cast<uint4*>(b->density), counters, 4);
  hipLaunchKernelGGL(k_morton, dim3(std::min(grid_for(m), 2048u)), dim3(kBlock), 0, s, points, m, partial, nparts, bounds,
                     b->dbox, b->codes);
  GRTX_LAUNCH_CHECK();
  // (eight passes: the result is where the codes were)
  GRTX_TRY((radix_sort<uint64_t, 8>(b->codes, b->perm, tkeys, tvals, m, sc, s, 8, nullptr, &b->codes, &b->perm)));
  if (proxy) {
    hipLaunchKernelGGL(k_proxy_leaves, dim3(grid_for(m)), dim3(kBlock), 0, s, b->perm, m, ttmp, tbox, b->tris,
                       b->boxes, cent, bounds, b->density);
  } else {
    float box_scale = 1.f;
    if (kind == GRTX_BVH_ICO_INSTANCE) {
      static const Ico ico = make_icosahedron();
      box_scale = std::sqrt(ico.v[0][0] * ico.v[0][0] + ico.v[0][1] * ico.v[0][1] + ico.v[0][2] * ico.v[0][2]);
    }
    hipLaunchKernelGGL(k_sphere_leaves, dim3(grid_for(m)), dim3(kBlock), 0, s, gi, b->perm, m, alpha_min, box_scale,
                       b->inst, b->boxes, bounds, b->density);
  }
  const uint32_t* tree_depth = nullptr;   // of the restructured tree
  const uint32_t* plain_depth = nullptr;
  if (nint > 0) {
    // boxes of 2, 4, 8, ... leaves
    BoxLevels lv{};
    lv.leaves = b->boxes + 6 * nint;
    lv.size[0] = m;
    lv.count = 1;
    int64_t total_up = 0;
    while (lv.size[lv.count - 1] > 1) {
      lv.at[lv.count] = total_up;
      lv.size[lv.count] = (lv.size[lv.count - 1] + 1) / 2;
      total_up += lv.size[lv.count++];
    }
    GRTX_TRY(sc.get(&lv.up, 6 * total_up));
    for (int from = 0; from + 1 < lv.count; from += 8)
      hipLaunchKernelGGL(k_box_levels, dim3(grid_for(lv.size[from])), dim3(kBlock), 0, s, lv, from);
    // (beyond one scan's reach neither restructuring nor the cut: the plain tree, and the trace
    // keeps its centre-out order)
    const bool reach = 2 * m - 1 <= (int64_t)kScanChunk * kScanChunk;
    const bool restructure = restructure_tree && nint > 1 && reach;
    const int ns = subtree_leaves(m);
    TopologyOut to{b->child, b->parent, range, count, b->boxes, nullptr, n_roots, b->cut, b->n_cut, nullptr};
    if (restructure) GRTX_TRY(sc.get(&to.roots, m));
    hipLaunchKernelGGL(k_topology, dim3(grid_for(nint)), dim3(kBlock), 0, s, b->codes, m, lv, to,
                       restructure ? (uint32_t)ns : 0u, reach ? (uint32_t)std::max<int64_t>(1, m / kCutDiv) : 0u,
                       (const uint32_t*)nullptr, 0);
    uint32_t* heights = nullptr;
    if (restructure) {
      // a workgroup per subtree, which mostly hold more than half of `ns` leaves (a stride over
      // the list takes any more); the costs are kept where the nodes above them need them
      const unsigned groups = (unsigned)std::min<int64_t>(m / (ns / 2) + 1, 1 << 16);
      const bool top_pass = m > kTopPassLeaves;
      float* costs = nullptr;
      if (top_pass) GRTX_TRY(sc.get(&costs, 2 * m - 1));
      if (ns == 256)
        hipLaunchKernelGGL(k_treelet<256>, dim3(groups), dim3(256), 0, s, m, to.roots, n_roots, range, b->child,
                           b->parent, b->boxes, costs, count, treelet_passes(m), top_pass ? nullptr : b->depth);
      else
        hipLaunchKernelGGL(k_treelet<128>, dim3(groups), dim3(128), 0, s, m, to.roots, n_roots, range, b->child,
                           b->parent, b->boxes, costs, count, treelet_passes(m), top_pass ? nullptr : b->depth);
      tree_depth = b->depth;
      if (top_pass) {
        uint32_t *arrivals = nullptr, *th = nullptr;
        GRTX_TRY(sc.get(&arrivals, nint));
        GRTX_TRY(sc.get(&th, nint));
        hipLaunchKernelGGL(k_fill_u32, dim3(grid_for(nint)), dim3(kBlock), 0, s, arrivals, nint, 0u);
        hipLaunchKernelGGL(k_fill_u32, dim3(grid_for(nint)), dim3(kBlock), 0, s, th, nint, 0u);
        const unsigned top_groups = (unsigned)((m + ns - 1) / ns);
        hipLaunchKernelGGL(k_treelet_top<128>, dim3(top_groups), dim3(128), 0, s, m, to.roots, n_roots, b->child,
                           b->parent, b->boxes, costs, count, arrivals);
        hipLaunchKernelGGL(k_tree_height, dim3(grid_for(m)), dim3(kBlock), 0, s, m, b->parent, th, max_depth,
                           (const uint32_t*)nullptr, 0);
        tree_depth = th;
      }
      // too deep: the plain tree again
      GRTX_TRY(sc.get(&heights, nint));
      to.heights = heights;
      hipLaunchKernelGGL(k_topology, dim3(grid_for(nint)), dim3(kBlock), 0, s, b->codes, m, lv, to, 0u, 0u, tree_depth,
                         max_depth);
    } else {
      GRTX_TRY(sc.get(&heights, nint));
      hipLaunchKernelGGL(k_fill_u32, dim3(grid_for(nint)), dim3(kBlock), 0, s, heights, nint, 0u);
    }
    hipLaunchKernelGGL(k_tree_height, dim3(grid_for(m)), dim3(kBlock), 0, s, m, b->parent, heights, GRTX_MAX_TREE_DEPTH,
                       tree_depth, max_depth);
    plain_depth = heights;
    // four-wide records of every internal node, then the reachable ones laid out
    float4* wide = nullptr;
    uint32_t *qold = nullptr, *ctr = nullptr;
    uint2* tasks = nullptr;
    GRTX_TRY(sc.get(&wide, kNodeF4 * nint));
    GRTX_TRY(sc.get(&qold, node_slots));
    GRTX_TRY(sc.get(&tasks, m));
    GRTX_TRY(sc.get(&ctr, 2));
    uint4* counts = nullptr;
    GRTX_TRY(sc.get(&counts, nint));
    hipLaunchKernelGGL(k_wide, dim3(grid_for(nint)), dim3(kBlock), 0, s, m, b->child, b->boxes, count, wide, counts);
    fin.tree = tree_depth;
    fin.plain = plain_depth;
    hipLaunchKernelGGL(k_layout_top, dim3(1), dim3(kLayoutBlock), 0, s, m, wide, counts, (uint32_t)top_cap, b->nodes,
                       qold, tasks, ctr, fin);
    // a wave per task; the tasks number about m / 64 (a grid-stride loop takes any more)
    hipLaunchKernelGGL(k_layout_tasks, dim3((unsigned)std::min<int64_t>(2048, m / (64 * (kBlock / 64)) + 1)),
                       dim3(kBlock), 0, s, wide, tasks, ctr, b->nodes);
  } else {
    hipLaunchKernelGGL(k_fill_u32, dim3(1), dim3(kBlock), 0, s, b->parent, 1, kNoParent);
    hipLaunchKernelGGL(k_finish, dim3(1), dim3(64), 0, s, fin);
  }
  GRTX_LAUNCH_CHECK();
  return GRTX_OK;
}

grtx_status export_topology(const Bvh* b, uint32_t* child, uint32_t* parent, uint64_t* morton, uint32_t* perm,
                            float* boxes, hipStream_t s) {
  const int64_t n = b->n_leaves;
  if (n == 0) return GRTX_OK;
  const int64_t nint = n - 1;
  if (child && nint > 0) GRTX_HIP(hipMemcpyAsync(child, b->child, sizeof(uint32_t) * 2 * nint, hipMemcpyDeviceToDevice, s));
  if (parent) GRTX_HIP(hipMemcpyAsync(parent, b->parent, sizeof(uint32_t) * (2 * n - 1), hipMemcpyDeviceToDevice, s));
  if (morton) GRTX_HIP(hipMemcpyAsync(morton, b->codes, sizeof(uint64_t) * n, hipMemcpyDeviceToDevice, s));
  if (perm) GRTX_HIP(hipMemcpyAsync(perm, b->perm, sizeof(uint32_t) * n, hipMemcpyDeviceToDevice, s));
  if (boxes) GRTX_HIP(hipMemcpyAsync(boxes, b->boxes, sizeof(float) * 6 * (2 * n - 1), hipMemcpyDeviceToDevice, s));
  return GRTX_OK;
}

grtx_status pinhole_rays(const grtx_camera* cam, float* origins, float* dirs, hipStream_t s) {
  CameraFrame cf;
  if (!camera_frame(cam->eye, cam->target, cam->up, cam->fov_y_deg, cam->width, cam->height, &cf)) {
    set_error("pinhole camera: degenerate eye/target/up");
    return GRTX_ERR_INVALID_ARG;
  }
  int64_t n = (int64_t)cam->width * cam->height;
  hipLaunchKernelGGL(k_pinhole, dim3(grid_for(n)), dim3(kBlock), 0, s, cf, cam->width, cam->height, origins, dirs);
  GRTX_LAUNCH_CHECK();
  return GRTX_OK;
}

grtx_status exclusive_scan_u32(const uint32_t* in, uint32_t* out, int64_t n, hipStream_t s) {
  if (n <= 0) return GRTX_OK;
  Scratch sc(s);
  const int nparts = (int)((n + kScanChunk - 1) / kScanChunk);
  if (nparts > kScanChunk) {
    set_error("scan: %lld values exceed the supported size", (long long)n);
    return GRTX_ERR_INVALID_ARG;
  }
  if (nparts > 1 && nparts <= kScanLoopChunks) {
    hipLaunchKernelGGL(k_scan_loop, dim3(1), dim3(kBlock), 0, s, in, n, out);
  } else if (nparts > 1) {
    uint32_t* part = nullptr;
    GRTX_TRY(sc.get(&part, nparts));
    hipLaunchKernelGGL(k_scan_reduce, dim3(nparts), dim3(kBlock), 0, s, in, n, part);
    hipLaunchKernelGGL(k_scan_partials, dim3(1), dim3(kBlock), 0, s, part, nparts);
    hipLaunchKernelGGL(k_scan_down, dim3(nparts), dim3(kBlock), 0, s, in, n, part, out);
  } else {
    hipLaunchKernelGGL(k_scan_down, dim3(1), dim3(kBlock), 0, s, in, n, (const uint32_t*)nullptr, out);
  }
  GRTX_LAUNCH_CHECK();
  return GRTX_OK;
}

grtx_status sort_positions(uint32_t* keys, uint32_t* vals, uint32_t* tkeys, uint32_t* tvals, int64_t n, int key_bits,
                           hipStream_t s, const uint32_t* n_dev, uint32_t** kres, uint32_t** vres) {
  *kres = keys;
  *vres = vals;
  if (n <= 0) return GRTX_OK;
  Scratch sc(s);
  // Nine bits a pass where that saves one (65k to 262k Gaussians: two passes of 115 us instead of
  // three of 109 us for 10.7M keys); a workgroup's digits then go two to a thread.
  const int by8 = std::max(1, (key_bits + 7) / 8), by9 = std::max(1, (key_bits + 8) / 9);
  if (by9 < by8) return radix_sort<uint32_t, 9>(keys, vals, tkeys, tvals, n, sc, s, by9, n_dev, kres, vres);
  return radix_sort<uint32_t, 8>(keys, vals, tkeys, tvals, n, sc, s, by8, n_dev, kres, vres);
}

}  // namespace grtx
