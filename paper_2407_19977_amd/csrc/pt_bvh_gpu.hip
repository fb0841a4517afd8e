// GPU construction of the BVH4 for gfx950 (the paper builds its BVH on the
// CPU once per scene and times that set-up separately, Sec. 5.1.1, Table 1).
//
// Two builders share the first and last steps:
//   1. triangle boxes, and the centroid bounds by a block reduction;
//   2. 30-bit Morton codes (10 bits per axis) of the centroids in cubic
//      cells (one scale, that of the centroid box's longest side, for all
//      three axes, so that neighbours along the curve are near in space);
//   3. an LSD radix sort of (code, index): four 8-bit passes, each a tile
//      histogram, one scan over (digit, tile) and a stable scatter that ranks
//      equal digits with wave ballots;
//   then a binary tree over the sorted triangles, either
//   4a. linear BVH (Karras 2012): the binary radix tree over the sorted codes,
//      every internal node in parallel (ties between equal codes broken by
//      the index), and node boxes bottom-up (each leaf walks towards the root
//      and the second thread to reach a node merges its children's boxes); or
//   4b. locally-ordered clustering (PLOC, Meister & Bittner 2018): clusters
//      in Morton order, each finds the neighbour within kPlocRadius places
//      whose merged box has the least surface area, mutual nearest
//      neighbours merge into a new node, the rest are compacted in order,
//      until one cluster is left (a greedy bottom-up SAH tree);
//   5. a top-down collapse to 128-byte BVH4 nodes, one launch per level, by
//      least SAH cost (the dynamic program of Ylitie, Karras and Laine 2017,
//      its costs computed where the binary nodes are made): a 4-wide node
//      takes the roots of the best split of its four slots; leaf subtrees
//      place their triangles in depth-first order;
//   6. the 48-byte triangle records in that (leaf) order.
// The result has the layout of the host builder's (root at node 0, empty
// child slots kEmpty with zero boxes, meta[0] = child count); only the tree
// differs.  Every closest hit is the same, since the hit is defined by the
// triangle test alone.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <vector>

#include "pt_internal.h"

namespace pt {
namespace {

constexpr int kBB = 256;               // threads per block
constexpr int kItems = 8;              // keys per thread and radix pass
constexpr int kTile = kBB * kItems;    // keys per radix tile
constexpr uint32_t kLeafRef = 0x80000000u;  // binary-tree child reference: leaf flag
constexpr int kMaxTreeLevels = 128;          // bound on any walk or level loop over the binary tree
#ifndef PT_PLOC_RADIUS
#define PT_PLOC_RADIUS 16
#endif
constexpr int kPlocRadius = PT_PLOC_RADIUS;  // clusters searched on either side
#ifndef PT_MORTON_CUBE
#define PT_MORTON_CUBE 1  // 1: Morton cells are cubes (one scale for the three axes), 0: one scale per axis
#endif
constexpr int kPlocMaxRounds = 4096;         // bound on the clustering rounds
// blocks of a clustering round up to which its merge kernel adds up the counts of the blocks before
// it itself; above, two scan launches (about 8 us) cost less than reading half of them in every block
constexpr int kPlocSumBlocks = 8192;
// blocks of the bounds reduction at most: each ends with six atomics on one line, 11 ns apiece
// (8192 blocks 123 us for 1.31M triangles)
constexpr int kBoundsGrid = 1024;
constexpr int kPlocBatch = 8;                // rounds enqueued between two reads of the cluster count
constexpr int kCollapseBatch = 8;            // collapse levels enqueued between two reads of the job count
#ifndef PT_GPU_COLLAPSE_DP
#define PT_GPU_COLLAPSE_DP 1
#endif
// 1: BVH4 nodes by least SAH cost over the binary tree; 0: each node opens its largest-area children
constexpr bool kGpuCollapseDp = PT_GPU_COLLAPSE_DP != 0;
#ifndef PT_SAH_TRAVERSAL
#define PT_SAH_TRAVERSAL 1.0
#endif
constexpr float kSahNode = (float)PT_SAH_TRAVERSAL;  // a node step, in triangle tests
// binary-node triangle counts carry this bit when the subtree becomes one BVH4 leaf
constexpr uint32_t kLeafBitCnt = 0x80000000u;

// Float <-> order-preserving unsigned, for atomic min / max of floats.
__device__ inline uint32_t f2ord(float f) {
  uint32_t u = __float_as_uint(f);
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}
__device__ inline float ord2f(uint32_t u) { return __uint_as_float((u & 0x80000000u) ? (u & 0x7FFFFFFFu) : ~u); }

__device__ inline uint32_t spread10(uint32_t v) {  // the 10 low bits of v to every third bit
  v &= 0x3FFu;
  v = (v | (v << 16)) & 0x030000FFu;
  v = (v | (v << 8)) & 0x0300F00Fu;
  v = (v | (v << 4)) & 0x030C30C3u;
  v = (v | (v << 2)) & 0x09249249u;
  return v;
}

// 1. boxes [n][6] (lo xyz, hi xyz) and centroid bounds cb[6] (ordered min xyz, max xyz)
__global__ __launch_bounds__(kBB) void k_tri_boxes(const float* __restrict__ soup, int64_t n, float* __restrict__ box,
                                                   uint32_t* __restrict__ cb) {
  __shared__ float red[6][kBB];
  float cmin[3] = {INFINITY, INFINITY, INFINITY}, cmax[3] = {-INFINITY, -INFINITY, -INFINITY};
  for (int64_t i = blockIdx.x * (int64_t)kBB + threadIdx.x; i < n; i += (int64_t)gridDim.x * kBB) {
    const float* p = soup + 9 * i;
    float lo[3], hi[3];
    for (int k = 0; k < 3; ++k) {
      lo[k] = fminf(fminf(p[k], p[3 + k]), p[6 + k]);
      hi[k] = fmaxf(fmaxf(p[k], p[3 + k]), p[6 + k]);
      box[6 * i + k] = lo[k];
      box[6 * i + 3 + k] = hi[k];
      const float c = 0.5f * (lo[k] + hi[k]);
      cmin[k] = fminf(cmin[k], c);
      cmax[k] = fmaxf(cmax[k], c);
    }
  }
  for (int k = 0; k < 3; ++k) {
    red[k][threadIdx.x] = cmin[k];
    red[3 + k][threadIdx.x] = cmax[k];
  }
  __syncthreads();
  for (int off = kBB / 2; off > 0; off >>= 1) {
    if ((int)threadIdx.x < off)
      for (int k = 0; k < 3; ++k) {
        red[k][threadIdx.x] = fminf(red[k][threadIdx.x], red[k][threadIdx.x + off]);
        red[3 + k][threadIdx.x] = fmaxf(red[3 + k][threadIdx.x], red[3 + k][threadIdx.x + off]);
      }
    __syncthreads();
  }
  if (threadIdx.x < 3) {
    atomicMin(&cb[threadIdx.x], f2ord(red[threadIdx.x][0]));
    atomicMax(&cb[3 + threadIdx.x], f2ord(red[3 + threadIdx.x][0]));
  }
}

__global__ void k_init_bounds(uint32_t* cb) {
  if (threadIdx.x < 3) cb[threadIdx.x] = 0xFFFFFFFFu;        // min: +inf of the order
  else if (threadIdx.x < 6) cb[threadIdx.x] = 0u;            // max: -inf of the order
}

// 2. Morton code of the centroid normalised to the centroid bounds; value = triangle index
__global__ __launch_bounds__(kBB) void k_morton(const float* __restrict__ box, int64_t n,
                                                const uint32_t* __restrict__ cb, uint32_t* __restrict__ key,
                                                uint32_t* __restrict__ val) {
  float lo[3], sc[3], ext[3], emax = 0.0f;
  for (int k = 0; k < 3; ++k) {
    lo[k] = ord2f(cb[k]);
    ext[k] = ord2f(cb[3 + k]) - lo[k];
    emax = fmaxf(emax, ext[k]);
  }
  for (int k = 0; k < 3; ++k) {
    const float e = PT_MORTON_CUBE ? emax : ext[k];
    sc[k] = e > 0.0f ? 1024.0f / e : 0.0f;
  }
  for (int64_t i = blockIdx.x * (int64_t)kBB + threadIdx.x; i < n; i += (int64_t)gridDim.x * kBB) {
    uint32_t q[3];
    for (int k = 0; k < 3; ++k) {
      const float c = 0.5f * (box[6 * i + k] + box[6 * i + 3 + k]);
      const float t = (c - lo[k]) * sc[k];
      q[k] = (uint32_t)fminf(fmaxf(t, 0.0f), 1023.0f);
    }
    key[i] = (spread10(q[0]) << 2) | (spread10(q[1]) << 1) | spread10(q[2]);
    val[i] = (uint32_t)i;
  }
}

// 3. radix sort passes over tiles of kTile keys (block b: keys [b kTile, (b + 1) kTile))
__global__ __launch_bounds__(kBB) void k_radix_hist(const uint32_t* __restrict__ key, int64_t n, int shift,
                                                    uint32_t* __restrict__ hist, int nb) {
  __shared__ uint32_t h[256];
  h[threadIdx.x] = 0u;
  __syncthreads();
  const int64_t base = (int64_t)blockIdx.x * kTile;
  for (int r = 0; r < kItems; ++r) {
    const int64_t i = base + r * kBB + threadIdx.x;
    if (i < n) atomicAdd(&h[(key[i] >> shift) & 0xFFu], 1u);
  }
  __syncthreads();
  hist[(size_t)threadIdx.x * nb + blockIdx.x] = h[threadIdx.x];
}

// Sum over the block's threads, in every thread (s_w: kBB / 64 words).
template <class T>
__device__ inline T block_sum(T v, T* s_w) {
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
  if (threadIdx.x % 64 == 0) s_w[threadIdx.x / 64] = v;
  __syncthreads();
  T t = 0;
  for (int w = 0; w < kBB / 64; ++w) t += s_w[w];
  __syncthreads();  // s_w may be reused
  return t;
}

// Exclusive scan of m counts in place, tiles of kScanTile counts: the tiles'
// sums, then every block adds up the sums before its own (at most 4096 of
// them for the largest build) and scans its tile from registers.  A single
// workgroup that walked 1024 strided segments took 343 us for the 164K radix
// counts of 1.31M triangles (uncoalesced, one CU); these two launches take 10.
constexpr int kScanPer = 16;
constexpr int kScanTile = kBB * kScanPer;

template <class T>
__global__ __launch_bounds__(kBB) void k_scan_sums(const T* __restrict__ a, int64_t m, T* __restrict__ sums) {
  __shared__ T s_w[kBB / 64];
  const int64_t base = (int64_t)blockIdx.x * kScanTile + threadIdx.x;
  T v = 0;
  for (int r = 0; r < kScanPer; ++r) {
    const int64_t i = base + r * kBB;
    if (i < m) v += a[i];
  }
  v = block_sum(v, s_w);
  if (threadIdx.x == 0) sums[blockIdx.x] = v;
}

template <class T>
__global__ __launch_bounds__(kBB) void k_scan_tiles(T* __restrict__ a, int64_t m, const T* __restrict__ sums) {
  __shared__ T s_w[kBB / 64], s_t[kScanTile];
  T before = 0;
  for (uint32_t k = threadIdx.x; k < blockIdx.x; k += kBB) before += sums[k];
  before = block_sum(before, s_w);
  const int64_t base = (int64_t)blockIdx.x * kScanTile;
  for (int r = 0; r < kScanPer; ++r) {
    const int64_t i = base + r * kBB + threadIdx.x;
    s_t[r * kBB + threadIdx.x] = i < m ? a[i] : T(0);
  }
  __syncthreads();
  T local[kScanPer], sum = 0;  // thread t: counts [t kScanPer, (t + 1) kScanPer) of the tile
  for (int r = 0; r < kScanPer; ++r) {
    local[r] = s_t[threadIdx.x * kScanPer + r];
    sum += local[r];
  }
  T incl = sum;
  for (int off = 1; off < 64; off <<= 1) {
    const T v = __shfl_up(incl, off);
    if ((int)(threadIdx.x % 64) >= off) incl += v;
  }
  if (threadIdx.x % 64 == 63) s_w[threadIdx.x / 64] = incl;
  __syncthreads();
  T run = before + incl - sum;
  for (int w = 0; w < (int)(threadIdx.x / 64); ++w) run += s_w[w];
  for (int r = 0; r < kScanPer; ++r) {
    s_t[threadIdx.x * kScanPer + r] = run;
    run += local[r];
  }
  __syncthreads();
  for (int r = 0; r < kScanPer; ++r) {
    const int64_t i = base + r * kBB + threadIdx.x;
    if (i < m) a[i] = s_t[r * kBB + threadIdx.x];
  }
}

// sums: ceil(m / kScanTile) counts of scratch
template <class T>
void launch_scan(T* a, int64_t m, T* sums, hipStream_t st) {
  const int tiles = (int)((m + kScanTile - 1) / kScanTile);
  if (tiles > 1) hipLaunchKernelGGL(k_scan_sums<T>, dim3(tiles), dim3(kBB), 0, st, a, m, sums);
  hipLaunchKernelGGL(k_scan_tiles<T>, dim3(tiles), dim3(kBB), 0, st, a, m, sums);
}

// Stable scatter: within each round of 256 keys a key's rank among equal
// digits comes from its wave's ballots (lane order) and the counts of the
// waves before it; rounds run in order and carry a per-digit running offset.
__global__ __launch_bounds__(kBB) void k_radix_scatter(const uint32_t* __restrict__ kin,
                                                       const uint32_t* __restrict__ vin, uint32_t* __restrict__ kout,
                                                       uint32_t* __restrict__ vout, int64_t n, int shift,
                                                       const uint32_t* __restrict__ offs, int nb) {
  __shared__ uint32_t run[256];
  __shared__ uint32_t wcnt[kBB / 64][256];
  const int tid = threadIdx.x, wave = tid / 64, lane = tid % 64;
  run[tid] = offs[(size_t)tid * nb + blockIdx.x];
  for (int w = 0; w < kBB / 64; ++w) wcnt[w][tid] = 0u;
  __syncthreads();
  const uint64_t lt = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
  const int64_t base = (int64_t)blockIdx.x * kTile;
  for (int r = 0; r < kItems; ++r) {
    const int64_t i = base + r * kBB + tid;
    const bool valid = i < n;
    const uint32_t k = valid ? kin[i] : 0u, v = valid ? vin[i] : 0u;
    const uint32_t d = (k >> shift) & 0xFFu;
    uint64_t peers = __ballot(valid);
    for (int b = 0; b < 8; ++b) {
      const bool bit = ((d >> b) & 1u) != 0u;
      const uint64_t m = __ballot(bit);
      peers &= bit ? m : ~m;
    }
    const uint32_t rank = (uint32_t)__popcll(peers & lt);
    if (valid && rank == 0u) wcnt[wave][d] = (uint32_t)__popcll(peers);
    __syncthreads();
    if (valid) {
      uint32_t pos = run[d] + rank;
      for (int w = 0; w < wave; ++w) pos += wcnt[w][d];
      kout[pos] = k;
      vout[pos] = v;
    }
    __syncthreads();
    uint32_t tot = 0u;
    for (int w = 0; w < kBB / 64; ++w) {
      tot += wcnt[w][tid];
      wcnt[w][tid] = 0u;
    }
    run[tid] += tot;
    __syncthreads();
  }
}

// 4a. binary radix tree (n - 1 internal nodes).  Child references: leaf
// (kLeafRef | sorted index) or internal node index; parents of leaves and of
// internal nodes (-1 for the root); the number of triangles under each node.
__device__ inline int delta(const uint32_t* key, int64_t n, int64_t i, int64_t j) {
  if (j < 0 || j >= n) return -1;
  const uint32_t a = key[i], b = key[j];
  if (a == b) return 32 + __clz((uint32_t)i ^ (uint32_t)j);
  return __clz(a ^ b);
}

__global__ __launch_bounds__(kBB) void k_radix_tree(const uint32_t* __restrict__ key, int64_t n,
                                                    uint2* __restrict__ child, int32_t* __restrict__ parent_leaf,
                                                    int32_t* __restrict__ parent_int, uint32_t* __restrict__ cnt,
                                                    uint32_t* __restrict__ err) {
  for (int64_t i = blockIdx.x * (int64_t)kBB + threadIdx.x; i < n - 1; i += (int64_t)gridDim.x * kBB) {
    const int d = delta(key, n, i, i + 1) - delta(key, n, i, i - 1) >= 0 ? 1 : -1;
    const int dmin = delta(key, n, i, i - d);
    int64_t lmax = 2;
    while (delta(key, n, i, i + lmax * d) > dmin) lmax <<= 1;
    int64_t l = 0;
    for (int64_t t = lmax >> 1; t >= 1; t >>= 1)
      if (delta(key, n, i, i + (l + t) * d) > dmin) l += t;
    const int64_t j = i + l * d;
    const int dnode = delta(key, n, i, j);
    int64_t s = 0, t = l;
    do {
      t = (t + 1) >> 1;
      if (delta(key, n, i, i + (s + t) * d) > dnode) s += t;
    } while (t > 1);
    const int64_t gamma = i + s * d + (d < 0 ? -1 : 0);
    const int64_t lo = i < j ? i : j, hi = i < j ? j : i;
    if (gamma < lo || gamma + 1 > hi) {  // only unsorted codes could get here: report, write nothing
      atomicOr(err, 1u);
      continue;
    }
    uint32_t cl, cr;
    if (lo == gamma) {
      cl = kLeafRef | (uint32_t)gamma;
      parent_leaf[gamma] = (int32_t)i;
    } else {
      cl = (uint32_t)gamma;
      parent_int[gamma] = (int32_t)i;
    }
    if (hi == gamma + 1) {
      cr = kLeafRef | (uint32_t)(gamma + 1);
      parent_leaf[gamma + 1] = (int32_t)i;
    } else {
      cr = (uint32_t)(gamma + 1);
      parent_int[gamma + 1] = (int32_t)i;
    }
    child[i] = make_uint2(cl, cr);
    const uint32_t c = (uint32_t)(hi - lo + 1);
    cnt[i] = c <= (uint32_t)kMaxLeafTris ? (c | kLeafBitCnt) : c;
  }
}

// box of a binary-tree reference: a leaf's triangle box (sorted index -> triangle) or a node box
__device__ inline void ref_box(uint32_t ref, const uint32_t* val, const float* tbox, const float* nbox, float b[6]) {
  const float* src = (ref & kLeafRef) ? tbox + 6 * (size_t)val[ref & ~kLeafRef] : nbox + 6 * (size_t)ref;
  for (int k = 0; k < 6; ++k) b[k] = src[k];
}

__device__ inline uint32_t ref_count(uint32_t ref, const uint32_t* cnt) {
  return (ref & kLeafRef) ? 1u : (cnt[ref] & ~kLeafBitCnt);
}

// the subtree of `ref` becomes one BVH4 leaf
__device__ inline bool ref_is_leaf_subtree(uint32_t ref, const uint32_t* cnt) {
  return (ref & kLeafRef) || (cnt[ref] & kLeafBitCnt);
}

// Collapse by least SAH cost (as the host builder's): per binary node o,
// dp[4 o + j - 1] is the least cost of covering its subtree with at most
// j = 1..4 roots (a root costs its area times one node step plus its
// children's costs, a leaf its area times its triangles), and dsp[o] holds,
// for j = 2..4 in bits 4 (j - 1) .. 4 (j - 1) + 3, the split of those slots
// (left count in the low two bits, right count in the high two; 0: the node
// is the one root), and in bits 16..19 the split of its own four slots when
// it is a 4-wide node.
__device__ inline void dp_of_ref(uint32_t ref, const float* dp, float tri_area, float D[4]) {
  for (int j = 0; j < 4; ++j) D[j] = (ref & kLeafRef) ? tri_area : dp[4 * (size_t)ref + j];
}

__device__ inline uint32_t dp_node(bool as_leaf, uint32_t c, float area, const float Da[4], const float Db[4],
                                   float D[4]) {
  if (as_leaf) {
    for (int j = 0; j < 4; ++j) D[j] = (float)c * area;
    return 0u;
  }
  float Ds[5];
  uint32_t ks[5] = {0u, 0u, 0u, 0u, 0u};
  for (int j = 2; j <= 4; ++j) {
    Ds[j] = INFINITY;
    for (int kl = 1; kl < j; ++kl) {
      const float v = Da[kl - 1] + Db[j - kl - 1];
      if (v < Ds[j]) {
        Ds[j] = v;
        ks[j] = (uint32_t)kl;
      }
    }
  }
  float best = kSahNode * area + Ds[4];
  uint32_t dec = 0u, bits = 0u;
  D[0] = best;
  for (int j = 2; j <= 4; ++j) {
    if (Ds[j] < best) {
      best = Ds[j];
      dec = ks[j] | ((uint32_t)(j - (int)ks[j]) << 2);
    }
    D[j - 1] = best;
    bits |= dec << (4 * (j - 1));
  }
  return bits | ((ks[4] | ((4u - ks[4]) << 2)) << 16);
}

__device__ inline float half_area(const float b[6]) {
  const float dx = b[3] - b[0], dy = b[4] - b[1], dz = b[5] - b[2];
  return dx * dy + dy * dz + dz * dx;
}

// boxes bottom-up: the second arrival at a node merges both children's boxes
__global__ __launch_bounds__(kBB) void k_boxes_up(int64_t n, const uint32_t* __restrict__ val,
                                                  const float* __restrict__ tbox, const uint2* __restrict__ child,
                                                  const int32_t* __restrict__ parent_leaf,
                                                  const int32_t* __restrict__ parent_int, float* nbox,
                                                  uint32_t* flag, const uint32_t* __restrict__ cnt, float* dp,
                                                  uint32_t* dsp) {
  for (int64_t i = blockIdx.x * (int64_t)kBB + threadIdx.x; i < n; i += (int64_t)gridDim.x * kBB) {
    int32_t p = n > 1 ? parent_leaf[i] : -1;
    // a radix tree over 30-bit codes and 32-bit indices is at most 63 levels deep; the bound only
    // guards the walk against a malformed tree
    for (int level = 0; p >= 0 && level < kMaxTreeLevels; ++level) {
      // release this subtree's box, acquire the sibling's
      if (__hip_atomic_fetch_add(&flag[p], 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT) == 0u) break;
      const uint2 c = child[p];
      float a[6], b[6];
      ref_box(c.x, val, tbox, nbox, a);
      ref_box(c.y, val, tbox, nbox, b);
      float u[6];
      for (int k = 0; k < 3; ++k) {
        u[k] = fminf(a[k], b[k]);
        u[3 + k] = fmaxf(a[3 + k], b[3 + k]);
        nbox[6 * (size_t)p + k] = u[k];
        nbox[6 * (size_t)p + 3 + k] = u[3 + k];
      }
      float Da[4], Db[4];
      dp_of_ref(c.x, dp, half_area(a), Da);
      dp_of_ref(c.y, dp, half_area(b), Db);
      const uint32_t cp = cnt[p];
      float D[4];
      dsp[p] = dp_node((cp & kLeafBitCnt) != 0u, cp & ~kLeafBitCnt, half_area(u), Da, Db, D);
      for (int j = 0; j < 4; ++j) dp[4 * (size_t)p + j] = D[j];
      p = parent_int[p];
    }
  }
}

// ---- 4b. locally-ordered clustering.  Cluster i of a round: a binary-tree
// reference cid[i] and its box cbox[k][i] (six planes of n floats); m clusters in
// Morton order.

__global__ __launch_bounds__(kBB) void k_ploc_init(const uint32_t* __restrict__ val, const float* __restrict__ tbox,
                                                   int64_t n, uint32_t* __restrict__ cid, float* __restrict__ cbox) {
  for (int64_t i = blockIdx.x * (int64_t)kBB + threadIdx.x; i < n; i += (int64_t)gridDim.x * kBB) {
    cid[i] = kLeafRef | (uint32_t)i;
    const float* b = tbox + 6 * (size_t)val[i];
    for (int k = 0; k < 6; ++k) cbox[(size_t)k * n + i] = b[k];
  }
}

// Nearest neighbour of cluster i of m: the least surface area of the merged
// box; among equal areas the nearer place, then an even lower index of the
// pair, then the lower index (one rank per pair, so mutual nearest neighbours
// always exist, and equal boxes pair up as (2k, 2k + 1)).  At one distance
// that is the lower place, unless it is odd and i is even.  G neighbouring
// lanes share a place: even lanes look below, odd ones above, each at every
// (G / 2)-th distance; the chain of one thread's comparisons is what a round
// lasts once few clusters are left.  Place i's box is s.get(at).  All G lanes
// return the neighbour, i if no area compares.
struct SharedBoxes {  // in LDS, read as 16 + 8 bytes
  float4* a;          // lo xyz, hi x
  float2* b;          // hi yz
  __device__ void put(int q, const float v[6]) const {
    a[q] = make_float4(v[0], v[1], v[2], v[3]);
    b[q] = make_float2(v[4], v[5]);
  }
  __device__ void get(int q, float v[6]) const {
    const float4 x = a[q];
    const float2 y = b[q];
    v[0] = x.x;
    v[1] = x.y;
    v[2] = x.z;
    v[3] = x.w;
    v[4] = y.x;
    v[5] = y.y;
  }
};

template <int G>
__device__ inline uint32_t ploc_nearest(const SharedBoxes& s, int at, uint32_t i, uint32_t m) {
  constexpr uint32_t kNone = 0xFFFFFFFFu;
  const uint32_t g = threadIdx.x % G;
  const bool up = (g & 1u) != 0u;
  const uint32_t reach = up ? m - 1u - i : i;
  const int step = up ? 1 : -1;
  float bi[6];
  s.get(at, bi);
  float best = INFINITY;
  uint32_t bd = kNone;
#pragma unroll
  for (int r = 0; r < 2 * kPlocRadius / G; ++r) {
    const uint32_t d = 1u + (g >> 1) + (uint32_t)(G / 2 * r);
    float u[6];
    s.get(at + step * (int)d, u);
    for (int k = 0; k < 3; ++k) {
      u[k] = fminf(bi[k], u[k]);
      u[3 + k] = fmaxf(bi[3 + k], u[3 + k]);
    }
    const float a = half_area(u);
    if (d <= reach && (a < best || (a == best && bd == kNone))) {
      best = a;
      bd = d;
    }
  }
  // rank of the place among equal areas
  uint32_t rank = bd == kNone ? kNone : 2u * bd + (uint32_t)(up != ((i & 1u) == 0u && (bd & 1u) != 0u));
  uint32_t j = bd == kNone ? i : (up ? i + bd : i - bd);
  for (int off = 1; off < G; off <<= 1) {
    const float oa = __shfl_xor(best, off);
    const uint32_t orank = __shfl_xor(rank, off), oj = __shfl_xor(j, off);
    if (oa < best || (oa == best && orank < rank)) {
      best = oa;
      rank = orank;
      j = oj;
    }
  }
  return j;
}

// A round's pairs.  mate[i]: the cluster that merges with i (mutual nearest
// neighbours), else i.  With over 99 % of the clusters of the round before
// kept (mc[1]: that round's own count, mc[0]: this round's) the pairs are
// (2k, 2k + 1) outright.  One block per kBB places; it also finds the
// neighbours of the kPlocRadius places on either side, so that it knows its
// pairs without another launch, and counts its kept places (low word) and
// its merges (high word) in bc (0 past the last cluster).  Two threads a
// place; bound by LDS reads of the 32 boxes a cluster is compared with (1.31M
// clusters 63 us; 84 with one thread a place and boxes in six planes).
constexpr int kNnThreads = 2 * (kBB + 2 * kPlocRadius);
static_assert(kNnThreads % 64 == 0 && kNnThreads <= 1024, "whole waves");
__global__ __launch_bounds__(kNnThreads) void k_ploc_nn(const float* __restrict__ cbox, uint32_t n,
                                                 const uint32_t* __restrict__ mc, int32_t* __restrict__ mate,
                                                 unsigned long long* __restrict__ bc) {
  constexpr int kNear = kBB + 2 * kPlocRadius;   // places whose neighbour is found here
  constexpr int kSpan = kBB + 4 * kPlocRadius;   // places compared
  __shared__ float4 s_a[kSpan];
  __shared__ float2 s_b[kSpan];
  const SharedBoxes boxes{s_a, s_b};
  __shared__ uint32_t s_nn[kNear];
  __shared__ unsigned long long s_w[kNnThreads / 64];
  const uint32_t m = mc[0];
  const bool forced = (uint64_t)m * 100u > (uint64_t)mc[1] * 99u;
  const int64_t b0 = (int64_t)blockIdx.x * kBB;
  if (b0 >= (int64_t)m) {
    if (threadIdx.x == 0) bc[blockIdx.x] = 0ull;
    return;
  }
  if (!forced) {
    for (int t = threadIdx.x; t < kSpan; t += kNnThreads) {
      const int64_t g = b0 - 2 * kPlocRadius + t;
      const bool in = g >= 0 && g < (int64_t)m;
      float v[6];
      for (int k = 0; k < 6; ++k) v[k] = in ? cbox[(size_t)k * n + g] : 0.0f;
      boxes.put(t, v);
    }
    __syncthreads();
  }
  const int t = threadIdx.x / 2;  // a pair of lanes takes the same branches
  const int64_t p = b0 - kPlocRadius + t;
  uint32_t near = 0;
  if (p >= 0 && p < (int64_t)m) {
    const uint32_t q = (uint32_t)p;
    near = forced ? ((q ^ 1u) < m ? q ^ 1u : q) : ploc_nearest<2>(boxes, t + kPlocRadius, q, m);
  }
  if (threadIdx.x % 2 == 0) s_nn[t] = near;
  __syncthreads();
  const uint32_t i = (uint32_t)b0 + threadIdx.x;
  bool kept = false, merges = false;
  if (threadIdx.x < kBB && i < m) {
    const uint32_t j = s_nn[threadIdx.x + kPlocRadius];
    // j is within kPlocRadius places of i
    const bool mutual = j != i && s_nn[(int)(j - (uint32_t)b0) + kPlocRadius] == i;
    mate[i] = (int32_t)(mutual ? j : i);
    kept = !(mutual && j < i);
    merges = mutual && i < j;
  }
  const unsigned long long w = (unsigned long long)__popcll(__ballot(kept)) |
                               ((unsigned long long)__popcll(__ballot(merges)) << 32);
  if (threadIdx.x % 64 == 0) s_w[threadIdx.x / 64] = w;
  __syncthreads();
  if (threadIdx.x == 0) {
    unsigned long long sum = 0;
    for (int k = 0; k < kBB / 64; ++k) sum += s_w[k];
    bc[blockIdx.x] = sum;
  }
}

// What the rounds know of a cluster's subtree: triangles (kLeafBitCnt: one
// BVH4 leaf), SAH cost and the costs of covering it with 1..4 roots.
struct SubTree {
  uint32_t cnt;
  float cost, D[4];
};

__device__ inline SubTree sub_tree(uint32_t ref, float area, const uint32_t* cnt, const float* ncost, const float* dp) {
  SubTree s;
  if (ref & kLeafRef) {
    s.cnt = 1u;
    s.cost = area;
    for (int j = 0; j < 4; ++j) s.D[j] = area;
  } else {
    s.cnt = cnt[ref];
    s.cost = ncost[ref];
    const float4 d = reinterpret_cast<const float4*>(dp)[ref];
    s.D[0] = d.x;
    s.D[1] = d.y;
    s.D[2] = d.z;
    s.D[3] = d.w;
  }
  return s;
}

// Binary node o of the clusters a and b (boxes ba, bb); its box replaces ba,
// what the next rounds need of it sa.  Its SAH cost (surface area x (kSahNode
// + the children's costs), a single triangle costing its area) decides whether
// its subtree becomes one BVH4 leaf: when it holds at most kMaxLeafTris
// triangles and testing them all costs no more.
__device__ inline void ploc_node(uint32_t o, uint32_t a, uint32_t b, float ba[6], const float bb[6], SubTree& sa,
                                 const SubTree& sc, uint2* __restrict__ child, float* __restrict__ nbox,
                                 uint32_t* __restrict__ cnt, float* __restrict__ dp, uint32_t* __restrict__ dsp) {
  for (int k = 0; k < 3; ++k) {
    ba[k] = fminf(ba[k], bb[k]);
    ba[3 + k] = fmaxf(ba[3 + k], bb[3 + k]);
  }
  for (int k = 0; k < 6; ++k) nbox[6 * (size_t)o + k] = ba[k];
  const uint32_t c = (sa.cnt & ~kLeafBitCnt) + (sc.cnt & ~kLeafBitCnt);
  const float area = half_area(ba);
  const float split = kSahNode * area + sa.cost + sc.cost, leaf = (float)c * area;
  const bool as_leaf = c <= (uint32_t)kMaxLeafTris && leaf <= split;
  float D[4];
  dsp[o] = dp_node(as_leaf, c, area, sa.D, sc.D, D);
  reinterpret_cast<float4*>(dp)[o] = make_float4(D[0], D[1], D[2], D[3]);
  child[o] = make_uint2(a, b);
  sa.cnt = as_leaf ? (c | kLeafBitCnt) : c;
  cnt[o] = sa.cnt;
  sa.cost = as_leaf ? leaf : split;
  for (int j = 0; j < 4; ++j) sa.D[j] = D[j];
}

// A round's merges and the compaction in one pass: pairs i < j become one node
// at place i, place j is dropped, and the kept clusters go in order to the
// next round's arrays.  After a tree of n leaves has come down to m clusters
// it has n - m inner nodes, so a merge's node index is n - m plus the merges
// before it: no counter is shared (one atomic per wave on one line took most
// of a 239 us first round of 1.31M clusters; this pass takes 25).  bc: this round's block
// counts, or with `scanned` their exclusive scan.  The last block writes the
// new count to mc_out[0] and this round's to mc_out[1].
__global__ __launch_bounds__(kBB) void k_ploc_merge(
    const uint32_t* __restrict__ cid, const float* __restrict__ cbox, uint32_t n, const uint32_t* __restrict__ mc,
    const int32_t* __restrict__ mate, const unsigned long long* __restrict__ bc, bool scanned,
    uint2* __restrict__ child, float* __restrict__ nbox, uint32_t* __restrict__ cnt, float* __restrict__ ncost,
    float* __restrict__ dp, uint32_t* __restrict__ dsp, uint32_t* __restrict__ cid2, float* __restrict__ cbox2,
    uint32_t* __restrict__ mc_out, uint32_t* __restrict__ err) {
  __shared__ unsigned long long s_w[kBB / 64];
  const uint32_t m = mc[0];
  const bool last = blockIdx.x == gridDim.x - 1;
  if ((int64_t)blockIdx.x * kBB >= (int64_t)m && !last) return;
  unsigned long long before = 0;
  if (scanned) {
    before = bc[blockIdx.x];
  } else {
    for (uint32_t k = threadIdx.x; k < blockIdx.x; k += kBB) before += bc[k];
    before = block_sum(before, s_w);
  }
  const uint32_t i = blockIdx.x * (uint32_t)kBB + threadIdx.x;
  const uint32_t j = i < m ? (uint32_t)mate[i] : i;
  const bool keep = i < m && j >= i, merge = i < m && j > i;
  const uint64_t bk = __ballot(keep), bm = __ballot(merge);
  const int wave = threadIdx.x / 64, lane = threadIdx.x % 64;
  if (lane == 0)
    s_w[wave] = (unsigned long long)__popcll(bk) | ((unsigned long long)__popcll(bm) << 32);
  __syncthreads();
  unsigned long long at = before, total = before;
  for (int q = 0; q < kBB / 64; ++q) {
    if (q < wave) at += s_w[q];
    total += s_w[q];
  }
  if (last && threadIdx.x == 0) {
    mc_out[0] = (uint32_t)total;
    mc_out[1] = m;
  }
  if (!keep) return;
  const uint64_t lt = lane == 0 ? 0ull : (~0ull >> (64 - lane));
  const uint32_t pos = (uint32_t)at + (uint32_t)__popcll(bk & lt);
  uint32_t id = cid[i];
  float ba[6];
  for (int k = 0; k < 6; ++k) ba[k] = cbox[(size_t)k * n + i];
  if (merge) {
    const uint32_t o = n - m + (uint32_t)(at >> 32) + (uint32_t)__popcll(bm & lt);
    if (o >= n - 1u || j >= m) {  // more merges than a binary tree of this size has nodes: report
      atomicOr(err, 4u);
    } else {
      const uint32_t b = cid[j];
      float bb[6];
      for (int k = 0; k < 6; ++k) bb[k] = cbox[(size_t)k * n + j];
      SubTree sa = sub_tree(id, half_area(ba), cnt, ncost, dp), sc = sub_tree(b, half_area(bb), cnt, ncost, dp);
      ploc_node(o, id, b, ba, bb, sa, sc, child, nbox, cnt, dp, dsp);
      ncost[o] = sa.cost;
      id = o;
    }
  }
  cid2[pos] = id;
  for (int k = 0; k < 6; ++k) cbox2[(size_t)k * n + pos] = ba[k];
}

// The last rounds of the clustering in one workgroup, once at most
// kFinishMax clusters are left: the same rounds (same ranks, same merges,
// same forced rounds) with the clusters and what is known of their subtrees in
// LDS and barriers between the steps instead of launches.  The barriers order
// LDS only, since no round reads what another stored.  Then the root's job.
// A chain of about 25 rounds, each as long as one thread's comparisons: 194 us
// with one thread a cluster and the subtrees in memory, 77 so.
constexpr int kFinishThreads = 1024;
constexpr int kFinishMax = 2048;
constexpr int kFinishPer = kFinishMax / kFinishThreads;
constexpr int kFinishSpan = kFinishMax + 2 * kPlocRadius;

__device__ inline void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

__device__ inline uint32_t block_excl_scan_1024(bool flag, uint32_t* s_w, uint32_t& total) {
  const int lane = threadIdx.x % 64, wave = threadIdx.x / 64;
  const uint64_t bal = __ballot(flag);
  const uint64_t lt = lane == 0 ? 0ull : (~0ull >> (64 - lane));
  if (lane == 0) s_w[wave] = (uint32_t)__popcll(bal);
  lds_barrier();
  uint32_t before = 0, t = 0;
  for (int w = 0; w < kFinishThreads / 64; ++w) {
    if (w < wave) before += s_w[w];
    t += s_w[w];
  }
  total = t;
  return before + (uint32_t)__popcll(bal & lt);
}

// Nearest neighbours of the m clusters in LDS, G lanes a cluster.  A place's
// window reaches past the arrays' ends: kPlocRadius boxes before and after.
template <int G>
__device__ inline void finish_nearest(const SharedBoxes& boxes, uint32_t* snn, uint32_t m) {
  for (uint32_t i = threadIdx.x / G; i < m; i += kFinishThreads / G) {
    const uint32_t j = ploc_nearest<G>(boxes, (int)i + kPlocRadius, i, m);
    if (threadIdx.x % G == 0) snn[i] = j;
  }
}

__global__ __launch_bounds__(kFinishThreads) void k_ploc_finish(
    const uint32_t* __restrict__ cid_in, const float* __restrict__ cbox_in, uint32_t n,
    const uint32_t* __restrict__ mc, uint2* __restrict__ child, float* __restrict__ nbox, uint32_t* __restrict__ cnt,
    const float* __restrict__ ncost, float* __restrict__ dp, uint32_t* __restrict__ dsp, uint4* __restrict__ jobs,
    uint32_t* __restrict__ err) {
  constexpr int kSub = 6;  // words of a SubTree
  __shared__ float4 s_a[kFinishSpan];
  __shared__ float2 s_b[kFinishSpan];
  const SharedBoxes boxes{s_a, s_b};
  __shared__ uint32_t s_sub[kSub * kFinishMax];
  __shared__ uint32_t sid[kFinishMax], snn[kFinishMax];
  __shared__ uint32_t s_w[kFinishPer][kFinishThreads / 64], s_nodes;
  uint32_t m = mc[0], prev = mc[1];
  if (m > (uint32_t)kFinishMax || m == 0u) {  // the host launches this only at or below kFinishMax clusters
    if (threadIdx.x == 0) atomicOr(err, 16u);
    return;
  }
  const auto load_sub = [&](uint32_t i) {
    SubTree s;
    s.cnt = s_sub[i];
    s.cost = __uint_as_float(s_sub[kFinishMax + i]);
    for (int k = 0; k < 4; ++k) s.D[k] = __uint_as_float(s_sub[(2 + k) * kFinishMax + i]);
    return s;
  };
  const auto store = [&](uint32_t i, uint32_t id, const float b[6], const SubTree& s) {
    sid[i] = id;
    boxes.put((int)i + kPlocRadius, b);
    s_sub[i] = s.cnt;
    s_sub[kFinishMax + i] = __float_as_uint(s.cost);
    for (int k = 0; k < 4; ++k) s_sub[(2 + k) * kFinishMax + i] = __float_as_uint(s.D[k]);
  };
  for (int e = 0; e < kFinishPer; ++e) {
    const uint32_t i = threadIdx.x + e * kFinishThreads;
    if (i < m) {
      const uint32_t id = cid_in[i];
      float b[6];
      for (int k = 0; k < 6; ++k) b[k] = cbox_in[(size_t)k * n + i];
      store(i, id, b, sub_tree(id, half_area(b), cnt, ncost, dp));
    }
  }
  if (threadIdx.x == 0) s_nodes = n - m;  // inner nodes so far
  lds_barrier();
  for (int round = 0; m > 1; ++round) {
    if (round >= kPlocMaxRounds) {
      if (threadIdx.x == 0) atomicOr(err, 16u);
      return;
    }
    const bool forced = (uint64_t)m * 100u > (uint64_t)prev * 99u;
    if (forced) {
      for (uint32_t i = threadIdx.x; i < m; i += kFinishThreads) snn[i] = (i ^ 1u) < m ? i ^ 1u : i;
    } else if (m > kFinishThreads / 8) {
      finish_nearest<2>(boxes, snn, m);
    } else {
      finish_nearest<8>(boxes, snn, m);
    }
    lds_barrier();
    // merges into registers, then the compaction in order: places tid (first) then
    // tid + kFinishThreads (second)
    bool keep[kFinishPer];
    uint32_t id_r[kFinishPer];
    float box_r[kFinishPer][6];
    SubTree sub_r[kFinishPer];
    uint32_t pos[kFinishPer], tot[kFinishPer];
    for (int e = 0; e < kFinishPer; ++e) {
      const uint32_t i = threadIdx.x + e * kFinishThreads;
      keep[e] = false;
      if (i >= m) continue;
      const uint32_t j = snn[i];
      const bool mutual = j != i && snn[j] == i;
      keep[e] = !(mutual && j < i);
      if (!keep[e]) continue;
      id_r[e] = sid[i];
      boxes.get((int)i + kPlocRadius, box_r[e]);
      sub_r[e] = load_sub(i);
      if (!mutual) continue;
      const uint32_t o = atomicAdd(&s_nodes, 1u);
      if (o >= n - 1u) {
        atomicOr(err, 4u);
        continue;
      }
      float bb[6];
      boxes.get((int)j + kPlocRadius, bb);
      const SubTree sc = load_sub(j);
      ploc_node(o, id_r[e], sid[j], box_r[e], bb, sub_r[e], sc, child, nbox, cnt, dp, dsp);
      id_r[e] = o;
    }
    for (int e = 0; e < kFinishPer; ++e) pos[e] = block_excl_scan_1024(keep[e], s_w[e], tot[e]);
    uint32_t base = 0;
    for (int e = 0; e < kFinishPer; ++e) {  // every thread has read its places before the scan's barriers
      if (keep[e]) store(base + pos[e], id_r[e], box_r[e], sub_r[e]);
      base += tot[e];
    }
    lds_barrier();
    prev = m;
    m = base;
  }
  if (threadIdx.x == 0) jobs[0] = make_uint4(sid[0], 0u, 0u, 0u);
}

// Cluster counts of the first round: n clusters, and no round before it.
__global__ void k_ploc_start(uint32_t* __restrict__ mc, uint32_t n) {
  mc[0] = n;
  mc[1] = 0xFFFFFFFFu;
}

// 5. one level of the collapse: job (binary reference, BVH4 node index, place
// of its first triangle in leaf order).  A leaf's triangles take consecutive
// places in depth-first order of its subtree: order[place] = sorted index.
__device__ inline void collapse_one(const uint4 job, uint4* __restrict__ next_jobs, uint32_t* __restrict__ n_next,
                                    uint32_t* __restrict__ n_nodes, uint32_t* __restrict__ max_leaf,
                                    const uint32_t* __restrict__ val, const float* __restrict__ tbox,
                                    const float* __restrict__ nbox, const uint2* __restrict__ child,
                                    const uint32_t* __restrict__ cnt, const uint32_t* __restrict__ dsp,
                                    BVHNode* __restrict__ out, uint32_t cap, uint32_t n_tris,
                                    uint32_t* __restrict__ order, uint32_t* __restrict__ err) {
  uint32_t kids[4];
  int nk = 0;
  if (ref_is_leaf_subtree(job.x, cnt)) {
    kids[nk++] = job.x;  // the whole tree is one leaf under a one-child root
  } else if (kGpuCollapseDp) {
    // the roots of the best split of the node's four slots, left before right
    // (the slots of the entries on the stack never add up to more than four)
    const uint2 c = child[job.x];
    const uint32_t s4 = dsp[job.x] >> 16;
    uint32_t stk_ref[4], stk_j[4];
    int sp = 0;
    stk_ref[sp] = c.y;
    stk_j[sp++] = s4 >> 2;
    stk_ref[sp] = c.x;
    stk_j[sp++] = s4 & 3u;
    while (sp > 0 && nk < 4) {
      --sp;
      const uint32_t y = stk_ref[sp], j = stk_j[sp];
      if (ref_is_leaf_subtree(y, cnt) || j <= 1u || j > 4u) {
        kids[nk++] = y;
        continue;
      }
      const uint32_t d = (dsp[y] >> (4u * (j - 1u))) & 15u;
      if ((d & 3u) == 0u || sp + 2 > 4) {
        kids[nk++] = y;
        continue;
      }
      const uint2 cc = child[y];
      stk_ref[sp] = cc.y;
      stk_j[sp++] = d >> 2;
      stk_ref[sp] = cc.x;
      stk_j[sp++] = d & 3u;
    }
    if (sp > 0) atomicOr(err, 32u);  // more roots than four slots: a malformed split
  } else {
    const uint2 c = child[job.x];
    kids[nk++] = c.x;
    kids[nk++] = c.y;
    while (nk < 4) {
      int pick = -1;
      float pa = -1.0f;
      for (int q = 0; q < nk; ++q) {
        if (!ref_is_leaf_subtree(kids[q], cnt)) {
          float b[6];
          ref_box(kids[q], val, tbox, nbox, b);
          const float a = half_area(b);
          if (a > pa) {
            pa = a;
            pick = q;
          }
        }
      }
      if (pick < 0) break;
      const uint2 cc = child[kids[pick]];
      for (int q = nk; q > pick + 1; --q) kids[q] = kids[q - 1];  // open in place: siblings keep their order
      kids[pick] = cc.x;
      kids[pick + 1] = cc.y;
      nk++;
    }
  }
  BVHNode node;
  for (int q = 0; q < 4; ++q) {
    node.lo_x[q] = node.hi_x[q] = node.lo_y[q] = node.hi_y[q] = node.lo_z[q] = node.hi_z[q] = 0.0f;
    node.child[q] = kEmpty;
    node.meta[q] = 0u;
  }
  node.meta[0] = (uint32_t)nk;
  uint32_t leaf_max = 0, place = job.z;
  // the node's inner children take consecutive node indices (siblings share lines of the cache)
  int n_inner = 0;
  for (int q = 0; q < nk; ++q) n_inner += ref_is_leaf_subtree(kids[q], cnt) ? 0 : 1;
  uint32_t o_next = 0, slot_next = 0;
  if (n_inner) {
    o_next = atomicAdd(n_nodes, (uint32_t)n_inner);
    slot_next = atomicAdd(n_next, (uint32_t)n_inner);
  }
  for (int q = 0; q < nk; ++q) {
    float b[6];
    ref_box(kids[q], val, tbox, nbox, b);
    node.lo_x[q] = b[0];
    node.lo_y[q] = b[1];
    node.lo_z[q] = b[2];
    node.hi_x[q] = b[3];
    node.hi_y[q] = b[4];
    node.hi_z[q] = b[5];
    const uint32_t c = ref_count(kids[q], cnt);
    if (place + c > n_tris) {  // counts that do not add up: report
      atomicOr(err, 8u);
      break;
    }
    if (ref_is_leaf_subtree(kids[q], cnt)) {
      node.child[q] = make_leaf(place, c);
      leaf_max = c > leaf_max ? c : leaf_max;
      // the subtree's leaves, left before right (at most kMaxLeafTris of them,
      // so the stack never holds more than that many entries)
      uint32_t stk[kMaxLeafTris];
      int sp = 0;
      uint32_t w = place;
      stk[sp++] = kids[q];
      while (sp > 0) {
        const uint32_t r = stk[--sp];
        if (r & kLeafRef) {
          if (w < place + c) order[w] = r & ~kLeafRef;
          w++;
        } else if (sp + 2 <= kMaxLeafTris) {
          const uint2 cc = child[r];
          stk[sp++] = cc.y;
          stk[sp++] = cc.x;
        } else {
          atomicOr(err, 8u);
          break;
        }
      }
      if (w != place + c) atomicOr(err, 8u);
    } else {
      const uint32_t o = o_next++, slot = slot_next++;
      if (o >= cap || slot >= cap) {  // more nodes than a tree of this size can have: report
        atomicOr(err, 2u);
        continue;
      }
      node.child[q] = o;
      next_jobs[slot] = make_uint4(kids[q], o, place, 0u);
    }
    place += c;
  }
  if (job.y < cap) out[job.y] = node;
  if (leaf_max) atomicMax(max_leaf, leaf_max);
}

// Level `level` of the collapse: its job count is jc[level % 3] (written by the
// level before), its jobs append to jc[(level + 1) % 3], and it zeroes
// jc[(level + 2) % 3] for the level after next; jc[3] counts the levels that
// had jobs.  Any grid (a grid-stride loop), so that levels are enqueued
// without the host reading the counts in between.
__global__ __launch_bounds__(kBB) void k_collapse(const uint4* __restrict__ jobs, uint32_t* __restrict__ jc, int level,
                                                  uint4* __restrict__ next_jobs, uint32_t* __restrict__ n_nodes,
                                                  uint32_t* __restrict__ max_leaf, const uint32_t* __restrict__ val,
                                                  const float* __restrict__ tbox, const float* __restrict__ nbox,
                                                  const uint2* __restrict__ child, const uint32_t* __restrict__ cnt,
                                                  const uint32_t* __restrict__ dsp, BVHNode* __restrict__ out,
                                                  uint32_t cap, uint32_t n_tris, uint32_t* __restrict__ order,
                                                  uint32_t* __restrict__ err) {
  const uint32_t n_jobs = min(jc[level % 3], cap);
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    jc[(level + 2) % 3] = 0u;
    if (n_jobs) atomicMax(jc + 3, (uint32_t)(level + 1));
  }
  for (uint32_t j = blockIdx.x * kBB + threadIdx.x; j < n_jobs; j += gridDim.x * kBB)
    collapse_one(jobs[j], next_jobs, jc + (level + 1) % 3, n_nodes, max_leaf, val, tbox, nbox, child, cnt, dsp, out,
                 cap, n_tris, order, err);
}

// 6. triangle records in leaf order
__global__ __launch_bounds__(kBB) void k_sorted_tris(const float* __restrict__ soup, const uint32_t* __restrict__ prim,
                                                     const uint32_t* __restrict__ mat, const uint32_t* __restrict__ val,
                                                     const uint32_t* __restrict__ order, int64_t n,
                                                     TriRec* __restrict__ tris) {
  for (int64_t i = blockIdx.x * (int64_t)kBB + threadIdx.x; i < n; i += (int64_t)gridDim.x * kBB) {
    const uint32_t t = val[order[i]];
    const float* p = soup + 9 * (size_t)t;
    TriRec r;
    r.a = make_float4(p[0], p[1], p[2], __uint_as_float(prim ? prim[t] : t));
    r.b = make_float4(p[3], p[4], p[5], __uint_as_float(mat[t]));
    r.c = make_float4(p[6], p[7], p[8], 0.0f);
    tris[i] = r;
  }
}

// A mesh's triangles as soup, its contents checked on the way: a bad index
// reads nothing and reports.  12 bytes of indices in and 36 of soup out per
// triangle (the vertices mostly stay in L2).
__global__ void k_gather_init(uint32_t* info) {
  if (threadIdx.x < (unsigned)kGatherWords)
    info[threadIdx.x] = threadIdx.x >= 2u && threadIdx.x < 5u ? 0xFFFFFFFFu : 0u;
}

__global__ __launch_bounds__(kBB) void k_check_vertices(const float* __restrict__ v, int64_t n,
                                                        uint32_t* __restrict__ info) {
  bool bad = false;
  for (int64_t i = blockIdx.x * (int64_t)kBB + threadIdx.x; i < n; i += (int64_t)gridDim.x * kBB)
    bad |= (__float_as_uint(v[i]) & 0x7F800000u) == 0x7F800000u;
  if (bad) atomicOr(info, 1u);
}

__global__ __launch_bounds__(kBB) void k_gather_soup(const float* __restrict__ v, int64_t nv,
                                                     const int32_t* __restrict__ idx, const uint32_t* __restrict__ mat,
                                                     int64_t n, float* __restrict__ soup, uint32_t* __restrict__ info) {
  __shared__ uint32_t red[8];
  if (threadIdx.x < 8) red[threadIdx.x] = threadIdx.x >= 2 && threadIdx.x < 5 ? 0xFFFFFFFFu : 0u;
  __syncthreads();
  uint32_t bad = 0u, top = 0u, lo[3] = {0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu}, hi[3] = {0u, 0u, 0u};
  for (int64_t i = blockIdx.x * (int64_t)kBB + threadIdx.x; i < n; i += (int64_t)gridDim.x * kBB) {
    const uint32_t m = mat[i];
    if (m & 0x80000000u) bad = 1u;
    else top = m > top ? m : top;
    for (int c = 0; c < 3; ++c) {
      const int64_t q = idx[3 * i + c];
      if (q < 0 || q >= nv) {
        bad = 1u;
        continue;
      }
      for (int k = 0; k < 3; ++k) {
        const float x = v[3 * q + k];
        soup[9 * i + 3 * c + k] = x;
        const uint32_t u = f2ord(x + 0.0f);  // -0 as 0
        lo[k] = u < lo[k] ? u : lo[k];
        hi[k] = u > hi[k] ? u : hi[k];
      }
    }
  }
  if (bad) atomicOr(&red[0], 1u);
  atomicMax(&red[1], top);
  for (int k = 0; k < 3; ++k) {
    atomicMin(&red[2 + k], lo[k]);
    atomicMax(&red[5 + k], hi[k]);
  }
  __syncthreads();
  if (threadIdx.x == 0 && red[0]) atomicOr(&info[0], 1u);
  if (threadIdx.x >= 2 && threadIdx.x < 5) atomicMin(&info[threadIdx.x], red[threadIdx.x]);
  if (threadIdx.x == 1 || (threadIdx.x >= 5 && threadIdx.x < 8)) atomicMax(&info[threadIdx.x], red[threadIdx.x]);
}

// Emissive triangles: a flag per primitive, scanned by the caller into places.
__global__ __launch_bounds__(kBB) void k_light_flags(const TriRec* __restrict__ tris, int64_t n,
                                                     const uint32_t* __restrict__ emits, uint32_t n_mats,
                                                     uint32_t* __restrict__ off) {
  for (int64_t i = blockIdx.x * (int64_t)kBB + threadIdx.x; i <= n; i += (int64_t)gridDim.x * kBB) {
    if (i == n) {
      off[n] = 0u;
    } else {
      const uint32_t prim = __float_as_uint(tris[i].a.w), m = __float_as_uint(tris[i].b.w);
      if (prim < (uint64_t)n) off[prim] = m < n_mats && emits[m] ? 1u : 0u;
    }
  }
}

__global__ __launch_bounds__(kBB) void k_light_list(const TriRec* __restrict__ tris, int64_t n,
                                                    const uint32_t* __restrict__ off, int32_t* __restrict__ tri_light,
                                                    uint32_t* __restrict__ list) {
  for (int64_t i = blockIdx.x * (int64_t)kBB + threadIdx.x; i < n; i += (int64_t)gridDim.x * kBB) {
    if (!off) {
      tri_light[i] = -1;
      continue;
    }
    const TriRec r = tris[i];
    const uint32_t prim = __float_as_uint(r.a.w);
    if (prim >= (uint64_t)n) continue;
    const uint32_t at = off[prim];
    const bool light = off[prim + 1] != at;
    tri_light[prim] = light ? (int32_t)at : -1;
    if (!light) continue;
    const float v[9] = {r.a.x, r.a.y, r.a.z, r.b.x, r.b.y, r.b.z, r.c.x, r.c.y, r.c.z};
    for (int k = 0; k < 9; ++k) list[(size_t)kLightWords * at + k] = __float_as_uint(v[k]);
    list[(size_t)kLightWords * at + 9] = __float_as_uint(r.b.w);
  }
}

int grid_of(int64_t n) { return (int)std::max<int64_t>(1, std::min<int64_t>((n + kBB - 1) / kBB, 8192)); }

// device workspace of one build, freed when it goes out of scope
// (one allocation sized for the whole build, carved in 256-byte aligned
// pieces; a piece that does not fit gets an allocation of its own)
struct Scratch {
  void* arena = nullptr;
  size_t cap = 0, used = 0;
  std::vector<void*> extra;
  explicit Scratch(size_t bytes) {
    if (hipMalloc(&arena, bytes) == hipSuccess) {
      cap = bytes;
    } else {
      arena = nullptr;
      (void)hipGetLastError();  // get() allocates piece by piece
    }
  }
  ~Scratch() {
    for (void* p : extra) (void)hipFree(p);
    if (arena) (void)hipFree(arena);
  }
  template <class T>
  hipError_t get(T** out, size_t count) {
    const size_t b = (std::max<size_t>(count * sizeof(T), 16) + 255) & ~size_t(255);
    if (arena && used + b <= cap) {
      *out = reinterpret_cast<T*>(static_cast<char*>(arena) + used);
      used += b;
      return hipSuccess;
    }
    void* p = nullptr;
    hipError_t e = hipMalloc(&p, b);
    if (e == hipSuccess) extra.push_back(p);
    else (void)hipGetLastError();
    *out = static_cast<T*>(p);
    return e;
  }
};

// workspace bytes per triangle of one build: boxes, keys, tree, jobs, clusters (an upper bound)
constexpr size_t kBuildBytesPerTri = 200;

}  // namespace

#define PT_TRY(x)                         \
  do {                                    \
    hipError_t e_ = (x);                  \
    if (e_ != hipSuccess) return e_;      \
  } while (0)

hipError_t gpu_build_bvh4(const float* soup, const uint32_t* prim, const uint32_t* mat, int64_t n, BVHNode* nodes,
                          TriRec* tris, hipStream_t st, GpuBvhStats* stats, int builder) {
  if (n <= 0 || n >= (int64_t)kLeafFirstMask) return hipErrorInvalidValue;
  if (builder != kGpuBvhPloc && builder != kGpuBvhLbvh) return hipErrorInvalidValue;
  Scratch S((size_t)n * kBuildBytesPerTri + (size_t)256 * 4 * (size_t)((n + kTile - 1) / kTile) + (64u << 10));
  float *tbox = nullptr, *nbox = nullptr;
  uint32_t *cb = nullptr, *keyA = nullptr, *valA = nullptr, *keyB = nullptr, *valB = nullptr, *hist = nullptr, *scan_sums = nullptr;
  uint32_t *counters = nullptr, *cnt = nullptr, *order = nullptr;
  uint2* child = nullptr;
  uint4* jobs[2] = {nullptr, nullptr};
  const int nb = (int)((n + kTile - 1) / kTile);
  const int64_t ni = std::max<int64_t>(1, n - 1);
  PT_TRY(S.get(&tbox, (size_t)n * 6));
  PT_TRY(S.get(&nbox, (size_t)ni * 6));
  PT_TRY(S.get(&cb, 6));
  PT_TRY(S.get(&keyA, (size_t)n));
  PT_TRY(S.get(&valA, (size_t)n));
  PT_TRY(S.get(&keyB, (size_t)n));
  PT_TRY(S.get(&valB, (size_t)n));
  PT_TRY(S.get(&hist, (size_t)256 * nb));
  PT_TRY(S.get(&scan_sums, ((size_t)256 * nb + kScanTile - 1) / kScanTile));
  // [0] BVH4 nodes, [1] jobs of the next level, [2] largest leaf, [3] error bits
  PT_TRY(S.get(&counters, 8));
  PT_TRY(S.get(&child, (size_t)ni));
  PT_TRY(S.get(&cnt, (size_t)ni));
  float* dp = nullptr;
  uint32_t* dsp = nullptr;
  PT_TRY(S.get(&dp, (size_t)ni * 4));
  PT_TRY(S.get(&dsp, (size_t)ni));
  PT_TRY(S.get(&order, (size_t)n));
  PT_TRY(S.get(&jobs[0], (size_t)n));
  PT_TRY(S.get(&jobs[1], (size_t)n));

  hipLaunchKernelGGL(k_init_bounds, dim3(1), dim3(64), 0, st, cb);
  hipLaunchKernelGGL(k_tri_boxes, dim3(std::min(grid_of(n), kBoundsGrid)), dim3(kBB), 0, st, soup, n, tbox, cb);
  hipLaunchKernelGGL(k_morton, dim3(grid_of(n)), dim3(kBB), 0, st, tbox, n, cb, keyA, valA);
  for (int pass = 0; pass < 4; ++pass) {  // codes have 30 bits
    const int shift = 8 * pass;
    hipLaunchKernelGGL(k_radix_hist, dim3(nb), dim3(kBB), 0, st, keyA, n, shift, hist, nb);
    launch_scan(hist, (int64_t)256 * nb, scan_sums, st);
    hipLaunchKernelGGL(k_radix_scatter, dim3(nb), dim3(kBB), 0, st, keyA, valA, keyB, valB, n, shift, hist, nb);
    std::swap(keyA, keyB);
    std::swap(valA, valB);
  }
  PT_TRY(hipMemsetAsync(counters, 0, 8 * sizeof(uint32_t), st));
  if (n > 1 && builder == kGpuBvhLbvh) {
    uint32_t* flag = nullptr;
    int32_t *parent_leaf = nullptr, *parent_int = nullptr;
    PT_TRY(S.get(&flag, (size_t)ni));
    PT_TRY(S.get(&parent_leaf, (size_t)n));
    PT_TRY(S.get(&parent_int, (size_t)ni));
    PT_TRY(hipMemsetAsync(flag, 0, (size_t)ni * sizeof(uint32_t), st));
    PT_TRY(hipMemsetAsync(parent_int, 0xFF, (size_t)ni * sizeof(int32_t), st));  // root: -1
    hipLaunchKernelGGL(k_radix_tree, dim3(grid_of(n - 1)), dim3(kBB), 0, st, keyA, n, child, parent_leaf, parent_int,
                       cnt, counters + 3);
    hipLaunchKernelGGL(k_boxes_up, dim3(grid_of(n)), dim3(kBB), 0, st, n, valA, tbox, child, parent_leaf, parent_int,
                       nbox, flag, cnt, dp, dsp);
    const uint4 root = make_uint4(0u, 0u, 0u, 0u);
    PT_TRY(hipMemcpyAsync(jobs[0], &root, sizeof(root), hipMemcpyHostToDevice, st));
  } else if (n > 1) {
    uint32_t *cid[2] = {nullptr, nullptr}, *mc = nullptr;
    float *cbox[2] = {nullptr, nullptr}, *ncost = nullptr;
    int32_t* mate = nullptr;
    unsigned long long *bc = nullptr, *bc_sums = nullptr;
    const int64_t nblk = (n + kBB - 1) / kBB;
    for (int k = 0; k < 2; ++k) {
      PT_TRY(S.get(&cid[k], (size_t)n));
      PT_TRY(S.get(&cbox[k], (size_t)n * 6));
    }
    PT_TRY(S.get(&bc, (size_t)nblk));
    PT_TRY(S.get(&bc_sums, (size_t)(nblk + kScanTile - 1) / kScanTile));
    PT_TRY(S.get(&mate, (size_t)n));
    PT_TRY(S.get(&ncost, (size_t)ni));
    PT_TRY(S.get(&mc, 4));  // cluster counts: [0..1] read by even rounds, [2..3] by odd rounds
    hipLaunchKernelGGL(k_ploc_init, dim3(grid_of(n)), dim3(kBB), 0, st, valA, tbox, n, cid[0], cbox[0]);
    hipLaunchKernelGGL(k_ploc_start, dim3(1), dim3(1), 0, st, mc, (uint32_t)n);
    // the counts stay on the device; the host reads them once per batch of rounds and sizes the
    // batch's grids by the count at its start (kernels skip the places past the current count; a
    // round with one cluster left copies it unchanged)
    uint32_t m = (uint32_t)n, m_host[2] = {0u, 0u};
    int cur = 0, rounds = 0;
    while (m > (uint32_t)kFinishMax) {
      if (rounds >= kPlocMaxRounds) return hipErrorUnknown;
      const int blocks = (int)((m + kBB - 1) / kBB);
      const bool scanned = blocks > kPlocSumBlocks;
      for (int r = 0; r < kPlocBatch; ++r, ++rounds) {
        const uint32_t* mc_in = mc + 2 * (rounds & 1);
        uint32_t* mc_out = mc + 2 * ((rounds & 1) ^ 1);
        hipLaunchKernelGGL(k_ploc_nn, dim3(blocks), dim3(kNnThreads), 0, st, cbox[cur], (uint32_t)n, mc_in, mate, bc);
        if (scanned) launch_scan(bc, (int64_t)blocks, bc_sums, st);
        hipLaunchKernelGGL(k_ploc_merge, dim3(blocks), dim3(kBB), 0, st, cid[cur], cbox[cur], (uint32_t)n, mc_in, mate,
                           bc, scanned, child, nbox, cnt, ncost, dp, dsp, cid[cur ^ 1], cbox[cur ^ 1], mc_out,
                           counters + 3);
        cur ^= 1;
      }
      PT_TRY(hipGetLastError());
      PT_TRY(hipMemcpyAsync(m_host, mc + 2 * (rounds & 1), sizeof(m_host), hipMemcpyDeviceToHost, st));
      PT_TRY(hipStreamSynchronize(st));
      if (m_host[0] == 0u || m_host[0] > m) return hipErrorUnknown;  // a round never loses every cluster
      m = m_host[0];
    }
    // the last rounds (at most kFinishMax clusters) in one workgroup; it also writes the root's job
    hipLaunchKernelGGL(k_ploc_finish, dim3(1), dim3(kFinishThreads), 0, st, cid[cur], cbox[cur], (uint32_t)n,
                       mc + 2 * (rounds & 1), child, nbox, cnt, ncost, dp, dsp, jobs[0], counters + 3);
  } else {
    const uint4 root = make_uint4(kLeafRef, 0u, 0u, 0u);
    PT_TRY(hipMemcpyAsync(jobs[0], &root, sizeof(root), hipMemcpyHostToDevice, st));
  }
  // collapse, level by level, from the root; the levels' job counts stay on the device and the host
  // reads the next one once per batch of levels
  const uint32_t cap = (uint32_t)ni;  // nodes of the output (and jobs of a level) at most
  uint32_t* jc = nullptr;  // job counts of three consecutive levels, [3]: levels that had jobs
  PT_TRY(S.get(&jc, 4));
  const uint32_t one = 1u, jc0[4] = {1u, 0u, 0u, 0u};
  PT_TRY(hipMemcpyAsync(counters, &one, sizeof(one), hipMemcpyHostToDevice, st));
  PT_TRY(hipMemcpyAsync(jc, jc0, sizeof(jc0), hipMemcpyHostToDevice, st));
  const int cgrid = grid_of(cap);
  int level = 0;
  uint32_t pending[2] = {1u, 0u};
  while (pending[0] > 0) {
    for (int r = 0; r < kCollapseBatch; ++r, ++level) {
      if (level >= kMaxTreeLevels) return hipErrorUnknown;
      hipLaunchKernelGGL(k_collapse, dim3(cgrid), dim3(kBB), 0, st, jobs[level & 1], jc, level, jobs[(level + 1) & 1],
                         counters, counters + 2, valA, tbox, nbox, child, cnt, dsp, nodes, cap, (uint32_t)n, order,
                         counters + 3);
    }
    PT_TRY(hipGetLastError());
    PT_TRY(hipMemcpyAsync(&pending[0], jc + level % 3, sizeof(uint32_t), hipMemcpyDeviceToHost, st));
    PT_TRY(hipMemcpyAsync(&pending[1], jc + 3, sizeof(uint32_t), hipMemcpyDeviceToHost, st));
    PT_TRY(hipStreamSynchronize(st));
  }
  const int levels = (int)pending[1];
  hipLaunchKernelGGL(k_sorted_tris, dim3(grid_of(n)), dim3(kBB), 0, st, soup, prim, mat, valA, order, n, tris);
  uint32_t fin[4];
  PT_TRY(hipMemcpyAsync(fin, counters, sizeof(fin), hipMemcpyDeviceToHost, st));
  PT_TRY(hipStreamSynchronize(st));
  if (fin[3] != 0u || fin[0] > cap) return hipErrorUnknown;  // malformed tree: no result
  stats->n_nodes = fin[0];
  stats->max_leaf = (int)fin[2];
  stats->depth = levels + 1;  // node levels, plus the leaves under the deepest nodes
  return hipGetLastError();
}

float gpu_ordered_float(uint32_t u) {
  u = (u & 0x80000000u) ? (u & 0x7FFFFFFFu) : ~u;
  float f;
  __builtin_memcpy(&f, &u, sizeof(f));
  return f;
}

hipError_t gpu_gather_init(uint32_t* info, hipStream_t st) {
  hipLaunchKernelGGL(k_gather_init, dim3(1), dim3(64), 0, st, info);
  return hipGetLastError();
}

hipError_t gpu_gather_mesh(const float* vertices, int64_t n_vertices, const int32_t* indices, const uint32_t* mat,
                           int64_t n, float* soup, uint32_t* info, hipStream_t st) {
  hipLaunchKernelGGL(k_check_vertices, dim3(std::min(grid_of(3 * n_vertices), kBoundsGrid)), dim3(kBB), 0, st,
                     vertices, 3 * n_vertices, info);
  hipLaunchKernelGGL(k_gather_soup, dim3(std::min(grid_of(n), kBoundsGrid)), dim3(kBB), 0, st, vertices, n_vertices,
                     indices, mat, n, soup, info);
  return hipGetLastError();
}

size_t gpu_count_lights_scratch(int64_t n) { return (size_t)((n + 1 + kScanTile - 1) / kScanTile); }

hipError_t gpu_count_lights(const TriRec* tris, int64_t n, const uint32_t* emits, uint32_t n_mats, uint32_t* off,
                            uint32_t* sums, hipStream_t st) {
  hipLaunchKernelGGL(k_light_flags, dim3(grid_of(n + 1)), dim3(kBB), 0, st, tris, n, emits, n_mats, off);
  launch_scan(off, n + 1, sums, st);
  return hipGetLastError();
}

hipError_t gpu_list_lights(const TriRec* tris, int64_t n, const uint32_t* off, int32_t* tri_light, uint32_t* list,
                           hipStream_t st) {
  hipLaunchKernelGGL(k_light_list, dim3(grid_of(n)), dim3(kBB), 0, st, tris, n, off, tri_light, list);
  return hipGetLastError();
}

}  // namespace pt
