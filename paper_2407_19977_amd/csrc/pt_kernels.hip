// Wavefront path-tracing kernels for gfx950 (wave64).
//
// One sampling pass traces one path per slot (one or more samples of every
// pixel of the tile) through the loop
//   generate -> [reset -> traverse -> bin -> shade<class>...] x (max_depth+1) -> traverse -> accumulate
// where traverse finds the closest hits of a bounce's rays together with the
// shadow rays of the previous bounce's shading.  From bounce 2 on, once few
// paths are alive, one persistent kernel (k_tail) finishes every remaining
// vertex instead.  Queues live in HBM and are compacted per workgroup: a
// ballot of the lanes that append, wave counts gathered in LDS, one atomic
// per workgroup on the queue tail and a lane prefix (mbcnt) for the slot.
// Queue lengths never leave the device, except the one count read to decide
// the tail hand-off: every kernel is launched over a fixed grid and strides
// over the length it reads from the counter array.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <mutex>

#include "pt_internal.h"
#include "pt_nrc.h"
#include "pt_shade.h"
#include "pt_trace.h"

namespace pt {

// ------------------------------------------------------------ wave helpers
__device__ inline uint32_t lane_id() { return __lane_id(); }

__device__ inline uint32_t lane_prefix(uint64_t mask) {
  return __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}

// A workgroup's share of a queue of n items in a grid of G workgroups:
// chunks of kShareChunk consecutive items dealt round-robin (chunk c to
// workgroup c mod G), so every workgroup gets items from all over the queue
// (regions of the image differ widely in cost) while a wave's refill still
// takes neighbouring items.  kShareChunk 0: one contiguous share each.
#ifndef PT_SHARE_CHUNK
#define PT_SHARE_CHUNK 256
#endif
constexpr uint32_t kShareChunk = PT_SHARE_CHUNK;
__device__ inline uint32_t share_size(uint32_t n, uint32_t wg, uint32_t G) {
  if (!kShareChunk) {
    const uint32_t per = (n + G - 1) / G, a = min(n, wg * per);
    return min(n, a + per) - a;
  }
  const uint32_t nc = (n + kShareChunk - 1) / kShareChunk;  // chunks, the last one possibly partial
  if (nc <= wg) return 0u;
  const uint32_t mine = (nc - 1 - wg) / G + 1;
  uint32_t items = mine * kShareChunk;
  if ((nc - 1) % G == wg) items -= nc * kShareChunk - n;  // this workgroup holds the partial chunk
  return items;
}
// queue index of item v (< share_size) of workgroup wg
__device__ inline uint32_t share_item(uint32_t v, uint32_t n, uint32_t wg, uint32_t G) {
  if (!kShareChunk) return min(n, wg * ((n + G - 1) / G)) + v;
  return ((v / kShareChunk) * G + wg) * kShareChunk + v % kShareChunk;
}

// Sum of a value over the wave's 64 lanes (every lane gets the sum).
__device__ inline uint32_t wave_sum(uint32_t v) {
  for (int d = 32; d >= 1; d >>= 1) v += (uint32_t)__shfl_xor((int)v, d);
  return v;
}

// ------------------------------------------------------------- signatures
constexpr uint64_t kFnvOffset = 0xcbf29ce484222325ull;
constexpr uint64_t kFnvPrime = 0x100000001b3ull;

__device__ inline uint64_t sig_word(uint64_t h, uint32_t w) {
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    h ^= (uint64_t)((w >> (8 * i)) & 0xFFu);
    h *= kFnvPrime;
  }
  return h;
}

// Tail events of a vertex, kept until the shadow ray of that vertex is
// resolved: lobe code (8 bits, 0xFF none), roulette (2 bits: 0 none,
// 1 survived, 2 killed), end reason (3 bits, 7 none).
__device__ inline uint32_t tail_pack(int lobe, int rr, int end) {
  return ((uint32_t)(lobe & 0xFF)) | ((uint32_t)rr << 8) | ((uint32_t)(end & 7) << 10);
}
__device__ inline uint64_t sig_tail(uint64_t h, uint32_t tail) {
  uint32_t lobe = tail & 0xFFu, rr = (tail >> 8) & 3u, end = (tail >> 10) & 7u;
  if (lobe != 0xFFu) { h = sig_word(h, 3); h = sig_word(h, lobe); }
  if (rr != 0u) { h = sig_word(h, 4); h = sig_word(h, rr == 2u ? 1u : 0u); }
  if (end != 7u) { h = sig_word(h, 6); h = sig_word(h, end); }
  return h;
}

// ----------------------------------------------------------------- stacks
// Traversal stack: the first kLdsStack entries of each lane in LDS as
// (ref, key) pairs, entry e of lane l at [e][l] (one 8-byte access per push
// or pop, conflict-free), deeper entries in a global spill area.  `top` is the
// place of the next entry as if all of them were in LDS; the pointer keeps its
// address space so pushes and pops are LDS accesses, not flat ones.
// The capacity (3 x BVH depth + 4) bounds a depth-first walk that pushes at
// most three siblings per level.
typedef __attribute__((address_space(3))) unsigned long long lds_u64;
__device__ inline unsigned long long stack_entry(uint32_t r, float k) {
  return (unsigned long long)r | ((unsigned long long)f2u(k) << 32);
}
struct DevStack {
  lds_u64 *base, *top;
  bool overflow;
  __device__ inline lds_u64* lds_end() const { return base + kLdsStack * kBlock; }
  __device__ inline bool room(int n) const { return top <= lds_end() - n * kBlock; }  // n more entries fit in LDS
  __device__ inline void push_lds(unsigned long long e) {
    *top = e;
    top += kBlock;
  }
  __device__ inline unsigned long long* spill_entry(const SceneDev& S, uint32_t i) const {
    return reinterpret_cast<unsigned long long*>(S.spill) + (size_t)i * S.spill_stride +
           (blockIdx.x * kBlock + threadIdx.x);
  }
  __device__ inline void push(const SceneDev& S, unsigned long long e) {
    if (room(1)) {
      push_lds(e);
      return;
    }
    const int i = (int)((uint32_t)(top - lds_end()) / kBlock);  // entries in the spill area
    if (i >= S.stack_cap - kLdsStack) {  // (a capacity below kLdsStack: none)
      overflow = true;
      return;
    }
    *spill_entry(S, (uint32_t)i) = e;
    top += kBlock;
  }
  __device__ inline unsigned long long pop(const SceneDev& S) {
    top -= kBlock;
    // the LDS read is unconditional (clamped place) so it stays an LDS access;
    // the rare spill read replaces it
    lds_u64* last = lds_end() - kBlock;
    unsigned long long w = *(top < last ? top : last);
    if (top > last)  // a relaxed atomic load is never merged with the LDS read into a flat load
      w = __hip_atomic_load(spill_entry(S, (uint32_t)(top - lds_end()) / kBlock), __ATOMIC_RELAXED,
                            __HIP_MEMORY_SCOPE_WAVEFRONT);
    return w;
  }
  __device__ inline void clear() { top = base; }
  __device__ inline bool empty() const { return top == base; }
};
__device__ inline DevStack make_stack(unsigned long long* shared_stack) {
  DevStack st;
  st.base = st.top = (lds_u64*)(shared_stack + threadIdx.x);
  st.overflow = false;
  return st;
}

// ------------------------------------------------------------------ lights
// sin(theta) as |(x, z)| and theta = atan2(|(x, z)|, y): near the poles
// acos(y) and sqrt(1 - y^2) lose most of their FP32 digits to cancellation
// (at 0.4 degrees from the zenith sqrt(1 - y^2) is off by ~1e-3 relative,
// which moves the environment's pdf and every MIS weight that uses it).
__device__ inline int env_texel(const SceneDev& S, V3 d, float& sin_t) {
  const float sxz = sqrtf(d.x * d.x + d.z * d.z);
  float th = atan2f(sxz, d.y), ph = atan2f(d.x, -d.z);
  float u = ph * (0.5f / kPi) + 0.5f, v = th * (1.0f / kPi);
  int c = (int)floorf(u * (float)S.env_w), r = (int)floorf(v * (float)S.env_h);
  c = min(max(c, 0), S.env_w - 1);
  r = min(max(r, 0), S.env_h - 1);
  sin_t = sxz;
  return r * S.env_w + c;
}

// e: the texel
__device__ inline float env_pdf_texel(const SceneDev& S, int texel, const float4& e, float sin_t) {
  int r = texel / S.env_w;
  float P = S.env_row_pmf[r] * e.w;
  if (!(sin_t > 0.0f)) return 0.0f;
  return (float)S.env_w * (float)S.env_h * P / (2.0f * kPi * kPi * sin_t);
}

// bucket i with cdf[i] <= u < cdf[i+1], skipping empty buckets
__device__ inline int cdf_invert(const float* cdf, int n, float u) {
  int lo = 0, hi = n;
  while (hi - lo > 1) {
    int mid = (lo + hi) >> 1;
    if (cdf[mid] <= u) lo = mid;
    else hi = mid;
  }
  int i = lo;
  while (i < n - 1 && !(cdf[i + 1] > cdf[i])) i++;
  while (i > 0 && !(cdf[i + 1] > cdf[i])) i--;
  return i;
}

// The same bucket through a guide table: guide[g] is the largest i with
// cdf[i] <= g/G, so for u in [g/G, (g+1)/G) the answer lies in
// [guide[g], guide[g+1]] and the binary search starts there (u * G is exact:
// u has 24 bits and G is a power of two).
__device__ inline int cdf_invert_guided(const float* cdf, int n, float u, const int32_t* guide, int G) {
  int g = min(G - 1, (int)(u * (float)G));
  int lo = guide[g], hi = g + 1 < G ? min(n, guide[g + 1] + 1) : n;
  while (hi - lo > 1) {
    int mid = (lo + hi) >> 1;
    if (cdf[mid] <= u) lo = mid;
    else hi = mid;
  }
  int i = lo;
  while (i < n - 1 && !(cdf[i + 1] > cdf[i])) i++;
  while (i > 0 && !(cdf[i + 1] > cdf[i])) i--;
  return i;
}

struct LightSample {
  V3 wl;
  float dist, pdf;
  V3 Le;
  uint32_t id;
  bool ok;
};

__device__ inline LightSample sample_light(const SceneDev& S, V3 p, float usel, float u1, float u2) {
  LightSample ls;
  ls.ok = false;
  ls.pdf = 0.0f;
  ls.dist = 0.0f;
  ls.Le = v3(0.0f, 0.0f, 0.0f);
  ls.wl = v3(0.0f, 0.0f, 1.0f);
  ls.id = 0xFFFFFFFFu;
  if (S.p_env <= 0.0f && S.n_lights == 0) return ls;
  if (usel < S.p_env) {
    int W = S.env_w, H = S.env_h;
    int r = cdf_invert_guided(S.env_row_cdf, H, u1, S.env_row_guide, kEnvRowGuide);
    float pr = S.env_row_pmf[r];
    float du = pr > 0.0f ? (u1 - S.env_row_cdf[r]) / pr : 0.5f;
    const float* ccdf = S.env_col_cdf + (size_t)r * (W + 1);
    int c = cdf_invert_guided(ccdf, W, u2, S.env_col_guide + (size_t)r * kEnvColGuide, kEnvColGuide);
    const float4 e = S.env[(size_t)r * W + c];
    float pc = e.w;
    float dv = pc > 0.0f ? (u2 - ccdf[c]) / pc : 0.5f;
    float uu = ((float)c + dv) / (float)W, vv = ((float)r + du) / (float)H;
    float th = kPi * vv, ph = 2.0f * kPi * (uu - 0.5f);
    float st, ct, sp, cp;
    sincosf(th, &st, &ct);
    sincosf(ph, &sp, &cp);
    ls.wl = v3(st * sp, ct, -st * cp);
    ls.dist = INFINITY;
    ls.id = 0x80000000u | (uint32_t)(r * W + c);
    if (!(st > 0.0f)) return ls;
    float P = pr * pc;
    ls.pdf = S.p_env * (float)W * (float)H * P / (2.0f * kPi * kPi * st);
    ls.Le = v3(e.x, e.y, e.z);
    ls.ok = ls.pdf > 0.0f;
    return ls;
  }
  float ut = S.p_env > 0.0f ? (usel - S.p_env) / (1.0f - S.p_env) : usel;
  int k = cdf_invert(S.light_cdf, S.n_lights, ut);
  ls.id = (uint32_t)k;
  const LightTri& L = S.lights[k];
  float sq = sqrtf(u1);
  float b0 = 1.0f - sq, b1 = u2 * sq;
  V3 q = v3(L.p0.x, L.p0.y, L.p0.z) * b0 + v3(L.p1.x, L.p1.y, L.p1.z) * b1 +
         v3(L.p2.x, L.p2.y, L.p2.z) * (1.0f - b0 - b1);
  V3 to = q - p;
  float d2 = dot(to, to);
  float dd = sqrtf(d2);
  if (!(dd > 0.0f)) return ls;
  ls.wl = to * (1.0f / dd);
  ls.dist = dd;
  float cl = -dot(v3(L.ng.x, L.ng.y, L.ng.z), ls.wl);
  if (cl <= 0.0f) return ls;
  ls.pdf = L.p1.w * d2 / (cl * L.p0.w);
  ls.Le = v3(L.Le.x, L.Le.y, L.Le.z);
  ls.ok = ls.pdf > 0.0f;
  return ls;
}

__device__ inline float pow_heuristic(float a, float b) {
  float a2 = a * a, b2 = b * b;
  return a2 + b2 > 0.0f ? a2 / (a2 + b2) : 0.0f;
}

__device__ inline bool finite3(V3 c) { return isfinite(c.x) && isfinite(c.y) && isfinite(c.z); }

// Pixel (x, y) of place p of a w x h tile: rows in bands of kPixBlock, each
// band in blocks of kPixBlock columns (the last band and block of a band may
// be narrower), row-major inside a block.  A bijection of [0, w h) for any w
// and h.  Neighbouring slots are then neighbouring pixels in both directions,
// and the samples of one pixel are adjacent, so a wave's rays start in a small
// square of the image.  Icosphere field 512x512, 100 spp: rows instead of
// blocks 20.1 ms, blocks of 4 19.8, of 8 19.9, of 16 19.9 with the samples
// apart (16 pixels, then their next sample); 19.3 with the samples adjacent.
#ifndef PT_PIX_BLOCK
#define PT_PIX_BLOCK 8
#endif
constexpr uint32_t kPixBlock = PT_PIX_BLOCK;
__device__ inline void place_pixel(uint32_t p, uint32_t w, uint32_t h, uint32_t& x, uint32_t& y) {
  const uint32_t band = p / (kPixBlock * w), r = p - band * (kPixBlock * w);
  const uint32_t bh = min(kPixBlock, h - band * kPixBlock);
  const uint32_t blk = bh == kPixBlock ? r / (kPixBlock * kPixBlock) : r / (kPixBlock * bh);
  const uint32_t q = r - blk * (kPixBlock * bh), bw = min(kPixBlock, w - blk * kPixBlock);
  const uint32_t ly = bw == kPixBlock ? q / kPixBlock : q / bw;
  x = blk * kPixBlock + (q - ly * bw);
  y = band * kPixBlock + ly;
}

// Pixel and random numbers of a path slot (`sample`: the pass's first): sampling
// paths (slot = place * spp + sample of the pass), then the radiance cache's
// training paths on their strided pixel set.
__device__ inline Rng slot_rng(const PathsDev& P, uint32_t slot, uint32_t sample, uint32_t k0, uint32_t k1,
                               uint32_t& px, uint32_t& py) {
  if (slot >= (uint32_t)P.n_render) {
    const uint32_t pix =
        (uint32_t)(((uint64_t)(slot - (uint32_t)P.n_render) * P.pix_stride + P.pix_off) % P.pix_total);
    px = pix % P.img_w;
    py = pix / P.img_w;
    return Rng{pix, P.train_sample, k0, k1};
  }
  const uint32_t place = slot / P.spp;
  place_pixel(place, (uint32_t)P.w, (uint32_t)P.h, px, py);
  px += (uint32_t)P.x0;
  py += (uint32_t)P.y0;
  return Rng{py * P.img_w + px, sample + (slot - place * P.spp), k0, k1};
}

// ------------------------------------------------------------------ queues
// A ray or shadow queue is kShards segments, each with its own counter on a
// 128-byte line of its own: atomics on one line take 11.4 ns each, one after
// the other, so a single counter held the shading of 33M paths (one append per
// 256 paths and queue) at 1.5 ms whatever else it did.  The shading kernels
// append block k of a class to segment k mod kShards, which fills the segments
// evenly, and workgroup g of a consumer takes from segment g mod kShards.
// The ray queue of the first vertex is every slot in order, with no array.
struct QueueShare {
  uint32_t n;       // items of the segment (kQueueAll: of the pass)
  uint32_t wg, G;   // this workgroup among those that share them
  const uint32_t* q;
  __device__ inline uint32_t slot(const PathsDev& P, uint32_t i) const { return q ? q[i] : i; }
};
__device__ inline QueueShare queue_share(const PathsDev& P, int cur) {
  if (cur == kQueueAll) return QueueShare{(uint32_t)P.n, blockIdx.x, gridDim.x, nullptr};
  const uint32_t seg = blockIdx.x % kShards;
  return QueueShare{P.counts[count_ray(seg, cur)], blockIdx.x / kShards, gridDim.x / kShards,
                    P.q_ray[cur] + (size_t)seg * P.seg_cap};
}

// ---------------------------------------------------------------- generate
template <bool DEBUG>
__global__ __launch_bounds__(kBlock) void k_generate(PathsDev P, CamDev C, uint32_t sample, uint32_t k0,
                                                     uint32_t k1) {
  int n = P.n;
  for (int slot = blockIdx.x * kBlock + threadIdx.x; slot < n; slot += gridDim.x * kBlock) {
    uint32_t px, py;
    const Rng rng = slot_rng(P, (uint32_t)slot, sample, k0, k1, px, py);
    U4 r = rng.block(0u, 0u);
    float fx = (float)px + u01(r.x), fy = (float)py + u01(r.y);
    float x = (2.0f * fx / (float)C.W - 1.0f) * C.tan_half * C.aspect;
    float y = (1.0f - 2.0f * fy / (float)C.H) * C.tan_half;
    V3 d = normalize(v3(C.R[0], C.R[1], C.R[2]) * x + v3(C.U[0], C.U[1], C.U[2]) * y + v3(C.F[0], C.F[1], C.F[2]));
    PathRec& rec = P.path[slot];
    rec.o = make_float4(C.eye[0], C.eye[1], C.eye[2], u2f(0xFFFFFFFFu));
    rec.d = make_float4(d.x, d.y, d.z, u2f(0xFFFFFFFFu));
    rec.hit = make_float4(INFINITY, 0.0f, 0.0f, u2f(0xFFFFFFFFu));
    rec.beta = make_float4(1.0f, 1.0f, 1.0f, 0.0f);
    P.L[slot] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    if (P.eta) P.eta[slot] = 1.0f;
    if (DEBUG) P.sig[slot] = kFnvOffset;
    if (P.rec && slot >= P.n_render)
      for (int r = 0; r < P.rec_depth; ++r)
        P.rec[((size_t)(slot - P.n_render) * P.rec_depth + r) * kNrcRecFloats + 18] = 0.0f;
  }
  if (blockIdx.x == 0) {
    if (threadIdx.x < kShards) P.counts[count_shadow(threadIdx.x)] = 0u;
    if (threadIdx.x == 0) P.counts[kCountQuery] = 0u;
  }
}

__global__ void k_zero_u32(uint32_t* p) { *p = 0u; }

// Empty the next ray queue and the class queues (the shadow queue is still
// being traced; k_bin empties it).
__global__ void k_reset_counts(uint32_t* counts, int next_queue) {
  const uint32_t i = threadIdx.x;
  if (i < kShards) counts[count_ray(i, next_queue)] = 0u;
  else if (i < kShards + kNumClasses) counts[count_class(i - kShards)] = 0u;
}

// ------------------------------------------------------------------ extend
// Persistent lanes: a workgroup takes its items of the ray queues (chunks of
// kShareChunk dealt round-robin; ray queries: one run of the array) through an
// LDS counter.  A lane advances its own walk one node or one leaf per loop
// iteration; once kRefill lanes of a wave are idle they take new rays, so the
// wave's SIMD lanes stay busy instead of waiting for the longest ray of a
// fixed batch.  Boxes are visited in the order of the recursive walk (entry
// distance, then reference); their test is wider than that walk's, never
// narrower, and the triangle test is the same, so the closest hit is unchanged
// bit for bit.
constexpr uint32_t kNoInst = 0xFFFFFFFFu;
#ifndef PT_REFILL
#define PT_REFILL 20  // 10 / 16 / 20 / 24: field 87.7 / 86.9 / 86.4 / 86.8 ms, instanced 117.4 / 114.3 / 112.9 / 112.6
#endif
constexpr uint32_t kRefill = PT_REFILL;  // idle lanes that trigger a refill
#ifndef PT_LEAF_WAIT
#define PT_LEAF_WAIT 1
#endif
#ifndef PT_LEAF_WAIT_DEN
#define PT_LEAF_WAIT_DEN 1
#endif
// traversal kernels: lanes at a leaf wait until kLeafWait x their number
// reaches kLeafWaitDen x the number of lanes at inner nodes (0: no waiting)
constexpr uint32_t kLeafWait = PT_LEAF_WAIT, kLeafWaitDen = PT_LEAF_WAIT_DEN;
#ifndef PT_TAIL_SHADE_WAIT
#define PT_TAIL_SHADE_WAIT 1
#endif
// tail kernel: lanes waiting to shade go ahead once kTailShadeWait x their
// number reaches the number of lanes still walking (a large value shades at
// once, as soon as a walk ends)
constexpr uint32_t kTailShadeWait = PT_TAIL_SHADE_WAIT;
#ifndef PT_TAIL_PATHS_PER_GROUP
#define PT_TAIL_PATHS_PER_GROUP 512
#endif
// tail kernel beside the next pass: paths per workgroup (two per lane)
constexpr uint64_t kTailPathsPerGroup = PT_TAIL_PATHS_PER_GROUP;
#ifndef PT_TRACE_WAVES
#define PT_TRACE_WAVES 6
#endif
// minimum waves per SIMD the traversal kernel is compiled for: 6 is the most that
// needs no scratch (field render at 4 / 5 / 6 / 7: 107.5 / 101.4 / 97.5 / 98.2 ms)
constexpr int kTraceWaves = PT_TRACE_WAVES;
#ifndef PT_TRACE_WAVES_2
#define PT_TRACE_WAVES_2 5
#endif
constexpr int kTraceWaves2 = PT_TRACE_WAVES_2;  // two-level scenes: the world-space ray takes registers too (6: 124.6 ms, 5: 119.4)

// Ray of a lane's walk in the space of the current level: what the triangle
// test reads (the same values as ray_prepare's, bit for bit) and the box test's
// constants.
struct LaneRay {
  float ox, oy, oz;
  float Sx, Sy, Sz;
  uint32_t k;  // kx, ky, kz, two bits each (never 0; two-level scenes: 0 while the box test's constants are the world ray's)
  // Box test of a plane p of axis a: t = fma(p, i_a, c) with c = -(o_a i_a) moved
  // by slack to the safe side, n_a for the plane the ray meets first and f_a for
  // the other.
  float ix, iy, iz, nx, ny, nz, fx, fy, fz;
  float wox, woy, woz, wdx, wdy, wdz;  // world-space ray (two-level scenes)
  uint32_t skip_inst, skip_prim;
  uint32_t cur;      // next reference to process, kEmpty: pop
  float cur_key;     // its entry distance (two-level scenes)
  uint32_t inst;     // instance of the current mesh walk, kNoInst at the top level
  lds_u64* base;     // stack top when that mesh walk started
  bool any;          // shadow ray: stop at the first accepted triangle (kWalkPerLane walks)
  // best hit so far (tri kEmpty: none, t is the ray's tmax)
  float t, b1, b2;
  uint32_t tri, best_inst;
  __device__ inline bool found() const { return tri != kEmpty; }
};

// ---- top of the tree in LDS
// A third of all node visits go to the first kTopNodes nodes in breadth-first
// order.  The traversal kernels keep copies of them in LDS (one per workgroup),
// where a read does not go through the CU's load path (2^20 incoherent rays 330
// -> 318 us); their references to each other carry kTopBit and the place in the
// table, others are as in the tree.  40 nodes fit six workgroups a CU (64 with
// five: the icosphere field renders in 101.4 ms against 97.5).
typedef __attribute__((address_space(3))) unsigned char lds_byte;
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) f32x4 lds_f32x4;
typedef __attribute__((address_space(3))) u32x4 lds_u32x4;
constexpr uint32_t kTopStride = 144;  // bytes per node in LDS: 16 more than the node, to spread the banks
constexpr uint32_t kTopLds = kTopNodes * kTopStride;
__device__ inline lds_byte* top_load(const SceneDev& S, unsigned char* shared) {
  for (uint32_t i = threadIdx.x; i < kTopNodes * 8u; i += kBlock)
    *(lds_u32x4*)((lds_byte*)shared + (i >> 3) * kTopStride + (i & 7u) * 16u) =
        reinterpret_cast<const u32x4*>(S.top)[i];
  return (lds_byte*)shared;
}

__device__ inline float widen_limit(float t) { return fmaf(fabsf(t), 1.9073486328125e-06f, t); }  // t + 2^-19 |t|

// Box-test constants of one axis.  The box only prunes, so it needs safe, not
// exact, distances: with inv within 1 ulp of 1/d, fma(p, inv, -(o inv)) is off by
// at most 4 u |t| + u |o inv| (u = 2^-24); the constants move by 4 u |o inv| to
// the safe side, the far distance and the pruning limit widen by 64 u and 32 u
// relative, so every box is at least as wide as one widened by 16 u computed from
// (p - o) / d.  A component smaller than tiny counts as tiny with a slack of
// reach in t: finite products instead of 0 x inf, and the axis still prunes.
// The ray leaves its true line by less than tiny t that way, the slack in space is
// tiny reach, so no box is lost before t = reach.
__device__ inline void box_axis(float o, float d, float reach, float& inv, float& n, float& f) {
  inv = __builtin_amdgcn_rcpf(d);
  const float c = o * inv, e = fmaf(fabsf(c), 2.384185791015625e-07f, reach);
  n = -c - e;
  f = -c + e;
}
// Byte offset in a node of the planes that a ray with inverse direction inv meets first on axis a (the others' is this ^ 16).
__device__ inline uint32_t near_offset(uint32_t a, float inv) { return (32u * a) | ((f2u(inv) >> 27) & 16u); }

// Both follow the direction's largest component m, for a ray of any length: tiny is
// 2^-100 m (2^-126 at least, whose reciprocal is finite) and reach 2^50 / m, about
// 10^15 units of space; the slack in space is 2^-50 (2^-76 / m below m = 2^-26).
// Below m = 2^-128 the triangle test's 1 / m is infinite and no hit is possible.
__device__ inline void lane_box(LaneRay& L, float ox, float oy, float oz, float dx, float dy, float dz) {
#pragma clang fp contract(off)
  const float ax = fabsf(dx), ay = fabsf(dy), az = fabsf(dz);
  float m = fmaxf(fmaxf(ax, ay), az), rx = 0.0f, ry = 0.0f, rz = 0.0f;
  const float kTiny = 7.888609052210118e-31f, kLeast = 1.1754943508222875e-38f;  // 2^-100, 2^-126
  if (fminf(fminf(ax, ay), az) < fmaxf(m * kTiny, kLeast)) {  // rare: most rays have no small component
    if (m < 2.938735877055719e-39f) m = 1.0f;  // 2^-128
    const float tiny = fmaxf(m * kTiny, kLeast), reach = __builtin_amdgcn_rcpf(m) * 1125899906842624.0f;  // 2^50
    if (ax < tiny) {
      dx = copysignf(tiny, dx);
      rx = reach;
    }
    if (ay < tiny) {
      dy = copysignf(tiny, dy);
      ry = reach;
    }
    if (az < tiny) {
      dz = copysignf(tiny, dz);
      rz = reach;
    }
  }
  box_axis(ox, dx, rx, L.ix, L.nx, L.fx);
  box_axis(oy, dy, ry, L.iy, L.ny, L.fy);
  box_axis(oz, dz, rz, L.iz, L.nz, L.fz);
}

// The ray (o, d) of the level whose triangles are tested next.
__device__ inline void lane_ray(LaneRay& L, float ox, float oy, float oz, float dx, float dy, float dz) {
  const RayPre r = ray_prepare(ox, oy, oz, dx, dy, dz);
  L.ox = ox;
  L.oy = oy;
  L.oz = oz;
  L.Sx = r.Sx;
  L.Sy = r.Sy;
  L.Sz = r.Sz;
  L.k = (uint32_t)(r.kx | (r.ky << 2) | (r.kz << 4));
  lane_box(L, ox, oy, oz, dx, dy, dz);
}

template <bool TWO>
__device__ inline void lane_start(LaneRay& L, float ox, float oy, float oz, float dx, float dy, float dz,
                                  float tmax, uint32_t skip_inst, uint32_t skip_prim, uint32_t root) {
  if (TWO) {  // the top level tests no triangles
    L.wox = ox;
    L.woy = oy;
    L.woz = oz;
    L.wdx = dx;
    L.wdy = dy;
    L.wdz = dz;
    lane_box(L, ox, oy, oz, dx, dy, dz);
    L.k = 0u;
  } else {
    lane_ray(L, ox, oy, oz, dx, dy, dz);
  }
  L.skip_inst = skip_inst;
  L.skip_prim = skip_prim;
  L.cur = root;
  L.cur_key = -INFINITY;
  L.inst = kNoInst;
  L.t = tmax;
  L.b1 = L.b2 = 0.0f;
  L.tri = L.best_inst = kEmpty;
}

// Walk kinds of lane_step: closest hit, any hit (shadow rays), or the kind
// the lane's own `any` flag names.
enum { kWalkClosest = 0, kWalkAny = 1, kWalkPerLane = 2 };

// Order two stack entries by key, then ref: as doubles, (key, ref) pairs with
// the key in the high word order as the keys do (keys are not NaN and at most
// +inf, whose pattern is a finite double's), and one 64-bit minimum and maximum
// take the place of a compare and four selects.  (asm: the builtins would first
// quieten every operand.)
__device__ inline void entry_sort(double& a, double& b) {
  double lo, hi;
  asm("v_min_f64 %0, %1, %2" : "=v"(lo) : "v"(a), "v"(b));
  asm("v_max_f64 %0, %1, %2" : "=v"(hi) : "v"(a), "v"(b));
  a = lo;
  b = hi;
}
__device__ inline float entry_key(double e) { return u2f((uint32_t)(__double_as_longlong(e) >> 32)); }
__device__ inline uint32_t entry_ref(double e) { return (uint32_t)__double_as_longlong(e); }
__device__ inline double entry_make(uint32_t ref, float key) {
  return __longlong_as_double((long long)stack_entry(ref, key));
}

struct TriRay {
  float ox, oy, oz, Sx, Sy, Sz;
  int kx, ky, kz;
};

// Test the triangles of a leaf (any: stop at the first accepted one); true if one was accepted.
template <bool COUNT, bool TWO>
__device__ inline bool lane_leaf(const SceneDev& S, LaneRay& L, float tmin, bool any, uint32_t& ntri) {
  const uint32_t first = leaf_first(L.cur), cnt = leaf_count(L.cur);
  const TriRay r{L.ox, L.oy, L.oz, L.Sx, L.Sy, L.Sz, (int)(L.k & 3u), (int)((L.k >> 2) & 3u), (int)(L.k >> 4)};
  bool found = false;
  for (uint32_t j = 0; j < cnt; ++j) {
    const TriRec tr = S.tris[first + j];
    if (COUNT) ntri++;
    const uint32_t prim = f2u(tr.a.w);
    // intersect before the origin-triangle check so the record's three loads
    // issue together instead of waiting on the primitive id first
    float t, b1, b2;
    if (!tri_intersect(r, tr.a, tr.b, tr.c, t, b1, b2)) continue;
    if (prim == L.skip_prim && (!TWO || L.inst == L.skip_inst)) continue;
    if (!(t > tmin && t <= L.t)) continue;
    if (t == L.t) {  // ties: the smallest (instance, primitive)
      if (!L.found()) continue;  // t is tmax
      if (TWO && L.inst != L.best_inst) {
        if (L.inst > L.best_inst) continue;
      } else if (prim >= f2u(S.tris[L.tri].a.w)) {
        continue;
      }
    }
    L.t = t;
    L.b1 = b1;
    L.b2 = b2;
    L.tri = first + j;
    if (TWO) L.best_inst = L.inst;
    found = true;
    if (any) return true;
  }
  return found;
}

// What bounds the walk (icosphere field, 33M paths a pass): a divergent 16-byte
// load costs the CU's load path one cycle per lane, so a node's seven parts cost
// seven cycles per lane, beside the node step's VALU work.  Sub and multiply per
// plane, minima for the near plane and compare-select sorting (0.92 / 0.81 VALU
// issue at bounces 0 / 1) became one fma per plane with the plane chosen by
// address and a 64-bit minimum sort: 3.85 -> 3.48 and 8.4 -> 7.6 ms at 0.67 / 0.61
// issue, 33 % fewer VALU instructions.  What is left is the latency of the ~14 of
// a wave's ~30 nodes that miss the L1.
// Slower: quads or the whole wave fetching nodes cooperatively into LDS (field
// render 121-130 ms against 99), rays sorted by direction (traversal +20 %).
//
// One step of a lane's walk: visit one node, or test one leaf, then pop the
// next entry that can still hold a closer hit.  In two-level scenes a
// top-level leaf pushes its instances as entries (leaf bit, count 0,
// instance id) that start a mesh walk on top of the stack.  Returns true when
// the walk is over (any-hit walks: also at the first accepted triangle).
// TOP: the walk started at the table's root (`top`: its copy in LDS).
template <int KIND, bool COUNT, bool TWO, bool TOP>
__device__ inline bool lane_step(const SceneDev& S, LaneRay& L, float tmin, DevStack& st, lds_byte* top,
                                 uint32_t& nvis, uint32_t& ntri, uint32_t& ninst) {
  const bool any = KIND == kWalkAny || (KIND == kWalkPerLane && L.any);
  const uint32_t cur = L.cur;
  if (cur != kEmpty) {
    if (!ref_is_leaf(cur)) {
      if (COUNT) nvis++;
      const float tlim = widen_limit(L.t);
      const uint32_t sx = near_offset(0, L.ix), sy = near_offset(1, L.iy), sz = near_offset(2, L.iz);
      const char* nodes = reinterpret_cast<const char*>(S.nodes);
      f32x4 an, af, bn, bf, cn, cf;
      u32x4 ch;
      if (TOP && (cur & kTopBit)) {
        lds_byte* q = top + (cur & ~kTopBit) * kTopStride;
        an = *(lds_f32x4*)(q + sx);
        af = *(lds_f32x4*)(q + (sx ^ 16u));
        bn = *(lds_f32x4*)(q + sy);
        bf = *(lds_f32x4*)(q + (sy ^ 16u));
        cn = *(lds_f32x4*)(q + sz);
        cf = *(lds_f32x4*)(q + (sz ^ 16u));
        ch = *(lds_u32x4*)(q + 96);
      } else if (S.small_nodes) {  // node bytes below 2^32: 32-bit offsets from the base
        const uint32_t o = cur << 7, x = o + sx, y = o + sy, z = o + sz;
        an = *reinterpret_cast<const f32x4*>(nodes + x);
        af = *reinterpret_cast<const f32x4*>(nodes + (x ^ 16u));
        bn = *reinterpret_cast<const f32x4*>(nodes + y);
        bf = *reinterpret_cast<const f32x4*>(nodes + (y ^ 16u));
        cn = *reinterpret_cast<const f32x4*>(nodes + z);
        cf = *reinterpret_cast<const f32x4*>(nodes + (z ^ 16u));
        ch = *reinterpret_cast<const u32x4*>(nodes + (o + 96u));
        asm volatile("; 32-bit node offsets" ::: "memory");  // keeps the two forms apart
      } else {
        const char* q = nodes + ((uint64_t)cur << 7);
        an = *reinterpret_cast<const f32x4*>(q + sx);
        af = *reinterpret_cast<const f32x4*>(q + (sx ^ 16u));
        bn = *reinterpret_cast<const f32x4*>(q + sy);
        bf = *reinterpret_cast<const f32x4*>(q + (sy ^ 16u));
        cn = *reinterpret_cast<const f32x4*>(q + sz);
        cf = *reinterpret_cast<const f32x4*>(q + (sz ^ 16u));
        ch = *reinterpret_cast<const u32x4*>(q + 96);
        asm volatile("; 64-bit node addresses" ::: "memory");
      }
      // entry of child c: its box's entry distance, +inf for a missed box
      auto child = [&](float ax, float ay, float az, float bx, float by, float bz, uint32_t ref) -> double {
        const float tn = fmaxf(fmaxf(fmaxf(fmaf(ax, L.ix, L.nx), fmaf(ay, L.iy, L.ny)), fmaf(az, L.iz, L.nz)), tmin);
        const float tf = fminf(fminf(fmaf(bx, L.ix, L.fx), fmaf(by, L.iy, L.fy)), fmaf(bz, L.iz, L.fz));
        const float te = fminf(fmaf(fabsf(tf), 3.814697265625e-06f, tf), tlim);  // tf + 2^-18 |tf|
        return entry_make(ref, tn <= te ? tn : INFINITY);
      };
      double e0 = child(an.x, bn.x, cn.x, af.x, bf.x, cf.x, ch.x), e1 = child(an.y, bn.y, cn.y, af.y, bf.y, cf.y, ch.y);
      double e2 = child(an.z, bn.z, cn.z, af.z, bf.z, cf.z, ch.z), e3 = child(an.w, bn.w, cn.w, af.w, bf.w, cf.w, ch.w);
      entry_sort(e0, e1);
      entry_sort(e2, e3);
      entry_sort(e0, e2);
      entry_sort(e1, e3);
      entry_sort(e1, e2);
      const bool h1 = entry_key(e1) < INFINITY, h2 = entry_key(e2) < INFINITY, h3 = entry_key(e3) < INFINITY;
      const auto bits = [](double e) { return (unsigned long long)__double_as_longlong(e); };
      if (st.room(3)) {
        if (h3) st.push_lds(bits(e3));
        if (h2) st.push_lds(bits(e2));
        if (h1) st.push_lds(bits(e1));
      } else {
        if (h3) st.push(S, bits(e3));
        if (h2) st.push(S, bits(e2));
        if (h1) st.push(S, bits(e1));
      }
      if (entry_key(e0) < INFINITY) {
        L.cur = entry_ref(e0);
        if (TWO) L.cur_key = entry_key(e0);
        return false;
      }
    } else if (TWO && L.inst == kNoInst) {
      const uint32_t first = leaf_first(cur), cnt = leaf_count(cur);
      if (cnt == 0) {  // an instance entry: walk its mesh in object space
        const InstRec& I = S.insts[first];
        if (COUNT) ninst++;
        float o[3], d[3];
        ray_to_object(I.w2o, L.wox, L.woy, L.woz, L.wdx, L.wdy, L.wdz, o, d);
        lane_ray(L, o[0], o[1], o[2], d[0], d[1], d[2]);
        L.inst = first;
        L.base = st.top;
        L.cur = I.blas_root;
        return false;
      }
      for (int j = (int)cnt - 1; j >= 0; --j) st.push(S, stack_entry(kLeafBit | S.tlas_items[first + j], L.cur_key));
    } else {
      if (lane_leaf<COUNT, TWO>(S, L, tmin, any, ntri) && any) return true;
    }
    L.cur = kEmpty;
  }
  while (true) {
    if (TWO && L.inst != kNoInst && st.top == L.base) L.inst = kNoInst;  // mesh walk over: back to the top level
    if (st.empty()) return true;
    const unsigned long long e = st.pop(S);
    const float k = u2f((uint32_t)(e >> 32));
    if (k <= widen_limit(L.t)) {
      L.cur = (uint32_t)e;
      if (TWO) L.cur_key = k;
      if (TWO && L.inst == kNoInst && L.k != 0u && !ref_is_leaf(L.cur)) {
        // a top-level node after a mesh walk: its boxes need the world ray's constants (most entries
        // here are instances, which do not)
        lane_box(L, L.wox, L.woy, L.woz, L.wdx, L.wdy, L.wdz);
        L.k = 0u;
      }
      return false;
    }
  }
}

// The persistent-lane loop shared by the traversal kernels.  Src supplies
// start(i, L) (load item i into the lane) and finish(i, L, found).  A lane whose
// walk has ended keeps its result until the next refill, where all such lanes
// finish together: one or two lanes end at almost every step, and finishing them
// at once put two dependent loads into every step of the wave (field of spheres
// 1920x1080 64 spp 88.4 -> 86.4 ms, instanced 115.4 -> 112.9).
template <int KIND, bool COUNT, bool TWO, class Src>
__device__ inline void persistent_trace(const SceneDev& S, Src& src, uint32_t count, unsigned long long* s_stack,
                                        lds_byte* top, uint32_t* s_next, uint32_t& nvis, uint32_t& ntri, bool& overflow) {
  const uint32_t per = (count + gridDim.x - 1) / gridDim.x;
  const uint32_t b0 = min(count, blockIdx.x * per), b1 = min(count, b0 + per);
  if (threadIdx.x == 0) *s_next = b0;
  __syncthreads();
  DevStack st = make_stack(s_stack);
  LaneRay L;
  bool busy = false, ended = false, drained = false;
  uint32_t item = 0;
  while (true) {
    const uint64_t idle = __ballot(!busy);
    const uint32_t n_idle = (uint32_t)__popcll((unsigned long long)idle);
    if ((!drained && n_idle >= kRefill) || n_idle == 64u) {
      if (ended) src.finish(item, L, L.found());
      ended = false;
      if (drained) break;
      uint32_t base = 0;
      if (lane_id() == 0) base = atomicAdd(s_next, n_idle);
      base = __shfl(base, 0);
      if (base + n_idle >= b1) drained = true;
      const uint32_t i = base + lane_prefix(idle);
      if (!busy && i < b1) {
        item = i;
        st.clear();
        src.start(i, L);
        busy = true;
      }
    }
    if (__ballot(busy) == 0) break;
    bool go = busy;
    if (kLeafWait) {
      // a lane at a leaf waits while there are many more lanes at inner
      // nodes, so that fewer iterations run both the node and the triangle
      // code
      const bool at_leaf = busy && L.cur != kEmpty && ref_is_leaf(L.cur);
      const uint32_t n_leaf = (uint32_t)__popcll((unsigned long long)__ballot(at_leaf));
      const uint32_t n_node = (uint32_t)__popcll((unsigned long long)__ballot(busy && !at_leaf));
      go = busy && (!at_leaf || kLeafWait * n_leaf >= kLeafWaitDen * n_node);
    }
    uint32_t ninst = 0;
    if (go && lane_step<KIND, COUNT, TWO, true>(S, L, src.tmin, st, top, nvis, ntri, ninst)) {
      busy = false;
      ended = true;
    }
  }
  overflow |= st.overflow;
}

template <bool TWO>
struct ExtendSrc {
  const SceneDev& S;
  const PathsDev& P;
  __device__ inline void start(uint32_t slot, LaneRay& L) {
    const float4 o = P.path[slot].o, d = P.path[slot].d;
    lane_start<TWO>(L, o.x, o.y, o.z, d.x, d.y, d.z, INFINITY, f2u(d.w), f2u(o.w), kTopBit);
  }
  __device__ inline void finish(uint32_t slot, const LaneRay& L, bool found) {
    int cls = kClsMiss;
    if (found) {
      P.path[slot].hit = make_float4(L.t, L.b1, L.b2, u2f(L.tri));
      uint32_t mid = f2u(S.tris[L.tri].b.w);
      if (TWO) {
        P.hit_inst[slot] = L.best_inst;
        int32_t ov = S.insts[L.best_inst].mat_override;
        if (ov >= 0) mid = (uint32_t)ov;
      }
      cls = S.mats[mid].cls;
    } else {
      P.path[slot].hit = make_float4(INFINITY, 0.0f, 0.0f, u2f(0xFFFFFFFFu));
    }
    P.cls[slot] = (uint8_t)cls;
  }
};

// Material binning of the rays just traced: a counting sort by class with
// one atomic per class per workgroup tile of kBinTile rays (atomics on one
// counter take 11.4 ns each however many workgroups issue them: with tiles of
// 1024 they were half of this kernel's 0.82 ms for 33M rays).
constexpr uint32_t kBinItems = 16, kBinTile = kBinItems * kBlock;
__global__ __launch_bounds__(kBlock) void k_bin(PathsDev P, int cur) {
  __shared__ uint32_t s_cnt[kNumClasses], s_base[kNumClasses];
  // the traversal launch before this one has traced the shadow queue: empty it for the shading
  if (blockIdx.x == 0 && threadIdx.x < kShards) P.counts[count_shadow(threadIdx.x)] = 0u;
  const QueueShare q = queue_share(P, cur);
  for (uint32_t blk = q.wg * kBinTile; blk < q.n; blk += q.G * kBinTile) {
    if (threadIdx.x < kNumClasses) s_cnt[threadIdx.x] = 0u;
    __syncthreads();
    uint32_t slot[kBinItems], pos[kBinItems];
    int cls[kBinItems];
#pragma unroll
    for (uint32_t k = 0; k < kBinItems; ++k) {
      const uint32_t i = blk + k * kBlock + threadIdx.x;
      cls[k] = -1;
      if (i < q.n) {
        slot[k] = q.slot(P, i);
        cls[k] = P.cls[slot[k]];
      }
    }
#pragma unroll
    for (uint32_t k = 0; k < kBinItems; ++k)
      if (cls[k] >= 0) pos[k] = atomicAdd(&s_cnt[cls[k]], 1u);  // LDS
    __syncthreads();
    if (threadIdx.x < kNumClasses) {
      uint32_t c = s_cnt[threadIdx.x];
      s_base[threadIdx.x] = c ? atomicAdd(&P.counts[count_class(threadIdx.x)], c) : 0u;
    }
    __syncthreads();
#pragma unroll
    for (uint32_t k = 0; k < kBinItems; ++k)
      if (cls[k] >= 0) P.q_cls[cls[k]][s_base[cls[k]] + pos[k]] = slot[k];
    __syncthreads();
  }
}

// ------------------------------------------------------------------- shade
struct ShadeOut {
  bool cont, shadow, query;  // next ray written / shadow ray below / path ended in the cache
  float4 sh_o, sh_d, sh_c;   // shadow ray: o, tmax; d, path slot; contribution, skip primitive
  uint32_t sh_inst;          // skip instance of the shadow ray
};

// Shade the hit (or miss) of path `slot` at vertex b: emission with MIS; at
// the last vertex stop; at the cache vertex write a query and stop;
// otherwise next-event estimation (a pre-weighted shadow ray), BSDF
// sampling, Russian roulette and the next ray.
template <int CLS, bool DEBUG, bool TWO>
__device__ inline void shade_one(const SceneDev& S, const PathsDev& P, uint32_t slot, int b, int max_depth,
                                 uint32_t sample, uint32_t k0, uint32_t k1, int nrc_bounce,
                                 ShadeOut& o, unsigned long long& nonfinite) {
  o.cont = o.shadow = o.query = false;
  PathRec& rec = P.path[slot];
  const float4 rd = rec.d, be = rec.beta;
  V3 beta = v3(be.x, be.y, be.z);
  float pdf_prev = be.w;
  bool prev_delta = !(pdf_prev > 0.0f);  // a sampled non-delta direction has a positive pdf
  // the path's radiance is touched only where something is added to it
  auto add_L = [&](V3 c) {
    const float4 l = P.L[slot];
    P.L[slot] = make_float4(l.x + c.x, l.y + c.y, l.z + c.z, 0.0f);
  };
  V3 d = v3(rd.x, rd.y, rd.z);
  uint64_t sig = DEBUG ? P.sig[slot] : 0ull;
  if (CLS == kClsMiss) {
    if (S.env_w > 0) {
      float st;
      int texel = env_texel(S, d, st);
      if (DEBUG) { sig = sig_word(sig, 2); sig = sig_word(sig, (uint32_t)texel); }
      float4 e = S.env[texel];
      float w = 1.0f;
      if (!prev_delta) w = pow_heuristic(pdf_prev, S.p_env * env_pdf_texel(S, texel, e, st));
      if (w > 0.0f) {
        V3 c = v3(beta.x * w * e.x, beta.y * w * e.y, beta.z * w * e.z);
        if (finite3(c)) add_L(c);
        else nonfinite++;
      }
    } else if (DEBUG) {
      sig = sig_word(sig, 2);
      sig = sig_word(sig, 0xFFFFFFFFu);
    }
    if (DEBUG) { sig = sig_word(sig, 6); sig = sig_word(sig, 0); }
    if (DEBUG) P.sig[slot] = sig;
  } else {
    const float4 hv = rec.hit;
    const TriRec tr = S.tris[f2u(hv.w)];
    uint32_t prim = f2u(tr.a.w), mid = f2u(tr.b.w);
    uint32_t inst = 0;
    V3 p0 = v3(tr.a.x, tr.a.y, tr.a.z), p1 = v3(tr.b.x, tr.b.y, tr.b.z), p2 = v3(tr.c.x, tr.c.y, tr.c.z);
    float b1 = hv.y, b2 = hv.z;
    V3 p = p0 * (1.0f - b1 - b2) + p1 * b1 + p2 * b2;
    V3 nc = cross(p1 - p0, p2 - p0);
    V3 axis = v3(S.axis[0], S.axis[1], S.axis[2]);
    int light_of_prim = -1;
    if (TWO) {
      inst = P.hit_inst[slot];
      const InstRec& I = S.insts[inst];
      if (I.mat_override >= 0) mid = (uint32_t)I.mat_override;
      const float* q = I.o2w;
      p = v3(q[0] * p.x + q[1] * p.y + q[2] * p.z + q[3], q[4] * p.x + q[5] * p.y + q[6] * p.z + q[7],
             q[8] * p.x + q[9] * p.y + q[10] * p.z + q[11]);
      nc = v3(q[0] * nc.x + q[1] * nc.y + q[2] * nc.z, q[4] * nc.x + q[5] * nc.y + q[6] * nc.z,
              q[8] * nc.x + q[9] * nc.y + q[10] * nc.z);
      axis = v3(q[2], q[6], q[10]);
      if (I.light_map >= 0) light_of_prim = S.light_map[I.light_map + (int)prim];
    } else {
      light_of_prim = S.tri_light[prim];
    }
    const MatRec& m = S.mats[mid];
    if (DEBUG) { sig = sig_word(sig, 1); sig = sig_word(sig, inst); sig = sig_word(sig, prim); }
    V3 ng = normalize(nc);
    V3 wo_w = d * -1.0f;
    float cos_ng = dot(ng, wo_w);
    // emission (front face only), MIS-weighted against light sampling
    if ((m.flags & kMatEmissive) && cos_ng > 0.0f) {
      float w = 1.0f;
      if (!prev_delta) {
        int k = light_of_prim;
        float pl = 0.0f;
        if (k >= 0 && S.n_lights > 0) {
          const LightTri& Lt = S.lights[k];
          pl = Lt.p1.w * hv.x * hv.x / (cos_ng * Lt.p0.w);
        }
        w = pow_heuristic(pdf_prev, pl);
      }
      if (w > 0.0f) {
        V3 c = v3(beta.x * w * m.Le[0], beta.y * w * m.Le[1], beta.z * w * m.Le[2]);
        if (finite3(c)) add_L(c);
        else nonfinite++;
      }
    }
    int lobe_ev = -1, rr_ev = 0, end_ev = 7;
    bool pending = false;
    uint32_t nee_id = 0xFFFFFFFFu, nee_out = 3u;
    bool nee_done = false;
    bool entering = cos_ng > 0.0f;
    V3 n = entering ? ng : ng * -1.0f;
    // adaptive termination (path spread): a0 = t^2 / (4 pi |cos|) at the primary vertex, then the
    // sum of sqrt(t^2 / (pdf |cos|)) over the non-delta bounces that led to each later vertex
    bool spread_end = false;
    if (P.spread_c > 0.0f && slot < (uint32_t)P.n_render && nrc_bounce >= 0 && b <= nrc_bounce) {
      const float t = hv.x, ac = fabsf(cos_ng);
      float2 sp = b == 0 ? make_float2(t * t / (4.0f * kPi * ac), 0.0f) : P.spread[slot];
      if (b >= 1) {
        if (!prev_delta) sp.y += sqrtf(t * t / (pdf_prev * ac));
        spread_end = sp.y * sp.y > P.spread_c * sp.x;
      }
      P.spread[slot] = sp;
    }
    if (b == max_depth) {
      end_ev = 1;
    } else if ((b == nrc_bounce || spread_end) && slot < (uint32_t)P.n_render) {
      // the path ends in the radiance cache: the query adds beta * cache(x) after the pass
      float* qr = P.nrc_q + (size_t)slot * kNrcQueryFloats;
      nrc_inputs(S.box_lo, S.box_inv, p, wo_w, n, m, qr);
      qr[12] = beta.x;
      qr[13] = beta.y;
      qr[14] = beta.z;
      o.query = true;
      end_ev = 4;
    } else if (b == P.train_end && slot >= (uint32_t)P.n_render) {
      // self-training: the training path ends in the cache; its terminal record (flag 2) is
      // answered by the cache before the targets of its earlier vertices are formed
      float* rr = P.rec + ((size_t)(slot - P.n_render) * P.rec_depth + b) * kNrcRecFloats;
      nrc_inputs(S.box_lo, S.box_inv, p, wo_w, n, m, rr);
      const float4 L = P.L[slot];
      rr[12] = L.x;
      rr[13] = L.y;
      rr[14] = L.z;
      rr[15] = beta.x;
      rr[16] = beta.y;
      rr[17] = beta.z;
      rr[18] = 2.0f;
      end_ev = 4;
    } else {
      if (P.rec && slot >= (uint32_t)P.n_render) {  // training record: inputs, radiance so far, throughput
        float* rr = P.rec + ((size_t)(slot - P.n_render) * P.rec_depth + b) * kNrcRecFloats;
        nrc_inputs(S.box_lo, S.box_inv, p, wo_w, n, m, rr);
        const float4 L = P.L[slot];
        rr[12] = L.x;
        rr[13] = L.y;
        rr[14] = L.z;
        rr[15] = beta.x;
        rr[16] = beta.y;
        rr[17] = beta.z;
        rr[18] = 1.0f;
      }
      V3 t, bt;
      make_frame(n, axis, t, bt);
      V3 wo = v3(dot(wo_w, t), dot(wo_w, bt), dot(wo_w, n));
      Bsdf B = bsdf_setup<CLS>(m, entering, wo.z);
      if (wo.z <= 0.0f) B.absorbed = true;
      uint32_t px, py;
      const Rng rng = slot_rng(P, slot, sample, k0, k1, px, py);
      U4 r0 = rng.block((uint32_t)b, 0u), r1 = rng.block((uint32_t)b, 1u);
      // next-event estimation
      if (!B.absorbed && bsdf_has_nondelta<CLS>(m, B)) {
        nee_done = true;
        U4 r2 = rng.block((uint32_t)b, 2u);
        LightSample ls = sample_light(S, p, u01(r1.w), u01(r2.x), u01(r2.y));
        nee_id = ls.id;
        if (ls.ok) {
          V3 wil = v3(dot(ls.wl, t), dot(ls.wl, bt), dot(ls.wl, n));
          float pb;
          V3 f = bsdf_eval<CLS>(m, B, wo, wil, pb);
          float w = pow_heuristic(ls.pdf, pb);
          float k = fabsf(wil.z) * w / ls.pdf;
          V3 c = v3(beta.x * f.x * ls.Le.x * k, beta.y * f.y * ls.Le.y * k, beta.z * f.z * ls.Le.z * k);
          if (c.x != 0.0f || c.y != 0.0f || c.z != 0.0f) {
            o.shadow = true;
            pending = true;
            float tmax = isinf(ls.dist) ? INFINITY : (1.0f - 1e-4f) * ls.dist;
            o.sh_o = make_float4(p.x, p.y, p.z, tmax);
            o.sh_d = make_float4(ls.wl.x, ls.wl.y, ls.wl.z, u2f(slot));
            o.sh_c = make_float4(c.x, c.y, c.z, u2f(prim));
            o.sh_inst = inst;
          } else {
            nee_out = 2u;
          }
        }
      }
      // BSDF sampling
      BsdfSample bs = bsdf_sample<CLS>(m, B, wo, u01(r0.z), u01(r1.x), u01(r1.y), u01(r1.z));
      lobe_ev = bs.lobe;
      if (!bs.ok || (bs.weight.x == 0.0f && bs.weight.y == 0.0f && bs.weight.z == 0.0f)) {
        end_ev = 2;
      } else {
        beta = v3(beta.x * bs.weight.x, beta.y * bs.weight.y, beta.z * bs.weight.z);
        pdf_prev = bs.pdf;  // 0 for a delta lobe
        float eta_scale = P.eta ? P.eta[slot] : 1.0f;
        if (bs.refract) {
          eta_scale *= B.eta * B.eta;
          P.eta[slot] = eta_scale;
        }
        bool killed = false;
        if (b >= 1) {
          float q = fmaxf(fmaxf(beta.x, beta.y), beta.z) * eta_scale;
          if (q < 0.995f) {  // no roulette within rounding of q = 1
            killed = u01(r0.w) >= q;
            rr_ev = killed ? 2 : 1;
            if (!killed) beta = beta * (1.0f / q);
          }
        }
        if (killed) {
          end_ev = 3;
        } else {
          V3 dn = normalize(t * bs.wi.x + bt * bs.wi.y + n * bs.wi.z);
          rec.o = make_float4(p.x, p.y, p.z, u2f(prim));
          rec.d = make_float4(dn.x, dn.y, dn.z, u2f(inst));
          rec.beta = make_float4(beta.x, beta.y, beta.z, pdf_prev);
          o.cont = true;
        }
      }
    }
    if (DEBUG) {
      uint32_t tail = tail_pack(lobe_ev, rr_ev, end_ev);
      if (pending) {
        P.dbg_nee[slot] = nee_id;
        P.dbg_tail[slot] = tail;
      } else {
        if (nee_done) {
          sig = sig_word(sig, 5);
          sig = sig_word(sig, nee_id);
          sig = sig_word(sig, nee_out);
        }
        sig = sig_tail(sig, tail);
      }
      P.sig[slot] = sig;
    }
  }
}

template <bool DEBUG, bool TWO>
__device__ inline void shade_any(int cls, const SceneDev& S, const PathsDev& P, uint32_t slot, int b, int max_depth,
                                 uint32_t sample, uint32_t k0, uint32_t k1, int nrc_bounce,
                                 ShadeOut& o, unsigned long long& nf) {
  const int q = nrc_bounce;
  switch (cls) {
    case kClsMiss: shade_one<kClsMiss, DEBUG, TWO>(S, P, slot, b, max_depth, sample, k0, k1, q, o, nf); break;
    case kClsAbsorb: shade_one<kClsAbsorb, DEBUG, TWO>(S, P, slot, b, max_depth, sample, k0, k1, q, o, nf); break;
    case kClsDiffuse: shade_one<kClsDiffuse, DEBUG, TWO>(S, P, slot, b, max_depth, sample, k0, k1, q, o, nf); break;
    case kClsMetal: shade_one<kClsMetal, DEBUG, TWO>(S, P, slot, b, max_depth, sample, k0, k1, q, o, nf); break;
    case kClsPlastic: shade_one<kClsPlastic, DEBUG, TWO>(S, P, slot, b, max_depth, sample, k0, k1, q, o, nf); break;
    case kClsGlass: shade_one<kClsGlass, DEBUG, TWO>(S, P, slot, b, max_depth, sample, k0, k1, q, o, nf); break;
    default: shade_one<kClsGeneral, DEBUG, TWO>(S, P, slot, b, max_depth, sample, k0, k1, q, o, nf); break;
  }
}

using ShadeAppend = uint32_t[3][kShadeBlock / 64 + 1];
// One workgroup's block of a class queue (items [base, base + kShadeBlock) of `count`): shades its
// paths and appends what they go on with.  s_app: per queue (next rays, shadow rays, cache queries)
// the wave counts, then the workgroup's base.
template <bool TWO, class Shade>
__device__ inline void shade_tile(const PathsDev& P, const uint32_t* q_cls, uint32_t count, uint32_t base, int next,
                                  ShadeAppend& s_app, Shade shade) {
  uint32_t i = base + threadIdx.x;
  bool active = i < count;
  uint32_t slot = 0;
  ShadeOut o;
  o.cont = o.shadow = o.query = false;
  if (active) {
    slot = q_cls[i];
    shade(slot, o);
  }
  // one atomic per queue per workgroup iteration
  const uint32_t shard = base / kShadeBlock % kShards;
  const size_t seg = (size_t)shard * P.seg_cap;
  const uint64_t m_cont = __ballot(o.cont), m_sh = __ballot(o.shadow), m_q = __ballot(o.query);
  const int w = (int)(threadIdx.x >> 6);
  if (lane_id() == 0) {
    s_app[0][w] = (uint32_t)__popcll(m_cont);
    s_app[1][w] = (uint32_t)__popcll(m_sh);
    s_app[2][w] = (uint32_t)__popcll(m_q);
  }
  __syncthreads();
  if (threadIdx.x < 3) {
    uint32_t tot = 0;
    for (int k = 0; k < kShadeBlock / 64; ++k) tot += s_app[threadIdx.x][k];
    uint32_t* ctr = threadIdx.x == 0   ? &P.counts[count_ray(shard, next)]
                    : threadIdx.x == 1 ? &P.counts[count_shadow(shard)]
                                       : &P.counts[kCountQuery];
    s_app[threadIdx.x][kShadeBlock / 64] = tot ? atomicAdd(ctr, tot) : 0u;
  }
  __syncthreads();
  uint32_t off[3];
  for (int q = 0; q < 3; ++q) {
    uint32_t acc = s_app[q][kShadeBlock / 64];
    for (int k = 0; k < w; ++k) acc += s_app[q][k];
    off[q] = acc;
  }
  __syncthreads();  // s_app is rewritten by the next iteration
  if (o.cont) P.q_ray[next][seg + off[0] + lane_prefix(m_cont)] = slot;
  if (o.query) P.q_nrc[off[2] + lane_prefix(m_q)] = slot;
  if (o.shadow) {
    const size_t spos = seg + off[1] + lane_prefix(m_sh);
    P.sh_o[spos] = o.sh_o;
    P.sh_d[spos] = o.sh_d;
    P.sh_c[spos] = o.sh_c;
    if (TWO) P.sh_inst[spos] = o.sh_inst;
  }
}

// Waves per SIMD that the shading kernel of a class is compiled for: 4 (128
// registers), 3 for the general class, which needs 153.  Material zoo 1024x768, 40
// spp, its launches at 4 / 3: 5.99 / 5.94 ms a render (6.52 / 5.99 while it needed 165
// and kept 144 bytes a lane in scratch at 4); coated 1.44 / 1.57, glass 0.58 / 0.64;
// instanced scene, glass 3.53 / 3.97.  Icosphere field render at 3 / 4 / 5 / 6: 89.1 /
// 88.4 / 94.5 / 99.5 ms.
constexpr int shade_waves(int cls) { return cls == kClsGeneral ? 3 : 4; }
template <int CLS, bool DEBUG, bool TWO>
__global__ __launch_bounds__(kShadeBlock, shade_waves(CLS)) void k_shade(SceneDev S, PathsDev P, int b, int max_depth, int next,
                                                  uint32_t sample, uint32_t k0, uint32_t k1,
                                                  int nrc_bounce) {
  __shared__ ShadeAppend s_app;
  const uint32_t count = P.counts[count_class(CLS)];
  unsigned long long nonfinite = 0;
  for (uint32_t base = blockIdx.x * kShadeBlock; base < count; base += gridDim.x * kShadeBlock)
    shade_tile<TWO>(P, P.q_cls[CLS], count, base, next, s_app, [&](uint32_t slot, ShadeOut& o) {
      shade_one<CLS, DEBUG, TWO>(S, P, slot, b, max_depth, sample, k0, k1, nrc_bounce, o, nonfinite);
    });
  if (nonfinite) atomicAdd(&P.stats[kStatNonFinite], nonfinite);
}

// All classes in one launch, for passes of few slots, whose launches last as long as one path's
// chain of dependent loads: a workgroup takes blocks of the class queues one after the other, each
// of one class, so that no wave runs the code of two (shade_all says up to which size, with figures).
template <bool DEBUG, bool TWO>
__global__ __launch_bounds__(kShadeBlock) void k_shade_classes(SceneDev S, PathsDev P, int b, int max_depth, int next,
                                                               uint32_t sample, uint32_t k0, uint32_t k1,
                                                               int nrc_bounce) {
  __shared__ ShadeAppend s_app;
  unsigned long long nonfinite = 0;
  uint32_t first = 0;  // blocks of the classes before
  for (int cls = 0; cls < kNumClasses; ++cls) {
    const uint32_t count = P.counts[count_class(cls)], blocks = (count + kShadeBlock - 1) / kShadeBlock;
    // this workgroup's first block of the class: those it takes are blockIdx.x, + gridDim.x, ... of all classes'
    uint32_t k = (blockIdx.x + gridDim.x - first % gridDim.x) % gridDim.x;
    for (; k < blocks; k += gridDim.x)
      shade_tile<TWO>(P, P.q_cls[cls], count, k * kShadeBlock, next, s_app, [&](uint32_t slot, ShadeOut& o) {
        shade_any<DEBUG, TWO>(cls, S, P, slot, b, max_depth, sample, k0, k1, nrc_bounce, o, nonfinite);
      });
    first += blocks;
  }
  if (nonfinite) atomicAdd(&P.stats[kStatNonFinite], nonfinite);
}

// ----------------------------------------------------------------- connect
template <bool DEBUG, bool TWO>
struct ConnectSrc {
  const SceneDev& S;
  const PathsDev& P;
  unsigned long long& nonfinite;
  __device__ inline void start(uint32_t i, LaneRay& L) {
    float4 o = P.sh_o[i], d = P.sh_d[i];
    uint32_t skip_prim = f2u(P.sh_c[i].w);
    if (TWO) lane_start<true>(L, o.x, o.y, o.z, d.x, d.y, d.z, o.w, P.sh_inst[i], skip_prim, kTopBit);
    else lane_start<false>(L, o.x, o.y, o.z, d.x, d.y, d.z, o.w, 0u, skip_prim, kTopBit);
  }
  __device__ inline void finish(uint32_t i, const LaneRay& L, bool occ) {
    uint32_t slot = f2u(P.sh_d[i].w);
    if (!occ) {
      float4 c = P.sh_c[i];
      V3 cc = v3(c.x, c.y, c.z);
      if (finite3(cc)) {
        float4 Lr = P.L[slot];
        P.L[slot] = make_float4(Lr.x + cc.x, Lr.y + cc.y, Lr.z + cc.z, Lr.w);
      } else {
        nonfinite++;
      }
    }
    if (DEBUG) {
      uint64_t sig = P.sig[slot];
      sig = sig_word(sig, 5);
      sig = sig_word(sig, P.dbg_nee[slot]);
      sig = sig_word(sig, occ ? 1u : 0u);
      sig = sig_tail(sig, P.dbg_tail[slot]);
      P.sig[slot] = sig;
    }
  }
};

// One traversal launch per bounce: the closest hits of the bounce's rays
// (queue `cur`, none if cur < 0) and the shadow rays of the previous bounce's
// shading.  A lane's walk kind is a per-lane flag, so lanes of both kinds can
// share a wave without running the walk code twice: the node step is the same
// and the leaf step differs only in stopping at the first accepted triangle.
// Each workgroup owns a share of both queues and takes its closest-hit rays
// first; its shadow rays fill the lanes that the last closest-hit walks leave
// idle, instead of every workgroup of the GPU draining at a kernel boundary.
template <bool DEBUG, bool COUNT, bool TWO>
__global__ __launch_bounds__(kBlock, TWO ? kTraceWaves2 : kTraceWaves) void k_traverse(SceneDev S, PathsDev P, int cur) {
  __shared__ unsigned long long s_stack[kLdsStack * kBlock];
  __shared__ __align__(16) unsigned char s_top[kTopLds];
  __shared__ uint32_t s_next;
  lds_byte* top = top_load(S, s_top);
  // closest-hit rays (queue `cur`; none if < 0) and shadow rays of this workgroup's segments
  QueueShare qe = queue_share(P, max(cur, 0));
  if (cur < 0) qe.n = 0u;
  const uint32_t seg = blockIdx.x % kShards, wg_s = blockIdx.x / kShards, G_s = gridDim.x / kShards;
  const uint32_t ns = P.counts[count_shadow(seg)], sh_first = seg * P.seg_cap;
  if (threadIdx.x == 0) {  // each count once
    if (qe.n && qe.wg == 0) atomicAdd(&P.stats[kStatExt], (unsigned long long)qe.n);
    if (ns && wg_s == 0) atomicAdd(&P.stats[kStatShadow], (unsigned long long)ns);
  }
  const uint32_t n_e = share_size(qe.n, qe.wg, qe.G), n_all = n_e + share_size(ns, wg_s, G_s);
  if (threadIdx.x == 0) s_next = 0u;
  __syncthreads();
  DevStack st = make_stack(s_stack);
  unsigned long long nonfinite = 0;
  ExtendSrc<TWO> es{S, P};
  ConnectSrc<DEBUG, TWO> cs{S, P, nonfinite};
  LaneRay L;
  L.any = false;
  bool busy = false, ended = false, drained = false, shadow = false;
  uint32_t item = 0;
  uint32_t rv = 0, rt = 0, nvis = 0, ntri = 0, svis = 0, stri = 0;  // node visits / triangle tests
  uint32_t ri = 0, ninst = 0;  // instances entered (both walk kinds)
  while (true) {
    const uint64_t idle = __ballot(!busy);
    const uint32_t n_idle = (uint32_t)__popcll((unsigned long long)idle);
    if ((!drained && n_idle >= kRefill) || n_idle == 64u) {
      if (ended) {  // the lanes whose walks have ended since the last refill
        const bool found = L.found();
        if (shadow) cs.finish(item, L, found);
        else es.finish(item, L, found);
        if (COUNT) {
          ninst += ri;
          if (shadow) {
            svis += rv;
            stri += rt;
          } else {
            nvis += rv;
            ntri += rt;
          }
        }
        ended = false;
      }
      if (drained) break;
      uint32_t base = 0;
      if (lane_id() == 0) base = atomicAdd(&s_next, n_idle);
      base = __shfl(base, 0);
      if (base + n_idle >= n_all) drained = true;
      const uint32_t v = base + lane_prefix(idle);
      if (!busy && v < n_all) {
        shadow = v >= n_e;
        item = shadow ? sh_first + share_item(v - n_e, ns, wg_s, G_s) : qe.slot(P, share_item(v, qe.n, qe.wg, qe.G));
        st.clear();
        if (shadow) cs.start(item, L);
        else es.start(item, L);
        L.any = shadow;
        busy = true;
        rv = rt = ri = 0;
      }
    }
    if (__ballot(busy) == 0) break;
    bool go = busy;
    if (kLeafWait) {
      // a lane at a leaf waits while there are many more lanes at inner
      // nodes, so that fewer iterations run both the node and the triangle
      // code
      const bool at_leaf = busy && L.cur != kEmpty && ref_is_leaf(L.cur);
      const uint32_t n_leaf = (uint32_t)__popcll((unsigned long long)__ballot(at_leaf));
      const uint32_t n_node = (uint32_t)__popcll((unsigned long long)__ballot(busy && !at_leaf));
      go = busy && (!at_leaf || kLeafWait * n_leaf >= kLeafWaitDen * n_node);
    }
    if (go && lane_step<kWalkPerLane, COUNT, TWO, true>(S, L, S.tmin, st, top, rv, rt, ri)) {
      busy = false;
      ended = true;
    }
  }
  if (COUNT) {
    atomicAdd(&P.stats[kStatNodes], (unsigned long long)nvis);
    atomicAdd(&P.stats[kStatTris], (unsigned long long)ntri);
    atomicAdd(&P.stats[kStatShadowNodes], (unsigned long long)svis);
    atomicAdd(&P.stats[kStatShadowTris], (unsigned long long)stri);
    if (TWO) atomicAdd(&P.stats[kStatInstances], (unsigned long long)ninst);
  }
  if (nonfinite) atomicAdd(&P.stats[kStatNonFinite], nonfinite);
  if (st.overflow) atomicAdd(&P.stats[kStatOverflow], 1ull);
}

// -------------------------------------------------------------------- tail
// Once few paths remain, one persistent-lane kernel finishes them: a lane
// takes a path and runs all its remaining vertices (closest hit, shading,
// shadow ray, next ray) with no kernel boundary between vertices, so short
// paths do not wait for the slowest ray of every later bounce.  Shading,
// walks and signatures are the same code as the wavefront kernels'.
template <bool DEBUG, bool COUNT, bool TWO>
__global__ __launch_bounds__(kBlock) void k_tail(SceneDev S, PathsDev P, int cur, int b_first, int max_depth,
                                                 uint32_t sample, uint32_t k0, uint32_t k1,
                                                 int nrc_bounce) {
  __shared__ unsigned long long s_stack[kLdsStack * kBlock];
  __shared__ uint32_t s_count;
  // Every wave takes paths from one device-wide counter (zeroed before the
  // launch), so the longest paths do not pile up in one workgroup's share.
  __shared__ uint32_t s_first[kShards];  // segments of the queue: the path number each starts at
  if (threadIdx.x == 0) {
    uint32_t n = 0;
    for (uint32_t g = 0; g < kShards; ++g) {
      s_first[g] = n;
      n += cur == kQueueAll ? 0u : P.counts[count_ray(g, cur)];
    }
    s_count = cur == kQueueAll ? (uint32_t)P.n : n;
  }
  __syncthreads();
  const uint32_t q1 = s_count;
  uint32_t* next_path = &P.counts[kCountTail];
  DevStack st = make_stack(s_stack);
  LaneRay L;
  // 0 idle, 1 closest-hit walk, 2 shadow-ray walk, 3 hit found and waiting to be shaded
  int phase = 0;
  bool drained = false, cont = false;
  uint32_t slot = 0;
  int b = b_first, cls = kClsMiss;
  float4 sh_c = make_float4(0, 0, 0, 0);
  uint32_t n_ext = 0, n_sh = 0, nvis = 0, ntri = 0, svis = 0, stri = 0;
  unsigned long long nonfinite = 0;
  bool overflow = false;
  uint32_t rv = 0, rt = 0, ri = 0;  // node visits / triangle tests / instances entered of the current walk
  uint32_t ninst = 0;
  auto start_closest = [&](void) {
    const float4 o = P.path[slot].o, d = P.path[slot].d;
    st.clear();
    lane_start<TWO>(L, o.x, o.y, o.z, d.x, d.y, d.z, INFINITY, f2u(d.w), f2u(o.w), S.root);
    L.any = false;
    rv = rt = ri = 0;
    phase = 1;
    n_ext++;
  };
  while (true) {
    const uint64_t idle = __ballot(phase == 0);
    const uint32_t n_idle = (uint32_t)__popcll((unsigned long long)idle);
    if (!drained && (n_idle >= kRefill || n_idle == 64u)) {
      uint32_t base = 0;
      if (lane_id() == 0) base = atomicAdd(next_path, n_idle);
      base = __shfl(base, 0);
      if (base + n_idle >= q1) drained = true;
      const uint32_t i = base + lane_prefix(idle);
      if (phase == 0 && i < q1) {
        if (cur == kQueueAll) {
          slot = i;
        } else {
          uint32_t g = kShards - 1;
          while (g > 0 && s_first[g] > i) --g;
          slot = P.q_ray[cur][(size_t)g * P.seg_cap + (i - s_first[g])];
        }
        b = b_first;
        start_closest();
      }
    }
    if (__ballot(phase != 0) == 0) break;
    // closest-hit and shadow walks share one walk step (kind per lane); a
    // lane at a leaf waits while lanes at inner nodes outnumber it
    const bool walking = phase == 1 || phase == 2;
    bool go = walking;
    if (kLeafWait) {
      const bool at_leaf = walking && L.cur != kEmpty && ref_is_leaf(L.cur);
      const uint32_t n_leaf = (uint32_t)__popcll((unsigned long long)__ballot(at_leaf));
      const uint32_t n_node = (uint32_t)__popcll((unsigned long long)__ballot(walking && !at_leaf));
      go = walking && (!at_leaf || kLeafWait * n_leaf >= kLeafWaitDen * n_node);
    }
    const bool done = go && lane_step<kWalkPerLane, COUNT, TWO, false>(S, L, S.tmin, st, nullptr, rv, rt, ri);
    if (done && COUNT) {
      ninst += ri;
      if (phase == 1) {
        nvis += rv;
        ntri += rt;
      } else {
        svis += rv;
        stri += rt;
      }
    }
    if (phase == 1) {
      if (done) {
        overflow |= st.overflow;
        cls = kClsMiss;
        if (L.found()) {
          P.path[slot].hit = make_float4(L.t, L.b1, L.b2, u2f(L.tri));
          uint32_t mid = f2u(S.tris[L.tri].b.w);
          if (TWO) {
            P.hit_inst[slot] = L.best_inst;
            int32_t ov = S.insts[L.best_inst].mat_override;
            if (ov >= 0) mid = (uint32_t)ov;
          }
          cls = S.mats[mid].cls;
        } else {
          P.path[slot].hit = make_float4(INFINITY, 0.0f, 0.0f, u2f(0xFFFFFFFFu));
        }
        phase = 3;
      }
    } else if (phase == 2) {
      if (done) {
        overflow |= st.overflow;
        const bool occ = L.found();
        if (!occ) {
          V3 cc = v3(sh_c.x, sh_c.y, sh_c.z);
          if (finite3(cc)) {
            float4 Lr = P.L[slot];
            P.L[slot] = make_float4(Lr.x + cc.x, Lr.y + cc.y, Lr.z + cc.z, Lr.w);
          } else {
            nonfinite++;
          }
        }
        if (DEBUG) {
          uint64_t sig = P.sig[slot];
          sig = sig_word(sig, 5);
          sig = sig_word(sig, P.dbg_nee[slot]);
          sig = sig_word(sig, occ ? 1u : 0u);
          sig = sig_tail(sig, P.dbg_tail[slot]);
          P.sig[slot] = sig;
        }
        if (cont) {
          b++;
          start_closest();
        } else {
          phase = 0;
        }
      }
    }
    // Shading is a long stretch of code per material class.  Lanes that found
    // their hit wait until they are at least as many as the lanes still
    // walking (or until no lane walks), so that one pass over the shading code
    // serves many lanes instead of one pass per walk that ends.
    const uint32_t n_ready = (uint32_t)__popcll((unsigned long long)__ballot(phase == 3));
    const uint32_t n_walk = (uint32_t)__popcll((unsigned long long)__ballot(phase == 1 || phase == 2));
    if (n_ready && kTailShadeWait * n_ready >= n_walk && phase == 3) {
      ShadeOut o;
      shade_any<DEBUG, TWO>(cls, S, P, slot, b, max_depth, sample, k0, k1, nrc_bounce, o, nonfinite);
      // paths that ended in the radiance cache join its query queue (one atomic per wave)
      const uint64_t m_q = __ballot(o.query);
      if (m_q) {
        const int leader = __ffsll((long long)m_q) - 1;
        uint32_t qbase = 0;
        if ((int)lane_id() == leader) qbase = atomicAdd(&P.counts[kCountQuery], (uint32_t)__popcll(m_q));
        qbase = __shfl(qbase, leader);
        if (o.query) P.q_nrc[qbase + lane_prefix(m_q)] = slot;
      }
      if (o.shadow) {
        st.clear();
        lane_start<TWO>(L, o.sh_o.x, o.sh_o.y, o.sh_o.z, o.sh_d.x, o.sh_d.y, o.sh_d.z, o.sh_o.w,
                        TWO ? o.sh_inst : 0u, f2u(o.sh_c.w), S.root);
        L.any = true;
        rv = rt = ri = 0;
        sh_c = o.sh_c;
        cont = o.cont;
        phase = 2;
        n_sh++;
      } else if (o.cont) {
        b++;
        start_closest();
      } else {
        phase = 0;
      }
    }
  }
  // statistics: one atomic per wave and counter
  n_ext = wave_sum(n_ext);
  n_sh = wave_sum(n_sh);
  if (lane_id() == 0) {
    atomicAdd(&P.stats[kStatExt], (unsigned long long)n_ext);
    atomicAdd(&P.stats[kStatTailExt], (unsigned long long)n_ext);
    atomicAdd(&P.stats[kStatShadow], (unsigned long long)n_sh);
    atomicAdd(&P.stats[kStatTailShadow], (unsigned long long)n_sh);
  }
  if (COUNT) {
    atomicAdd(&P.stats[kStatTailNodes], (unsigned long long)nvis);
    atomicAdd(&P.stats[kStatTailTris], (unsigned long long)ntri);
    atomicAdd(&P.stats[kStatTailShadowNodes], (unsigned long long)svis);
    atomicAdd(&P.stats[kStatTailShadowTris], (unsigned long long)stri);
    if (TWO) atomicAdd(&P.stats[kStatTailInstances], (unsigned long long)ninst);
  }
  if (nonfinite) atomicAdd(&P.stats[kStatNonFinite], nonfinite);
  if (overflow) atomicAdd(&P.stats[kStatOverflow], 1ull);
}

// -------------------------------------------------------------- accumulate
// FP64 per-pixel running sums: one writer per pixel per pass, no atomics; the
// pass's samples are added one by one in sample order, so the sums do not
// depend on how many samples a pass takes.
// A workgroup stages its pixels' radiance through LDS, kAccumTile slots at a
// time, so that every lane reads neighbouring slots (a pixel per lane, 256 bytes
// apart at 16 samples: 3.1 GB fetched for 0.53, 450 us for 33M slots).
constexpr uint32_t kAccumTile = 2048;
__global__ __launch_bounds__(kBlock) void k_accumulate(PathsDev P, double* sum, int W, float* per_sample,
                                                       uint64_t* sig_out, int spp_total, int first_index) {
  __shared__ float4 s_L[kAccumTile + kAccumTile / 8];  // one more entry after every eight: spread over the banks
  const uint32_t places = (uint32_t)P.w * (uint32_t)P.h;
  const uint32_t part = min(P.spp, kAccumTile);                  // samples of a pixel per tile
  const uint32_t tile = min((uint32_t)kBlock, kAccumTile / part);  // pixels per tile
  for (uint32_t p0 = blockIdx.x * tile; p0 < places; p0 += gridDim.x * tile) {
    const uint32_t np = min(tile, places - p0), p = p0 + threadIdx.x;
    const bool mine = threadIdx.x < np;
    uint32_t x = 0, y = 0;
    double* s = nullptr;
    double sx = 0.0, sy = 0.0, sz = 0.0;
    if (mine) {
      place_pixel(p, (uint32_t)P.w, (uint32_t)P.h, x, y);
      if (sum) {
        s = sum + 3 * ((size_t)(P.y0 + y) * W + (P.x0 + x));
        sx = s[0];
        sy = s[1];
        sz = s[2];
      }
    }
    for (uint32_t k0 = 0; k0 < P.spp; k0 += part) {  // more than one round only for spp > kAccumTile (one pixel a tile)
      const uint32_t nk = min(part, P.spp - k0);
      __syncthreads();
      for (uint32_t i = threadIdx.x; i < np * nk; i += kBlock) s_L[i + i / 8u] = P.L[(size_t)p0 * P.spp + k0 + i];
      __syncthreads();
      if (!mine) continue;
      for (uint32_t k = 0; k < nk; ++k) {
        const uint32_t i = threadIdx.x * nk + k;
        const float4 v = s_L[i + i / 8u];
        if (sum) {
          sx += (double)v.x;
          sy += (double)v.y;
          sz += (double)v.z;
        }
        if (per_sample) {
          const size_t o = ((size_t)y * P.w + x) * spp_total + first_index + k0 + k;
          per_sample[3 * o] = v.x;
          per_sample[3 * o + 1] = v.y;
          per_sample[3 * o + 2] = v.z;
          sig_out[o] = P.sig[(size_t)p * P.spp + k0 + k];
        }
      }
    }
    if (s) {
      s[0] = sx;
      s[1] = sy;
      s[2] = sz;
    }
  }
}

__global__ __launch_bounds__(kBlock) void k_resolve(const double* sum, float* out, int64_t n, double inv) {
  for (int64_t i = blockIdx.x * (int64_t)kBlock + threadIdx.x; i < n; i += (int64_t)gridDim.x * kBlock)
    out[i] = (float)(sum[i] * inv);
}

__global__ __launch_bounds__(kBlock) void k_zero_f64(double* p, int64_t n) {
  for (int64_t i = blockIdx.x * (int64_t)kBlock + threadIdx.x; i < n; i += (int64_t)gridDim.x * kBlock) p[i] = 0.0;
}

__global__ __launch_bounds__(kBlock) void k_zero_u64(unsigned long long* p, int64_t n) {
  for (int64_t i = blockIdx.x * (int64_t)kBlock + threadIdx.x; i < n; i += (int64_t)gridDim.x * kBlock) p[i] = 0ull;
}

// ------------------------------------------------------- ray query kernels
// The first kTopNodes nodes of the tree in breadth-first order from `root`, with
// references to each other replaced by kTopBit | place.  One wave; lanes expand
// the places found so far, kTopNodes at most, until no place is left to expand.
__global__ __launch_bounds__(64) void k_top_nodes(const BVHNode* nodes, uint32_t root, BVHNode* top) {
  __shared__ uint32_t s_node[kTopNodes];
  const uint32_t lane = threadIdx.x;
  if (lane == 0) s_node[0] = root;
  __syncthreads();
  uint32_t n = 1;
  for (uint32_t done = 0; done < n;) {  // places [done, n) are expanded together, at most 64 of them
    const uint32_t batch = min(64u, n - done);
    BVHNode v;
    uint32_t inner = 0;
    if (lane < batch) {
      v = nodes[s_node[done + lane]];
      for (int c = 0; c < 4; ++c) inner += (int)v.child[c] >= 0 ? 1u : 0u;
    }
    uint32_t before = inner;  // inclusive prefix over the lanes
    for (int d = 1; d < 64; d <<= 1) {
      const uint32_t o = (uint32_t)__shfl_up((int)before, d);
      if ((int)lane >= d) before += o;
    }
    const uint32_t total = (uint32_t)__shfl((int)before, 63);
    uint32_t place = n + before - inner;
    if (lane < batch) {
      for (int c = 0; c < 4; ++c) {
        if ((int)v.child[c] < 0) continue;  // a leaf or empty
        if (place < kTopNodes) {
          s_node[place] = v.child[c];
          v.child[c] = kTopBit | place;
        }
        ++place;
      }
      top[done + lane] = v;
    }
    __syncthreads();
    done += batch;
    n = min(n + total, kTopNodes);
  }
}

hipError_t launch_top_nodes(const BVHNode* nodes, uint32_t root, BVHNode* top, hipStream_t st) {
  hipLaunchKernelGGL(k_top_nodes, dim3(1), dim3(64), 0, st, nodes, root, top);
  return hipGetLastError();
}

// Closest hits of a ray array ([n][8]: o, tmin, d, tmax) -> [n][6] words.
__device__ inline void write_hit(uint32_t* H, const Hit& h) {
  bool hit = h.tri != 0xFFFFFFFFu;
  H[0] = f2u(h.t);
  H[1] = hit ? h.inst : 0xFFFFFFFFu;
  H[2] = hit ? h.prim : 0xFFFFFFFFu;
  H[3] = hit ? f2u(h.b1) : 0u;
  H[4] = hit ? f2u(h.b2) : 0u;
  H[5] = hit ? 1u : 0u;
}

template <bool TWO>
struct RaysSrc {
  const SceneDev& S;
  const float* rays;
  uint32_t* hits;
  float tmin;  // of the lane's ray
  __device__ inline void start(uint32_t i, LaneRay& L) {
    const float* R = rays + 8 * (size_t)i;
    tmin = R[3];
    lane_start<TWO>(L, R[0], R[1], R[2], R[4], R[5], R[6], R[7], 0xFFFFFFFFu, 0xFFFFFFFFu, kTopBit);
  }
  __device__ inline void finish(uint32_t i, const LaneRay& L, bool found) {
    Hit h;
    hit_clear(h);
    if (found) {
      h.t = L.t;
      h.b1 = L.b1;
      h.b2 = L.b2;
      h.inst = TWO ? L.best_inst : 0u;
      h.tri = L.tri;
      h.prim = f2u(S.tris[L.tri].a.w);
    }
    write_hit(hits + 6 * (size_t)i, h);
  }
};

template <bool TWO>
__global__ __launch_bounds__(kBlock) void k_trace_rays(SceneDev S, const float* rays, uint32_t n, uint32_t* hits,
                                                       unsigned long long* stats) {
  __shared__ unsigned long long s_stack[kLdsStack * kBlock];
  __shared__ __align__(16) unsigned char s_top[kTopLds];
  __shared__ uint32_t s_next;
  uint32_t nvis = 0, ntri = 0;
  bool overflow = false;
  RaysSrc<TWO> src{S, rays, hits, 0.0f};
  persistent_trace<kWalkClosest, false, TWO>(S, src, n, s_stack, top_load(S, s_top), &s_next, nvis, ntri, overflow);
  if (overflow) atomicAdd(&stats[kStatOverflow], 1ull);
}

// The same definition by testing every triangle (and every instance).
template <bool TWO>
__global__ __launch_bounds__(kBlock) void k_trace_rays_brute(SceneDev S, const float* rays, uint32_t n,
                                                             uint32_t* hits) {
  for (uint32_t i = blockIdx.x * kBlock + threadIdx.x; i < n; i += gridDim.x * kBlock) {
    const float* R = rays + 8 * (size_t)i;
    Hit h;
    hit_clear(h);
    uint32_t nt = 0;
    RayPre r = ray_prepare(R[0], R[1], R[2], R[4], R[5], R[6]);
    if (TWO) brute_force_two_level(S.insts, S.n_insts, S.tris, S.mesh_tri_first, S.mesh_tri_count, r, R[3], R[7], h);
    else brute_force<false>(S.tris, S.n_tris, r, R[3], R[7], 0u, h, nt);
    write_hit(hits + 6 * (size_t)i, h);
  }
}

// --------------------------------------------------------------- launchers
int trace_grid_blocks() { return 2048; }

// Workgroups of the tail kernel.  Alone, every resident workgroup (about one
// path per lane: the tail ends with its longest path).  Beside the next
// pass's dense bounces (second stream), about three paths per lane and at
// most one workgroup per CU, which leaves most of each CU to them.
int tail_grid(int grid_trace, uint32_t paths, bool beside) {
  static int cus = 0, resident = 0;
  if (!cus) {
    int dev = 0, per = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus < 1)
      cus = 256;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, k_tail<true, true, true>, kBlock, 0) != hipSuccess ||
        per < 1)
      per = 1;
    resident = cus * per;
  }
  if (!beside) return std::max(1, std::min(grid_trace, resident));
  int want = (int)std::min<uint64_t>((uint64_t)cus, std::max<uint64_t>(8, ((uint64_t)paths + kTailPathsPerGroup - 1) /
                                                                                 kTailPathsPerGroup));
  return std::max(1, std::min(grid_trace, want));
}

// The traversal kernels keep one resident set of workgroups (persistent
// lanes); more would only queue behind them.
int traversal_grid(int64_t rays, bool two_level) {
  const int64_t need = std::max<int64_t>(1, (rays + kBlock - 1) / kBlock);
  static int resident[2] = {0, 0};
  if (!resident[two_level]) {
    int dev = 0, cus = 0, per = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus < 1)
      cus = 256;
    const hipError_t e = two_level
                             ? hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, k_traverse<false, false, true>, kBlock, 0)
                             : hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, k_traverse<false, false, false>, kBlock, 0);
    if (e != hipSuccess || per < 1) per = 1;
    resident[two_level] = std::max(1, cus * per);
  }
  // a multiple of the queues' segments, which the workgroups share out among them
  const int64_t g = std::min<int64_t>(need, resident[two_level]);
  return (int)std::max<int64_t>(kShards, need <= resident[two_level] ? (g + kShards - 1) / kShards * kShards
                                                                      : g / kShards * kShards);
}

// One shading launch per material class, one after the other: each fills the
// chip, and side by side on three streams they took as long together (33M
// paths: 3.45 ms either way) plus 20-30 us a vertex for the joins (box 512x512,
// 64 spp 5.86 ms against 5.32, icosphere field 13.4 / 13.0, material zoo 16.5 /
// 15.5).  In a pass of up to kOneShadeSlots slots no class fills it, and each
// launch lasts as long as one path's chain; all classes then share one launch.
// A wavefront render of one sample and 6 bounces in us, one launch each / one in
// all: zoo 64x64 1488 / 1074, 512x512 1714 / 1188, 1024x1024 2225 / 1786; field
// (82K triangles) 1206 / 1019, 1645 / 1461, 2173 / 1961; instanced 2973 / 2633, 2769 /
// 2380, 3628 / 3312; box 304 / 280, 424 / 398, 630 / 611.  From there on a scene
// of few classes loses to the lower occupancy (164 registers for every class):
// 2048x1024 with the hand-off, box 696 / 713, field 2475 / 2435.
static constexpr int32_t kOneShadeSlots = 1 << 20;
template <bool DEBUG, bool TWO>
static hipError_t shade_all(const SceneDev& S, const PathsDev& P, const PassArgs& A, int b, int next, hipStream_t st) {
  dim3 g(std::max(1, A.grid * kBlock / kShadeBlock)), blk(kShadeBlock);
  if (P.n <= kOneShadeSlots && __builtin_popcount(A.class_mask) > 2) {
    hipLaunchKernelGGL((k_shade_classes<DEBUG, TWO>), g, blk, 0, st, S, P, b, A.max_depth, next, A.sample, A.k0, A.k1,
                       A.nrc_bounce);
    return hipGetLastError();
  }
  for (int c = 0; c < kNumClasses; ++c) {
    if (!(A.class_mask & (1u << c))) continue;
    switch (c) {
#define PT_SHADE(C)                                                                                       \
  case C:                                                                                                 \
    hipLaunchKernelGGL((k_shade<C, DEBUG, TWO>), g, blk, 0, st, S, P, b, A.max_depth, next, A.sample, A.k0, \
                       A.k1, A.nrc_bounce);                                                               \
    break;
      PT_SHADE(kClsMiss)
      PT_SHADE(kClsAbsorb)
      PT_SHADE(kClsDiffuse)
      PT_SHADE(kClsMetal)
      PT_SHADE(kClsPlastic)
      PT_SHADE(kClsGlass)
      PT_SHADE(kClsGeneral)
#undef PT_SHADE
    }
  }
  return hipGetLastError();
}

// Unless the caller set the hand-off (then what it set holds as it is):
// the hand-off fraction counts from at most this many slots, so the tail
// kernel never takes more than max_fraction of them however large the pass:
// its lanes are 18 % active, the wavefront kernels fill the chip with a few
// hundred thousand paths.  Icosphere field 1080p 64 spp in passes of 2^25
// slots: 0.7M 103.8 ms, 1.4M 103.5, 2M 102.9, 3M 106.5, no bound (2^24
// slots) 121.9; instanced scene 32 spp: 151.7 / 153.7 / 150.8 / 153.7 ms.
static constexpr int32_t kTailPassSlots = 1 << 21;
// And a pass of few slots runs in the tail kernel from its first vertex: the
// wavefront's launches and count reads take longer than its better lane use
// saves.  Render of 6 bounces in us, hand-off from vertex 2 / whole pass: box 262K
// slots 437 / 312, 524K 490 / 455; material zoo 1485 / 1410, 1648 / 2097; icosphere
// field (1.31M triangles) 16K 1236 / 857, 262K 1458 / 1064, 524K 1665 / 1528;
// instanced 262K 2529 / 2083, 524K 2835 / 3247.
// Not so short paths where the general class is among the materials: a wave of
// the tail kernel runs the code of every class its lanes wait for (zoo 640x512,
// one sample: 2 bounces 599 / 948, 3 777 / 1168, 4 1016 / 1333; at 5 bounces 1444
// whole, 1459 with three streams and a hand-off).
// A frame of the radiance cache, beside which the next one runs, is whole where
// its training paths, which live longest, are a third of it or more, and then on
// the whole chip: the following frames queue behind it on the second stream.
// Eight frames, 65,536 training paths, 6 bounces, in us, wavefront first / whole:
// box 160x120 3437 / 3356, 400x300 3540 / 3655, 640x400 3693 / 4057; zoo 13234 / 11373,
// 13799 / 11979, 14343 / 14132; field 10463 / 8924, 10037 / 9287, 10026 / 10940;
// instanced 16166 / 15908, 18828 / 16799, 20019 / 19928.  160x120, 3 bounces: zoo
// 6184 / 8026, field 7878 / 7623, instanced 10616 / 11257; 4 bounces: zoo 8495 / 9501,
// instanced 12328 / 13056, field 9123 / 8231, box 3101 / 3008 (so 4 bounces are enough in
// single-level scenes without the general class).  64x48, 8,192 training paths:
// zoo 10151 / 12087, field 8389 / 8487, instanced 12889 / 16630.  A grid of one
// workgroup per CU instead of all that fit: field 400x300 10933 / 9321, zoo 14181 /
// 12118, 1000x60 7817 / 7978.
static constexpr int32_t kWholePassSlots = 5 << 16;
static constexpr int32_t kWholeFrameSlots = 3 << 16;
static constexpr uint32_t kWholeTrainPaths = 1u << 15;
static constexpr int kWholeDepth = 5;
static bool whole_pass(const PathsDev& P, const PassArgs& A) {
  if (!A.tail_sized) return false;
  const bool general = (A.class_mask & (1u << kClsGeneral)) != 0u;
  const bool deep = A.max_depth >= kWholeDepth - (general || A.two_level ? 0 : 1);
  if (!A.tail_stream) return P.n <= kWholePassSlots && (deep || !general);
  return deep && P.n <= kWholeFrameSlots && A.tail_bound >= kWholeTrainPaths && 3u * A.tail_bound >= (uint32_t)P.n;
}

template <bool DEBUG, bool COUNT, bool TWO>
static hipError_t bounce_loop(const SceneDev& S, const PathsDev& P, const CamDev& C, const PassArgs& A,
                              hipStream_t st) {
  dim3 blk(kBlock);
  if (A.wavefront_bounces) *A.wavefront_bounces = A.max_depth + 1;
  int n_trace = 0;
  // closest hits of queue q (none if q < 0) and the shadow rays of the last shading, on stream on
  auto traverse = [&](int q, hipStream_t on) {
    if (A.ext_events) hipEventRecord(A.ext_events[2 * n_trace], on);
    hipLaunchKernelGGL((k_traverse<DEBUG, COUNT, TWO>), dim3(A.grid_trace), blk, 0, on, S, P, q);
    if (A.ext_events) hipEventRecord(A.ext_events[2 * n_trace + 1], on);
    n_trace++;
  };
  bool shadow_pending = false;  // the last shading queued shadow rays that no launch has traced yet
  bool query_pending = false;   // the cache queries wait for the tail kernel's stream
  auto query = [&](hipStream_t q) -> hipError_t {
    if (A.query_wait) {  // the weights of the last training must be in place
      hipError_t e1 = hipStreamWaitEvent(q, A.query_wait, 0);
      if (e1 != hipSuccess) return e1;
    }
    if (A.nrc_events) hipEventRecord(A.nrc_events[0], q);
    hipError_t e2 = nrc_launch_query(P, A.nrc_fwd, std::min(A.grid, 1024), q);
    if (A.nrc_events) hipEventRecord(A.nrc_events[1], q);
    return e2;
  };
  const double tail_limit = A.tail_fraction * (double)(A.tail_sized ? std::min(P.n, kTailPassSlots) : P.n);
  const bool whole = whole_pass(P, A);
  for (int b = 0; b <= A.max_depth; ++b) {
    const int next = (b & 1) ^ 1, cur = b == 0 ? kQueueAll : b & 1;
    if (A.tail_host_count && (whole || b >= A.tail_min_bounce)) {
      // hand the remaining vertices to one persistent kernel once few paths are left
      uint32_t alive = 0;
      if (A.tail_bound && A.nrc_bounce >= 0 && b > A.nrc_bounce &&
          (double)A.tail_bound <= tail_limit) {
        alive = A.tail_bound;  // a bound known on the host: no need to read the count
      } else if (cur == kQueueAll) {
        alive = (uint32_t)P.n;
      } else {
        hipError_t e0 = hipMemcpyAsync(A.tail_host_count, P.counts, kShardWords * sizeof(uint32_t),
                                       hipMemcpyDeviceToHost, st);
        if (e0 == hipSuccess) e0 = hipStreamSynchronize(st);
        if (e0 != hipSuccess) return e0;
        for (uint32_t g = 0; g < kShards; ++g) alive += A.tail_host_count[count_ray(g, cur)];
      }
      if (whole || (double)alive <= tail_limit) {
        if (A.wavefront_bounces) *A.wavefront_bounces = b;
        hipStream_t ts = st;
        if (A.tail_stream) {  // continue on the second stream; the caller's stream is free for the next pass
          hipError_t e1 = hipEventRecord(A.tail_ready, st);
          if (e1 == hipSuccess) e1 = hipStreamWaitEvent(A.tail_stream, A.tail_ready, 0);
          if (e1 != hipSuccess) return e1;
          ts = A.tail_stream;
          if (A.tail_launched) *A.tail_launched = true;
        }
        if (shadow_pending) {  // the previous vertex's shadow rays come before the tail's next vertex
          traverse(-1, ts);
          shadow_pending = false;
        }
        if (query_pending) {  // the queries run on the tail kernel's stream, before it
          hipError_t e2 = query(ts);
          if (e2 != hipSuccess) return e2;
          query_pending = false;
        }
        hipLaunchKernelGGL(k_zero_u32, dim3(1), dim3(1), 0, ts, P.counts + kCountTail);
        if (A.tail_events) hipEventRecord(A.tail_events[0], ts);
        hipLaunchKernelGGL((k_tail<DEBUG, COUNT, TWO>),
                           dim3(tail_grid(A.grid_trace, alive, A.tail_stream && !whole)), blk, 0, ts,
                           S, P, cur, b, A.max_depth, A.sample, A.k0, A.k1, A.nrc_bounce);
        if (A.tail_events) hipEventRecord(A.tail_events[1], ts);
        if (A.nrc_bounce >= 0 && b <= A.nrc_bounce) {
          // the tail kernel took over at or before the query vertex: the paths it ends in the
          // cache join the query queue, so the queries run after it, on its stream
          hipError_t e2 = query(ts);
          if (e2 != hipSuccess) return e2;
        }
        break;
      }
    }
    hipLaunchKernelGGL(k_reset_counts, dim3(1), dim3(64), 0, st, P.counts, next);
    traverse(cur, st);  // this bounce's closest hits and the previous bounce's shadow rays
    shadow_pending = false;
    hipLaunchKernelGGL(k_bin, dim3(A.grid_bin), blk, 0, st, P, cur);  // also empties the shadow queue
    hipError_t e = shade_all<DEBUG, TWO>(S, P, A, b, next, st);
    if (e != hipSuccess) return e;
    shadow_pending = b < A.max_depth;
    if (b == A.nrc_bounce) {  // every path still alive ended in the cache at this vertex
      // (a path that ends in the cache casts no shadow ray at that vertex, so
      // the pending shadow rays touch other paths; the queries touch only the
      // paths that ended here, so they can wait for the tail kernel's stream)
      if (A.query_beside && A.tail_stream && P.n > P.n_render) {
        query_pending = true;
      } else {
        hipError_t e2 = query(st);
        if (e2 != hipSuccess) return e2;
      }
      if (P.n == P.n_render) break;  // no training paths: nothing continues
    }
  }
  if (shadow_pending) traverse(-1, st);
  if (query_pending) {  // no hand-off: the queries run here after all
    hipError_t e2 = query(st);
    if (e2 != hipSuccess) return e2;
  }
  if (A.trace_launches) *A.trace_launches = n_trace;
  return hipGetLastError();
}

hipError_t launch_pass(const SceneDev& S, const PathsDev& paths, const CamDev& C, const PassArgs& A, hipStream_t st) {
  dim3 blk(kBlock);
  PathsDev P = paths;
  P.seg_cap = (uint32_t)queue_segment(P.n);
  P.img_w = (uint32_t)C.W;
  if (A.debug) hipLaunchKernelGGL((k_generate<true>), dim3(A.grid), blk, 0, st, P, C, A.sample, A.k0, A.k1);
  else hipLaunchKernelGGL((k_generate<false>), dim3(A.grid), blk, 0, st, P, C, A.sample, A.k0, A.k1);
  const int sel = (A.debug ? 4 : 0) | (A.count ? 2 : 0) | (A.two_level ? 1 : 0);
  switch (sel) {
    case 0: return bounce_loop<false, false, false>(S, P, C, A, st);
    case 1: return bounce_loop<false, false, true>(S, P, C, A, st);
    case 2: return bounce_loop<false, true, false>(S, P, C, A, st);
    case 3: return bounce_loop<false, true, true>(S, P, C, A, st);
    case 4: return bounce_loop<true, false, false>(S, P, C, A, st);
    case 5: return bounce_loop<true, false, true>(S, P, C, A, st);
    case 6: return bounce_loop<true, true, false>(S, P, C, A, st);
    default: return bounce_loop<true, true, true>(S, P, C, A, st);
  }
}

static int blocks_for(int64_t n) {
  int64_t b = (n + kBlock - 1) / kBlock;
  if (b < 1) b = 1;
  if (b > 4096) b = 4096;
  return (int)b;
}

hipError_t launch_accumulate(const PathsDev& P, double* sum, int W, float* per_sample, uint64_t* sig_out,
                             int spp_total, int first_index, hipStream_t st) {
  const uint32_t part = std::min(P.spp, kAccumTile), tile = std::min((uint32_t)kBlock, kAccumTile / part);
  hipLaunchKernelGGL(k_accumulate, dim3(blocks_for((int64_t)P.w * P.h * kBlock / tile)), dim3(kBlock), 0, st, P, sum, W, per_sample,
                     sig_out, spp_total, first_index);
  return hipGetLastError();
}

hipError_t launch_resolve(const double* sum, float* out, int64_t n, double inv, hipStream_t st) {
  hipLaunchKernelGGL(k_resolve, dim3(blocks_for(n)), dim3(kBlock), 0, st, sum, out, n, inv);
  return hipGetLastError();
}

hipError_t launch_zero_f64(double* p, int64_t n, hipStream_t st) {
  hipLaunchKernelGGL(k_zero_f64, dim3(blocks_for(n)), dim3(kBlock), 0, st, p, n);
  return hipGetLastError();
}

hipError_t launch_zero_u64(unsigned long long* p, int64_t n, hipStream_t st) {
  hipLaunchKernelGGL(k_zero_u64, dim3(blocks_for(n)), dim3(kBlock), 0, st, p, n);
  return hipGetLastError();
}

hipError_t launch_trace_rays(const SceneDev& S, const float* rays, int64_t n, uint32_t* hits, bool brute,
                             bool two_level, int grid, unsigned long long* stats, hipStream_t st) {
  dim3 g(grid), blk(kBlock);
  const uint32_t nn = (uint32_t)n;
  if (brute && two_level) hipLaunchKernelGGL((k_trace_rays_brute<true>), g, blk, 0, st, S, rays, nn, hits);
  else if (brute) hipLaunchKernelGGL((k_trace_rays_brute<false>), g, blk, 0, st, S, rays, nn, hits);
  else if (two_level) hipLaunchKernelGGL((k_trace_rays<true>), g, blk, 0, st, S, rays, nn, hits, stats);
  else hipLaunchKernelGGL((k_trace_rays<false>), g, blk, 0, st, S, rays, nn, hits, stats);
  return hipGetLastError();
}

// ------------------------------------------------ allocation-free scratch
// Device memory of the allocation-free closest-hit call: a file-scope array,
// one copy per GPU, held until the process ends and shared by every call on
// that GPU.  In host code its name is not a device address: kernels receive
// the address hipGetSymbolAddress returns for the current device.
static __device__ __align__(256) unsigned char scratch[kNoAllocScratchBytes];

namespace {
constexpr int kMaxScratchDevices = 64;
std::mutex g_scratch_mu;
unsigned char* g_scratch_ptr[kMaxScratchDevices];
}  // namespace

hipError_t noalloc_scratch(int dev, unsigned char** out) {
  *out = nullptr;
  if (dev < 0 || dev >= kMaxScratchDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (!p) return hipErrorInvalidSymbol;
    g_scratch_ptr[dev] = static_cast<unsigned char*>(p);
  }
  *out = g_scratch_ptr[dev];
  return hipSuccess;
}

}  // namespace pt
