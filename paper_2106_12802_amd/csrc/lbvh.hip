// Linear BVH construction on the GPU (Karras, "Maximizing parallelism in the
// construction of BVHs, octrees, and k-d trees", HPG 2012).
//
//  1. centroid bounds (two-level min/max reduction)
//  2. 30-bit Morton code per triangle centroid, quantised in those bounds
//  3. stable LSD radix sort of (code, primitive) pairs, 8-bit digits; since the
//     primitives start in ascending order, the result is the order of the
//     unique 64-bit keys (code << 32 | primitive)
//  4. one internal node per adjacent key pair, its range and split found from
//     common-prefix lengths of the 64-bit keys (clz of xor)
//  5. leaf-to-root refit: each leaf walks up; the second thread to reach a
//     node (atomic visit counter) unions its children's boxes and continues.
//
//  6. collapse to a four-wide BVH, top down one level per launch (the first
//     levels in one block, the others with their sizes left on the device): a node
//     starts from its two binary children and twice opens the child of
//     largest surface area; binary subtrees of at most leaf_max triangles
//     become leaves (their leaf records are contiguous); nodes are then
//     renumbered densely in binary-node order.
//
// Binary node record (64 B): child boxes as 12 floats (left lo, left hi, right
// lo, right hi), two child references (bit 31 = leaf) and the node's range of
// leaf records (first, last).
//
// A second builder replaces steps 4-5 by agglomerative clustering over the
// Morton order (PLOC: Meister & Bittner, "Parallel Locally-Ordered Clustering
// for Bounding Volume Hierarchy Construction", IEEE TVCG 2018): every cluster
// finds, among the clusters within R places of it, the one whose union box has
// the smallest surface area; mutual nearest neighbours merge; the survivors are
// compacted in order; repeat until one cluster is left.  Ties are broken by a
// total order on cluster pairs, so some pair is always mutual and every round
// merges (identical boxes pair up with their neighbours, see ploc_nearest).
// The tree is then laid out depth first: internal nodes numbered in
// preorder (root 0) and leaf records in leaf order, so every subtree's leaves
// are a contiguous range as the BVH4 collapse needs.  Its trees have a lower
// surface-area cost than the Morton-split tree (10-15% on the procedural
// scenes), hence fewer node visits and triangle tests per ray.
//
// A build is bound by its chain of small dependent launches, not by its data (100k
// triangles: 28 MB, 6 us at the rate of a copy; 69 clustering rounds and 15
// levels).  So the rounds of at most 4096 clusters run in one block, larger ones
// take three launches with the counts left on the device (the host looks every
// eighth round), leaf counts and parents are written as clusters merge instead of
// by a walk with device-scope fences (266 us), and one allocation holds all
// scratch.  Measured, build of 20k / 100k / 200k triangles: 2.77 / 4.60 / 5.49 ms
// with five launches and a read-back per round, 0.69 / 1.01 / 1.53 ms now.
#include "mrs_internal.hpp"
#include "devmath.hpp"

namespace mrs {
namespace {

constexpr int RS_THREADS = 256;
constexpr int RS_ITEMS = 4;
constexpr int RS_TILE = RS_THREADS * RS_ITEMS;  // keys per block
constexpr int PLOC_RADIUS = 12;  // clusters searched on each side (fastest frame of 2..24)
constexpr int PLOC_MAX_ROUNDS = 256;
constexpr int PLOC_BATCH = 8;     // rounds enqueued between two looks at the cluster count
constexpr int PLOC_SMALL = 4096;  // clusters that one block finishes by itself (128 KB of LDS)

__device__ __forceinline__ f3 centroid(const float4* tri, int i) {
  f3 a = xyz(tri[3 * i]), b = xyz(tri[3 * i + 1]), c = xyz(tri[3 * i + 2]);
  return (a + b + c) * (1.0f / 3.0f);
}

// Half the surface area of a box of sides dx, dy, dz, in a fixed order of roundings: areas
// of nearly equal boxes decide which clusters merge and which child is opened, and the
// compiler contracts the plain sum in one way here and in another there.
__device__ __forceinline__ float half_area(float dx, float dy, float dz) {
  return fmaf(dx, dz, fmaf(dx, dy, dy * dz));
}

__global__ __launch_bounds__(256) void k_bounds_partial(const float4* __restrict__ tri, int n,
                                                        float* __restrict__ part) {
  __shared__ float s[6][256];
  float lo[3] = {INFINITY, INFINITY, INFINITY}, hi[3] = {-INFINITY, -INFINITY, -INFINITY};
  for (int i = blockIdx.x * 256 + threadIdx.x; i < n; i += gridDim.x * 256) {
    f3 c = centroid(tri, i);
    lo[0] = fminf(lo[0], c.x); lo[1] = fminf(lo[1], c.y); lo[2] = fminf(lo[2], c.z);
    hi[0] = fmaxf(hi[0], c.x); hi[1] = fmaxf(hi[1], c.y); hi[2] = fmaxf(hi[2], c.z);
  }
  for (int a = 0; a < 3; ++a) {
    s[a][threadIdx.x] = lo[a];
    s[3 + a][threadIdx.x] = hi[a];
  }
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) {
      for (int a = 0; a < 3; ++a) {
        s[a][threadIdx.x] = fminf(s[a][threadIdx.x], s[a][threadIdx.x + w]);
        s[3 + a][threadIdx.x] = fmaxf(s[3 + a][threadIdx.x], s[3 + a][threadIdx.x + w]);
      }
    }
    __syncthreads();
  }
  if (threadIdx.x < 6) part[blockIdx.x * 6 + threadIdx.x] = s[threadIdx.x][0];
}

// One wave per component (min x, y, z, max x, y, z).
__global__ __launch_bounds__(384) void k_bounds_final(const float* __restrict__ part, int nparts,
                                                      float* __restrict__ out) {
  const int a = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const bool is_lo = a < 3;
  float v = is_lo ? INFINITY : -INFINITY;
  for (int b = lane; b < nparts; b += 64) {
    const float x = part[b * 6 + a];
    v = is_lo ? fminf(v, x) : fmaxf(v, x);
  }
  for (int w = 32; w > 0; w >>= 1) {
    const float x = __shfl_xor(v, w);
    v = is_lo ? fminf(v, x) : fmaxf(v, x);
  }
  if (lane == 0) out[a] = v;
}

__device__ __forceinline__ uint32_t spread10(uint32_t v) {
  v = (v * 0x00010001u) & 0xFF0000FFu;
  v = (v * 0x00000101u) & 0x0F00F00Fu;
  v = (v * 0x00000011u) & 0xC30C30C3u;
  v = (v * 0x00000005u) & 0x49249249u;
  return v;
}

__device__ __forceinline__ uint32_t quant10(float x, float lo, float ext) {
  float q = ext > 0.0f ? (x - lo) / ext : 0.0f;
  q = fminf(fmaxf(q * 1024.0f, 0.0f), 1023.0f);
  return (uint32_t)q;
}

__global__ __launch_bounds__(256) void k_morton(const float4* __restrict__ tri, int n,
                                                const float* __restrict__ bounds,
                                                uint32_t* __restrict__ keys,
                                                uint32_t* __restrict__ vals) {
  int i = blockIdx.x * 256 + threadIdx.x;
  if (i >= n) return;
  f3 c = centroid(tri, i);
  uint32_t x = quant10(c.x, bounds[0], bounds[3] - bounds[0]);
  uint32_t y = quant10(c.y, bounds[1], bounds[4] - bounds[1]);
  uint32_t z = quant10(c.z, bounds[2], bounds[5] - bounds[2]);
  keys[i] = (spread10(x) << 2) | (spread10(y) << 1) | spread10(z);
  vals[i] = (uint32_t)i;
}

// ---------------------------------------------------------------- radix sort
// counts layout: digit-major, counts[d * nblocks + b]
__global__ __launch_bounds__(RS_THREADS) void k_rs_hist(const uint32_t* __restrict__ keys, int n,
                                                        int shift, int nblocks,
                                                        uint32_t* __restrict__ counts) {
  __shared__ uint32_t h[256];
  h[threadIdx.x] = 0;
  __syncthreads();
  const int base = blockIdx.x * RS_TILE;
  for (int k = 0; k < RS_ITEMS; ++k) {
    int i = base + k * RS_THREADS + threadIdx.x;
    if (i < n) atomicAdd(&h[(keys[i] >> shift) & 255u], 1u);
  }
  __syncthreads();
  counts[(size_t)threadIdx.x * nblocks + blockIdx.x] = h[threadIdx.x];
}

__device__ __forceinline__ uint32_t lanes_below(uint64_t m) {
  return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

// Inclusive scan over the 256 threads of a block (sh: 4 words of LDS, free again
// on return); *total gets the sum.
__device__ __forceinline__ uint32_t block_scan256(uint32_t v, uint32_t* sh, uint32_t* total) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const uint32_t y = __shfl_up(v, d);
    if (lane >= d) v += y;
  }
  if (lane == 63) sh[w] = v;
  __syncthreads();
  uint32_t before = 0, all = 0;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const uint32_t c = sh[k];
    before += k < w ? c : 0u;
    all += c;
  }
  __syncthreads();
  *total = all;
  return v + before;
}

// Sum of v[0 .. n - 1] over the threads of a 256-thread block (sh: 4 words).
__device__ __forceinline__ uint32_t block_sum(const uint32_t* __restrict__ v, int n,
                                              uint32_t* sh) {
  uint32_t x = 0, total;
  for (int i = threadIdx.x; i < n; i += 256) x += v[i];
  (void)block_scan256(x, sh, &total);
  return total;
}

// Exclusive scan of each digit's block counts (one block per digit) and the
// digit's total; the scatter adds the totals of the smaller digits.
__global__ __launch_bounds__(RS_THREADS) void k_rs_rows(uint32_t* __restrict__ counts, int nblocks,
                                                        uint32_t* __restrict__ totals) {
  __shared__ uint32_t sh[4];
  uint32_t* row = counts + (size_t)blockIdx.x * nblocks;
  uint32_t carry = 0;
  for (int b0 = 0; b0 < nblocks; b0 += RS_THREADS) {
    const int b = b0 + threadIdx.x;
    const uint32_t c = b < nblocks ? row[b] : 0u;
    uint32_t total;
    const uint32_t incl = block_scan256(c, sh, &total);
    if (b < nblocks) row[b] = carry + incl - c;
    carry += total;
  }
  if (threadIdx.x == 0) totals[blockIdx.x] = carry;
}

// Stable scatter: keys of a tile are ranked in tile order, 256 per round.  The
// rank among equal digits inside a wave comes from 8 ballots (one per digit
// bit); across the 4 waves of the block from per-wave digit counts in LDS.
__global__ __launch_bounds__(RS_THREADS) void k_rs_scatter(
    const uint32_t* __restrict__ keys, const uint32_t* __restrict__ vals, int n, int shift,
    int nblocks, const uint32_t* __restrict__ offsets, const uint32_t* __restrict__ totals,
    uint32_t* __restrict__ keys_out, uint32_t* __restrict__ vals_out) {
  __shared__ uint32_t base[256];
  __shared__ uint32_t wcnt[4][256];
  __shared__ uint32_t sh[4];
  const int t = threadIdx.x;
  const int wave = t >> 6;
  const uint32_t mine = totals[t];
  uint32_t all;
  base[t] = block_scan256(mine, sh, &all) - mine + offsets[(size_t)t * nblocks + blockIdx.x];
  for (int w = 0; w < 4; ++w) wcnt[w][t] = 0;
  __syncthreads();
  const int tile = blockIdx.x * RS_TILE;
  for (int k = 0; k < RS_ITEMS; ++k) {
    const int i = tile + k * RS_THREADS + t;
    const bool valid = i < n;
    uint32_t key = valid ? keys[i] : 0u;
    uint32_t val = valid ? vals[i] : 0u;
    uint32_t dig = (key >> shift) & 255u;
    uint64_t peers = __ballot(valid);
#pragma unroll
    for (int b = 0; b < 8; ++b) {
      const bool bit = (dig >> b) & 1u;
      const uint64_t bb = __ballot(bit);
      peers &= bit ? bb : ~bb;
    }
    const uint32_t rank = lanes_below(peers);
    if (valid && rank == 0) wcnt[wave][dig] = (uint32_t)__popcll(peers);
    __syncthreads();
    if (valid) {
      uint32_t off = base[dig] + rank;
      for (int w = 0; w < wave; ++w) off += wcnt[w][dig];
      if (off < (uint32_t)n) {  // always true for consistent counts; guards the write
        keys_out[off] = key;
        vals_out[off] = val;
      }
    }
    __syncthreads();
    base[t] += wcnt[0][t] + wcnt[1][t] + wcnt[2][t] + wcnt[3][t];
    for (int w = 0; w < 4; ++w) wcnt[w][t] = 0;
    __syncthreads();
  }
}

// ---------------------------------------------------------------- hierarchy
__device__ __forceinline__ int delta(const uint32_t* code, const uint32_t* prim, int n, int i,
                                     int j) {
  if (j < 0 || j >= n) return -1;
  uint64_t a = ((uint64_t)code[i] << 32) | prim[i];
  uint64_t b = ((uint64_t)code[j] << 32) | prim[j];
  return __clzll((long long)(a ^ b));
}

__global__ __launch_bounds__(256) void k_hierarchy(const uint32_t* __restrict__ code,
                                                   const uint32_t* __restrict__ prim, int n,
                                                   float4* __restrict__ nodes,
                                                   uint32_t* __restrict__ parent_int,
                                                   uint32_t* __restrict__ parent_leaf) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i >= n - 1) return;
  const int d = (delta(code, prim, n, i, i + 1) - delta(code, prim, n, i, i - 1)) >= 0 ? 1 : -1;
  const int dmin = delta(code, prim, n, i, i - d);
  int lmax = 2;
  while (delta(code, prim, n, i, i + lmax * d) > dmin) lmax <<= 1;
  int l = 0;
  for (int t = lmax >> 1; t >= 1; t >>= 1)
    if (delta(code, prim, n, i, i + (l + t) * d) > dmin) l += t;
  const int j = i + l * d;
  const int dnode = delta(code, prim, n, i, j);
  int s = 0;
  int t = l;
  do {
    t = (t + 1) >> 1;
    if (delta(code, prim, n, i, i + (s + t) * d) > dnode) s += t;
  } while (t > 1);
  const int g = i + s * d + min(d, 0);
  const int lo = min(i, j), hi = max(i, j);
  if (g < lo || g + 1 > hi) return;  // cannot happen for unique keys; guards the writes
  uint32_t left, right;
  if (lo == g) {
    left = LEAF_BIT | (uint32_t)g;
    parent_leaf[g] = (uint32_t)i;
  } else {
    left = (uint32_t)g;
    parent_int[g] = (uint32_t)i;
  }
  if (hi == g + 1) {
    right = LEAF_BIT | (uint32_t)(g + 1);
    parent_leaf[g + 1] = (uint32_t)i;
  } else {
    right = (uint32_t)(g + 1);
    parent_int[g + 1] = (uint32_t)i;
  }
  nodes[4 * i + 3] = make_float4(__uint_as_float(left), __uint_as_float(right),
                                 __uint_as_float((uint32_t)lo), __uint_as_float((uint32_t)hi));
}

__global__ __launch_bounds__(256) void k_fill_u32(uint32_t* p, int n, uint32_t v) {
  int i = blockIdx.x * 256 + threadIdx.x;
  if (i < n) p[i] = v;
}

// Leaf records in leaf order, then the bottom-up refit.
__global__ __launch_bounds__(256) void k_leaves_refit(const float4* __restrict__ tri_src,
                                                      const uint32_t* __restrict__ leaf_prim,
                                                      int n, float4* __restrict__ leaf_tri,
                                                      float* __restrict__ nodes_f,
                                                      const uint32_t* __restrict__ parent_int,
                                                      const uint32_t* __restrict__ parent_leaf,
                                                      uint32_t* __restrict__ visits) {
  const int k = blockIdx.x * 256 + threadIdx.x;
  if (k >= n) return;
  const uint32_t p = leaf_prim[k];
  const f3 v0 = xyz(tri_src[3 * p]), v1 = xyz(tri_src[3 * p + 1]), v2 = xyz(tri_src[3 * p + 2]);
  const f3 e1 = v1 - v0, e2 = v2 - v0;
  leaf_tri[3 * k + 0] = make_float4(v0.x, v0.y, v0.z, __uint_as_float(p));
  leaf_tri[3 * k + 1] = make_float4(e1.x, e1.y, e1.z, 0.0f);
  leaf_tri[3 * k + 2] = make_float4(e2.x, e2.y, e2.z, 0.0f);
  if (n < 2) return;
  float lo[3] = {fminf(v0.x, fminf(v1.x, v2.x)), fminf(v0.y, fminf(v1.y, v2.y)),
                 fminf(v0.z, fminf(v1.z, v2.z))};
  float hi[3] = {fmaxf(v0.x, fmaxf(v1.x, v2.x)), fmaxf(v0.y, fmaxf(v1.y, v2.y)),
                 fmaxf(v0.z, fmaxf(v1.z, v2.z))};
  uint32_t child = LEAF_BIT | (uint32_t)k;
  uint32_t node = parent_leaf[k];
  for (int guard = 0; guard < 2 * MAX_STACK + 2; ++guard) {
    if (node >= (uint32_t)(n - 1)) return;  // parents are always internal nodes
    float* nf = nodes_f + 16 * (size_t)node;
    const uint32_t left_ref = __float_as_uint(nf[12]);
    const int slot = (left_ref == child) ? 0 : 6;
    for (int a = 0; a < 3; ++a) {
      __hip_atomic_store(nf + slot + a, lo[a], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      __hip_atomic_store(nf + slot + 3 + a, hi[a], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    const uint32_t prev =
        __hip_atomic_fetch_add(visits + node, 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT);
    if (prev == 0) return;  // the sibling subtree is not finished; its thread continues
    const int other = 6 - slot;
    for (int a = 0; a < 3; ++a) {
      lo[a] = fminf(lo[a], __hip_atomic_load(nf + other + a, __ATOMIC_RELAXED,
                                             __HIP_MEMORY_SCOPE_AGENT));
      hi[a] = fmaxf(hi[a], __hip_atomic_load(nf + other + 3 + a, __ATOMIC_RELAXED,
                                             __HIP_MEMORY_SCOPE_AGENT));
    }
    if (node == 0) return;  // root: its box is not stored
    child = node;
    node = parent_int[node];
  }
}

// ---------------------------------------------------------------- PLOC
constexpr uint32_t NO_PARENT = 0xffffffffu;
// Device words of a clustering build: merges so far, 1 once one cluster is left
// and every merge is made, deepest leaf or node, a fault (below), root.
enum { PC_MERGES = 0, PC_DONE, PC_DEPTH, PC_BAD, PC_ROOT, PLOC_CTR };
enum { BAD_TREE = 1, BAD_STUCK = 2 };  // PC_BAD: malformed, a round without a merge

__device__ __forceinline__ float box_half_area(float4 lo, float4 hi) {
  return half_area(hi.x - lo.x, hi.y - lo.y, hi.z - lo.z);
}

// Clusters start as the leaves in Morton order: reference LEAF_BIT | k, lo.w = the
// cluster's leaf count.
__global__ __launch_bounds__(256) void k_ploc_init(const float4* __restrict__ tri_src,
                                                   const uint32_t* __restrict__ prim, int n,
                                                   uint32_t* __restrict__ cref,
                                                   float4* __restrict__ clo,
                                                   float4* __restrict__ chi,
                                                   uint32_t* __restrict__ mcount,
                                                   uint32_t* __restrict__ ctr) {
  const int k = blockIdx.x * 256 + threadIdx.x;
  if (k == 0) mcount[0] = (uint32_t)n;
  if (k < PLOC_CTR) ctr[k] = 0u;
  if (k >= n) return;
  const uint32_t p = prim[k];
  const f3 a = xyz(tri_src[3 * p]), b = xyz(tri_src[3 * p + 1]), c = xyz(tri_src[3 * p + 2]);
  cref[k] = LEAF_BIT | (uint32_t)k;
  clo[k] = make_float4(fminf(a.x, fminf(b.x, c.x)), fminf(a.y, fminf(b.y, c.y)),
                       fminf(a.z, fminf(b.z, c.z)), __uint_as_float(1u));
  chi[k] = make_float4(fmaxf(a.x, fmaxf(b.x, c.x)), fmaxf(a.y, fmaxf(b.y, c.y)),
                       fmaxf(a.z, fmaxf(b.z, c.z)), 0.0f);
}

// Nearest neighbour by union surface area among the clusters within PLOC_RADIUS
// places of cluster c of m; l(j) and h(j) return cluster j's box.  Equal areas are
// settled by a total order of pairs: nearer pairs first, then pairs whose smaller
// member is even, then by smaller member.  Among equal costs (equal boxes, regular
// grids) clusters thus pair up as (0, 1), (2, 3), ...: every cluster merges and
// the tree stays balanced, where a plain index order would merge one pair per
// round.  Candidates come by distance, left before right, so an equal one replaces
// the best only where it is the right one of the same odd distance and c is even; the
// first of infinite cost is equal to no pair yet and taken, one that is not a number
// (boxes beyond FP32's range) is no candidate.
// No branches: the boxes of several candidates are in flight at once (one after
// the other the LDS latency bounds it).
template <class L, class H>
__device__ __forceinline__ int ploc_nearest(int c, int m, L l, H h) {
  const float4 lo = l(c), hi = h(c);
  float best = INFINITY;
  int bj = -1;
  const bool even = (c & 1) == 0;
  constexpr int G = 4;  // distances in flight
  static_assert(PLOC_RADIUS % G == 0, "whole groups of distances");
#pragma unroll 1
  for (int d0 = 1; d0 <= PLOC_RADIUS; d0 += G) {
    float4 cl[2 * G], ch[2 * G];
#pragma unroll
    for (int u = 0; u < 2 * G; ++u) {
      const int d = d0 + (u >> 1), j = (u & 1) ? min(c + d, m - 1) : max(c - d, 0);
      cl[u] = l(j);
      ch[u] = h(j);
    }
#pragma unroll
    for (int u = 0; u < 2 * G; ++u) {
      const int d = d0 + (u >> 1), j = (u & 1) ? c + d : c - d;
      const bool in = (u & 1) ? j < m : j >= 0;
      float a = box_half_area(make_float4(fminf(lo.x, cl[u].x), fminf(lo.y, cl[u].y),
                                          fminf(lo.z, cl[u].z), 0.0f),
                              make_float4(fmaxf(hi.x, ch[u].x), fmaxf(hi.y, ch[u].y),
                                          fmaxf(hi.z, ch[u].z), 0.0f));
      const bool tie = (bj < 0) | ((u & 1) ? (bj == c - d) & ((d & 1) != 0) & even : false);
      const bool take = in & ((a < best) | ((a == best) & tie));
      best = take ? a : best;
      bj = take ? j : bj;
    }
  }
  return bj;
}

// A block's boxes and its neighbours' go through LDS.
__global__ __launch_bounds__(256) void k_ploc_nn(const uint32_t* __restrict__ mcount,
                                                 const float4* __restrict__ clo,
                                                 const float4* __restrict__ chi,
                                                 int* __restrict__ nn) {
  __shared__ float4 sl[256 + 2 * PLOC_RADIUS], sh[256 + 2 * PLOC_RADIUS];
  const int m = (int)*mcount, c0 = blockIdx.x * 256 - PLOC_RADIUS;
  if ((int)blockIdx.x * 256 >= m) return;
  for (int i = threadIdx.x; i < 256 + 2 * PLOC_RADIUS; i += 256) {
    const int j = c0 + i;
    if (j >= 0 && j < m) {
      sl[i] = clo[j];
      sh[i] = chi[j];
    }
  }
  __syncthreads();
  const int c = blockIdx.x * 256 + threadIdx.x;
  if (c >= m) return;
  nn[c] = ploc_nearest(
      c, m, [&](int j) { return sl[j - c0]; }, [&](int j) { return sh[j - c0]; });
}

// Cluster pair (c, j), c < j, becomes internal node t: the node's record, its
// children's parents ((parent << 1) | side) and leaf counts; returns the merged
// cluster in place of c.
struct PlocTree {
  float* tnodes;
  uint32_t *par_int, *par_leaf, *sz2;
};
__device__ __forceinline__ void ploc_merge(const PlocTree& T, uint32_t t, uint32_t& ref, float4& lo,
                                           float4& hi, uint32_t ref2, float4 l2, float4 h2) {
  float4* o = reinterpret_cast<float4*>(T.tnodes) + 4 * (size_t)t;
  o[0] = make_float4(lo.x, lo.y, lo.z, hi.x);
  o[1] = make_float4(hi.y, hi.z, l2.x, l2.y);
  o[2] = make_float4(l2.z, h2.x, h2.y, h2.z);
  o[3] = make_float4(__uint_as_float(ref), __uint_as_float(ref2), 0.0f, 0.0f);
  auto parent = [&](uint32_t r, uint32_t side) {
    if (r & LEAF_BIT) T.par_leaf[r & ~LEAF_BIT] = (t << 1) | side;
    else T.par_int[r] = (t << 1) | side;
  };
  parent(ref, 0u);
  parent(ref2, 1u);
  const uint32_t n1 = __float_as_uint(lo.w), n2 = __float_as_uint(l2.w);
  T.sz2[2 * (size_t)t] = n1;
  T.sz2[2 * (size_t)t + 1] = n2;
  ref = t;
  lo = make_float4(fminf(lo.x, l2.x), fminf(lo.y, l2.y), fminf(lo.z, l2.z),
                   __uint_as_float(n1 + n2));
  hi = make_float4(fmaxf(hi.x, h2.x), fmaxf(hi.y, h2.y), fmaxf(hi.z, h2.z), 0.0f);
}

// Mutual nearest neighbours c < j merge into a new internal node (in place of
// c; j is dropped); counts the clusters each block keeps.
__global__ __launch_bounds__(256) void k_ploc_merge(const uint32_t* __restrict__ mcount, int nint,
                                                    const int* __restrict__ nn,
                                                    uint32_t* __restrict__ cref,
                                                    float4* __restrict__ clo,
                                                    float4* __restrict__ chi, PlocTree T,
                                                    uint32_t* __restrict__ ctr,
                                                    uint32_t* __restrict__ keep,
                                                    uint32_t* __restrict__ bcount) {
  __shared__ uint32_t wc[4];
  const int m = (int)*mcount, c = blockIdx.x * 256 + threadIdx.x;
  if ((int)blockIdx.x * 256 >= m) return;
  const int j = c < m ? nn[c] : -1;
  const bool mutual = j >= 0 && j < m && nn[j] == c;
  const bool kept = c < m && !(mutual && c > j), merge = mutual && c < j;
  const uint64_t mm = __ballot(merge), mk = __ballot(kept);
  if (c < m) keep[c] = kept ? 1u : 0u;
  uint32_t t = 0;
  if (__lane_id() == 0 && mm) t = atomicAdd(ctr + PC_MERGES, (uint32_t)__popcll(mm));
  t = __shfl(t, 0) + lanes_below(mm);
  if (merge && t < (uint32_t)nint) {  // always: n leaves make n - 1 merges
    uint32_t ref = cref[c];
    float4 lo = clo[c], hi = chi[c];
    ploc_merge(T, t, ref, lo, hi, cref[j], clo[j], chi[j]);
    cref[c] = ref;
    clo[c] = lo;
    chi[c] = hi;
  }
  if ((threadIdx.x & 63) == 0) wc[threadIdx.x >> 6] = (uint32_t)__popcll(mk);
  __syncthreads();
  if (threadIdx.x == 0) bcount[blockIdx.x] = wc[0] + wc[1] + wc[2] + wc[3];
}

// Kept clusters in order into the other arrays, SUB tiles of 256 per block (its
// offset: the sum of the counts before it); the last cluster's thread writes the
// new count.
template <int SUB>
__global__ __launch_bounds__(256) void k_ploc_scatter(
    const uint32_t* __restrict__ mcount, const uint32_t* __restrict__ keep,
    const uint32_t* __restrict__ bcount, const uint32_t* __restrict__ cref,
    const float4* __restrict__ clo, const float4* __restrict__ chi, uint32_t* __restrict__ cref2,
    float4* __restrict__ clo2, float4* __restrict__ chi2, uint32_t* __restrict__ mnext) {
  __shared__ uint32_t sh[4], wc[4];
  const int m = (int)*mcount;
  if ((int64_t)blockIdx.x * SUB * 256 >= m) return;
  uint32_t base = block_sum(bcount, blockIdx.x * SUB, sh);
  for (int q = 0; q < SUB; ++q) {
    const int c = (blockIdx.x * SUB + q) * 256 + threadIdx.x;
    const bool k = c < m && keep[c];
    const uint64_t b = __ballot(k);
    const int w = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) wc[w] = (uint32_t)__popcll(b);
    __syncthreads();
    uint32_t pos = base + lanes_below(b);
    for (int v = 0; v < w; ++v) pos += wc[v];
    if (k && pos < (uint32_t)m) {
      cref2[pos] = cref[c];
      clo2[pos] = clo[c];
      chi2[pos] = chi[c];
    }
    if (c == m - 1) *mnext = pos + (k ? 1u : 0u);
    base += wc[0] + wc[1] + wc[2] + wc[3];
    __syncthreads();
  }
}

// The rounds from at most PLOC_SMALL clusters on, in one block: the boxes stay in
// LDS, each thread holds up to four clusters while they are merged and compacted.
// A round costs its LDS reads and a few barriers; as five launches and a count
// read back by the host it cost about 50 us; 53 of the 69 rounds of 100,000 triangles
// run here, in 248 us (a round of more clusters: 16 us in three launches).  4096 clusters
// are what LDS holds; smaller lines were not measured.
// Ends with PC_DONE = 1 and PC_ROOT when one cluster is left, with PC_DONE = 0
// after max_rounds.
__global__ __launch_bounds__(1024) void k_ploc_small(const uint32_t* __restrict__ mcount, int nint,
                                                     const uint32_t* __restrict__ cref,
                                                     const float4* __restrict__ clo,
                                                     const float4* __restrict__ chi, PlocTree T,
                                                     uint32_t* __restrict__ ctr, int max_rounds) {
  constexpr int PER = PLOC_SMALL / 1024;
  __shared__ float4 slo[PLOC_SMALL], shi[PLOC_SMALL];  // lo.w: leaf count, hi.w: reference
  __shared__ uint16_t snn[PLOC_SMALL];
  __shared__ uint32_t wk[PER * 16], wm[PER * 16], tot[2];
  static_assert(PER * 16 == 64, "one wave scans the counts of all waves");
  const int tid = threadIdx.x, wave = tid >> 6;
  int m = (int)*mcount;
  if (m > PLOC_SMALL || m < 1) return;
  uint32_t merges = ctr[PC_MERGES];
  bool stuck = false;
  auto put = [&](int c, uint32_t ref, float4 lo, float4 hi) {
    slo[c] = lo;
    shi[c] = make_float4(hi.x, hi.y, hi.z, __uint_as_float(ref));
  };
  auto get = [&](int c, uint32_t& ref, float4& lo, float4& hi) {
    lo = slo[c];
    hi = shi[c];
    ref = __float_as_uint(hi.w);
  };
  for (int c = tid; c < m; c += 1024) put(c, cref[c], clo[c], chi[c]);
  __syncthreads();
  for (int round = 0; m > 1 && round < max_rounds; ++round) {
#pragma unroll 1
    for (int c = tid; c < m; c += 1024)
      snn[c] = (uint16_t)ploc_nearest(
          c, m, [&](int j) { return slo[j]; }, [&](int j) { return shi[j]; });
    __syncthreads();
    uint32_t ref[PER];
    float4 lo[PER], hi[PER];
    uint64_t bk[PER], bm[PER];
    bool kept[PER], merge[PER];
#pragma unroll
    for (int q = 0; q < PER; ++q) {
      const int c = q * 1024 + tid;
      const int j = c < m ? (int)snn[c] : -1;
      const bool mutual = j >= 0 && j < m && (int)snn[j] == c;
      kept[q] = c < m && !(mutual && c > j);
      merge[q] = mutual && c < j;
      bk[q] = __ballot(kept[q]);
      bm[q] = __ballot(merge[q]);
      if ((tid & 63) == 0) {
        wk[q * 16 + wave] = (uint32_t)__popcll(bk[q]);
        wm[q * 16 + wave] = (uint32_t)__popcll(bm[q]);
      }
    }
    __syncthreads();
    if (wave < 2) {  // exclusive scan of the waves' counts, in cluster order
      uint32_t* v = wave ? wm : wk;
      const uint32_t own = v[tid & 63];
      uint32_t x = own;
#pragma unroll
      for (int d = 1; d < 64; d <<= 1) {
        const uint32_t y = __shfl_up(x, d);
        if ((tid & 63) >= d) x += y;
      }
      v[tid & 63] = x - own;
      if ((tid & 63) == 63) tot[wave] = x;
    }
    __syncthreads();
    const uint32_t nk = tot[0], nm = tot[1];
    uint32_t pos[PER];
#pragma unroll
    for (int q = 0; q < PER; ++q) {
      const uint32_t t = merges + wm[q * 16 + wave] + lanes_below(bm[q]);
      pos[q] = wk[q * 16 + wave] + lanes_below(bk[q]);
      const int c = q * 1024 + tid;
      if (kept[q]) {
        get(c, ref[q], lo[q], hi[q]);
        if (merge[q] && t < (uint32_t)nint) {
          uint32_t r2;
          float4 l2, h2;
          get(snn[c], r2, l2, h2);
          ploc_merge(T, t, ref[q], lo[q], hi[q], r2, l2, h2);
        }
      }
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < PER; ++q)
      if (kept[q]) put((int)pos[q], ref[q], lo[q], hi[q]);
    merges += nm;
    stuck = nm == 0;  // some pair is mutual unless costs are not numbers
    if (stuck) break;
    m = (int)nk;
    __syncthreads();
  }
  if (tid == 0) {
    const uint32_t root = __float_as_uint(shi[0].w);
    const bool ok = m == 1 && merges == (uint32_t)nint && root < (uint32_t)nint;
    if (ok) T.par_int[root] = NO_PARENT;
    ctr[PC_MERGES] = merges;
    ctr[PC_ROOT] = root;
    ctr[PC_DONE] = ok ? 1u : 0u;
    if (m == 1 && !ok) ctr[PC_BAD] = BAD_TREE;
    if (stuck) ctr[PC_BAD] = BAD_STUCK;
  }
}

// Depth-first layout, each node and leaf walking up to the root: a left child
// comes right after its parent in preorder and shares its first leaf; a right
// child follows the left subtree (its leaf count L): preorder + L, first leaf + L.
__global__ __launch_bounds__(256) void k_ploc_order(int n, int nint,
                                                    const uint32_t* __restrict__ par_int,
                                                    const uint32_t* __restrict__ par_leaf,
                                                    const uint32_t* __restrict__ sz2,
                                                    uint32_t* __restrict__ pre_int,
                                                    uint32_t* __restrict__ first_int,
                                                    uint32_t* __restrict__ first_leaf,
                                                    uint32_t* __restrict__ ctr) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (!ctr[PC_DONE]) return;
  uint32_t depth = 0;
  if (i < nint + n) {
    uint32_t x = i < nint ? par_int[i] : par_leaf[i - nint];
    uint32_t pre = 0, first = 0;
    for (; x != NO_PARENT; ++depth) {
      if (depth >= 4 * MAX_STACK) break;  // too deep (the caller falls back)
      const uint32_t p = x >> 1;
      if (p >= (uint32_t)nint) {  // cannot happen for a tree
        atomicOr(ctr + PC_BAD, (uint32_t)BAD_TREE);
        break;
      }
      const uint32_t L = sz2[2 * (size_t)p], up = par_int[p];
      pre += x & 1u ? L : 1u;
      first += x & 1u ? L : 0u;
      x = up;
    }
    if (i < nint) {
      pre_int[i] = pre;
      first_int[i] = first;
    } else {
      first_leaf[i - nint] = first;
    }
  }
  // one atomic per wave: 2 n of them on one word took most of this kernel
  for (int w = 32; w > 0; w >>= 1) depth = max(depth, (uint32_t)__shfl_xor((int)depth, w));
  if (__lane_id() == 0) atomicMax(ctr + PC_DEPTH, depth);
}

// Final binary records: temporary node t goes to its preorder place, with its
// references and leaf range in the final numbering.
__global__ __launch_bounds__(256) void k_ploc_emit(int nint, int n, const float* __restrict__ tnodes,
                                                   const uint32_t* __restrict__ pre_int,
                                                   const uint32_t* __restrict__ first_int,
                                                   const uint32_t* __restrict__ first_leaf,
                                                   const uint32_t* __restrict__ sz2,
                                                   const uint32_t* __restrict__ ctr,
                                                   float* __restrict__ nodes_f) {
  const int t = blockIdx.x * 256 + threadIdx.x;
  if (t >= nint || !ctr[PC_DONE]) return;
  const uint32_t d = pre_int[t];
  if (d >= (uint32_t)nint) return;  // cannot happen for a tree
  const float4* src = reinterpret_cast<const float4*>(tnodes) + 4 * (size_t)t;
  float4* o = reinterpret_cast<float4*>(nodes_f) + 4 * (size_t)d;
  const float4 r4 = src[3];
  auto ref = [&](uint32_t r) {
    return (r & LEAF_BIT) ? LEAF_BIT | first_leaf[min(r & ~LEAF_BIT, (uint32_t)n - 1)]
                          : pre_int[min(r, (uint32_t)nint - 1)];
  };
  const uint32_t first = first_int[t];
  const uint32_t last = first + sz2[2 * (size_t)t] + sz2[2 * (size_t)t + 1] - 1u;
  for (int a = 0; a < 3; ++a) o[a] = src[a];
  o[3] = make_float4(__uint_as_float(ref(__float_as_uint(r4.x))),
                     __uint_as_float(ref(__float_as_uint(r4.y))), __uint_as_float(first),
                     __uint_as_float(last));
}

// Morton position k -> leaf position first_leaf[k]: primitives, codes and leaf
// records (v0, primitive id) (e1) (e2) in leaf order.
__global__ __launch_bounds__(256) void k_ploc_leaves(
    int n, const float4* __restrict__ tri_src, const uint32_t* __restrict__ prim,
    const uint32_t* __restrict__ code, const uint32_t* __restrict__ first_leaf,
    const uint32_t* __restrict__ ctr, uint32_t* __restrict__ leaf_prim,
    uint32_t* __restrict__ leaf_code, float4* __restrict__ leaf_tri) {
  const int k = blockIdx.x * 256 + threadIdx.x;
  if (k >= n || !ctr[PC_DONE]) return;
  const uint32_t pos = first_leaf[k], p = prim[k];
  if (pos >= (uint32_t)n) return;  // cannot happen for a tree
  leaf_prim[pos] = p;
  leaf_code[pos] = code[k];
  const f3 v0 = xyz(tri_src[3 * p]), v1 = xyz(tri_src[3 * p + 1]), v2 = xyz(tri_src[3 * p + 2]);
  const f3 e1 = v1 - v0, e2 = v2 - v0;
  float4* o = leaf_tri + 3 * (size_t)pos;
  o[0] = make_float4(v0.x, v0.y, v0.z, __uint_as_float(p));
  o[1] = make_float4(e1.x, e1.y, e1.z, 0.0f);
  o[2] = make_float4(e2.x, e2.y, e2.z, 0.0f);
}

// ---------------------------------------------------------------- BVH4 collapse
struct Cand {
  uint32_t ref;
  float lo[3], hi[3];
};

__device__ __forceinline__ void binary_children(const float* __restrict__ nf, Cand& l, Cand& r) {
  for (int a = 0; a < 3; ++a) {
    l.lo[a] = nf[a];
    l.hi[a] = nf[3 + a];
    r.lo[a] = nf[6 + a];
    r.hi[a] = nf[9 + a];
  }
  l.ref = __float_as_uint(nf[12]);
  r.ref = __float_as_uint(nf[13]);
}

__device__ __forceinline__ float half_area(const Cand& c) {
  return half_area(c.hi[0] - c.lo[0], c.hi[1] - c.lo[1], c.hi[2] - c.lo[2]);
}

// leaf-record range of a binary reference
__device__ __forceinline__ void ref_range(const float* __restrict__ nodes_f, uint32_t ref,
                                          uint32_t& first, uint32_t& last) {
  if (ref & LEAF_BIT) {
    first = last = ref & ~LEAF_BIT;
  } else {
    first = __float_as_uint(nodes_f[16 * (size_t)ref + 14]);
    last = __float_as_uint(nodes_f[16 * (size_t)ref + 15]);
  }
}

// Binary node b becomes BVH4 node b (sparse numbering); its children that are
// nodes themselves are queued for the next level.
__device__ __forceinline__ void collapse_node(const float* __restrict__ nodes_f, uint32_t b,
                                              uint32_t* __restrict__ q_out,
                                              uint32_t* __restrict__ cnt_out,
                                              float4* __restrict__ sparse4,
                                              uint32_t* __restrict__ is4, int leaf_max) {
  Cand c[4];
  binary_children(nodes_f + 16 * (size_t)b, c[0], c[1]);
  int nc = 2;
  for (int open = 0; open < 2; ++open) {
    int best = -1;
    float best_area = -1.0f;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      if (k >= nc || (c[k].ref & LEAF_BIT)) continue;
      uint32_t f, l;
      ref_range(nodes_f, c[k].ref, f, l);
      if (l - f + 1 <= (uint32_t)leaf_max) continue;
      const float a = half_area(c[k]);
      if (a > best_area) {
        best_area = a;
        best = k;
      }
    }
    if (best < 0) break;
    Cand l, r;
    uint32_t opened = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k)
      if (k == best) opened = c[k].ref;
    binary_children(nodes_f + 16 * (size_t)opened, l, r);
    // c[best] <- l, c[best + 1] <- r, later children shift right by one
#pragma unroll
    for (int k = 3; k >= 1; --k)
      if (k > best + 1 && k <= nc) c[k] = c[k - 1];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      if (k == best) c[k] = l;
      if (k == best + 1) c[k] = r;
    }
    ++nc;
  }
  float box[6][4];
  uint32_t refs[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    if (k < nc) {
      uint32_t f, l;
      ref_range(nodes_f, c[k].ref, f, l);
      if ((c[k].ref & LEAF_BIT) || l - f + 1 <= (uint32_t)leaf_max) {
        refs[k] = leaf4_ref(f, l - f + 1);
      } else {
        refs[k] = c[k].ref;
        q_out[atomicAdd(cnt_out, 1u)] = c[k].ref;
      }
      for (int a = 0; a < 3; ++a) {
        box[a][k] = c[k].lo[a];
        box[3 + a][k] = c[k].hi[a];
      }
    } else {
      refs[k] = EMPTY4;
      for (int a = 0; a < 3; ++a) {
        box[a][k] = INFINITY;
        box[3 + a][k] = -INFINITY;
      }
    }
  }
  float4* o = sparse4 + 8 * (size_t)b;
  for (int a = 0; a < 6; ++a) o[a] = make_float4(box[a][0], box[a][1], box[a][2], box[a][3]);
  o[6] = make_float4(__uint_as_float(refs[0]), __uint_as_float(refs[1]),
                     __uint_as_float(refs[2]), __uint_as_float(refs[3]));
  o[7] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
  is4[b] = 1u;
}

// The levels have one counter each, cnt[0 .. C4_LEVELS] (level l's items in queue
// l % 2), so that they are enqueued without a look at their sizes.
constexpr int C4_LEVELS = 4 * MAX_STACK;
constexpr int C4_TOP = 5;     // levels of at most 4^5 items that one block does by itself
constexpr int C4_BATCH = 14;  // levels enqueued between two looks

// The root and the first C4_TOP levels.
__global__ __launch_bounds__(1024) void k_collapse_top(const float* __restrict__ nodes_f,
                                                       uint32_t* __restrict__ q0,
                                                       uint32_t* __restrict__ q1,
                                                       uint32_t* __restrict__ cnt,
                                                       float4* __restrict__ sparse4,
                                                       uint32_t* __restrict__ is4, int leaf_max) {
  for (int l = threadIdx.x; l <= C4_LEVELS; l += 1024) cnt[l] = l == 0 ? 1u : 0u;
  if (threadIdx.x == 0) q0[0] = 0u;  // the root is the one item of level 0
  __threadfence();
  __syncthreads();
  for (int l = 0; l < C4_TOP; ++l) {
    const uint32_t n = __hip_atomic_load(cnt + l, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const uint32_t* q = l & 1 ? q1 : q0;
    for (uint32_t i = threadIdx.x; i < n; i += 1024)
      collapse_node(nodes_f, __hip_atomic_load(q + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT),
                    l & 1 ? q0 : q1, cnt + l + 1, sparse4, is4, leaf_max);
    __threadfence();
    __syncthreads();
  }
}

__global__ __launch_bounds__(256) void k_collapse(const float* __restrict__ nodes_f,
                                                  const uint32_t* __restrict__ q_in,
                                                  const uint32_t* __restrict__ cnt,
                                                  uint32_t* __restrict__ q_out,
                                                  uint32_t* __restrict__ cnt_out,
                                                  float4* __restrict__ sparse4,
                                                  uint32_t* __restrict__ is4, int leaf_max) {
  const uint32_t n = *cnt;
  for (uint32_t i = blockIdx.x * 256 + threadIdx.x; i < n; i += gridDim.x * 256)
    collapse_node(nodes_f, q_in[i], q_out, cnt_out, sparse4, is4, leaf_max);
}

// Dense numbering of the BVH4 nodes in binary-node order: nodes per block of 1024
// binary nodes, then each node's number (the counts before its block are summed).
__global__ __launch_bounds__(1024) void k_count4(const uint32_t* __restrict__ is4, int nint,
                                                 uint32_t* __restrict__ bcount) {
  __shared__ uint32_t wc[16];
  const int b = blockIdx.x * 1024 + threadIdx.x;
  const uint64_t m = __ballot(b < nint && is4[b]);
  if ((threadIdx.x & 63) == 0) wc[threadIdx.x >> 6] = (uint32_t)__popcll(m);
  __syncthreads();
  if (threadIdx.x == 0) {
    uint32_t s = 0;
    for (int w = 0; w < 16; ++w) s += wc[w];
    bcount[blockIdx.x] = s;
  }
}

__global__ __launch_bounds__(256) void k_number4(const uint32_t* __restrict__ is4, int nint,
                                                 const uint32_t* __restrict__ bcount,
                                                 uint32_t* __restrict__ idx,
                                                 uint32_t* __restrict__ count4) {
  __shared__ uint32_t sh[4];
  uint32_t base = block_sum(bcount, blockIdx.x, sh);
  for (int q = 0; q < 4; ++q) {
    const int b = blockIdx.x * 1024 + q * 256 + threadIdx.x;
    const uint32_t k = b < nint && is4[b] ? 1u : 0u;
    uint32_t total;
    const uint32_t incl = block_scan256(k, sh, &total);
    if (b < nint) idx[b] = base + incl - k;
    base += total;
  }
  if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) *count4 = base;
}

// Dense renumbering (binary-node order): node b moves to idx[b]; internal
// references are renumbered the same way.
__global__ __launch_bounds__(256) void k_compact4(const float4* __restrict__ sparse4,
                                                  const uint32_t* __restrict__ is4,
                                                  const uint32_t* __restrict__ idx, int nint,
                                                  float4* __restrict__ dense4) {
  const int b = blockIdx.x * 256 + threadIdx.x;
  if (b >= nint || !is4[b]) return;
  const float4* src = sparse4 + 8 * (size_t)b;
  float4* dst = dense4 + 8 * (size_t)idx[b];
  for (int a = 0; a < 6; ++a) dst[a] = src[a];
  const float4 r = src[6];
  uint32_t refs[4] = {__float_as_uint(r.x), __float_as_uint(r.y), __float_as_uint(r.z),
                      __float_as_uint(r.w)};
  for (int k = 0; k < 4; ++k)
    if (refs[k] != EMPTY4 && !(refs[k] & LEAF_BIT)) refs[k] = idx[refs[k]];
  dst[6] = make_float4(__uint_as_float(refs[0]), __uint_as_float(refs[1]),
                       __uint_as_float(refs[2]), __uint_as_float(refs[3]));
  dst[7] = src[7];
}

// Quantized copy of a BVH4 node (64 bytes, 4 float4): the node's box origin p
// (minus a margin) and per-axis power-of-two steps s = 2^e, then each child's
// box as 8-bit steps from p, rounded outward, and the child references:
//   [0] p.x, p.y, p.z, bits(biased e_x | e_y << 8 | e_z << 16)
//   [1] lo_x, lo_y, lo_z, hi_x  (one byte per child: byte c = child c)
//   [2] hi_y, hi_z, 0, 0
//   [3] child references (as in the full node)
// Every quantized child box contains the exact one with a margin of at least
// m = 2^-18 max(|node coordinates|, |scene coordinates|) on every side, so the
// traversal's FP32 rounding never culls a box the full node would keep.
__global__ __launch_bounds__(256) void k_quantize4(const float4* __restrict__ nodes4, int count,
                                                   float4* __restrict__ q4) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i >= count) return;
  const float4* nd = nodes4 + 8 * (size_t)i;
  const float4* root = nodes4;
  const float4 rf = nd[6];
  const uint32_t ref[4] = {__float_as_uint(rf.x), __float_as_uint(rf.y), __float_as_uint(rf.z),
                           __float_as_uint(rf.w)};
  auto comp = [](const float4& v, int c) { return c == 0 ? v.x : c == 1 ? v.y : c == 2 ? v.z : v.w; };
  double scene = 0.0;  // largest coordinate magnitude of the scene (the root's child boxes)
  {
    const uint32_t rr[4] = {__float_as_uint(root[6].x), __float_as_uint(root[6].y),
                            __float_as_uint(root[6].z), __float_as_uint(root[6].w)};
    for (int c = 0; c < 4; ++c)
      if (rr[c] != EMPTY4)
        for (int a = 0; a < 6; ++a) scene = fmax(scene, fabs((double)comp(root[a], c)));
  }
  float P[3];
  uint32_t E = 0, qlo[3] = {0u, 0u, 0u}, qhi[3] = {0u, 0u, 0u};
  for (int a = 0; a < 3; ++a) {
    double lo = INFINITY, hi = -INFINITY, mag = scene;
    for (int c = 0; c < 4; ++c) {
      if (ref[c] == EMPTY4) continue;
      const double l = comp(nd[a], c), h = comp(nd[3 + a], c);
      lo = fmin(lo, l);
      hi = fmax(hi, h);
      mag = fmax(mag, fmax(fabs(l), fabs(h)));
    }
    if (!(lo <= hi)) lo = hi = 0.0;  // no child (cannot happen in a built tree)
    const double m = ldexp(fmax(mag, 1e-30), -18);
    // origin: an FP32 value at or below lo - m
    float p = (float)(lo - m);
    if ((double)p > lo - m) p = nextafterf(p, -INFINITY);
    // step: the smallest power of two with 255 steps covering [p, hi + m]
    const double need = (hi + m - (double)p) / 255.0;
    int e;
    (void)frexp(fmax(need, 1e-37), &e);  // need <= 2^e
    e = max(-126, min(127, e));
    const double sc = ldexp(1.0, e);
    P[a] = p;
    E |= (uint32_t)(e + 127) << (8 * a);
    for (int c = 0; c < 4; ++c) {
      uint32_t ql = 0u, qh = 0u;
      if (ref[c] != EMPTY4) {
        const double l = comp(nd[a], c) - m, h = comp(nd[3 + a], c) + m;
        int lq = (int)floor((l - (double)p) / sc), hq = (int)ceil((h - (double)p) / sc);
        lq = max(0, min(255, lq));
        hq = max(0, min(255, hq));
        while (lq > 0 && (double)p + lq * sc > l) --lq;   // exact in FP64
        while (hq < 255 && (double)p + hq * sc < h) ++hq;
        ql = (uint32_t)lq;
        qh = (uint32_t)hq;
      }
      qlo[a] |= ql << (8 * c);
      qhi[a] |= qh << (8 * c);
    }
  }
  float4* o = q4 + 4 * (size_t)i;
  o[0] = make_float4(P[0], P[1], P[2], __uint_as_float(E));
  o[1] = make_float4(__uint_as_float(qlo[0]), __uint_as_float(qlo[1]), __uint_as_float(qlo[2]),
                     __uint_as_float(qhi[0]));
  o[2] = make_float4(__uint_as_float(qhi[1]), __uint_as_float(qhi[2]), 0.0f, 0.0f);
  o[3] = rf;
}

inline int cdiv(long a, long b) { return (int)((a + b - 1) / b); }

// Scratch of the collapse.
struct Collapse4 {
  uint32_t *q[2], *cnt, *is4, *idx, *bcount, *count4;
  float4* sparse4;
};

// Enqueues the collapse's first C4_TOP levels.
void collapse4_begin(const float4* nodes, int n, hipStream_t st, int leaf_max,
                     const Collapse4& c) {
  const int nint = n - 1;
  k_fill_u32<<<cdiv(nint, 256), 256, 0, st>>>(c.is4, nint, 0u);
  k_collapse_top<<<1, 1024, 0, st>>>((const float*)nodes, c.q[0], c.q[1], c.cnt, c.sparse4, c.is4,
                                     leaf_max);
}

// Enqueues levels from .. to - 1, the dense numbering and the node count.
void collapse4_levels(const float4* nodes, int n, hipStream_t st, int leaf_max,
                      const Collapse4& c, int from, int to) {
  const int nint = n - 1;
  const int blocks = std::min(cdiv(nint, 256), 1024);
  for (int l = from; l < to; ++l)
    k_collapse<<<blocks, 256, 0, st>>>((const float*)nodes, c.q[l & 1], c.cnt + l, c.q[~l & 1],
                                       c.cnt + l + 1, c.sparse4, c.is4, leaf_max);
  const int nb = cdiv(nint, 1024);
  k_count4<<<nb, 1024, 0, st>>>(c.is4, nint, c.bcount);
  k_number4<<<nb, 256, 0, st>>>(c.is4, nint, c.bcount, c.idx, c.count4);
}

// Top-down collapse of the binary tree, then dense renumbering.  Synchronises to
// learn the node count (and, for a tree of more than C4_TOP + C4_BATCH levels, whether
// levels are left).
mrs_status collapse4(mrs_scene* s, hipStream_t st, int leaf_max, const Collapse4& c) {
  const int n = s->ntris;
  collapse4_begin(s->d_nodes, n, st, leaf_max, c);
  uint32_t count4 = 0;
  for (int from = C4_TOP;;) {
    const int to = std::min(from + C4_BATCH, C4_LEVELS);
    collapse4_levels(s->d_nodes, n, st, leaf_max, c, from, to);
    MRS_TRY_HIP(hipGetLastError());
    uint32_t left = 0;
    MRS_TRY_HIP(hipMemcpyAsync(&left, c.cnt + to, sizeof left, hipMemcpyDeviceToHost, st));
    MRS_TRY_HIP(hipMemcpyAsync(&count4, c.count4, sizeof count4, hipMemcpyDeviceToHost, st));
    MRS_TRY_HIP(hipStreamSynchronize(st));
    if (!left) break;
    if (to == C4_LEVELS)
      return fail(MRS_ERR_DEVICE, "mrs_build_bvh: BVH4 collapse does not end");
    from = to;
  }
  if (count4 == 0 || count4 > (uint32_t)(n - 1))
    return fail(MRS_ERR_DEVICE, "mrs_build_bvh: BVH4 collapse made no tree");
  // the nodes and their quantized copies in one allocation
  if (s->d_nodes4) (void)hipFree(s->d_nodes4);
  s->d_nodes4 = s->d_nodes4q = nullptr;
  if (hipMalloc(&s->d_nodes4, sizeof(float4) * 12 * (size_t)count4) != hipSuccess) {
    (void)hipGetLastError();
    s->d_nodes4 = nullptr;
    return fail(MRS_ERR_OUT_OF_MEMORY, "mrs_build_bvh: BVH4 allocation failed");
  }
  s->d_nodes4q = s->d_nodes4 + 8 * (size_t)count4;
  k_compact4<<<cdiv(n - 1, 256), 256, 0, st>>>(c.sparse4, c.is4, c.idx, n - 1, s->d_nodes4);
  k_quantize4<<<cdiv(count4, 256), 256, 0, st>>>(s->d_nodes4, (int)count4, s->d_nodes4q);
  MRS_TRY_HIP(hipGetLastError());
  s->count4 = count4;
  s->root4 = 0u;  // binary root 0 is the first BVH4 node
  return MRS_OK;
}

// PLOC over the Morton-sorted primitives (code, prim): binary records into
// s->d_nodes (preorder, root 0), primitives and codes in leaf order into
// s->d_leaf_prim / s->d_morton, leaf records into s->d_leaf_tri.  *used is
// false when the tree would be deeper than the Morton-split tree may be (64
// levels): the caller builds that one instead, which writes all of these again.
struct PlocScratch {
  uint32_t* cref[2];
  float4 *clo[2], *chi[2];
  int* nn;
  uint32_t *keep, *bcount, *mcount, *pre_int, *first_int, *first_leaf, *ctr;
  PlocTree tree;
};

mrs_status ploc_build(mrs_scene* s, hipStream_t st, const uint32_t* code, const uint32_t* prim,
                      const PlocScratch& c, bool* used) {
  *used = false;
  const int n = s->ntris, nint = n - 1;
  const int nb = cdiv(n, 256);
  k_ploc_init<<<nb, 256, 0, st>>>(s->d_tri_src, prim, n, c.cref[0], c.clo[0], c.chi[0], c.mcount,
                                  c.ctr);
  // mcount[r]: clusters before round r.  The host looks at the counts every
  // PLOC_BATCH rounds; between two looks the launches are sized by the last one
  // seen and take the count from the device.
  int round = 0;
  uint32_t m = (uint32_t)n;
  while (m > (uint32_t)PLOC_SMALL) {
    // a healthy build takes 50-70 rounds; this many means chains (deep trees)
    if (round >= PLOC_MAX_ROUNDS) return MRS_OK;  // the caller falls back
    const int mb = cdiv(m, 256);
    for (int k = 0; k < PLOC_BATCH; ++k) {
      const int r = round + k, cur = r & 1;
      const uint32_t* mc = c.mcount + r;
      k_ploc_nn<<<mb, 256, 0, st>>>(mc, c.clo[cur], c.chi[cur], c.nn);
      k_ploc_merge<<<mb, 256, 0, st>>>(mc, nint, c.nn, c.cref[cur], c.clo[cur], c.chi[cur],
                                       c.tree, c.ctr, c.keep, c.bcount);
      // few blocks sum the counts before them quickly; many take longer tiles
      if (mb <= 2048)
        k_ploc_scatter<1><<<mb, 256, 0, st>>>(mc, c.keep, c.bcount, c.cref[cur], c.clo[cur],
                                              c.chi[cur], c.cref[1 - cur], c.clo[1 - cur],
                                              c.chi[1 - cur], c.mcount + r + 1);
      else
        k_ploc_scatter<8><<<cdiv(mb, 8), 256, 0, st>>>(
            mc, c.keep, c.bcount, c.cref[cur], c.clo[cur], c.chi[cur], c.cref[1 - cur],
            c.clo[1 - cur], c.chi[1 - cur], c.mcount + r + 1);
    }
    MRS_TRY_HIP(hipGetLastError());
    uint32_t seen[PLOC_BATCH];
    MRS_TRY_HIP(hipMemcpyAsync(seen, c.mcount + round + 1, sizeof seen, hipMemcpyDeviceToHost, st));
    MRS_TRY_HIP(hipStreamSynchronize(st));
    for (int k = 0; k < PLOC_BATCH; ++k) {
      if (m > 1 && (seen[k] >= m || seen[k] == 0))
        return fail(MRS_ERR_DEVICE, "mrs_build_bvh: a clustering round merged nothing");
      m = seen[k];
    }
    round += PLOC_BATCH;
  }
  const int cur = round & 1;
  k_ploc_small<<<1, 1024, 0, st>>>(c.mcount + round, nint, c.cref[cur], c.clo[cur], c.chi[cur],
                                   c.tree, c.ctr, PLOC_MAX_ROUNDS - round);
  k_ploc_order<<<cdiv(nint + n, 256), 256, 0, st>>>(n, nint, c.tree.par_int, c.tree.par_leaf,
                                                    c.tree.sz2, c.pre_int, c.first_int,
                                                    c.first_leaf, c.ctr);
  k_ploc_emit<<<cdiv(nint, 256), 256, 0, st>>>(nint, n, c.tree.tnodes, c.pre_int, c.first_int,
                                               c.first_leaf, c.tree.sz2, c.ctr, (float*)s->d_nodes);
  k_ploc_leaves<<<nb, 256, 0, st>>>(n, s->d_tri_src, prim, code, c.first_leaf, c.ctr,
                                    s->d_leaf_prim, s->d_morton, s->d_leaf_tri);
  MRS_TRY_HIP(hipGetLastError());
  uint32_t h[PLOC_CTR];
  MRS_TRY_HIP(hipMemcpyAsync(h, c.ctr, sizeof h, hipMemcpyDeviceToHost, st));
  MRS_TRY_HIP(hipStreamSynchronize(st));
  if (h[PC_BAD] & BAD_STUCK)
    return fail(MRS_ERR_DEVICE, "mrs_build_bvh: a clustering round merged nothing");
  if (h[PC_BAD]) return fail(MRS_ERR_DEVICE, "mrs_build_bvh: clustered tree is malformed");
  // not done in PLOC_MAX_ROUNDS, or too deep: the caller falls back
  *used = h[PC_DONE] && h[PC_DEPTH] <= (uint32_t)MAX_STACK;
  return MRS_OK;
}

}  // namespace

mrs_status lbvh_build(mrs_scene* s, hipStream_t st, int leaf_max, int builder) {
  const int n = s->ntris;
  s->bvh_built = false;
  s->leaf_max = leaf_max;
  if (n == 0) {
    s->root = 0;
    s->root4 = EMPTY4;
    s->count4 = 0;
    s->bvh_built = true;
    return MRS_OK;
  }
  // scratch: bounds partials, keys/vals ping-pong, counts, parents, visits
  const int nb = std::min(1024, cdiv(n, 256));
  const int rs_blocks = cdiv(n, RS_TILE);
  const size_t count_len = (size_t)256 * rs_blocks;
  size_t bytes = 0;
  auto carve = [&](size_t sz) {
    size_t off = bytes;
    bytes += (sz + 255) & ~(size_t)255;
    return off;
  };
  const bool ploc = builder == MRS_BVH_PLOC && n >= 2;
  const int nint = std::max(n - 1, 1);
  const size_t o_part = carve(sizeof(float) * 6 * nb);
  const size_t o_bounds = carve(sizeof(float) * 6);
  const size_t o_k0 = carve(sizeof(uint32_t) * n);
  const size_t o_v0 = carve(sizeof(uint32_t) * n);
  const size_t o_k1 = carve(sizeof(uint32_t) * n);
  const size_t o_v1 = carve(sizeof(uint32_t) * n);
  const size_t o_cnt = carve(sizeof(uint32_t) * count_len);
  const size_t o_tot = carve(sizeof(uint32_t) * 256);
  const size_t o_pi = carve(sizeof(uint32_t) * n);
  const size_t o_pl = carve(sizeof(uint32_t) * n);
  const size_t o_vis = carve(sizeof(uint32_t) * n);
  const size_t o_q0 = carve(sizeof(uint32_t) * n);
  const size_t o_q1 = carve(sizeof(uint32_t) * n);
  const size_t o_qc = carve(sizeof(uint32_t) * (C4_LEVELS + 2));
  const size_t o_is4 = carve(sizeof(uint32_t) * n);
  const size_t o_idx = carve(sizeof(uint32_t) * n);
  const size_t o_bc4 = carve(sizeof(uint32_t) * cdiv(n, 1024));
  const size_t o_sp4 = carve(sizeof(float4) * 8 * (size_t)nint);
  // clustering; its arrays end before the collapse starts, but a fallback needs
  // the sorted keys and the collapse's scratch again
  size_t o_ref[2] = {0, 0}, o_lo[2] = {0, 0}, o_hi[2] = {0, 0};
  size_t o_nn = 0, o_keep = 0, o_bc = 0, o_mc = 0, o_pre = 0, o_fi = 0, o_fl = 0, o_ctr = 0,
         o_tn = 0, o_sz = 0;
  if (ploc) {
    for (int b = 0; b < 2; ++b) {
      o_ref[b] = carve(sizeof(uint32_t) * n);
      o_lo[b] = carve(sizeof(float4) * n);
      o_hi[b] = carve(sizeof(float4) * n);
    }
    o_nn = carve(sizeof(int) * n);
    o_keep = carve(sizeof(uint32_t) * n);
    o_bc = carve(sizeof(uint32_t) * cdiv(n, 256));
    o_mc = carve(sizeof(uint32_t) * (PLOC_MAX_ROUNDS + PLOC_BATCH + 1));
    o_pre = carve(sizeof(uint32_t) * nint);
    o_fi = carve(sizeof(uint32_t) * nint);
    o_fl = carve(sizeof(uint32_t) * n);
    o_ctr = carve(sizeof(uint32_t) * PLOC_CTR);
    o_tn = carve(sizeof(float4) * 4 * (size_t)nint);
    o_sz = carve(sizeof(uint32_t) * 2 * (size_t)nint);
  }
  char* scratch = nullptr;
  if (hipMalloc(&scratch, bytes) != hipSuccess) {
    (void)hipGetLastError();
    return fail(MRS_ERR_OUT_OF_MEMORY, "mrs_build_bvh: scratch allocation failed");
  }
  float* part = (float*)(scratch + o_part);
  float* bounds = (float*)(scratch + o_bounds);
  uint32_t* k0 = (uint32_t*)(scratch + o_k0);
  uint32_t* v0 = (uint32_t*)(scratch + o_v0);
  uint32_t* k1 = (uint32_t*)(scratch + o_k1);
  uint32_t* v1 = (uint32_t*)(scratch + o_v1);
  uint32_t* counts = (uint32_t*)(scratch + o_cnt);
  uint32_t* totals = (uint32_t*)(scratch + o_tot);
  uint32_t* pint = (uint32_t*)(scratch + o_pi);
  uint32_t* pleaf = (uint32_t*)(scratch + o_pl);
  uint32_t* visits = (uint32_t*)(scratch + o_vis);

  k_bounds_partial<<<nb, 256, 0, st>>>(s->d_tri_src, n, part);
  k_bounds_final<<<1, 384, 0, st>>>(part, nb, bounds);
  k_morton<<<cdiv(n, 256), 256, 0, st>>>(s->d_tri_src, n, bounds, k0, v0);
  for (int shift = 0; shift < 32; shift += 8) {
    k_rs_hist<<<rs_blocks, RS_THREADS, 0, st>>>(k0, n, shift, rs_blocks, counts);
    k_rs_rows<<<256, RS_THREADS, 0, st>>>(counts, rs_blocks, totals);
    k_rs_scatter<<<rs_blocks, RS_THREADS, 0, st>>>(k0, v0, n, shift, rs_blocks, counts, totals, k1,
                                                   v1);
    std::swap(k0, k1);
    std::swap(v0, v1);
  }
  // 4 passes: the sorted data is back in the first buffers (k0/v0 after swaps)
  bool clustered = false;
  mrs_status rc = MRS_OK;
  if (ploc) {
    PlocScratch c;
    for (int b = 0; b < 2; ++b) {
      c.cref[b] = (uint32_t*)(scratch + o_ref[b]);
      c.clo[b] = (float4*)(scratch + o_lo[b]);
      c.chi[b] = (float4*)(scratch + o_hi[b]);
    }
    c.nn = (int*)(scratch + o_nn);
    c.keep = (uint32_t*)(scratch + o_keep);
    c.bcount = (uint32_t*)(scratch + o_bc);
    c.mcount = (uint32_t*)(scratch + o_mc);
    c.pre_int = (uint32_t*)(scratch + o_pre);
    c.first_int = (uint32_t*)(scratch + o_fi);
    c.first_leaf = (uint32_t*)(scratch + o_fl);
    c.ctr = (uint32_t*)(scratch + o_ctr);
    c.tree.tnodes = (float*)(scratch + o_tn);
    c.tree.par_int = pint;
    c.tree.par_leaf = pleaf;
    c.tree.sz2 = (uint32_t*)(scratch + o_sz);
    rc = ploc_build(s, st, k0, v0, c, &clustered);
    if (rc != MRS_OK) {
      (void)hipStreamSynchronize(st);
      (void)hipFree(scratch);
      return rc;
    }
  }
  if (!clustered) {
    MRS_TRY_HIP(
        hipMemcpyAsync(s->d_morton, k0, sizeof(uint32_t) * n, hipMemcpyDeviceToDevice, st));
    MRS_TRY_HIP(
        hipMemcpyAsync(s->d_leaf_prim, v0, sizeof(uint32_t) * n, hipMemcpyDeviceToDevice, st));
    if (n >= 2) {
      k_hierarchy<<<cdiv(n - 1, 256), 256, 0, st>>>(s->d_morton, s->d_leaf_prim, n, s->d_nodes,
                                                    pint, pleaf);
      k_fill_u32<<<cdiv(n, 256), 256, 0, st>>>(visits, n, 0u);
    }
    k_leaves_refit<<<cdiv(n, 256), 256, 0, st>>>(s->d_tri_src, s->d_leaf_prim, n, s->d_leaf_tri,
                                                 (float*)s->d_nodes, pint, pleaf, visits);
    MRS_TRY_HIP(hipGetLastError());
  }
  s->builder = clustered ? MRS_BVH_PLOC : MRS_BVH_LBVH;
  if (n >= 2) {
    Collapse4 c;
    c.q[0] = (uint32_t*)(scratch + o_q0);
    c.q[1] = (uint32_t*)(scratch + o_q1);
    c.cnt = (uint32_t*)(scratch + o_qc);
    c.count4 = c.cnt + C4_LEVELS + 1;
    c.is4 = (uint32_t*)(scratch + o_is4);
    c.idx = (uint32_t*)(scratch + o_idx);
    c.bcount = (uint32_t*)(scratch + o_bc4);
    c.sparse4 = (float4*)(scratch + o_sp4);
    rc = collapse4(s, st, leaf_max, c);
  }
  // The scratch must outlive the kernels: wait, then free.
  MRS_TRY_HIP(hipStreamSynchronize(st));
  MRS_TRY_HIP(hipFree(scratch));
  if (rc != MRS_OK) return rc;
  s->root = n >= 2 ? 0u : LEAF_BIT;
  if (n < 2) {
    s->root4 = leaf4_ref(0, 1);
    s->count4 = 0;
  }
  s->bvh_built = true;
  return MRS_OK;
}

}  // namespace mrs
