// bvh_gpu.hip -- linear BVH on the GPU: Morton codes of the triangle
// centroids, a radix sort, the binary radix tree of Karras ("Maximizing
// parallelism in the construction of BVHs, octrees, and k-d trees", HPG
// 2012), and a collapse of every other level into the four-wide quantised
// nodes the traversal kernels read.  Every inner node covers a contiguous
// range of the sorted triangles, so a subtree of at most max_leaf triangles
// becomes one leaf without copying, and a node's box is a range query over
// the sorted triangles' boxes (an implicit binary tree over the positions,
// three launches to fill for two million triangles).  A refit keeps the tree
// and recomputes triangles, normals, boxes and node frames from moved
// vertices; a four-wide tree built on the host is refitted one launch per
// depth of its nodes.
//
// Every kernel here moves a few hundred megabytes at most, so what bounded
// them was elsewhere: same-address atomics (one per wave and counter: 62,000
// at about 10 ns each), 33 launches for the boxes, float64 divisions and
// dynamically indexed arrays in the node frames.  On two million triangles:
// k_prep 730 -> 65 us, k_heads 723 -> 50, boxes 345 -> 40, k_emit 413 -> 90;
// a refit's normals and leaves 175 -> 75, its k_emit 251 -> 91.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>

#include <rocprim/device/device_radix_sort.hpp>
#include <rocprim/device/device_scan.hpp>

#include "bvh_gpu.h"

#pragma clang fp contract(off)

namespace rr {

namespace {

constexpr int kB = 256;
// misc words: [0..2] centroid minimum and [3..5] maximum (order-preserving
// encodings), [6] largest coordinate magnitude (float bits, >= 1), [7]
// hittable triangles, [8] four-wide nodes, [9] leaves, [10] deepest
// four-wide node
constexpr int kMiscWords = 16;

__device__ __forceinline__ uint32_t fenc(float f) {
  const uint32_t b = __float_as_uint(f);
  return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}
__device__ __forceinline__ float fdec(uint32_t u) {
  return __uint_as_float((u & 0x80000000u) ? (u & 0x7fffffffu) : ~u);
}

// triangle j: vertices, edges, geometric normal (the host build's float32
// operations, so normals match bit for bit); nn > 0 marks a hittable one
struct Tri {
  float p0[3], p1[3], p2[3], e1[3], e2[3], n[3], nn;
};
__device__ __forceinline__ void load_tri(const GpuBvh& g, uint32_t j, Tri& t) {
  const float* a = g.V + 3u * g.F[3u * j + 0u];
  const float* b = g.V + 3u * g.F[3u * j + 1u];
  const float* c = g.V + 3u * g.F[3u * j + 2u];
  for (int k = 0; k < 3; ++k) {
    t.p0[k] = a[k];
    t.p1[k] = b[k];
    t.p2[k] = c[k];
    t.e1[k] = t.p1[k] - t.p0[k];
    t.e2[k] = t.p2[k] - t.p0[k];
  }
  t.n[0] = t.e1[1] * t.e2[2] - t.e1[2] * t.e2[1];
  t.n[1] = t.e1[2] * t.e2[0] - t.e1[0] * t.e2[2];
  t.n[2] = t.e1[0] * t.e2[1] - t.e1[1] * t.e2[0];
  t.nn = dot3(t.n[0], t.n[1], t.n[2], t.n[0], t.n[1], t.n[2]);
}

__device__ __forceinline__ void tri_box(const Tri& t, float lo[3], float hi[3]) {
  for (int k = 0; k < 3; ++k) {
    lo[k] = fminf(fminf(t.p0[k], t.p1[k]), t.p2[k]);
    hi[k] = fmaxf(fmaxf(t.p0[k], t.p1[k]), t.p2[k]);
  }
}

__device__ __forceinline__ float4 aux_of(const GpuBvh& g, uint32_t j, const Tri& t) {
  if (!(t.nn > 0.0f)) return make_float4(0.0f, 0.0f, 0.0f, 0.0f);
  const float len = sqrtf(t.nn);
  return make_float4(t.n[0] / len, t.n[1] / len, t.n[2] / len, __uint_as_float((uint32_t)g.M[j]));
}

// leaf record of triangle `orig`: first vertex and id, the two edges.  A
// triangle that a refit made degenerate keeps zero edges, so the ray test's
// determinant is exactly zero and it is never hit (a build leaves it out).
__device__ __forceinline__ void store_tri(float4* rec, uint32_t orig, const Tri& t) {
  const float k = t.nn > 0.0f ? 1.0f : 0.0f;
  rec[0] = make_float4(t.p0[0], t.p0[1], t.p0[2], __uint_as_float(orig));
  rec[1] = make_float4(k * t.e1[0], k * t.e1[1], k * t.e1[2], 0.0f);
  rec[2] = make_float4(k * t.e2[0], k * t.e2[1], k * t.e2[2], 0.0f);
}

__global__ void k_init_misc(uint32_t* misc, bool refit) {
  const uint32_t i = threadIdx.x;
  if (i >= (uint32_t)kMiscWords) return;
  if (refit) {
    if (i == 6) misc[i] = __float_as_uint(1.0f);
    return;
  }
  misc[i] = i < 3 ? 0xffffffffu : (i == 6 ? __float_as_uint(1.0f) : 0u);
}

// Kernels that end in one atomic per block and scalar use large blocks, so
// that 512 of them fill the chip: same-address atomics take about 10 ns each.
constexpr int kBig = 1024;

// Combines one value per lane over the block (kLanes lanes) with `op`; the
// result is valid in thread 0.  `buf` holds one word per wave.
template <int kLanes = kBig, class Op>
__device__ __forceinline__ uint32_t block_reduce(uint32_t v, uint32_t* buf, Op op) {
  for (int d = 32; d >= 1; d >>= 1) v = op(v, (uint32_t)__shfl_xor((int)v, d));
  __syncthreads();
  if ((threadIdx.x & 63u) == 0) buf[threadIdx.x >> 6] = v;
  __syncthreads();
  if (threadIdx.x == 0)
    for (int w = 1; w < kLanes / 64; ++w) v = op(v, buf[w]);
  return v;
}
__device__ __forceinline__ uint32_t op_min(uint32_t a, uint32_t b) { return a < b ? a : b; }
__device__ __forceinline__ uint32_t op_max(uint32_t a, uint32_t b) { return a > b ? a : b; }
__device__ __forceinline__ uint32_t op_add(uint32_t a, uint32_t b) { return a + b; }

__device__ __forceinline__ float tri_magnitude(const float lo[3], const float hi[3], float mag) {
  for (int k = 0; k < 3; ++k) mag = fmaxf(mag, fmaxf(fabsf(lo[k]), fabsf(hi[k])));
  return mag;
}

// Build, per triangle: normal record, hittable count, centroid (into `cen`),
// centroid bounds and the largest coordinate magnitude.  Each lane keeps its
// own bounds over its triangles; one atomic per block and scalar at the end.
__global__ void __launch_bounds__(kBig) k_prep(GpuBvh g, float4* aux, float4* cen) {
  __shared__ uint32_t buf[kBig / 64];
  uint32_t blo[3] = {0xffffffffu, 0xffffffffu, 0xffffffffu}, bhi[3] = {0u, 0u, 0u}, cnt = 0;
  float mag = 1.0f;
  for (uint32_t j = blockIdx.x * kBig + threadIdx.x; j < g.nt; j += gridDim.x * kBig) {
    Tri t;
    load_tri(g, j, t);
    aux[j] = aux_of(g, j, t);
    if (t.nn > 0.0f) {
      float lo[3], hi[3], c[3];
      tri_box(t, lo, hi);
      mag = tri_magnitude(lo, hi, mag);
      for (int k = 0; k < 3; ++k) {
        c[k] = 0.5f * (lo[k] + hi[k]);
        blo[k] = op_min(blo[k], fenc(c[k]));
        bhi[k] = op_max(bhi[k], fenc(c[k]));
      }
      cen[j] = make_float4(c[0], c[1], c[2], 1.0f);
      ++cnt;
    } else {
      cen[j] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    }
  }
  for (int k = 0; k < 3; ++k) {
    const uint32_t lo = block_reduce(blo[k], buf, op_min), hi = block_reduce(bhi[k], buf, op_max);
    if (threadIdx.x == 0) {
      atomicMin(g.misc + k, lo);
      atomicMax(g.misc + 3 + k, hi);
    }
  }
  // positive floats order as their bits
  const uint32_t m = block_reduce(__float_as_uint(mag), buf, op_max), n = block_reduce(cnt, buf, op_add);
  if (threadIdx.x == 0) {
    atomicMax(g.misc + 6, m);
    atomicAdd(g.misc + 7, n);
  }
}

// Refit of a host-built tree, per triangle: normal record and the largest
// coordinate magnitude.
__global__ void __launch_bounds__(kBig) k_normals(GpuBvh g, float4* aux) {
  __shared__ uint32_t buf[kBig / 64];
  float mag = 1.0f;
  for (uint32_t j = blockIdx.x * kBig + threadIdx.x; j < g.nt; j += gridDim.x * kBig) {
    Tri t;
    load_tri(g, j, t);
    aux[j] = aux_of(g, j, t);
    if (t.nn > 0.0f) {
      float lo[3], hi[3];
      tri_box(t, lo, hi);
      mag = tri_magnitude(lo, hi, mag);
    }
  }
  const uint32_t m = block_reduce(__float_as_uint(mag), buf, op_max);
  if (threadIdx.x == 0) atomicMax(g.misc + 6, m);
}

__device__ __forceinline__ uint32_t spread10(uint32_t x) {
  x = (x * 0x00010001u) & 0xFF0000FFu;
  x = (x * 0x00000101u) & 0x0F00F00Fu;
  x = (x * 0x00000011u) & 0xC30C30C3u;
  x = (x * 0x00000005u) & 0x49249249u;
  return x;
}

// 30-bit Morton key of the centroid in the centroid bounds; unhittable
// triangles get a key above every valid one and sort last
__global__ void __launch_bounds__(kB) k_morton(GpuBvh g, const float4* cen) {
  const uint32_t j = blockIdx.x * kB + threadIdx.x;
  if (j >= g.nt) return;
  const float4 c = cen[j];
  uint32_t key = 0xffffffffu;
  if (c.w > 0.0f) {
    const float cc[3] = {c.x, c.y, c.z};
    uint32_t q[3];
    for (int k = 0; k < 3; ++k) {
      const float lo = fdec(g.misc[k]), hi = fdec(g.misc[3 + k]);
      const float ext = hi - lo;
      float u = ext > 0.0f ? (cc[k] - lo) / ext * 1024.0f : 0.0f;
      u = fminf(fmaxf(u, 0.0f), 1023.0f);
      q[k] = (uint32_t)u;
    }
    key = (spread10(q[0]) << 2) | (spread10(q[1]) << 1) | spread10(q[2]);
  }
  g.keys[j] = key;
  g.ids[j] = j;
}

// common-prefix length of sorted keys a and b (index bits break ties)
__device__ __forceinline__ int delta(const uint32_t* key, int m, int a, int b) {
  if (b < 0 || b >= m) return -1;
  const uint32_t ka = key[a], kb = key[b];
  if (ka == kb) return 32 + __clz((uint32_t)(a ^ b));
  return __clz(ka ^ kb);
}

// inner node i of the binary radix tree: its key range and split
__global__ void __launch_bounds__(kB) k_internal(GpuBvh g) {
  const int m = (int)g.misc[7];
  const int i = (int)(blockIdx.x * kB + threadIdx.x);
  if (i >= m - 1) return;
  const uint32_t* key = g.keys + g.nt;  // sorted keys
  const int d = (delta(key, m, i, i + 1) - delta(key, m, i, i - 1)) >= 0 ? 1 : -1;
  const int dmin = delta(key, m, i, i - d);
  int lmax = 2;
  while (delta(key, m, i, i + lmax * d) > dmin) lmax *= 2;
  int l = 0;
  for (int t = lmax / 2; t >= 1; t /= 2)
    if (delta(key, m, i, i + (l + t) * d) > dmin) l += t;
  const int j = i + l * d;
  const int dnode = delta(key, m, i, j);
  int s = 0;
  for (int t = (l + 1) / 2; t >= 1; t = t == 1 ? 0 : (t + 1) / 2)
    if (delta(key, m, i, i + (s + t) * d) > dnode) s += t;
  const int split = i + s * d + (d < 0 ? -1 : 0);
  const int first = min(i, j), last = max(i, j);
  const int left = first == split ? ~split : split;
  const int right = last == split + 1 ? ~(split + 1) : split + 1;
  g.child[2 * i + 0] = left;
  g.child[2 * i + 1] = right;
  g.range[2 * i + 0] = (uint32_t)first;
  g.range[2 * i + 1] = (uint32_t)last;
  g.parent[left >= 0 ? left : (m - 1) + ~left] = i;
  g.parent[right >= 0 ? right : (m - 1) + ~right] = i;
  if (i == 0) g.parent[0] = -1;
}

// Per sorted position: the leaf-order triangle and its box.  kRefit: also the
// normal record of the position's triangle (unhittable ones, sorted last,
// have no leaf) and the largest coordinate magnitude, so that a refit reads
// the moved vertices once.
template <bool kRefit>
__global__ void __launch_bounds__(kBig) k_leaves(GpuBvh g, float4* tris, float4* aux) {
  __shared__ uint32_t buf[kBig / 64];
  const uint32_t m = g.misc[7], n = kRefit ? g.nt : m;
  float mag = 1.0f;
  for (uint32_t p = blockIdx.x * kBig + threadIdx.x; p < n; p += gridDim.x * kBig) {
    const uint32_t orig = g.sorted[p];
    Tri t;
    load_tri(g, orig, t);
    float lo[3], hi[3];
    tri_box(t, lo, hi);
    if (kRefit) {
      aux[orig] = aux_of(g, orig, t);
      if (t.nn > 0.0f) mag = tri_magnitude(lo, hi, mag);
    }
    if (p < m) {
      store_tri(tris + 3 * (size_t)p, orig, t);
      float* b = g.box + 6 * (size_t)(m - 1u + p);
      for (int k = 0; k < 3; ++k) {
        b[k] = lo[k];
        b[3 + k] = hi[k];
      }
    }
  }
  if (kRefit) {
    const uint32_t top = block_reduce(__float_as_uint(mag), buf, op_max);
    if (threadIdx.x == 0) atomicMax(g.misc + 6, top);
  }
}

// Boxes over the sorted positions as an implicit binary tree: node t covers
// nodes 2t and 2t + 1, position p is node m + p, node t is slot t - 1 of the
// box array.  One block fills the subtree below root r over kSegLevels levels
// whose deepest one is level `top` of the tree (levels deeper than that are
// positions or filled by the launch before); nodes at m or above are
// positions.
constexpr int kSegLevels = 9;
__global__ void __launch_bounds__(kB) k_seg(GpuBvh g, uint32_t root_level, uint32_t levels) {
  __shared__ float s_box[2][kB][6];
  const uint32_t m = g.misc[7];
  const uint32_t r = (1u << root_level) + blockIdx.x;
  // levels - 1 .. 0 below the root; the deepest one's children are in memory
  for (int h = (int)levels - 1; h >= 0; --h) {
    const uint32_t j = threadIdx.x;
    const uint64_t t = ((uint64_t)r << h) + j;
    const int cur = h & 1;
    if (j < (1u << h) && t < m) {
      float c[2][6];
      for (int k = 0; k < 2; ++k) {
        const uint64_t child = 2 * t + (uint64_t)k;
        const float* b = g.box + 6 * (size_t)(child - 1);
        const bool here = h < (int)levels - 1 && child < m;  // computed by this block's last round
        for (int a = 0; a < 6; ++a) c[k][a] = here ? s_box[cur ^ 1][2 * j + k][a] : b[a];
      }
      float* o = g.box + 6 * (size_t)(t - 1);
      for (int a = 0; a < 6; ++a) {
        const float v = a < 3 ? fminf(c[0][a], c[1][a]) : fmaxf(c[0][a], c[1][a]);
        s_box[cur][j][a] = v;
        o[a] = v;
      }
    }
    __syncthreads();
  }
}

// box of sorted positions first..last
__device__ __forceinline__ void range_box(const GpuBvh& g, uint32_t m, uint32_t first, uint32_t last, float lo[3],
                                          float hi[3]) {
  for (int a = 0; a < 3; ++a) {
    lo[a] = INFINITY;
    hi[a] = -INFINITY;
  }
  auto take = [&](uint64_t t) {
    const float* b = g.box + 6 * (size_t)(t - 1);
    for (int a = 0; a < 3; ++a) {
      lo[a] = fminf(lo[a], b[a]);
      hi[a] = fmaxf(hi[a], b[3 + a]);
    }
  };
  for (uint64_t l = (uint64_t)m + first, r = (uint64_t)m + last + 1u; l < r; l >>= 1, r >>= 1) {
    if (l & 1u) take(l++);
    if (r & 1u) take(--r);
  }
}

// four-wide nodes sit at even binary depths; a subtree of at most max_leaf
// triangles is a leaf and is not opened
__global__ void __launch_bounds__(kBig) k_heads(GpuBvh g) {
  __shared__ uint32_t buf[kBig / 64];
  const int m = (int)g.misc[7];
  uint32_t deepest = 0;
  for (uint32_t i = blockIdx.x * kBig + threadIdx.x; i < g.nt; i += gridDim.x * kBig) {
    uint32_t is_head = 0;
    if ((int)i < m - 1) {
      int depth = 0;
      for (int n = g.parent[i]; n >= 0 && depth < (int)kMaxTreeDepth - 1; n = g.parent[n]) ++depth;
      const uint32_t count = g.range[2 * i + 1] - g.range[2 * i] + 1u;
      is_head = (i == 0 || ((depth & 1) == 0 && count > g.max_leaf)) ? 1u : 0u;
      if (is_head) deepest = op_max(deepest, (uint32_t)depth / 2u);
    }
    g.flag[i] = is_head;
  }
  deepest = block_reduce(deepest, buf, op_max);
  if (threadIdx.x == 0) atomicMax(g.misc + 10, deepest);
}

// node index of each head, and the head of each node
__global__ void __launch_bounds__(kB) k_head_index(GpuBvh g, const uint32_t* scanned) {
  const int m = (int)g.misc[7];
  const int i = (int)(blockIdx.x * kB + threadIdx.x);
  if (i >= m - 1) return;
  const uint32_t node = scanned[i];
  g.head[i] = g.flag[i] ? (int32_t)node : -1;
  if (g.flag[i]) g.order[node] = (uint32_t)i;
  if (i == m - 2) g.misc[8] = node + g.flag[i];
}

// the host build's node frame: origin at the low corner, the smallest power
// of two step with the extent within 255 steps.  With ext = f 2^x, f in
// [1/2, 1), that is 2^(x - 8) when f <= 255 / 256 and 2^(x - 7) otherwise.
__device__ __forceinline__ void quantise_axis(float lo, float hi, float& origin, uint32_t& ebyte) {
  origin = lo;
  const double ext = (double)hi - (double)lo;
  int e = 0;  // a node with no box at all keeps step 1 (see the host build)
  if (ext > 0.0) {
    int x;
    const double f = frexp(ext, &x);
    e = max(f <= 255.0 / 256.0 ? x - 8 : x - 7, -126);
  }
  ebyte = (uint32_t)(e + 127);
}

struct Kid {
  int32_t ref;
  float lo[3], hi[3];
  bool empty;
};

// (steps are powers of two, so dividing by one is an exact scaling)
__device__ __forceinline__ void write_node(Node4* out, const Kid (&kids)[4], float pad) {
  float clo[4][3], chi[4][3];
  float nlo[3] = {INFINITY, INFINITY, INFINITY}, nhi[3] = {-INFINITY, -INFINITY, -INFINITY};
#pragma unroll
  for (int j = 0; j < 4; ++j)
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      clo[j][a] = kids[j].empty ? 0.0f : kids[j].lo[a] - pad;
      chi[j][a] = kids[j].empty ? 0.0f : kids[j].hi[a] + pad;
      if (!kids[j].empty) {
        nlo[a] = fminf(nlo[a], clo[j][a]);
        nhi[a] = fmaxf(nhi[a], chi[j][a]);
      }
    }
#pragma unroll
  for (int a = 0; a < 3; ++a)
    if (!(nlo[a] <= nhi[a])) nlo[a] = nhi[a] = 0.0f;
  float origin[3];
  uint32_t eb[3];
#pragma unroll
  for (int a = 0; a < 3; ++a) quantise_axis(nlo[a], nhi[a], origin[a], eb[a]);
  uint32_t qlo[3] = {0u, 0u, 0u}, qhi[3] = {0u, 0u, 0u};
  int32_t ref[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      const double lo = floor(ldexp((double)clo[j][a] - (double)origin[a], 127 - (int)eb[a]));
      const double hi = ceil(ldexp((double)chi[j][a] - (double)origin[a], 127 - (int)eb[a]));
      const uint32_t ql = (uint32_t)fmin(255.0, fmax(0.0, lo));
      const uint32_t qh = (uint32_t)fmin(255.0, fmax(0.0, hi));
      qlo[a] |= ql << (8 * j);
      qhi[a] |= qh << (8 * j);
    }
    ref[j] = kids[j].ref;
  }
  invert_empty_slots(ref, qlo, qhi);
  Node4 nd;
  pack_node4(nd, origin, eb, qlo, qhi, ref);
  *out = nd;
}

__device__ __forceinline__ bool leaf_sized(const GpuBvh& g, int x) {
  return x < 0 || g.range[2 * x + 1] - g.range[2 * x] + 1u <= g.max_leaf;
}

// child x (an inner node, or ~position) of a four-wide node; none: an empty
// slot.  Returns 1 for a leaf.
__device__ __forceinline__ uint32_t kid_of(const GpuBvh& g, uint32_t m, bool none, int x, Kid& k) {
  k.empty = none;
  k.ref = kEmpty;
  for (int a = 0; a < 3; ++a) k.lo[a] = k.hi[a] = 0.0f;
  if (none) return 0u;
  const uint32_t first = x >= 0 ? g.range[2 * x] : (uint32_t)~x;
  const uint32_t last = x >= 0 ? g.range[2 * x + 1] : (uint32_t)~x;
  const bool leaf = x < 0 || last - first + 1u <= g.max_leaf;
  k.ref = leaf ? leaf_ref_encode(first, last - first + 1u) : g.head[x];
  range_box(g, m, first, last, k.lo, k.hi);
  return leaf ? 1u : 0u;
}

// One four-wide node per head: its two binary children, each opened into its
// own two children unless it is a leaf.  A refit takes the children from the
// node's own references and their ranges of sorted positions from what the
// build left in g.keys: three dependent loads before the boxes instead of
// six (refit of two million triangles, 550,000 nodes, and a scan: 352 -> 337
// us).
template <bool kRefit>
__global__ void __launch_bounds__(kB) k_emit(GpuBvh g, Node4* nodes) {
  __shared__ uint32_t buf[kB / 64];
  const uint32_t m = g.misc[7];
  const float pad = __uint_as_float(g.misc[6]) * (1.0f / 262144.0f);
  uint2* const span = reinterpret_cast<uint2*>(g.keys);
  uint32_t leaves = 0;
  if (m < 2) {
    // the root must be an inner node: at most one triangle hangs below it
    if (blockIdx.x == 0 && threadIdx.x == 0) {
      Kid k[4];
      leaves = kid_of(g, m, m == 0, ~0, k[0]);
      for (int j = 1; j < 4; ++j) kid_of(g, m, true, 0, k[j]);
      write_node(nodes, k, pad);
    }
  } else {
    const uint32_t n = g.misc[8];
    for (uint32_t node = blockIdx.x * kB + threadIdx.x; node < n; node += gridDim.x * kB) {
      Kid k[4];
      if constexpr (kRefit) {
        const int4 w = nodes[node].w3;
        const int32_t ref[4] = {w.x, w.y, w.z, w.w};
        uint2 r[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          if (ref[j] < 0)  // (kEmpty too: its range is not used)
            r[j] = make_uint2(leaf_start(ref[j]), leaf_start(ref[j]) + leaf_count(ref[j]) - 1u);
          else
            r[j] = span[ref[j]];
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          k[j].empty = ref[j] == kEmpty;
          k[j].ref = ref[j];
          for (int a = 0; a < 3; ++a) k[j].lo[a] = k[j].hi[a] = 0.0f;
          if (!k[j].empty) range_box(g, m, r[j].x, r[j].y, k[j].lo, k[j].hi);
        }
      } else {
        const uint32_t i = g.order[node];
        span[node] = make_uint2(g.range[2 * i], g.range[2 * i + 1]);
        const int a = g.child[2 * i], b = g.child[2 * i + 1];
        const bool la = leaf_sized(g, a), lb = leaf_sized(g, b);
        const int a0 = la ? a : g.child[2 * a], a1 = la ? 0 : g.child[2 * a + 1];
        const int b0 = lb ? b : g.child[2 * b], b1 = lb ? 0 : g.child[2 * b + 1];
        // in order, without gaps
        leaves += kid_of(g, m, false, a0, k[0]);
        leaves += kid_of(g, m, false, la ? b0 : a1, k[1]);
        leaves += kid_of(g, m, la && lb, la ? b1 : b0, k[2]);
        leaves += kid_of(g, m, la || lb, b1, k[3]);
      }
      write_node(nodes + node, k, pad);
    }
  }
  if constexpr (!kRefit) {
    leaves = block_reduce<kB>(leaves, buf, op_add);
    if (threadIdx.x == 0) atomicAdd(g.misc + 9, leaves);
  }
}

inline dim3 grid_for(uint32_t n) { return dim3(n ? (n + kB - 1) / kB : 1u); }
// grid of kBig-lane blocks whose lanes take several items each
inline dim3 grid_strided(uint32_t n) { return dim3(std::min(n ? (n + kBig - 1) / kBig : 1u, 512u)); }

}  // namespace

hipError_t gpu_bvh_build(GpuBvh& g, Node4* nodes, float4* tris, float4* aux, hipStream_t st) {
  const uint32_t nt = g.nt;
  hipError_t e;
#define RR_GB(x)                           \
  do {                                     \
    if ((e = (x)) != hipSuccess) return e; \
  } while (0)
  hipLaunchKernelGGL(k_init_misc, dim3(1), dim3(64), 0, st, g.misc, false);
  RR_GB(hipGetLastError());
  float4* cen = reinterpret_cast<float4*>(g.box);  // scratch until the boxes are formed
  hipLaunchKernelGGL(k_prep, grid_strided(nt), dim3(kBig), 0, st, g, aux, cen);
  RR_GB(hipGetLastError());
  hipLaunchKernelGGL(k_morton, grid_for(nt), dim3(kB), 0, st, g, cen);
  RR_GB(hipGetLastError());
  size_t bytes = g.temp_bytes;
  RR_GB(rocprim::radix_sort_pairs(g.temp, bytes, g.keys, g.keys + nt, g.ids, g.sorted, nt, 0u, 32u, st));
  hipLaunchKernelGGL(k_internal, grid_for(nt), dim3(kB), 0, st, g);
  RR_GB(hipGetLastError());
  hipLaunchKernelGGL(k_heads, grid_strided(nt), dim3(kBig), 0, st, g);
  RR_GB(hipGetLastError());
  // node index of each head: exclusive scan of the head flags into the
  // first half of the key array (free after the sort)
  bytes = g.temp_bytes;
  RR_GB(rocprim::exclusive_scan(g.temp, bytes, g.flag, g.keys, 0u, (size_t)nt, rocprim::plus<uint32_t>(), st));
  hipLaunchKernelGGL(k_head_index, grid_for(nt), dim3(kB), 0, st, g, g.keys);
  RR_GB(hipGetLastError());
  uint32_t h[kMiscWords];
  RR_GB(hipMemcpyAsync(h, g.misc, sizeof h, hipMemcpyDeviceToHost, st));
  RR_GB(hipStreamSynchronize(st));
  g.m = h[7];
  RR_GB(gpu_bvh_refit(g, nodes, tris, aux, st, false));
  RR_GB(hipMemcpyAsync(h, g.misc, sizeof h, hipMemcpyDeviceToHost, st));
  RR_GB(hipStreamSynchronize(st));
  g.n_nodes = g.m >= 2 ? h[8] : 1u;
  g.n_leaves = h[9];
  g.max_depth = g.m >= 2 ? h[10] : 0u;
  // a node pushes at most three of its children; the path to the deepest
  // node has max_depth + 1 nodes
  g.max_stack = 3u * (g.max_depth + 1u);
  g.pad = __builtin_bit_cast(float, h[6]) * (1.0f / 262144.0f);
  return hipSuccess;
}

hipError_t gpu_bvh_refit(const GpuBvh& g, Node4* nodes, float4* tris, float4* aux, hipStream_t st, bool refit) {
  hipError_t e;
  if (refit) {
    hipLaunchKernelGGL(k_init_misc, dim3(1), dim3(64), 0, st, g.misc, true);
    RR_GB(hipGetLastError());
    hipLaunchKernelGGL(k_leaves<true>, grid_strided(g.nt), dim3(kBig), 0, st, g, tris, aux);
  } else {
    hipLaunchKernelGGL(k_leaves<false>, grid_strided(g.m), dim3(kBig), 0, st, g, tris, aux);
  }
  RR_GB(hipGetLastError());
  if (g.m >= 2) {
    // inner nodes 1 .. m - 1: levels floor(log2(m - 1)) .. 0, kSegLevels a launch
    for (int deep = 31 - __builtin_clz(g.m - 1u); deep >= 0;) {
      const int root = std::max(deep - kSegLevels + 1, 0);
      hipLaunchKernelGGL(k_seg, dim3(1u << root), dim3(kB), 0, st, g, (uint32_t)root, (uint32_t)(deep - root + 1));
      RR_GB(hipGetLastError());
      deep = root - 1;
    }
  }
  const dim3 grid(std::min(grid_for(refit ? g.n_nodes : g.m).x, 2048u));
  if (refit)
    hipLaunchKernelGGL(k_emit<true>, grid, dim3(kB), 0, st, g, nodes);
  else
    hipLaunchKernelGGL(k_emit<false>, grid, dim3(kB), 0, st, g, nodes);
  RR_GB(hipGetLastError());
#undef RR_GB
  return hipSuccess;
}

// ---------------------------------------------------------------- refit of a host-built tree
namespace {

// leaf-order triangle li: vertex and edges from the moved vertices of its
// original triangle (the original id stays in the first word's w)
__global__ void __launch_bounds__(kB) k_hr_tris(GpuBvh g, float4* tris, uint32_t n) {
  const uint32_t li = blockIdx.x * kB + threadIdx.x;
  if (li >= n) return;
  const uint32_t orig = __float_as_uint(tris[3u * li].w);
  if (orig >= g.nt) return;
  Tri t;
  load_tri(g, orig, t);
  store_tri(tris + 3u * li, orig, t);
}

// the nodes of one depth: child boxes (inner children from the deeper level
// just refitted, leaves from their triangles), the quantised node and its
// own box for its parent.  All four slots are rewritten; a slot without a
// child gets the inverted box, as in the builds, so a refit with unmoved
// vertices rewrites every byte as built.
__global__ void __launch_bounds__(kB) k_hr_level(GpuBvh g, Node4* nodes, const float4* tris, float* nbox,
                                                 const uint32_t* order, uint32_t first, uint32_t count,
                                                 uint32_t n_nodes, uint32_t n_leaf_tris) {
  const uint32_t k = blockIdx.x * kB + threadIdx.x;
  if (k >= count) return;
  const uint32_t id = order[first + k];
  if (id >= n_nodes) return;
  const float pad = __uint_as_float(g.misc[6]) * (1.0f / 262144.0f);
  const Node4 nd = nodes[id];
  const int32_t refs[4] = {nd.w3.x, nd.w3.y, nd.w3.z, nd.w3.w};
  Kid kids[4];
  float nlo[3] = {INFINITY, INFINITY, INFINITY}, nhi[3] = {-INFINITY, -INFINITY, -INFINITY};
  for (int j = 0; j < 4; ++j) {
    Kid& kd = kids[j];
    kd.ref = refs[j];
    kd.empty = true;
    for (int a = 0; a < 3; ++a) {
      kd.lo[a] = INFINITY;
      kd.hi[a] = -INFINITY;
    }
    if (refs[j] == kEmpty) continue;
    if (refs[j] >= 0) {
      if ((uint32_t)refs[j] < n_nodes) {
        const float* b = nbox + 6u * (uint32_t)refs[j];
        for (int a = 0; a < 3; ++a) {
          kd.lo[a] = b[a];
          kd.hi[a] = b[3 + a];
        }
      }
    } else {
      const uint32_t start = leaf_start(refs[j]), cnt = leaf_count(refs[j]);
      for (uint32_t u = 0; u < cnt; ++u) {
        const uint32_t li = start + u;
        if (li >= n_leaf_tris) break;
        const uint32_t orig = __float_as_uint(tris[3u * li].w);
        if (orig >= g.nt) continue;
        Tri t;
        load_tri(g, orig, t);
        float lo[3], hi[3];
        tri_box(t, lo, hi);
        for (int a = 0; a < 3; ++a) {
          kd.lo[a] = fminf(kd.lo[a], lo[a]);
          kd.hi[a] = fmaxf(kd.hi[a], hi[a]);
        }
      }
    }
    kd.empty = !(kd.lo[0] <= kd.hi[0] && kd.lo[1] <= kd.hi[1] && kd.lo[2] <= kd.hi[2]);
    if (!kd.empty)
      for (int a = 0; a < 3; ++a) {
        nlo[a] = fminf(nlo[a], kd.lo[a]);
        nhi[a] = fmaxf(nhi[a], kd.hi[a]);
      }
  }
  write_node(nodes + id, kids, pad);
  for (int a = 0; a < 3; ++a) {
    nbox[6u * id + (uint32_t)a] = nlo[a];
    nbox[6u * id + 3u + (uint32_t)a] = nhi[a];
  }
}

}  // namespace

hipError_t host_refit_setup(HostRefit& r, const Node4* nodes, uint32_t n_nodes, uint32_t n_leaf_tris,
                            const uint32_t* F, const uint16_t* M, uint32_t nt) {
  hipError_t e;
  host_refit_free(r);
  r.nt = nt;
  r.n_nodes = n_nodes;
  r.n_leaf_tris = n_leaf_tris;
  // depth of every node from the root (children are emitted after parents)
  std::vector<uint32_t> depth(n_nodes, 0u);
  uint32_t max_d = 0;
  for (uint32_t i = 0; i < n_nodes; ++i) {
    const int32_t refs[4] = {nodes[i].w3.x, nodes[i].w3.y, nodes[i].w3.z, nodes[i].w3.w};
    for (int j = 0; j < 4; ++j) {
      if (refs[j] < 0) continue;
      if ((uint32_t)refs[j] >= n_nodes || (uint32_t)refs[j] <= i) return hipErrorInvalidValue;
      depth[(uint32_t)refs[j]] = depth[i] + 1u;
      max_d = std::max(max_d, depth[i] + 1u);
    }
  }
  r.level_cnt.assign(max_d + 1u, 0u);
  r.level_off.assign(max_d + 1u, 0u);
  for (uint32_t i = 0; i < n_nodes; ++i) ++r.level_cnt[depth[i]];
  for (uint32_t d = 1; d <= max_d; ++d) r.level_off[d] = r.level_off[d - 1] + r.level_cnt[d - 1];
  std::vector<uint32_t> order(std::max<uint32_t>(n_nodes, 1u)), cur = r.level_off;
  for (uint32_t i = 0; i < n_nodes; ++i) order[cur[depth[i]]++] = i;
  if ((e = hipMalloc(&r.F, 12 * (size_t)std::max<uint32_t>(nt, 1u))) != hipSuccess) return e;
  if ((e = hipMalloc(&r.M, 2 * (size_t)std::max<uint32_t>(nt, 1u))) != hipSuccess) return e;
  if ((e = hipMalloc(&r.order, 4 * order.size())) != hipSuccess) return e;
  if ((e = hipMalloc(&r.nbox, 24 * (size_t)std::max<uint32_t>(n_nodes, 1u))) != hipSuccess) return e;
  if ((e = hipMalloc(&r.misc, 4 * (size_t)kMiscWords)) != hipSuccess) return e;
  if (nt) {
    if ((e = hipMemcpy(r.F, F, 12 * (size_t)nt, hipMemcpyHostToDevice)) != hipSuccess) return e;
    if ((e = hipMemcpy(r.M, M, 2 * (size_t)nt, hipMemcpyHostToDevice)) != hipSuccess) return e;
  }
  return hipMemcpy(r.order, order.data(), 4 * order.size(), hipMemcpyHostToDevice);
}

hipError_t host_refit(HostRefit& r, const float* V, uint32_t nv, Node4* nodes, float4* tris, float4* aux,
                      hipStream_t st) {
  GpuBvh g;  // a view: the mesh and the scalars only
  g.nv = nv;
  g.nt = r.nt;
  g.V = const_cast<float*>(V);
  g.F = r.F;
  g.M = r.M;
  g.misc = r.misc;
  hipError_t e;
  hipLaunchKernelGGL(k_init_misc, dim3(1), dim3(64), 0, st, r.misc, true);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  hipLaunchKernelGGL(k_normals, grid_strided(r.nt), dim3(kBig), 0, st, g, aux);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  hipLaunchKernelGGL(k_hr_tris, grid_for(r.n_leaf_tris), dim3(kB), 0, st, g, tris, r.n_leaf_tris);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  for (int d = (int)r.level_cnt.size() - 1; d >= 0; --d) {
    const uint32_t c = r.level_cnt[(size_t)d];
    if (!c) continue;
    hipLaunchKernelGGL(k_hr_level, grid_for(c), dim3(kB), 0, st, g, nodes, tris, r.nbox, r.order,
                       r.level_off[(size_t)d], c, r.n_nodes, r.n_leaf_tris);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  return hipSuccess;
}

void host_refit_free(HostRefit& r) {
  if (r.F) (void)hipFree(r.F);
  if (r.M) (void)hipFree(r.M);
  if (r.order) (void)hipFree(r.order);
  if (r.nbox) (void)hipFree(r.nbox);
  if (r.misc) (void)hipFree(r.misc);
  r.F = nullptr;
  r.M = nullptr;
  r.order = nullptr;
  r.nbox = nullptr;
  r.misc = nullptr;
}

hipError_t rocprim_sizes(size_t n, size_t* sort_bytes, size_t* scan_bytes) {
  hipError_t e = rocprim::radix_sort_pairs(nullptr, *sort_bytes, (uint32_t*)nullptr, (uint32_t*)nullptr,
                                           (uint32_t*)nullptr, (uint32_t*)nullptr, n, 0u, 32u);
  if (e != hipSuccess) return e;
  return rocprim::exclusive_scan(nullptr, *scan_bytes, (uint32_t*)nullptr, (uint32_t*)nullptr, 0u, n,
                                 rocprim::plus<uint32_t>());
}

void gpu_bvh_free(GpuBvh& g) {
  void* ptrs[] = {g.V, g.F, g.M, g.sorted, g.child, g.parent, g.range, g.head, g.box, g.flag, g.misc, g.temp,
                  g.keys, g.ids, g.order};
  for (void* p : ptrs)
    if (p) (void)hipFree(p);
  g = GpuBvh();
}

}  // namespace rr
