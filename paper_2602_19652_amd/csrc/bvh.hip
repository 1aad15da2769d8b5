// Scene build on the device:
//  1. triangle boxes, centroid bounds, per-object boxes (field-of-view test of Sec. III-D)
//  2. 30-bit Morton codes of centroids, stable radix sort
//  3. agglomerative clustering over the Morton order (PLOC, Meister & Bittner 2018): each
//     cluster's nearest neighbour within a window is the one whose merged box has the
//     smallest surface area (the surface-area heuristic's cost driver); mutual nearest
//     neighbours merge; repeat until one cluster remains
//  4. packing into 64-byte binary nodes and the four-wide traversal nodes formed from them, triangles repacked
//     in leaf order
//  5. curvature metric C_i of Eq. (1) with the Meyer et al. cotangent operator, FP64
#include "internal.hpp"

#include <algorithm>
#include <cmath>
#include <vector>

namespace et {

namespace {

constexpr int BS = 256;

__device__ inline uint32_t f2o(float f) {
  uint32_t u = __float_as_uint(f);
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}
__device__ inline float o2f(uint32_t u) { return __uint_as_float((u & 0x80000000u) ? (u & 0x7fffffffu) : ~u); }

__global__ void k_init_bounds(uint32_t* cb, uint32_t* ob, int32_t n_obj) {
  int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < 6) cb[i] = (i < 3) ? 0xffffffffu : 0u;
  if (i < n_obj * 6) ob[i] = ((i % 6) < 3) ? 0xffffffffu : 0u;
}

// Triangle bounds (centroid bounds, object boxes) and the device checks of the mesh: vertex and
// object indices in range, finite vertex coordinates, materials >= 0 (their largest value goes
// to *mat_max when mat_max is not NULL, for the host's check against a pose's tables).
// Bound by the atomics, which land on few lines: those on the scene's own bounds and material are one per workgroup of
// few large ones, and those on object boxes are gathered in LDS (190,000 triangles in 200 objects: 78 us
// with the scene's per 256 triangles and the material's per triangle, 51 us with only the objects' per wave, 16 us so).
constexpr int TBB = 1024, TB_BLOCKS = 128, OBJ_LDS = 64;
__global__ __launch_bounds__(TBB) void k_tri_bounds(const float* __restrict__ V, const int32_t* __restrict__ tris,
                             const int32_t* __restrict__ obj, const int32_t* __restrict__ mat, int64_t T, int64_t nV,
                             int32_t n_obj, uint32_t* cb, uint32_t* ob, uint32_t* err, int32_t* mat_max) {
  __shared__ float red[7][TBB / 64];
  __shared__ uint32_t lob[6 * OBJ_LDS];
  __shared__ int32_t lowest;
  float cmin[3] = {INFINITY, INFINITY, INFINITY};      // bounds of this thread's centroids
  float cmax[3] = {-INFINITY, -INFINITY, -INFINITY};
  int32_t qm = 0;
  for (int64_t i0 = (int64_t)blockIdx.x * TBB; i0 < T; i0 += (int64_t)gridDim.x * TBB) {
    const int64_t i = i0 + threadIdx.x;
    float lo[3] = {INFINITY, INFINITY, INFINITY}, hi[3] = {-INFINITY, -INFINITY, -INFINITY};
    int32_t key = -1;   // object of a valid triangle, else -1
    if (i < T && mat_max) {
      const int32_t q = mat[i];
      if (q < 0) atomicOr(err, DEV_ERR_INDEX);
      else qm = max(qm, q);
    }
    if (i < T) {
      int32_t a = tris[3 * i], b = tris[3 * i + 1], cc = tris[3 * i + 2];
      int32_t o = obj[i];
      if (a < 0 || b < 0 || cc < 0 || a >= nV || b >= nV || cc >= nV || o < 0 || o >= n_obj) {
        atomicOr(err, DEV_ERR_INDEX);
      } else {
        key = o;
        bool finite = true;
        for (int k = 0; k < 3; ++k) {
          float x0 = V[3 * (int64_t)a + k], x1 = V[3 * (int64_t)b + k], x2 = V[3 * (int64_t)cc + k];
          finite = finite && isfinite(x0) && isfinite(x1) && isfinite(x2);
          lo[k] = fminf(x0, fminf(x1, x2));
          hi[k] = fmaxf(x0, fmaxf(x1, x2));
        }
        if (!finite) {   // a NaN or infinite coordinate: no box, and the call reports it
          atomicOr(err, DEV_ERR_VERTEX);
          key = -1;
          for (int k = 0; k < 3; ++k) {
            lo[k] = INFINITY;
            hi[k] = -INFINITY;
          }
        } else {
          for (int k = 0; k < 3; ++k) {
            const float c = 0.5f * (lo[k] + hi[k]);
            cmin[k] = fminf(cmin[k], c);
            cmax[k] = fmaxf(cmax[k], c);
          }
        }
      }
    }
    // Object boxes: triangles of an object are usually contiguous, so the workgroup gathers the boxes of up to
    // OBJ_LDS objects from its lowest on in LDS, a wave whose lanes all hold one object its own box first, and
    // issues one atomic per box and side.
    if (threadIdx.x < 6 * OBJ_LDS) lob[threadIdx.x] = threadIdx.x % 6 < 3 ? 0xffffffffu : 0u;
    if (threadIdx.x == 0) lowest = INT32_MAX;
    __syncthreads();
    int32_t low = key < 0 ? INT32_MAX : key;
    for (int off = 32; off > 0; off >>= 1) low = min(low, __shfl_xor(low, off));
    if ((threadIdx.x & 63) == 0 && low != INT32_MAX) atomicMin(&lowest, low);
    __syncthreads();
    const int32_t key0 = __shfl(key, 0);
    const bool one = __all(key == key0) && key0 >= 0;
    if (one)
      for (int k = 0; k < 3; ++k)
        for (int off = 32; off > 0; off >>= 1) {
          lo[k] = fminf(lo[k], __shfl_xor(lo[k], off));
          hi[k] = fmaxf(hi[k], __shfl_xor(hi[k], off));
        }
    if (key >= 0 && (!one || (threadIdx.x & 63) == 0)) {
      uint32_t* box = key - lowest < OBJ_LDS ? &lob[6 * (key - lowest)] : &ob[6 * (int64_t)key];
      for (int k = 0; k < 3; ++k) {
        atomicMin(&box[k], f2o(lo[k]));
        atomicMax(&box[3 + k], f2o(hi[k]));
      }
    }
    __syncthreads();
    if (threadIdx.x < 6 * OBJ_LDS) {
      const int side = threadIdx.x % 6;
      const uint32_t v = lob[threadIdx.x];
      if (side < 3 && v != 0xffffffffu) atomicMin(&ob[6 * (int64_t)lowest + threadIdx.x], v);
      if (side >= 3 && v != 0u) atomicMax(&ob[6 * (int64_t)lowest + threadIdx.x], v);
    }
    __syncthreads();
  }
  // the workgroup's centroid bounds and material: waves, then one thread per quantity
  for (int off = 32; off > 0; off >>= 1) {
    for (int k = 0; k < 3; ++k) {
      cmin[k] = fminf(cmin[k], __shfl_xor(cmin[k], off));
      cmax[k] = fmaxf(cmax[k], __shfl_xor(cmax[k], off));
    }
    qm = max(qm, __shfl_xor(qm, off));
  }
  if ((threadIdx.x & 63) == 0) {
    for (int k = 0; k < 3; ++k) {
      red[k][threadIdx.x >> 6] = cmin[k];
      red[3 + k][threadIdx.x >> 6] = -cmax[k];
    }
    red[6][threadIdx.x >> 6] = __int_as_float(qm);
  }
  __syncthreads();
  if (threadIdx.x < 6) {
    float v = INFINITY;
    for (int w = 0; w < TBB / 64; ++w) v = fminf(v, red[threadIdx.x][w]);
    if (v < INFINITY) {
      if (threadIdx.x < 3) atomicMin(&cb[threadIdx.x], f2o(v));
      else atomicMax(&cb[threadIdx.x], f2o(-v));
    }
  } else if (threadIdx.x == 6 && mat_max) {
    int32_t q = 0;
    for (int w = 0; w < TBB / 64; ++w) q = max(q, __float_as_int(red[6][w]));
    atomicMax(mat_max, q);
  }
}

__device__ inline uint32_t spread10(uint32_t x) {
  x &= 0x3ffu;
  x = (x | (x << 16)) & 0x030000FFu;
  x = (x | (x << 8)) & 0x0300F00Fu;
  x = (x | (x << 4)) & 0x030C30C3u;
  x = (x | (x << 2)) & 0x09249249u;
  return x;
}

__global__ void k_morton(const float* __restrict__ V, const int32_t* __restrict__ tris, int64_t T,
                         const uint32_t* __restrict__ cb, uint32_t* __restrict__ keys, int32_t* __restrict__ vals) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= T) return;
  uint32_t q[3];
  for (int k = 0; k < 3; ++k) {
    float x0 = V[3 * (int64_t)tris[3 * i] + k], x1 = V[3 * (int64_t)tris[3 * i + 1] + k],
          x2 = V[3 * (int64_t)tris[3 * i + 2] + k];
    float c = 0.5f * (fminf(x0, fminf(x1, x2)) + fmaxf(x0, fmaxf(x1, x2)));
    float lo = o2f(cb[k]), hi = o2f(cb[3 + k]);
    float u = hi > lo ? (c - lo) / (hi - lo) : 0.5f;
    u = fminf(fmaxf(u, 0.f), 1.f);
    q[k] = (uint32_t)fminf(u * 1024.f, 1023.f);
  }
  keys[i] = (spread10(q[0]) << 2) | (spread10(q[1]) << 1) | spread10(q[2]);
  vals[i] = (int32_t)i;
}

__global__ void k_leaves(const float* __restrict__ V, const int32_t* __restrict__ tris, const int32_t* __restrict__ mat,
                         const int32_t* __restrict__ perm, int64_t T, NodeB* __restrict__ nodes,
                         float4* __restrict__ tri4, int32_t* __restrict__ tri_orig, int32_t* __restrict__ tri_pos,
                         int32_t* __restrict__ clusters) {
  int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= T) return;
  int32_t t = perm[p];
  float v[3][3];
  for (int c = 0; c < 3; ++c)
    for (int k = 0; k < 3; ++k) v[c][k] = V[3 * (int64_t)tris[3 * (int64_t)t + c] + k];
  NodeB n;
  n.lox = fminf(v[0][0], fminf(v[1][0], v[2][0]));
  n.loy = fminf(v[0][1], fminf(v[1][1], v[2][1]));
  n.loz = fminf(v[0][2], fminf(v[1][2], v[2][2]));
  n.hix = fmaxf(v[0][0], fmaxf(v[1][0], v[2][0]));
  n.hiy = fmaxf(v[0][1], fmaxf(v[1][1], v[2][1]));
  n.hiz = fmaxf(v[0][2], fmaxf(v[1][2], v[2][2]));
  n.left = -1;
  n.right = -1;
  nodes[p] = n;
  tri4[3 * p + 0] = make_float4(v[0][0], v[0][1], v[0][2], __int_as_float(t));
  tri4[3 * p + 1] = make_float4(v[1][0], v[1][1], v[1][2], __int_as_float(mat[t]));
  tri4[3 * p + 2] = make_float4(v[2][0], v[2][1], v[2][2], 0.f);
  tri_orig[p] = t;
  tri_pos[t] = (int32_t)p;
  clusters[p] = (int32_t)p;
}

// Clustering state: current cluster count, next node id, which of the two cluster lists is current.  An iteration
// reads one copy and writes the other.
struct Ploc {
  int64_t n, next;
  int32_t list, pad;
};

__device__ inline float merged_area(float alx, float aly, float alz, float ahx, float ahy, float ahz, float blx, float bly,
                                    float blz, float bhx, float bhy, float bhz) {
  float dx = fmaxf(ahx, bhx) - fminf(alx, blx);
  float dy = fmaxf(ahy, bhy) - fminf(aly, bly);
  float dz = fmaxf(ahz, bhz) - fminf(alz, blz);
  return dx * dy + dy * dz + dz * dx;   // half the surface area (constant factor is irrelevant)
}

// Nearest neighbour of cluster i of n among i + d, d0 <= d < d1, the boxes from cluster `first` on in LDS.
struct Near {
  float a;
  int j;
};
template <int W>
__device__ inline Near nearest(const float (&box)[6][W], int64_t i, int64_t first, int64_t n, int d0, int d1) {
  const int k = (int)(i - first);
  Near b{INFINITY, -1};
#pragma unroll 4
  for (int d = d0; d < d1; ++d) {
    const int64_t j = i + d;
    if (d == 0 || j < 0 || j >= n) continue;
    const float a = merged_area(box[0][k], box[1][k], box[2][k], box[3][k], box[4][k], box[5][k], box[0][k + d],
                                box[1][k + d], box[2][k + d], box[3][k + d], box[4][k + d], box[5][k + d]);
    if (a < b.a) b = Near{a, (int)j};   // increasing j: ties keep the smaller index
  }
  return b;
}

__device__ inline NodeB merged_node(const NodeB& x, const NodeB& y, int32_t a, int32_t b) {
  NodeB m;
  m.lox = fminf(x.lox, y.lox); m.loy = fminf(x.loy, y.loy); m.loz = fminf(x.loz, y.loz);
  m.hix = fmaxf(x.hix, y.hix); m.hiy = fmaxf(x.hiy, y.hiy); m.hiz = fmaxf(x.hiz, y.hiz);
  m.left = a;
  m.right = b;
  return m;
}

// An iteration is two launches; the host reads the count after several (66 iterations and as many host waits made
// 190,000 triangles' clustering 2.5 of the build's 3.2 ms).  At PLOC_TAIL clusters both stop, and k_ploc_tail does the
// rest in one workgroup.
constexpr int PLOC_TAIL = 2048;
constexpr int PLOC_OWN = BS - 2 * PLOC_RADIUS;   // clusters per workgroup; its threads also find the window's neighbours
constexpr int64_t PLOC_SUM_BLOCKS = 1024;        // up to these the merging workgroups sum the counts before theirs

// 190,000 triangles: 27 iterations to the tail, 350 us in the kernels, of which 240 in this one (vector instructions of
// the 32 merged areas per cluster), and 200 us in the tail; the whole build 3.2 -> 1.1 ms.
// The clusters that merge: pair[i] = the partner j > i of a mutual pair's first cluster, -2 for its second (which goes),
// -1 for the others; per workgroup the clusters that stay and (high half) the merges.
__global__ __launch_bounds__(BS) void k_ploc_pairs(const int32_t* __restrict__ clA, const int32_t* __restrict__ clB,
                                                   const Ploc* __restrict__ st, const NodeB* __restrict__ nodes,
                                                   int32_t* __restrict__ pair, uint64_t* __restrict__ counts) {
  constexpr int R = PLOC_RADIUS, W = BS + 2 * R;
  __shared__ float box[6][W];
  __shared__ int nn[BS];
  __shared__ uint32_t sums[2][BS / 64];
  const int64_t n = st->n;
  const int64_t own = (int64_t)blockIdx.x * PLOC_OWN;
  if (n <= PLOC_TAIL || own >= n) {
    if (threadIdx.x == 0) counts[blockIdx.x] = 0;
    return;
  }
  const int32_t* cl = st->list ? clB : clA;
  const int64_t first = own - 2 * R;
  for (int k = threadIdx.x; k < W; k += BS) {
    const int64_t i = first + k;
    if (i >= 0 && i < n) {
      const NodeB b = nodes[cl[i]];
      box[0][k] = b.lox; box[1][k] = b.loy; box[2][k] = b.loz;
      box[3][k] = b.hix; box[4][k] = b.hiy; box[5][k] = b.hiz;
    }
  }
  __syncthreads();
  const int64_t i = own - R + threadIdx.x;
  const int j = i >= 0 && i < n ? nearest(box, i, first, n, -R, R + 1).j : -1;
  nn[threadIdx.x] = j;
  __syncthreads();
  const bool mine = threadIdx.x >= R && threadIdx.x < R + PLOC_OWN && i < n;
  const bool mutual = mine && j >= 0 && nn[j - (own - R)] == (int)i;
  if (mine) pair[i] = mutual ? (i < j ? j : -2) : -1;
  const uint64_t stay = __ballot(mine && !(mutual && j < i)), merge = __ballot(mutual && i < j);
  if ((threadIdx.x & 63) == 0) {
    sums[0][threadIdx.x >> 6] = (uint32_t)__popcll(stay);
    sums[1][threadIdx.x >> 6] = (uint32_t)__popcll(merge);
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    uint64_t t = 0;
    for (int w = 0; w < BS / 64; ++w) t += (uint64_t)sums[0][w] | (uint64_t)sums[1][w] << 32;
    counts[blockIdx.x] = t;
  }
}

// The next list and the merged nodes, in order.  before: the counts' exclusive sums, or NULL.
__global__ __launch_bounds__(BS) void k_ploc_merge(int32_t* __restrict__ clA, int32_t* __restrict__ clB,
                                                   const Ploc* __restrict__ st, Ploc* __restrict__ next,
                                                   const int32_t* __restrict__ pair, const uint64_t* __restrict__ counts,
                                                   const uint64_t* __restrict__ before, NodeB* __restrict__ nodes) {
  __shared__ uint64_t red[BS / 64];
  __shared__ uint32_t sums[2][BS / 64];
  const Ploc s = *st;
  const int64_t n = s.n, own = (int64_t)blockIdx.x * PLOC_OWN;
  if (n <= PLOC_TAIL) {
    if (blockIdx.x == 0 && threadIdx.x == 0) *next = s;
    return;
  }
  if (own >= n) return;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  uint64_t base = 0;
  if (before) {
    base = before[blockIdx.x];
  } else {
    for (int b = threadIdx.x; b < (int)blockIdx.x; b += BS) base += counts[b];
    for (int o = 32; o > 0; o >>= 1) base += __shfl_xor(base, o);
    if (lane == 0) red[wv] = base;
  }
  const int64_t i = own + threadIdx.x;
  const bool mine = threadIdx.x < PLOC_OWN && i < n;
  const int p = mine ? pair[i] : -2;
  const uint64_t stay = __ballot(p != -2), merge = __ballot(p >= 0);
  if (lane == 0) {
    sums[0][wv] = (uint32_t)__popcll(stay);
    sums[1][wv] = (uint32_t)__popcll(merge);
  }
  __syncthreads();
  if (!before) base = red[0] + red[1] + red[2] + red[3];
  const uint64_t below = (1ull << lane) - 1ull;
  int64_t at = (int64_t)(base & 0xffffffffu) + __popcll(stay & below);
  int64_t id = s.next + (int64_t)(base >> 32) + __popcll(merge & below);
  uint64_t all = base;
  for (int w = 0; w < BS / 64; ++w) {
    if (w < wv) { at += sums[0][w]; id += sums[1][w]; }
    all += (uint64_t)sums[0][w] | (uint64_t)sums[1][w] << 32;
  }
  const int32_t* cl = s.list ? clB : clA;
  int32_t* out = s.list ? clA : clB;
  if (p >= 0) {
    const int32_t a = cl[i], b = cl[p];
    nodes[id] = merged_node(nodes[a], nodes[b], a, b);
    out[at] = (int32_t)id;
  } else if (p == -1) {
    out[at] = cl[i];
  }
  if (own + PLOC_OWN >= n && threadIdx.x == 0) {   // the last workgroup with clusters
    next->n = (int64_t)(all & 0xffffffffu);
    next->next = s.next + (int64_t)(all >> 32);
    next->list = s.list ^ 1;
  }
}

// The last PLOC_TAIL clusters: boxes and ids in LDS, every iteration in this workgroup, until one is left (or no two
// merge, which the host reports).  Bound by the chain of iterations, 39 of 5 us in the room (6.4 us with a lane per
// cluster throughout).
constexpr int TAIL_T = 1024;
constexpr double PLOC_RATE = 0.17;   // -log of the share of clusters that an iteration leaves (room, foliage)
__global__ __launch_bounds__(TAIL_T) void k_ploc_tail(const int32_t* __restrict__ clA, const int32_t* __restrict__ clB,
                                                      const Ploc* __restrict__ st, Ploc* __restrict__ next,
                                                      NodeB* __restrict__ nodes) {
  constexpr int E = PLOC_TAIL / TAIL_T;
  __shared__ float box[6][PLOC_TAIL];
  __shared__ int32_t ids[PLOC_TAIL], nn[PLOC_TAIL];
  __shared__ uint32_t sums[2][E * TAIL_T / 64];
  const Ploc s = *st;
  if (s.n > PLOC_TAIL) {
    if (threadIdx.x == 0) *next = s;
    return;
  }
  int n = (int)s.n;
  int64_t id0 = s.next;
  const int32_t* cl = s.list ? clB : clA;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  for (int i = threadIdx.x; i < n; i += TAIL_T) {
    const int32_t c = cl[i];
    const NodeB b = nodes[c];
    ids[i] = c;
    box[0][i] = b.lox; box[1][i] = b.loy; box[2][i] = b.loz;
    box[3][i] = b.hix; box[4][i] = b.hiy; box[5][i] = b.hiz;
  }
  __syncthreads();
  while (n > 1) {
    if (n > TAIL_T / 2) {
      for (int i = threadIdx.x; i < n; i += TAIL_T) nn[i] = nearest(box, i, 0, n, -PLOC_RADIUS, PLOC_RADIUS + 1).j;
    } else {
      // as many lanes a cluster as there are threads for, up to 16, each over its part of the window
      const int lg = min(4, 31 - __builtin_clz(TAIL_T / n)), part = 2 * PLOC_RADIUS >> lg;
      const int i = threadIdx.x >> lg, p = threadIdx.x & ((1 << lg) - 1);
      const int d0 = -PLOC_RADIUS + p * part;
      Near b{INFINITY, -1};
      if (i < n) b = nearest(box, i, 0, n, d0, d0 + part + (p + 1 == 1 << lg ? 1 : 0));
      for (int o = 1; o < 1 << lg; o <<= 1) {
        const float a = __shfl_xor(b.a, o);
        const int j = __shfl_xor(b.j, o);
        if (j >= 0 && (b.j < 0 || a < b.a || (a == b.a && j < b.j))) b = Near{a, j};
      }
      if (i < n && p == 0) nn[i] = b.j;
    }
    __syncthreads();
    NodeB m[E];
    int32_t own[E];
    bool stays[E], merges[E];
#pragma unroll
    for (int e = 0; e < E; ++e) {
      const int i = threadIdx.x + e * TAIL_T;
      const int j = i < n ? nn[i] : -1;
      const bool mutual = j >= 0 && nn[j] == i;
      stays[e] = i < n && !(mutual && j < i);
      merges[e] = mutual && i < j;
      own[e] = i < n ? ids[i] : -1;
      if (stays[e]) {
        const NodeB x{box[0][i], box[1][i], box[2][i], 0, box[3][i], box[4][i], box[5][i], 0};
        m[e] = x;
        if (merges[e]) {
          const NodeB y{box[0][j], box[1][j], box[2][j], 0, box[3][j], box[4][j], box[5][j], 0};
          m[e] = merged_node(x, y, own[e], ids[j]);
        }
      }
      const uint64_t sb = __ballot(stays[e]), mb = __ballot(merges[e]);
      if (lane == 0) {
        sums[0][e * (TAIL_T / 64) + wv] = (uint32_t)__popcll(sb);
        sums[1][e * (TAIL_T / 64) + wv] = (uint32_t)__popcll(mb);
      }
    }
    __syncthreads();
    int total = 0, merged = 0;
    int at[E], rank[E];
    for (int w = 0; w < E * TAIL_T / 64; ++w) {
#pragma unroll
      for (int e = 0; e < E; ++e)
        if (w == e * (TAIL_T / 64) + wv) { at[e] = total; rank[e] = merged; }
      total += (int)sums[0][w];
      merged += (int)sums[1][w];
    }
#pragma unroll
    for (int e = 0; e < E; ++e) {
      const uint64_t below = (1ull << lane) - 1ull;
      const uint64_t sb = __ballot(stays[e]), mb = __ballot(merges[e]);
      if (!stays[e]) continue;
      const int p = at[e] + __popcll(sb & below);
      int32_t id = own[e];
      if (merges[e]) {
        id = (int32_t)(id0 + rank[e] + __popcll(mb & below));
        nodes[id] = m[e];
      }
      ids[p] = id;
      box[0][p] = m[e].lox; box[1][p] = m[e].loy; box[2][p] = m[e].loz;
      box[3][p] = m[e].hix; box[4][p] = m[e].hiy; box[5][p] = m[e].hiz;
    }
    n = total;
    id0 += merged;
    __syncthreads();
    if (merged == 0) break;
  }
  if (threadIdx.x == 0) *next = Ploc{n, id0, s.list, 0};
}

__global__ void k_ploc_start(Ploc* st, int64_t T) { *st = Ploc{T, T, 0, 0}; }

__global__ void k_pack(const NodeB* __restrict__ nb, int64_t T, Node2* __restrict__ out) {
  int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= T - 1) return;
  NodeB b = nb[T + k];
  NodeB c0 = nb[b.left], c1 = nb[b.right];
  Node2 n;
  n.xy0 = make_float4(c0.lox, c0.hix, c0.loy, c0.hiy);
  n.xy1 = make_float4(c1.lox, c1.hix, c1.loy, c1.hiy);
  n.zz = make_float4(c0.loz, c0.hiz, c1.loz, c1.hiz);
  int e0 = b.left >= T ? (int)(b.left - T) : ~b.left;
  int e1 = b.right >= T ? (int)(b.right - T) : ~b.right;
  n.ch = make_int4(e0, e1, -1, 0);
  out[k] = n;
}

__global__ void k_parents(Node2* __restrict__ nodes, int64_t n_inner) {
  int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= n_inner) return;
  int4 ch = nodes[k].ch;
  if (ch.x >= 0) nodes[ch.x].ch.z = (int)k;
  if (ch.y >= 0) nodes[ch.y].ch.z = (int)k;
}

// Adds the workgroup's (BS threads) sum of v to *out with one atomic.
__device__ inline void add_block(double v, double* out) {
  __shared__ double red[BS / 64];
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < BS / 64; ++w) v += red[w];
    atomicAdd(out, v);
  }
}
constexpr int SUM_BLOCKS = 256;   // workgroups of the sums over a tree (their atomics land on one address)

__device__ inline double half_area(const NodeB& b) {
  return (double)(b.hix - b.lox) * (b.hiy - b.loy) + (double)(b.hiy - b.loy) * (b.hiz - b.loz) +
         (double)(b.hiz - b.loz) * (b.hix - b.lox);
}

// SAH cost of the built tree: the areas of all 2 T - 1 nodes over the root's (190,000 triangles: 60 us with an atomic per
// triangle).
__global__ __launch_bounds__(BS) void k_sah(const NodeB* __restrict__ nb, int64_t T, int root_id, double* sah) {
  const double ra = half_area(nb[root_id]);
  double sum = 0.0;
  if (ra > 0)
    for (int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; p < 2 * T - 1; p += (int64_t)gridDim.x * blockDim.x)
      sum += half_area(nb[p]) / ra;
  add_block(sum, sah);
}

// ------------------------------------------------------------------ curvature (Eq. 1)
// The arithmetic below follows the paper's definition through the Meyer et al. operator
// with the operations in a fixed order and no contraction, so that C_i is reproducible
// to the last bit by any IEEE double implementation evaluating the same expressions.
#pragma clang fp contract(off)

__global__ void k_vcount(const int32_t* __restrict__ tris, int64_t T, uint64_t* __restrict__ cnt) {
  int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= T) return;
  for (int c = 0; c < 3; ++c) atomicAdd((unsigned long long*)&cnt[tris[3 * t + c]], 1ull);
}

// (vertex, triangle) pairs in triangle order; a stable sort by vertex leaves each vertex's
// triangles in ascending order, the order in which the operator below sums them.
__global__ void k_vkeys(const int32_t* __restrict__ tris, int64_t n3, uint32_t* __restrict__ key,
                        int32_t* __restrict__ val) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n3) return;
  key[i] = (uint32_t)tris[i];
  val[i] = (int32_t)(i / 3);
}

struct d3 { double x, y, z; };
__device__ inline d3 dsub(d3 a, d3 b) { return {a.x - b.x, a.y - b.y, a.z - b.z}; }
__device__ inline double ddot(d3 a, d3 b) { return a.x * b.x + a.y * b.y + a.z * b.z; }
__device__ inline d3 dcross(d3 a, d3 b) { return {a.y * b.z - a.z * b.y, a.z * b.x - a.x * b.z, a.x * b.y - a.y * b.x}; }
__device__ inline d3 dload(const float* V, int32_t i) {
  return {(double)V[3 * (int64_t)i], (double)V[3 * (int64_t)i + 1], (double)V[3 * (int64_t)i + 2]};
}

// The terms of triangle t at its corners in v (one corner, unless it repeats v).
struct Corners {
  int n;
  double x[3], y[3], z[3], m[3];
};
__device__ inline Corners corners(const float* __restrict__ V, const int32_t* __restrict__ tris, int64_t t, int32_t v) {
  Corners o;
  o.n = 0;
  int32_t id[3] = {tris[3 * t], tris[3 * t + 1], tris[3 * t + 2]};
  d3 P[3] = {dload(V, id[0]), dload(V, id[1]), dload(V, id[2])};
  d3 cr = dcross(dsub(P[1], P[0]), dsub(P[2], P[0]));
  double area2 = sqrt(ddot(cr, cr));
  double area = 0.5 * area2;
  if (area < 1e-20) return o;
  double dotc[3], cot[3];
  for (int c = 0; c < 3; ++c) {
    dotc[c] = ddot(dsub(P[(c + 1) % 3], P[c]), dsub(P[(c + 2) % 3], P[c]));
    cot[c] = dotc[c] / area2;
  }
  bool obtuse = dotc[0] < 0.0 || dotc[1] < 0.0 || dotc[2] < 0.0;
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    if (id[c] != v) continue;
    int c1 = (c + 1) % 3, c2 = (c + 2) % 3;
    d3 ea = dsub(P[c], P[c1]), eb = dsub(P[c], P[c2]);
    const double x = cot[c2] * ea.x + cot[c1] * eb.x, y = cot[c2] * ea.y + cot[c1] * eb.y,
                 z = cot[c2] * ea.z + cot[c1] * eb.z;
    double m;
    if (!obtuse) m = (ddot(ea, ea) * cot[c2] + ddot(eb, eb) * cot[c1]) / 8.0;   // Voronoi region
    else if (dotc[c] < 0.0) m = area / 2.0;
    else m = area / 4.0;
#pragma unroll
    for (int k = 0; k < 3; ++k)
      if (k == o.n) { o.x[k] = x; o.y[k] = y; o.z[k] = z; o.m[k] = m; }
    ++o.n;
  }
  return o;
}

// Eight lanes per vertex, a triangle each; a vertex of more triangles takes the whole wave.  The terms are then
// added in the triangles' order.  Bound by the vertex with most triangles (the room's 97,000 vertices, the fans'
// centres with 120: 102 us with a lane per vertex, 52 us with eight for all, 26 us so).
__global__ __launch_bounds__(BS) void k_vertex_curv(const float* __restrict__ V, const int32_t* __restrict__ tris,
                              const uint64_t* __restrict__ offs, const uint64_t* __restrict__ cnt,
                              const int32_t* __restrict__ adj, int64_t v0, int64_t nV, double* __restrict__ G) {
  const int64_t v = v0 + (((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 3);
  __shared__ double term[BS / 64][4][3 * 64];
  const int lane = threadIdx.x & 63, sub = threadIdx.x & 7, wv = threadIdx.x >> 6;
  double Kx = 0.0, Ky = 0.0, Kz = 0.0, Am = 0.0;
  const int64_t n = v < nV ? (int64_t)cnt[v] : 0;
  const int64_t at = n > 0 ? (int64_t)offs[v] : 0;
  Corners o;
  o.n = 0;
  const int few = n <= 8 ? (int)n : 0;
  if (sub < few) o = corners(V, tris, adj[at + sub], (int32_t)v);
  for (int l = 0; l < 8 && __any(l < few); ++l) {
    const int nt = l < few ? __shfl(o.n, l, 8) : 0;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      if (!__any(k < nt)) break;
      const double x = __shfl(o.x[k], l, 8), y = __shfl(o.y[k], l, 8), z = __shfl(o.z[k], l, 8), m = __shfl(o.m[k], l, 8);
      if (k < nt) { Kx += x; Ky += y; Kz += z; Am += m; }
    }
  }
  for (uint64_t many = __ballot(sub == 0 && n > 8); many; many &= many - 1) {
    const int src = (int)__builtin_ctzll(many);
    const int64_t vs = __shfl(v, src), ns = __shfl(n, src), as = __shfl(at, src);
    double sum = 0.0;   // lane c: component c (x, y, z, area) of four
    for (int64_t e0 = 0; e0 < ns; e0 += 64) {
      Corners c;
      c.n = 0;
      if (e0 + lane < ns) c = corners(V, tris, adj[as + e0 + lane], (int32_t)vs);
      const uint64_t n1 = __ballot(c.n > 0), n2 = __ballot(c.n > 1), n3 = __ballot(c.n > 2), below = (1ull << lane) - 1ull;
      const int first = __popcll(n1 & below) + __popcll(n2 & below) + __popcll(n3 & below);
#pragma unroll
      for (int k = 0; k < 3; ++k)
        if (k < c.n) {
          term[wv][0][first + k] = c.x[k];
          term[wv][1][first + k] = c.y[k];
          term[wv][2][first + k] = c.z[k];
          term[wv][3][first + k] = c.m[k];
        }
      const int count = __popcll(n1) + __popcll(n2) + __popcll(n3);
      wave_order();
#pragma unroll 8
      for (int i = 0; i < count; ++i) sum += term[wv][lane & 3][i];
      wave_order();
    }
    const double sx = __shfl(sum, 0), sy = __shfl(sum, 1), sz = __shfl(sum, 2), sm = __shfl(sum, 3);
    if (lane >> 3 == src >> 3) { Kx = sx; Ky = sy; Kz = sz; Am = sm; }
  }
  if (v >= nV || sub != 0) return;
  double kn = sqrt(Kx * Kx + Ky * Ky + Kz * Kz);
  G[v] = Am > 0.0 ? kn / (4.0 * Am) : 0.0;   // G = |K| / 2 with K = sum / (2 A_mixed)
}

// In launches of 2^28 vertices (a launch holds fewer than 2^32 threads).
void vertex_curv(const float* V, const int32_t* tris, const uint64_t* offs, const uint64_t* cnt, const int32_t* adj,
                 int64_t nV, double* G, hipStream_t s) {
  constexpr int64_t PER = (int64_t)1 << 28;
  for (int64_t v0 = 0; v0 < nV; v0 += PER)
    k_vertex_curv<<<(unsigned)((8 * std::min(nV - v0, PER) + BS - 1) / BS), BS, 0, s>>>(V, tris, offs, cnt, adj, v0, nV, G);
}

__global__ void k_tri_curv(const float* __restrict__ V, const int32_t* __restrict__ tris, int64_t T,
                           const double* __restrict__ G, double a_ref, double* __restrict__ C) {
  int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= T) return;
  double g0 = G[tris[3 * t]], g1 = G[tris[3 * t + 1]], g2 = G[tris[3 * t + 2]];
  double dG = fmax(g0, fmax(g1, g2)) - fmin(g0, fmin(g1, g2));
  d3 P0 = dload(V, tris[3 * t]), P1 = dload(V, tris[3 * t + 1]), P2 = dload(V, tris[3 * t + 2]);
  d3 cr = dcross(dsub(P1, P0), dsub(P2, P0));
  double area = 0.5 * sqrt(ddot(cr, cr));
  double w = a_ref > 0.0 ? fmin(1.0, area / a_ref) : 1.0;
  C[t] = w * dG;
}

#pragma clang fp contract(on)

// checks (build): the error word and the largest material, side by side for the host.
__global__ void k_obj_box(const uint32_t* __restrict__ ob, int32_t n_obj, float* __restrict__ out,
                          const uint32_t* __restrict__ err, const int32_t* __restrict__ mat_max, uint32_t* __restrict__ checks) {
  int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n_obj * 6) out[i] = o2f(ob[i]);
  if (i == 0 && checks) {
    checks[0] = *err;
    checks[1] = (uint32_t)*mat_max;
  }
}

// Slot q of the four-wide node of binary node n (see internal.hpp); one node per binary node, so that a build or a refit
// forms them in one launch without finding which of them a traversal can reach.  A lane per slot, so that a
// node is stored as one line (190,000 triangles: 19 us with a lane per node).
__device__ inline void widen(const Node2* nodes, const Node2& n, int q, float4* __restrict__ out) {
  const int n0 = n.ch.x < 0 ? 1 : 2, n1 = n.ch.y < 0 ? 1 : 2;
  float4 xy = make_float4(0.f, 0.f, 0.f, 0.f);
  float lz = 0.f, hz = 0.f;
  int child = INT32_MIN;
  if (q < n0 + n1) {
    const bool second = q >= n0;
    child = second ? n.ch.y : n.ch.x;
    xy = second ? n.xy1 : n.xy0;
    lz = second ? n.zz.z : n.zz.x;
    hz = second ? n.zz.w : n.zz.y;
    if (child >= 0) {
      const Node2 m = nodes[child];
      const bool right = (second ? q - n0 : q) != 0;
      child = right ? m.ch.y : m.ch.x;
      xy = right ? m.xy1 : m.xy0;
      lz = right ? m.zz.z : m.zz.x;
      hz = right ? m.zz.w : m.zz.y;
    }
  }
  out[2 * q] = xy;
  out[2 * q + 1] = make_float4(lz, hz, __int_as_float(child), 0.f);
}

__global__ void k_widen(const Node2* __restrict__ nodes, int64_t n_inner, float4* __restrict__ wide) {
  const int64_t k = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 2;
  if (k < n_inner) widen(nodes, nodes[k], threadIdx.x & 3, wide + 8 * k);
}

__global__ void k_single_leaf(Node2* nodes, float4* wide) {
  Node2 n;
  // both children are leaf 0: child 0 with an infinite box, child 1 with its planes swapped, which the slab test orders
  // (every ray tests the one triangle twice)
  n.xy0 = make_float4(-INFINITY, INFINITY, -INFINITY, INFINITY);
  n.xy1 = make_float4(INFINITY, -INFINITY, INFINITY, -INFINITY);
  n.zz = make_float4(-INFINITY, INFINITY, INFINITY, -INFINITY);
  n.ch = make_int4(~0, ~0, -1, 0);
  nodes[0] = n;
  for (int q = 0; q < 4; ++q) widen(nodes, n, q, wide);
}

// ------------------------------------------------------------------ refit (dynamic scenes)
// Same topology, new vertex positions.  The build groups the inner nodes by depth; a refit
// rewrites the repacked triangles, then visits the levels from the deepest up, one launch per
// wide level and per run of narrow ones (190,000 triangles, 38 levels: 16 launches): each node forms its two child boxes from its children (a leaf's triangle bounds, or
// the union of an inner child's two slots, final since the previous level).  Every node
// writes only its own slots, so no thread waits on or fences against another, and every box
// is the exact union of its leaves' FP32 bounds, as the build produces it.

// Clears some bits of the deferred error word (the others keep what earlier calls reported).
__global__ void k_clear_bits(uint32_t* err, uint32_t bits) { atomicAnd(err, ~bits); }

__global__ void k_fill_u32(uint32_t* __restrict__ a, int64_t n, uint32_t v) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    a[i] = v;
}

__global__ void k_refit_leaves(const float* __restrict__ V, const int32_t* __restrict__ tris,
                               const int32_t* __restrict__ mat, const int32_t* __restrict__ tri_orig, int64_t T,
                               float4* __restrict__ tri4) {
  const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= T) return;
  const int32_t t = tri_orig[p];
  float v[3][3];
  for (int c = 0; c < 3; ++c)
    for (int k = 0; k < 3; ++k) v[c][k] = V[3 * (int64_t)tris[3 * (int64_t)t + c] + k];
  tri4[3 * p + 0] = make_float4(v[0][0], v[0][1], v[0][2], __int_as_float(t));
  tri4[3 * p + 1] = make_float4(v[1][0], v[1][1], v[1][2], __int_as_float(mat[t]));
  tri4[3 * p + 2] = make_float4(v[2][0], v[2][1], v[2][2], 0.f);
}

struct Box6 { float lx, hx, ly, hy, lz, hz; };

__device__ inline Box6 child_box(const Node2* nodes, const float4* __restrict__ tri4, int link) {
  if (link < 0) {
    const int64_t p = ~(int64_t)link;
    const float4 a = tri4[3 * p], b = tri4[3 * p + 1], c = tri4[3 * p + 2];
    return {fminf(a.x, fminf(b.x, c.x)), fmaxf(a.x, fmaxf(b.x, c.x)), fminf(a.y, fminf(b.y, c.y)),
            fmaxf(a.y, fmaxf(b.y, c.y)), fminf(a.z, fminf(b.z, c.z)), fmaxf(a.z, fmaxf(b.z, c.z))};
  }
  const Node2 m = nodes[link];
  return {fminf(m.xy0.x, m.xy1.x), fmaxf(m.xy0.y, m.xy1.y), fminf(m.xy0.z, m.xy1.z),
          fmaxf(m.xy0.w, m.xy1.w), fminf(m.zz.x, m.zz.z), fmaxf(m.zz.y, m.zz.w)};
}

__device__ inline void refit_node(int k, int4 ch, const float4* __restrict__ tri4, Node2* nodes) {
  const Box6 b0 = child_box(nodes, tri4, ch.x), b1 = child_box(nodes, tri4, ch.y);
  nodes[k].xy0 = make_float4(b0.lx, b0.hx, b0.ly, b0.hy);
  nodes[k].xy1 = make_float4(b1.lx, b1.hx, b1.ly, b1.hy);
  nodes[k].zz = make_float4(b0.lz, b0.hz, b1.lz, b1.hz);
}

__global__ void k_refit_level(const int32_t* __restrict__ level, int64_t n, const float4* __restrict__ tri4,
                              Node2* nodes) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) refit_node(level[i], nodes[level[i]].ch, tri4, nodes);
}

// Consecutive narrow levels, from the deepest, in one workgroup.  Bound by the chain of levels; the next level's nodes
// and links, which a refit leaves as they are, are read before the barrier (24 levels 60 us without).
constexpr int NARROW = 2048, NARROW_LEVELS = 32;
struct LevelRun {
  int32_t first[NARROW_LEVELS], n[NARROW_LEVELS];
  int32_t levels;
};
__global__ __launch_bounds__(1024) void k_refit_narrow(LevelRun run, const int32_t* __restrict__ lvl_nodes,
                                                       const float4* __restrict__ tri4, Node2* nodes) {
  constexpr int E = NARROW / 1024;
  int k[E];
  int4 ch[E];
  auto fetch = [&](int l) {
#pragma unroll
    for (int e = 0; e < E; ++e) {
      const int i = threadIdx.x + 1024 * e;
      k[e] = i < run.n[l] ? lvl_nodes[run.first[l] + i] : -1;
      if (k[e] >= 0) ch[e] = nodes[k[e]].ch;
    }
  };
  fetch(0);
  for (int l = 0; l < run.levels; ++l) {
#pragma unroll
    for (int e = 0; e < E; ++e)
      if (k[e] >= 0) refit_node(k[e], ch[e], tri4, nodes);
    if (l + 1 < run.levels) fetch(l + 1);
    __threadfence_block();
    __syncthreads();
  }
}

// Depth of every inner node (root 0) by walking its parent links; histogram per depth.
template <int NL>
__global__ void k_node_depth(const Node2* __restrict__ nodes, int64_t n_inner, uint32_t* __restrict__ key,
                             int32_t* __restrict__ val, uint32_t* __restrict__ hist) {
  __shared__ uint32_t h[NL + 1];
  for (int i = threadIdx.x; i <= NL; i += blockDim.x) h[i] = 0u;
  __syncthreads();
  const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (k < n_inner) {
    int d = 0;
    for (int node = nodes[k].ch.z; node >= 0 && d < NL; node = nodes[node].ch.z) ++d;
    key[k] = (uint32_t)d;
    val[k] = (int32_t)k;
    atomicAdd(&h[d], 1u);
  }
  __syncthreads();
  for (int i = threadIdx.x; i <= NL; i += blockDim.x)
    if (h[i]) atomicAdd(&hist[i], h[i]);
}

// SAH cost of the refitted tree (C_node = C_tri = 1, normalised by the root area): the root
// contributes 1 and every other node its box area, read from its parent's child slot.
__device__ inline double slot_area(float lx, float hx, float ly, float hy, float lz, float hz) {
  return (double)(hx - lx) * (hy - ly) + (double)(hy - ly) * (hz - lz) + (double)(hz - lz) * (hx - lx);
}

// The four-wide nodes are formed in the same pass over the binary ones.
__global__ __launch_bounds__(BS) void k_refit_sah(const Node2* __restrict__ nodes, int64_t n_inner, int root,
                                                  float4* __restrict__ wide, double* sah) {
  const Node2 r = nodes[root];
  const double ra = slot_area(fminf(r.xy0.x, r.xy1.x), fmaxf(r.xy0.y, r.xy1.y), fminf(r.xy0.z, r.xy1.z),
                              fmaxf(r.xy0.w, r.xy1.w), fminf(r.zz.x, r.zz.z), fmaxf(r.zz.y, r.zz.w));
  double s = 0.0;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < 4 * n_inner; i += (int64_t)gridDim.x * blockDim.x) {
    const int64_t k = i >> 2;
    const Node2 n = nodes[k];
    widen(nodes, n, (int)(i & 3), wide + 8 * k);
    if (i & 3) continue;
    if (k == root) s += 1.0;
    if (ra > 0)
      s += (slot_area(n.xy0.x, n.xy0.y, n.xy0.z, n.xy0.w, n.zz.x, n.zz.y) +
            slot_area(n.xy1.x, n.xy1.y, n.xy1.z, n.xy1.w, n.zz.z, n.zz.w)) / ra;
  }
  add_block(s, sah);
}

inline unsigned nblk(int64_t n) { return (unsigned)((n + BS - 1) / BS > 0 ? (n + BS - 1) / BS : 1); }
inline size_t al(size_t b) { return (b + 255) / 256 * 256; }

}  // namespace

// [6] u32 centroid bounds, then a double at byte 64; zero between calls, so that a refit to
// the build's own vertices leaves the whole blob as the build left it
constexpr size_t REFIT_SCRATCH = 256;
constexpr int MAX_LEVEL = TRAV_STACK + 1;
// What the host reads of a built tree: SAH cost, inner nodes per depth.
struct TreeSummary {
  double sah;
  uint32_t hist[MAX_LEVEL + 1];
};

size_t scene_blob_bytes(int64_t T, int64_t V, int32_t n_obj) {
  size_t b = 0;
  b += al(sizeof(Node2) * (size_t)std::max<int64_t>(1, T - 1));
  b += al(sizeof(float4) * 8 * (size_t)std::max<int64_t>(1, T - 1));
  b += al(sizeof(float4) * 3 * (size_t)std::max<int64_t>(1, T));
  b += 2 * al(sizeof(int32_t) * (size_t)std::max<int64_t>(1, T));   // tri_orig, tri_pos
  b += al(sizeof(double) * (size_t)std::max<int64_t>(1, T));
  b += al(sizeof(double) * (size_t)std::max<int64_t>(1, V));
  b += al(sizeof(float) * 6 * (size_t)std::max<int32_t>(1, n_obj));
  // kept for refits: inner nodes by depth, vertex-triangle lists, refit scratch
  b += al(sizeof(int32_t) * (size_t)std::max<int64_t>(1, T - 1));
  b += 2 * al(sizeof(uint64_t) * (size_t)std::max<int64_t>(1, V));
  b += al(sizeof(int32_t) * 3 * (size_t)std::max<int64_t>(1, T));
  b += al(REFIT_SCRATCH);
  return b;
}

size_t scene_scratch_bytes(int64_t T, int64_t V) {
  const int64_t Tm = std::max<int64_t>(T, 1), Vm = std::max<int64_t>(V, 1);
  size_t b = 0;
  b += al(sizeof(uint32_t) * 6) + al(sizeof(uint32_t) * 6 * 1);   // centroid bounds (object bounds sized below)
  b += al(sizeof(uint32_t) * Tm) + al(sizeof(int32_t) * Tm);       // morton keys / perm
  b += sort_temp_bytes(Tm, 4);
  b += al(sizeof(NodeB) * (size_t)(2 * Tm));                       // build nodes
  b += 2 * al(sizeof(int32_t) * Tm);                               // clusters ping-pong
  b += al(sizeof(int32_t) * Tm);                                   // nn
  b += 2 * al(sizeof(uint64_t) * Tm);                              // clustering counts and their sums, per workgroup
  b += scan_temp_bytes(std::max(Tm, Vm));
  b += al(sizeof(int64_t) * 8);                                    // clustering states
  b += al(sizeof(TreeSummary));
  b += al(sizeof(uint32_t) * 3 * Tm) + sort_temp_bytes(3 * Tm, 4);  // vertex-triangle pair keys, sort
  return b;
}

void scene_build(et_scene* sc, const et_mesh_desc* mesh, void* blob, void* scratch, uint32_t* dev_err, hipStream_t s) {
  const int64_t T = mesh->T, V = mesh->V;
  const int32_t n_obj = mesh->n_objects;
  SceneDev& d = sc->d;
  d.T = T; d.V = V; d.n_obj = n_obj;
  d.verts = mesh->vertices; d.tris = mesh->tris; d.mat = mesh->tri_material; d.obj = mesh->tri_object;
  // blob layout
  char* bp = (char*)blob;
  auto takeb = [&](size_t bytes) { char* p = bp; bp += al(bytes); return (void*)p; };
  d.nodes = (Node2*)takeb(sizeof(Node2) * (size_t)std::max<int64_t>(1, T - 1));
  d.wide = (float4*)takeb(sizeof(float4) * 8 * (size_t)std::max<int64_t>(1, T - 1));
  d.tri4 = (float4*)takeb(sizeof(float4) * 3 * (size_t)std::max<int64_t>(1, T));
  d.tri_orig = (int32_t*)takeb(sizeof(int32_t) * (size_t)std::max<int64_t>(1, T));
  d.tri_pos = (int32_t*)takeb(sizeof(int32_t) * (size_t)std::max<int64_t>(1, T));
  d.C = (double*)takeb(sizeof(double) * (size_t)std::max<int64_t>(1, T));
  d.G = (double*)takeb(sizeof(double) * (size_t)std::max<int64_t>(1, V));
  d.obj_box = (float*)takeb(sizeof(float) * 6 * (size_t)std::max<int32_t>(1, n_obj));
  sc->lvl_nodes = (int32_t*)takeb(sizeof(int32_t) * (size_t)std::max<int64_t>(1, T - 1));
  sc->vcnt = (uint64_t*)takeb(sizeof(uint64_t) * (size_t)std::max<int64_t>(1, V));
  sc->voff = (uint64_t*)takeb(sizeof(uint64_t) * (size_t)std::max<int64_t>(1, V));
  sc->adj = (int32_t*)takeb(sizeof(int32_t) * 3 * (size_t)std::max<int64_t>(1, T));
  sc->rscratch = takeb(REFIT_SCRATCH);
  // scratch layout
  const int64_t Tm = std::max<int64_t>(T, 1), Vm = std::max<int64_t>(V, 1);
  char* sp = (char*)scratch;
  auto take = [&](size_t bytes) { char* p = sp; sp += al(bytes); return (void*)p; };
  uint32_t* cb = (uint32_t*)take(sizeof(uint32_t) * 6);
  int32_t* mat_max = (int32_t*)take(sizeof(uint32_t) * 6);   // [0]: largest material index
  uint32_t* checks = (uint32_t*)mat_max + 2;                 // [2]: error word, material, for the host
  uint32_t* keys = (uint32_t*)take(sizeof(uint32_t) * Tm);
  int32_t* perm = (int32_t*)take(sizeof(int32_t) * Tm);
  void* sort_tmp = take(sort_temp_bytes(Tm, 4));
  NodeB* nb = (NodeB*)take(sizeof(NodeB) * (size_t)(2 * Tm));
  int32_t* clA = (int32_t*)take(sizeof(int32_t) * Tm);
  int32_t* clB = (int32_t*)take(sizeof(int32_t) * Tm);
  int32_t* nn = (int32_t*)take(sizeof(int32_t) * Tm);
  uint64_t* flags = (uint64_t*)take(sizeof(uint64_t) * Tm);
  uint64_t* offs = (uint64_t*)take(sizeof(uint64_t) * Tm);
  void* scan_tmp = take(scan_temp_bytes(std::max(Tm, Vm)));
  int64_t* ctr = (int64_t*)take(sizeof(int64_t) * 8);      // two clustering states
  TreeSummary* tree = (TreeSummary*)take(sizeof(TreeSummary));
  uint32_t* vkey = (uint32_t*)take(sizeof(uint32_t) * 3 * Tm);
  void* vsort_tmp = take(sort_temp_bytes(3 * Tm, 4));
  uint64_t* vcnt = sc->vcnt;
  uint64_t* voff = sc->voff;
  int32_t* adj = sc->adj;
  // object boxes live in the blob as floats; build them as ordered uints in the blob memory
  uint32_t* ob = (uint32_t*)d.obj_box;

  hipEvent_t e0, e1;
  ET_HIP(hipEventCreate(&e0));
  ET_HIP(hipEventCreate(&e1));
  ET_HIP(hipEventRecord(e0, s));

  k_init_bounds<<<nblk(6 * (int64_t)std::max(n_obj, 1)), BS, 0, s>>>(cb, ob, n_obj);
  k_fill_u32<<<1, 1, 0, s>>>((uint32_t*)mat_max, 1, 0u);
  if (T > 0) {
    k_tri_bounds<<<(unsigned)std::min<int64_t>((T + TBB - 1) / TBB, TB_BLOCKS), TBB, 0, s>>>(d.verts, d.tris, d.obj, d.mat, T, V, n_obj, cb, ob, dev_err, mat_max);
  }
  k_obj_box<<<nblk(6 * (int64_t)std::max(n_obj, 1)), BS, 0, s>>>(ob, n_obj, d.obj_box, dev_err, mat_max, checks);
  ET_HIP(hipGetLastError());
  // the index check must pass before any kernel dereferences triangle indices
  uint32_t hchecks[2] = {0, 0};
  ET_HIP(hipMemcpyAsync(hchecks, checks, sizeof(hchecks), hipMemcpyDeviceToHost, s));
  ET_HIP(hipStreamSynchronize(s));
  const uint32_t herr = hchecks[0];
  ET_CHECK(!(herr & DEV_ERR_INDEX), ET_E_INVALID,
           "mesh index out of range (triangle vertex or object index, or a negative material)");
  ET_CHECK(!(herr & DEV_ERR_VERTEX), ET_E_INVALID, "non-finite vertex coordinate in a triangle");
  sc->max_mat = T > 0 ? (int32_t)hchecks[1] : -1;

  if (T >= 1) {
    k_morton<<<nblk(T), BS, 0, s>>>(d.verts, d.tris, T, cb, keys, perm);
    radix_sort_u32(keys, perm, T, 30, sort_tmp, s);
    k_leaves<<<nblk(T), BS, 0, s>>>(d.verts, d.tris, d.mat, perm, T, nb, d.tri4, d.tri_orig, d.tri_pos, clA);
    ET_HIP(hipGetLastError());
  }
  int root_id = 0;
  if (T >= 2) {
    // agglomerative clustering; the cluster count lives on the device, and the host reads it after as many
    // iterations as usually reach the tail (too many cost empty launches, 5 us each; too few another wait, 25 us)
    Ploc* st[2] = {(Ploc*)ctr, (Ploc*)ctr + 1};
    k_ploc_start<<<1, 1, 0, s>>>(st[0], T);
    int64_t n = T;
    int cur = 0;
    while (n > 1) {
      const int64_t blocks = (n + PLOC_OWN - 1) / PLOC_OWN;
      const bool scan = blocks > PLOC_SUM_BLOCKS;
      int iters = n > PLOC_TAIL ? 1 + (int)std::ceil(std::log((double)n / PLOC_TAIL) / PLOC_RATE) : 0;
      if (scan) iters = std::min(iters, 4);   // (the grids shrink at the next read)
      for (int k = 0; k < iters; ++k, cur ^= 1) {
        k_ploc_pairs<<<(unsigned)blocks, BS, 0, s>>>(clA, clB, st[cur], nb, nn, flags);
        if (scan) scan_exclusive_u64(flags, offs, blocks, nullptr, blocks, nullptr, scan_tmp, s);
        k_ploc_merge<<<(unsigned)blocks, BS, 0, s>>>(clA, clB, st[cur], st[cur ^ 1], nn, flags, scan ? offs : nullptr, nb);
      }
      k_ploc_tail<<<1, TAIL_T, 0, s>>>(clA, clB, st[cur], st[cur ^ 1], nb);
      cur ^= 1;
      ET_HIP(hipGetLastError());
      Ploc h;
      ET_HIP(hipMemcpyAsync(&h, st[cur], sizeof(Ploc), hipMemcpyDeviceToHost, s));
      ET_HIP(hipStreamSynchronize(s));
      ET_CHECK(h.n < n && h.n >= 1 && (h.n == 1 || h.n > PLOC_TAIL), ET_E_INTERNAL, "BVH clustering made no progress");
      n = h.n;
      if (n == 1) ET_CHECK(h.next == 2 * T - 1, ET_E_INTERNAL, "BVH node count mismatch");
    }
    root_id = (int)(2 * T - 2);
    k_pack<<<nblk(T - 1), BS, 0, s>>>(nb, T, d.nodes);
    k_parents<<<nblk(T - 1), BS, 0, s>>>(d.nodes, T - 1);
    k_widen<<<nblk(4 * (T - 1)), BS, 0, s>>>(d.nodes, T - 1, d.wide);
    k_fill_u32<<<1, BS, 0, s>>>((uint32_t*)tree, sizeof(TreeSummary) / 4, 0u);
    k_sah<<<std::min(nblk(T), (unsigned)SUM_BLOCKS), BS, 0, s>>>(nb, T, root_id, &tree->sah);
    // inner nodes grouped by depth for refits (stable sort: the order is deterministic)
    k_node_depth<MAX_LEVEL><<<nblk(T - 1), BS, 0, s>>>(d.nodes, T - 1, keys, sc->lvl_nodes, tree->hist);
    radix_sort_u32(keys, sc->lvl_nodes, T - 1, 7, sort_tmp, s);
    ET_HIP(hipGetLastError());
    d.root = (int)(T - 2);   // the last node created is the root; packed index = id - T
    sc->n_nodes = T - 1;
  } else {
    k_single_leaf<<<1, 1, 0, s>>>(d.nodes, d.wide);
    d.root = 0;
    sc->n_nodes = 1;
  }

  k_fill_u32<<<1, BS, 0, s>>>((uint32_t*)sc->rscratch, REFIT_SCRATCH / 4, 0u);
  // curvature (Eq. 1)
  if (T > 0 && V > 0) {
    k_fill_u32<<<std::min(nblk(2 * V), 1u << 20), BS, 0, s>>>((uint32_t*)vcnt, 2 * V, 0u);
    k_vcount<<<nblk(T), BS, 0, s>>>(d.tris, T, vcnt);
    scan_exclusive_u64(vcnt, voff, V, nullptr, V, nullptr, scan_tmp, s);
    k_vkeys<<<nblk(3 * T), BS, 0, s>>>(d.tris, 3 * T, vkey, adj);
    int vbits = 1;
    while (vbits < 32 && ((int64_t)1 << vbits) < V) ++vbits;
    radix_sort_u32(vkey, adj, 3 * T, vbits, vsort_tmp, s);
    vertex_curv(d.verts, d.tris, voff, vcnt, adj, V, d.G, s);
    k_tri_curv<<<nblk(T), BS, 0, s>>>(d.verts, d.tris, T, d.G, mesh->area_ref, d.C);
    ET_HIP(hipGetLastError());
  }
  ET_HIP(hipEventRecord(e1, s));
  ET_HIP(hipEventSynchronize(e1));
  float ms = 0;
  ET_HIP(hipEventElapsedTime(&ms, e0, e1));
  sc->build_ms = ms;
  ET_HIP(hipEventDestroy(e0));
  ET_HIP(hipEventDestroy(e1));
  if (T >= 2) {
    TreeSummary h;
    ET_HIP(hipMemcpyAsync(&h, tree, sizeof(h), hipMemcpyDeviceToHost, s));
    ET_HIP(hipStreamSynchronize(s));
    sc->sah = h.sah;
    const uint32_t* hist = h.hist;
    int levels = MAX_LEVEL + 1;
    while (levels > 0 && hist[levels - 1] == 0) --levels;
    sc->lvl_off.assign(1, 0);
    sc->depth = levels + 1;   // inner nodes and a leaf
    for (int l = 0; l < levels; ++l) sc->lvl_off.push_back(sc->lvl_off.back() + hist[l]);
    ET_CHECK(sc->lvl_off.back() == T - 1, ET_E_INTERNAL, "BVH level grouping lost nodes");
  } else {
    sc->depth = T;
    sc->sah = T;
  }
  ET_CHECK(sc->depth <= TRAV_STACK, ET_E_UNSUPPORTED, "BVH deeper than the traversal stack");
}

}  // namespace et

namespace et {

void scene_refit(et_scene* sc, const float* vertices, double area_ref, uint32_t* dev_err, hipStream_t s) {
  SceneDev& d = sc->d;
  const int64_t T = d.T, V = d.V;
  const int32_t n_obj = d.n_obj;
  d.verts = vertices;
  uint32_t* cb = (uint32_t*)sc->rscratch;
  double* sah = (double*)((char*)sc->rscratch + 64);
  uint32_t* ob = (uint32_t*)d.obj_box;
  hipEvent_t e0, e1;
  ET_HIP(hipEventCreate(&e0));
  ET_HIP(hipEventCreate(&e1));
  ET_HIP(hipEventRecord(e0, s));
  k_clear_bits<<<1, 1, 0, s>>>(dev_err, DEV_ERR_VERTEX);
  k_init_bounds<<<nblk(6 * (int64_t)std::max(n_obj, 1)), BS, 0, s>>>(cb, ob, n_obj);
  if (T > 0) k_tri_bounds<<<(unsigned)std::min<int64_t>((T + TBB - 1) / TBB, TB_BLOCKS), TBB, 0, s>>>(d.verts, d.tris, d.obj, d.mat, T, V, n_obj, cb, ob, dev_err, nullptr);
  k_obj_box<<<nblk(6 * (int64_t)std::max(n_obj, 1)), BS, 0, s>>>(ob, n_obj, d.obj_box, nullptr, nullptr, nullptr);
  if (T > 0) k_refit_leaves<<<nblk(T), BS, 0, s>>>(d.verts, d.tris, d.mat, d.tri_orig, T, d.tri4);
  if (T >= 2) {
    for (int l = (int)sc->lvl_off.size() - 2; l >= 0;) {
      const int64_t a = sc->lvl_off[l], n = sc->lvl_off[l + 1] - a;
      if (n > NARROW) {
        k_refit_level<<<nblk(n), BS, 0, s>>>(sc->lvl_nodes + a, n, d.tri4, d.nodes);
        --l;
        continue;
      }
      LevelRun run{};
      for (; l >= 0 && run.levels < NARROW_LEVELS && sc->lvl_off[l + 1] - sc->lvl_off[l] <= NARROW; --l) {
        run.first[run.levels] = (int32_t)sc->lvl_off[l];
        run.n[run.levels++] = (int32_t)(sc->lvl_off[l + 1] - sc->lvl_off[l]);
      }
      k_refit_narrow<<<1, 1024, 0, s>>>(run, sc->lvl_nodes, d.tri4, d.nodes);
    }
    k_fill_u32<<<1, BS, 0, s>>>((uint32_t*)sah, 2, 0u);
    k_refit_sah<<<std::min(nblk(4 * (T - 1)), (unsigned)SUM_BLOCKS * 2), BS, 0, s>>>(d.nodes, T - 1, d.root, d.wide, sah);
  }
  if (T > 0 && V > 0) {   // the vertex-triangle lists depend on the topology only
    vertex_curv(d.verts, d.tris, sc->voff, sc->vcnt, sc->adj, V, d.G, s);
    k_tri_curv<<<nblk(T), BS, 0, s>>>(d.verts, d.tris, T, d.G, area_ref, d.C);
  }
  ET_HIP(hipGetLastError());
  ET_HIP(hipEventRecord(e1, s));
  ET_HIP(hipEventSynchronize(e1));
  float ms = 0;
  ET_HIP(hipEventElapsedTime(&ms, e0, e1));
  sc->refit_ms = ms;
  ET_HIP(hipEventDestroy(e0));
  ET_HIP(hipEventDestroy(e1));
  if (T >= 2) ET_HIP(hipMemcpyAsync(&sc->sah, sah, sizeof(double), hipMemcpyDeviceToHost, s));
  k_fill_u32<<<1, BS, 0, s>>>((uint32_t*)sc->rscratch, REFIT_SCRATCH / 4, 0u);
  ET_HIP(hipGetLastError());
  uint32_t herr = 0;
  ET_HIP(hipMemcpyAsync(&herr, dev_err, sizeof(uint32_t), hipMemcpyDeviceToHost, s));
  k_clear_bits<<<1, 1, 0, s>>>(dev_err, DEV_ERR_VERTEX);   // reported by this call's status only
  ET_HIP(hipGetLastError());
  ET_HIP(hipStreamSynchronize(s));
  ET_CHECK(!(herr & DEV_ERR_VERTEX), ET_E_INVALID,
           "non-finite vertex coordinate in a triangle (refit again with finite vertices before tracing)");
}

}  // namespace et
