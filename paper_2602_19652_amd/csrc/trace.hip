// Ray tracing of one pose (Sec. III-C, Algorithm 1) and diffraction sampling (Sec. III-D).
//
// Per bounce j, over the list of active rays:
//   k_walk      FP32 closest-hit BVH traversal of the FP64 ray rounded to FP32 (which triangle), FP64 plane
//               intersection, specular reflection about the face normal and path-length update (where);
//               in the same launch the FP32 any-hit line-of-sight rays of the previous bounce's records
//               toward x_ref (or each receiver)
//   k_mask_sums sums of the waves' hit and continue masks (large ray sets; small ones are summed in place)
//   k_records   stable compaction: records in ray order after the earlier bounces' records, the list of the
//               rays that go on in ray order
// Ray order: a ray set larger than one round of the walks' grid (the threads the chip holds at
// once) is first sorted (stably) by a 16-bit octahedral Morton key of its world direction, so
// that the rays of a wave walk nearby parts of the BVH; the stable compaction keeps that order
// through the bounces, and records carry their ray.  Whole pose in the room with 2^20 rays: 11.98 ms
// sorted, the sort included, against 12.28 ms in seeded order; smaller sets keep their given order.
// Traversal: four lanes per ray over four-wide nodes (see walk_rays), nearest child first, stacks in LDS, leaves
// tested together (after Aila & Laine, HPG 2009), watertight ray-triangle test
// (Woop, Benthin & Wald, JCGT 2013), conservative slab test (Ize 2013).
#include "internal.hpp"

#include <algorithm>
#include <atomic>
#include <cmath>

namespace et {

namespace {

constexpr int BS = TRAV_BLOCK;
constexpr int EMPTY = INT32_MIN;
// Grids of up to 8192 blocks (then whole rounds of resident ones, see trace_run): the room's 2^20 rays and their
// line-of-sight rays are 32,768 chunks of 64, one or two to a wave, so the hardware dispatcher balances uneven chunks
// (1536 blocks, one round that strides: 3% slower poses, foliage 6%).
constexpr int MAX_BLOCKS = 8192;

// Waves that a traversal of few rays is spread over, 16 rays to a wave at the least (see k_walk).
constexpr int64_t RS_WAVES = 2560;

inline unsigned nblk(int64_t n) { return (unsigned)std::max<int64_t>(1, std::min<int64_t>((n + BS - 1) / BS, MAX_BLOCKS)); }
inline unsigned nblk_full(int64_t n) { return (unsigned)std::max<int64_t>(1, (n + BS - 1) / BS); }

struct Ray32 {
  float ox, oy, oz;
  float ix, iy, iz;          // reciprocal direction (tiny components clamped)
  float okx, oky, okz;       // origin permuted for the watertight test
  float Sx, Sy, Sz;          // shear constants
  int kx, ky, kz;
};

__device__ inline float sel3(float a, float b, float c, int k) { return k == 0 ? a : (k == 1 ? b : c); }

__device__ inline float safe_rcp(float d) {
  const float tiny = 1e-30f;
  return 1.0f / (fabsf(d) < tiny ? (d < 0.f ? -tiny : tiny) : d);
}

__device__ inline Ray32 make_ray(double ox, double oy, double oz, double dx, double dy, double dz) {
  Ray32 r;
  r.ox = (float)ox; r.oy = (float)oy; r.oz = (float)oz;
  const float fx = (float)dx, fy = (float)dy, fz = (float)dz;
  r.ix = safe_rcp(fx); r.iy = safe_rcp(fy); r.iz = safe_rcp(fz);
  const float ax = fabsf(fx), ay = fabsf(fy), az = fabsf(fz);
  int kz = (ax >= ay && ax >= az) ? 0 : (ay >= az ? 1 : 2);
  int kx = kz + 1 == 3 ? 0 : kz + 1;
  int ky = kx + 1 == 3 ? 0 : kx + 1;
  const float dkz = sel3(fx, fy, fz, kz);
  if (dkz < 0.f) { int t = kx; kx = ky; ky = t; }
  r.kx = kx; r.ky = ky; r.kz = kz;
  r.Sx = sel3(fx, fy, fz, kx) / dkz;
  r.Sy = sel3(fx, fy, fz, ky) / dkz;
  r.Sz = 1.0f / dkz;
  r.okx = sel3(r.ox, r.oy, r.oz, kx);
  r.oky = sel3(r.ox, r.oy, r.oz, ky);
  r.okz = sel3(r.ox, r.oy, r.oz, kz);
  return r;
}

// Watertight ray-triangle test, two-sided.  Returns t (or a negative value on a miss).
__device__ inline float tri_test(const float4 a, const float4 b, const float4 c, const Ray32& r) {
#pragma clang fp contract(off)
  const float Ax0 = sel3(a.x, a.y, a.z, r.kx) - r.okx, Ay0 = sel3(a.x, a.y, a.z, r.ky) - r.oky,
              Az0 = sel3(a.x, a.y, a.z, r.kz) - r.okz;
  const float Bx0 = sel3(b.x, b.y, b.z, r.kx) - r.okx, By0 = sel3(b.x, b.y, b.z, r.ky) - r.oky,
              Bz0 = sel3(b.x, b.y, b.z, r.kz) - r.okz;
  const float Cx0 = sel3(c.x, c.y, c.z, r.kx) - r.okx, Cy0 = sel3(c.x, c.y, c.z, r.ky) - r.oky,
              Cz0 = sel3(c.x, c.y, c.z, r.kz) - r.okz;
  const float Ax = Ax0 - r.Sx * Az0, Ay = Ay0 - r.Sy * Az0;
  const float Bx = Bx0 - r.Sx * Bz0, By = By0 - r.Sy * Bz0;
  const float Cx = Cx0 - r.Sx * Cz0, Cy = Cy0 - r.Sy * Cz0;
  float U = Cx * By - Cy * Bx;
  float V = Ax * Cy - Ay * Cx;
  float W = Bx * Ay - By * Ax;
  if (U == 0.f || V == 0.f || W == 0.f) {   // exact edge: decide in double (watertightness)
    U = (float)((double)Cx * (double)By - (double)Cy * (double)Bx);
    V = (float)((double)Ax * (double)Cy - (double)Ay * (double)Cx);
    W = (float)((double)Bx * (double)Ay - (double)By * (double)Ax);
  }
  if ((U < 0.f || V < 0.f || W < 0.f) && (U > 0.f || V > 0.f || W > 0.f)) return -1.f;
  const float det = U + V + W;
  if (det == 0.f) return -1.f;
  const float Az = r.Sz * Az0, Bz = r.Sz * Bz0, Cz = r.Sz * Cz0;
  const float T = U * Az + V * Bz + W * Cz;
  return T / det;
}

struct PoseArgs {
  double s[3];
  double R[9];
  double xref[3];
  int64_t N;
  int32_t B;
  double maxd;
  double t_eps;
};

// One job of a fused batch: its scene, pose and ray directions.  Rays [ray0, ray0 + a.N) of
// the batch belong to it; in the ray state and the records the ray field holds the job.
struct TraceJob {
  SceneDev S;
  PoseArgs a;
  const float* dirs;
  int64_t ray0;
};

// Four lanes (a quad) walk a ray: each tests one child box of a four-wide node, and up to four leaves at the top of the
// stack are tested at once, one per lane.  A quad's stack is a column of LDS: entry i (1 .. cap) at col[i * QW], entry 0
// always EMPTY, so that an empty stack yields EMPTY.
template <int TB>
struct QuadLds {
  static constexpr int QW = TB / 4;             // quads per block
  int stack[(QUAD_STACK + 1) * QW];
  int2 res[TB];                                 // hit position and distance bits of each wave's 64 rays
};

struct QuadStack {
  int cap;        // entries a quad may hold: QUAD_STACK (lower only when a test forces overflows)
  int overflow;   // dropped pushes
};

template <int CTRL>
__device__ inline int quad_perm(int v) {
  return __builtin_amdgcn_update_dpp(0, v, CTRL, 0xf, 0xf, true);
}
constexpr int QP1 = 0xB1, QP2 = 0x4E, QP3 = 0x1B;   // lane q reads lane q ^ 1, q ^ 2, q ^ 3 of its quad
__device__ inline int quad_or(int v) { v |= quad_perm<QP1>(v); return v | quad_perm<QP2>(v); }
__device__ inline int quad_sum(int v) { v += quad_perm<QP1>(v); return v + quad_perm<QP2>(v); }
__device__ inline float quad_min(float v) {
  v = fminf(v, __int_as_float(quad_perm<QP1>(__float_as_int(v))));
  return fminf(v, __int_as_float(quad_perm<QP2>(__float_as_int(v))));
}
__device__ inline int from_lane(int v, int src4) { return __builtin_amdgcn_ds_bpermute(src4, v); }
__device__ inline float from_lane(float v, int src4) {
  return __int_as_float(__builtin_amdgcn_ds_bpermute(src4, __float_as_int(v)));
}

// Closest hits (any = false) or any hits (any = true) of the wave's rays: lane l < nr holds ray l; t in (tmin, tmax),
// excluding the leaf position excl; walked = false: the ray hits nothing.  Called by all 64 lanes; leaves ray
// l's leaf position (-1: none) and distance in pos, t of lane l.  Closest-hit ties in t go to the smaller original
// triangle index.
// Boxes are culled against the current best distance widened by 2^-19 relative (about 16
// ulps, more than the rounding of a box entry plus that of a triangle's t): a triangle whose
// computed t ties the best (or lies within rounding of it, as on a shared edge or a box face
// whose slab entry equals the hit distance) is always tested, so the hit does not depend on
// the traversal order, and a refitted tree hits what a rebuilt one hits.
// Bound by the chain of dependent steps where rays are few (a step: node from L2, boxes, stack), by vector
// instructions and node bytes where they are many.  One lane per ray over binary nodes took twice the steps,
// ran them with half of the lanes or fewer (32 of 64 in the room, 24 in foliage), and
// fetched 64 B per ray and step through 64 different lines.  Measured (walks of a pose, before and after): 16,384
// rays 105 -> 50 us, 50,003 rays in the room 403 -> 204 us, 2^20 there 2.12 -> 1.94 ms, 2^20 in foliage 7.1 -> 6.4 ms.
// Leaves wait for three eighths of the quads: for a quarter, poses took 3% longer in the room and 1% in foliage, for
// an eighth 4 and 9%, for half foliage 2%, for all 16%.  Handing out rays at 4 or 6 free quads instead of 2 cost 1
// to 2%, at every free one as much.
constexpr float T_WIDEN = 1.0f + 1.9073486328125e-6f;   // 1 + 2^-19
constexpr int REFILL_LANES = 8;   // lanes of quads without a ray that make the wave hand out rays
template <bool COUNT, int TB>
__device__ inline void walk_rays(const SceneDev& S, const Ray32& r, bool walked, float tmin, float tmax, int excl, int nr,
                                 bool any, QuadLds<TB>& L, QuadStack& st, int& pos, float& t, int64_t& cn, int64_t& ct) {
  constexpr int QW = QuadLds<TB>::QW;
  const int lane = threadIdx.x & 63, q = lane & 3;
  int* col = L.stack + (threadIdx.x >> 2);
  int2* res = L.res + (threadIdx.x & ~63);
  const int pack = r.kx | r.ky << 2 | r.kz << 4 | (walked ? 64 : 0);
  const float4* wide = S.wide + 2 * q;
  const float4* tri4 = S.tri4;
  Ray32 u;                     // the quad's ray
  int ex = -1, cur = -1;       // its excluded leaf, its lane
  int node = EMPTY, sp = 0;    // >= 0 inner node, < 0 leaf ~position, EMPTY: done
  float bt = 0.f, tb = 0.f, tbw = 0.f;         // this lane's best, the quad's best, widened
  int best = -1, borig = INT32_MAX;
  int taken = 0;
  while (true) {
    const uint64_t idle = __ballot(node == EMPTY);
    const int n_idle = __popcll(idle);
    if (taken < nr ? n_idle >= REFILL_LANES : n_idle == 64) {
      // finished quads hand in the best of their lanes
      if (node == EMPTY && cur >= 0) {
#pragma unroll
        for (int m = 0; m < 2; ++m) {
          const int tj = m ? quad_perm<QP2>(__float_as_int(bt)) : quad_perm<QP1>(__float_as_int(bt));
          const int oj = m ? quad_perm<QP2>(borig) : quad_perm<QP1>(borig);
          const int bj = m ? quad_perm<QP2>(best) : quad_perm<QP1>(best);
          const float tf = __int_as_float(tj);
          if (tf < bt || (tf == bt && oj < borig)) { bt = tf; borig = oj; best = bj; }
        }
        if (q == 0) res[cur] = make_int2(best, __float_as_int(bt));
        cur = -1;
      }
      wave_order();   // (lane `cur` reads the result)
      if (taken >= nr) break;
      // and take the next rays
      const int nx = taken + (int)(__builtin_amdgcn_mbcnt_hi((uint32_t)(idle >> 32),
                                                             __builtin_amdgcn_mbcnt_lo((uint32_t)idle, 0u)) >> 2);
      const bool get = node == EMPTY && nx < nr;
      const int src = (get ? nx : lane) * 4;
      const float ox = from_lane(r.ox, src), oy = from_lane(r.oy, src), oz = from_lane(r.oz, src);
      const float ix = from_lane(r.ix, src), iy = from_lane(r.iy, src), iz = from_lane(r.iz, src);
      const float Sx = from_lane(r.Sx, src), Sy = from_lane(r.Sy, src), tx = from_lane(tmax, src);
      const int pk = from_lane(pack, src), e = from_lane(excl, src);
      if (get) {
        u.ox = ox; u.oy = oy; u.oz = oz;
        u.ix = ix; u.iy = iy; u.iz = iz;
        u.Sx = Sx; u.Sy = Sy;
        u.kx = pk & 3; u.ky = pk >> 2 & 3; u.kz = pk >> 4 & 3;
        u.Sz = sel3(ix, iy, iz, u.kz);     // (the largest component's reciprocal is not clamped)
        u.okx = sel3(ox, oy, oz, u.kx); u.oky = sel3(ox, oy, oz, u.ky); u.okz = sel3(ox, oy, oz, u.kz);
        ex = e;
        cur = nx;
        node = (pk & 64) ? S.root : EMPTY;
        sp = 0;
        bt = tb = tx;
        tbw = tx * T_WIDEN;
        best = -1;
        borig = INT32_MAX;
      }
      taken = min(nr, taken + (n_idle >> 2));
    }
    // inner nodes, until three eighths of the quads that were at one have left for a leaf or finished
    int left = __popcll(__ballot(node >= 0));
    const int enough = left * 5;
    while (left > 0) {
      if (node >= 0) {
        const float4 a = wide[(int64_t)node * 8], b = wide[(int64_t)node * 8 + 1];
        const int top = col[sp * QW];
        if (COUNT && q == 0) ++cn;
        // slab test; far distances widened by 1 + 2*gamma(3) (Ize 2013)
        // so that FP32 rounding never rejects a box that the exact ray meets
        const float up = 1.0f + 2.0f * 3.5762786865234375e-7f;   // 1 + 2 * gamma_3, gamma_n = n u / (1 - n u)
        const float lx = (a.x - u.ox) * u.ix, hx = (a.y - u.ox) * u.ix;
        const float ly = (a.z - u.oy) * u.iy, hy = (a.w - u.oy) * u.iy;
        const float lz = (b.x - u.oz) * u.iz, hz = (b.y - u.oz) * u.iz;
        const float tn = fmaxf(fmaxf(fminf(lx, hx), fminf(ly, hy)), fmaxf(fminf(lz, hz), tmin));
        const float tf = fminf(fminf(fmaxf(lx, hx), fmaxf(ly, hy)), fmaxf(lz, hz)) * up;
        const int child = __float_as_int(b.z);
        const bool h = (tn <= fminf(tf, tbw)) & (child != EMPTY);
        // rank among the quad's children by entry distance (tn >= 0: its bits are ordered; the low two bits
        // make the keys distinct); rank 0 comes next, the others go on the stack, the farthest lowest
        const uint32_t key = h ? (((uint32_t)__float_as_int(tn) & ~3u) | (uint32_t)q) : 0xffffffffu;
        const int rank = (int)((uint32_t)quad_perm<QP1>((int)key) < key) + (int)((uint32_t)quad_perm<QP2>((int)key) < key) +
                         (int)((uint32_t)quad_perm<QP3>((int)key) < key);
        const int c = quad_sum((int)h);
        if (h & (rank > 0)) {
          const int i = sp + c - rank;
          if (i <= st.cap) col[i * QW] = child;
          else ++st.overflow;
        }
        wave_order();   // (the quad's other lanes read the entry)
        const int first = quad_or((h && rank == 0) ? child : 0);
        node = c ? first : top;
        sp = min(sp + c - 1, st.cap);
      }
      left = __popcll(__ballot(node >= 0));
      if (left * 8 <= enough) break;
    }
    // leaves: a lane each, of the run of leaves on top of the quad's stack
    if (node < 0 && node != EMPTY) {
      const int e = q == 0 ? node : col[max(sp + 1 - q, 0) * QW];
      const bool lf = (e < 0) & (e != EMPTY);
      const int n0 = lf ? 0 : 1 << q;                       // bit q: the run ends before lane q
      const int run = __builtin_ctz(quad_or(n0) | 16);
      const int nxt = col[(sp + 1 - run) * QW];
      bool acc = false;
      if (q < run && ~e != ex) {
        const int64_t p = ~(int64_t)e;
        const float4 a = tri4[3 * p], b = tri4[3 * p + 1], c = tri4[3 * p + 2];
        const float tt = tri_test(a, b, c, u);
        const int orig = __float_as_int(a.w);
        acc = (tt > tmin) & (tt <= tb) & ((tt < bt) | (!any & (tt == bt) & (orig < borig)));
        if (acc) { bt = tt; borig = orig; best = ~e; }
      }
      if (COUNT && q < run) ++ct;
      sp -= run;
      node = nxt;
      tb = quad_min(bt);
      tbw = tb * T_WIDEN;
      if (any && quad_or((int)acc)) node = EMPTY;
    }
  }
  const int2 v = lane < nr ? res[lane] : make_int2(-1, 0);
  wave_order();   // (the next call's rays leave theirs there)
  pos = v.x;
  t = __int_as_float(v.y);
}

// Job tables reach the device through kernel arguments, a few jobs per launch, so that no
// host buffer has to outlive the call (and graph capture records the values).
constexpr int JOB_PACK = 8;
struct TraceJobPack {
  TraceJob j[JOB_PACK];
  int32_t first, n;
};
static_assert(sizeof(TraceJobPack) <= 4000, "job pack must fit the kernel argument space");

__global__ void k_put_trace_jobs(TraceJobPack pk, TraceJob* __restrict__ dst) {
  if ((int)threadIdx.x < pk.n) dst[pk.first + threadIdx.x] = pk.j[threadIdx.x];
}

__device__ inline double dnorm3(double x, double y, double z) { return sqrt(x * x + y * y + z * z); }

// carry: a later job wave of a batch; the totals of the statistics carry over.  misses: rays of a scene without
// triangles (every ray misses at its first segment).
__device__ inline void trace_init(Ctl* ctl, int64_t N, int carry, int64_t misses) {
  ctl->act[0] = N;
  ctl->base[0] = 0;
  if (carry) {
    ctl->rec_prev += ctl->rec_base;
  } else {
    ctl->rec_prev = 0;
    ctl->seg = 0;
    ctl->shadow = 0;
    ctl->overflow = 0;
    for (int i = 0; i < 6; ++i) ctl->cnt[i] = 0;
  }
  ctl->seg += misses;
  ctl->cnt[4] += misses;
  ctl->rec_base = 0;
  ctl->cmax_bits = 0;
  ctl->n_elig = 0;
  ctl->diff_kept = 0;
  ctl->n_groups = 0;
  ctl->n_draw = 0;
  for (int i = 0; i < 4; ++i) ctl->tot[i] = 0;
}

__global__ void k_trace_init(Ctl* ctl, int64_t N, int carry, int64_t misses) { trace_init(ctl, N, carry, misses); }

// The job of batch ray g (the last job with ray0 <= g; jobs without rays share ray0 with the next).
__device__ inline int ray_job(const TraceJob* __restrict__ jobs, int32_t J, int64_t g) {
  int lo = 0, hi = J - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (jobs[mid].ray0 <= g) lo = mid;
    else hi = mid - 1;
  }
  return lo;
}

constexpr int RAY_KEY_BITS = 16;   // direction cells of the ray sort: 2^16 on the octahedral map

__device__ inline uint32_t spread8(uint32_t v) {   // bit i -> bit 2i
  v = (v | (v << 4)) & 0x0F0Fu;
  v = (v | (v << 2)) & 0x3333u;
  v = (v | (v << 1)) & 0x5555u;
  return v;
}

// Sort key of ray g: Morton code of its world direction on the octahedral map (the top
// RAY_KEY_BITS of 8 + 8 bits), the job above it in a batch.  perm[g] = g (the sort's values).
template <bool BATCH>
__global__ void k_ray_keys(PoseArgs a0, const float* __restrict__ dirs0, const TraceJob* __restrict__ jobs, int32_t J,
                           uint32_t* __restrict__ keys, int32_t* __restrict__ perm) {
  const int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (g >= a0.N) return;
  const float* dirs = dirs0;
  double R[9];
#pragma unroll
  for (int k = 0; k < 9; ++k) R[k] = a0.R[k];
  int64_t li = g;
  uint32_t hi = 0;
  if (BATCH) {
    const int j = ray_job(jobs, J, g);
    dirs = jobs[j].dirs;
#pragma unroll
    for (int k = 0; k < 9; ++k) R[k] = jobs[j].a.R[k];
    li = g - jobs[j].ray0;
    hi = (uint32_t)j << RAY_KEY_BITS;
  }
  const float lx = dirs[3 * li], ly = dirs[3 * li + 1], lz = dirs[3 * li + 2];
  float x = (float)(R[0] * lx + R[1] * ly + R[2] * lz);
  float y = (float)(R[3] * lx + R[4] * ly + R[5] * lz);
  float z = (float)(R[6] * lx + R[7] * ly + R[8] * lz);
  const float s = fabsf(x) + fabsf(y) + fabsf(z);
  uint32_t ux = 0, uy = 0;
  if (s > 0.f && s < INFINITY) {
    x /= s; y /= s; z /= s;
    if (z < 0.f) {
      const float tx = (1.f - fabsf(y)) * (x >= 0.f ? 1.f : -1.f), ty = (1.f - fabsf(x)) * (y >= 0.f ? 1.f : -1.f);
      x = tx; y = ty;
    }
    ux = (uint32_t)fminf(fmaxf((x * 0.5f + 0.5f) * 256.f, 0.f), 255.f);
    uy = (uint32_t)fminf(fmaxf((y * 0.5f + 0.5f) * 256.f, 0.f), 255.f);
  }
  keys[g] = hi | ((spread8(ux) | (spread8(uy) << 1)) >> (16 - RAY_KEY_BITS));
  perm[g] = (int32_t)g;
}

// BATCH: a0.N is the batch's total ray count and each ray finds its job in the table.
// Slot i starts ray perm[i] (rays in key order).
template <bool BATCH>
__global__ void k_ray_init(PoseArgs a0, const float* __restrict__ dirs0, const TraceJob* __restrict__ jobs, int32_t J,
                           const int32_t* __restrict__ perm, TraceWS w, Ctl* ctl) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (!BATCH && i == 0) trace_init(ctl, a0.N, 0, 0);
  if (i >= a0.N) return;
  const int64_t g = perm ? perm[i] : i;
  PoseArgs a = a0;
  const float* dirs = dirs0;
  int64_t li = g;
  int32_t tag = (int32_t)g;
  if (BATCH) {
    const int j = ray_job(jobs, J, g);
    a = jobs[j].a;
    dirs = jobs[j].dirs;
    li = g - jobs[j].ray0;
    tag = j;
  }
  const double lx = dirs[3 * li], ly = dirs[3 * li + 1], lz = dirs[3 * li + 2];
  // CalculateWorldDirection: world = R * local, normalised in FP64
  double dx = a.R[0] * lx + a.R[1] * ly + a.R[2] * lz;
  double dy = a.R[3] * lx + a.R[4] * ly + a.R[5] * lz;
  double dz = a.R[6] * lx + a.R[7] * ly + a.R[8] * lz;
  double nrm = dnorm3(dx, dy, dz);
  if (!(nrm > 0.0) || !isfinite(nrm)) {
    atomicOr(&ctl->err, DEV_ERR_RAYDIR);
    nrm = 1.0;
    dx = 1.0; dy = 0.0; dz = 0.0;
  }
  w.st[0][i] = a.s[0]; w.st[1][i] = a.s[1]; w.st[2][i] = a.s[2];
  w.st[3][i] = dx / nrm; w.st[4][i] = dy / nrm; w.st[5][i] = dz / nrm;
  w.st[6][i] = 0.0;
  w.prev[i] = -1;
  w.ray[i] = tag;
}

// One launch per bounce (and a last one) walks two kinds of rays, each kind in whole waves: the closest hits of
// the act[j] active rays, and the line-of-sight rays of the records that bounce j - 1 left, which nothing
// waits for until the end.  A small pose is bound by the length of one walk after the other (16,384 rays: 48 us
// a bounce with both walks in one thread, and one line-of-sight ray per receiver made that 720 us for 8
// receivers); apart, the two walks of a ray run beside each other.
// The ray state is updated in place: slot s of the state holds the point, reflected direction, path length and
// leaf of the ray's last hit, which k_records copies into the record; act lists hold the slots that go on.
// Each wave leaves its 64 rays' hit and continue flags as two masks.
// BATCH: each ray reads its scene and pose from the job table (the ray field is the job).
// PERRX: one line-of-sight ray from the hit to each of the M receivers at rxp (bit m of the result) instead of one
// toward the pose's reference point.
// Six waves per SIMD (80 registers, 25 KB of stacks per 256 threads; the few spills lie outside the traversal loop):
// measured 4% faster on the room's pose and 7% on foliage's than five, 6% and 22% than four.
// A wave takes 1 << rs rays: 64 where there are waves enough to fill the chip, down to the 16 that its quads
// hold in a small pose.
// TB: threads per block: 64 while the rays leave compute units without a wave, else 256.
template <int TB, bool COUNT, bool BATCH, bool PERRX>
__global__ __launch_bounds__(TB) __attribute__((amdgpu_waves_per_eu(TRAV_WAVES_PER_SIMD))) void k_walk(
    SceneDev S0, PoseArgs a0, const TraceJob* __restrict__ jobs, TraceWS w, Ctl* ctl, et_paths P, int j, int last,
    int rs, const double* __restrict__ rxp, int32_t M) {
  __shared__ QuadLds<TB> lds;
  const int lane = threadIdx.x & 63;
  const int64_t n = last ? 0 : ctl->act[j];
  const int64_t r0 = j > 0 ? ctl->base[j - 1] : 0;
  const int64_t n_los = j > 0 ? (min(ctl->base[j], P.capacity) - r0) * (PERRX ? M : 1) : 0;
  const int64_t gtid = (int64_t)blockIdx.x * TB + threadIdx.x;
  const int64_t waves = (int64_t)gridDim.x * (TB / 64);
  const int R = 1 << rs;
  const int64_t nc = (n + R - 1) >> rs, nl = n_los > 0 ? (n_los + R - 1) >> rs : 0;
  const int32_t* list = j > 0 ? w.list[j & 1] : nullptr;
  QuadStack st{w.stack_cap, 0};
  lds.stack[threadIdx.x >> 2] = EMPTY;
  int64_t cn_c = 0, ct_c = 0, cn_a = 0, ct_a = 0, rays_a = 0;
  for (int64_t c = __builtin_amdgcn_readfirstlane((int)(gtid >> 6)); c < nc + nl; c += waves) {
    const bool los = c >= nc;
    const int64_t i0 = (los ? c - nc : c) << rs;
    const int nr = (int)min((int64_t)R, (los ? n_los : n) - i0);
    // the wave's rays, one per lane
    Ray32 ray{};
    bool walked = false;
    float tmax = INFINITY;
    int excl = -1, job = 0;
    if (lane < nr) {
      if (!los) {
        const int64_t s = list ? list[i0 + lane] : i0 + lane;
        if (BATCH) job = w.ray[s];
        ray = make_ray(w.st[0][s], w.st[1][s], w.st[2][s], w.st[3][s], w.st[4][s], w.st[5][s]);
        excl = w.prev[s];
        walked = !BATCH || jobs[job].S.T > 0;
      } else {
        // line of sight from a record's point toward the receiver reference point (or receiver m)
        const int64_t e = i0 + lane, rec = r0 + (PERRX ? e / M : e);
        const int m = PERRX ? (int)(e - (rec - r0) * M) : 0;
        if (BATCH) job = P.ray[rec];
        const PoseArgs& a = BATCH ? jobs[job].a : a0;
        const double px = P.p[3 * rec], py = P.p[3 * rec + 1], pz = P.p[3 * rec + 2];
        const double tx = PERRX ? rxp[3 * m] : a.xref[0], ty = PERRX ? rxp[3 * m + 1] : a.xref[1],
                     tz = PERRX ? rxp[3 * m + 2] : a.xref[2];
        const double wx = tx - px, wy = ty - py, wz = tz - pz;
        const double len = dnorm3(wx, wy, wz);
        if (len > 2.0 * a.t_eps) {
          excl = BATCH ? jobs[job].S.tri_pos[P.tri[rec]] : S0.tri_pos[P.tri[rec]];
          ray = make_ray(px, py, pz, wx / len, wy / len, wz / len);
          tmax = (float)(len - a.t_eps);
          walked = true;
          ++rays_a;
        }
      }
    }
    int pos;
    float th;
    int64_t cn = 0, ct = 0;
    if (!BATCH) {
      walk_rays<COUNT>(S0, ray, walked, (float)a0.t_eps, tmax, excl, nr, los, lds, st, pos, th, cn, ct);
    } else {
      // job after job (rays and records come in job order, so nearly every wave holds one)
      pos = -1;
      th = 0.f;
      for (uint64_t rest = __ballot(walked); rest;) {
        const int jb = __builtin_amdgcn_readlane(job, (int)__builtin_ctzll(rest));
        const bool mine = walked && job == jb;
        int p;
        float t;
        walk_rays<COUNT>(jobs[jb].S, ray, mine, (float)jobs[jb].a.t_eps, tmax, excl, nr, los, lds, st, p, t, cn, ct);
        if (mine) { pos = p; th = t; }
        rest &= ~__ballot(mine);
      }
    }
    if (COUNT) {
      cn_c += los ? 0 : cn; ct_c += los ? 0 : ct;
      cn_a += los ? cn : 0; ct_a += los ? ct : 0;
    }
    // The FP64 ray state (and a batch ray's job) is read again after the traversal instead of being held in
    // registers through it; the compiler barrier keeps the two reads apart, so the traversal loop runs
    // with fewer live registers (more waves per SIMD).
    __asm__ volatile("" ::: "memory");
    if (!los) {
      bool hit = false, cont = false;
      if (lane < nr && pos >= 0) {
        const int64_t s = list ? list[i0 + lane] : i0 + lane;
        SceneDev S = S0;
        PoseArgs a = a0;
        if (BATCH) {
          const TraceJob* tj = jobs + w.ray[s];
          S = tj->S;
          a = tj->a;
        }
        const double ox = w.st[0][s], oy = w.st[1][s], oz = w.st[2][s];
        const double dx = w.st[3][s], dy = w.st[4][s], dz = w.st[5][s];
        const double rtot = w.st[6][s];
        // FP64 refinement on the chosen triangle: plane intersection, normal, reflection
        const float4 A = S.tri4[3 * (int64_t)pos], Bv = S.tri4[3 * (int64_t)pos + 1], Cv = S.tri4[3 * (int64_t)pos + 2];
        const double e1x = (double)Bv.x - A.x, e1y = (double)Bv.y - A.y, e1z = (double)Bv.z - A.z;
        const double e2x = (double)Cv.x - A.x, e2y = (double)Cv.y - A.y, e2z = (double)Cv.z - A.z;
        double nx = e1y * e2z - e1z * e2y, ny = e1z * e2x - e1x * e2z, nz = e1x * e2y - e1y * e2x;
        const double nn = dnorm3(nx, ny, nz);
        nx /= nn; ny /= nn; nz /= nn;
        const double dn = dx * nx + dy * ny + dz * nz;
        const double hp = ((double)A.x - ox) * nx + ((double)A.y - oy) * ny + ((double)A.z - oz) * nz;
        const double t = dn != 0.0 ? hp / dn : (double)th;
        const double px = ox + t * dx, py = oy + t * dy, pz = oz + t * dz;
        const double rnew = (j == 0) ? dnorm3(px - a.s[0], py - a.s[1], pz - a.s[2]) : rtot + t;
        w.st[0][s] = px; w.st[1][s] = py; w.st[2][s] = pz;
        w.st[3][s] = dx - 2.0 * dn * nx; w.st[4][s] = dy - 2.0 * dn * ny; w.st[5][s] = dz - 2.0 * dn * nz;
        w.st[6][s] = rnew;
        w.prev[s] = pos;
        hit = true;
        cont = (j + 1 < a.B) && !(rnew >= a.maxd);
      }
      const uint64_t hm = __ballot(hit), cm = __ballot(cont);
      if (lane == 0) w.masks[c] = make_ulonglong2(hm, cm);
    } else if (lane < nr && pos < 0) {
      const int64_t e = i0 + lane, rec = r0 + (PERRX ? e / M : e);
      P.flags[rec] = 1;
      if (PERRX) atomicOr((unsigned long long*)&P.rx_vis[rec], 1ull << (int)(e - (rec - r0) * M));
    }
  }
  if (st.overflow) atomicAdd((unsigned long long*)&ctl->overflow, (unsigned long long)st.overflow);
  if (st.overflow) atomicOr(&ctl->err, DEV_ERR_STACK);
  if (COUNT) {
    atomicAdd((unsigned long long*)&ctl->cnt[0], (unsigned long long)cn_c);
    atomicAdd((unsigned long long*)&ctl->cnt[1], (unsigned long long)ct_c);
    atomicAdd((unsigned long long*)&ctl->cnt[2], (unsigned long long)cn_a);
    atomicAdd((unsigned long long*)&ctl->cnt[3], (unsigned long long)ct_a);
    atomicAdd((unsigned long long*)&ctl->cnt[5], (unsigned long long)rays_a);
  }
}

// Record counts of the finished trace.
__device__ inline void trace_final(Ctl* ctl, const et_paths& P, int diff, int32_t n_passive) {
  const int64_t spec = ctl->rec_base;
  const int64_t dk = diff ? (int64_t)ctl->tot[3] : 0;
  ctl->diff_kept = dk;
  const int64_t total = spec + dk + n_passive;
  P.count[0] = total;
  P.count[1] = spec;
  P.count[2] = dk;
  P.count[3] = ctl->seg;
}

// Hits (low half) and continuing rays (high half) of a wave's masks.
__device__ inline uint64_t mask_counts(ulonglong2 m) {
  return (uint64_t)__popcll(m.x) | (uint64_t)__popcll(m.y) << 32;
}

// Exclusive sums of the masks' counts within blocks of 1024, and the blocks' sums (more masks than
// SCAN_IN_PLACE, eight per thread of k_records' workgroups; fewer are summed by k_records itself).
constexpr int CHUNKS = 1024;
constexpr int64_t SCAN_IN_PLACE = 2048;
__global__ __launch_bounds__(BS) void k_mask_sums(TraceWS w, const Ctl* ctl, int j, int rs) {
  __shared__ uint64_t wsum[BS / 64];
  const int64_t nc = (ctl->act[j] + (1 << rs) - 1) >> rs;
  const int64_t c0 = (int64_t)blockIdx.x * CHUNKS + 4 * threadIdx.x;
  if ((int64_t)blockIdx.x * CHUNKS >= nc) return;
  uint64_t v[4], s = 0;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    v[k] = c0 + k < nc ? mask_counts(w.masks[c0 + k]) : 0;
    s += v[k];
  }
  uint64_t inc = s;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  for (int o = 1; o < 64; o <<= 1) {
    const uint64_t t = __shfl_up(inc, o);
    if (lane >= o) inc += t;
  }
  if (lane == 63) wsum[wv] = inc;
  __syncthreads();
  uint64_t ex = inc - s, tot = 0;
  for (int k = 0; k < BS / 64; ++k) {
    if (k < wv) ex += wsum[k];
    tot += wsum[k];
  }
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    if (c0 + k < nc) w.pre[c0 + k] = ex;
    ex += v[k];
  }
  if (threadIdx.x == 0) w.bsum[blockIdx.x] = tot;
}

__device__ inline uint64_t block_sum(uint64_t v, uint64_t* red) {
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  v = 0;
  for (int k = 0; k < BS / 64; ++k) v += red[k];
  __syncthreads();
  return v;
}

// The records of bounce j in ray order after the earlier bounces', the list of the slots that go on, and (last
// workgroup, which has no rays) the counts of the next bounce.  A workgroup takes 256 rays, the masks of 256 >> rs waves; what lies
// before them comes from k_mask_sums, or (IN_PLACE) from summing the masks before it.  fin: this is the last
// bounce and no other records follow.
template <bool BATCH, bool IN_PLACE>
__global__ __launch_bounds__(BS) void k_records(SceneDev S, const TraceJob* __restrict__ jobs, TraceWS w, Ctl* ctl,
                                                et_paths P, int j, int rs, int perrx, int fin) {
  __shared__ uint64_t red[BS / 64];
  const int64_t n = ctl->act[j], nc = (n + (1 << rs) - 1) >> rs;
  const int64_t base = ctl->base[j];
  const int32_t* list = j > 0 ? w.list[j & 1] : nullptr;
  int32_t* next = w.list[(j + 1) & 1];
  const unsigned groups = gridDim.x - 1;
  if (blockIdx.x == groups) {
    uint64_t t = 0;
    if (IN_PLACE) {
      for (int64_t c = threadIdx.x; c < nc; c += BS) t += mask_counts(w.masks[c]);
    } else {
      for (int64_t b = threadIdx.x; b < (nc + CHUNKS - 1) / CHUNKS; b += BS) t += w.bsum[b];
    }
    t = block_sum(t, red);
    if (threadIdx.x == 0) {
      const int64_t hits = (int64_t)(t & 0xffffffffull);
      ctl->seg += n;
      atomicAdd((unsigned long long*)&ctl->shadow, (unsigned long long)hits);   // (diffraction adds beside)
      ctl->cnt[4] += n;
      ctl->act[j + 1] = (int64_t)(t >> 32);
      ctl->base[j + 1] = base + hits;
      ctl->rec_base = base + hits;
      if (fin) trace_final(ctl, P, 0, 0);
    }
    return;
  }
  const int bit = threadIdx.x & ((1 << rs) - 1);
  for (int64_t i0 = (int64_t)blockIdx.x * BS; i0 < n; i0 += (int64_t)groups * BS) {
    const int64_t cb = i0 >> rs, c = cb + (threadIdx.x >> rs);   // the workgroup's first mask, this thread's
    uint64_t before;
    if (IN_PLACE) {
      uint64_t t = 0;
      for (int64_t k = threadIdx.x; k < cb; k += BS) t += mask_counts(w.masks[k]);
      before = block_sum(t, red);
      for (int64_t k = cb; k < c && k < nc; ++k) before += mask_counts(w.masks[k]);
    } else {
      uint64_t t = 0;
      const int64_t b = cb / CHUNKS;   // (a workgroup's masks share a block of sums)
      for (int64_t k = threadIdx.x; k < b; k += BS) t += w.bsum[k];
      before = block_sum(t, red);
      if (c < nc) before += w.pre[c];
    }
    const int64_t i = i0 + threadIdx.x;
    if (i >= n) continue;
    const ulonglong2 m = w.masks[c];
    const uint64_t below = (1ull << bit) - 1ull;
    if (!((m.x >> bit) & 1ull)) continue;
    const int64_t s = list ? list[i] : i;
    const int64_t ri = base + (int64_t)(before & 0xffffffffull) + __popcll(m.x & below);
    const int32_t* tri_orig = S.tri_orig;
    const int32_t* matp = S.mat;
    const int32_t tag = w.ray[s];
    if (BATCH) {
      const TraceJob* tj = jobs + tag;
      tri_orig = tj->S.tri_orig;
      matp = tj->S.mat;
    }
    const int orig = tri_orig[w.prev[s]];
    if (ri < P.capacity) {
      P.p[3 * ri] = w.st[0][s]; P.p[3 * ri + 1] = w.st[1][s]; P.p[3 * ri + 2] = w.st[2][s];
      P.dout[3 * ri] = (float)w.st[3][s]; P.dout[3 * ri + 1] = (float)w.st[4][s]; P.dout[3 * ri + 2] = (float)w.st[5][s];
      P.rtot[ri] = w.st[6][s];
      P.tri[ri] = orig;
      P.mat[ri] = matp[orig];
      P.ray[ri] = tag;
      P.bounce[ri] = (uint8_t)j;
      P.flags[ri] = 0;   // (set by the line-of-sight ray of the next launch)
      if (P.prev) P.prev[ri] = j > 0 ? w.prec[s] : -1;
      if (perrx) P.rx_vis[ri] = 0;
    } else {
      atomicOr(&ctl->err, DEV_ERR_CAPACITY);
    }
    if ((m.y >> bit) & 1ull) {
      next[(int64_t)(before >> 32) + __popcll(m.y & below)] = (int32_t)s;
      w.prec[s] = ri;
    }
  }
}

// ------------------------------------------------------------------ diffraction (Sec. III-D)
// Decisions that pick integers (eligibility, weights, CDF search, sample points, incidence
// test) are FP64 without contraction, in a fixed operation order.
#pragma clang fp contract(off)

__device__ inline uint64_t splitmix(uint64_t key, uint64_t counter) {
  uint64_t z = key + (counter + 1ull) * 0x9E3779B97F4A7C15ull;
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return z ^ (z >> 31);
}
__device__ inline double u01(uint64_t x) { return (double)(x >> 11) * 0x1p-53; }

struct DiffArgs {
  double s[3];
  double axis[3];
  double cone;
  double tau;
  double cos_max;
  uint64_t seed;
  int64_t K;            // draws (per mesh with per_mesh)
  double t_eps;
  int per_mesh;
  int64_t max_meshes;
  uint64_t rx_all;      // per-receiver reading: every receiver's bit (no receiver-side test), else 0
};

__global__ void k_obj_fov(SceneDev S, DiffArgs a, uint8_t* oel) {
  int o = blockIdx.x * blockDim.x + threadIdx.x;
  if (o >= S.n_obj) return;
  const float* b = S.obj_box + 6 * o;
  const double lx = b[0], ly = b[1], lz = b[2], hx = b[3], hy = b[4], hz = b[5];
  if (!(lx <= hx)) { oel[o] = 0; return; }
  const double cx = 0.5 * (lx + hx), cy = 0.5 * (ly + hy), cz = 0.5 * (lz + hz);
  const double ex = hx - lx, ey = hy - ly, ez = hz - lz;
  const double rad = 0.5 * sqrt(ex * ex + ey * ey + ez * ez);
  const double wx = cx - a.s[0], wy = cy - a.s[1], wz = cz - a.s[2];
  const double dist = sqrt(wx * wx + wy * wy + wz * wz);
  if (dist <= rad) { oel[o] = 1; return; }
  const double qx = wy * a.axis[2] - wz * a.axis[1], qy = wz * a.axis[0] - wx * a.axis[2],
               qz = wx * a.axis[1] - wy * a.axis[0];
  const double psi = atan2(sqrt(qx * qx + qy * qy + qz * qz), wx * a.axis[0] + wy * a.axis[1] + wz * a.axis[2]);
  oel[o] = psi <= a.cone + asin(rad / dist);
}

// Largest C_i over the triangles of eligible objects, as the bit pattern of a non-negative double
// (ordered like the value): a grid-strided maximum per thread, then per wave and per block, and
// one atomic per block (one per wave left the room's 193,212 triangles waiting on about 3000 atomics).
__global__ __launch_bounds__(BS) void k_cmax(SceneDev S, const uint8_t* __restrict__ oel, Ctl* ctl) {
  __shared__ long long wmax[BS / 64];
  long long v = 0;
  for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < S.T; t += (int64_t)gridDim.x * blockDim.x) {
    if (oel[S.obj[t]]) {
      const double c = S.C[t];
      if (c > 0.0) {
        const long long b = __double_as_longlong(c);
        v = b > v ? b : v;
      }
    }
  }
  for (int off = 32; off > 0; off >>= 1) {
    const long long o = __shfl_xor(v, off);
    v = o > v ? o : v;
  }
  if ((threadIdx.x & 63) == 0) wmax[threadIdx.x >> 6] = v;
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int i = 1; i < BS / 64; ++i) v = wmax[i] > v ? wmax[i] : v;
    if (v > 0) atomicMax((unsigned long long*)&ctl->cmax_bits, (unsigned long long)v);
  }
}

__global__ void k_qweight(SceneDev S, DiffArgs a, const uint8_t* __restrict__ oel, const Ctl* ctl,
                          uint64_t* __restrict__ q, uint64_t* __restrict__ flag) {
  int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= S.T) return;
  const double cmax = __longlong_as_double((long long)ctl->cmax_bits);
  const double c = S.C[t];
  uint64_t qq = 0;
  if (cmax > 0.0 && oel[S.obj[t]] && c > 0.0 && c >= a.tau * cmax) {
    // dithered integer weight: stochastic rounding of (C / Cmax) * 2^32
    const double x = c / cmax * 4294967296.0 + u01(splitmix(a.seed ^ 1ull, (uint64_t)t));
    qq = (uint64_t)floor(x);
  }
  q[t] = qq;
  flag[t] = qq > 0 ? 1ull : 0ull;
}

// Sort keys of the eligible triangles, listed in increasing index: weight descending (one
// CDF), or the mesh first and then weight descending (per mesh).  The radix sort is stable,
// so equal weights keep increasing indices without the index in the key (32 key bits, four
// passes, for one CDF).
__global__ void k_elig_keys(SceneDev S, int per_mesh, const uint64_t* __restrict__ q, const uint64_t* __restrict__ flag,
                            const uint64_t* __restrict__ offs, uint64_t* __restrict__ keys, int32_t* __restrict__ vals) {
  int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= S.T || !flag[t]) return;
  const int64_t p = (int64_t)offs[t];
  keys[p] = per_mesh ? ((uint64_t)S.obj[t] << 32) | (4294967296ull - q[t]) : (4294967296ull - q[t]);
  vals[p] = (int32_t)t;
}

__global__ void k_sorted_q(const uint64_t* __restrict__ keys, const Ctl* ctl, uint64_t* __restrict__ qs) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= ctl->n_elig) return;
  qs[i] = 4294967296ull - (keys[i] & 0xffffffffull);
}

// Group starts in the sorted list: a group per mesh.
__global__ void k_group_flags(const uint64_t* __restrict__ keys, const Ctl* ctl, uint64_t* __restrict__ flag) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= ctl->n_elig) return;
  flag[i] = (i == 0 || (keys[i] >> 32) != (keys[i - 1] >> 32)) ? 1ull : 0ull;
}

__global__ void k_group_starts(const uint64_t* __restrict__ flag, const uint64_t* __restrict__ rank, const Ctl* ctl,
                               int64_t* __restrict__ gstart) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < ctl->n_elig && flag[i]) gstart[rank[i]] = i;
}

// Group count and draws (one CDF: one group); more meshes than max_meshes keeps the first ones and reports a
// capacity error.  The last kept group ends where the first dropped one starts (its entry of
// gstart is already that start), so only an untruncated list gets the end marker n_elig.
__global__ void k_group_count(Ctl* ctl, DiffArgs a, int64_t* __restrict__ gstart) {
  int64_t g = a.per_mesh ? (int64_t)ctl->tot[2] : (ctl->n_elig > 0 ? 1 : 0);
  if (!a.per_mesh) gstart[0] = 0;
  if (a.per_mesh && g > a.max_meshes) {
    atomicOr(&ctl->err, DEV_ERR_CAPACITY);
    g = a.max_meshes;
  } else {
    gstart[g] = ctl->n_elig;
  }
  ctl->n_groups = g;
  ctl->n_draw = a.per_mesh ? a.K * g : (ctl->n_elig > 0 ? a.K : 0);
}

__global__ __launch_bounds__(BS) void k_diff_sample(SceneDev S, DiffArgs a, const uint64_t* __restrict__ W_ex,
                                                    const uint64_t* __restrict__ qs, const int32_t* __restrict__ vals,
                                                    TraceWS w, Ctl* ctl, int rs) {
  __shared__ QuadLds<BS> lds;
  const int lane = threadIdx.x & 63;
  const int64_t waves = (int64_t)gridDim.x * (BS / 64);
  QuadStack st{w.stack_cap, 0};
  lds.stack[threadIdx.x >> 2] = EMPTY;
  const int64_t n_draw = ctl->n_draw;
  int64_t dummy0 = 0, dummy1 = 0, rays = 0;
  const int first = __builtin_amdgcn_readfirstlane((int)(blockIdx.x * (BS / 64) + (threadIdx.x >> 6)));
  for (int64_t k0 = (int64_t)first << rs; k0 < n_draw; k0 += waves << rs) {
    const int nr = (int)min((int64_t)1 << rs, n_draw - k0);
    const int64_t k = k0 + lane;
    Ray32 ray{};
    bool ok = false;
    float tmax = INFINITY;
    int pos = -1;
    if (lane < nr) {
      // this draw's group (its mesh, or the one CDF) and the group's running sums
      const int64_t g = a.per_mesh ? k / a.K : 0;
      const int64_t j0 = w.gstart[g], j1 = w.gstart[g + 1];
      const uint64_t base = W_ex[j0], total = W_ex[j1 - 1] + qs[j1 - 1] - base;
      const uint64_t ks = a.seed ^ 2ull;
      const uint64_t U = splitmix(ks, 3ull * (uint64_t)k);
      const uint64_t idx = __umul64hi(U, total);
      // first position of the group whose inclusive running sum exceeds idx
      int64_t lo = j0, hi = j1;
      while (lo < hi) {
        const int64_t mid = (lo + hi) >> 1;
        if (W_ex[mid] + qs[mid] - base > idx) hi = mid; else lo = mid + 1;
      }
      const int32_t t = vals[lo];
      const double u1 = u01(splitmix(ks, 3ull * (uint64_t)k + 1ull)), u2 = u01(splitmix(ks, 3ull * (uint64_t)k + 2ull));
      const double su = sqrt(u1);
      const double wa = 1.0 - su, wb = su * (1.0 - u2), wc = su * u2;   // uniform point on the triangle
      pos = S.tri_pos[t];
      const float4 A = S.tri4[3 * (int64_t)pos], B = S.tri4[3 * (int64_t)pos + 1], C = S.tri4[3 * (int64_t)pos + 2];
      const double ax = A.x, ay = A.y, az = A.z, bx = B.x, by = B.y, bz = B.z, cx = C.x, cy = C.y, cz = C.z;
      const double ox = wa * ax + wb * bx + wc * cx, oy = wa * ay + wb * by + wc * cy, oz = wa * az + wb * bz + wc * cz;
      double nx = (by - ay) * (cz - az) - (bz - az) * (cy - ay);
      double ny = (bz - az) * (cx - ax) - (bx - ax) * (cz - az);
      double nz = (bx - ax) * (cy - ay) - (by - ay) * (cx - ax);
      const double nn = sqrt(nx * nx + ny * ny + nz * nz);
      const double inn = 1.0 / nn;
      nx = nx * inn; ny = ny * inn; nz = nz * inn;
      const double wx = a.s[0] - ox, wy = a.s[1] - oy, wz = a.s[2] - oz;
      const double L = sqrt(wx * wx + wy * wy + wz * wz);
      const double iL = 1.0 / L;
      const double vx = wx * iL, vy = wy * iL, vz = wz * iL;
      const double ci = fabs(nx * vx + ny * vy + nz * vz);
      ok = ci >= a.cos_max;                                        // incidence-angle constraint
      if (ok) {                                                    // line of sight to the source
        ray = make_ray(ox, oy, oz, vx, vy, vz);
        tmax = (float)(L - a.t_eps);
        ++rays;
      }
      w.stri[k] = t;
      w.so[3 * k] = ox; w.so[3 * k + 1] = oy; w.so[3 * k + 2] = oz;
      w.sr[k] = L;
    }
    int blk;
    float tv;
    walk_rays<false>(S, ray, ok, (float)a.t_eps, tmax, pos, nr, true, lds, st, blk, tv, dummy0, dummy1);
    if (lane < nr) w.skeep[k] = ok && blk < 0 ? 1ull : 0ull;
  }
  if (st.overflow) {
    atomicAdd((unsigned long long*)&ctl->overflow, (unsigned long long)st.overflow);
    atomicOr(&ctl->err, DEV_ERR_STACK);
  }
  // (one addition per wave: one per thread took most of this kernel's 100 us for 65,536 draws)
  for (int o = 32; o > 0; o >>= 1) rays += __shfl_xor(rays, o);
  if ((threadIdx.x & 63) == 0 && rays) atomicAdd((unsigned long long*)&ctl->shadow, (unsigned long long)rays);
}

__global__ void k_diff_scatter(SceneDev S, DiffArgs a, TraceWS w, Ctl* ctl, et_paths P) {
  const int64_t base = ctl->rec_base;
  const int64_t n_draw = ctl->n_draw;
  for (int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; k < n_draw; k += (int64_t)gridDim.x * blockDim.x) {
    if (!w.skeep[k]) continue;
    const int64_t ri = base + (int64_t)w.soffs[k];
    if (ri >= P.capacity) { atomicOr(&ctl->err, DEV_ERR_CAPACITY); continue; }
    const int32_t t = w.stri[k];
    P.p[3 * ri] = w.so[3 * k]; P.p[3 * ri + 1] = w.so[3 * k + 1]; P.p[3 * ri + 2] = w.so[3 * k + 2];
    P.dout[3 * ri] = 0.f; P.dout[3 * ri + 1] = 0.f; P.dout[3 * ri + 2] = 0.f;
    P.rtot[ri] = w.sr[k];
    P.tri[ri] = t;
    P.mat[ri] = S.mat[t];
    P.ray[ri] = (int32_t)k;
    P.bounce[ri] = 0;
    P.flags[ri] = 3;   // visible | diffraction
    if (P.prev) P.prev[ri] = -1;
    if (a.rx_all) P.rx_vis[ri] = a.rx_all;
  }
}

#pragma clang fp contract(on)

// Passive component: one line-of-sight ray from the emitter to each receiver (no triangle
// excluded) and one record per receiver after the specular and diffraction records: the
// emitter as the point, path 0, the receiver in `mat` and `ray`, kind 2 in the flags.
__global__ __launch_bounds__(BS) void k_passive(SceneDev S, PoseArgs a, const double* __restrict__ rx, int32_t M,
                                                int diff, TraceWS w, Ctl* ctl, et_paths P, int perrx) {
  __shared__ QuadLds<BS> lds;
  const int lane = threadIdx.x & 63;
  QuadStack st{w.stack_cap, 0};
  lds.stack[threadIdx.x >> 2] = EMPTY;
  const int64_t base = ctl->rec_base + (diff ? (int64_t)ctl->tot[3] : 0);
  int64_t dummy0 = 0, dummy1 = 0, rays = 0;
  const int64_t waves = (int64_t)gridDim.x * (BS / 64);
  const int first = __builtin_amdgcn_readfirstlane((int)(blockIdx.x * (BS / 64) + (threadIdx.x >> 6)));
  for (int64_t m0 = (int64_t)first << 4; m0 < M; m0 += waves << 4) {
    const int nr = (int)min((int64_t)16, M - m0);
    const int64_t m = m0 + lane;
    Ray32 ray{};
    bool walked = false;
    float tmax = INFINITY;
    if (lane < nr) {
      const double wx = rx[3 * m] - a.s[0], wy = rx[3 * m + 1] - a.s[1], wz = rx[3 * m + 2] - a.s[2];
      const double L = dnorm3(wx, wy, wz);
      if (L > 2.0 * a.t_eps && S.T > 0) {
        ray = make_ray(a.s[0], a.s[1], a.s[2], wx / L, wy / L, wz / L);
        tmax = (float)(L - a.t_eps);
        walked = true;
        ++rays;
      }
    }
    int pos;
    float tv;
    walk_rays<false>(S, ray, walked, (float)a.t_eps, tmax, -1, nr, true, lds, st, pos, tv, dummy0, dummy1);
    if (lane >= nr) continue;
    const int vis = pos < 0;
    const int64_t ri = base + m;
    if (ri < P.capacity) {
      P.p[3 * ri] = a.s[0]; P.p[3 * ri + 1] = a.s[1]; P.p[3 * ri + 2] = a.s[2];
      P.dout[3 * ri] = 0.f; P.dout[3 * ri + 1] = 0.f; P.dout[3 * ri + 2] = 0.f;
      P.rtot[ri] = 0.0;
      P.tri[ri] = -1;
      P.mat[ri] = (int32_t)m;
      P.ray[ri] = (int32_t)m;
      P.bounce[ri] = 0;
      P.flags[ri] = (uint8_t)(vis | 4);   // visible | kind 2
      if (P.prev) P.prev[ri] = -1;
      if (perrx) P.rx_vis[ri] = vis && m < 64 ? 1ull << m : 0ull;
    } else {
      atomicOr(&ctl->err, DEV_ERR_CAPACITY);
    }
  }
  if (st.overflow) {
    atomicAdd((unsigned long long*)&ctl->overflow, (unsigned long long)st.overflow);
    atomicOr(&ctl->err, DEV_ERR_STACK);
  }
  if (rays) atomicAdd((unsigned long long*)&ctl->shadow, (unsigned long long)rays);
}

__global__ void k_trace_final(Ctl* ctl, et_paths P, int diff, int32_t n_passive) { trace_final(ctl, P, diff, n_passive); }

inline size_t al(size_t b) { return (b + 255) / 256 * 256; }

}  // namespace

size_t trace_ws_layout(int64_t N, int64_t T, int32_t n_obj, int64_t K, char* base, TraceWS* w) {
  const int64_t Nm = std::max<int64_t>(N, 1), Tm = std::max<int64_t>(T, 1), Km = std::max<int64_t>(K, 1);
  size_t off = 0;
  auto take = [&](size_t bytes) -> void* {
    void* p = base ? (void*)(base + off) : nullptr;
    off += al(bytes);
    return p;
  };
  TraceWS x{};
  for (int k = 0; k < 7; ++k) x.st[k] = (double*)take(sizeof(double) * Nm);
  x.prev = (int32_t*)take(sizeof(int32_t) * Nm);
  x.ray = (int32_t*)take(sizeof(int32_t) * Nm);
  x.prec = (int64_t*)take(sizeof(int64_t) * Nm);
  for (int b = 0; b < 2; ++b) x.list[b] = (int32_t*)take(sizeof(int32_t) * Nm);
  // (small sets take down to 16 rays per wave)
  const int64_t waves = std::max<int64_t>((Nm + 63) / 64, std::min<int64_t>((Nm + 15) / 16, 2 * RS_WAVES));
  x.masks = (ulonglong2*)take(sizeof(ulonglong2) * waves);
  x.pre = (uint64_t*)take(sizeof(uint64_t) * waves);
  x.bsum = (uint64_t*)take(sizeof(uint64_t) * ((waves + CHUNKS - 1) / CHUNKS));
  x.scan_tmp = take(scan_temp_bytes(std::max(std::max(Nm, Tm), Km)));
  x.rkeys = (uint32_t*)take(sizeof(uint32_t) * Nm);
  x.rperm = (int32_t*)take(sizeof(int32_t) * Nm);
  x.rsort_tmp = take(sort_temp_bytes(Nm, 4));
  x.stack_cap = QUAD_STACK;
  if (K > 0) {
    x.oel = (uint8_t*)take((size_t)std::max<int32_t>(n_obj, 1));
    x.dkeys = (uint64_t*)take(sizeof(uint64_t) * Tm);
    x.dvals = (int32_t*)take(sizeof(int32_t) * Tm);
    x.dq = (uint64_t*)take(sizeof(uint64_t) * Tm);
    x.dflags = (uint64_t*)take(sizeof(uint64_t) * Tm);
    x.doffs = (uint64_t*)take(sizeof(uint64_t) * Tm);
    x.sort_tmp = take(sort_temp_bytes(Tm, 8));
    x.stri = (int32_t*)take(sizeof(int32_t) * Km);
    x.so = (double*)take(sizeof(double) * 3 * Km);
    x.sr = (double*)take(sizeof(double) * Km);
    x.skeep = (uint64_t*)take(sizeof(uint64_t) * Km);
    x.soffs = (uint64_t*)take(sizeof(uint64_t) * Km);
    x.goffs = (uint64_t*)take(sizeof(uint64_t) * Tm);
    x.gstart = (int64_t*)take(sizeof(int64_t) * (Tm + 1));
  }
  if (w) *w = x;
  return off;
}

namespace {
// Threads of k_walk that the current device holds at once (blocks per compute unit
// at its occupancy, times the compute units), queried once per device.
int64_t bounce_resident_threads() {
  static std::atomic<int64_t> cache[64];
  int dev = 0;
  ET_HIP(hipGetDevice(&dev));
  std::atomic<int64_t>* slot = (dev >= 0 && dev < 64) ? &cache[dev] : nullptr;
  if (slot) {
    const int64_t v = slot->load(std::memory_order_relaxed);
    if (v > 0) return v;
  }
  int per_cu = 0, cus = 0;
  ET_HIP(hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_walk<BS, false, false, false>, BS, 0));
  ET_HIP(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
  const int64_t v = std::max<int64_t>(1, (int64_t)per_cu * cus) * BS;
  if (slot) slot->store(v, std::memory_order_relaxed);
  return v;
}

// A bounce's walk: tb threads per block.
template <bool BATCH, bool PERRX>
void launch_walk(int tb, bool counting, unsigned blocks, hipStream_t s, const SceneDev& S, const PoseArgs& a,
                 const TraceJob* jobs, const TraceWS& w, Ctl* ctl, const et_paths& P, int j, int last, int rs,
                 const double* rx, int32_t M) {
  if (tb == 64) {
    if (counting) k_walk<64, true, BATCH, PERRX><<<blocks, 64, 0, s>>>(S, a, jobs, w, ctl, P, j, last, rs, rx, M);
    else k_walk<64, false, BATCH, PERRX><<<blocks, 64, 0, s>>>(S, a, jobs, w, ctl, P, j, last, rs, rx, M);
  } else {
    if (counting) k_walk<BS, true, BATCH, PERRX><<<blocks, BS, 0, s>>>(S, a, jobs, w, ctl, P, j, last, rs, rx, M);
    else k_walk<BS, false, BATCH, PERRX><<<blocks, BS, 0, s>>>(S, a, jobs, w, ctl, P, j, last, rs, rx, M);
  }
}

// The records of bounce j and the next bounce's list and counts; N: the most rays.
template <bool BATCH>
void launch_records(int64_t N, const SceneDev& S, const TraceJob* jobs, const TraceWS& w, Ctl* ctl, const et_paths& P, int j,
                    int rs, int perrx, int fin, hipStream_t s) {
  const int64_t masks = (N + (1 << rs) - 1) >> rs;
  if (masks <= SCAN_IN_PLACE) {
    k_records<BATCH, true><<<nblk(N) + 1, BS, 0, s>>>(S, jobs, w, ctl, P, j, rs, perrx, fin);
  } else {
    k_mask_sums<<<(unsigned)((masks + CHUNKS - 1) / CHUNKS), BS, 0, s>>>(w, ctl, j, rs);
    k_records<BATCH, false><<<nblk(N) + 1, BS, 0, s>>>(S, jobs, w, ctl, P, j, rs, perrx, fin);
  }
}

PoseArgs pose_args(const et_sim_desc* sim) {
  PoseArgs a;
  for (int k = 0; k < 3; ++k) { a.s[k] = sim->emitter_pos[k]; a.xref[k] = sim->x_ref[k]; }
  for (int k = 0; k < 9; ++k) a.R[k] = sim->emitter_rot[k];
  a.N = (sim->flags & ET_SPECULAR) ? sim->N : 0;
  a.B = sim->max_bounces;
  a.maxd = sim->max_distance;
  a.t_eps = sim->t_eps;
  return a;
}
}  // namespace

size_t trace_batch_jobs_bytes(int32_t J) { return sizeof(TraceJob) * (size_t)std::max(J, 1); }

int64_t trace_batch_rays(int32_t J, const et_job* jobs) {
  int64_t n = 0;
  for (int32_t i = 0; i < J; ++i) n += (jobs[i].sim->flags & ET_SPECULAR) ? jobs[i].sim->N : 0;
  return n;
}

void trace_batch_run(int32_t J, const et_job* jobs, void* dev_jobs, const et_paths* paths, const TraceWS& w,
                     Ctl* ctl, bool counting, int32_t blocks, hipStream_t s, bool carry) {
  TraceJob* dj = (TraceJob*)dev_jobs;
  TraceJobPack pk{};
  int64_t N = 0;
  int B = 0;
  for (int32_t i = 0; i < J; ++i) {
    TraceJob& t = pk.j[pk.n++];
    t.S = jobs[i].scene->d;
    t.a = pose_args(jobs[i].sim);
    t.dirs = jobs[i].sim->ray_dirs;
    t.ray0 = N;
    N += t.a.N;
    B = std::max(B, (int)t.a.B);
    if (pk.n == JOB_PACK || i + 1 == J) {
      k_put_trace_jobs<<<1, JOB_PACK, 0, s>>>(pk, dj);
      pk.first += pk.n;
      pk.n = 0;
    }
  }
  PoseArgs all{};
  all.N = N;
  const et_paths P = *paths;
  k_trace_init<<<1, 1, 0, s>>>(ctl, N, carry ? 1 : 0, 0);
  ET_HIP(hipGetLastError());
  // walks' grid: the tuned block count
  const int64_t cap_blocks = std::max<int64_t>(1, blocks);
  const unsigned gb = (unsigned)std::max<int64_t>(1, std::min<int64_t>((N + BS - 1) / BS, cap_blocks));
  if (N > 0) {
    const bool sorted = N > (int64_t)gb * BS;
    if (sorted) {
      int jb = 0;
      while ((1ll << jb) < (int64_t)J) ++jb;
      k_ray_keys<true><<<nblk_full(N), BS, 0, s>>>(all, nullptr, dj, J, w.rkeys, w.rperm);
      radix_sort_u32(w.rkeys, w.rperm, N, RAY_KEY_BITS + jb, w.rsort_tmp, s);
    }
    k_ray_init<true><<<nblk_full(N), BS, 0, s>>>(all, nullptr, dj, J, sorted ? w.rperm : nullptr, w, ctl);
    for (int j = 0; j <= B; ++j) {
      launch_walk<true, false>(64, counting, gb * (BS / 64), s, SceneDev{}, all, dj, w, ctl, P, j, j == B, 6, nullptr, 0);
      if (j < B) launch_records<true>(N, SceneDev{}, dj, w, ctl, P, j, 6, 0, 0, s);
    }
    ET_HIP(hipGetLastError());
  }
  k_trace_final<<<1, 1, 0, s>>>(ctl, P, 0, 0);
  ET_HIP(hipGetLastError());
}

void trace_run(const SceneDev& S, const et_sim_desc* sim, const et_paths* paths, const TraceWS& w, Ctl* ctl,
               bool counting, hipStream_t s, const SideStream* side) {
  const PoseArgs a = pose_args(sim);
  const et_paths P = *paths;
  const bool perrx = (sim->flags & ET_PER_RX_VISIBILITY) != 0;
  const bool diff = (sim->flags & ET_DIFFRACTION) && sim->diff_K > 0 && S.T > 0;
  const int32_t n_passive = (sim->flags & ET_PASSIVE) ? sim->M : 0;
  const bool fin = !diff && n_passive == 0 && a.N > 0 && S.T > 0;   // the last bounce's records end the trace
  if (a.N > 0 && S.T > 0) {
    const bool sorted = a.N > bounce_resident_threads() || a.N > (int64_t)nblk(a.N) * BS;
    if (sorted) {
      k_ray_keys<false><<<nblk_full(a.N), BS, 0, s>>>(a, sim->ray_dirs, nullptr, 0, w.rkeys, w.rperm);
      radix_sort_u32(w.rkeys, w.rperm, a.N, RAY_KEY_BITS, w.rsort_tmp, s);
    }
    k_ray_init<false><<<nblk_full(a.N), BS, 0, s>>>(a, sim->ray_dirs, nullptr, 0, sorted ? w.rperm : nullptr, w, ctl);
    // The diffraction samples depend on the pose alone, so with a side stream they are drawn beside the walks, which
    // leave compute units idle in a small pose (some twenty launches of 2 to 10 us: 50,003 rays in the
    // room with samples on 61 meshes 500 us in order, 382 us beside; an animated frame 980 and 847 us).
    if (diff && side) ET_HIP(hipEventRecord(side->fork, s));
    // walks' grid: whole rounds of resident blocks (no partly filled last round), the chunks taken by grid
    // stride (2^20 rays, room and foliage pose: 12.10 and 8.30 ms; a block per four chunks 12.20 and 8.48; one round
    // 12.48 and 8.81)
    const double* rx = perrx ? sim->rx_pos : nullptr;
    const int32_t M = perrx ? sim->M : 1;
    const int64_t res_blocks = std::max<int64_t>(1, bounce_resident_threads() / BS);
    // rays per wave: the most that leaves RS_WAVES waves (two and a half per SIMD), from 64 down to 16
    const int64_t most = a.N * (1 + M);
    int rs = 6;
    while (rs > 4 && (most >> rs) < RS_WAVES) --rs;
    for (int j = 0; j <= a.B; ++j) {
      // closest hits of at most N rays and the line-of-sight rays of as many records
      const int64_t waves = (((j < a.B ? a.N : 0) + (j > 0 ? a.N * M : 0)) >> rs) + 2;
      const int64_t nb = std::min<int64_t>((waves + BS / 64 - 1) / (BS / 64), MAX_BLOCKS);
      const int tb = waves <= 4 * res_blocks / TRAV_WAVES_PER_SIMD ? 64 : BS;
      const unsigned gb = (unsigned)(tb == 64 ? waves : nb > res_blocks ? nb / res_blocks * res_blocks : nb);
      if (perrx) launch_walk<false, true>(tb, counting, gb, s, S, a, nullptr, w, ctl, P, j, j == a.B, rs, rx, M);
      else launch_walk<false, false>(tb, counting, gb, s, S, a, nullptr, w, ctl, P, j, j == a.B, rs, rx, M);
      if (j < a.B) launch_records<false>(a.N, S, nullptr, w, ctl, P, j, rs, perrx ? 1 : 0, fin && j + 1 == a.B, s);
    }
    ET_HIP(hipGetLastError());
  } else {
    // no rays, or an empty scene: every ray misses at its first segment
    k_trace_init<<<1, 1, 0, s>>>(ctl, a.N, 0, a.N);
    ET_HIP(hipGetLastError());
  }
  if (diff) {
    if (!(a.N > 0)) side = nullptr;   // (nothing to run beside)
    const hipStream_t main = s;
    if (side) {
      ET_HIP(hipStreamWaitEvent(side->stream, side->fork, 0));
      s = side->stream;
    }
    DiffArgs d;
    for (int k = 0; k < 3; ++k) { d.s[k] = sim->emitter_pos[k]; d.axis[k] = sim->emitter_rot[3 * k]; }
    d.cone = sim->diff_cone_half_angle;
    d.tau = sim->diff_tau;
    d.cos_max = std::cos(sim->diff_max_incidence);
    d.seed = sim->diff_seed;
    d.K = sim->diff_K;
    d.t_eps = sim->t_eps;
    d.per_mesh = (sim->flags & ET_DIFF_PER_MESH) ? 1 : 0;
    d.rx_all = perrx ? (sim->M >= 64 ? ~0ull : (1ull << sim->M) - 1ull) : 0ull;
    d.max_meshes = d.per_mesh ? sim->diff_max_meshes : 1;
    const int64_t max_draw = d.K * d.max_meshes;
    int obj_bits = 1;
    while (obj_bits < 31 && ((int64_t)1 << obj_bits) < S.n_obj) ++obj_bits;
    k_obj_fov<<<nblk_full(S.n_obj), BS, 0, s>>>(S, d, w.oel);
    k_cmax<<<(unsigned)std::min<int64_t>(nblk_full(S.T), 256), BS, 0, s>>>(S, w.oel, ctl);
    k_qweight<<<nblk_full(S.T), BS, 0, s>>>(S, d, w.oel, ctl, w.dq, w.dflags);
    scan_exclusive_u64(w.dflags, w.doffs, S.T, nullptr, S.T, (uint64_t*)&ctl->n_elig, w.scan_tmp, s);
    k_elig_keys<<<nblk_full(S.T), BS, 0, s>>>(S, d.per_mesh, w.dq, w.dflags, w.doffs, w.dkeys, w.dvals);
    radix_sort_u64(w.dkeys, w.dvals, 0, &ctl->n_elig, S.T, d.per_mesh ? 32 + obj_bits : 32, w.sort_tmp, s);
    // weights in sorted order, then their exclusive prefix sums (the CDF) and total
    k_sorted_q<<<nblk_full(S.T), BS, 0, s>>>(w.dkeys, ctl, w.dq);
    scan_exclusive_u64(w.dq, w.doffs, 0, &ctl->n_elig, S.T, nullptr, w.scan_tmp, s);
    // groups of the sorted list (meshes, or one) and the number of draws
    if (d.per_mesh) {
      k_group_flags<<<nblk_full(S.T), BS, 0, s>>>(w.dkeys, ctl, w.dflags);
      scan_exclusive_u64(w.dflags, w.goffs, 0, &ctl->n_elig, S.T, &ctl->tot[2], w.scan_tmp, s);
      k_group_starts<<<nblk_full(S.T), BS, 0, s>>>(w.dflags, w.goffs, ctl, w.gstart);
    }
    k_group_count<<<1, 1, 0, s>>>(ctl, d, w.gstart);
    int rs = 6;
    while (rs > 4 && (max_draw >> rs) < RS_WAVES) --rs;
    k_diff_sample<<<nblk(max_draw << (6 - rs)), BS, 0, s>>>(S, d, w.doffs, w.dq, w.dvals, w, ctl, rs);
    scan_exclusive_u64(w.skeep, w.soffs, 0, &ctl->n_draw, max_draw, &ctl->tot[3], w.scan_tmp, s);
    if (side) {
      ET_HIP(hipEventRecord(side->join, s));
      ET_HIP(hipStreamWaitEvent(main, side->join, 0));
      s = main;
    }
    k_diff_scatter<<<nblk(max_draw), BS, 0, s>>>(S, d, w, ctl, P);   // (after the walks' records)
    ET_HIP(hipGetLastError());
  }
  if (n_passive > 0)
    k_passive<<<nblk(4 * (int64_t)n_passive), BS, 0, s>>>(S, a, sim->rx_pos, n_passive, diff ? 1 : 0, w, ctl, P, perrx ? 1 : 0);
  if (!fin) k_trace_final<<<1, 1, 0, s>>>(ctl, P, diff ? 1 : 0, n_passive);
  ET_HIP(hipGetLastError());
}

}  // namespace et
