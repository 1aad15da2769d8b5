// Echo synthesis (Eqs. 2-4 specular, 7-8 diffraction) and its adjoint.
//
// For record n (point p, path rtot to it, reflected direction d', material q) and receiver
// m at x_m, with r = rtot + |x_m - p| and f_k = f_lo + k df:
//   H_m[k] += A_nmk exp(j 2 pi sigma f_k r / c)
//   A_nmk = r^-p 10^(-(a0 + a1 f_k) r / 20) * I[b(k)] * D_m[bd(k)]
//   I[b] = k_qb exp(-gamma^2 / (2 beta_qb^2)) (specular),  I_d,qb (diffraction),  I_p,b (passive)
// where gamma is the angle between d' and the direction from p to x_m.  Records whose
// line-of-sight ray was blocked contribute nothing; a first pass compacts the indices of
// the visible records so that no kernel spends work on the others.  Two alternative
// readings switch per pose: the path product (k_qb replaced by the product of k over the
// ray's reflections so far, through per-record band tables) and per-receiver line of sight
// (a record reaches receiver m only when its bit m is set).
//
// Precision: the receiver leg, total path and the delay in cycles at f_lo and per bin are
// FP64 (the phase needs the path to ~1e-8 m at 100-200 kHz); sin/cos/exp2 and the
// accumulation are FP32 (v_sin/v_cos take revolutions, so the FP64 reduction hands them
// a fraction of a cycle).
//
// Three kernels compute the same sum.  With k = 64 k1 + k2, amplitude and phase separate as
//   A e^{j phi} = X[n,k1] * Y[n,k2],
//   X = exp2(base + 64 k1 slope + band(k1)) e^{j 2 pi (c0 + 64 k1 cb)},
//   Y = exp2(k2 slope) e^{j 2 pi k2 cb},
// where the material/directivity bands are constant over a run of 64 bins, so
// H_m[k1, k2] = sum_n X[n,k1] Y[n,k2] is a complex matrix product contracting over the records.  X and Y themselves
// come from 32 exp2/sin/cos factors per (record, receiver) (a second 8 x 8 split) plus the band factors, so only
// about 40 transcendental triples remain of the 4096 per (record, receiver) of a 4096-bin grid.
//  * k_synth_mfma (bands on whole runs of 64 bins): on the f16 matrix cores (v_mfma_f32_32x32x16_f16), every FP32
//    operand split into two f16 halves and three half products per real product, FP32 accumulation.
//  * k_synth_rows (other layouts): rows cut at the band edges, on the FP32 matrix cores (v_mfma_f32_32x32x2_f32).
//  * k_synth_direct (many bands in few bins, or asked for): one sin/cos/exp2 per (record, receiver, bin).
// Each writes per-chunk partial spectra that a final kernel sums in a fixed order
// (bit-reproducible results).
#include "internal.hpp"

#include <algorithm>
#include <cmath>
#include <vector>

namespace et {

namespace {

constexpr double LOG2_10 = 3.32192809488736234787;
constexpr float LOG2E_F = 1.44269504088896340736f;
constexpr float PI_F = 3.14159265358979323846f;

struct SynthArgs {
  int32_t M, F, Q, Bk, Bd, El, Az, sigma;
  double f_lo, df, c, A0, A1, ps;
  const double* rx_pos;
  const double* rx_rot;
  const float* refl_k;
  const float* beta;
  const float* dcoef;
  const float* dir;
  int32_t P;               // record chunks
  double kc0, kcb;         // sigma f_lo / c and sigma df / c: cycles per metre of path
  double kbase, kslope;    // log2 absorption per metre at f_lo and per bin
  const float* lk;         // [Q][Bk] log2 k
  const float* lc;         // [Q][Bk] log2(e) / (2 beta^2)
  const float* ld;         // [Q][Bk] log2 I_d
  const float* pcoef;      // [Bk] passive source magnitude I_p (NULL without the passive component)
  const float* lp;         // [Bk] log2 I_p
  const float* lmax;       // [3 Q + 1] per material: max_b log2 k, min_b lobe coefficient, max_b log2 I_d;
                           // then max_b log2 I_p (bounds on the band factors, used with rec_rows 0)
  int32_t rec_rows;        // 1 (path-product reading): lk, lc, ld have a row per record and a
                           // record's `mat` in the kernels is its index; 0: a row per material
  const uint64_t* rxv;     // per-receiver line of sight [records] (NULL: the records' visible bit)
  const int2* rows;        // [nrows + 1] row table (FOLD 0): first bin and bands of each row, then F
  int32_t nrows;
};

constexpr int K2 = 64;        // bins per inner run (k = 64 k1 + k2)
constexpr int KT1 = 64;       // rows per workgroup
constexpr int SMAX = 16;      // band segments (runs of equal material and directivity band) per tile of rows

// Rows of the factorised kernels: runs of bins within one block of 64 (an outer index) and within
// one material and one directivity band, so a row starts at every multiple of 64 and at every band
// edge.  With the band edges on multiples of 64 bins the rows are the outer indices; otherwise an
// outer index that holds an edge has a row per band, each computing the 64 bins and keeping its own.
// Returns their number; *max_seg (optional): the most band segments in a tile of KT1 rows.
int synth_rows(const et_sim_desc* sim, int* max_seg) {
  const int64_t F = sim->F;
  std::vector<int64_t> edge;   // first bin of every band but the first
  for (int pass = 0; pass < 2; ++pass) {
    const int64_t B = pass == 0 ? sim->Bk : (sim->directivity ? sim->Bd : 0);
    for (int64_t b = 1; b < B; ++b) {
      const int64_t k = (b * F + B - 1) / B;
      if (k > 0 && k < F) edge.push_back(k);
    }
  }
  std::sort(edge.begin(), edge.end());
  edge.erase(std::unique(edge.begin(), edge.end()), edge.end());
  int64_t rows = (F + K2 - 1) / K2;
  for (int64_t e : edge) rows += (e % K2) != 0;
  if (max_seg) {
    // segments of the tile that starts at each row: band edges among its rows, and the first one
    int most = 1, seg = 1;
    int64_t v = 0, k = 0;
    size_t ie = 0;
    while (k < F) {
      if (v % KT1 == 0) seg = 1;
      else if (ie > 0 && edge[ie - 1] == k) ++seg;
      most = std::max(most, seg);
      int64_t next = (k / K2 + 1) * K2;
      if (ie < edge.size() && edge[ie] <= next) next = edge[ie++];
      k = next;
      ++v;
    }
    *max_seg = most;
  }
  return (int)std::min<int64_t>(rows, INT32_MAX);
}

SynthArgs make_args(const et_sim_desc* sim, int32_t P) {
  SynthArgs a;
  a.M = sim->M; a.F = sim->F; a.Q = sim->Q; a.Bk = sim->Bk;
  a.Bd = sim->directivity ? sim->Bd : 0;
  a.El = sim->El; a.Az = sim->Az;
  a.sigma = sim->phase_sign;
  a.f_lo = sim->f_lo;
  a.df = sim->F > 1 ? (sim->f_hi - sim->f_lo) / (double)(sim->F - 1) : 0.0;
  a.c = sim->c; a.A0 = sim->atm_a0; a.A1 = sim->atm_a1; a.ps = sim->spreading_p;
  a.rx_pos = sim->rx_pos; a.rx_rot = sim->rx_rot;
  a.refl_k = sim->refl_k; a.beta = sim->lobe_beta; a.dcoef = sim->diff_coef;
  a.dir = sim->directivity;
  a.P = P;
  a.kc0 = (double)a.sigma * a.f_lo / a.c;
  a.kcb = (double)a.sigma * a.df / a.c;
  a.kbase = -(a.A0 + a.A1 * a.f_lo) / 20.0 * LOG2_10;
  a.kslope = -a.A1 * a.df / 20.0 * LOG2_10;
  a.pcoef = (sim->flags & ET_PASSIVE) ? sim->passive_coef : nullptr;
  a.lk = a.lc = a.ld = a.lp = a.lmax = nullptr;
  a.rec_rows = 0;
  a.rxv = nullptr;
  a.rows = nullptr;
  a.nrows = synth_rows(sim, nullptr);
  return a;
}

// Per (record, receiver) quantities shared by every bin.
struct Pair {
  double c0, cb;     // delay in cycles at f_lo and per bin
  float base;        // log2 amplitude at f_lo without band factors
  float slope;       // log2 amplitude change per bin
  double base64, slope64;
  double r, l;
  double u[3];
  float gamma;
  int mat;           // row of the band tables: the material, or the record (rec_rows)
  int kind;
};

// Cell of the cell-centred directivity grid that a direction of arrival falls into: offsets of its
// two elevation rows and azimuth columns and the weights of the bilinear interpolation.
struct DirCell {
  int r0, r1, i0, i1;   // row offsets (row times Az) and columns
  float ta, te;
};

__device__ inline DirCell dir_cell(int El, int Az, float vx, float vy, float vz) {
  const float az = atan2f(vy, vx);
  const float el = atan2f(vz, hypotf(vx, vy));
  float fa = (az + PI_F) / (2.0f * PI_F) * (float)Az - 0.5f;
  float fe = (el + 0.5f * PI_F) / PI_F * (float)El - 0.5f;
  if (!(fa == fa)) fa = 0.f;   // undefined direction (receiver on the point): any cell, indices stay in range
  if (!(fe == fe)) fe = 0.f;
  DirCell c;
  const float fl = floorf(fa);
  c.ta = fa - fl;
  c.i0 = (int)fl % Az;
  if (c.i0 < 0) c.i0 += Az;
  c.i1 = (c.i0 + 1) % Az;
  int j0, j1;
  if (fe <= 0.f) { j0 = j1 = 0; c.te = 0.f; }
  else if (fe >= (float)(El - 1)) { j0 = j1 = El - 1; c.te = 0.f; }
  else { j0 = min((int)floorf(fe), El - 1); j1 = min(j0 + 1, El - 1); c.te = fe - (float)j0; }
  c.r0 = j0 * Az;
  c.r1 = j1 * Az;
  return c;
}

template <typename T>
__device__ inline float dir_lerp(const T* tab, const DirCell& c) {
  const float a0 = (1.f - c.ta) * tab[c.r0 + c.i0] + c.ta * tab[c.r0 + c.i1];
  const float a1 = (1.f - c.ta) * tab[c.r1 + c.i0] + c.ta * tab[c.r1 + c.i1];
  return (1.f - c.te) * a0 + c.te * a1;
}

__device__ inline float dir_gain(const float* tab, int El, int Az, float vx, float vy, float vz) {
  return dir_lerp(tab, dir_cell(El, Az, vx, vy, vz));
}

// The gain of dir_gain and its gradient (gx, gy, gz) with respect to the direction v: the
// derivative of the bilinear interpolant inside the cell that holds v, through
// fa = (az + pi) Az / 2pi - 1/2, fe = (el + pi/2) El / pi - 1/2, az = atan2(y, x) and
// el = atan2(z, rho); zero across the clamped elevation rows and on the poles.
__device__ inline float dir_gain_dv(const float* tab, int El, int Az, float vx, float vy, float vz, float& gx,
                                    float& gy, float& gz) {
  const float az = atan2f(vy, vx);
  const float rho2 = vx * vx + vy * vy, rho = sqrtf(rho2);
  const float el = atan2f(vz, rho);
  float fa = (az + PI_F) / (2.0f * PI_F) * (float)Az - 0.5f;
  float fe = (el + 0.5f * PI_F) / PI_F * (float)El - 0.5f;
  if (!(fa == fa)) fa = 0.f;
  if (!(fe == fe)) fe = 0.f;
  const float fl = floorf(fa);
  const float ta = fa - fl;
  int i0 = (int)fl % Az;
  if (i0 < 0) i0 += Az;
  const int i1 = (i0 + 1) % Az;
  int j0, j1;
  float te;
  bool inner = false;
  if (fe <= 0.f) { j0 = j1 = 0; te = 0.f; }
  else if (fe >= (float)(El - 1)) { j0 = j1 = El - 1; te = 0.f; }
  else { j0 = min((int)floorf(fe), El - 1); j1 = min(j0 + 1, El - 1); te = fe - (float)j0; inner = true; }
  const float t00 = tab[j0 * Az + i0], t01 = tab[j0 * Az + i1], t10 = tab[j1 * Az + i0], t11 = tab[j1 * Az + i1];
  const float a0 = (1.f - ta) * t00 + ta * t01;
  const float a1 = (1.f - ta) * t10 + ta * t11;
  const float daz = ((1.f - te) * (t01 - t00) + te * (t11 - t10)) * (float)Az / (2.0f * PI_F);
  const float del = inner ? (a1 - a0) * (float)El / PI_F : 0.f;
  const float n2 = rho2 + vz * vz;
  if (rho2 > 0.f && n2 > 0.f) {
    gx = -daz * vy / rho2 - del * vx * vz / (rho * n2);
    gy = daz * vx / rho2 - del * vy * vz / (rho * n2);
    gz = del * rho / n2;
  } else {
    gx = gy = gz = 0.f;
  }
  return (1.f - te) * a0 + te * a1;
}

// Returns false if the record does not contribute to receiver m (not visible, hidden from
// receiver m under the per-receiver line of sight, or a passive record of another receiver).
__device__ inline bool pair_setup(const SynthArgs& a, const et_paths& P, int64_t n, int m, Pair& q) {
  const uint8_t fl = P.flags[n];
  if (!(fl & 1)) return false;
  if (a.rxv && !((a.rxv[n] >> m) & 1ull)) return false;   // per-receiver line of sight
  q.kind = (fl >> 1) & 3;
  if (q.kind == 2 && P.mat[n] != m) return false;
  const double px = P.p[3 * n], py = P.p[3 * n + 1], pz = P.p[3 * n + 2];
  const double wx = a.rx_pos[3 * m] - px, wy = a.rx_pos[3 * m + 1] - py, wz = a.rx_pos[3 * m + 2] - pz;
  q.l = sqrt(wx * wx + wy * wy + wz * wz);
  q.u[0] = wx / q.l; q.u[1] = wy / q.l; q.u[2] = wz / q.l;
  q.r = P.rtot[n] + q.l;                                   // emitter -> point -> receiver
  const double sc = (double)a.sigma * q.r / a.c;
  q.c0 = sc * a.f_lo;
  q.cb = sc * a.df;
  q.base64 = -a.ps * log2(q.r) - (a.A0 + a.A1 * a.f_lo) * q.r / 20.0 * LOG2_10;
  q.slope64 = -a.A1 * a.df * q.r / 20.0 * LOG2_10;
  q.base = (float)q.base64;
  q.slope = (float)q.slope64;
  q.mat = a.rec_rows ? (int)n : P.mat[n];
  q.gamma = 0.f;
  if (q.kind == 0) {
    const float dx = P.dout[3 * n], dy = P.dout[3 * n + 1], dz = P.dout[3 * n + 2];
    const float ux = (float)q.u[0], uy = (float)q.u[1], uz = (float)q.u[2];
    const float cx = dy * uz - dz * uy, cy = dz * ux - dx * uz, cz = dx * uy - dy * ux;
    q.gamma = atan2f(sqrtf(cx * cx + cy * cy + cz * cz), dx * ux + dy * uy + dz * uz);
  }
  return true;
}

// log2 of the band factor: k exp(-gamma^2 / (2 beta^2)) (specular), I_d (diffraction) or
// I_p (passive)
// KFREE: specular records without the factor k (the adjoint's dH/dk, H being linear in k).
template <bool KFREE = false>
__device__ inline float band_log2_v(const SynthArgs& a, int kind, int mat, float gamma, int b) {
  const int64_t i = (int64_t)mat * a.Bk + b;
  return kind == 0 ? (KFREE ? 0.f : a.lk[i]) - gamma * gamma * a.lc[i] : kind == 1 ? a.ld[i] : a.lp[b];
}

__device__ inline void band_table_entry(const SynthArgs& a, int i, float* lk, float* lc, float* ld, float* lp) {
  const float bt = a.beta[i];
  lk[i] = log2f(a.refl_k[i]);
  lc[i] = LOG2E_F / (2.0f * bt * bt);
  ld[i] = log2f(a.dcoef[i]);
  if (i < a.Bk) lp[i] = a.pcoef ? log2f(a.pcoef[i]) : -INFINITY;
}

// Per-material bounds of material q (and, for q = 0, of the passive factors) from the same
// expressions as the table entries, so that each bound equals the extreme of its entries.
__device__ inline void band_bound_entry(const SynthArgs& a, int q, float* lmax) {
  float mk = -INFINITY, mc = INFINITY, md = -INFINITY;
  for (int b = 0; b < a.Bk; ++b) {
    const int i = q * a.Bk + b;
    const float bt = a.beta[i];
    mk = fmaxf(mk, log2f(a.refl_k[i]));
    mc = fminf(mc, LOG2E_F / (2.0f * bt * bt));
    md = fmaxf(md, log2f(a.dcoef[i]));
  }
  lmax[q] = mk;
  lmax[a.Q + q] = mc;
  lmax[2 * a.Q + q] = md;
  if (q == 0) {
    float mp = -INFINITY;
    if (a.pcoef)
      for (int b = 0; b < a.Bk; ++b) mp = fmaxf(mp, log2f(a.pcoef[b]));
    lmax[3 * a.Q] = mp;
  }
}

// Band of bin k of F in B bands (32-bit arithmetic where k B fits).
__device__ inline int band_of(int k, int B, int F) {
  return F < (1 << 25) ? (int)(((uint32_t)k * (uint32_t)B) / (uint32_t)F) : (int)(((int64_t)k * B) / F);
}

// Row table of a pose (see synth_rows): (first bin, material band + directivity band << 16) per row,
// closed by an entry with first bin F.  One workgroup of 256 threads, each a run of the bins.
__device__ inline void row_table(const SynthArgs& a, int2* __restrict__ rows) {
  __shared__ int wsum[4];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int per = (int)(((int64_t)a.F + 255) / 256);
  const int64_t k0 = (int64_t)tid * per, k1 = min(k0 + per, (int64_t)a.F);
  int at = 0;
  for (int pass = 0; pass < 2; ++pass) {
    int n = 0;
    if (k0 < k1) {
      int pb = k0 > 0 ? band_of((int)k0 - 1, a.Bk, a.F) : -1, pd = k0 > 0 && a.Bd ? band_of((int)k0 - 1, a.Bd, a.F) : 0;
      for (int64_t k = k0; k < k1; ++k) {
        const int b = band_of((int)k, a.Bk, a.F), d = a.Bd ? band_of((int)k, a.Bd, a.F) : 0;
        if (k % K2 == 0 || b != pb || d != pd) {
          if (pass == 1) rows[at + n] = make_int2((int)k, b | (d << 16));
          ++n;
        }
        pb = b;
        pd = d;
      }
    }
    if (pass == 1) break;
    int inc = n;   // exclusive sum of the counts over the workgroup
    for (int o = 1; o < 64; o <<= 1) {
      const int v = __shfl_up(inc, o);
      if (lane >= o) inc += v;
    }
    if (lane == 63) wsum[wv] = inc;
    __syncthreads();
    at = inc - n;
    for (int w = 0; w < wv; ++w) at += wsum[w];
  }
  if (tid == 0) rows[a.nrows] = make_int2(a.F, 0);
}

__device__ inline float band_log2(const SynthArgs& a, const Pair& q, int b) {
  return band_log2_v(a, q.kind, q.mat, q.gamma, b);
}

// direction of arrival in the receiver frame: v = R_m^T (p - x_m) / l = -R_m^T u
__device__ inline void arrival(const SynthArgs& a, const Pair& q, int m, float& vx, float& vy, float& vz) {
  const double ux = -q.u[0], uy = -q.u[1], uz = -q.u[2];
  if (a.rx_rot) {
    const double* R = a.rx_rot + 9 * m;
    vx = (float)(R[0] * ux + R[3] * uy + R[6] * uz);
    vy = (float)(R[1] * ux + R[4] * uy + R[7] * uz);
    vz = (float)(R[2] * ux + R[5] * uy + R[8] * uz);
  } else {
    vx = (float)ux; vy = (float)uy; vz = (float)uz;
  }
}

__device__ inline double frac(double x) { return x - floor(x); }

__device__ inline void chunk_range(int64_t n, int32_t P, int p, int64_t& lo, int64_t& hi) {
  const int64_t per = (n + P - 1) / P;
  lo = std::min<int64_t>((int64_t)p * per, n);
  hi = std::min<int64_t>(lo + per, n);
}

// Chunks of a fused batch: the visible records are sorted by job, job j owns positions
// [lo[j], hi[j]) and chunks [off[j], off[j + 1]) of at most `per` records each, so no chunk
// mixes jobs.  off[J] is the batch's chunk count.
struct ChunkTab {
  const int64_t* off;   // [J + 1]
  const int64_t* lo;    // [J]
  const int64_t* hi;    // [J]
  const int64_t* per;   // [1]
  int32_t J;
};

// Resolves chunk c to its job and record range; false if c is past the batch's chunks.
__device__ inline bool batch_chunk(const ChunkTab& ct, int64_t c, int& j, int64_t& lo, int64_t& hi) {
  if (c >= ct.off[ct.J]) return false;
  int a = 0, b = ct.J - 1;   // last job with off <= c (jobs without chunks share off with the next)
  while (a < b) {
    const int mid = (a + b + 1) >> 1;
    if (ct.off[mid] <= c) a = mid;
    else b = mid - 1;
  }
  j = a;
  lo = ct.lo[a] + (c - ct.off[a]) * ct.per[0];
  hi = std::min<int64_t>(lo + ct.per[0], ct.hi[a]);
  return true;
}

// Common prologue: the workgroup's arguments and record range, plain or batched.
// Workgroup -> (record chunk, receiver, tile).  Workgroups reach the eight XCDs in turn (linear
// id mod 8).  With a chunk count that is a multiple of 8 the linear id reads as (chunk group,
// receiver and tile, XCD): every XCD works through its chunks one at a time with all receivers
// and tiles of a chunk together, so they share that XCD's L2 for the chunk's records.  Other
// chunk counts keep the grid's own coordinates.
__device__ inline void block_coords(int& p, int& m, int& t) {
  const int64_t nx = gridDim.x, ny = gridDim.y, nz = gridDim.z;
  if (nx % 8 != 0) {
    p = blockIdx.x; m = blockIdx.y; t = blockIdx.z;
    return;
  }
  const int64_t L = blockIdx.x + nx * (blockIdx.y + ny * blockIdx.z);
  const int64_t q = L >> 3, inner = ny * nz;
  const int64_t mt = q % inner;
  p = (int)((q / inner) * 8 + (L & 7));
  m = (int)(mt % ny);
  t = (int)(mt / ny);
}

#define SYNTH_RESOLVE()                                                      \
  int bp, bm, bt;                                                            \
  block_coords(bp, bm, bt);                                                  \
  SynthArgs a = a0;                                                          \
  int64_t lo, hi;                                                            \
  int jb = 0;                                                                \
  if (BATCH) {                                                               \
    if (!batch_chunk(ct, bp, jb, lo, hi)) return;                            \
    a = jobs[jb];                                                            \
  } else {                                                                   \
    chunk_range(ctl->n_vis, a.P, bp, lo, hi);                                \
  }

// ------------------------------------------------------------------ visible-record list

// The number of records of a call: what the paths hold, at most their capacity.
__device__ inline int64_t record_count(const et_paths& P) { return min(P.count[0], P.capacity); }

// Tiles of the records for the visible list: 2048 records, more where that would make over 2048 tiles (every
// tile sums the counts of those before it).
constexpr int VIS_TILE = 2048;
constexpr int64_t VIS_MAX_TILES = 2048;
__host__ __device__ inline int64_t vis_tile(int64_t cap) {
  const int64_t t = (cap + VIS_MAX_TILES - 1) / VIS_MAX_TILES;
  return (t + VIS_TILE - 1) / VIS_TILE * VIS_TILE;
}

__device__ inline uint64_t wave_sum_u64(uint64_t v) {
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
  return v;
}

// Visible records of tile t (workgroup of 256 threads).
__device__ inline void vis_count(const et_paths& P, Ctl* ctl, int64_t t, int64_t tile, uint64_t* __restrict__ vsum) {
  __shared__ uint64_t red[4];
  const int64_t n = record_count(P);
  const int64_t lo = t * tile, hi = min(lo + tile, n);
  uint64_t c = 0;
  for (int64_t i = lo + threadIdx.x; i < hi; i += 256) c += P.flags[i] & 1;
  c = wave_sum_u64(c);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = c;
  __syncthreads();
  if (threadIdx.x == 0) {
    vsum[t] = red[0] + red[1] + red[2] + red[3];
    if (t == 0) ctl->n_rec = n;
  }
}

__global__ __launch_bounds__(256) void k_vis_count(et_paths P, Ctl* ctl, int64_t tile, uint64_t* __restrict__ vsum) {
  vis_count(P, ctl, blockIdx.x, tile, vsum);
}

// The indices of the visible records in order; each wave takes 512 consecutive ones of a tile at a time.
__global__ __launch_bounds__(256) void k_vis_list(et_paths P, Ctl* ctl, int64_t tile, const uint64_t* __restrict__ vsum,
                                                  int32_t* __restrict__ idx) {
  __shared__ uint64_t red[4];
  __shared__ uint64_t cnt[4];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int64_t n = ctl->n_rec;
  const int64_t lo = blockIdx.x * tile, hi = min(lo + tile, n);
  if (blockIdx.x > 0 && lo >= n) return;
  uint64_t s = 0;   // before the tile; the last tile with records also leaves the total
  for (int64_t k = tid; k < (int64_t)blockIdx.x; k += 256) s += vsum[k];
  s = wave_sum_u64(s);
  if (lane == 0) red[wv] = s;
  __syncthreads();
  uint64_t at = red[0] + red[1] + red[2] + red[3];
  if (tid == 0 && hi >= n) ctl->n_vis = (int64_t)(at + vsum[blockIdx.x]);
  for (int64_t base = lo; base < hi; base += VIS_TILE) {
    const int64_t w0 = base + wv * (VIS_TILE / 4);
    uint64_t m[8];
    uint64_t c = 0;
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const int64_t i = w0 + 64 * k + lane;
      m[k] = __ballot(i < hi && (P.flags[i] & 1));
      c += __popcll(m[k]);
    }
    __syncthreads();
    if (lane == 0) cnt[wv] = c;
    __syncthreads();
    uint64_t o = at;
    for (int k = 0; k < wv; ++k) o += cnt[k];
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      if ((m[k] >> lane) & 1ull) idx[o + __popcll(m[k] & ((1ull << lane) - 1ull))] = (int32_t)(w0 + 64 * k + lane);
      o += __popcll(m[k]);
    }
    at += cnt[0] + cnt[1] + cnt[2] + cnt[3];
  }
}

// no list: the kernels walk every record
__global__ void k_vis_all(et_paths P, Ctl* ctl) { ctl->n_vis = ctl->n_rec = record_count(P); }

// ------------------------------------------------------------------ factorised MFMA kernel

constexpr int RB = 32;        // records per stage (contraction depth per stage)
constexpr int RPW = RB / 4;   // records per wave and stage

typedef float floatx4 __attribute__((ext_vector_type(4)));

__device__ inline uint32_t q32(double cyc) {   // fraction of a cycle in Q0.32 (mod 2^32)
  return (uint32_t)(__builtin_amdgcn_fract(cyc) * 4294967296.0);   // in [0, 2^32); the conversion saturates
}

// Lean per-(record, receiver) setup: FP64 only for the receiver leg, the path and the delay
// reductions.  Phases of the generated values are integer phase accumulators in Q0.32
// (a32 + k1 bx32 for X, k2 by32 for Y), exact mod 1 up to the quantisation of the steps
// (<= 128 * 2^-33 cycles).
typedef __attribute__((address_space(1))) float GlobalFloat;

// The lobe coefficients of the records that have no lobe (diffraction and passive ones), for up to 64 bands: a
// material's own may be infinite (a lobe of width 0), and 0 times that is no factor.
__device__ const float NO_LOBE[64] = {};

struct PairLean {
  uint32_t a32, bx32, by32;
  float base, slope, gamma;
  DirCell cell;          // directivity cell of the arrival (forward, with directivity)
  int mat, kind;         // mat: row of the band tables (the material, or the record: rec_rows)
  float lbm;             // bound on the log2 band factor (with directivity) over every band: the
                         // generating factors carry it, so Xa stays below the record's bound and
                         // the per-segment factors below 1
  const GlobalFloat *t1, *t2;   // forward: the record's rows of the band tables, log2 factor = t1[b] - gamma^2 t2[b]
  // the adjoint's receiver-gradient coefficients, d/dx_m of (ln A + j phi) = (c1 + c2 f + j c3 f) u - lobe
  float gux, guy, guz;   // u = (x_m - p) / l
  float gc1;             // -p / r - ln10 a0 / 20
  float glx, gly, glz;   // 2 (gamma / sin gamma) (d' - cos(gamma) u) / l (specular; 0 otherwise)
};

// Element e of the visible-record list (without a list: every record, hidden ones skipped at set-up).
__device__ inline int64_t record_at(const int32_t* __restrict__ idx, int64_t e) { return idx ? (int64_t)idx[e] : e; }

// Set-up of record n for receiver m (forward): every field of the record is read at once, whether it counts
// or not, so that a group waits for memory once and not for the index, the flags and the fields in
// turn.  What a record that does not count holds is never used: its point and direction may be anything (its
// gamma and bound are set to 0), and its material, like the receiver that a passive record keeps there, is no
// index of the tables.  valid: the lane has a record of the range.  dmax: the receiver's largest log2 directivity gain
// (0 without directivity).
template <bool DIR>
__device__ __forceinline__ void pair_fwd(const SynthArgs& a, const et_paths& P, int64_t n, bool valid, int m, float dmax,
                                         PairLean& q) {
  const uint8_t fl = P.flags[n];
  const int mat = P.mat[n];
  const double px = P.p[3 * n], py = P.p[3 * n + 1], pz = P.p[3 * n + 2], rtot = P.rtot[n];
  const float dx = P.dout[3 * n], dy = P.dout[3 * n + 1], dz = P.dout[3 * n + 2];
  bool ok = valid && (fl & 1);
  if (a.rxv) ok = ok && ((a.rxv[n] >> m) & 1ull);   // per-receiver line of sight
  q.kind = (fl >> 1) & 3;
  ok = ok && !(q.kind == 2 && mat != m);            // a passive record reaches its own receiver only
  const double wx = a.rx_pos[3 * m] - px, wy = a.rx_pos[3 * m + 1] - py, wz = a.rx_pos[3 * m + 2] - pz;
  const double l = sqrt(wx * wx + wy * wy + wz * wz), il = 1.0 / l;
  const double r = rtot + l;                        // emitter -> point -> receiver
  const double cb = r * a.kcb;
  q.a32 = ok ? q32(r * a.kc0) : 0u;
  q.bx32 = ok ? q32((double)K2 * cb) : 0u;
  q.by32 = ok ? q32(cb) : 0u;
  const float base = -(float)a.ps * log2f((float)r) + (float)(r * a.kbase);
  q.slope = ok ? (float)(r * a.kslope) : 0.f;
  // rows of the band tables: the material's (with per-record tables the record's), one row for passive
  // records; the lobe is the specular records' (per-record tables hold 0 for the others)
  const int q1 = ok && q.kind < 2 ? mat : 0;
  const int64_t row = a.rec_rows ? n : (int64_t)q1;
  const float* t1 = q.kind == 0 ? a.lk : q.kind == 1 ? a.ld : a.lp;
  q.t1 = (const GlobalFloat*)(t1 + (q.kind >= 2 ? 0 : row * a.Bk));
  q.t2 = (const GlobalFloat*)(q.kind == 0 || a.rec_rows ? a.lc + row * a.Bk : NO_LOBE);
  const float ux = (float)(wx * il), uy = (float)(wy * il), uz = (float)(wz * il);
  const float cx = dy * uz - dz * uy, cy = dz * ux - dx * uz, cz = dx * uy - dy * ux;
  const float gam = atan2f(sqrtf(cx * cx + cy * cy + cz * cz), dx * ux + dy * uy + dz * uz);
  q.gamma = ok && q.kind == 0 ? gam : 0.f;
  if (DIR) {   // direction of arrival in the receiver frame: -R_m^T u
    q.cell = DirCell{0, 0, 0, 0, 0.f, 0.f};
    if (a.Bd) {
      float vx = -ux, vy = -uy, vz = -uz;
      if (a.rx_rot) {
        const double* R = a.rx_rot + 9 * m;
        vx = -(float)(R[0] * ux + R[3] * uy + R[6] * uz);
        vy = -(float)(R[1] * ux + R[4] * uy + R[7] * uz);
        vz = -(float)(R[2] * ux + R[5] * uy + R[8] * uz);
      }
      q.cell = dir_cell(a.El, a.Az, vx, vy, vz);
    }
  }
  // bound on the log2 band factor over every band: from the per-material bounds (at least the largest factor:
  // k and the lobe's coefficient may peak on different bands), or by taking every band of per-record tables
  float bm = -INFINITY;
  if (!a.rec_rows) {
    const int top = q.kind == 0 ? q1 : q.kind == 1 ? 2 * a.Q + q1 : 3 * a.Q;
    const float lobe = q.kind == 0 ? a.lmax[a.Q + q1] : 0.f;
    bm = a.lmax[top] - q.gamma * q.gamma * lobe;
  } else {
    for (int b = 0; b < a.Bk; ++b) bm = fmaxf(bm, q.t1[b] - q.gamma * q.gamma * q.t2[b]);
  }
  q.lbm = bm + dmax;
  // nothing to add when every band factor is zero (lbm stays finite)
  q.base = ok && q.lbm != -INFINITY ? base : -INFINITY;
  if (!ok || q.lbm == -INFINITY) q.lbm = 0.f;
}

// Set-up of the adjoint: receiver-gradient coefficients, band factors without k.
__device__ inline void pair_adj(const SynthArgs& a, const et_paths& P, const int32_t* __restrict__ idx, int64_t e,
                                int64_t hi, int m, PairLean& q) {
  q.a32 = q.bx32 = q.by32 = 0;
  q.base = -INFINITY;
  q.lbm = 0.f;
  q.slope = q.gamma = 0.f;
  q.mat = q.kind = 0;
  q.gux = q.guy = q.guz = q.gc1 = q.glx = q.gly = q.glz = 0.f;
  if (e >= hi) return;
  const int64_t n = record_at(idx, e);
  const uint8_t fl = P.flags[n];
  if (!(fl & 1)) return;
  if (a.rxv && !((a.rxv[n] >> m) & 1ull)) return;   // per-receiver line of sight
  const int kind = (fl >> 1) & 3;
  if (kind == 2 && P.mat[n] != m) return;   // a passive record reaches its own receiver only
  q.kind = kind;
  const double wx = a.rx_pos[3 * m] - P.p[3 * n], wy = a.rx_pos[3 * m + 1] - P.p[3 * n + 1],
               wz = a.rx_pos[3 * m + 2] - P.p[3 * n + 2];
  const double l = sqrt(wx * wx + wy * wy + wz * wz), il = 1.0 / l;
  const double r = P.rtot[n] + l;                          // emitter -> point -> receiver
  const double cb = r * a.kcb;
  q.a32 = q32(r * a.kc0);
  q.bx32 = q32((double)K2 * cb);
  q.by32 = q32(cb);
  q.base = -(float)a.ps * log2f((float)r) + (float)(r * a.kbase);
  q.slope = (float)(r * a.kslope);
  q.mat = P.mat[n];
  const float ux = (float)(wx * il), uy = (float)(wy * il), uz = (float)(wz * il);
  if (q.kind == 0) {
    const float dx = P.dout[3 * n], dy = P.dout[3 * n + 1], dz = P.dout[3 * n + 2];
    const float cx = dy * uz - dz * uy, cy = dz * ux - dx * uz, cz = dx * uy - dy * ux;
    const float sc = sqrtf(cx * cx + cy * cy + cz * cz), cc = dx * ux + dy * uy + dz * uz;
    q.gamma = atan2f(sc, cc);
    // d(gamma^2)/dx_m = -(2 gamma / sin gamma) (h - cos(gamma) u) / l with h = d' / |d'|
    const float idn = 1.0f / sqrtf(dx * dx + dy * dy + dz * dz);
    const float sg = sc * idn, cg = cc * idn;
    const float ratio = q.gamma < 1e-4f ? 2.0f : 2.0f * q.gamma / sg;
    const float c = ratio * (float)(2.0 * il);
    q.glx = c * (dx * idn - cg * ux);
    q.gly = c * (dy * idn - cg * uy);
    q.glz = c * (dz * idn - cg * uz);
  }
  q.gux = ux; q.guy = uy; q.guz = uz;
  q.gc1 = (float)(-a.ps / r - 2.30258509299404568402 * a.A0 / 20.0);
  // bound on the log2 band factor without k, over every band
  q.lbm = q.kind == 0 ? -q.gamma * q.gamma * a.lmax[a.Q + q.mat] : a.lmax[q.kind == 1 ? 2 * a.Q + q.mat : 3 * a.Q];
  if (q.lbm == -INFINITY) {   // every band factor is zero: nothing to add (lbm stays finite)
    q.base = -INFINITY;
    q.lbm = 0.f;
  }
}

// The contractions run on the f16 matrix cores with FP32 accumulation.  Each FP32 operand v is split
// into two halves, hi = f16(v) and lo = f16(v - hi), about 22 significant bits together; a real
// product takes three half products, hi hi + hi lo + lo hi (lo lo lies below 2^-22 of it), and the
// complex product the four real ones re re, im im, re im, im re.  f16 has a narrow exponent range: X
// is scaled by 2^(XTOP - E) with E a wave-wide bound on log2 |X| over each group of 64 records, taken
// before the group is generated; when a group's bound exceeds E the accumulators are rescaled by a
// power of two (exact).  A record far below the bound loses relative precision in proportion to its
// negligible share of the sum.
typedef _Float16 halfx8 __attribute__((ext_vector_type(8)));
constexpr float XTOP = 12.f;     // log2 of the largest scaled |X| (|Y| <= 1 for non-negative absorption)

typedef _Float16 half2v __attribute__((ext_vector_type(2)));
typedef float float2v __attribute__((ext_vector_type(2)));

// The halves of two values: h = (f16(v0), f16(v1)), l the halves of the differences (see split8).
__device__ __forceinline__ void split2(float v0, float v1, uint32_t& h, uint32_t& l) {
  h = __builtin_bit_cast(uint32_t, __builtin_convertvector((float2v){v0, v1}, half2v));
  uint32_t lo;
  asm("v_fma_mixlo_f16 %0, -%1, 1.0, %2 op_sel_hi:[1,0,0]" : "=v"(lo) : "v"(h), "v"(v0));
  asm("v_fma_mixhi_f16 %0, -%1, 1.0, %2 op_sel:[1,0,0] op_sel_hi:[1,0,0]" : "+v"(lo) : "v"(h), "v"(v1));
  l = lo;
}

// hi = f16(v) two at a time (round to nearest even); lo = f16(v - hi), the difference taken
// exactly by a mixed-precision fma from the f16 hi and the f32 v, written into the low, then
// the high half of one register (the fma leaves the other half as it is).
__device__ inline void split8(const float (&v)[8], halfx8& h, halfx8& l) {
  union { halfx8 h8; uint32_t u[4]; } H, L;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const uint32_t xu = __builtin_bit_cast(uint32_t, __builtin_convertvector((float2v){v[2 * i], v[2 * i + 1]}, half2v));
    uint32_t lo;
    asm("v_fma_mixlo_f16 %0, -%1, 1.0, %2 op_sel_hi:[1,0,0]" : "=v"(lo) : "v"(xu), "v"(v[2 * i]));
    asm("v_fma_mixhi_f16 %0, -%1, 1.0, %2 op_sel:[1,0,0] op_sel_hi:[1,0,0]" : "+v"(lo) : "v"(xu), "v"(v[2 * i + 1]));
    H.u[i] = xu;
    L.u[i] = lo;
  }
  h = H.h8;
  l = L.h8;
}

// Two-level generation: X[8a+b] = Xa[a] Xb[b] bf[seg(8a+b)] and Y[8a+b] = Ya[a] Yb[b]:
// 32 exp2/sin/cos factors per record instead of 128 values, plus one real band factor
// bf = 2^(band + directivity log2) per segment of outer indices with equal bands.
struct WaveScratch {
  float2 xa[RPW][8], xb[RPW][8], ya[RPW][8], yb[RPW][8];
  union {
    float bf[RPW][SMAX + 1];   // [nseg]: zero, for rows past the tile
    float2 xh[RPW][8];         // FOLD: Xa of rows 8 a + 4 .. 8 a + 7 (their half group's band)
  };
};

// Band segments of a tile of outer indices: segment s covers the rows whose material band
// is sb[s] and directivity band sd[s].
struct SegTable {
  int32_t sb[SMAX], sd[SMAX];   // material and directivity band of segment s
  int32_t s0[SMAX], s1[SMAX];   // its rows [s0, s1) within the tile
  int32_t bseg[16];             // segment of material band b, -1 if none (used without directivity)
};

// Band segments of the tile [k1_0, k1_0 + nk1) (the host guarantees bands constant per row
// and at most SMAX segments).  Every thread learns nseg and the segment of its lane's row
// (nseg for a row past the tile).
__device__ inline void seg_init(const SynthArgs& a, int k1_0, int nk1, int tid, SegTable& st, int& nseg, int& myseg) {
  const int lane = tid & 63, wv = tid >> 6;
  const int kr = (k1_0 + min(lane, nk1 - 1)) * K2;
  const int bb = (int)(((int64_t)kr * a.Bk) / a.F), bd = a.Bd ? (int)(((int64_t)kr * a.Bd) / a.F) : 0;
  const int bb_prev = __shfl(bb, lane - 1), bd_prev = __shfl(bd, lane - 1);
  const bool starts = lane < nk1 && (lane == 0 || bb != bb_prev || bd != bd_prev);
  const uint64_t sm = __ballot(starts);
  nseg = __popcll(sm);
  // rows past the tile take the extra segment nseg, whose band factor is zero
  myseg = lane < nk1 ? __popcll(sm & (~0ull >> (63 - lane))) - 1 : nseg;
  if (tid < 16) st.bseg[tid] = -1;
  __syncthreads();
  if (wv == 0 && starts && myseg < SMAX) {
    st.sb[myseg] = bb;
    st.sd[myseg] = bd;
    st.s0[myseg] = lane;
    if (bb < 16) st.bseg[bb] = myseg;
  }
  __syncthreads();
  if (tid < nseg && tid < SMAX) st.s1[tid] = tid + 1 < nseg ? st.s0[tid + 1] : nk1;
  __syncthreads();
}

// 2^lg e^(2 pi j rev) from the hardware exp2, sin and cos (a result below 2^-126 flushes to zero:
// such a value is below 2^-138 of the tile's largest term)
__device__ inline float2 cexp2(float lg, float rev) {
  const float amp = __builtin_amdgcn_exp2f(lg);
  return make_float2(amp * __builtin_amdgcn_cosf(rev), amp * __builtin_amdgcn_sinf(rev));
}
__device__ inline float2 cmul(float2 a, float2 b) { return make_float2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x); }

// (Adjoint.)  One wave computes the generating factors of RPW records (sub-stage t of its 64 set-up
// records): Xa, Xb, Ya, Yb (8 each) and the band factor of every (record, band segment) of the
// tile, into its WaveScratch.  esh (log2) scales every X of the sub-stage.
// The specular band factor leaves out k (see band_log2_v).
// FOLD 4: every band segment is a union of whole half groups of 4 rows (segl, segh: the segments
// of rows 8 j and 8 j + 4 of this lane's group j): the band factor is folded into Xa, one copy
// per half group (Xa for rows 8 j .. 8 j + 3, Xh for 8 j + 4 .. 8 j + 7), and no table is written.
// FOLD 8: whole groups of 8 rows, one copy (Xa).
template <int FOLD>
__device__ inline void gen_factors(const SynthArgs& a, const PairLean& q, int t, int k1_0, int nk1, int lane, int nseg,
                                   const SegTable& st, float esh, WaveScratch& W, int segl, int segh) {
  const int r = lane >> 3, j = lane & 7;
  const int src = t * RPW + r;                 // lane that set up record r of this sub-stage
  const float base_r = __shfl(q.base, src), slope_r = __shfl(q.slope, src);
  const uint32_t a_r = (uint32_t)__shfl((int)q.a32, src), bx_r = (uint32_t)__shfl((int)q.bx32, src),
                 by_r = (uint32_t)__shfl((int)q.by32, src);
  const float lbm_r = __shfl(q.lbm, src);
  const bool ok = base_r != -INFINITY;
  const uint32_t k1a = (uint32_t)(k1_0 + 8 * j);   // first outer index of group j
  // Xa is zero for a record that adds nothing (and past the tile); then X is zero whatever the
  // other factors (finite for every record: a skipped record has slope 0 and phase steps 0)
  const float S = 2.3283064365386963e-10f;   // 2^-32: Q0.32 cycles to revolutions
  const float lg0 = base_r + (float)(k1a * K2) * slope_r + esh;
  if (FOLD) {
    // the band factors of the two half groups (no record's bound needed: each is its own)
    const float g_r = __shfl(q.gamma, src);
    const int m_r = __shfl(q.mat, src), k_r = __shfl(q.kind, src);
    float ll = band_log2_v<true>(a, k_r, m_r, g_r, st.sb[segl]);
    float lh = FOLD == 4 ? band_log2_v<true>(a, k_r, m_r, g_r, st.sb[segh]) : 0.f;
    const float rev = (float)(int32_t)(a_r + k1a * bx_r) * S;
    const float c = __builtin_amdgcn_cosf(rev), sn = __builtin_amdgcn_sinf(rev);
    const float al = ok && 8 * j < nk1 ? __builtin_amdgcn_exp2f(lg0 + ll) : 0.f;
    W.xa[r][j] = make_float2(al * c, al * sn);
    if (FOLD == 4) {
      const float ah = ok && 8 * j + 4 < nk1 ? __builtin_amdgcn_exp2f(lg0 + lh) : 0.f;
      W.xh[r][j] = make_float2(ah * c, ah * sn);
    }
  } else {
    // the record's band bound lbm rides on Xa; the band factors (<= 1) go to the table below
    const float lg = ok && 8 * j < nk1 ? lg0 + lbm_r : -INFINITY;
    W.xa[r][j] = cexp2(lg, (float)(int32_t)(a_r + k1a * bx_r) * S);
  }
  W.xb[r][j] = cexp2((float)(j * K2) * slope_r, (float)(int32_t)((uint32_t)j * bx_r) * S);
  W.ya[r][j] = cexp2((float)(8 * j) * slope_r, (float)(int32_t)((uint32_t)(8 * j) * by_r) * S);
  W.yb[r][j] = cexp2((float)j * slope_r, (float)(int32_t)((uint32_t)j * by_r) * S);
  // band factors of every (record, segment), and zero for the segment past the tile
  if (!FOLD) {
    // the pairs enumerated over the wave, each lane fetching its record's data (fewer registers live across the
    // loop: measured faster)
    for (int i0 = 0; i0 < RPW * nseg; i0 += 64) {
      const int i = i0 + lane;
      const int rr = min(i / nseg, RPW - 1), sg = i - (i / nseg) * nseg;
      const int sr = t * RPW + rr;
      const float g2 = __shfl(q.gamma, sr), b2 = __shfl(q.base, sr), lm2 = __shfl(q.lbm, sr);
      const int m2 = __shfl(q.mat, sr), k2 = __shfl(q.kind, sr);
      if (i < RPW * nseg) W.bf[rr][sg] = b2 != -INFINITY ? exp2f(band_log2_v<true>(a, k2, m2, g2, st.sb[sg]) - lm2) : 0.f;
    }
  }
  if (!FOLD && j == 7) W.bf[r][nseg] = 0.f;
  // the factors are read back by other lanes of this wave only
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// Maximum over the wave's lanes, the same (scalar) value in every lane: lane moves within rows of 16,
// then the four rows' values.
template <int CTRL>
__device__ inline float dpp_mov(float x) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), CTRL, 0xF, 0xF, false));
}
__device__ inline float wave_max(float v) {
  v = fmaxf(v, dpp_mov<0xB1>(v));    // quad_perm [1, 0, 3, 2]
  v = fmaxf(v, dpp_mov<0x4E>(v));    // quad_perm [2, 3, 0, 1]
  v = fmaxf(v, dpp_mov<0x141>(v));   // row_half_mirror
  v = fmaxf(v, dpp_mov<0x140>(v));   // row_mirror
  const int u = __builtin_bit_cast(int, v);
  float r[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) r[i] = __builtin_bit_cast(float, __builtin_amdgcn_readlane(u, 16 * i));
  return fmaxf(fmaxf(r[0], r[1]), fmaxf(r[2], r[3]));
}

// Upper bound on log2 |X[k1] Y[k2]| over the tile for the record set up in q (-inf for none):
// the amplitude at the tile's first or last row, the record's band bound lbm (at least its
// largest band factor with its lobe, plus the receiver's largest log2 directivity gain), and
// what |Y| can exceed 1 by.
__device__ inline float record_bound(const PairLean& q, int k1_0, int nk1) {
  if (q.base == -INFINITY) return -INFINITY;
  const float s64 = (float)K2 * q.slope;
  return q.base + fmaxf((float)k1_0 * s64, (float)(k1_0 + nk1 - 1) * s64) + fmaxf(0.f, (float)(K2 - 1) * q.slope) +
         q.lbm;
}

// Largest log2 directivity gain of receiver m over every band and cell (the bilinear gain never
// exceeds it); 0 without directivity.  Every thread of the workgroup calls it.
__device__ inline float dir_log2_max(const SynthArgs& a, int m, int tid, float* red) {
  if (!a.Bd) return 0.f;
  const float* tab = a.dir + (size_t)m * a.Bd * a.El * a.Az;
  const int n = a.Bd * a.El * a.Az;
  float v = 0.f;
  for (int i = tid; i < n; i += 256) v = fmaxf(v, tab[i]);
  v = wave_max(v);
  if ((tid & 63) == 0) red[tid >> 6] = v;
  __syncthreads();
  v = fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
  __syncthreads();
  return log2f(v);
}

typedef float floatx16 __attribute__((ext_vector_type(16)));

// The generating factors of a wave's U records (private to it): rows [factor][record] with a pad of 16
// bytes, so that the lanes that read different factors of the same records land on distinct banks.
// Factors: Xa of the G = 4 NRB row groups, with FOLD 4 Xa of their upper halves, then Xb, Ya and Yb
// (8 each); bf: the band factor per (segment, record) with FOLD 0.
template <int NRB, int FOLD, int U>
struct Factors {
  static constexpr int G = 4 * NRB, XH = G, XB = FOLD == 4 ? 2 * G : G, YA = XB + 8, YB = YA + 8;
  float2 f[YB + 8][U + 2];
  float bf[FOLD == 0 ? SMAX + 1 : 1][FOLD == 0 ? U + 4 : 4];
};

__device__ inline const GlobalFloat* shfl_ptr(const GlobalFloat* p, int src) {
  const uint64_t v = (uint64_t)p;
  const uint32_t lo = (uint32_t)__shfl((int)(uint32_t)v, src), hi = (uint32_t)__shfl((int)(uint32_t)(v >> 32), src);
  return (const GlobalFloat*)((uint64_t)hi << 32 | lo);
}

// One wave computes the generating factors of records U s .. U s + U - 1 of the 64 its lanes have set up:
// with U = 64 every lane those of its own record, with U = 32 lane (r = lane % 32, h = lane / 32) half of
// record r's.  esh (log2) scales X.  key: with FOLD the bands of the eight row groups, material |
// directivity << 8 of the first half group, << 16 of the second; with FOLD 0 the bands of the segments.
template <int NRB, int FOLD, int U, bool DIR>
__device__ __forceinline__ void gen_factors_u(const SynthArgs& a, const PairLean& q0, int s, int m, int k1_0, int nk1,
                                              int lane, float esh, int nseg, const int* __restrict__ key,
                                              Factors<NRB, FOLD, U>& W) {
  using FT = Factors<NRB, FOLD, U>;
  constexpr int NH = 64 / U;                     // lanes per record
  const int r = lane & (U - 1), h = U == 64 ? 0 : lane / U;
  PairLean q = q0;
  if (U != 64) {
    const int src = U * s + r;
    q.base = __shfl(q0.base, src); q.slope = __shfl(q0.slope, src); q.gamma = __shfl(q0.gamma, src);
    q.a32 = (uint32_t)__shfl((int)q0.a32, src);
    q.bx32 = (uint32_t)__shfl((int)q0.bx32, src);
    q.by32 = (uint32_t)__shfl((int)q0.by32, src);
    q.t1 = shfl_ptr(q0.t1, src);
    q.t2 = shfl_ptr(q0.t2, src);
    if (DIR) {
      q.cell.r0 = __shfl(q0.cell.r0, src); q.cell.r1 = __shfl(q0.cell.r1, src);
      q.cell.i0 = __shfl(q0.cell.i0, src); q.cell.i1 = __shfl(q0.cell.i1, src);
      q.cell.ta = __shfl(q0.cell.ta, src); q.cell.te = __shfl(q0.cell.te, src);
    }
    if (FOLD == 0) q.lbm = __shfl(q0.lbm, src);
  }
  const GlobalFloat* dtab = (const GlobalFloat*)a.dir + (size_t)m * a.Bd * a.El * a.Az;
  const size_t dcells = (size_t)a.El * a.Az;
  const bool dir = DIR && a.Bd != 0;
  const float g2 = q.gamma * q.gamma;
  // Xa is zero for a record that adds nothing (and past the tile); then X is zero whatever the
  // other factors (finite for every record: a skipped record has slope 0 and phase steps 0)
  const bool ok = q.base != -INFINITY;
  const float S = 2.3283064365386963e-10f;   // 2^-32: Q0.32 cycles to revolutions
  // the groups' log2 band factors: all the table reads at once, in flight while Xb, Ya and Yb are formed
  constexpr int NG = FT::G / NH;
  const int j0 = NG * h;
  float ll[NG], lh[FOLD == 4 ? NG : 1];
  if (FOLD) {
    uint32_t kb[NG];
#pragma unroll
    for (int jj = 0; jj < NG; ++jj) {
      kb[jj] = (uint32_t)key[j0 + jj];
      if (U == 64) kb[jj] = (uint32_t)__builtin_amdgcn_readfirstlane((int)kb[jj]);
    }
#pragma unroll
    for (int jj = 0; jj < NG; ++jj) {
      ll[jj] = q.t1[kb[jj] & 255] - g2 * q.t2[kb[jj] & 255];
      if (FOLD == 4) lh[jj] = q.t1[(kb[jj] >> 16) & 255] - g2 * q.t2[(kb[jj] >> 16) & 255];
    }
    if (dir) {
#pragma unroll
      for (int jj = 0; jj < NG; ++jj) {
        ll[jj] += log2f(dir_lerp(dtab + ((kb[jj] >> 8) & 255) * dcells, q.cell));
        if (FOLD == 4) lh[jj] += log2f(dir_lerp(dtab + (kb[jj] >> 24) * dcells, q.cell));
      }
    }
  }
  {
    // (phases by repeated addition: exact modulo a cycle; with U = 64 the factors 0, which are 1, are written
    // once by the kernel)
    constexpr int JJ0 = U == 64 ? 1 : 0;
    const int i0 = 8 / NH * h;
    uint32_t pb = (uint32_t)(i0 + JJ0) * q.bx32, pyb = (uint32_t)(i0 + JJ0) * q.by32, pya = 8u * pyb;
    const uint32_t by8 = 8u * q.by32;
#pragma unroll 4
    for (int jj = JJ0; jj < 8 / NH; ++jj) {
      const int j = i0 + jj;
      const float fj = (float)j;
      W.f[FT::XB + j][r] = cexp2((fj * K2) * q.slope, (float)(int32_t)pb * S);
      W.f[FT::YA + j][r] = cexp2((fj * 8.f) * q.slope, (float)(int32_t)pya * S);
      W.f[FT::YB + j][r] = cexp2(fj * q.slope, (float)(int32_t)pyb * S);
      pb += q.bx32;
      pya += by8;
      pyb += q.by32;
    }
  }
  {
    uint32_t pa = q.a32 + (uint32_t)(k1_0 + 8 * j0) * q.bx32;
    const uint32_t bx8 = 8u * q.bx32;
#pragma unroll
    for (int jj = 0; jj < NG; ++jj) {
      const int j = j0 + jj;
      const float lg0 = q.base + (float)((k1_0 + 8 * j) * K2) * q.slope + esh;
      const float rev = (float)(int32_t)pa * S;
      pa += bx8;
      const float c = __builtin_amdgcn_cosf(rev), sn = __builtin_amdgcn_sinf(rev);
      // with FOLD the group's (FOLD 4: its halves') band factor rides on Xa, else the record's band bound lbm
      const float al = ok && 8 * j < nk1 ? __builtin_amdgcn_exp2f(lg0 + (FOLD ? ll[jj] : q.lbm)) : 0.f;
      W.f[j][r] = make_float2(al * c, al * sn);
      if (FOLD == 4) {
        const float ah = ok && 8 * j + 4 < nk1 ? __builtin_amdgcn_exp2f(lg0 + lh[jj]) : 0.f;
        W.f[FT::XH + j][r] = make_float2(ah * c, ah * sn);
      }
    }
  }
  if (FOLD == 0) {
    for (int sg = h; sg < nseg; sg += NH) {
      const int kb = key[sg];
      float lb = q.t1[kb & 0xffff] - g2 * q.t2[kb & 0xffff];
      if (dir) lb += log2f(dir_lerp(dtab + (kb >> 16) * dcells, q.cell));
      W.bf[sg][r] = ok ? __builtin_amdgcn_exp2f(lb - q.lbm) : 0.f;   // <= 1
    }
  }
  // the factors are read back by other lanes of this wave only
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// Eight records of one row (X) or bin (Y) as a matrix operand: halves of the real and imaginary parts,
// records 2 e, 2 e + 1 in u[e].
union Half8 {
  halfx8 h;
  uint32_t u[4];
};
struct Operand {
  Half8 rh, rl, ih, il;
};

// Two records of an operand's two factors (and their band factors f with FOLD 0), in registers.
struct Pair2 {
  float4 a, b;
  __device__ __forceinline__ void load(const char* pa, const char* pb) {
    a = *reinterpret_cast<const float4*>(pa);
    b = *reinterpret_cast<const float4*>(pb);
  }
  __device__ __forceinline__ void scale(const char* pf) {
    const float2 f = *reinterpret_cast<const float2*>(pf);
    a.x *= f.x; a.y *= f.x;
    a.z *= f.y; a.w *= f.y;
  }
  // the products of the factors (into a), then their halves
  __device__ __forceinline__ void multiply() {
    const float2 v0 = cmul(make_float2(a.x, a.y), make_float2(b.x, b.y));
    const float2 v1 = cmul(make_float2(a.z, a.w), make_float2(b.z, b.w));
    a = make_float4(v0.x, v0.y, v1.x, v1.y);
  }
  __device__ __forceinline__ void split(int e, Operand& o) const {
    split2(a.x, a.z, o.rh.u[e], o.rl.u[e]);
    split2(a.y, a.w, o.ih.u[e], o.il.u[e]);
  }
};

// One 32 x 32 block and 16 records: Re += Xr Yr - Xi Yi, Im += Xr Yi + Xi Yr, three half products per real
// product, with slice(k) placed after product k (k < 12): the vector work that the matrix pipe covers.
template <class G>
__device__ __forceinline__ void contract12(const Operand& x, const Operand& y, floatx16& re, floatx16& im, G&& slice) {
  Half8 nx;   // -Xi, its high halves, then its low ones
#define ET_MM(A, B, C, K)                                              \
  C = __builtin_amdgcn_mfma_f32_32x32x16_f16(A.h, B.h, C, 0, 0, 0);    \
  slice(K);                                                            \
  __builtin_amdgcn_sched_barrier(0)
  ET_MM(x.rh, y.rh, re, 0);
  ET_MM(x.rh, y.ih, im, 1);
  ET_MM(x.rh, y.rl, re, 2);
  ET_MM(x.rh, y.il, im, 3);
  ET_MM(x.rl, y.rh, re, 4);
  ET_MM(x.rl, y.ih, im, 5);
#pragma unroll
  for (int e = 0; e < 4; ++e) nx.u[e] = x.ih.u[e] ^ 0x80008000u;
  ET_MM(nx, y.ih, re, 6);
  ET_MM(x.ih, y.rh, im, 7);
  ET_MM(nx, y.il, re, 8);
  ET_MM(x.ih, y.rl, im, 9);
#pragma unroll
  for (int e = 0; e < 4; ++e) nx.u[e] = x.il.u[e] ^ 0x80008000u;
  ET_MM(nx, y.ih, re, 10);
  ET_MM(x.il, y.rh, im, 11);
#undef ET_MM
}

// Rows [v0, v0 + nk) of the row table as a tile: its outer indices [k1_0, k1_0 + nk1), its band segments (nseg, their
// bands in key) and, of this lane's rows l % 32 + 32 i, the outer index - k1_0 | segment << 8 (rows past the tile: the
// extra segment nseg).
template <int NRB>
__device__ __forceinline__ void tile_rows(const SynthArgs& a, int v0, int nk, int lane, int wv, int* __restrict__ key,
                                          int& k1_0, int& nk1, int& nseg, int (&rinfo)[NRB]) {
  const int2 row = a.rows[v0 + min(lane, nk - 1)];
  k1_0 = __shfl(row.x, 0) >> 6;
  nk1 = (__shfl(row.x, 63) >> 6) - k1_0 + 1;
  const int prev = __shfl(row.y, (lane + 63) & 63);
  const uint64_t sm = __ballot(lane == 0 || (lane < nk && row.y != prev));
  const int seg = __popcll(sm & (~0ull >> (63 - lane))) - 1;
  nseg = min(__popcll(sm), SMAX);
  if (wv == 0 && ((sm >> lane) & 1) && seg < SMAX) key[seg] = row.y;
  const int info = ((row.x >> 6) - k1_0) | (lane < nk ? min(seg, SMAX - 1) : nseg) << 8;
#pragma unroll
  for (int i = 0; i < NRB; ++i) rinfo[i] = __shfl(info, (lane & 31) + 32 * i);
}

// The four waves' sums acc [re, im][row block][column block] of a tile, times us, as the chunk's partial spectrum.
// Accumulator v of lane l in block (i, jc): row 32 i + 8 (v / 4) + 4 (l / 32) + v % 4, bin 32 jc + l % 32 of the
// row's 64; the waves' values are added in wave order, a block at a time.  ROWS: rows of the row table, each
// keeping its own bins of the 64.  sums: LDS [wave][v][lane].
template <int NRB, bool ROWS>
__device__ __forceinline__ void write_tile(const SynthArgs& a, const floatx16 (&acc)[2][NRB][2], float us,
                                           float2* __restrict__ sums, int p, int m, int v0, int nk, int k1_0, bool two,
                                           int tid, float* __restrict__ part) {
  const int lane = tid & 63, wv = tid >> 6;
  float2* out = reinterpret_cast<float2*>(part + (((size_t)p * a.M + m) * a.F) * 2);
#pragma unroll
  for (int i = 0; i < NRB; ++i) {
    if (i == 1 && !two) break;
#pragma unroll
    for (int jc = 0; jc < 2; ++jc) {
      __syncthreads();
#pragma unroll
      for (int v = 0; v < 16; ++v)
        sums[(wv * 16 + v) * 64 + lane] = make_float2(acc[0][i][jc][v] * us, acc[1][i][jc][v] * us);
      __syncthreads();
#pragma unroll
      for (int e0 = 0; e0 < 1024; e0 += 256) {
        const int e = e0 + tid, v = e >> 6, l = e & 63;
        const int row = 32 * i + 8 * (v >> 2) + 4 * (l >> 5) + (v & 3), k2 = 32 * jc + (l & 31);
        if (row < nk) {
          int k = (k1_0 + row) * K2 + k2;
          bool in = true;
          if (ROWS) {
            const int r0 = a.rows[v0 + row].x, r1 = a.rows[v0 + row + 1].x;
            k = (r0 & ~(K2 - 1)) + k2;
            in = k >= r0 && k < r1;
          }
          if (in) {
            float2 t = sums[e];
#pragma unroll
            for (int w = 1; w < 4; ++w) {
              const float2 o = sums[w * 1024 + e];
              t.x += o.x;
              t.y += o.y;
            }
            out[k] = t;
          }
        }
      }
    }
  }
}

// Workgroup = (record chunk p, receiver m, tile of 64 rows), four waves, each with records of its own: a
// wave sets up 64 records (one per lane), writes the generating factors of U of them to its own LDS, and per
// 16 records forms X and Y straight into the registers that the matrix instruction takes
// (v_mfma_f32_32x32x16_f16: lane l holds records 8 (l / 32) .. + 7 of row, or bin, l % 32) and contracts the
// whole 64 x 64 tile, accumulating Re and Im.  The blocks go in serpentine order (X0 Ya, X0 Yb, X1 Yb, X1 Ya,
// then Yb first), so that one operand is free at a time, and the next one is formed between the twelve
// products of a block: the matrix pipe works through the forming of the operands.  At the end the
// four waves' sums are added in wave order and written as the chunk's partial spectrum.
// What bounds it: per 32 records and receiver about 3100 cycles of a SIMD's matrix pipe and 4500 of its vector
// unit (products and splits of the operands 1900, factors 1500, set-up 900).  The form before this one
// shared the operands of four waves through LDS (64 KB read and 32 KB written per 32 records besides the
// factors, LDS busy two thirds of the time, two barriers per stage, matrix and vector work one after the other).
// Measured: 2.9 million records x 32 receivers x 4096 bins 10.7 -> 9.2 ms (992 TFLOP/s executed, 82% of the 1.2 PFLOP/s
// that a large fp16 product reaches on the card: under this load the clock falls to 2.05 GHz), 100,000 x 16 x
// 2048 158 -> 140 us.
// NRB: blocks of 32 rows (1: tiles of at most 32 rows).
// FOLD 4 (8): every band edge falls on a multiple of 4 (8) outer indices and the grid holds whole groups of
// that many (bins a multiple of 256, 512): the band factor rides on Xa.  FOLD 0: other bands on whole runs of 64 bins,
// rows from the row table, a band factor per (segment, record).
// DIR: some pose has a receiver directivity.
template <bool BATCH, int NRB, int FOLD, bool DIR>
__global__ __launch_bounds__(256, 2) void k_synth_mfma(SynthArgs a0, const SynthArgs* __restrict__ jobs,
                                                                      ChunkTab ct, et_paths P,
                                                                      const int32_t* __restrict__ idx, const Ctl* ctl,
                                                                      float* __restrict__ part) {
  SYNTH_RESOLVE();
  // records per generation: 64 (a lane per record) where the factors of two workgroups fit a CU's 160 KB; with a
  // directivity and two row blocks 64 would spill 50 registers in the loop (foliage pose 8.30 ms, 32 records 7.96 ms)
  constexpr int U = (FOLD == 8 && !(DIR && NRB == 2)) || (FOLD == 4 && NRB == 1) ? 64 : 32;
  using FT = Factors<NRB, FOLD, U>;
  constexpr size_t FAC_BYTES = sizeof(FT) * 4, SUM_BYTES = sizeof(float2) * 4 * 16 * 64;
  __shared__ __align__(16) char lds[FAC_BYTES > SUM_BYTES ? FAC_BYTES : SUM_BYTES];
  __shared__ int key[SMAX];
  __shared__ float red[4];
  const int p = bp, m = bm;
  const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, hf = lane >> 5;
  const int v0 = bt * KT1;                       // first row of the tile
  const int nk = min(KT1, (FOLD ? a.F / K2 : a.nrows) - v0);   // its rows
  if (nk <= 0) return;                           // (a batch's job with fewer rows than others)
  int k1_0 = v0, nk1 = nk;                       // outer indices [k1_0, k1_0 + nk1) that the rows fall into
  int nseg = 0;
  int rinfo[NRB];                                // FOLD 0: of rows l32 + 32 i: outer index - k1_0 | segment << 8
  FT& W = reinterpret_cast<FT*>(lds)[wv];
  if (FOLD) {
    if (tid < 8) {
      const int r0 = (k1_0 + min(8 * tid, nk - 1)) * K2, r1 = (k1_0 + min(8 * tid + 4, nk - 1)) * K2;
      uint32_t kb = (uint32_t)band_of(r0, a.Bk, a.F) | (uint32_t)band_of(r1, a.Bk, a.F) << 16;
      if (a.Bd) kb |= (uint32_t)band_of(r0, a.Bd, a.F) << 8 | (uint32_t)band_of(r1, a.Bd, a.F) << 24;
      key[tid] = (int)kb;
    }
  } else {
    tile_rows<NRB>(a, v0, nk, lane, wv, key, k1_0, nk1, nseg, rinfo);
    if (hf == 0) W.bf[nseg][l32] = 0.f;   // rows past the tile take the extra segment, whose factor is zero
  }
  if (U == 64) W.f[FT::XB][lane] = W.f[FT::YA][lane] = W.f[FT::YB][lane] = make_float2(1.f, 0.f);
  __syncthreads();
  const float dmax = DIR ? dir_log2_max(a, m, tid, red) : 0.f;
  const bool two = NRB == 2 && nk > 32;          // rows in the second block
  floatx16 acc[2][NRB][2];                       // [re, im][row block][column block]
#pragma unroll
  for (int c = 0; c < 2; ++c)
#pragma unroll
    for (int i = 0; i < NRB; ++i)
#pragma unroll
      for (int jc = 0; jc < 2; ++jc)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[c][i][jc][v] = 0.f;
  float E = -INFINITY;   // current exponent bound of the wave
  // the wave's share of the chunk: whole pairs of steps, 32 records
  const int64_t pw = ((hi - lo + 3) / 4 + 31) / 32 * 32;
  const int64_t wlo = lo + wv * pw, whi = min(wlo + pw, hi);
  int64_t rec = 0;       // this lane's record of the group (the range's last one past its end), read a group ahead
  if (wlo < whi) rec = record_at(idx, min(wlo + lane, whi - 1));
  for (int64_t g = wlo; g < whi; g += 64) {
    PairLean q;
    pair_fwd<DIR>(a, P, rec, g + lane < whi, m, dmax, q);
    rec = record_at(idx, min(g + 64 + lane, whi - 1));
    const float Eg = ceilf(wave_max(record_bound(q, k1_0, nk1)));
    if (Eg > E) {
      if (E != -INFINITY) {
        const float r = exp2f(E - Eg);
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
          for (int i = 0; i < NRB; ++i)
#pragma unroll
            for (int jc = 0; jc < 2; ++jc) acc[c][i][jc] *= r;
      }
      E = Eg;
    }
    const float esh = E != -INFINITY ? XTOP - E : 0.f;
    const int nrec = (int)min<int64_t>(64, whi - g);
    for (int s = 0; U * s < nrec; ++s) {
      gen_factors_u<NRB, FOLD, U, DIR>(a, q, s, m, k1_0, nk1, lane, esh, nseg, key, W);
      const int steps = (min(U, nrec - U * s) + 31) / 32 * 2;   // of 16 records, in pairs
      // Where the factors of this lane's operands lie for its records (8 hf .. + 7) of a step: bin l32 + 32 jc, row
      // l32 + 32 i; o: the step's and the pair's offset.  (Formed here, from a lane number that the compiler
      // cannot carry over, so that the addresses hold no registers while the factors are generated.)
      int ln = lane;
      asm volatile("" : "+v"(ln));
      constexpr int ROW = sizeof(W.f[0]), STEP = 16 * sizeof(float2);
      const int lb = ln & 31, lh8 = 8 * (ln >> 5);
      const char* const wb = reinterpret_cast<const char*>(&W) + lh8 * sizeof(float2);
      const char* const py_a = wb + (FT::YA + (lb >> 3)) * ROW;
      const char* const py_b = wb + (FT::YB + (lb & 7)) * ROW;
      const char *px_a[NRB], *px_b[NRB], *px_f[NRB];
#pragma unroll
      for (int i = 0; i < NRB; ++i) {
        const int ri = FOLD ? 0 : rinfo[i];
        const int ga = FOLD ? (lb >> 3) + 4 * i : (ri & 63) >> 3, gb = FOLD ? lb & 7 : ri & 7;
        px_a[i] = wb + (FOLD == 4 && (lb & 4) ? FT::XH + ga : ga) * ROW;
        px_b[i] = wb + (FT::XB + gb) * ROW;
        px_f[i] = reinterpret_cast<const char*>(&W.bf[FOLD == 0 ? ri >> 8 : 0][0]) + lh8 * sizeof(float);
      }
      auto load_y = [&](Pair2& t, int jc, int o, int e) { t.load(py_a + 4 * jc * ROW + o + 16 * e, py_b + o + 16 * e); };
      auto load_x = [&](Pair2& t, int i, int o, int e) {
        const int ii = i < NRB ? i : 0;
        if (FOLD) t.load(px_a[0] + 4 * ii * ROW + o + 16 * e, px_b[0] + o + 16 * e);
        else t.load(px_a[ii] + o + 16 * e, px_b[ii] + o + 16 * e);
      };
      auto scale_x = [&](Pair2& t, int i, int o, int e) { if (FOLD == 0) t.scale(px_f[i < NRB ? i : 0] + o / 2 + 8 * e); };
      Operand x0, x1, ya, yb;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        Pair2 t, u;
        load_x(t, 0, 0, e);
        load_y(u, 0, 0, e);
        scale_x(t, 0, 0, e);
        t.multiply();
        u.multiply();
        t.split(e, x0);
        u.split(e, ya);
      }
      // The slices of a block that form one operand: two records at a time, loaded three products ahead,
      // multiplied after one product and split after the next (about seven vector instructions per product,
      // which take as long as the product does).
      Pair2 t[2];
#define ET_SLICE_Y(JC, O, DST)                                                      \
  [&](int k) {                                                                      \
    if (k >= 4 && k % 2 == 0 && k <= 10) t[(k - 4) / 2 % 2].split((k - 4) / 2, DST); \
    if (k % 2 == 0 && k < 8) load_y(t[k / 2 % 2], JC, O, k / 2);                    \
    if (k >= 3 && k % 2 == 1 && k <= 9) t[(k - 3) / 2 % 2].multiply();              \
  }
#define ET_SLICE_X(I, O, DST)                                                       \
  [&](int k) {                                                                      \
    if (k >= 4 && k % 2 == 0 && k <= 10) t[(k - 4) / 2 % 2].split((k - 4) / 2, DST); \
    if (k % 2 == 0 && k < 8) load_x(t[k / 2 % 2], I, O, k / 2);                     \
    if (k >= 3 && k % 2 == 1 && k <= 9) {                                           \
      scale_x(t[(k - 3) / 2 % 2], I, O, (k - 3) / 2);                               \
      t[(k - 3) / 2 % 2].multiply();                                                \
    }                                                                               \
  }
      if constexpr (NRB == 2) {
        for (int st = 0; st < steps; st += 2) {
          const int o = st * STEP, on = o + STEP, onn = st + 2 < steps ? o + 2 * STEP : o;
          contract12(x0, ya, acc[0][0][0], acc[1][0][0], ET_SLICE_Y(1, o, yb));
          contract12(x0, yb, acc[0][0][1], acc[1][0][1], ET_SLICE_X(1, o, x1));
          contract12(x1, yb, acc[0][NRB - 1][1], acc[1][NRB - 1][1], ET_SLICE_X(0, on, x0));
          contract12(x1, ya, acc[0][NRB - 1][0], acc[1][NRB - 1][0], ET_SLICE_Y(1, on, yb));
          contract12(x0, yb, acc[0][0][1], acc[1][0][1], ET_SLICE_Y(0, on, ya));
          contract12(x0, ya, acc[0][0][0], acc[1][0][0], ET_SLICE_X(1, on, x1));
          contract12(x1, ya, acc[0][NRB - 1][0], acc[1][NRB - 1][0], ET_SLICE_X(0, onn, x0));
          contract12(x1, yb, acc[0][NRB - 1][1], acc[1][NRB - 1][1], ET_SLICE_Y(0, onn, ya));
        }
      } else {
        Pair2 u[2];
        Operand y1;
        for (int st = 0; st < steps; ++st) {
          const int o = st * STEP, on = st + 1 < steps ? o + STEP : o;
          contract12(x0, ya, acc[0][0][0], acc[1][0][0], ET_SLICE_Y(1, o, yb));
          contract12(x0, yb, acc[0][0][1], acc[1][0][1], [&](int k) {
            if (k >= 4 && k % 2 == 0 && k <= 10) {
              t[(k - 4) / 2 % 2].split((k - 4) / 2, x1);
              u[(k - 4) / 2 % 2].split((k - 4) / 2, y1);
            }
            if (k % 2 == 0 && k < 8) {
              load_x(t[k / 2 % 2], 0, on, k / 2);
              load_y(u[k / 2 % 2], 0, on, k / 2);
            }
            if (k >= 3 && k % 2 == 1 && k <= 9) {
              scale_x(t[(k - 3) / 2 % 2], 0, on, (k - 3) / 2);
              t[(k - 3) / 2 % 2].multiply();
              u[(k - 3) / 2 % 2].multiply();
            }
          });
          x0 = x1;
          ya = y1;
        }
      }
#undef ET_SLICE_X
#undef ET_SLICE_Y
      __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");   // the factors are rewritten next
      __builtin_amdgcn_wave_barrier();
    }
  }
  write_tile<NRB, FOLD == 0>(a, acc, E != -INFINITY ? exp2f(E - XTOP) : 0.f, reinterpret_cast<float2*>(lds), p, m, v0, nk,
                             k1_0, two, tid, part);
}

// ------------------------------------------------------------------ factorised FP32 kernel

// The factorised sum for bands that end inside a block of 64 bins, over the rows of the row table.  What a row does
// not hold of its 64 bins is computed and dropped.  Everything is FP32 or more: the operands go to the FP32 matrix
// cores as they are, so that a band or a path far below the tile's largest keeps its own precision, as per term
// (halves under one exponent per tile lose it: 5e-4 of a band 1e-7 below the others), and the factors' exponents and
// phases are reduced exactly, so that four factors per term add no more error than the one of a term by itself.

// The generating factors of a wave's 32 records, rows [factor][record] as in Factors: Xa of the 4 NRB groups of outer
// indices (without the amplitude at f_lo and the band), Xb, Ya and Yb (8 each); bf: amplitude at f_lo times band
// factor per (segment, record).
constexpr int RU = 32;
template <int NRB>
struct RowFactors {
  static constexpr int G = 4 * NRB, XB = G, YA = XB + 8, YB = YA + 8;
  float2 f[YB + 8][RU + 2];
  float bf[SMAX + 1][RU + 4];
};

// 2^lg, the whole part of lg exactly (zero, infinite or not a number where lg says so).
__device__ inline float exp2_64(double lg) {
  const double x = fmin(fmax(lg, -4096.0), 4096.0), n = rint(x);
  const float v = __builtin_amdgcn_ldexpf(__builtin_amdgcn_exp2f((float)(x - n)), (int)n);
  return lg == lg ? v : NAN;
}
// e^(2 pi j ph) of a phase in Q0.32 cycles: the nearest quarter turn exactly, the rest (at most an eighth) by the
// Taylor series of sine and cosine, whose first terms left out are 2e-9.
__device__ inline float2 cis_q32(uint32_t ph) {
  const uint32_t q = (ph + 0x20000000u) >> 30;
  const float t = (float)(int32_t)(ph - (q << 30)) * 1.4629180792671596e-9f;   // 2 pi 2^-32
  const float u = t * t;
  const float sn = t * fmaf(u, fmaf(u, fmaf(u, fmaf(u, 1.f / 362880.f, -1.f / 5040.f), 1.f / 120.f), -1.f / 6.f), 1.f);
  const float cs = fmaf(u, fmaf(u, fmaf(u, fmaf(u, fmaf(u, -1.f / 3628800.f, 1.f / 40320.f), -1.f / 720.f), 1.f / 24.f), -0.5f), 1.f);
  const float x = q & 1 ? sn : cs, y = q & 1 ? cs : sn;
  return make_float2((q ^ (q << 1)) & 2 ? -x : x, q & 2 ? -y : y);
}
// 2^(k slope) e^(2 pi j ph), slope = hi + lo with 12 bits in hi: k hi is exact for the multiples k that a factor takes (up
// to 3 bits and a power of two), and so is its fraction.
__device__ inline float2 row_factor(float k, float hi, float lo, uint32_t ph) {
  const float n = rintf(k * hi);
  const float amp = __builtin_amdgcn_ldexpf(__builtin_amdgcn_exp2f(fmaf(k, lo, fmaf(k, hi, -n))), (int)n);
  const float2 c = cis_q32(ph);
  return make_float2(amp * c.x, amp * c.y);
}

// Workgroup and waves as in k_synth_mfma.  A wave sets up 64 records and, 32 at a time, writes their factors to its own
// LDS; lane l forms X of row l % 32 (+ 32) and Y of bin l % 32 (+ 32) for records 4 j + 2 (l / 32) and the next, two
// steps of v_mfma_f32_32x32x2_f32 (a record per half wave).
// Bound by the FP32 matrix pipe where records are many (250,000 x 32 receivers x 2000 bins: 1.75 ms, 105 TFLOP/s
// executed, two thirds of the peak; per term 6.7 ms), and by the set-up and the factors of part-filled groups where a wave
// has few (60,000 x 6 receivers x 3000 bins in 7 bands: 129 us, matrix pipe 42% and vector unit 23% busy; per term 540).
// Error against 64 bits over 70 random grids of 192 to 4160 bins 1.7e-7 to 6.0e-7 of the norm, per term 2.1e-7 to 1.3e-6,
// lower in each.
template <bool BATCH, int NRB, bool DIR>
__global__ __launch_bounds__(256, 2) void k_synth_rows(SynthArgs a0, const SynthArgs* __restrict__ jobs, ChunkTab ct,
                                                       et_paths P, const int32_t* __restrict__ idx, const Ctl* ctl,
                                                       float* __restrict__ part) {
  SYNTH_RESOLVE();
  using FT = RowFactors<NRB>;
  constexpr size_t FAC_BYTES = sizeof(FT) * 4, SUM_BYTES = sizeof(float2) * 4 * 16 * 64;
  __shared__ __align__(16) char lds[FAC_BYTES > SUM_BYTES ? FAC_BYTES : SUM_BYTES];
  __shared__ int key[SMAX];
  const int m = bm;
  const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, hf = lane >> 5;
  const int v0 = bt * KT1;                       // first row of the tile
  const int nk = min(KT1, a.nrows - v0);         // its rows
  if (nk <= 0) return;                           // (a batch's job with fewer rows than others)
  int k1_0, nk1, nseg, rinfo[NRB];
  tile_rows<NRB>(a, v0, nk, lane, wv, key, k1_0, nk1, nseg, rinfo);
  FT& W = reinterpret_cast<FT*>(lds)[wv];
  if (hf == 0) W.bf[nseg][l32] = 0.f;            // rows past the tile
  __syncthreads();
  const bool two = NRB == 2 && nk > 32;          // rows in the second block
  const float* dtab = a.dir + (size_t)m * a.Bd * a.El * a.Az;
  const size_t dcells = (size_t)a.El * a.Az;
  const bool dir = DIR && a.Bd != 0;
  floatx16 acc[2][NRB][2];
#pragma unroll
  for (int c = 0; c < 2; ++c)
#pragma unroll
    for (int i = 0; i < NRB; ++i)
#pragma unroll
      for (int jc = 0; jc < 2; ++jc)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[c][i][jc][v] = 0.f;
  const int64_t pw = ((hi - lo + 3) / 4 + 3) / 4 * 4;   // the wave's share of the chunk: whole steps of 4 records
  const int64_t wlo = lo + wv * pw, whi = min(wlo + pw, hi);
  for (int64_t g = wlo; g < whi; g += 64) {
    Pair q;
    DirCell cell{0, 0, 0, 0, 0.f, 0.f};
    bool ok = false;
    if (g + lane < whi) ok = pair_setup(a, P, record_at(idx, g + lane), m, q);
    // phases of the first row's first bin, and steps of 8 rows, a row, 8 bins and a bin
    uint32_t pa = 0, pa8 = 0, px = 0, py8 = 0, py = 0;
    float shi = 0.f, slo = 0.f;
    if (!ok) {
      q.base64 = q.slope64 = 0.0;
      q.gamma = 0.f;
      q.kind = q.mat = 0;
    } else {
      pa = q32(q.c0 + (double)(k1_0 * K2) * q.cb);
      pa8 = q32((double)(8 * K2) * q.cb);
      px = q32((double)K2 * q.cb);
      py8 = q32(8.0 * q.cb);
      py = q32(q.cb);
      shi = __uint_as_float(__float_as_uint((float)q.slope64) & 0xfffff000u);
      slo = (float)(q.slope64 - (double)shi);
    }
    if (dir && ok) {
      float vx, vy, vz;
      arrival(a, q, m, vx, vy, vz);
      cell = dir_cell(a.El, a.Az, vx, vy, vz);
    }
    const int nrec = (int)min<int64_t>(64, whi - g);
    for (int s = 0; RU * s < nrec; ++s) {
      const int r = l32, src = RU * s + r;       // lanes r and r + 32: half of record r's factors each
      {
        // (the tile's first row may lie at any multiple of the slope)
        const float amp0 = exp2_64(__shfl((double)(k1_0 * K2) * q.slope64, src));
        const float hi = __shfl(shi, src), lo = __shfl(slo, src);
        const uint32_t ba = (uint32_t)__shfl((int)pa, src), b8 = (uint32_t)__shfl((int)pa8, src);
#pragma unroll
        for (int jj = 0; jj < FT::G / 2; ++jj) {
          const int j = FT::G / 2 * hf + jj;
          const float2 v = row_factor((float)(8 * K2 * j), hi, lo, ba + (uint32_t)j * b8);
          W.f[j][r] = make_float2(amp0 * v.x, amp0 * v.y);
        }
        const uint32_t bx = (uint32_t)__shfl((int)px, src), by8 = (uint32_t)__shfl((int)py8, src), by = (uint32_t)__shfl((int)py, src);
#pragma unroll
        for (int jj = 0; jj < 4; ++jj) {
          const int j = 4 * hf + jj;
          W.f[FT::XB + j][r] = row_factor((float)(K2 * j), hi, lo, (uint32_t)j * bx);
          W.f[FT::YA + j][r] = row_factor((float)(8 * j), hi, lo, (uint32_t)j * by8);
          W.f[FT::YB + j][r] = row_factor((float)j, hi, lo, (uint32_t)j * by);
        }
      }
      {
        const double base = __shfl(q.base64, src);
        const float gamma = __shfl(q.gamma, src);
        const int mat = __shfl(q.mat, src), kind = __shfl(q.kind, src);
        const bool on = __shfl((int)ok, src) != 0;
        DirCell c = cell;
        if (dir) {
          c.r0 = __shfl(cell.r0, src); c.r1 = __shfl(cell.r1, src);
          c.i0 = __shfl(cell.i0, src); c.i1 = __shfl(cell.i1, src);
          c.ta = __shfl(cell.ta, src); c.te = __shfl(cell.te, src);
        }
        for (int sg = hf; sg < nseg; sg += 2) {
          float v = 0.f;
          if (on) {
            const int kb = key[sg];
            const int64_t at = (int64_t)mat * a.Bk + (kb & 0xffff);
            double lb = kind == 0 ? (double)a.lk[at] - (double)gamma * (double)gamma * (double)a.lc[at]
                                  : (double)(kind == 1 ? a.ld[at] : a.lp[kb & 0xffff]);
            if (dir) lb += (double)log2f(dir_lerp(dtab + (kb >> 16) * dcells, c));
            v = exp2_64(base + lb);
          }
          W.bf[sg][r] = v;
        }
      }
      // the factors are read back by other lanes of this wave only
      __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
      __builtin_amdgcn_wave_barrier();
      const float2 *px_a[NRB], *px_b[NRB];
      const float* px_f[NRB];
#pragma unroll
      for (int i = 0; i < NRB; ++i) {
        px_a[i] = &W.f[(rinfo[i] & 63) >> 3][2 * hf];
        px_b[i] = &W.f[FT::XB + (rinfo[i] & 7)][2 * hf];
        px_f[i] = &W.bf[rinfo[i] >> 8][2 * hf];
      }
      const float2 *py_a = &W.f[FT::YA + (l32 >> 3)][2 * hf], *py_b = &W.f[FT::YB + (l32 & 7)][2 * hf];
      constexpr int Y1 = 4 * (RU + 2);           // bins l + 32: four groups of 8 on
      const int n4 = (min(RU, nrec - RU * s) + 3) / 4;
      for (int j = 0; j < n4; ++j) {
        float2 y[2][2], x[NRB][2];               // [block][step]
#pragma unroll
        for (int jc = 0; jc < 2; ++jc) {
          const float4 u = *reinterpret_cast<const float4*>(py_a + jc * Y1 + 4 * j), v = *reinterpret_cast<const float4*>(py_b + 4 * j);
          y[jc][0] = cmul(make_float2(u.x, u.y), make_float2(v.x, v.y));
          y[jc][1] = cmul(make_float2(u.z, u.w), make_float2(v.z, v.w));
        }
#pragma unroll
        for (int i = 0; i < NRB; ++i) {
          const float4 u = *reinterpret_cast<const float4*>(px_a[i] + 4 * j), v = *reinterpret_cast<const float4*>(px_b[i] + 4 * j);
          const float2 f = *reinterpret_cast<const float2*>(px_f[i] + 4 * j);
          x[i][0] = cmul(make_float2(u.x * f.x, u.y * f.x), make_float2(v.x, v.y));
          x[i][1] = cmul(make_float2(u.z * f.y, u.w * f.y), make_float2(v.z, v.w));
        }
#pragma unroll
        for (int i = 0; i < NRB; ++i) {
          if (i == 1 && !two) break;
#pragma unroll
          for (int st = 0; st < 2; ++st) {
#pragma unroll
            for (int jc = 0; jc < 2; ++jc) {
              acc[0][i][jc] = __builtin_amdgcn_mfma_f32_32x32x2f32(x[i][st].x, y[jc][st].x, acc[0][i][jc], 0, 0, 0);
              acc[1][i][jc] = __builtin_amdgcn_mfma_f32_32x32x2f32(x[i][st].x, y[jc][st].y, acc[1][i][jc], 0, 0, 0);
            }
#pragma unroll
            for (int jc = 0; jc < 2; ++jc) {
              acc[0][i][jc] = __builtin_amdgcn_mfma_f32_32x32x2f32(-x[i][st].y, y[jc][st].y, acc[0][i][jc], 0, 0, 0);
              acc[1][i][jc] = __builtin_amdgcn_mfma_f32_32x32x2f32(x[i][st].y, y[jc][st].x, acc[1][i][jc], 0, 0, 0);
            }
          }
        }
      }
      __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");   // the factors are rewritten next
      __builtin_amdgcn_wave_barrier();
    }
  }
  write_tile<NRB, true>(a, acc, 1.f, reinterpret_cast<float2*>(lds), bp, m, v0, nk, k1_0, two, tid, part);
}

// ------------------------------------------------------------------ direct kernel

constexpr int DB = 256;       // threads
constexpr int DPT = 4;        // bins per thread
constexpr int DTILE = DB * DPT;
constexpr int DRB = 64;       // records per batch
constexpr int DBMAX = 64;

struct DirectLds {
  uint32_t a32[DRB], b32[DRB];
  float base[DRB], slope[DRB];
  float band[DRB][DBMAX];
  float dirl[DRB][DBMAX];
};

template <bool BATCH>
__global__ __launch_bounds__(DB) void k_synth_direct(SynthArgs a0, const SynthArgs* __restrict__ jobs, ChunkTab ct,
                                                     et_paths P, const int32_t* __restrict__ idx, const Ctl* ctl,
                                                     float* __restrict__ part) {
  SYNTH_RESOLVE();
  __shared__ DirectLds L;
  const int p = bp, m = bm;
  const int tid = threadIdx.x;
  const int kbase = bt * DTILE + tid * DPT;
  int bk[DPT], bd[DPT];
#pragma unroll
  for (int i = 0; i < DPT; ++i) {
    const int64_t k = kbase + i;
    bk[i] = (int)(((k < a.F ? k : a.F - 1) * a.Bk) / a.F);
    bd[i] = a.Bd ? (int)(((k < a.F ? k : a.F - 1) * a.Bd) / a.F) : 0;
  }
  float re[DPT], im[DPT];
#pragma unroll
  for (int i = 0; i < DPT; ++i) re[i] = im[i] = 0.f;
  for (int64_t n0 = lo; n0 < hi; n0 += DRB) {
    __syncthreads();
    if (tid < DRB) {
      const int64_t e = n0 + tid;
      Pair q;
      if (e < hi && pair_setup(a, P, idx ? (int64_t)idx[e] : e, m, q)) {
        // integer phase accumulator (Q0.32 cycles): phase_k = a32 + k b32 mod 2^32
        L.a32[tid] = (uint32_t)(uint64_t)llrint(frac(q.c0) * 4294967296.0);
        L.b32[tid] = (uint32_t)(uint64_t)llrint(frac(q.cb) * 4294967296.0);
        L.base[tid] = q.base;
        L.slope[tid] = q.slope;
        for (int b = 0; b < a.Bk; ++b) L.band[tid][b] = band_log2(a, q, b);
        if (a.Bd) {
          float vx, vy, vz;
          arrival(a, q, m, vx, vy, vz);
          const float* tab = a.dir + (size_t)m * a.Bd * a.El * a.Az;
          for (int b = 0; b < a.Bd; ++b) L.dirl[tid][b] = log2f(dir_gain(tab + (size_t)b * a.El * a.Az, a.El, a.Az, vx, vy, vz));
        }
      } else {
        L.a32[tid] = 0; L.b32[tid] = 0;
        L.base[tid] = -INFINITY; L.slope[tid] = 0.f;
        for (int b = 0; b < a.Bk; ++b) L.band[tid][b] = 0.f;
        for (int b = 0; b < a.Bd; ++b) L.dirl[tid][b] = 0.f;
      }
    }
    __syncthreads();
    const int nb = (int)min<int64_t>(DRB, hi - n0);
    for (int r = 0; r < nb; ++r) {
      const uint32_t A32 = L.a32[r], B32 = L.b32[r];
      const float base = L.base[r], slope = L.slope[r];
#pragma unroll
      for (int i = 0; i < DPT; ++i) {
        const int k = kbase + i;
        const uint32_t ph = A32 + (uint32_t)k * B32;
        const float rev = (float)(int32_t)ph * 2.3283064365386963e-10f;   // 2^-32
        float lg = base + (float)k * slope + L.band[r][bk[i]];
        if (a.Bd) lg += L.dirl[r][bd[i]];
        const float amp = exp2f(lg);
        re[i] += amp * __builtin_amdgcn_cosf(rev);
        im[i] += amp * __builtin_amdgcn_sinf(rev);
      }
    }
  }
  float* out = part + (((size_t)p * a.M + m) * a.F) * 2;
#pragma unroll
  for (int i = 0; i < DPT; ++i) {
    const int k = kbase + i;
    if (k < a.F) { out[2 * k] = re[i]; out[2 * k + 1] = im[i]; }
  }
}

// Sum of the chunks' partial spectra: a workgroup takes 64 complex outputs, its S waves the chunks w,
// w + S, ... each (eight loads in flight), and the S sums are added in wave order, so the result does not
// depend on scheduling.  S = 16 while the outputs alone leave the chip idle: one thread per output walked
// its 256 chunks one load after the other (68 us for 2 x 1024 bins).
template <int S>
__global__ __launch_bounds__(64 * S) void k_reduce_partials(const float2* __restrict__ part, int32_t P, int64_t MF,
                                                            float2* __restrict__ out) {
  __shared__ float2 red[S][64];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int64_t i = (int64_t)blockIdx.x * 64 + lane;
  float2 s = make_float2(0.f, 0.f);
  if (i < MF) {
    int c = w;
    for (; c + 7 * S < P; c += 8 * S) {
      float2 v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) v[u] = part[(size_t)(c + u * S) * MF + i];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        s.x += v[u].x;
        s.y += v[u].y;
      }
    }
    for (; c < P; c += S) {
      const float2 v = part[(size_t)c * MF + i];
      s.x += v.x;
      s.y += v.y;
    }
  }
  red[w][lane] = s;
  __syncthreads();
  if (w == 0 && i < MF) {
#pragma unroll
    for (int k = 1; k < S; ++k) {
      s.x += red[k][lane].x;
      s.y += red[k][lane].y;
    }
    out[i] = s;
  }
}

void reduce_partials(const float* part, int32_t P, int64_t MF, float* out, hipStream_t s) {
  const unsigned nb = (unsigned)((MF + 63) / 64);
  // sixteen waves per 64 outputs up to 64 K outputs (1024 workgroups of sixteen waves fill the chip twice)
  if (MF <= 65536 && P > 8)
    k_reduce_partials<16><<<nb, 1024, 0, s>>>((const float2*)part, P, MF, (float2*)out);
  else
    k_reduce_partials<4><<<nb, 256, 0, s>>>((const float2*)part, P, MF, (float2*)out);
}

// ------------------------------------------------------------------ adjoint

constexpr int GB = 256;
constexpr int GANCHOR = 32;   // bins between exact re-anchoring of the rotation recurrence

template <bool BATCH>
__global__ __launch_bounds__(GB) void k_synth_bwd(SynthArgs a0, const SynthArgs* __restrict__ jobs, ChunkTab ct,
                                                 et_paths P, const int32_t* __restrict__ idx, const Ctl* ctl,
                                                 const float* __restrict__ g, double* __restrict__ gpx,
                                                 double* __restrict__ gpk) {
  SYNTH_RESOLVE();
  if (BATCH) g += (size_t)jb * a.M * a.F * 2;
  extern __shared__ float2 gl[];   // dL/dconj(H) of this receiver, [F]
  __shared__ double red[GB];
  __shared__ double kval[16][GB];
  __shared__ int kmat[GB];
  __shared__ double kacc[16 * 16];
  const int p = bp, m = bm, tid = threadIdx.x;
  for (int k = tid; k < a.F; k += GB) gl[k] = make_float2(g[((size_t)m * a.F + k) * 2], g[((size_t)m * a.F + k) * 2 + 1]);
  for (int i = tid; i < a.Q * a.Bk; i += GB) kacc[i] = 0.0;
  double gx0 = 0, gx1 = 0, gx2 = 0;
  const double ln10 = 2.30258509299404568402;
  __syncthreads();
  for (int64_t n0 = lo; n0 < hi; n0 += GB) {
    const int64_t e = n0 + tid;
    double sb[16];
#pragma unroll
    for (int b = 0; b < 16; ++b) sb[b] = 0.0;
    int mat = -1;
    Pair q;
    int64_t n = -1;
    if (e < hi) n = idx[e];
    if (n >= 0 && pair_setup(a, P, n, m, q)) {
      mat = q.kind == 0 ? q.mat : -1;
      // step of the rotation recurrence: exp2(slope) e^{j 2 pi cb}
      const float wrev = (float)frac(q.cb);
      const float wamp = exp2f(q.slope);
      const float wr = wamp * __builtin_amdgcn_cosf(wrev), wi = wamp * __builtin_amdgcn_sinf(wrev);
      // S_b = sum_{k in band b} conj(g_k) T_k and S1 = sum_k f_k conj(g_k) T_k.  Within a
      // block of GANCHOR bins the FP32 sums carry the small weights (k - ka); blocks combine
      // in FP64 as S1 += f_ka sum z + df sum (k - ka) z.
      double s1r = 0.0, s1i = 0.0;
      // receiver directivity: direction of arrival in the receiver frame, and the sum over
      // directivity bands d of Re(S_d) grad_v ln D_d(v)
      float vx = 0.f, vy = 0.f, vz = 0.f;
      if (a.Bd) arrival(a, q, m, vx, vy, vz);
      double gvx = 0.0, gvy = 0.0, gvz = 0.0;
      for (int b = 0; b < a.Bk; ++b) {
        const int k0 = (int)(((int64_t)b * a.F + a.Bk - 1) / a.Bk);
        const int k1 = (int)(((int64_t)(b + 1) * a.F + a.Bk - 1) / a.Bk);
        // specular records: the band's terms without the factor k (H is linear in k, Eq. 2, so
        // this sum is dH/dk also where k = 0); k multiplies the band's share of the other sums
        const float blog = q.kind == 0 ? -q.gamma * q.gamma * a.lc[(int64_t)q.mat * a.Bk + b] : band_log2(a, q, b);
        const double kf = q.kind == 0 ? (double)a.refl_k[(int64_t)q.mat * a.Bk + b] : 1.0;
        double sbr = 0.0, b1r = 0.0, b1i = 0.0, bgx = 0.0, bgy = 0.0, bgz = 0.0;
        // the band's bins in runs of one directivity band (one run without directivity)
        for (int ks = k0; ks < k1;) {
          int kr = k1;
          float dlog = 0.f, dgx = 0.f, dgy = 0.f, dgz = 0.f;
          if (a.Bd) {
            const int d = (int)(((int64_t)ks * a.Bd) / a.F);
            kr = min(k1, (int)(((int64_t)(d + 1) * a.F + a.Bd - 1) / a.Bd));
            const float D = dir_gain_dv(a.dir + ((size_t)m * a.Bd + d) * a.El * a.Az, a.El, a.Az, vx, vy, vz, dgx,
                                        dgy, dgz);
            dlog = log2f(D);
            const float iD = D > 0.f ? 1.f / D : 0.f;
            dgx *= iD; dgy *= iD; dgz *= iD;
          }
          double srun = 0.0;
          for (int ka = ks; ka < kr; ka += GANCHOR) {
            const int ke = min(ka + GANCHOR, kr);
            const float rev = (float)frac(q.c0 + (double)ka * q.cb);
            const float amp = exp2f(q.base + (float)ka * q.slope + blog + dlog);
            float tr = amp * __builtin_amdgcn_cosf(rev), ti = amp * __builtin_amdgcn_sinf(rev);
            float w = 0.f;
            float c0r = 0.f, c0i = 0.f, c1r = 0.f, c1i = 0.f;
            for (int k = ka; k < ke; ++k) {
              const float2 gg = gl[k];
              const float zr = gg.x * tr + gg.y * ti;   // Re(conj(g) T)
              const float zi = gg.x * ti - gg.y * tr;   // Im(conj(g) T)
              c0r += zr;
              c0i += zi;
              c1r += w * zr;
              c1i += w * zi;
              const float nr = tr * wr - ti * wi;
              ti = tr * wi + ti * wr;
              tr = nr;
              w += 1.f;
            }
            const double fa = a.f_lo + (double)ka * a.df;
            srun += (double)c0r;
            b1r += fa * (double)c0r + a.df * (double)c1r;
            b1i += fa * (double)c0i + a.df * (double)c1i;
          }
          sbr += srun;
          bgx += srun * (double)dgx; bgy += srun * (double)dgy; bgz += srun * (double)dgz;
          ks = kr;
        }
        s1r += kf * b1r;
        s1i += kf * b1i;
        gvx += kf * bgx; gvy += kf * bgy; gvz += kf * bgz;
#pragma unroll
        for (int bb = 0; bb < 16; ++bb)
          if (bb == b) sb[bb] = sbr;
      }
      // sb: band sums without k for specular records; s0 = sum over bands of k * sb
      double s0 = 0;
#pragma unroll
      for (int b = 0; b < 16; ++b)
        if (b < a.Bk) s0 += (q.kind == 0 ? (double)a.refl_k[(int64_t)q.mat * a.Bk + b] : 1.0) * sb[b];
      // d(ln A + j phi)/dx_m = [(-p/r - ln10 (a0 + a1 f)/20) + j sigma 2 pi f / c] u - d(gamma^2)/dx / (2 beta^2)
      const double cu = (-a.ps / q.r - ln10 * a.A0 / 20.0) * s0 - ln10 * a.A1 / 20.0 * (double)s1r -
                        (double)a.sigma * 2.0 * M_PI / a.c * (double)s1i;
      double g0 = 2.0 * cu * q.u[0], g1 = 2.0 * cu * q.u[1], g2 = 2.0 * cu * q.u[2];
      if (q.kind == 0) {
        const double dx = P.dout[3 * n], dy = P.dout[3 * n + 1], dz = P.dout[3 * n + 2];
        const double dnn = sqrt(dx * dx + dy * dy + dz * dz);
        const double hx = dx / dnn, hy = dy / dnn, hz = dz / dnn;
        const double cg = hx * q.u[0] + hy * q.u[1] + hz * q.u[2];
        const double qx = hy * q.u[2] - hz * q.u[1], qy = hz * q.u[0] - hx * q.u[2], qz = hx * q.u[1] - hy * q.u[0];
        const double sg = sqrt(qx * qx + qy * qy + qz * qz);
        const double gam = atan2(sg, cg);
        const double ratio = gam < 1e-8 ? 2.0 : 2.0 * gam / sg;
        // d(gamma^2)/dx = -(2 gamma / sin gamma) (d' - cos(gamma) u) / l
        const double d0 = -ratio * (hx - cg * q.u[0]) / q.l, d1 = -ratio * (hy - cg * q.u[1]) / q.l,
                     d2 = -ratio * (hz - cg * q.u[2]) / q.l;
        double wsum = 0.0;
#pragma unroll
        for (int b = 0; b < 16; ++b) {
          if (b < a.Bk) {
            const double bt = (double)a.beta[q.mat * a.Bk + b];
            wsum += (double)a.refl_k[q.mat * a.Bk + b] * sb[b] / (2.0 * bt * bt);
          }
        }
        g0 -= 2.0 * wsum * d0; g1 -= 2.0 * wsum * d1; g2 -= 2.0 * wsum * d2;
        // dL/dk of the record's (material, band): 2 Re sum conj(g) dT/dk
#pragma unroll
        for (int b = 0; b < 16; ++b) sb[b] = 2.0 * sb[b];
      }
      if (a.Bd) {
        // v = -R^T u and du/dx_m = (I - u u^T) / l: d ln D / dx_m = -(I - u u^T) R grad_v ln D / l
        double w0 = gvx, w1 = gvy, w2 = gvz;
        if (a.rx_rot) {
          const double* R = a.rx_rot + 9 * m;
          w0 = R[0] * gvx + R[1] * gvy + R[2] * gvz;
          w1 = R[3] * gvx + R[4] * gvy + R[5] * gvz;
          w2 = R[6] * gvx + R[7] * gvy + R[8] * gvz;
        }
        const double uw = q.u[0] * w0 + q.u[1] * w1 + q.u[2] * w2;
        const double c = 2.0 / q.l;
        g0 -= c * (w0 - uw * q.u[0]);
        g1 -= c * (w1 - uw * q.u[1]);
        g2 -= c * (w2 - uw * q.u[2]);
      }
      gx0 += g0; gx1 += g1; gx2 += g2;
    }
    // deterministic per-batch reduction of the band-coefficient gradient by material
    kmat[tid] = mat;
#pragma unroll
    for (int b = 0; b < 16; ++b) kval[b][tid] = sb[b];
    __syncthreads();
    for (int i = tid; i < a.Q * a.Bk; i += GB) {
      const int qq = i / a.Bk, b = i % a.Bk;
      double s = 0.0;
      for (int t = 0; t < GB; ++t)
        if (kmat[t] == qq) s += kval[b][t];
      kacc[i] += s;
    }
    __syncthreads();
  }
  // receiver gradient: block tree reduction
  const double gv[3] = {gx0, gx1, gx2};
  for (int c = 0; c < 3; ++c) {
    red[tid] = gv[c];
    __syncthreads();
    for (int s = GB / 2; s > 0; s >>= 1) {
      if (tid < s) red[tid] += red[tid + s];
      __syncthreads();
    }
    if (tid == 0) gpx[((size_t)p * a.M + m) * 3 + c] = red[0];
    __syncthreads();
  }
  for (int i = tid; i < a.Q * a.Bk; i += GB) gpk[((size_t)p * a.M + m) * a.Q * a.Bk + i] = kacc[i];
}

// Factorised adjoint.  For record n and receiver m the adjoint needs, per material band b,
//   S_b = sum_{k in b} conj(g_k) T_k   and   S1 = sum_k f_k conj(g_k) T_k,
// with T_k = X[k1] Y[k2] as in the forward kernel and G = conj(g) as a [k1][k2] matrix:
//   S_b = sum_{k1 in b} X[k1] Z[k1],   Z[k1]  = sum_k2 G[k1, k2] Y[k2],
//   S1  = sum_k1 X[k1] Z'[k1],         Z'[k1] = sum_k2 f_k G[k1, k2] Y[k2],
// f_k the frequency of bin k = 64 k1 + k2.  Z and Z' are complex matrix products contracting
// over k2 on the f16 matrix cores with split operands (as in the forward kernel): G = conj(g)
// and f_k G sit in registers as halves, each scaled into the f16 range by a power of two per
// wave, and Y is written as halves, record-major (8 inner indices per lane, 16-byte reads).
// The per-row products go to LDS; per record, band sums and the weighted sum run in FP32 in a
// fixed order, and the chain rule of the direct adjoint turns them into dL/dk and dL/dx_m
// (accumulated over records in FP64).
// LDS record stride of the adjoint's per-row products R0: with 68 = 4 (mod 64) the 16-byte
// writes of four consecutive rows are conflict-free per quarter wave.
constexpr int BS68 = 68;

// Group-major sums (stride 36): the eight threads of each of a wave's eight records reading
// groups 2 j + i fall on 64 distinct banks.
// X carries the band factor without k for specular records: Re(X Z) summed over a band's rows
// is then dH/dk of that band (also where k = 0), and k enters the other sums per row.
constexpr int YROW = 9;     // halfx8 per record row of Y halves: 64 inner indices and a pad (144-byte rows)
template <int FOLD>
struct __align__(16) BwdBuf {
  halfx8 Y[4][RB][YROW];     // Y halves [re hi, re lo, im hi, im lo][record][chunk of 8 inner indices]
  float R0[FOLD ? 1 : RB][BS68];   // Re(X Z) per (record, row) (band edges off the 4-row groups)
  float Rg[FOLD ? 16 : 1][36];     // Re(X Z) summed over a group of 4 rows, per (group, record) (FOLD)
  float2 R1[16][36];         // sum over 4 rows of k X Z' per (row group, record)
  float kv[16][RB];          // 2 S_b of each specular record of the stage (0 for the others), [band][record]
  int32_t kmat[RB];          // the material of each specular record of the stage, -1 for the others
  double dk[4][256];         // per wave: dL/dk of (material, band) over its records so far
  float lobe_w[256];         // per (material, band): 1 / (2 beta^2)
  float kf[256 + 16];        // per (material, band): k; then a row of ones (records of other kinds)
  int32_t recb[RB];          // per record of the stage: its row of kf (mat Bk, or the ones row)
};

// The adjoint's matrix-product operand of the sub-stage's records: Y as f16 halves record-major,
// lane (r, c) = (lane / 8, lane % 8) forming inner indices 8 c .. 8 c + 7 of record r:
// Y[8 c + i] = Ya[c] Yb[i].  (X is formed where it is used, from the factors.)
template <int FOLD>
__device__ inline void write_bwd(const WaveScratch& W, int lane, int wv, BwdBuf<FOLD>& bb) {
  const int row0 = wv * RPW;
  const int r = lane >> 3, c = lane & 7;
  const float2 ya = W.ya[r][c];
  float yr[8], yi[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const float2 y = cmul(ya, W.yb[r][i]);
    yr[i] = y.x;
    yi[i] = y.y;
  }
  split8(yr, bb.Y[0][row0 + r][c], bb.Y[1][row0 + r][c]);
  split8(yi, bb.Y[2][row0 + r][c], bb.Y[3][row0 + r][c]);
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// Sum of v over each group of 8 consecutive lanes, valid in the group's first lane, added as
// ((v0 + v1) + (v2 + v3)) + ((v4 + v5) + (v6 + v7)) by lane moves within rows of 16 (no LDS).
__device__ inline float sum8_first(float v) {
  v += dpp_mov<0xB1>(v);    // quad_perm [1, 0, 3, 2]: lane ^ 1
  v += dpp_mov<0x4E>(v);    // quad_perm [2, 3, 0, 1]: lane ^ 2
  v += dpp_mov<0x104>(v);   // row_shl 4: lane + 4 within the row
  return v;
}

// dL/dk over the wave's 8 records n of the stage (8 wv .. 8 wv + 7): (material q, band b) adds
// 2 S_b of the specular records of material q.  As a matrix product, kv [band][record] times the
// records' one-hot materials [record][material], on the FP32 matrix cores (the products are
// exact: 0 or the value) in tiles of 16 materials; each lane adds its four sums to the wave's
// FP64 totals in LDS (one lane per (material, band)).  With at most 16 materials the sums stay
// in the FP32 accumulator dkc over a group of 8 stages (64 records) and go to the totals when
// flush is set.  Every lane of the wave calls it.
template <int FOLD>
__device__ inline void dk_wave(BwdBuf<FOLD>& bb, int wv, int lane, int Q, int Bk, floatx4& dkc, bool flush) {
  const int col = lane & 15;   // A: band row; B: material column within the tile
  float av[2];
  int mv[2];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int n = 8 * wv + 4 * h + (lane >> 4);
    av[h] = col < Bk ? bb.kv[col][n] : 0.f;
    mv[h] = bb.kmat[n];
  }
  if (Q <= 16) {
#pragma unroll
    for (int h = 0; h < 2; ++h) dkc = __builtin_amdgcn_mfma_f32_16x16x4f32(av[h], mv[h] == col ? 1.f : 0.f, dkc, 0, 0, 0);
    if (flush) {
      if (col < Q) {
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int b = 4 * (lane >> 4) + v;
          if (b < Bk) bb.dk[wv][col * Bk + b] += (double)dkc[v];
        }
      }
      dkc = floatx4{0.f, 0.f, 0.f, 0.f};
    }
    return;
  }
  for (int q0 = 0; q0 < Q; q0 += 16) {
    floatx4 c = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int h = 0; h < 2; ++h) c = __builtin_amdgcn_mfma_f32_16x16x4f32(av[h], mv[h] == q0 + col ? 1.f : 0.f, c, 0, 0, 0);
    // c[v]: band 4 (lane / 16) + v, material q0 + lane % 16
    const int qq = q0 + col;
    if (qq < Q) {
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int b = 4 * (lane >> 4) + v;
        if (b < Bk) bb.dk[wv][qq * Bk + b] += (double)c[v];
      }
    }
  }
}

// FOLD 4 (8): every band edge of the grid falls on a group of 4 (8) rows (a multiple of 256, 512
// bins) and the grid holds whole groups: each lane's four rows of the matrix-product output belong
// to one band and are summed in registers, and the band factor rides on Xa as in the forward
// kernel.
// Bound by latency between its phases (factors, products, row sums, record sums, with two barriers a stage of 32
// records): matrix cores 21%, vector units 36% busy with two workgroups per CU.  With folded bands and at most 32 rows
// the buffers leave room for three (51 KB of LDS, 168 registers, 11 spilled outside the stages): 100,000
// records x 16 receivers x 2048 bins 443 -> 372 us, a batch's adjoint 8.05 -> 6.8 ms.
template <bool BATCH, bool SPLIT, int FOLD>
__global__ __launch_bounds__(256, SPLIT && FOLD ? 3 : 2) void k_synth_bwd_mfma(SynthArgs a0, const SynthArgs* __restrict__ jobs,
                                                        ChunkTab ct, et_paths P, const int32_t* __restrict__ idx,
                                                        const Ctl* ctl, const float* __restrict__ g,
                                                        double* __restrict__ gpx, double* __restrict__ gpk) {
  SYNTH_RESOLVE();
  if (BATCH) g += (size_t)jb * a.M * a.F * 2;
  __shared__ __align__(16) BwdBuf<FOLD> bb;
  __shared__ WaveScratch wscr[4];
  __shared__ SegTable st;
  __shared__ double red[256];
  const int p = bp, m = bm, k1t = bt;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int K1 = a.F / K2;
  const int k1_0 = k1t * KT1;
  const int nk1 = min(KT1, K1 - k1_0);
  int nseg, myseg;
  seg_init(a, k1_0, nk1, tid, st, nseg, myseg);
  // segments of the two half groups of row group lane % 8 (FOLD)
  const int segl = min(__shfl(myseg, 8 * (lane & 7)), nseg - 1), segh = min(__shfl(myseg, 8 * (lane & 7) + 4), nseg - 1);
  // wave -> block of 16 rows; SPLIT (a tile of at most 32 rows, two blocks) gives each wave
  // pair one block and each wave of a pair one of the stage's two record blocks
  constexpr int NB = SPLIT ? 1 : 2;              // record blocks of 16 per wave and stage
  const int rbw = SPLIT ? (wv & 1) : wv;
  const int nb0 = SPLIT ? (wv >> 1) : 0;
  // A operands: rows k1 = 16 rbw + lane % 16 of G = conj(g) and of f_k G (f_k the bin's
  // frequency), inner indices k2 = 32 h + 8 (lane / 16) + i (h < 2, i < 8), as f16 halves
  // [re hi, re lo, im hi, im lo], scaled by 2^eg and 2^eg2 (per wave) so that the largest
  // magnitude is near 2^12
  halfx8 ga[2][4], gw[2][4];
  float usz, usw;   // 2^-eg, 2^-eg2: undo the scales on Z and Z'
  {
    const int r1g = rbw * 16 + (lane & 15);
    float gr[2][8], gi[2][8], fk[2][8];
    float mz = 0.f, mw = 0.f;
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const int k2 = 32 * h + 8 * (lane >> 4) + i;
        const int k = (k1_0 + r1g) * K2 + k2;
        float vr = 0.f, vi = 0.f;
        if (r1g < nk1) {
          vr = g[((size_t)m * a.F + k) * 2];
          vi = -g[((size_t)m * a.F + k) * 2 + 1];
        }
        gr[h][i] = vr;
        gi[h][i] = vi;
        fk[h][i] = (float)(a.f_lo + (double)k * a.df);
        const float mg = fmaxf(fabsf(vr), fabsf(vi));
        mz = fmaxf(mz, mg);
        mw = fmaxf(mw, mg * fabsf(fk[h][i]));
      }
    mz = wave_max(mz);
    mw = wave_max(mw);
    const float ez = mz > 0.f ? 12.f - ceilf(log2f(mz)) : 0.f, ew = mw > 0.f ? 12.f - ceilf(log2f(mw)) : 0.f;
    const float sz = exp2f(ez), sw = exp2f(ew);
    usz = exp2f(-ez);
    usw = exp2f(-ew);
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      float zr[8], zi[8], wr[8], wi[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        zr[i] = gr[h][i] * sz;
        zi[i] = gi[h][i] * sz;
        wr[i] = gr[h][i] * fk[h][i] * sw;
        wi[i] = gi[h][i] * fk[h][i] * sw;
      }
      split8(zr, ga[h][0], ga[h][1]);
      split8(zi, ga[h][2], ga[h][3]);
      split8(wr, gw[h][0], gw[h][1]);
      split8(wi, gw[h][2], gw[h][3]);
    }
  }
  const int64_t nst = (hi - lo + 8 * RB - 1) / (8 * RB) * 8;
  const double ln10 = 2.30258509299404568402;
  const double c2 = -ln10 * a.A1 / 20.0, c3 = -(double)a.sigma * 2.0 * M_PI / a.c;
  const int QB = a.Q * a.Bk;
  double gx0 = 0.0, gx1 = 0.0, gx2 = 0.0;
  for (int i = tid; i < QB; i += 256) {
    const double bt = (double)a.beta[i];
    bb.lobe_w[i] = (float)(1.0 / (2.0 * bt * bt));
    bb.kf[i] = a.refl_k[i];
  }
  if (tid < a.Bk) bb.kf[QB + tid] = 1.f;
  for (int i = lane; i < QB; i += 64) bb.dk[wv][i] = 0.0;   // (each wave's own totals)
  // material band and band segment of each of this lane's four epilogue rows (rows past the grid:
  // the last band, and the segment past the tile, whose band factor is zero)
  int rband[4], rseg[4];
  {
    const int r10 = rbw * 16 + (lane >> 4) * 4;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int64_t kr = (int64_t)min(k1_0 + r10 + v, K1 - 1) * K2;
      rband[v] = (int)((kr * a.Bk) / a.F);
      rseg[v] = __shfl(myseg, r10 + v);
    }
  }
  // rows [br0[h], br1[h]) of the tile in band (tid % 8) + 8 h, the bands this thread sums in the
  // per-record epilogue (empty for a band not in the tile)
  int br0[2], br1[2];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int b = (tid & 7) + 8 * h, sg = b < a.Bk ? st.bseg[b] : -1;
    br0[h] = sg >= 0 ? st.s0[sg] : 0;
    br1[h] = sg >= 0 ? st.s1[sg] : 0;
  }
  floatx4 dkc = {0.f, 0.f, 0.f, 0.f};
  PairLean q;
  for (int64_t s = 0; s < nst; ++s) {
    const int t = (int)(s & 7);
    if (t == 0) pair_adj(a, P, idx, lo + (s >> 3) * (8 * RB) + wv * 64 + lane, hi, m, q);
    gen_factors<FOLD>(a, q, t, k1_0, nk1, lane, nseg, st, 0.f, wscr[wv], segl, segh);
    write_bwd(wscr[wv], lane, wv, bb);
    {
      // each generated record's row of k factors
      const int src = t * RPW + (lane & 7);
      const int m_r = __shfl(q.mat, src), k_r = __shfl(q.kind, src);
      if (lane < RPW) bb.recb[wv * RPW + lane] = k_r == 0 ? m_r * a.Bk : QB;
    }
    __syncthreads();
    // acc[0..2]: Z as Gr Yr, Gi Yi, Gr Yi + Gi Yr; acc[3..5]: Z' likewise (f_k G)
    floatx4 acc[6][NB];
#pragma unroll
    for (int i = 0; i < 6; ++i)
#pragma unroll
      for (int j = 0; j < NB; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int h = 0; h < 2; ++h) {
#pragma unroll
      for (int j = 0; j < NB; ++j) {
        const int nn = (nb0 + j) * 16 + (lane & 15);
        halfx8 y[4];
#pragma unroll
        for (int f = 0; f < 4; ++f) y[f] = bb.Y[f][nn][4 * h + (lane >> 4)];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          const halfx8* A = u ? gw[h] : ga[h];
          floatx4 rr = acc[3 * u][j], ii = acc[3 * u + 1][j], im = acc[3 * u + 2][j];
          rr = __builtin_amdgcn_mfma_f32_16x16x32_f16(A[0], y[0], rr, 0, 0, 0);
          rr = __builtin_amdgcn_mfma_f32_16x16x32_f16(A[0], y[1], rr, 0, 0, 0);
          rr = __builtin_amdgcn_mfma_f32_16x16x32_f16(A[1], y[0], rr, 0, 0, 0);
          ii = __builtin_amdgcn_mfma_f32_16x16x32_f16(A[2], y[2], ii, 0, 0, 0);
          ii = __builtin_amdgcn_mfma_f32_16x16x32_f16(A[2], y[3], ii, 0, 0, 0);
          ii = __builtin_amdgcn_mfma_f32_16x16x32_f16(A[3], y[2], ii, 0, 0, 0);
          im = __builtin_amdgcn_mfma_f32_16x16x32_f16(A[0], y[2], im, 0, 0, 0);
          im = __builtin_amdgcn_mfma_f32_16x16x32_f16(A[0], y[3], im, 0, 0, 0);
          im = __builtin_amdgcn_mfma_f32_16x16x32_f16(A[1], y[2], im, 0, 0, 0);
          im = __builtin_amdgcn_mfma_f32_16x16x32_f16(A[2], y[0], im, 0, 0, 0);
          im = __builtin_amdgcn_mfma_f32_16x16x32_f16(A[2], y[1], im, 0, 0, 0);
          im = __builtin_amdgcn_mfma_f32_16x16x32_f16(A[3], y[0], im, 0, 0, 0);
          acc[3 * u][j] = rr;
          acc[3 * u + 1][j] = ii;
          acc[3 * u + 2][j] = im;
        }
      }
    }
    // accumulator (j, v) of lane l: row 16 rbw + 4 (l / 16) + v, record 16 (nb0 + j) + l % 16
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      const int nb = nb0 + j;
      const int n = nb * 16 + (lane & 15);
      const int r10 = rbw * 16 + (lane >> 4) * 4;   // this lane's four rows r10 .. r10 + 3
      // X of record n at these rows from its factors (wave n / 8 generated it): Xa (or Xh, the
      // upper half group with FOLD 4) of group r10 / 8 times Xb of r10 % 8 .. + 3, times the
      // row's band factor without FOLD
      float xrv[4], xiv[4];
      {
        const WaveScratch& W = wscr[n >> 3];
        const int rr = n & 7, ga = r10 >> 3, gb = r10 & 7;
        const float2 xa = FOLD == 4 && gb >= 4 ? W.xh[rr][ga] : W.xa[rr][ga];
        const float4 b01 = *reinterpret_cast<const float4*>(&W.xb[rr][gb]);
        const float4 b23 = *reinterpret_cast<const float4*>(&W.xb[rr][gb + 2]);
        const float2 xb[4] = {make_float2(b01.x, b01.y), make_float2(b01.z, b01.w), make_float2(b23.x, b23.y),
                              make_float2(b23.z, b23.w)};
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          float2 x = cmul(xa, xb[v]);
          if (!FOLD) {
            const float f = W.bf[rr][rseg[v]];
            x.x *= f;
            x.y *= f;
          }
          xrv[v] = x.x;
          xiv[v] = x.y;
        }
      }
      const float* kfr = bb.kf + bb.recb[n];
      float crv[4];
      float s1r = 0.f, s1i = 0.f;
      // Re(X Z) per row (the band sums) and X Z' (the frequency-weighted sum), both before the
      // scales 2^-eg, 2^-eg2, which are applied once per lane below
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const float zr = acc[0][j][v] - acc[1][j][v], zi = acc[2][j][v];
        const float wr = acc[3][j][v] - acc[4][j][v], wi = acc[5][j][v];
        const float xr = xrv[v], xi = xiv[v];
        crv[v] = xr * zr - xi * zi;
        const float tr = xr * wr - xi * wi, ti = xr * wi + xi * wr;
        if (FOLD) {   // one band over the four rows: k applies to their sum
          s1r += tr;
          s1i += ti;
        } else {
          const float kv = kfr[rband[v]];
          s1r += kv * tr;
          s1i += kv * ti;
        }
      }
      const int grp = rbw * 4 + (lane >> 4);
      if (FOLD) {
        const float kv = kfr[rband[0]] * usw;
        bb.Rg[grp][n] = ((crv[0] + crv[1]) + (crv[2] + crv[3])) * usz;
        bb.R1[grp][n] = make_float2(kv * s1r, kv * s1i);
      } else {
        *reinterpret_cast<float4*>(&bb.R0[n][r10]) =
            make_float4(crv[0] * usz, crv[1] * usz, crv[2] * usz, crv[3] * usz);
        bb.R1[grp][n] = make_float2(s1r * usw, s1i * usw);
      }
    }
    __syncthreads();
    {
      // eight threads per record: row sums in FP64, bands j and j + 8.  Record n of this stage
      // was set up by lane 8 t + n % 8 of this same wave: its data arrive by shuffle.
      const int n = tid >> 3, j = tid & 7;
      const int src = t * RPW + (n & 7);
      const bool valid = __shfl(q.base, src) != -INFINITY;
      const int mat = __shfl(q.mat, src), kind = __shfl(q.kind, src);
      const float gux = __shfl(q.gux, src), guy = __shfl(q.guy, src), guz = __shfl(q.guz, src);
      const float gc1 = __shfl(q.gc1, src);
      const float glx = __shfl(q.glx, src), gly = __shfl(q.gly, src), glz = __shfl(q.glz, src);
      // partial sums of this thread (row groups 2 j, 2 j + 1; bands j, j + 8) in FP32, combined
      // over the record's eight threads in a fixed order
      float s1r = 0.f, s1i = 0.f;
      const int ngroups = SPLIT ? 8 : 16;   // row groups of 4 written this stage
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        if (2 * j + i >= ngroups) continue;
        const float2 c = bb.R1[2 * j + i][n];
        s1r += c.x;
        s1i += c.y;
      }
      float s0 = 0.f, wl = 0.f;
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int b = j + 8 * h;
        float sb = 0.f;
        if (FOLD) {
          for (int gg = br0[h] >> 2; gg < br1[h] >> 2; ++gg) sb += bb.Rg[gg][n];
        } else {
          // the band's rows in four interleaved partial sums (independent LDS reads)
          const int e = br1[h];
          int r1 = br0[h];
          float p0 = 0.f, p1 = 0.f, p2 = 0.f, p3 = 0.f;
          for (; r1 + 4 <= e; r1 += 4) {
            p0 += bb.R0[n][r1];
            p1 += bb.R0[n][r1 + 1];
            p2 += bb.R0[n][r1 + 2];
            p3 += bb.R0[n][r1 + 3];
          }
          for (; r1 < e; ++r1) p0 += bb.R0[n][r1];
          sb = (p0 + p1) + (p2 + p3);
        }
        // sb leaves out k for specular records: k sb is the band's share of H's sums, 2 sb its dL/dk
        float kvv = 0.f;
        if (b < a.Bk) {
          const float kb = kind == 0 ? bb.kf[mat * a.Bk + b] : 1.f;
          s0 += kb * sb;
          if (valid && kind == 0) {
            wl += kb * sb * bb.lobe_w[mat * a.Bk + b];
            kvv = 2.f * sb;
          }
        }
        if (b < a.Bk) bb.kv[b][n] = kvv;
      }
      s1r = sum8_first(s1r);
      s1i = sum8_first(s1i);
      s0 = sum8_first(s0);
      wl = sum8_first(wl);
      if (j == 0) bb.kmat[n] = valid && kind == 0 ? mat : -1;
      if (j == 0 && valid) {
        // d(ln A + j phi)/dx_m = [(-p/r - ln10 (a0 + a1 f)/20) + j sigma 2 pi f / c] u - d(gamma^2)/dx / (2 beta^2)
        const double cu = (double)gc1 * (double)s0 + c2 * (double)s1r + c3 * (double)s1i;
        const double g0 = 2.0 * cu * (double)gux + (double)wl * (double)glx;
        const double g1 = 2.0 * cu * (double)guy + (double)wl * (double)gly;
        const double g2 = 2.0 * cu * (double)guz + (double)wl * (double)glz;
        gx0 += g0; gx1 += g1; gx2 += g2;
      }
    }
    // the wave's records of this stage into dL/dk (their kv and kmat were written by this wave)
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
    dk_wave(bb, wv, lane, a.Q, a.Bk, dkc, t == 7);   // (nst is a multiple of 8)
  }
  __syncthreads();
  const size_t slot = ((size_t)p * gridDim.z + k1t) * a.M + m;
  const double gv[3] = {gx0, gx1, gx2};
  for (int c = 0; c < 3; ++c) {
    red[tid] = gv[c];
    __syncthreads();
    for (int h = 128; h > 0; h >>= 1) {
      if (tid < h) red[tid] += red[tid + h];
      __syncthreads();
    }
    if (tid == 0) gpx[slot * 3 + c] = red[0];
    __syncthreads();
  }
  // the four waves' totals of each (material, band), in wave order
  if (tid < QB) gpk[slot * QB + tid] = ((bb.dk[0][tid] + bb.dk[1][tid]) + bb.dk[2][tid]) + bb.dk[3][tid];
}

// One workgroup per output value (QB band coefficients, then 3 M receiver coordinates): its
// threads sum fixed strided subsets of the partials in FP64 and a fixed-shape tree in LDS adds
// the 256 sums, so the result does not depend on scheduling.
constexpr int RED_T = 256;
__global__ __launch_bounds__(RED_T) void k_bwd_reduce(const double* __restrict__ gpx, const double* __restrict__ gpk,
                                                      int32_t P, int32_t M, int32_t QB, double* __restrict__ grad_k,
                                                      double* __restrict__ grad_x) {
  __shared__ double red[RED_T];
  const int o = blockIdx.x, tid = threadIdx.x;
  double s = 0.0;
  if (o < QB) {
    const int64_t n = (int64_t)P * M;   // partial (p, m) at gpk[((p M) + m) QB + o]
    for (int64_t e = tid; e < n; e += RED_T) s += gpk[e * QB + o];
  } else {
    const int i = o - QB;               // coordinate i = 3 m + c at gpx[p 3 M + i]
    for (int64_t p = tid; p < P; p += RED_T) s += gpx[p * M * 3 + i];
  }
  red[tid] = s;
  __syncthreads();
  for (int h = RED_T / 2; h > 0; h >>= 1) {
    if (tid < h) red[tid] += red[tid + h];
    __syncthreads();
  }
  if (tid == 0) {
    if (o < QB) grad_k[o] = red[0];
    else grad_x[o - QB] = red[0];
  }
}

inline size_t al(size_t b) { return (b + 255) / 256 * 256; }

// Tiles of at most 64 rows of a pose's spectrum.
int64_t row_tiles(const et_sim_desc* sim) { return ((int64_t)synth_rows(sim, nullptr) + KT1 - 1) / KT1; }

// Record chunks of a launch of the kernel fk (the factorised adjoint as FWD_HALVES).
int choose_P(const et_sim_desc* sim, int64_t cap, FwdKernel fk) {
  // kernels in halves: about sixteen workgroups per CU over the launch (measured on the
  // room's 32 x 4096 adjoint: 2048 workgroups 20.16 ms, 3072 20.05, 4096 19.87, 6144 19.98, 8192
  // 19.92 ms).  Chunk count a multiple of 8 so that every receiver's workgroups of one chunk share an
  // XCD's L2.
  const int64_t tiles = (int64_t)sim->M * (fk != FWD_TERM ? row_tiles(sim) : (sim->F + DTILE - 1) / DTILE);
  const int64_t target = fk == FWD_HALVES ? 4096 : 2048;
  int64_t P = std::max<int64_t>(1, (target + tiles - 1) / tiles);
  if (P >= 8) P = (P + 7) / 8 * 8;
  int64_t most = std::max<int64_t>(1, cap / 64);
  if (fk == FWD_ROWS) {
    // no fewer chunks than per term has for as many tiles: a wave then sums a quarter of the records in a row (with 1024
    // workgroups 60,000 records x 6 receivers x 3000 bins take 113 us instead of 130, but sums of many records in few
    // bins came out less accurate than per term); chunks of 128 records (20,011 x 4 x 1500: 29 us, of 64 36, of
    // 512 34) beyond the first 16
    P = std::max<int64_t>(1, 2048 / tiles);
    if (P >= 8) P = P / 8 * 8;
    most = std::max(std::min<int64_t>(most, 16), cap / 128);
  }
  P = std::min(P, most);
  return (int)std::min<int64_t>(P, 256);
}

size_t vis_ws(int64_t cap, char* base, size_t off, uint64_t** sum, int32_t** idx) {
  auto take = [&](size_t b) -> void* { void* p = base ? (void*)(base + off) : nullptr; off += al(b); return p; };
  // (as many tiles as any smaller capacity has, so that what is queried for a pose's most records serves paths of
  // fewer: tiles grow in steps)
  *sum = (uint64_t*)take(sizeof(uint64_t) * (size_t)std::min<int64_t>((cap + VIS_TILE - 1) / VIS_TILE, VIS_MAX_TILES));
  *idx = (int32_t*)take(sizeof(int32_t) * (size_t)cap);
  return off;
}

// What a call needs before its kernels, in one launch: the visible records of each tile (vis workgroups), the
// band tables, and the row table if asked for.
__global__ __launch_bounds__(256) void k_synth_prep(et_paths P, Ctl* ctl, int64_t tile, unsigned vis,
                                                    uint64_t* __restrict__ vsum, SynthArgs a, float* lk, float* lc,
                                                    float* ld, float* lp, float* lmax, int2* rows) {
  if (blockIdx.x < vis) {
    vis_count(P, ctl, blockIdx.x, tile, vsum);
    return;
  }
  if (rows && blockIdx.x + 1 == gridDim.x) {
    row_table(a, rows);
    return;
  }
  const int i = (blockIdx.x - vis) * blockDim.x + threadIdx.x;
  if (i < a.Q) band_bound_entry(a, i, lmax);
  if (i < a.Q * a.Bk) band_table_entry(a, i, lk, lc, ld, lp);
}

// Band tables (and with rows the row table, for the factorised kernels' FOLD 0), and with list the visible-record
// list of the paths.
void build_prep(SynthArgs& a, const SynthWS& ws, const et_paths& P, bool list, bool rows, Ctl* ctl, hipStream_t s) {
  a.lk = ws.lk;
  a.lc = ws.lc;
  a.ld = ws.ld;
  a.lp = ws.lp;
  a.lmax = ws.lmax;
  a.rows = rows ? (const int2*)ws.rows : nullptr;
  const int n = a.Q * a.Bk;
  const int64_t tile = vis_tile(ws.cap);
  const unsigned vis = list ? (unsigned)((ws.cap + tile - 1) / tile) : 0u;
  k_synth_prep<<<vis + (n + 255) / 256 + (rows ? 1 : 0), 256, 0, s>>>(P, ctl, tile, vis, ws.vsum, a, ws.lk, ws.lc, ws.ld,
                                                                    ws.lp, ws.lmax, rows ? (int2*)ws.rows : nullptr);
  if (list) k_vis_list<<<vis, 256, 0, s>>>(P, ctl, tile, ws.vsum, ws.vidx);
  ET_HIP(hipGetLastError());
}

// Path-product reading: band tables with a row per record.  Specular record n: the sum of
// log2 k over its ray's specular records up to n (itself and its predecessors through prev)
// and its own lobe coefficient; a diffraction record: its material's log2 I_d.
__global__ void k_path_tables(et_paths P, SynthArgs a, const Ctl* ctl, float* __restrict__ plk,
                              float* __restrict__ plc) {
  const int Bk = a.Bk;
  const int64_t n_rec = ctl->n_rec;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n_rec * Bk;
       i += (int64_t)gridDim.x * blockDim.x) {
    const int64_t n = i / Bk;
    const int b = (int)(i - n * Bk);
    const int kind = (P.flags[n] >> 1) & 3;
    const int mat = P.mat[n];
    float s = 0.f, lobe = 0.f;
    if (kind == 0) {
      lobe = a.lc[mat * Bk + b];
      int64_t r = n;
      for (int guard = 0; guard < 256 && r >= 0; ++guard) {   // a ray has at most 255 reflections
        s += a.lk[P.mat[r] * Bk + b];
        const int64_t pr = P.prev[r];
        r = pr < r ? pr : -1;                                    // predecessors have smaller indices
      }
    } else if (kind == 1) {
      s = a.ld[mat * Bk + b];
    }
    plk[i] = s;
    plc[i] = lobe;
  }
}

// Per-receiver line of sight and the path-product reading for one pose's synthesis.
void set_readings(SynthArgs& a, const et_sim_desc* sim, const et_paths& P, const SynthWS& ws, Ctl* ctl,
                  hipStream_t s) {
  a.rxv = (sim->flags & ET_PER_RX_VISIBILITY) ? P.rx_vis : nullptr;
  if (sim->flags & ET_PATH_PRODUCT) {
    const int64_t n = ws.cap * sim->Bk;
    k_path_tables<<<(unsigned)std::max<int64_t>(1, std::min<int64_t>((n + 255) / 256, 16384)), 256, 0, s>>>(
        P, a, ctl, ws.plk, ws.plc);
    ET_HIP(hipGetLastError());
    a.lk = ws.plk;
    a.lc = ws.plc;
    a.ld = ws.plk;
    a.rec_rows = 1;
  }
}

size_t table_ws(const et_sim_desc* sim, char* base, size_t off, SynthWS& w) {
  const size_t n = (size_t)sim->Q * sim->Bk;
  w.lk = (float*)(base ? base + off : nullptr);
  off += al(sizeof(float) * n);
  w.lc = (float*)(base ? base + off : nullptr);
  off += al(sizeof(float) * n);
  w.ld = (float*)(base ? base + off : nullptr);
  off += al(sizeof(float) * n);
  w.lp = (float*)(base ? base + off : nullptr);
  off += al(sizeof(float) * sim->Bk);
  w.lmax = (float*)(base ? base + off : nullptr);
  off += al(sizeof(float) * (3 * (size_t)sim->Q + 1));
  w.rows = base ? base + off : nullptr;
  off += al(sizeof(int2) * ((size_t)synth_rows(sim, nullptr) + 1));
  return off;
}

// ------------------------------------------------------------------ fused batches

constexpr int SJOB_PACK = 16;
struct SynthJobPack {
  SynthArgs j[SJOB_PACK];
  int32_t first, n;
};
static_assert(sizeof(SynthJobPack) <= 4032, "job pack must fit the kernel argument space");

__global__ void k_put_synth_jobs(SynthJobPack pk, SynthArgs* __restrict__ dst) {
  if ((int)threadIdx.x < pk.n) dst[pk.first + threadIdx.x] = pk.j[threadIdx.x];
}

// workgroup j fills job j's band tables (its lk / lc / ld / lp point into the batch's table block)
__global__ void k_band_tables_batch(const SynthArgs* __restrict__ jobs) {
  const SynthArgs a = jobs[blockIdx.x];
  for (int i = threadIdx.x; i < a.Q * a.Bk; i += blockDim.x)
    band_table_entry(a, i, const_cast<float*>(a.lk), const_cast<float*>(a.lc), const_cast<float*>(a.ld),
                     const_cast<float*>(a.lp));
  for (int q = threadIdx.x; q < a.Q; q += blockDim.x) band_bound_entry(a, q, const_cast<float*>(a.lmax));
  if (a.rows) row_table(a, const_cast<int2*>(a.rows));
}

// sort key of each visible record: its job (the ray field of a batch record)
__global__ void k_vis_jobkeys(et_paths P, const int32_t* __restrict__ idx, const Ctl* ctl, uint64_t* __restrict__ keys) {
  const int64_t n = ctl->n_vis;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    keys[i] = (uint64_t)(uint32_t)P.ray[idx[i]];
}

// Per-job ranges of the job-sorted visible list and chunk offsets: chunks of
// per = ceil(n_vis / target) records, never crossing a job.  One workgroup.
__global__ void k_job_chunks(const uint64_t* __restrict__ keys, const Ctl* ctl, int32_t J, int64_t target,
                             int64_t* __restrict__ off, int64_t* __restrict__ lo, int64_t* __restrict__ hi,
                             int64_t* __restrict__ per) {
  const int64_t n = ctl->n_vis;
  const int64_t pc = std::max<int64_t>(1, (n + target - 1) / target);
  for (int j = threadIdx.x; j < J; j += blockDim.x) {
    int64_t a = 0, b = n;   // first position with key >= j
    while (a < b) {
      const int64_t mid = (a + b) >> 1;
      if (keys[mid] < (uint64_t)j) a = mid + 1;
      else b = mid;
    }
    const int64_t l = a;
    b = n;                  // first position with key >= j + 1
    while (a < b) {
      const int64_t mid = (a + b) >> 1;
      if (keys[mid] < (uint64_t)j + 1) a = mid + 1;
      else b = mid;
    }
    lo[j] = l;
    hi[j] = a;
    off[j + 1] = (a - l + pc - 1) / pc;   // chunk count, turned into offsets below
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    off[0] = 0;
    for (int j = 0; j < J; ++j) off[j + 1] += off[j];
    per[0] = pc;
  }
}

__global__ void k_reduce_batch(const float* __restrict__ part, ChunkTab ct, int64_t MF2, float* __restrict__ out) {
  const int64_t total = (int64_t)ct.J * MF2;
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < total; e += (int64_t)gridDim.x * blockDim.x) {
    const int64_t j = e / MF2, r = e - j * MF2;
    float s = 0.f;
    for (int64_t c = ct.off[j]; c < ct.off[j + 1]; ++c) s += part[c * MF2 + r];
    out[e] = s;
  }
}

// Per job dL/dk[Q Bk] and dL/dx[M][3], a workgroup per value as in k_bwd_reduce: its threads sum fixed strided subsets of
// the job's partials over chunks, tiles (and receivers), and a fixed-shape tree in LDS adds the 256 sums (24
// jobs of 128 band coefficients and 8 receivers: 83 us with a thread per value, one load after the other).
__global__ __launch_bounds__(RED_T) void k_bwd_reduce_batch(const double* __restrict__ gpx, const double* __restrict__ gpk,
                                                            ChunkTab ct, int32_t T1, int32_t M, int32_t QB,
                                                            double* __restrict__ grad_k, double* __restrict__ grad_x) {
  __shared__ double red[RED_T];
  const int o = blockIdx.x, tid = threadIdx.x;
  const int64_t j = blockIdx.y, c0 = ct.off[j], c1 = ct.off[j + 1];
  double s = 0.0;
  if (o < QB) {
    for (int64_t e = c0 * T1 * M + tid; e < c1 * T1 * M; e += RED_T) s += gpk[e * QB + o];
  } else {
    for (int64_t e = c0 * T1 + tid; e < c1 * T1; e += RED_T) s += gpx[e * M * 3 + o - QB];
  }
  red[tid] = s;
  __syncthreads();
  for (int h = RED_T / 2; h > 0; h >>= 1) {
    if (tid < h) red[tid] += red[tid + h];
    __syncthreads();
  }
  if (tid == 0) {
    if (o < QB) grad_k[j * QB + o] = red[0];
    else grad_x[j * 3 * M + o - QB] = red[0];
  }
}

}  // namespace

// Every material (and directivity) band edge on a multiple of g outer indices (64 g bins) and
// the bins a multiple of 64 g.
bool bands_on_groups(const et_sim_desc* sim, int64_t g) {
  const int64_t F = sim->F, Bk = sim->Bk, Bd = sim->directivity ? sim->Bd : 0, K1 = F / K2;
  if (F % (K2 * g)) return false;
  for (int64_t k1 = 1; k1 < K1; ++k1) {
    if (k1 % g == 0) continue;
    const int64_t k = k1 * K2, kp = k - K2;
    if (k * Bk / F != kp * Bk / F) return false;
    if (Bd && k * Bd / F != kp * Bd / F) return false;
  }
  return true;
}

// How the band factor rides on the generating factors (forward and adjoint): 8 when every band
// edge falls on a multiple of 512 bins and the bins are a multiple of 512, 4 for 256, 0 (a table
// of band factors) otherwise.
int bands_fold(const et_sim_desc* sim) { return bands_on_groups(sim, 8) ? 8 : bands_on_groups(sim, 4) ? 4 : 0; }

template <bool BATCH, int NRB, bool DIR>
void launch_fwd_fold(int fold, dim3 grid, hipStream_t s, const SynthArgs& a, const SynthArgs* jobs, const ChunkTab& ct,
                     const et_paths& P, const int32_t* idx, const Ctl* ctl, float* part) {
  if (fold == 8) k_synth_mfma<BATCH, NRB, 8, DIR><<<grid, 256, 0, s>>>(a, jobs, ct, P, idx, ctl, part);
  else if (fold == 4) k_synth_mfma<BATCH, NRB, 4, DIR><<<grid, 256, 0, s>>>(a, jobs, ct, P, idx, ctl, part);
  else k_synth_mfma<BATCH, NRB, 0, DIR><<<grid, 256, 0, s>>>(a, jobs, ct, P, idx, ctl, part);
}

template <bool BATCH, int NRB, bool DIR>
void launch_fwd_tiles(FwdKernel fk, int fold, dim3 grid, hipStream_t s, const SynthArgs& a, const SynthArgs* jobs,
                      const ChunkTab& ct, const et_paths& P, const int32_t* idx, const Ctl* ctl, float* part) {
  if (fk == FWD_ROWS) k_synth_rows<BATCH, NRB, DIR><<<grid, 256, 0, s>>>(a, jobs, ct, P, idx, ctl, part);
  else launch_fwd_fold<BATCH, NRB, DIR>(fold, grid, s, a, jobs, ct, P, idx, ctl, part);
}

// rows: the most rows of a job; tiles of 64 rows, or one block of 32 when that holds them all
template <bool BATCH>
void launch_fwd(FwdKernel fk, int rows, int fold, bool dir, int chunks, int M, hipStream_t s, const SynthArgs& a,
                const SynthArgs* jobs, const ChunkTab& ct, const et_paths& P, const int32_t* idx, const Ctl* ctl,
                float* part) {
  if (fk == FWD_TERM) {
    k_synth_direct<BATCH><<<dim3(chunks, M, (a.F + DTILE - 1) / DTILE), DB, 0, s>>>(a, jobs, ct, P, idx, ctl, part);
    return;
  }
  const dim3 grid(chunks, M, (rows + KT1 - 1) / KT1);
  if (rows <= 32) {
    if (dir) launch_fwd_tiles<BATCH, 1, true>(fk, fold, grid, s, a, jobs, ct, P, idx, ctl, part);
    else launch_fwd_tiles<BATCH, 1, false>(fk, fold, grid, s, a, jobs, ct, P, idx, ctl, part);
  } else {
    if (dir) launch_fwd_tiles<BATCH, 2, true>(fk, fold, grid, s, a, jobs, ct, P, idx, ctl, part);
    else launch_fwd_tiles<BATCH, 2, false>(fk, fold, grid, s, a, jobs, ct, P, idx, ctl, part);
  }
}

// Bands on whole runs of 64 bins: what k_synth_mfma and the factorised adjoint take.
bool synth_factorised_ok(const et_sim_desc* sim) {
  // needs k = 64 k1 + k2, material / directivity bands constant over each run of 64 bins
  // (the band factor is per outer index), and at most SMAX band segments per tile of KT1
  // outer indices
  if (sim->flags & ET_SYNTH_DIRECT) return false;
  if (sim->F < K2 || sim->F % K2) return false;
  const int64_t F = sim->F, Bk = sim->Bk, Bd = sim->directivity ? sim->Bd : 0;
  int nseg = 0;
  int64_t pb = -1, pd = -1;
  for (int64_t k1 = 0; k1 < F / K2; ++k1) {
    const int64_t ka = k1 * K2, kb = ka + K2 - 1;
    const int64_t b = ka * Bk / F, d = Bd ? ka * Bd / F : 0;
    if (b != kb * Bk / F) return false;
    if (Bd && d != kb * Bd / F) return false;
    if (k1 % KT1 == 0) nseg = 0;
    if (k1 % KT1 == 0 || b != pb || d != pd) ++nseg;
    if (nseg > SMAX) return false;
    pb = b;
    pd = d;
  }
  return true;
}

// The forward kernel of a pose: in halves where the bands lie on whole runs of 64 bins, in FP32 over rows for any other
// layout whose tiles of 64 rows hold at most SMAX band segments (their factors sit in LDS per segment), else per
// term.  Per term the 60,000 records x 6 receivers x 3000 bins in 7 bands take 540 us, most of it three
// transcendentals per term.
FwdKernel fwd_kernel(const et_sim_desc* sim) {
  if (sim->flags & ET_SYNTH_DIRECT) return FWD_TERM;
  if (synth_factorised_ok(sim)) return FWD_HALVES;
  int seg = 0;
  synth_rows(sim, &seg);
  return seg <= SMAX ? FWD_ROWS : FWD_TERM;
}

size_t synth_ws_layout(const et_sim_desc* sim, int64_t cap, char* base, SynthWS* ws) {
  cap = std::max<int64_t>(cap, 1);
  const int P = choose_P(sim, cap, fwd_kernel(sim));
  size_t off = 0;
  SynthWS w{};
  w.P = P;
  w.cap = cap;
  w.partial = (float*)(base ? base + off : nullptr);
  off += al(sizeof(float) * 2 * (size_t)P * sim->M * sim->F);
  off = vis_ws(cap, base, off, &w.vsum, &w.vidx);
  off = table_ws(sim, base, off, w);
  if (sim->flags & ET_PATH_PRODUCT) {
    w.plk = (float*)(base ? base + off : nullptr);
    off += al(sizeof(float) * (size_t)cap * sim->Bk);
    w.plc = (float*)(base ? base + off : nullptr);
    off += al(sizeof(float) * (size_t)cap * sim->Bk);
  }
  if (ws) *ws = w;
  return off;
}

int synth_run(const et_sim_desc* sim, const et_paths* paths, const SynthWS& ws, Ctl* ctl, float* spectra, hipStream_t s,
              hipEvent_t kb, hipEvent_t ke) {
  const FwdKernel fk = fwd_kernel(sim);
  const int fold = fk == FWD_HALVES ? bands_fold(sim) : 0;
  SynthArgs a = make_args(sim, ws.P);
  const et_paths P = *paths;
  build_prep(a, ws, P, true, fk != FWD_TERM && fold == 0, ctl, s);
  set_readings(a, sim, P, ws, ctl, s);
  if (kb) ET_HIP(hipEventRecord(kb, s));
  launch_fwd<false>(fk, a.nrows, fold, sim->directivity != nullptr, ws.P, sim->M, s, a, nullptr, ChunkTab{}, P, ws.vidx, ctl,
                    ws.partial);
  if (ke) ET_HIP(hipEventRecord(ke, s));
  reduce_partials(ws.partial, ws.P, (int64_t)sim->M * sim->F, spectra, s);
  ET_HIP(hipGetLastError());
  return fk;
}

int synth_run_noalloc(const et_sim_desc* sim, const et_paths* paths, void* buf, size_t bytes, Ctl* ctl,
                      float* spectra, hipStream_t s, hipEvent_t kb, hipEvent_t ke) {
  ET_CHECK(!(sim->flags & ET_PATH_PRODUCT), ET_E_UNSUPPORTED,
           "ET_PATH_PRODUCT needs per-record tables (a workspace): use et_synthesize");
  FwdKernel fk = fwd_kernel(sim);
  const int fold = fk == FWD_HALVES ? bands_fold(sim) : 0;
  const int64_t cap = std::max<int64_t>(paths->capacity, 1);
  SynthWS w{};
  // the row table comes last: left out where the kernel has no use for it, or where only without it one chunk
  // fits the scratch (then per term)
  const size_t row_bytes = al(sizeof(int2) * ((size_t)synth_rows(sim, nullptr) + 1));
  size_t tables = table_ws(sim, nullptr, 0, w);
  const size_t chunk = al(sizeof(float) * 2 * (size_t)sim->M * sim->F);
  if (fk != FWD_TERM && fold == 0 && tables + chunk > bytes) fk = FWD_TERM;
  if (fk == FWD_TERM || fold != 0) tables -= row_bytes;
  ET_CHECK(tables + chunk <= bytes, ET_E_UNSUPPORTED,
           "receivers x bins too large for the device scratch of the allocation-free call");
  // record chunks: the usual choice, as many as the scratch holds, a multiple of 8 above 8
  int64_t P = std::min<int64_t>(choose_P(sim, cap, fk), (int64_t)((bytes - tables) / chunk));
  if (P > 8) P = P / 8 * 8;
  char* base = (char*)buf;
  table_ws(sim, base, 0, w);
  w.partial = (float*)(base + tables);
  w.P = (int)P;
  w.cap = cap;
  SynthArgs a = make_args(sim, w.P);
  const et_paths Pth = *paths;
  k_vis_all<<<1, 1, 0, s>>>(Pth, ctl);
  build_prep(a, w, Pth, false, fk != FWD_TERM && fold == 0, ctl, s);
  a.rxv = (sim->flags & ET_PER_RX_VISIBILITY) ? Pth.rx_vis : nullptr;
  if (kb) ET_HIP(hipEventRecord(kb, s));
  launch_fwd<false>(fk, a.nrows, fold, sim->directivity != nullptr, w.P, sim->M, s, a, nullptr, ChunkTab{}, Pth, nullptr, ctl,
                    w.partial);
  if (ke) ET_HIP(hipEventRecord(ke, s));
  reduce_partials(w.partial, w.P, (int64_t)sim->M * sim->F, spectra, s);
  ET_HIP(hipGetLastError());
  return fk;
}

bool synth_bwd_factorised_ok(const et_sim_desc* sim) { return !sim->directivity && synth_factorised_ok(sim); }

template <bool BATCH, bool SPLIT>
void launch_bwd_fold(int fold, dim3 grid, hipStream_t s, const SynthArgs& a, const SynthArgs* jobs, const ChunkTab& ct,
                     const et_paths& P, const int32_t* idx, const Ctl* ctl, const float* g, double* gpx,
                     double* gpk) {
  if (fold == 8) k_synth_bwd_mfma<BATCH, SPLIT, 8><<<grid, 256, 0, s>>>(a, jobs, ct, P, idx, ctl, g, gpx, gpk);
  else if (fold == 4) k_synth_bwd_mfma<BATCH, SPLIT, 4><<<grid, 256, 0, s>>>(a, jobs, ct, P, idx, ctl, g, gpx, gpk);
  else k_synth_bwd_mfma<BATCH, SPLIT, 0><<<grid, 256, 0, s>>>(a, jobs, ct, P, idx, ctl, g, gpx, gpk);
}

template <bool BATCH>
void launch_bwd_mfma(bool split, int fold, dim3 grid, hipStream_t s, const SynthArgs& a, const SynthArgs* jobs,
                     const ChunkTab& ct, const et_paths& P, const int32_t* idx, const Ctl* ctl, const float* g,
                     double* gpx, double* gpk) {
  if (split) launch_bwd_fold<BATCH, true>(fold, grid, s, a, jobs, ct, P, idx, ctl, g, gpx, gpk);
  else launch_bwd_fold<BATCH, false>(fold, grid, s, a, jobs, ct, P, idx, ctl, g, gpx, gpk);
}

size_t synth_bwd_ws_layout(const et_sim_desc* sim, int64_t cap, char* base, SynthWS* ws) {
  cap = std::max<int64_t>(cap, 1);
  const bool mf = synth_bwd_factorised_ok(sim);
  const int64_t T1 = mf ? (sim->F / K2 + KT1 - 1) / KT1 : 1;
  int64_t P;
  if (mf) {
    P = choose_P(sim, cap, FWD_HALVES);
  } else {
    P = std::max<int64_t>(1, (1024 + sim->M - 1) / sim->M);
    P = std::min<int64_t>(P, std::max<int64_t>(1, (cap + GB - 1) / GB));
    P = std::min<int64_t>(P, 256);
  }
  size_t off = 0;
  SynthWS w{};
  w.gchunks = (int)P;
  w.gtiles = (int)T1;
  w.cap = cap;
  w.gpart_x = (double*)(base ? base + off : nullptr);
  off += al(sizeof(double) * 3 * (size_t)P * T1 * sim->M);
  w.gpart_k = (double*)(base ? base + off : nullptr);
  off += al(sizeof(double) * (size_t)P * T1 * sim->M * sim->Q * sim->Bk);
  off = vis_ws(cap, base, off, &w.vsum, &w.vidx);
  off = table_ws(sim, base, off, w);
  if (ws) *ws = w;
  return off;
}

int synth_bwd_run(const et_sim_desc* sim, const et_paths* paths, const float* grad_spectra, const SynthWS& ws,
                  Ctl* ctl, double* grad_k, double* grad_rx, hipStream_t s, hipEvent_t kb, hipEvent_t ke) {
  const bool mf = synth_bwd_factorised_ok(sim);
  SynthArgs a = make_args(sim, ws.gchunks);
  const et_paths P = *paths;
  build_prep(a, ws, P, true, false, ctl, s);
  a.rxv = (sim->flags & ET_PER_RX_VISIBILITY) ? P.rx_vis : nullptr;   // (no path product in the adjoint)
  if (kb) ET_HIP(hipEventRecord(kb, s));
  if (mf) {
    dim3 grid(ws.gchunks, sim->M, ws.gtiles);
    launch_bwd_mfma<false>(sim->F / K2 <= 32, bands_fold(sim), grid, s, a, nullptr, ChunkTab{}, P, ws.vidx, ctl,
                           grad_spectra, ws.gpart_x, ws.gpart_k);
  } else {
    dim3 grid(ws.gchunks, sim->M);
    const size_t shm = sizeof(float2) * (size_t)sim->F;
    k_synth_bwd<false><<<grid, GB, shm, s>>>(a, nullptr, ChunkTab{}, P, ws.vidx, ctl, grad_spectra, ws.gpart_x,
                                             ws.gpart_k);
  }
  if (ke) ET_HIP(hipEventRecord(ke, s));
  const int QB = sim->Q * sim->Bk;
  k_bwd_reduce<<<QB + 3 * sim->M, RED_T, 0, s>>>(ws.gpart_x, ws.gpart_k, ws.gchunks * ws.gtiles, sim->M, QB, grad_k,
                                                grad_rx);
  ET_HIP(hipGetLastError());
  return mf ? 1 : 2;
}


// ------------------------------------------------------------------ fused batches (host)

namespace {
int chunk_target(const et_sim_desc* s0, bool mf, int32_t wgs) {
  // record chunks over the whole batch for about `wgs` workgroups of the main kernel
  const int64_t per_chunk = (int64_t)s0->M * (mf ? row_tiles(s0) : (s0->F + DTILE - 1) / DTILE);
  return (int)std::max<int64_t>(1, (wgs + per_chunk - 1) / per_chunk);
}
}  // namespace

size_t synth_batch_ws_layout(int32_t J, const et_job* jobs, int64_t cap, const BatchTune& tune, bool adjoint,
                             char* base, SynthBatchWS* ws) {
  const et_sim_desc* s0 = jobs[0].sim;
  cap = std::max<int64_t>(cap, 1);
  SynthBatchWS w{};
  w.J = J;
  w.cap = cap;
  // one kernel for every job: in halves if each allows it, else FP32 over rows if each allows that (a job with its
  // bands on whole runs too), else per term
  w.fwd = FWD_HALVES;
  w.rows = 0;
  for (int32_t i = 0; i < J; ++i) {
    const FwdKernel k = fwd_kernel(jobs[i].sim);
    if (k == FWD_TERM || (k == FWD_ROWS && w.fwd == FWD_HALVES)) w.fwd = k;
    if (w.fwd == FWD_TERM) break;
  }
  for (int32_t i = 0; i < J; ++i) w.rows = std::max(w.rows, synth_rows(jobs[i].sim, nullptr));
  w.mf_bwd = adjoint;
  for (int32_t i = 0; i < J; ++i) w.mf_bwd = w.mf_bwd && synth_bwd_factorised_ok(jobs[i].sim);
  w.fold = 8;   // the coarsest folding every job allows
  for (int32_t i = 0; i < J; ++i) w.fold = std::min(w.fold, bands_fold(jobs[i].sim));
  const bool mf = w.fwd != FWD_TERM;
  w.target = chunk_target(s0, mf, tune.synth_wgs);
  w.target_bwd = chunk_target(s0, w.mf_bwd, tune.adjoint_wgs);
  // grid size: the chunk count is at most target + J (sum_j ceil(n_j / per)); buffers are
  // sized for the largest target the tuner tries, so that tuning keeps the workspace valid
  w.chunks = w.target + J;
  w.chunks_bwd = w.target_bwd + J;
  const int64_t cmax = chunk_target(s0, mf, TUNE_MAX_WGS) + J;
  const int64_t cmax_bwd = chunk_target(s0, w.mf_bwd, TUNE_MAX_WGS) + J;
  w.T1 = w.mf_bwd ? (int)((s0->F / K2 + KT1 - 1) / KT1) : 1;
  size_t off = 0;
  auto take = [&](size_t b) -> void* { void* p = base ? (void*)(base + off) : nullptr; off += al(b); return p; };
  const size_t MF2 = (size_t)s0->M * s0->F * 2;
  w.partial = (float*)take(sizeof(float) * MF2 * (size_t)std::max<int64_t>(cmax, w.chunks));
  if (adjoint) {
    const size_t cb = (size_t)std::max<int64_t>(cmax_bwd, w.chunks_bwd);
    w.gpart_x = (double*)take(sizeof(double) * 3 * cb * w.T1 * s0->M);
    w.gpart_k = (double*)take(sizeof(double) * cb * w.T1 * s0->M * s0->Q * s0->Bk);
  }
  off = vis_ws(cap, base, off, &w.vsum, &w.vidx);
  w.keys = (uint64_t*)take(sizeof(uint64_t) * (size_t)cap);
  w.sort_tmp = take(sort_temp_bytes(cap, 8));
  w.tab = (int64_t*)take(sizeof(int64_t) * (size_t)(3 * J + 2) * 2);
  w.jobs = take(sizeof(SynthArgs) * (size_t)J);
  w.tables = (float*)take(sizeof(float) * (size_t)J * (4 * (size_t)s0->Q * s0->Bk + 3 * s0->Q + 1));
  w.row_tables = take(sizeof(int2) * (size_t)J * (w.rows + 1));
  if (ws) *ws = w;
  return off;
}

namespace {
ChunkTab chunk_tab(const SynthBatchWS& w, int which) {
  int64_t* t = w.tab + (size_t)which * (3 * w.J + 2);
  return ChunkTab{t, t + w.J + 1, t + 2 * w.J + 1, t + 3 * w.J + 1, w.J};
}
}  // namespace

int synth_batch_run(int32_t J, const et_job* jobs, const et_paths* paths, const SynthBatchWS& w, Ctl* ctl,
                    float* spectra, const float* grad, double* grad_k, double* grad_rx, int* adjoint_kernel,
                    const hipEvent_t* ev, hipStream_t s) {
  const et_sim_desc* s0 = jobs[0].sim;
  const et_paths P = *paths;
  const int QB = s0->Q * s0->Bk;
  // job table with per-job band tables
  SynthArgs* dj = (SynthArgs*)w.jobs;
  const bool row_tables = w.fwd == FWD_ROWS || (w.fwd == FWD_HALVES && w.fold == 0);
  SynthJobPack pk{};
  for (int32_t i = 0; i < J; ++i) {
    SynthArgs a = make_args(jobs[i].sim, 0);
    a.lk = w.tables + (size_t)i * (4 * QB + 3 * s0->Q + 1);
    a.lc = a.lk + QB;
    a.ld = a.lc + QB;
    a.lp = a.ld + QB;
    a.lmax = a.lp + QB;
    if (row_tables) a.rows = (const int2*)w.row_tables + (size_t)i * (w.rows + 1);
    pk.j[pk.n++] = a;
    if (pk.n == SJOB_PACK || i + 1 == J) {
      k_put_synth_jobs<<<1, SJOB_PACK, 0, s>>>(pk, dj);
      pk.first += pk.n;
      pk.n = 0;
    }
  }
  k_band_tables_batch<<<J, 256, 0, s>>>(dj);
  // visible records, sorted by job (stable: each job keeps its record order)
  const int64_t tile = vis_tile(w.cap);
  const unsigned tiles = (unsigned)((w.cap + tile - 1) / tile);
  k_vis_count<<<tiles, 256, 0, s>>>(P, ctl, tile, w.vsum);
  k_vis_list<<<tiles, 256, 0, s>>>(P, ctl, tile, w.vsum, w.vidx);
  const unsigned nb = (unsigned)std::max<int64_t>(1, std::min<int64_t>((w.cap + 255) / 256, 4096));
  k_vis_jobkeys<<<nb, 256, 0, s>>>(P, w.vidx, ctl, w.keys);
  int bits = 0;
  while ((1ll << bits) < (int64_t)J) ++bits;
  if (bits > 0) radix_sort_u64(w.keys, w.vidx, 0, &ctl->n_vis, w.cap, bits, w.sort_tmp, s);
  const int64_t MF2 = (int64_t)s0->M * s0->F * 2;
  // forward
  {
    const ChunkTab ct = chunk_tab(w, 0);
    k_job_chunks<<<1, 256, 0, s>>>(w.keys, ctl, J, w.target, const_cast<int64_t*>(ct.off), const_cast<int64_t*>(ct.lo),
                                   const_cast<int64_t*>(ct.hi), const_cast<int64_t*>(ct.per));
    const SynthArgs a0 = make_args(s0, 0);
    if (ev) ET_HIP(hipEventRecord(ev[0], s));
    bool dir = false;
    for (int32_t i = 0; i < J; ++i) dir = dir || jobs[i].sim->directivity != nullptr;
    launch_fwd<true>(w.fwd, w.rows, w.fold, dir, w.chunks, s0->M, s, a0, dj, ct, P, w.vidx, ctl, w.partial);
    if (ev) ET_HIP(hipEventRecord(ev[1], s));
    k_reduce_batch<<<(unsigned)std::min<int64_t>((J * MF2 + 255) / 256, 8192), 256, 0, s>>>(w.partial, ct, MF2, spectra);
  }
  if (grad) {
    const ChunkTab ct = chunk_tab(w, 1);
    k_job_chunks<<<1, 256, 0, s>>>(w.keys, ctl, J, w.target_bwd, const_cast<int64_t*>(ct.off),
                                   const_cast<int64_t*>(ct.lo), const_cast<int64_t*>(ct.hi), const_cast<int64_t*>(ct.per));
    const SynthArgs a0 = make_args(s0, 0);
    if (ev) ET_HIP(hipEventRecord(ev[2], s));
    if (w.mf_bwd) {
      dim3 grid(w.chunks_bwd, s0->M, w.T1);
      launch_bwd_mfma<true>(s0->F / K2 <= 32, w.fold, grid, s, a0, dj, ct, P, w.vidx, ctl, grad, w.gpart_x,
                            w.gpart_k);
    } else {
      dim3 grid(w.chunks_bwd, s0->M);
      k_synth_bwd<true><<<grid, GB, sizeof(float2) * (size_t)s0->F, s>>>(a0, dj, ct, P, w.vidx, ctl, grad, w.gpart_x,
                                                                         w.gpart_k);
    }
    if (ev) ET_HIP(hipEventRecord(ev[3], s));
    for (int32_t j0 = 0; j0 < J; j0 += 65535) {   // (the grid's second dimension)
      ChunkTab part = ct;
      part.off += j0;
      k_bwd_reduce_batch<<<dim3(QB + 3 * s0->M, std::min(J - j0, 65535)), RED_T, 0, s>>>(
          w.gpart_x, w.gpart_k, part, w.T1, s0->M, QB, grad_k + (size_t)j0 * QB, grad_rx + (size_t)j0 * 3 * s0->M);
    }
    if (adjoint_kernel) *adjoint_kernel = w.mf_bwd ? 1 : 2;
  }
  ET_HIP(hipGetLastError());
  return w.fwd;
}

__global__ void k_sum_spectra(const float* __restrict__ in, int32_t J, int64_t n, float* __restrict__ out) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
    float acc = 0.f;
    for (int32_t j = 0; j < J; ++j) acc += in[(size_t)j * n + i];
    out[i] = acc;
  }
}

void sum_spectra(const float* in, int32_t J, int64_t n, float* out, hipStream_t s) {
  const unsigned grid = (unsigned)std::max<int64_t>(1, std::min<int64_t>((n + 255) / 256, 16384));
  k_sum_spectra<<<grid, 256, 0, s>>>(in, J, n, out);
  ET_HIP(hipGetLastError());
}

}  // namespace et
