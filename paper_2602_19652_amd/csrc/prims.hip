// Device primitives: exclusive scan (u64) and stable LSD radix sort (8-bit digits).
// Both take the element count either from the host or from device memory, so that they
// can run behind kernels whose output size is only known on the device (no host sync).
#include "internal.hpp"

#include <algorithm>

namespace et {

namespace {

constexpr int SB = 256;          // threads per block
constexpr int SI = 8;            // items per thread
constexpr int TILE = SB * SI;    // elements per block

__device__ inline int64_t get_n(int64_t n_host, const int64_t* n_dev) { return n_dev ? *n_dev : n_host; }

// Inclusive scan of one value per lane across the 64-lane wave.
template <typename T>
__device__ inline T wave_incl_scan(T v) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    T o = __shfl_up(v, d, 64);
    if (lane >= d) v += o;
  }
  return v;
}

// Exclusive scan across the block (SB threads); returns the block total in *total.
template <typename T>
__device__ inline T block_excl_scan(T v, T* total) {
  __shared__ T wsum[SB / 64];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  T inc = wave_incl_scan(v);
  if (lane == 63) wsum[w] = inc;
  __syncthreads();
  T off = 0, tot = 0;
#pragma unroll
  for (int i = 0; i < SB / 64; ++i) {
    if (i < w) off += wsum[i];
    tot += wsum[i];
  }
  __syncthreads();
  *total = tot;
  return off + inc - v;
}

__global__ void k_scan_reduce(const uint64_t* __restrict__ in, int64_t n_host, const int64_t* n_dev,
                              uint64_t* __restrict__ bsum) {
  const int64_t n = get_n(n_host, n_dev);
  const int64_t base = (int64_t)blockIdx.x * TILE;
  if (base >= n) return;
  uint64_t s = 0;
#pragma unroll
  for (int i = 0; i < SI; ++i) {
    int64_t idx = base + (int64_t)i * SB + threadIdx.x;
    if (idx < n) s += in[idx];
  }
  uint64_t tot;
  block_excl_scan<uint64_t>(s, &tot);
  if (threadIdx.x == 0) bsum[blockIdx.x] = tot;
}

// Single block: exclusive scan of the block sums, in chunks with a running carry.
__global__ void k_scan_blocks(uint64_t* __restrict__ bsum, int64_t n_host, const int64_t* n_dev,
                              uint64_t* __restrict__ total) {
  const int64_t n = get_n(n_host, n_dev);
  const int64_t nb = (n + TILE - 1) / TILE;
  uint64_t carry = 0;
  for (int64_t c = 0; c < nb; c += SB) {
    int64_t i = c + threadIdx.x;
    uint64_t v = i < nb ? bsum[i] : 0;
    uint64_t tot;
    uint64_t ex = block_excl_scan<uint64_t>(v, &tot);
    if (i < nb) bsum[i] = carry + ex;
    carry += tot;
  }
  if (threadIdx.x == 0 && total) *total = carry;
}

// IN_PLACE: bsum holds the blocks' sums, and each workgroup adds up those before its own (the first one all
// of them, for the total); else their exclusive scan (k_scan_blocks).
template <bool IN_PLACE>
__global__ void k_scan_apply(const uint64_t* __restrict__ in, uint64_t* __restrict__ out, int64_t n_host,
                             const int64_t* n_dev, const uint64_t* __restrict__ bsum, uint64_t* __restrict__ total) {
  const int64_t n = get_n(n_host, n_dev);
  const int64_t base = (int64_t)blockIdx.x * TILE;
  if (base >= n && blockIdx.x > 0) return;
  uint64_t before = IN_PLACE ? 0 : base < n ? bsum[blockIdx.x] : 0;
  if (IN_PLACE) {
    const int64_t nb = blockIdx.x > 0 ? (int64_t)blockIdx.x : (n + TILE - 1) / TILE;
    uint64_t s = 0, tot;
    for (int64_t k = threadIdx.x; k < nb; k += SB) s += bsum[k];
    block_excl_scan<uint64_t>(s, &tot);
    if (blockIdx.x > 0) before = tot;
    else if (threadIdx.x == 0 && total) *total = tot;
  }
  if (base >= n) return;
  // thread t owns the contiguous items [base + t*SI, base + t*SI + SI)
  uint64_t v[SI];
  uint64_t s = 0;
#pragma unroll
  for (int i = 0; i < SI; ++i) {
    int64_t idx = base + (int64_t)threadIdx.x * SI + i;
    v[i] = idx < n ? in[idx] : 0;
    s += v[i];
  }
  uint64_t tot;
  uint64_t ex = block_excl_scan<uint64_t>(s, &tot) + before;
#pragma unroll
  for (int i = 0; i < SI; ++i) {
    int64_t idx = base + (int64_t)threadIdx.x * SI + i;
    if (idx < n) out[idx] = ex;
    ex += v[i];
  }
}

// Short arrays (at most SCAN_ONE_MAX elements, e.g. a radix pass's digit counts): one
// workgroup scans the tiles in turn with a running carry, one launch instead of three.  Past
// two tiles the three-launch scan, whose workgroups run in parallel, is faster (measured at
// 16384 elements).  The count is clamped to the caller's bound n_max.
constexpr int64_t SCAN_ONE_MAX = 2 * TILE;
// Up to this many blocks (two million elements) a workgroup sums the block sums before its own itself, at most
// four loads per thread; a launch of its own for them takes 4 us.
constexpr int64_t SCAN_IN_PLACE_BLOCKS = 1024;

__global__ void k_scan_one(const uint64_t* __restrict__ in, uint64_t* __restrict__ out, int64_t n_host,
                           const int64_t* n_dev, int64_t n_max, uint64_t* __restrict__ total) {
  int64_t n = get_n(n_host, n_dev);
  n = n < n_max ? n : n_max;
  uint64_t carry = 0;
  for (int64_t base = 0; base < n; base += TILE) {
    // thread t owns the contiguous items [base + t*SI, base + t*SI + SI)
    uint64_t v[SI];
    uint64_t s = 0;
#pragma unroll
    for (int i = 0; i < SI; ++i) {
      const int64_t idx = base + (int64_t)threadIdx.x * SI + i;
      v[i] = idx < n ? in[idx] : 0;
      s += v[i];
    }
    uint64_t tot;
    uint64_t ex = block_excl_scan<uint64_t>(s, &tot) + carry;
#pragma unroll
    for (int i = 0; i < SI; ++i) {
      const int64_t idx = base + (int64_t)threadIdx.x * SI + i;
      if (idx < n) out[idx] = ex;
      ex += v[i];
    }
    carry += tot;
  }
  if (threadIdx.x == 0 && total) *total = carry;
}

// ------------------------------------------------------------------ radix sort

// 8-bit digits, two launches per pass: per-block digit counts, then the scatter, whose workgroups add up the
// counts before their own block themselves (a row of 256 counts per block, read by one thread per digit).  The
// passes of 4-bit digits before took three to five launches each, twice as many passes, and ranked the items
// with 16 counters per thread in LDS (8 us a pass for 45,000 keys; a pass of 8 bits takes 4 + 9 us, so half as
// much a key).  Bound by the scatter's reads of the other blocks' counts and its scattered writes.
constexpr int RBITS = 8;
constexpr int RADIX = 1 << RBITS;
constexpr int RT = 256;   // threads per block: one per digit

// Lanes of the wave whose active item has the same digit as this lane's.
__device__ inline uint64_t same_digit(uint32_t d, bool active) {
  uint64_t m = __ballot(active);
#pragma unroll
  for (int b = 0; b < RBITS; ++b) {
    const uint64_t s = __ballot((d >> b) & 1u);
    m &= ((d >> b) & 1u) ? s : ~s;
  }
  return m;
}

// Counts of each digit in this block's items: hist[block][digit].  per: items per block.
template <typename K>
__global__ __launch_bounds__(RT) void k_radix_hist(const K* __restrict__ keys, int64_t n_host, const int64_t* n_dev,
                                                   int64_t per, int shift, uint32_t* __restrict__ hist) {
  const int64_t n = get_n(n_host, n_dev);
  __shared__ uint32_t cnt[RADIX];
  cnt[threadIdx.x] = 0;
  __syncthreads();
  const int64_t lo = blockIdx.x * per, hi = lo + per < n ? lo + per : n;
  for (int64_t i = lo + threadIdx.x; i < hi; i += RT) atomicAdd(&cnt[(uint32_t)(keys[i] >> shift) & (RADIX - 1)], 1u);
  __syncthreads();
  hist[(int64_t)blockIdx.x * RADIX + threadIdx.x] = cnt[threadIdx.x];
}

// Stable scatter, 2048 items of the block at a time in registers.  Each wave owns 512 consecutive ones and ranks
// them 64 at a time in order: an item's place is its digit's start, plus the counts of earlier blocks, of
// earlier waves, and of its wave's items before it (by comparing digits over the wave).
constexpr int RSTEPS = 8;
constexpr int RTILE = RT * RSTEPS;
template <typename K>
__global__ __launch_bounds__(RT) void k_radix_scatter(const K* __restrict__ kin, const int32_t* __restrict__ vin,
                                                      K* __restrict__ kout, int32_t* __restrict__ vout, int64_t n_host,
                                                      const int64_t* n_dev, int64_t per, int shift,
                                                      const uint32_t* __restrict__ hist, int nblocks) {
  const int64_t n = get_n(n_host, n_dev);
  const int64_t lo = blockIdx.x * per, hi = lo + per < n ? lo + per : n;
  if (lo >= n) return;
  __shared__ uint32_t wcnt[RT / 64][RADIX];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  // digit tid: items of earlier blocks, and of all blocks
  uint32_t before = 0, all = 0;
  {
    int b = 0;
    for (; b + 16 <= nblocks; b += 16) {
      uint32_t v[16];
#pragma unroll
      for (int k = 0; k < 16; ++k) v[k] = hist[(int64_t)(b + k) * RADIX + tid];
#pragma unroll
      for (int k = 0; k < 16; ++k) {
        all += v[k];
        before += b + k < (int)blockIdx.x ? v[k] : 0u;
      }
    }
    for (; b < nblocks; ++b) {
      const uint32_t v = hist[(int64_t)b * RADIX + tid];
      all += v;
      before += b < (int)blockIdx.x ? v : 0u;
    }
  }
  uint32_t tot;
  uint32_t start = block_excl_scan<uint32_t>(all, &tot) + before;
  for (int64_t t0 = lo; t0 < hi; t0 += RTILE) {
    const int64_t w0 = t0 + wv * (RTILE / (RT / 64)) + lane;
    K k[RSTEPS];
    int32_t v[RSTEPS];
    uint32_t at[RSTEPS];
#pragma unroll
    for (int i = 0; i < RSTEPS; ++i) {
      const int64_t e = w0 + 64 * i;
      k[i] = e < hi ? kin[e] : K{};
      v[i] = e < hi ? vin[e] : 0;
    }
#pragma unroll
    for (int w = 0; w < RT / 64; ++w) wcnt[w][tid] = 0;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < RSTEPS; ++i) {
      const bool in = w0 + 64 * i < hi;
      const uint32_t d = (uint32_t)(k[i] >> shift) & (RADIX - 1);
      const uint64_t m = same_digit(d, in);
      const uint64_t below = m & ((1ull << lane) - 1ull);
      const uint32_t c = in ? wcnt[wv][d] : 0u;
      at[i] = c + (uint32_t)__popcll(below);
      __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
      __builtin_amdgcn_wave_barrier();
      if (in && below == 0) wcnt[wv][d] = c + (uint32_t)__popcll(m);   // the first lane of the digit
      __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
      __builtin_amdgcn_wave_barrier();
    }
    __syncthreads();
#pragma unroll
    for (int w = 0; w < RT / 64; ++w) {
      const uint32_t c = wcnt[w][tid];
      wcnt[w][tid] = start;
      start += c;
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < RSTEPS; ++i) {
      if (w0 + 64 * i < hi) {
        const uint32_t pos = wcnt[wv][(uint32_t)(k[i] >> shift) & (RADIX - 1)] + at[i];
        kout[pos] = k[i];
        vout[pos] = v[i];
      }
    }
    __syncthreads();
  }
}

int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

}  // namespace

size_t scan_temp_bytes(int64_t n_max) { return (size_t)(ceil_div(n_max > 0 ? n_max : 1, TILE) + 1) * sizeof(uint64_t); }

void scan_exclusive_u64(const uint64_t* in, uint64_t* out, int64_t n_host, const int64_t* n_dev, int64_t n_max,
                        uint64_t* total, void* temp, hipStream_t s) {
  if (n_max <= 0) n_max = 1;
  if (n_max <= SCAN_ONE_MAX) {
    k_scan_one<<<1, SB, 0, s>>>(in, out, n_host, n_dev, n_max, total);
    ET_HIP(hipGetLastError());
    return;
  }
  const int64_t nb = ceil_div(n_max, TILE);
  uint64_t* bsum = (uint64_t*)temp;
  k_scan_reduce<<<(unsigned)nb, SB, 0, s>>>(in, n_host, n_dev, bsum);
  if (nb <= SCAN_IN_PLACE_BLOCKS) {
    k_scan_apply<true><<<(unsigned)nb, SB, 0, s>>>(in, out, n_host, n_dev, bsum, total);
  } else {
    k_scan_blocks<<<1, SB, 0, s>>>(bsum, n_host, n_dev, total);
    k_scan_apply<false><<<(unsigned)nb, SB, 0, s>>>(in, out, n_host, n_dev, bsum, nullptr);
  }
  ET_HIP(hipGetLastError());
}

namespace {
// Items per block of a radix pass: 2048, more where that would make over 512 blocks (every block of the scatter
// reads the others' counts, 1 KB each).
constexpr int64_t RADIX_BLOCKS = 512;
int64_t radix_per(int64_t n) { return ceil_div(ceil_div(n, RADIX_BLOCKS), RTILE) * RTILE; }
}  // namespace

size_t sort_temp_bytes(int64_t n, int key_bytes) {
  if (n <= 0) n = 1;
  size_t b = 0;
  b += (size_t)n * key_bytes + 256;          // key ping-pong
  b += (size_t)n * sizeof(int32_t) + 256;    // value ping-pong
  // digit counts, of as many blocks as any smaller array has (radix_per grows in steps, at which the blocks
  // become fewer: a scratch sized for an array serves every shorter one)
  b += (size_t)RADIX * std::min<int64_t>(ceil_div(n, RTILE), RADIX_BLOCKS) * sizeof(uint32_t) + 256;
  return b;
}

// An odd number of passes ends with a copy back, by a kernel (a captured graph records no copy of n_max bytes
// whose tail nothing wrote).
template <typename K>
__global__ __launch_bounds__(RT) void k_copy_pairs(const K* __restrict__ kin, const int32_t* __restrict__ vin,
                                                   K* __restrict__ kout, int32_t* __restrict__ vout, int64_t n_host,
                                                   const int64_t* n_dev) {
  const int64_t n = get_n(n_host, n_dev);
  for (int64_t i = (int64_t)blockIdx.x * RT + threadIdx.x; i < n; i += (int64_t)gridDim.x * RT) {
    kout[i] = kin[i];
    vout[i] = vin[i];
  }
}

template <typename K>
static void radix_sort_impl(K* keys, int32_t* vals, int64_t n_host, const int64_t* n_dev, int64_t n_max, int bits,
                            void* temp, hipStream_t s) {
  if (n_max <= 0) return;
  const int64_t per = radix_per(n_max), nb = ceil_div(n_max, per);
  char* t = (char*)temp;
  auto take = [&](size_t bytes) { char* p = t; t += (bytes + 255) / 256 * 256; return (void*)p; };
  K* k2 = (K*)take((size_t)n_max * sizeof(K));
  int32_t* v2 = (int32_t*)take((size_t)n_max * sizeof(int32_t));
  uint32_t* hist = (uint32_t*)take((size_t)RADIX * nb * sizeof(uint32_t));
  K* ka = keys; int32_t* va = vals; K* kb = k2; int32_t* vb = v2;
  const int passes = (bits + RBITS - 1) / RBITS;
  for (int p = 0; p < passes; ++p) {
    const int shift = p * RBITS;
    k_radix_hist<K><<<(unsigned)nb, RT, 0, s>>>(ka, n_host, n_dev, per, shift, hist);
    k_radix_scatter<K><<<(unsigned)nb, RT, 0, s>>>(ka, va, kb, vb, n_host, n_dev, per, shift, hist, (int)nb);
    ET_HIP(hipGetLastError());
    K* tk = ka; ka = kb; kb = tk;
    int32_t* tv = va; va = vb; vb = tv;
  }
  if (ka != keys) {
    k_copy_pairs<K><<<(unsigned)std::min<int64_t>(ceil_div(n_max, RT), 4096), RT, 0, s>>>(ka, va, keys, vals, n_host, n_dev);
    ET_HIP(hipGetLastError());
  }
}

void radix_sort_u32(uint32_t* keys, int32_t* vals, int64_t n, int bits, void* temp, hipStream_t s) {
  radix_sort_impl<uint32_t>(keys, vals, n, nullptr, n, bits, temp, s);
}

void radix_sort_u64(uint64_t* keys, int32_t* vals, int64_t n_host, const int64_t* n_dev, int64_t n_max, int bits,
                    void* temp, hipStream_t s) {
  radix_sort_impl<uint64_t>(keys, vals, n_host, n_dev, n_max, bits, temp, s);
}

}  // namespace et
