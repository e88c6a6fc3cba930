// Load-time build kernels for gfx950 (Sec. 3.1 data structure, Sec. 3.3 Eq. 1).
//
//  Morton orders: cloud box and finite check -> 63-bit Morton codes -> stable
//  sort (radix passes over the code's leading bits, then the runs that these
//  leave equal, in LDS) -> records of position and colour -> per batch: gather,
//  box, Eq. 1 words (one kernel).  Input order: the last kernel alone.
//  Uneven clouds, where a run is too long for LDS: the sort goes on over every
//  bit, and the kernels after it, which did nothing, run then.  A build with one
//  point 1,000 extents away, by one sort of every bit in 8-bit passes as it was at
//  first, by a build that was made and thrown away, and now: 2e5 points 460, 890,
//  421 us; 2e7 4.30, 8.20, 3.14 ms; 5e8 74-79, 195-200, 72.5 ms.
//
// Boxes order binary32 values by IEEE totalOrder (-0 below +0) through the
// monotone integer map okey(), so a box depends only on the point set, not on
// the order of a parallel reduction.
#include "internal.h"

namespace ptr {
namespace {

__device__ __forceinline__ uint32_t okey(float f) {
  const uint32_t u = __float_as_uint(f);
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}
__device__ __forceinline__ float okey_inv(uint32_t k) {
  return __uint_as_float((k & 0x80000000u) ? (k & 0x7FFFFFFFu) : ~k);
}

// Workgroups are dealt to the eight XCDs in turn, each with an L2 of its own.
// Where neighbouring tiles write parts of the same lines, or read them, workgroup
// b takes tile (b mod 8) per + b / 8 instead of tile b: an XCD then works on one
// contiguous eighth and its L2 puts the parts together.  The grid is 8 per; a
// tile at or past tiles is none.
constexpr uint32_t XCDS = 8;
inline uint32_t xcd_grid(uint64_t tiles) { return (uint32_t)((tiles + XCDS - 1) / XCDS * XCDS); }
__device__ __forceinline__ uint32_t xcd_tile() { return blockIdx.x % XCDS * (gridDim.x / XCDS) + blockIdx.x / XCDS; }

// ---------------------------------------------------------- finite check
__global__ void __launch_bounds__(256) k_finite(const uint32_t* __restrict__ w, uint64_t nwords,
                                                uint32_t* __restrict__ flag) {
  const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
  bool bad = false;
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < nwords; i += stride)
    bad |= (w[i] & 0x7F800000u) == 0x7F800000u;
  if (__ballot(bad) != 0 && (threadIdx.x & 63) == 0) atomicOr(flag, 1u);
}

__global__ void __launch_bounds__(256) k_iota(uint32_t* __restrict__ p, uint64_t n) {
  const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) p[i] = (uint32_t)i;
}

// ------------------------------------------------------------- cloud box
struct Box {
  uint32_t mn[3], mx[3];
};
__device__ __forceinline__ Box empty_box() {
  return {{0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu}, {0u, 0u, 0u}};
}
__device__ __forceinline__ void grow(Box& b, int a, float f) {
  const uint32_t k = okey(f);
  b.mn[a] = min(b.mn[a], k);
  b.mx[a] = max(b.mx[a], k);
}
// The workgroup's box (every thread gets it).  red: LDS, one Box per wave.
__device__ __forceinline__ Box block_box(Box b, Box* red) {
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    for (int o = 32; o > 0; o >>= 1) {
      b.mn[a] = min(b.mn[a], (uint32_t)__shfl_xor((int)b.mn[a], o));
      b.mx[a] = max(b.mx[a], (uint32_t)__shfl_xor((int)b.mx[a], o));
    }
  }
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = b;
  __syncthreads();
  for (uint32_t w = 0; w < blockDim.x / 64; ++w) {
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      b.mn[a] = min(b.mn[a], red[w].mn[a]);
      b.mx[a] = max(b.mx[a], red[w].mx[a]);
    }
  }
  return b;
}
__device__ __forceinline__ bool not_finite(float f) { return (__float_as_uint(f) & 0x7F800000u) == 0x7F800000u; }
// A look first: where every wave has cause, the atomics of millions of waves on one word would queue.
__device__ __forceinline__ void raise(uint32_t* flag, bool bad) {
  if (__ballot(bad) != 0 && (threadIdx.x & 63) == 0 &&
      __hip_atomic_load(flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == 0)
    atomicOr(flag, 1u);
}

// The cloud box, and the finite check on the same loads (flag: set if a
// coordinate is NaN or Inf).  One box per workgroup, reduced by a second
// launch: 4,096 workgroups combining theirs by atomics on one line took 1.14
// ms for any cloud (28 % of a 2e7-point build), 40 us with the partial boxes.
constexpr uint32_t BOX_BLOCKS = 1024;
__global__ void __launch_bounds__(256) k_aabb(const float* __restrict__ xyz, uint64_t n, Box* __restrict__ part,
                                              uint32_t* __restrict__ flag) {
  __shared__ Box red[4];
  Box box = empty_box();
  bool bad = false;
  const uint64_t stride = (uint64_t)gridDim.x * blockDim.x, n4 = n / 4;
  const uint64_t t0 = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const float4* const v4 = reinterpret_cast<const float4*>(xyz);
  for (uint64_t g = t0; g < n4; g += stride) {  // four points: three 16-byte loads
    const float4 u = v4[3 * g], v = v4[3 * g + 1], w = v4[3 * g + 2];
    const float f[12] = {u.x, u.y, u.z, u.w, v.x, v.y, v.z, v.w, w.x, w.y, w.z, w.w};
#pragma unroll
    for (int j = 0; j < 12; ++j) {
      bad |= not_finite(f[j]);
      grow(box, j % 3, f[j]);
    }
  }
  for (uint64_t i = 4 * n4 + t0; i < n; i += stride) {
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      bad |= not_finite(xyz[3 * i + a]);
      grow(box, a, xyz[3 * i + a]);
    }
  }
  raise(flag, bad);
  box = block_box(box, red);
  if (threadIdx.x == 0) part[blockIdx.x] = box;
}
__global__ void __launch_bounds__(256) k_aabb_top(const Box* __restrict__ part, uint32_t blocks,
                                                  uint32_t* __restrict__ aabb) {
  __shared__ Box red[4];
  Box box = empty_box();
  for (uint32_t i = threadIdx.x; i < blocks; i += 256) {
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      box.mn[a] = min(box.mn[a], part[i].mn[a]);
      box.mx[a] = max(box.mx[a], part[i].mx[a]);
    }
  }
  box = block_box(box, red);
  if (threadIdx.x == 0) {
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      aabb[a] = box.mn[a];
      aabb[3 + a] = box.mx[a];
    }
  }
}

// ---------------------------------------------------------- Morton codes
__device__ __forceinline__ uint64_t spread3(uint64_t x) {  // bit b -> bit 3b (21 bits)
  x &= 0x1FFFFFull;
  x = (x | (x << 32)) & 0x1F00000000FFFFull;
  x = (x | (x << 16)) & 0x1F0000FF0000FFull;
  x = (x | (x << 8)) & 0x100F00F00F00F00Full;
  x = (x | (x << 4)) & 0x10C30C30C30C30C3ull;
  x = (x | (x << 2)) & 0x1249249249249249ull;
  return x;
}

// min(floor(fl(d scale / s)), scale - 1) for d = x - lo, s = hi - lo in
// binary64, scale a power of two up to 2^30, with the quotient rounded once as
// the contract says; 0 for an empty extent.  The quotient comes from the axis's
// reciprocal (two roundings, off by less than 2^-20 below 2^30); unless it lies
// that close to a whole number, its floor is the rounded quotient's floor too.
// The rest, about one coordinate in 2^19, takes the division.
struct Axis {
  double lo, s, inv;  // inv = scale / s, 0 for an empty extent
};
__device__ __forceinline__ Axis make_axis(float lo, float hi, double scale) {
  Axis a;
  a.lo = (double)lo;
  a.s = (double)hi - (double)lo;
  a.inv = a.s == 0.0 ? 0.0 : scale / a.s;
  return a;
}
__device__ __forceinline__ uint32_t axis_cell(const Axis& a, float x, double scale) {
  const double d = (double)x - a.lo, q = d * a.inv, f = floor(q), r = q - f;
  uint32_t c = (uint32_t)f;
  if (!(r > 0x1p-20 && r < 1.0 - 0x1p-20)) {
    const double e = a.s == 0.0 ? 0.0 : floor((d * scale) / a.s);
    c = e > scale - 1.0 ? (uint32_t)(scale - 1.0) : (uint32_t)e;
  }
  return c;
}

// ------------------------------------------------------------ radix sort
// Stable LSD radix sort of (u64 key, u32 value) pairs, RS_BITS bits per pass,
// of the leading bits only; k_fix_runs orders what these leave equal.  Each
// workgroup owns a tile of RS_TILE consecutive elements.  count: per-tile digit
// histogram, stored digit-major (hist[d * nblk + blk]); an exclusive scan of
// that array gives every (digit, tile) its output offset; scatter: the tile is
// ranked in input order and leaves in digit runs.
constexpr int RS_BITS = 9, RS_DIGITS = 1 << RS_BITS;
constexpr int RS_THREADS = 512, RS_WAVES = RS_THREADS / 64;
constexpr int RS_ITEMS = 16;
constexpr uint64_t RS_TILE = (uint64_t)RS_THREADS * RS_ITEMS;
constexpr uint64_t SCAN_CHUNK = 4096;
constexpr int KEY_BITS = 63;

__device__ __forceinline__ uint32_t digit_of(uint64_t key, int shift) {
  return (uint32_t)(key >> shift) & (uint32_t)(RS_DIGITS - 1);
}
__device__ __forceinline__ void put_histogram(const uint32_t* h, uint32_t* hist, uint64_t nblk) {
  static_assert(RS_DIGITS <= RS_THREADS, "one digit per thread");
  if (threadIdx.x < RS_DIGITS) hist[(uint64_t)threadIdx.x * nblk + blockIdx.x] = h[threadIdx.x];
}

// Morton codes of a tile, and the histogram of their digit at shift (the first pass needs no count launch).
__global__ void __launch_bounds__(RS_THREADS) k_morton(const float* __restrict__ xyz, uint64_t n,
                                                       const uint32_t* __restrict__ aabb, uint64_t* __restrict__ keys,
                                                       int shift, uint32_t* __restrict__ hist, uint64_t nblk) {
  __shared__ uint32_t h[RS_DIGITS];
  if (threadIdx.x < RS_DIGITS) h[threadIdx.x] = 0;
  __syncthreads();
  constexpr double SCALE = 2097152.0;  // 21 bits per axis
  Axis ax[3];
#pragma unroll
  for (int a = 0; a < 3; ++a) ax[a] = make_axis(okey_inv(aabb[a]), okey_inv(aabb[3 + a]), SCALE);
  const uint64_t base = (uint64_t)blockIdx.x * RS_TILE;
#pragma unroll 4
  for (int it = 0; it < RS_ITEMS; ++it) {
    const uint64_t i = base + (uint64_t)it * RS_THREADS + threadIdx.x;
    if (i < n) {
      const uint64_t qx = axis_cell(ax[0], xyz[3 * i], SCALE);
      const uint64_t qy = axis_cell(ax[1], xyz[3 * i + 1], SCALE);
      const uint64_t qz = axis_cell(ax[2], xyz[3 * i + 2], SCALE);
      const uint64_t key = spread3(qx) | (spread3(qy) << 1) | (spread3(qz) << 2);
      keys[i] = key;
      atomicAdd(&h[digit_of(key, shift)], 1u);
    }
  }
  __syncthreads();
  put_histogram(h, hist, nblk);
}

__global__ void __launch_bounds__(RS_THREADS) k_radix_count(const uint64_t* __restrict__ keys, uint64_t n, int shift,
                                                            uint32_t* __restrict__ hist, uint64_t nblk) {
  __shared__ uint32_t h[RS_DIGITS];
  if (threadIdx.x < RS_DIGITS) h[threadIdx.x] = 0;
  __syncthreads();
  const uint64_t base = (uint64_t)blockIdx.x * RS_TILE;
  uint64_t k[RS_ITEMS];
#pragma unroll
  for (int it = 0; it < RS_ITEMS; ++it) {
    const uint64_t i = base + (uint64_t)it * RS_THREADS + threadIdx.x;
    k[it] = i < n ? keys[i] : 0ull;
  }
#pragma unroll
  for (int it = 0; it < RS_ITEMS; ++it)
    if (base + (uint64_t)it * RS_THREADS + threadIdx.x < n) atomicAdd(&h[digit_of(k[it], shift)], 1u);
  __syncthreads();
  put_histogram(h, hist, nblk);
}

// exclusive scan of m u32 values: partial sums, top-level scan, apply
__global__ void __launch_bounds__(256) k_scan_partials(const uint32_t* __restrict__ x, uint64_t m,
                                                       uint32_t* __restrict__ part) {
  const uint64_t base = (uint64_t)blockIdx.x * SCAN_CHUNK;
  uint32_t s = 0;
  for (uint64_t i = base + threadIdx.x; i < base + SCAN_CHUNK && i < m; i += 256) s += x[i];
  for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o);
  __shared__ uint32_t ws[4];
  if ((threadIdx.x & 63) == 0) ws[threadIdx.x >> 6] = s;
  __syncthreads();
  if (threadIdx.x == 0) part[blockIdx.x] = ws[0] + ws[1] + ws[2] + ws[3];
}

// Block-wide exclusive scan of one value per thread (WAVES waves); returns the
// exclusive prefix and writes the block total to *total.
template <int WAVES = 4>
__device__ __forceinline__ uint32_t block_exclusive_scan(uint32_t v, uint32_t* total) {
  __shared__ uint32_t ws[WAVES];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  uint32_t inc = v;
  for (int o = 1; o < 64; o <<= 1) {
    const uint32_t y = __shfl_up(inc, o);
    if (lane >= o) inc += y;
  }
  if (lane == 63) ws[wave] = inc;
  __syncthreads();
  uint32_t wbase = 0;
  uint32_t tot = 0;
  for (int w = 0; w < WAVES; ++w) {
    if (w < wave) wbase += ws[w];
    tot += ws[w];
  }
  __syncthreads();
  *total = tot;
  return wbase + inc - v;
}

__global__ void __launch_bounds__(256) k_scan_top(uint32_t* __restrict__ part, uint64_t np) {
  uint32_t carry = 0;
  for (uint64_t base = 0; base < np; base += 256) {
    const uint64_t i = base + threadIdx.x;
    const uint32_t v = i < np ? part[i] : 0u;
    uint32_t tot;
    const uint32_t ex = block_exclusive_scan(v, &tot);
    if (i < np) part[i] = carry + ex;
    carry += tot;
  }
}

__global__ void __launch_bounds__(256) k_scan_apply(uint32_t* __restrict__ x, uint64_t m,
                                                    const uint32_t* __restrict__ part) {
  const uint64_t base = (uint64_t)blockIdx.x * SCAN_CHUNK;
  uint32_t carry = part[blockIdx.x];
  for (uint64_t off = 0; off < SCAN_CHUNK; off += 256) {
    const uint64_t i = base + off + threadIdx.x;
    const uint32_t v = i < m ? x[i] : 0u;
    uint32_t tot;
    const uint32_t ex = block_exclusive_scan(v, &tot);
    if (i < m) x[i] = carry + ex;
    carry += tot;
  }
}

// The same scan of up to SCAN_SMALL values (8,192-point tiles of about a million points) by one workgroup in one
// launch, all loads in flight together.  SMALL_FIGURES
constexpr int SS_WAVES = 16, SS_THREADS = 64 * SS_WAVES, SS_ITEMS = 16;  // items of four values per thread
constexpr uint64_t SCAN_SMALL = 4ull * SS_ITEMS * SS_THREADS;
__global__ void __launch_bounds__(SS_THREADS) k_scan_small(uint32_t* __restrict__ x, uint64_t m) {
  __shared__ uint32_t sums[SS_ITEMS * SS_WAVES];
  static_assert(SS_ITEMS * SS_WAVES == 256, "four sums per lane of the first wave");
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const uint32_t m4 = (uint32_t)(m / 4);  // m is a multiple of the digits of a pass
  uint4* const x4 = reinterpret_cast<uint4*>(x);
  uint4 v[SS_ITEMS];
  uint32_t ex[SS_ITEMS];
#pragma unroll
  for (int j = 0; j < SS_ITEMS; ++j) {
    const uint32_t i = j * SS_THREADS + threadIdx.x;
    v[j] = i < m4 ? x4[i] : make_uint4(0, 0, 0, 0);
  }
#pragma unroll
  for (int j = 0; j < SS_ITEMS; ++j) {
    const uint32_t own = v[j].x + v[j].y + v[j].z + v[j].w;
    uint32_t inc = own;
    for (int o = 1; o < 64; o <<= 1) {
      const uint32_t y = __shfl_up(inc, o);
      if (lane >= o) inc += y;
    }
    ex[j] = inc - own;
    if (lane == 63) sums[j * SS_WAVES + wave] = inc;
  }
  __syncthreads();
  if (wave == 0) {
    const uint4 s = reinterpret_cast<uint4*>(sums)[lane];
    const uint32_t own = s.x + s.y + s.z + s.w;
    uint32_t inc = own;
    for (int o = 1; o < 64; o <<= 1) {
      const uint32_t y = __shfl_up(inc, o);
      if (lane >= o) inc += y;
    }
    const uint32_t e = inc - own;
    reinterpret_cast<uint4*>(sums)[lane] = make_uint4(e, e + s.x, e + s.x + s.y, e + s.x + s.y + s.z);
  }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < SS_ITEMS; ++j) {
    const uint32_t i = j * SS_THREADS + threadIdx.x, e = ex[j] + sums[j * SS_WAVES + wave];
    if (i < m4) x4[i] = make_uint4(e, e + v[j].x, e + v[j].x + v[j].y, e + v[j].x + v[j].y + v[j].z);
  }
}

// Scatter of one pass.  Each wave ranks its 1,024 consecutive elements alone,
// against digit counters of its own (ballots give the rank among equal digits
// of a 64-element row, the counter carries it over the rows): no barrier until
// the whole tile is ranked, where one counter row per 256 elements took three.
// The tile then moves through LDS in digit order, keys first, values after them
// in the same space, so that consecutive threads write consecutive slots of one
// digit's range.  The first pass's values are the indices themselves (vin null).
// Bound by memory: 24 bytes an element; the runs of a digit (16 elements, 128 and
// 64 bytes, unaligned) of neighbouring tiles share lines, so the tiles are dealt
// to the XCDs in contiguous eighths (5e8 elements: 2.66 ms, 4.5 TB/s; tiles dealt
// in turn 5.9 ms; the earlier scatter of 4,096-element tiles and 8-bit digits 5.6).
__global__ void __launch_bounds__(RS_THREADS) k_radix_scatter(
    const uint64_t* __restrict__ kin, const uint32_t* __restrict__ vin, uint64_t* __restrict__ kout,
    uint32_t* __restrict__ vout, uint64_t n, int shift, const uint32_t* __restrict__ offs, uint64_t nblk) {
  __shared__ uint64_t stage[RS_TILE];
  __shared__ uint16_t cnt[RS_WAVES][RS_DIGITS];  // a wave's count of a digit, then the digit's start in the wave's part
  __shared__ uint32_t gout[RS_DIGITS];           // output slot of the tile's LDS slot 0, as seen from digit d
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const uint64_t blk = xcd_tile();
  if (blk >= nblk) return;
  const uint64_t base = blk * RS_TILE, wbase = base + (uint64_t)wave * (64 * RS_ITEMS);
  uint64_t key[RS_ITEMS];
  uint32_t val[RS_ITEMS];
#pragma unroll
  for (int it = 0; it < RS_ITEMS; ++it) {
    const uint64_t i = wbase + it * 64 + lane;
    key[it] = i < n ? kin[i] : 0ull;
    val[it] = vin ? (i < n ? vin[i] : 0u) : (uint32_t)i;
  }
  for (int d = lane; d < RS_DIGITS; d += 64) cnt[wave][d] = 0;
  __builtin_amdgcn_wave_barrier();
  const uint64_t lt_mask = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
  uint16_t rank[RS_ITEMS];
#pragma unroll
  for (int it = 0; it < RS_ITEMS; ++it) {
    const bool valid = wbase + it * 64 + lane < n;
    const uint32_t d = digit_of(key[it], shift);
    uint64_t peers = __ballot(valid);
#pragma unroll
    for (int bit = 0; bit < RS_BITS; ++bit) {
      const bool set = (d >> bit) & 1u;
      const uint64_t mk = __ballot(set);
      peers &= set ? mk : ~mk;
    }
    const uint32_t r = __popcll(peers & lt_mask);
    const uint32_t before = cnt[wave][d];
    __builtin_amdgcn_wave_barrier();  // every lane has read the counter before its first peer adds
    if (valid && r == 0) cnt[wave][d] = (uint16_t)(before + __popcll(peers));
    __builtin_amdgcn_wave_barrier();
    rank[it] = (uint16_t)(before + r);
  }
  __syncthreads();
  uint32_t sum = 0;
  if (tid < RS_DIGITS) {
    for (int w = 0; w < RS_WAVES; ++w) sum += cnt[w][tid];
  }
  uint32_t total;
  uint32_t start = block_exclusive_scan<RS_WAVES>(sum, &total);  // of the digit in the tile
  if (tid < RS_DIGITS) {
    gout[tid] = offs[(uint64_t)tid * nblk + blk] - start;  // wraps; added to an LDS slot it does not
    for (int w = 0; w < RS_WAVES; ++w) {
      const uint32_t c = cnt[w][tid];
      cnt[w][tid] = (uint16_t)start;  // below RS_TILE
      start += c;
    }
  }
  __syncthreads();
  static_assert(RS_TILE <= 65536, "slots in 16 bits");
  const uint32_t nt = (uint32_t)(n - base < RS_TILE ? n - base : RS_TILE);
#pragma unroll
  for (int it = 0; it < RS_ITEMS; ++it) {
    const bool valid = wbase + it * 64 + lane < n;
    rank[it] = (uint16_t)(rank[it] + cnt[wave][digit_of(key[it], shift)]);
    if (valid) stage[rank[it]] = key[it];
  }
  __syncthreads();
  uint32_t pos[RS_ITEMS];
#pragma unroll
  for (int it = 0; it < RS_ITEMS; ++it) {
    const uint32_t p = it * RS_THREADS + tid;
    pos[it] = ~0u;
    if (p < nt) {
      const uint64_t k = stage[p];
      pos[it] = gout[digit_of(k, shift)] + p;
      if (pos[it] < n) kout[pos[it]] = k;  // always true for a consistent histogram; never write outside
    }
  }
  __syncthreads();
  uint32_t* const vstage = reinterpret_cast<uint32_t*>(stage);
#pragma unroll
  for (int it = 0; it < RS_ITEMS; ++it)
    if (wbase + it * 64 + lane < n) vstage[rank[it]] = val[it];
  __syncthreads();
#pragma unroll
  for (int it = 0; it < RS_ITEMS; ++it) {
    const uint32_t p = it * RS_THREADS + tid;
    if (p < nt && pos[it] < n) vout[pos[it]] = vstage[p];
  }
}

// Orders the runs of elements whose keys agree from bit shift up, by the whole
// key, stably, and writes the values alone (the keys stay as they are).  An
// element moves left by the number of earlier ones of its run with a larger key
// and right by the number of later ones with a smaller key.  Runs of more than
// RUN_MAX + 1 elements are left as they are; flag is set if one of them is out
// of order (one of equal keys is not, however long).
//
// Bound by its memory traffic where runs are short: 16 bytes an element at 4.8
// TB/s (5e8 points of an even surface: 1.66 ms; 1.75 when every element walked
// to the ends of its run).  How far a run reaches is found first, by doubling and
// halving steps, so that no element of a long run walks it.  Whole builds, with
// the walk and now: 5e8 points with a third of them equal 77 -> 42 ms, with the
// box 8 times wider than the points (about a hundred a run) 59 -> 47.
constexpr int FIX_THREADS = 256, FIX_ITEMS = 8, RUN_MAX = 256;
constexpr int FIX_TILE = FIX_THREADS * FIX_ITEMS;

// Elements of the run of mine = k[at] on one side (DIR -1: before it, 1: after it), RUN_MAX + 1 at most.  The keys are
// in the order of their leading bits, so a run has no gaps.
template <int DIR>
__device__ __forceinline__ int run_side(const uint64_t* k, int at, uint64_t mine, int shift) {
  const auto same = [&](int d) { return ((k[at + DIR * d] ^ mine) >> shift) == 0; };
  int in = 0, out = 1;
  while (out <= RUN_MAX && same(out)) {
    in = out;
    out *= 2;
  }
  out = min(out, RUN_MAX + 2);
  while (out - in > 1) {
    const int mid = (in + out) / 2;
    if (same(mid)) in = mid;
    else out = mid;
  }
  return in;
}

__global__ void __launch_bounds__(FIX_THREADS) k_fix_runs(const uint64_t* __restrict__ keys,
                                                          const uint32_t* __restrict__ vin, uint64_t n, int shift,
                                                          uint32_t* __restrict__ vout, uint32_t* __restrict__ flag) {
  constexpr int SPAN = FIX_TILE + 2 * RUN_MAX + 2, LOADS = (SPAN + FIX_THREADS - 1) / FIX_THREADS;
  __shared__ uint64_t k[LOADS * FIX_THREADS];
  const int64_t base = (int64_t)blockIdx.x * FIX_TILE, lo = base - RUN_MAX - 1;  // k[0] is element lo
  // all loads in flight before the first is used
  uint64_t key[LOADS];
  uint32_t val[FIX_ITEMS];
#pragma unroll
  for (int l = 0; l < LOADS; ++l) {
    const int64_t i = lo + l * FIX_THREADS + threadIdx.x;
    key[l] = i >= 0 && i < (int64_t)n ? keys[i] : ~0ull;  // ~0 agrees with no 63-bit key
  }
#pragma unroll
  for (int it = 0; it < FIX_ITEMS; ++it) {
    const int64_t i = base + it * FIX_THREADS + threadIdx.x;
    val[it] = i < (int64_t)n ? vin[i] : 0u;
  }
#pragma unroll
  for (int l = 0; l < LOADS; ++l) k[l * FIX_THREADS + threadIdx.x] = key[l];
  __syncthreads();
  bool unsorted = false;
#pragma unroll
  for (int it = 0; it < FIX_ITEMS; ++it) {
    const int64_t i = base + it * FIX_THREADS + threadIdx.x;
    if (i >= (int64_t)n) break;
    const int at = (int)(i - lo);
    const uint64_t mine = k[at];
    const int left = run_side<-1>(k, at, mine, shift), right = run_side<1>(k, at, mine, shift);
    int move = 0;
    if (left + right > RUN_MAX) {
      unsorted |= right > 0 && k[at + 1] < mine;
    } else {
#pragma unroll 4
      for (int j = 1; j <= left; ++j) move -= k[at - j] > mine ? 1 : 0;
#pragma unroll 4
      for (int j = 1; j <= right; ++j) move += k[at + j] < mine ? 1 : 0;
    }
    vout[i + move] = val[it];
  }
  raise(flag, unsorted);
}

// ----------------------------------------------------------------- gather
// The kernels after the sort do nothing where it has raised its flag (unsorted):
// the keys, the order so far and the input stay for the second sort, and the
// host need not wait for the flag before it enqueues them.

// Positions and colours of the input as one 16-byte record per point, in
// input order: the gather then reads one record (one cache line) per output
// instead of a position and a colour from two arrays.
__global__ void __launch_bounds__(256) k_interleave(const float* __restrict__ xyz, const uint32_t* __restrict__ rgba,
                                                    uint64_t n, uint4* __restrict__ rec,
                                                    const uint32_t* __restrict__ unsorted) {
  if (*unsorted) return;
  const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride)
    rec[i] = make_uint4(__float_as_uint(xyz[3 * i]), __float_as_uint(xyz[3 * i + 1]), __float_as_uint(xyz[3 * i + 2]),
                        rgba[i]);
}

// The batches of a spread build: each batch of c points is stored in the
// order position r <- Morton rank (r * m) mod c (m: step for a full batch,
// m_last for the last batch when it is shorter).
struct Spread {
  uint64_t S, m, c_last, m_last;
};
__device__ __forceinline__ uint64_t spread_source(uint64_t i, const Spread& sp, uint64_t n) {
  const uint64_t b0 = i - i % sp.S;
  const bool full = b0 + sp.S <= n;
  const uint64_t c = full ? sp.S : sp.c_last, m = full ? sp.m : sp.m_last;
  return b0 + ((i - b0) * m) % c;
}

// Four consecutive outputs per thread: one 16-byte load of their sources, the
// four record reads in flight together, 48 + 16 contiguous bytes written.
// The outputs past the last multiple of four go one per thread.  SPREAD: the
// sources come from the Morton positions of the spread order.  perm_out
// receives the sources.
template <bool SPREAD>
__global__ void __launch_bounds__(256) k_gather(const uint4* __restrict__ rec, const uint32_t* __restrict__ perm,
                                                uint32_t* __restrict__ perm_out, Spread sp, uint64_t n,
                                                float* __restrict__ xyz_out, uint32_t* __restrict__ colors,
                                                const uint32_t* __restrict__ unsorted) {
  if (*unsorted) return;
  const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
  const uint64_t n4 = n / 4;
  for (uint64_t g = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; g < n4; g += stride) {
    uint64_t s[4];
    if constexpr (SPREAD) {
      uint32_t q[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const uint64_t src = spread_source(4 * g + j, sp, n);
        q[j] = perm[src < n ? src : 4 * g + j];
        s[j] = q[j];
      }
      reinterpret_cast<uint4*>(perm_out)[g] = make_uint4(q[0], q[1], q[2], q[3]);
    } else {
      const uint4 p = reinterpret_cast<const uint4*>(perm)[g];
      s[0] = p.x;
      s[1] = p.y;
      s[2] = p.z;
      s[3] = p.w;
      reinterpret_cast<uint4*>(perm_out)[g] = p;
    }
    uint4 r[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      if (s[j] >= n) s[j] = 4 * g + j;  // a permutation never triggers this; it keeps reads in bounds
      r[j] = rec[s[j]];
    }
    float4* const xo = reinterpret_cast<float4*>(xyz_out + 12 * g);
    xo[0] = make_float4(__uint_as_float(r[0].x), __uint_as_float(r[0].y), __uint_as_float(r[0].z), __uint_as_float(r[1].x));
    xo[1] = make_float4(__uint_as_float(r[1].y), __uint_as_float(r[1].z), __uint_as_float(r[2].x), __uint_as_float(r[2].y));
    xo[2] = make_float4(__uint_as_float(r[2].z), __uint_as_float(r[3].x), __uint_as_float(r[3].y), __uint_as_float(r[3].z));
    reinterpret_cast<uint4*>(colors)[g] = make_uint4(r[0].w, r[1].w, r[2].w, r[3].w);
  }
  for (uint64_t i = 4 * n4 + (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
    uint64_t s;
    if constexpr (SPREAD) {
      const uint64_t src = spread_source(i, sp, n);
      s = perm[src < n ? src : i];
    } else {
      s = perm[i];
    }
    perm_out[i] = (uint32_t)s;
    if (s >= n) s = i;
    const uint4 r = rec[s];
    xyz_out[3 * i] = __uint_as_float(r.x);
    xyz_out[3 * i + 1] = __uint_as_float(r.y);
    xyz_out[3 * i + 2] = __uint_as_float(r.z);
    colors[i] = r.w;
  }
}

// ------------------------------------------------------------ batch boxes
// One block per batch: batch b is [b S, min((b + 1) S, n)), or, with spans,
// [out[b].first, out[b].first + out[b].count) as set by the host.  unsorted: as
// above, or null.
__global__ void __launch_bounds__(256) k_batch_bbox(const float* __restrict__ xyz, uint64_t n, uint32_t S,
                                                    BatchRec* __restrict__ out, int spans,
                                                    const uint32_t* __restrict__ unsorted) {
  if (unsorted && *unsorted) return;
  const uint64_t first = spans ? out[blockIdx.x].first : (uint64_t)blockIdx.x * S;
  const uint64_t end = spans ? first + out[blockIdx.x].count : (first + S < n ? first + S : n);
  uint32_t mn[3] = {0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu}, mx[3] = {0, 0, 0};
  for (uint64_t i = first + threadIdx.x; i < end; i += 256) {
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      const uint32_t k = okey(xyz[3 * i + a]);
      mn[a] = min(mn[a], k);
      mx[a] = max(mx[a], k);
    }
  }
  __shared__ uint32_t red[4][6];
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    for (int o = 32; o > 0; o >>= 1) {
      mn[a] = min(mn[a], (uint32_t)__shfl_xor((int)mn[a], o));
      mx[a] = max(mx[a], (uint32_t)__shfl_xor((int)mx[a], o));
    }
  }
  const int wave = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) {
    for (int a = 0; a < 3; ++a) {
      red[wave][a] = mn[a];
      red[wave][3 + a] = mx[a];
    }
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    BatchRec r;
    r.first = (uint32_t)first;
    r.count = (uint32_t)(end - first);
    for (int a = 0; a < 3; ++a) {
      uint32_t lo = red[0][a], hi = red[0][3 + a];
      for (int w = 1; w < 4; ++w) {
        lo = min(lo, red[w][a]);
        hi = max(hi, red[w][3 + a]);
      }
      r.mn[a] = okey_inv(lo);
      r.mx[a] = okey_inv(hi);
    }
    out[blockIdx.x] = r;
  }
}

// --------------------------------------------------------------- quantise
// Eq. 1: X30 = min(floor(2^30 (x - min) / size), 2^30 - 1) in binary64 with
// one correctly rounded division (0 for size 0); low = bits 29..20, med =
// bits 19..10, high = bits 9..0, each packed x | y << 10 | z << 20.
constexpr double EQ1_SCALE = 1073741824.0;
struct Words3 {
  uint32_t low, med, high;
};
__device__ __forceinline__ Words3 eq1(const Axis (&ax)[3], float x, float y, float z) {
  const float f[3] = {x, y, z};
  Words3 w = {0, 0, 0};
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    const uint32_t X30 = axis_cell(ax[a], f[a], EQ1_SCALE);
    w.low |= ((X30 >> 20) & 1023u) << (10 * a);
    w.med |= ((X30 >> 10) & 1023u) << (10 * a);
    w.high |= (X30 & 1023u) << (10 * a);
  }
  return w;
}

__global__ void __launch_bounds__(256) k_quantize(const float* __restrict__ xyz, uint64_t n, uint32_t S,
                                                  const BatchRec* __restrict__ batches, uint32_t* __restrict__ low,
                                                  uint32_t* __restrict__ med, uint32_t* __restrict__ high,
                                                  const uint32_t* __restrict__ unsorted) {
  if (unsorted && *unsorted) return;
  const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
    const BatchRec& B = batches[(uint32_t)i / S];  // i < 2^32
    Axis ax[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) ax[a] = make_axis(B.mn[a], B.mx[a], EQ1_SCALE);
    const Words3 w = eq1(ax, xyz[3 * i], xyz[3 * i + 1], xyz[3 * i + 2]);
    low[i] = w.low;
    med[i] = w.med;
    high[i] = w.high;
  }
}

// Variable-size batches: one block per batch, Eq. 1 relative to its box.
__global__ void __launch_bounds__(256) k_quantize_spans(const float* __restrict__ xyz,
                                                        const BatchRec* __restrict__ batches,
                                                        uint32_t* __restrict__ low, uint32_t* __restrict__ med,
                                                        uint32_t* __restrict__ high) {
  const BatchRec B = batches[blockIdx.x];
  Axis ax[3];
#pragma unroll
  for (int a = 0; a < 3; ++a) ax[a] = make_axis(B.mn[a], B.mx[a], EQ1_SCALE);
  for (uint64_t i = (uint64_t)B.first + threadIdx.x; i < (uint64_t)B.first + B.count; i += 256) {
    const Words3 w = eq1(ax, xyz[3 * i], xyz[3 * i + 1], xyz[3 * i + 2]);
    low[i] = w.low;
    med[i] = w.med;
    high[i] = w.high;
  }
}

// ------------------------------------------------------------ whole batches
// One batch per workgroup, its points in registers from the first read to the
// last word: source (ORDER 0: the input itself, with the finite check; 1 and 2:
// records gathered through the sorted order, 2 in the spread order) -> position,
// colour and permutation -> box -> Eq. 1 words.  Against a gather, a box pass and
// a word pass of their own it saves reading the positions twice more, and the
// box and division work hides behind the gather's scattered reads (5e8 points in
// no order: 16.3 ms, as the gather alone took, instead of 16.2 + 0.8 + 0.95 + 4.3
// with its copy of the order; each record is a line of its own there, 64 GB of
// lines; all steps' reads issued up front gained nothing).  Each thread owns
// groups of four consecutive points, so that every buffer is written in 16-byte
// words.
constexpr int WB_STEPS = 5;  // groups of four points per thread
template <int ORDER, int THREADS>
__global__ void __launch_bounds__(THREADS) __attribute__((amdgpu_waves_per_eu(4)))
k_batch(const float* __restrict__ xyz, const uint32_t* __restrict__ rgba, const uint4* __restrict__ rec,
        const uint32_t* __restrict__ order, Spread sp, uint64_t n, uint32_t S, float* __restrict__ xyz_out,
        uint32_t* __restrict__ colors, uint32_t* __restrict__ perm, BatchRec* __restrict__ batches,
        uint32_t* __restrict__ low, uint32_t* __restrict__ med, uint32_t* __restrict__ high,
        uint32_t* __restrict__ nonfinite, const uint32_t* __restrict__ unsorted) {
  __shared__ Box red[THREADS / 64];
  const uint64_t batch = xcd_tile(), first = batch * S;
  if (first >= n) return;
  if constexpr (ORDER != 0) {
    if (*unsorted) return;
  }
  const uint32_t count = (uint32_t)(first + S <= n ? S : n - first);
  const uint32_t step = (uint32_t)(count == S ? sp.m : sp.m_last);
  float p[WB_STEPS][12];
  Box box = empty_box();
  bool bad = false;
#pragma unroll
  for (int k = 0; k < WB_STEPS; ++k) {
    const uint32_t r = 4u * (k * THREADS + threadIdx.x);
    if (r >= count) break;
    const uint64_t i = first + r;
    const uint32_t m = min(4u, count - r);
    uint32_t src[4], col[4];
    if constexpr (ORDER == 0) {
      if (m == 4) {
        const float4* const v = reinterpret_cast<const float4*>(xyz + 3 * i);
        const float4 u0 = v[0], u1 = v[1], u2 = v[2];
        const uint4 c = *reinterpret_cast<const uint4*>(rgba + i);
        const float f[12] = {u0.x, u0.y, u0.z, u0.w, u1.x, u1.y, u1.z, u1.w, u2.x, u2.y, u2.z, u2.w};
#pragma unroll
        for (int j = 0; j < 12; ++j) p[k][j] = f[j];
        col[0] = c.x, col[1] = c.y, col[2] = c.z, col[3] = c.w;
#pragma unroll
        for (int j = 0; j < 4; ++j) src[j] = (uint32_t)i + j;
      } else {
#pragma unroll
        for (int j = 0; j < 4; ++j) {  // past the end the last point again
          src[j] = (uint32_t)i + min((uint32_t)j, m - 1u);
#pragma unroll
          for (int a = 0; a < 3; ++a) p[k][3 * j + a] = xyz[3 * (uint64_t)src[j] + a];
          col[j] = rgba[src[j]];
        }
      }
#pragma unroll
      for (int j = 0; j < 12; ++j) bad |= not_finite(p[k][j]);
    } else {
      if constexpr (ORDER == 2) {
        uint32_t o = (r * step) % count;  // rank of position r; r step < 2^32 for batches of 20,480 points
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          src[j] = order[first + o];
          o += step;
          if (o >= count) o -= count;
        }
      } else {
#pragma unroll
        for (int j = 0; j < 4; ++j) src[j] = order[i + min((uint32_t)j, m - 1u)];
      }
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        if (src[j] >= n) src[j] = (uint32_t)i;  // a permutation never triggers this; it keeps reads in bounds
        const uint4 q = rec[src[j]];
        p[k][3 * j] = __uint_as_float(q.x);
        p[k][3 * j + 1] = __uint_as_float(q.y);
        p[k][3 * j + 2] = __uint_as_float(q.z);
        col[j] = q.w;
      }
      if (m == 4) {
        float4* const x = reinterpret_cast<float4*>(xyz_out + 3 * i);
        x[0] = make_float4(p[k][0], p[k][1], p[k][2], p[k][3]);
        x[1] = make_float4(p[k][4], p[k][5], p[k][6], p[k][7]);
        x[2] = make_float4(p[k][8], p[k][9], p[k][10], p[k][11]);
      }
    }
    if (m == 4) {
      *reinterpret_cast<uint4*>(colors + i) = make_uint4(col[0], col[1], col[2], col[3]);
      *reinterpret_cast<uint4*>(perm + i) = make_uint4(src[0], src[1], src[2], src[3]);
    } else {
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        if ((uint32_t)j < m) {
          if constexpr (ORDER != 0) {
#pragma unroll
            for (int a = 0; a < 3; ++a) xyz_out[3 * (i + j) + a] = p[k][3 * j + a];
          }
          colors[i + j] = col[j];
          perm[i + j] = src[j];
        }
      }
    }
#pragma unroll
    for (int j = 0; j < 12; ++j) grow(box, j % 3, p[k][j]);
  }
  if constexpr (ORDER == 0) raise(nonfinite, bad);
  box = block_box(box, red);
  Axis ax[3];
#pragma unroll
  for (int a = 0; a < 3; ++a) ax[a] = make_axis(okey_inv(box.mn[a]), okey_inv(box.mx[a]), EQ1_SCALE);
  if (threadIdx.x == 0) {
    BatchRec b;
    b.first = (uint32_t)first;
    b.count = count;
    for (int a = 0; a < 3; ++a) {
      b.mn[a] = okey_inv(box.mn[a]);
      b.mx[a] = okey_inv(box.mx[a]);
    }
    batches[batch] = b;
  }
#pragma unroll
  for (int k = 0; k < WB_STEPS; ++k) {
    const uint32_t r = 4u * (k * THREADS + threadIdx.x);
    if (r >= count) break;
    const uint64_t i = first + r;
    Words3 w[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) w[j] = eq1(ax, p[k][3 * j], p[k][3 * j + 1], p[k][3 * j + 2]);
    if (r + 4 <= count) {
      *reinterpret_cast<uint4*>(low + i) = make_uint4(w[0].low, w[1].low, w[2].low, w[3].low);
      *reinterpret_cast<uint4*>(med + i) = make_uint4(w[0].med, w[1].med, w[2].med, w[3].med);
      *reinterpret_cast<uint4*>(high + i) = make_uint4(w[0].high, w[1].high, w[2].high, w[3].high);
    } else {
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        if (r + j < count) {
          low[i + j] = w[j].low;
          med[i + j] = w[j].med;
          high[i + j] = w[j].high;
        }
      }
    }
  }
}

inline uint32_t grid_for(uint64_t work, uint32_t per_block = 256, uint32_t cap = 65536) {
  uint64_t b = (work + per_block - 1) / per_block;
  if (b < 1) b = 1;
  if (b > cap) b = cap;
  return (uint32_t)b;
}

inline uint64_t align256(uint64_t x) { return (x + 255) & ~255ull; }

}  // namespace

uint64_t small_scratch_bytes() { return 4096; }

uint64_t sort_scratch_bytes(uint64_t n) {
  const uint64_t tiles = n ? (n + 4095) / 4096 : 1, m = 256 * tiles;
  return 256 + 2 * align256(8 * n) + align256(4 * n) + align256(4 * m) + align256(4 * ((m + 4095) / 4096));
}

// The sort area starts 1 KiB before the end of the small scratch, whose first
// 256 bytes hold the cloud box: with tiles of 8,192 points and 512 digits the
// histograms take at most 1 KiB more than sort_scratch_bytes counts for them.
void sort_scratch_layout(uint64_t n, uint8_t* scratch, SortScratch* out) {
  SortScratch s{};
  s.nblk = (n + RS_TILE - 1) / RS_TILE;
  if (s.nblk == 0) s.nblk = 1;
  const uint64_t m = RS_DIGITS * s.nblk;
  s.npart = (m + SCAN_CHUNK - 1) / SCAN_CHUNK;
  s.aabb = reinterpret_cast<uint32_t*>(scratch);
  uint64_t off = small_scratch_bytes() - 1024;
  auto take = [&](uint64_t bytes) {
    uint8_t* const p = scratch + off;
    off += align256(bytes);
    return p;
  };
  s.keys0 = reinterpret_cast<uint64_t*>(take(8 * n));
  s.keys1 = reinterpret_cast<uint64_t*>(take(8 * n));
  s.vals1 = reinterpret_cast<uint32_t*>(take(4 * n));
  s.hist = reinterpret_cast<uint32_t*>(take(4 * m));
  s.part = reinterpret_cast<uint32_t*>(take(4 * s.npart));
  s.end = off;
  *out = s;
}

hipError_t launch_finite_check(const float* xyz, uint64_t n, uint32_t* flag, hipStream_t s) {
  hipLaunchKernelGGL(k_finite, dim3(grid_for(3 * n, 256 * 8)), dim3(256), 0, s,
                     reinterpret_cast<const uint32_t*>(xyz), 3 * n, flag);
  return hipGetLastError();
}

hipError_t launch_iota(uint32_t* p, uint64_t n, hipStream_t s) {
  hipLaunchKernelGGL(k_iota, dim3(grid_for(n, 256 * 4)), dim3(256), 0, s, p, n);
  return hipGetLastError();
}

// Radix passes over the leading bits before the runs are ordered: enough that
// a surface, which fills about 4^levels of the cells, leaves some 16 points a
// run at most (5e8 points: 4 passes, 30 a run, 50.5 ms; 5 passes, 45.7 ms).
int sort_passes(uint64_t n) {
  int passes = 2;
  while (passes < 5 && (n >> (2 * 3 * passes)) > 16) ++passes;  // 9 bits: 3 levels
  return passes;
}

namespace {
constexpr int FULL_PASSES = KEY_BITS / RS_BITS;  // every bit of the key
static_assert(FULL_PASSES * RS_BITS == KEY_BITS, "whole passes");

// Passes over the digits from bit 63 - 9 passes up, of the keys in kin and the values in vin (null: the indices, and
// the first digit's histogram is counted already).  The values end in vals_last, the keys in kin or the other buffer.
hipError_t radix_passes(const SortScratch& sc, uint64_t n, int passes, uint64_t* kin, const uint32_t* vin,
                        uint32_t* vals_last, uint32_t* vals_other, hipStream_t s) {
  const uint64_t m = RS_DIGITS * sc.nblk;
  for (int p = 0; p < passes; ++p) {
    const int shift = KEY_BITS - RS_BITS * (passes - p);
    uint64_t* const kout = kin == sc.keys0 ? sc.keys1 : sc.keys0;
    uint32_t* const vout = (passes - 1 - p) % 2 ? vals_other : vals_last;
    if (vin)
      hipLaunchKernelGGL(k_radix_count, dim3((uint32_t)sc.nblk), dim3(RS_THREADS), 0, s, kin, n, shift, sc.hist, sc.nblk);
    if (m <= SCAN_SMALL) {
      hipLaunchKernelGGL(k_scan_small, dim3(1), dim3(SS_THREADS), 0, s, sc.hist, m);
    } else {
      hipLaunchKernelGGL(k_scan_partials, dim3((uint32_t)sc.npart), dim3(256), 0, s, sc.hist, m, sc.part);
      hipLaunchKernelGGL(k_scan_top, dim3(1), dim3(256), 0, s, sc.part, sc.npart);
      hipLaunchKernelGGL(k_scan_apply, dim3((uint32_t)sc.npart), dim3(256), 0, s, sc.hist, m, sc.part);
    }
    hipLaunchKernelGGL(k_radix_scatter, dim3(xcd_grid(sc.nblk)), dim3(RS_THREADS), 0, s, kin, vin, kout, vout, n, shift,
                       sc.hist, sc.nblk);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    kin = kout;
    vin = vout;
  }
  return hipSuccess;
}

// Where the passes of the first sort leave its keys.
uint64_t* sorted_keys(const SortScratch& sc, uint64_t n) { return sort_passes(n) % 2 ? sc.keys1 : sc.keys0; }
}  // namespace

hipError_t launch_morton_sort(const SortScratch& sc, const float* xyz, uint32_t* perm, uint64_t n, uint32_t* nonfinite,
                              uint32_t* unsorted, hipStream_t s) {
  if (n == 0) return hipSuccess;
  // the partial boxes lie in the second key buffer, not in use yet (24 bytes per 1,024 points, or one in 256)
  Box* const part = reinterpret_cast<Box*>(sc.keys1);
  const uint32_t blocks = grid_for(n, 1024, BOX_BLOCKS);
  hipLaunchKernelGGL(k_aabb, dim3(blocks), dim3(256), 0, s, xyz, n, part, nonfinite);
  hipLaunchKernelGGL(k_aabb_top, dim3(1), dim3(256), 0, s, part, blocks, sc.aabb);
  const int passes = sort_passes(n), shift = KEY_BITS - RS_BITS * passes;
  hipLaunchKernelGGL(k_morton, dim3((uint32_t)sc.nblk), dim3(RS_THREADS), 0, s, xyz, n, sc.aabb, sc.keys0, shift,
                     sc.hist, sc.nblk);
  const hipError_t e = radix_passes(sc, n, passes, sc.keys0, nullptr, perm, sc.vals1, s);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_fix_runs, dim3((uint32_t)((n + FIX_TILE - 1) / FIX_TILE)), dim3(FIX_THREADS), 0, s,
                     sorted_keys(sc, n), perm, n, shift, sc.vals1, unsorted);
  return hipGetLastError();
}

hipError_t launch_morton_resort(const SortScratch& sc, uint32_t* perm, uint64_t n, hipStream_t s) {
  return radix_passes(sc, n, FULL_PASSES, sorted_keys(sc, n), perm, sc.vals1, perm, s);
}

uint64_t spread_step(uint64_t c) {
  uint64_t m = c / 4 + 1;
  for (;;) {
    uint64_t a = m, b = c;
    while (b) {
      const uint64_t t = a % b;
      a = b;
      b = t;
    }
    if (a == 1) return m;
    ++m;
  }
}

namespace {
Spread make_spread(uint64_t n, uint32_t S) {
  Spread sp;
  sp.S = S;
  sp.m = spread_step(S);
  sp.c_last = n % S ? n % S : S;
  sp.m_last = spread_step(sp.c_last);
  return sp;
}

template <int ORDER, int THREADS>
hipError_t launch_batch_t(const BuildArgs& a, const uint4* rec, const uint32_t* order, hipStream_t s) {
  const uint64_t nb = (a.n + a.S - 1) / a.S;
  hipLaunchKernelGGL((k_batch<ORDER, THREADS>), dim3(xcd_grid(nb)), dim3(THREADS), 0, s, a.xyz, a.rgba, rec, order,
                     ORDER == 2 ? make_spread(a.n, a.S) : Spread{}, a.n, a.S, a.xyz, a.colors, a.perm, a.batches, a.low,
                     a.med, a.high, a.nonfinite, a.unsorted);
  return hipGetLastError();
}
template <int ORDER>
hipError_t launch_batch(const BuildArgs& a, const uint4* rec, const uint32_t* order, hipStream_t s) {
  if (a.S <= 256u * 4 * WB_STEPS) return launch_batch_t<ORDER, 256>(a, rec, order, s);
  if (a.S <= 512u * 4 * WB_STEPS) return launch_batch_t<ORDER, 512>(a, rec, order, s);
  return launch_batch_t<ORDER, 1024>(a, rec, order, s);
}
// Batches that one workgroup of k_batch holds in registers (20 points a thread)
// and that fill at least two of its waves; larger and smaller ones take the separate
// kernels (2e7 points in their order, whole builds: 508 points a batch 447 us, 512 359, 1,024
// 304, 20,480 328, 20,484 450; sorted: 1.77, 1.63, 1.64, 1.68, 1.77 ms).
bool whole_batches(uint32_t S) { return S >= 512 && S <= 1024u * 4 * WB_STEPS; }

hipError_t boxes_and_words(const BuildArgs& a, const uint32_t* unsorted, hipStream_t s) {
  const uint64_t nb = (a.n + a.S - 1) / a.S;
  hipLaunchKernelGGL(k_batch_bbox, dim3((uint32_t)nb), dim3(256), 0, s, a.xyz, a.n, a.S, a.batches, 0, unsorted);
  hipLaunchKernelGGL(k_quantize, dim3(grid_for(a.n, 256 * 4)), dim3(256), 0, s, a.xyz, a.n, a.S, a.batches, a.low, a.med,
                     a.high, unsorted);
  return hipGetLastError();
}
}  // namespace

hipError_t launch_build_input(const BuildArgs& a, hipStream_t s) {
  if (a.n == 0) return hipSuccess;
  if (whole_batches(a.S)) return launch_batch<0>(a, nullptr, nullptr, s);
  hipError_t e = launch_finite_check(a.xyz, a.n, a.nonfinite, s);
  if (e == hipSuccess) e = launch_iota(a.perm, a.n, s);
  if (e == hipSuccess) e = hipMemcpyAsync(a.colors, a.rgba, 4 * a.n, hipMemcpyDeviceToDevice, s);
  return e == hipSuccess ? boxes_and_words(a, nullptr, s) : e;
}

hipError_t launch_build_sorted(const BuildArgs& a, const SortScratch& sc, bool spread, hipStream_t s) {
  if (a.n == 0) return hipSuccess;
  // the records take the two key buffers, free once the sort is done (keys0 then keys1: 16 n bytes)
  uint4* const rec = reinterpret_cast<uint4*>(sc.keys0);
  if (reinterpret_cast<uint8_t*>(sc.keys1) + 8 * a.n < reinterpret_cast<uint8_t*>(rec) + 16 * a.n) return hipErrorInvalidValue;
  const dim3 grid(grid_for(a.n, 256 * 4));
  hipLaunchKernelGGL(k_interleave, grid, dim3(256), 0, s, a.xyz, a.rgba, a.n, rec, a.unsorted);
  if (whole_batches(a.S)) return spread ? launch_batch<2>(a, rec, sc.vals1, s) : launch_batch<1>(a, rec, sc.vals1, s);
  if (spread)
    hipLaunchKernelGGL(k_gather<true>, grid, dim3(256), 0, s, rec, sc.vals1, a.perm, make_spread(a.n, a.S), a.n, a.xyz,
                       a.colors, a.unsorted);
  else
    hipLaunchKernelGGL(k_gather<false>, grid, dim3(256), 0, s, rec, sc.vals1, a.perm, Spread{}, a.n, a.xyz, a.colors,
                       a.unsorted);
  return boxes_and_words(a, a.unsorted, s);
}

hipError_t launch_batch_bbox_spans(const float* xyz, uint64_t nb, BatchRec* recs, hipStream_t s) {
  if (nb == 0) return hipSuccess;
  hipLaunchKernelGGL(k_batch_bbox, dim3((uint32_t)nb), dim3(256), 0, s, xyz, (uint64_t)0, 0u, recs, 1,
                     (const uint32_t*)nullptr);
  return hipGetLastError();
}

hipError_t launch_quantize_spans(const float* xyz, uint64_t nb, const BatchRec* recs, uint32_t* low, uint32_t* med,
                                 uint32_t* high, hipStream_t s) {
  if (nb == 0) return hipSuccess;
  hipLaunchKernelGGL(k_quantize_spans, dim3((uint32_t)nb), dim3(256), 0, s, xyz, recs, low, med, high);
  return hipGetLastError();
}

}  // namespace ptr
