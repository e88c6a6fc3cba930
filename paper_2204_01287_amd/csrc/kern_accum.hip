// High-quality shading pass (Sec. 3.6) for gfx950: the sums of the colours of
// the points near each pixel's closest depth, and their average.
//
// What bounds it: the device's atomics where batches add straight into global
// sums (25 G 64-byte lines/s), and the latency chain of a batch (record,
// thresholds, words, flush) with two workgroups per CU.  At 5e8 points, one
// 2016x2240 eye of 1.4e4 live batches: 495 us with both words of a pixel in
// instructions of their own, a point's threshold read and addition before the
// next point's, and sums and thresholds staged before the words were asked
// for; 480 with one instruction per pixel in the flush; 385 with the same for
// the untiled batches (6 % of the points); 370 as it stands.  Smaller
// workgroups with smaller tiles (4 or 5 waves, 2032 pixels: 435 and 445 us)
// and larger ones (10 or 16 waves: 525 and 490) are slower.
//
// Its own translation unit: the pass runs eight-wave workgroups (two per CU,
// each with an 80 KiB LDS tile of thresholds and sums) over the point loops
// of raster_core.h.
#define PR_WAVES 8
#include "raster_core.h"

namespace ptr {
namespace {

// ------------------------------------------------------------------ shading
// High-quality shading (Sec. 3.6), second pass over the live batches of the
// frame's render: every drawn point within the depth window of its pixel
// adds its colour and a count.  Tiled batches whose rectangle fits HQS_TILE
// pixels stage the thresholds of the rectangle in LDS, add into LDS sums and
// flush each covered pixel with two global additions; the others read the
// visibility buffer and add globally per point.  Integer sums: the result
// does not depend on the order of the additions.

// Row of entry e of a rectangle of tw columns, m = row_magic(tw): exact while
// e * tw < 2^32.
__device__ __forceinline__ uint32_t row_magic(uint32_t tw) { return 0xFFFFFFFFu / tw + 1u; }  // 0 for one column
__device__ __forceinline__ uint32_t row_of(uint32_t e, uint32_t m) { return m ? __umulhi(e, m) : e; }

// Thresholds fl32(closest depth * window) of a tw x th rectangle at (x0, y0)
// into the LDS tile, four reads of a thread in flight.
__device__ __forceinline__ void stage_band(const RenderArgs& a, float* thr, uint32_t tid, uint32_t x0, uint32_t y0,
                                           uint32_t tw, uint32_t th) {
  const uint32_t n = tw * th, m = row_magic(tw);
  const uint32_t* const depth = reinterpret_cast<const uint32_t*>(a.vb + ((uint64_t)y0 * a.W + x0)) + 1;
  for (uint32_t b = tid; b < n; b += 4 * THREADS) {
    uint32_t d[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const uint32_t e = min(b + j * THREADS, n - 1u), ly = row_of(e, m);
      d[j] = depth[2 * (uint64_t)(ly * a.W + (e - ly * tw))];
    }
#pragma unroll
    for (int j = 0; j < 4; ++j)
      if (b + j * THREADS < n) thr[b + j * THREADS] = __uint_as_float(d[j]) * a.window;
  }
}

// Every pixel of the rectangle with a point in its sums: two global additions,
// by neighbouring lanes; the sums are left zero for the next batch.  The
// device's atomics cost by the 64-byte line of an instruction (25 G lines/s),
// so the two words of a pixel go into one.
__device__ __forceinline__ void flush_band(const RenderArgs& a, uint64_t* sums, uint32_t tid, uint32_t x0, uint32_t y0,
                                           uint32_t tw, uint32_t th) {
  const uint32_t n = tw * th, m = row_magic(tw), half = tid & 1u;
  uint64_t* const base = a.accum + 2 * ((uint64_t)y0 * a.W + x0) + half;
  for (uint32_t e = tid >> 1; e < n; e += THREADS / 2) {
    const uint64_t bn = sums[HQS_TILE + e];
    if (bn >> 32) {
      const uint64_t v = half ? bn : sums[e];
      sums[half * HQS_TILE + e] = 0;  // after both lanes' reads: they are lanes of one wave
      const uint32_t ly = row_of(e, m);
      __hip_atomic_fetch_add(base + 2 * (uint64_t)(ly * a.W + (e - ly * tw)), v, __ATOMIC_RELAXED,
                             __HIP_MEMORY_SCOPE_AGENT);
    }
  }
}

__global__ void __launch_bounds__(THREADS) k_accum(RenderArgs a) {
  __shared__ float thr[HQS_TILE];
  __shared__ uint64_t sums[2 * HQS_TILE];
  __shared__ uint32_t s_next;
  const uint32_t tid = threadIdx.x, wave = uni(tid >> 6), lane = tid & 63;
  const uint32_t q = blockIdx.x % RENDER_QUEUES;
  uint32_t* const qc = &a.hdr->queue[q][0];
  // batch order (Morton order for sorted clouds): the sums' lines of neighbouring
  // batches stay in the caches; measured faster than the render's order here
  const uint32_t nlive = a.hdr->live_count + a.hdr->direct_count;
  const Cut cut = cut_of(nlive);
  for (uint32_t e = tid; e < 2 * HQS_TILE; e += THREADS) sums[e] = 0;
  const Streams st = {a.low, a.med, a.high, a.colors};
  __syncthreads();
  uint32_t item, slice;
  cut.at(first_position(cut, qc, q, &s_next), item, slice);
  uint32_t natom = 0;
  while (item < nlive) {
    uint32_t grab = 0;
    if (tid == 0) grab = next_position(cut, qc, q);
    const LiveBatch& rec = a.live[uni(a.order[item])];
    Loop L;
#pragma unroll
    for (int r = 0; r < 3; ++r) {
#pragma unroll
      for (int j = 0; j < 3; ++j) L.P[r][j] = rec.P[r][j];
      L.t[r] = rec.t[r];
    }
    L.W = a.W;
    L.H = a.H;
    L.vb = a.vb;
    L.window = a.window;
    L.acc = a.accum;
    L.thr = thr;
    const uint32_t mode = rec.mode, rxy = rec.rect_xy, rwh = rec.rect_wh;
    Span b = {rec.first, rec.count};
    const uint32_t x0 = rxy & 0xFFFFu, y0 = rxy >> 16;
    L.tw = rwh & 0xFFFFu;
    L.th = rwh >> 16;
    L.tw8 = L.tw * 8u;
    const int k = (int)(mode & 0xFFu), cls = (int)((mode >> 8) & 0xFFu);
    const uint32_t n = L.tw * L.th;
    const bool tiled = ((mode >> 16) & 1u) && n <= HQS_TILE;
    // 10-bit batches with a proven rectangle too large for the tile but at most
    // one tile wide: band by band (stage the band's thresholds, add, flush)
    const bool banded = !tiled && k == 10 && ((mode >> 16) & 3u) && L.tw <= HQS_TILE;
    if (banded) {
      const uint32_t bh = HQS_TILE / L.tw;
      uint32_t by0 = 0, by1 = L.th;
      if (cut.shift) {
        b = banded_part({uni(b.first), uni(b.count)}, uni(L.tw), uni(L.th), bh, slice, cut, by0, by1);
        if (b.count == 0) {  // nothing in this slice
          by0 = 0;
          by1 = 1;
        }
      }
      const uint32_t first = b.first, count = b.count;
      L.cx = in_vgpr(uni(0x4B000000u + x0));
      for (uint32_t by = by0; by < by1; by += bh) {
        L.th = min(bh, by1 - by);
        L.cy = in_vgpr(uni(0x4B000000u + y0 + by));
        raster_by_class<10, true, true, true>(cls, L, st, sums, first, count, wave, lane, natom, [&] {
          stage_band(a, thr, tid, x0, y0 + by, L.tw, L.th);
          __syncthreads();
        });
        __syncthreads();  // the band's sums are complete; s_next has been read
        if (by == by0 && tid == 0) s_next = grab;
        flush_band(a, sums, tid, x0, y0 + by, L.tw, L.th);
        __syncthreads();  // tile free again
      }
      cut.at(uni(s_next), item, slice);
      continue;
    }
    if (cut.shift) {
      b = {uni(b.first), uni(b.count)};
      b = tiled ? tiled_part(b, uni(n), slice, cut.shift) : points_part(b, slice, 1u << cut.shift);
    }
    const uint32_t first = b.first, count = b.count;
    L.cx = in_vgpr(uni(0x4B000000u + (tiled ? x0 : 0u)));
    L.cy = in_vgpr(uni(0x4B000000u + (tiled ? y0 : 0u)));
    if (tiled) {
      // the thresholds are read while the wave's first words are on their way
      const auto stage = [&] {
        stage_band(a, thr, tid, x0, y0, L.tw, L.th);
        __syncthreads();
      };
      if (k == 10) raster_by_class<10, true, true>(cls, L, st, sums, first, count, wave, lane, natom, stage);
      else if (k == 20) raster_by_class<20, true, true>(cls, L, st, sums, first, count, wave, lane, natom, stage);
      else raster_by_class<30, true, true>(cls, L, st, sums, first, count, wave, lane, natom, stage);
    } else {
      if (k == 10) raster_by_class<10, false, true>(cls, L, st, sums, first, count, wave, lane, natom);
      else if (k == 20) raster_by_class<20, false, true>(cls, L, st, sums, first, count, wave, lane, natom);
      else raster_by_class<30, false, true>(cls, L, st, sums, first, count, wave, lane, natom);
    }
    __syncthreads();  // the batch's sums are complete; s_next has been read
    if (tid == 0) s_next = grab;
    if (tiled && count != 0) flush_band(a, sums, tid, x0, y0, L.tw, L.th);
    __syncthreads();  // tile free for the next batch; s_next visible
    cut.at(uni(s_next), item, slice);
  }
}

// Zeroes the sums and, in its first block, the work-queue counters that the
// frame's render has used up.
__global__ void __launch_bounds__(256) k_zero_sums(uint64_t* p, uint64_t n, FrameHeader* hdr) {
  const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
  if (blockIdx.x == 0 && threadIdx.x < RENDER_QUEUES && hdr) hdr->queue[threadIdx.x][0] = 0;
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) p[i] = 0;
}

// The average of the sums: each channel (sum + n / 2) / n, alpha 255; the
// clear colour where no point joined.
__global__ void __launch_bounds__(256) k_resolve_hqs(const uint64_t* __restrict__ acc, uint64_t npix,
                                                     uint32_t clear_rgba, uint32_t* __restrict__ fb) {
  const uint64_t p = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= npix) return;
  const uint64_t rg = acc[2 * p], bn = acc[2 * p + 1];
  const uint64_t n = bn >> 32;
  if (n == 0) {
    fb[p] = clear_rgba;
    return;
  }
  const uint64_t r = ((rg & 0xFFFFFFFFull) + n / 2) / n, g = ((rg >> 32) + n / 2) / n;
  const uint64_t b = ((bn & 0xFFFFFFFFull) + n / 2) / n;
  fb[p] = (uint32_t)r | ((uint32_t)g << 8) | ((uint32_t)b << 16) | (255u << 24);
}

}  // namespace

uint32_t accum_grid(int device) {
  int per_cu = 0, cus = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_accum, THREADS, 0) != hipSuccess || per_cu < 1)
    per_cu = 1;
  if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, device) != hipSuccess || cus < 1) cus = 1;
  return (uint32_t)(per_cu * cus);
}

hipError_t launch_accumulate(const RenderArgs& a, hipStream_t s) {
  const uint64_t n = 2ull * a.W * a.H;
  uint64_t blocks = (n + 255) / 256;
  if (blocks > 4096) blocks = 4096;
  // the shading pass walks the render's live list with fresh work-queue counters
  hipLaunchKernelGGL(k_zero_sums, dim3((uint32_t)blocks), dim3(256), 0, s, a.accum, n, a.nb ? a.hdr : nullptr);
  if (a.nb == 0) return hipGetLastError();
  const uint64_t items = (uint64_t)a.nb << MAX_SLICE_SHIFT;
  const uint32_t blocks_r = a.grid < items ? a.grid : (uint32_t)items;
  hipLaunchKernelGGL(k_accum, dim3(blocks_r), dim3(THREADS), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_resolve_hqs(const uint64_t* accum, uint64_t npix, uint32_t clear_rgba, uint32_t* fb,
                              hipStream_t s) {
  const uint64_t blocks = (npix + 255) / 256;
  if (blocks == 0) return hipSuccess;
  hipLaunchKernelGGL(k_resolve_hqs, dim3((uint32_t)blocks), dim3(256), 0, s, accum, npix, clear_rgba, fb);
  return hipGetLastError();
}

}  // namespace ptr
