// Per-(view, surfel) culling and EWA projection (Eq. 5, supp. Sec. 2.1), tile
// counts and visible counts per block, their scans, and the generic scan.
//
// One block per (range of 256 surfels, view): a thread projects one surfel
// into one view (the other views' blocks of a surfel range find its
// parameters in the cache); per-view results land in "slot" arrays indexed
// v * N + i.
#include <math.h>

#include <algorithm>

#include "rogs_internal.h"

namespace rogs {

namespace {

// (range, view) pairs from which a list pays: its launch costs about 10 us and a
// culled block of the direct launch 1.2 ns.  Listed against direct: 70000 pairs
// (6 views of 3M surfels) 73 / 95 us, 75000 (24 of 800k, fewer of them culled)
// 204 / 209, 11700 (one view of 3M) 22 / 19, 4700 (an export's chunk) 41 / 24.
constexpr int64_t kProjListMin = 32768;
constexpr int64_t kProjListBlocks = 6144;   // blocks that stride over it

__device__ __forceinline__ uint32_t nonzero_bytes4(uint32_t x) {
  return ((x & 0xffu) != 0u) + ((x & 0xff00u) != 0u) + ((x & 0xff0000u) != 0u) +
         ((x & 0xff000000u) != 0u);
}

// Extra blocks of the fused step's projection launch, chunk c of view v: the
// nonzero bytes of chunk c (kMaskChunk bytes) of view v's loss mask into
// mpart[v * nmb + c] (summed per view by the count-table scan), and a share
// of clearing the n_zero per-tile pair counters.  Work the step needs
// anyway, done here instead of in two launches of its own.
__device__ void project_side_block(const ViewDev* __restrict__ views, int V, int c, int v,
                                   const uint8_t* __restrict__ mask, int nmb,
                                   uint32_t* __restrict__ mpart, uint32_t* __restrict__ zero_words,
                                   int64_t n_zero, uint32_t* s_w) {
  const ViewDev& vw = views[v];
  const int64_t npix = (int64_t)vw.w * vw.h;
  const uint8_t* m = mask + vw.pix_off;
  uint32_t cnt = 0;
#pragma unroll
  for (int it = 0; it < kMaskChunk / (16 * kProjBlock); ++it) {
    const int64_t p = (int64_t)c * kMaskChunk + 16 * ((int64_t)it * kProjBlock + threadIdx.x);
    if (p >= npix) continue;
    const uint8_t* g = m + p;
    if (p + 16 <= npix && (reinterpret_cast<uintptr_t>(g) & 15u) == 0) {
      const uint4 x = *reinterpret_cast<const uint4*>(g);
      cnt += nonzero_bytes4(x.x) + nonzero_bytes4(x.y) + nonzero_bytes4(x.z) + nonzero_bytes4(x.w);
    } else {
      const int n = (int)min<int64_t>(16, npix - p);
      for (int k = 0; k < n; ++k) cnt += g[k] ? 1u : 0u;
    }
  }
  cnt = wave_sum_u32(cnt);
  if ((threadIdx.x & 63) == 0) s_w[threadIdx.x >> 6] = cnt;
  __syncthreads();
  if (threadIdx.x == 0) {
    uint32_t t = 0;
    for (int w = 0; w < kProjBlock / 64; ++w) t += s_w[w];
    mpart[(size_t)v * nmb + c] = t;
  }
  const int64_t nside = (int64_t)V * nmb;
  for (int64_t k = ((int64_t)v * nmb + c) * kProjBlock + threadIdx.x; k < n_zero;
       k += nside * kProjBlock)
    zero_words[k] = 0u;
}

struct ProjLds {
  uint32_t w[kProjBlock / 64], v[kProjBlock / 64];
  Span sp[kProjBlock];            // per-record span set-up
  uint32_t roff[kProjBlock];      // first row item of each lane in its wave
  uint32_t y0[kProjBlock], y1[kProjBlock], cnt[kProjBlock];
};

// The projection of one range of surfels into view v.  Surfels that certainly
// lie outside (the contract's first tests, frustum_outside) skip it, and so do
// waves and blocks of such surfels.  A block without a candidate does not write
// its slots' counts: every reader of per-slot arrays tests the block's visible
// count (partv) first.
__device__ __forceinline__ void project_block(
    ProjLds& L, const ViewDev* __restrict__ views, int N, int nb, int range, int v, float eps,
    float qcut, double r_cut, double sqrt_eps, const float* __restrict__ px,
    const float* __restrict__ py, const float* __restrict__ pz, const float* __restrict__ pq,
    const float* __restrict__ ps, uint32_t* __restrict__ cnt, float4* __restrict__ rec,
    uint2* __restrict__ rect, uint16_t* __restrict__ rspan, uint32_t* __restrict__ part,
    uint32_t* __restrict__ partv) {
  const int i = range * kProjBlock + threadIdx.x;
  const int lane = threadIdx.x & 63, wbase = threadIdx.x & ~63;
  const bool valid = i < N;
  const ViewDev& vw = views[v];
  const size_t slot = (size_t)v * N + i;
  const size_t pb = (size_t)v * nb + range;
  float zf = 0.0f, sxf = 0.0f, syf = 0.0f;
  bool cand = false;
  if (valid && ground_inside(vw, px[i], py[i])) {
    zf = pz[i];
    sxf = ps[i];
    syf = ps[N + i];
    cand = !frustum_outside(vw, r_cut, sqrt_eps, px[i], py[i], zf, sxf, syf);
  }
  if (!__syncthreads_or(cand)) {
    if (threadIdx.x == 0) part[pb] = partv[pb] = 0u;
    return;
  }
  uint32_t nt = 0, rows = 0;
  Proj p;
  p.vis = false;
  p.y0 = 0;
  if (cand) {
    p = project_contract(vw, eps, qcut, px[i], py[i], zf, pq[i], pq[N + i],
                         pq[2 * (size_t)N + i], pq[3 * (size_t)N + i], sxf, syf);
    if (p.vis) {
      const Span sp = span_setup(p.uh, p.vh, p.ul, p.vl, p.A, p.B, p.C, qcut, p.x0, p.x1);
      if (sp.full) {
        nt = (uint32_t)((p.x1 - p.x0) * (p.y1 - p.y0));
        if (span_desc_ok(p.x0, p.x1, p.y0, p.y1))
          for (int r = 0; r < p.y1 - p.y0; ++r)
            rspan[slot * kSpanRows + r] = (uint16_t)((p.x1 - p.x0) << 8);
      } else {
        rows = (uint32_t)(p.y1 - p.y0);
      }
      L.sp[threadIdx.x] = sp;
      rec[2 * slot] = make_float4(p.uh, p.vh, p.ul, p.vl);
      rec[2 * slot + 1] = make_float4(p.A, p.B, p.C, p.tz);
      rect[slot] = make_uint2((uint32_t)p.x0 | ((uint32_t)p.x1 << 16),
                              (uint32_t)p.y0 | ((uint32_t)p.y1 << 16));
    }
  }
  // the wave's rectangle rows, spread evenly over its lanes: the row spans
  // of one record are summed into its lane's counter (integer adds)
  const uint32_t incl = wave_incl_scan(rows, lane);
  const uint32_t R = __shfl(incl, 63, 64);
  L.roff[threadIdx.x] = incl - rows;
  L.y0[threadIdx.x] = (uint32_t)p.y0;
  L.y1[threadIdx.x] = (uint32_t)p.y1;
  L.cnt[threadIdx.x] = 0;
  __syncthreads();
  for (uint32_t k = (uint32_t)lane; k < R; k += 64) {
    const int j = wbase + last_le(L.roff + wbase, 64, k);
    const int r = (int)(k - L.roff[j]);
    const Span& sj = L.sp[j];
    int lo, hi;
    span_row(sj, vw.tw, vw.th, vw.w, vw.h, (int)L.y0[j] + r, lo, hi);
    if (hi > lo) atomicAdd(&L.cnt[j], (uint32_t)(hi - lo));
    if (span_desc_ok(sj.x0, sj.x1, (int)L.y0[j], (int)L.y1[j]))
      rspan[((size_t)v * N + range * kProjBlock + (j & (kProjBlock - 1))) * kSpanRows + r] =
          (uint16_t)((lo - sj.x0) | ((hi - sj.x0) << 8));
  }
  __syncthreads();
  nt += L.cnt[threadIdx.x];
  if (valid) cnt[slot] = nt;
  uint32_t ws = wave_sum_u32(nt);
  const uint32_t wvis = (uint32_t)__popcll(__ballot(nt != 0));
  if (lane == 0) {
    L.w[threadIdx.x >> 6] = ws;
    L.v[threadIdx.x >> 6] = wvis;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    uint32_t t = 0, tv = 0;
    for (int w = 0; w < kProjBlock / 64; ++w) {
      t += L.w[w];
      tv += L.v[w];
    }
    part[pb] = t;
    partv[pb] = tv;
  }
}

// The (range, view) pairs that the projection has to look at: a wave per range
// of kProjBlock surfels, four to a lane, tests them against every view's ground
// rectangle and image (frustum_outside), appends the pairs with a candidate, as
// index v * nb + range, to list, and writes the zero counts of the others.
// Most pairs of a long road go here (82 % of 24 views of a 200 m strip, more of
// a longer one), and a block of the projection's own launch for each of them is
// bound by the rate at which blocks start (kProjListMin).  Extra blocks as in
// project_side_block from block range_blocks on; this launch's blocks start at
// first_block.
__global__ __launch_bounds__(kProjBlock) void k_project_list(
    const ViewDev* __restrict__ views, int V, int N, int nb, int first_block, int range_blocks,
    double r_cut, double sqrt_eps, const float* __restrict__ px, const float* __restrict__ py,
    const float* __restrict__ pz, const float* __restrict__ ps, uint32_t* __restrict__ part,
    uint32_t* __restrict__ partv, uint32_t* __restrict__ list, uint32_t* __restrict__ misc,
    const uint8_t* __restrict__ mask, int nmb, uint32_t* __restrict__ mpart,
    uint32_t* __restrict__ zero_words, int64_t n_zero) {
  __shared__ uint32_t s_w[kProjBlock / 64];
  const int block = first_block + (int)blockIdx.x;
  if (block >= range_blocks) {
    const int k = block - range_blocks;
    project_side_block(views, V, k % nmb, k / nmb, mask, nmb, mpart, zero_words, n_zero, s_w);
    return;
  }
  constexpr int kPer = kProjBlock / 64;
  const int lane = threadIdx.x & 63;
  const int range = block * kPer + (int)(threadIdx.x >> 6);
  if (range >= nb) return;
  const int i0 = range * kProjBlock + lane;
  float x[kPer], y[kPer];
#pragma unroll
  for (int u = 0; u < kPer; ++u) {
    // (past the end: the range's first surfel once more, which adds no candidate)
    const int i = i0 + 64 * u < N ? i0 + 64 * u : range * kProjBlock;
    x[u] = px[i];
    y[u] = py[i];
  }
  for (int v0 = 0; v0 < V; v0 += 64) {
    // bit k: some surfel of the range may be visible in view v0 + k
    const int vn = min(64, V - v0);
    unsigned long long any = 0ull;
    for (int k = 0; k < vn; ++k) {
      const ViewDev& vw = views[v0 + k];
      bool c = false;
#pragma unroll
      for (int u = 0; u < kPer; ++u) c = c || ground_inside(vw, x[u], y[u]);
      if (__ballot(c)) any |= 1ull << k;
    }
    if (any) {
      float z[kPer], sx[kPer], sy[kPer];
#pragma unroll
      for (int u = 0; u < kPer; ++u) {
        const int i = i0 + 64 * u < N ? i0 + 64 * u : range * kProjBlock;
        z[u] = pz[i];
        sx[u] = ps[i];
        sy[u] = ps[N + i];
      }
      for (unsigned long long m = any; m; m &= m - 1ull) {
        const int k = __builtin_ctzll(m);
        const ViewDev& vw = views[v0 + k];
        bool c = false;
        for (int u = 0; u < kPer; ++u)
          c = c || (ground_inside(vw, x[u], y[u]) &&
                    !frustum_outside(vw, r_cut, sqrt_eps, x[u], y[u], z[u], sx[u], sy[u]));
        if (!__ballot(c)) any &= ~(1ull << k);
      }
    }
    uint32_t base = 0;
    if (lane == 0 && any) base = atomicAdd(&misc[kMiscList], (uint32_t)__popcll(any));
    base = __shfl(base, 0, 64);
    if (lane < vn) {
      const size_t pb = (size_t)(v0 + lane) * nb + range;
      if ((any >> lane) & 1ull) {
        list[base + (uint32_t)__popcll(any & ((1ull << lane) - 1ull))] = (uint32_t)pb;
      } else {
        part[pb] = 0u;
        partv[pb] = 0u;
      }
    }
  }
}

// One (range, view) pair per block: each thread projects one surfel.  With
// kListed, the blocks stride over the pairs that k_project_list left; without,
// the pair is the block's own (grid.x = range, grid.y = view).  Two kernels: as
// one both took the 93 registers of the loop, 5 waves per SIMD; without it the
// direct one takes 72, 6 waves, the most that its LDS block allows (24 views that
// all see 400k surfels 331 -> 309 us).
template <bool kListed>
__global__ __launch_bounds__(kProjBlock) void k_project(
    const ViewDev* __restrict__ views, int V, int N, int nb, float eps, float qcut, double r_cut,
    double sqrt_eps, const float* __restrict__ px, const float* __restrict__ py,
    const float* __restrict__ pz,
    const float* __restrict__ pq, const float* __restrict__ ps,
    uint32_t* __restrict__ cnt, float4* __restrict__ rec, uint2* __restrict__ rect,
    uint16_t* __restrict__ rspan, uint32_t* __restrict__ part, uint32_t* __restrict__ partv,
    const uint32_t* __restrict__ list, const uint32_t* __restrict__ misc,
    const uint8_t* __restrict__ mask, int nmb,
    uint32_t* __restrict__ mpart, uint32_t* __restrict__ zero_words, int64_t n_zero) {
  __shared__ ProjLds L;
  if constexpr (kListed) {
    const uint32_t n = misc[kMiscList];
    for (uint32_t w = blockIdx.x; w < n; w += gridDim.x) {
      const uint32_t pb = list[w];
      const int v = (int)(pb / (uint32_t)nb);
      project_block(L, views, N, nb, (int)(pb - (uint32_t)v * (uint32_t)nb), v, eps, qcut, r_cut,
                    sqrt_eps, px, py, pz, pq, ps, cnt, rec, rect, rspan, part, partv);
      __syncthreads();
    }
    return;
  }
  if (blockIdx.x >= (unsigned)nb) {
    project_side_block(views, V, (int)blockIdx.x - nb, (int)blockIdx.y, mask, nmb, mpart,
                       zero_words, n_zero, L.w);
    return;
  }
  project_block(L, views, N, nb, (int)blockIdx.x, (int)blockIdx.y, eps, qcut, r_cut, sqrt_eps, px,
                py, pz, pq, ps, cnt, rec, rect, rspan, part, partv);
}

// Feature records of the surfel ranges (projection blocks) that some view sees,
// between the projection and the scan of its counts (partv still holds the
// visible slots of each block).  Bound by the bytes of the ranges that are
// packed: packing every surfel of a 3M-surfel map with 16 classes moved 480 MB
// (120 us) for a view that sees 2 % of it; 7 us with the test.
__global__ __launch_bounds__(kProjBlock) void k_pack_feat(int V, int N, int nb, int C, int FS,
                                                          const uint32_t* __restrict__ partv,
                                                          const float* __restrict__ pa,
                                                          const float* __restrict__ prgb,
                                                          const float* __restrict__ psem,
                                                          float4* __restrict__ feat) {
  bool seen = false;
  for (int v = threadIdx.x; v < V; v += kProjBlock)
    seen = seen || partv[(size_t)v * nb + blockIdx.x] != 0u;
  if (__syncthreads_or(seen)) pack_features(blockIdx.x, N, C, FS, pa, prgb, psem, feat);
}

// Per-view mask counts from the projection's side blocks (exact integer
// sums): per view, the block's threads stride over the chunks, then a wave
// sum and the waves' totals.  blockDim.x is a multiple of 64, at most 1024.
// One block for all views (small batches, inside k_scan_part) ...
__device__ __forceinline__ void sum_mask_parts_all(const uint32_t* __restrict__ mpart, int nmb,
                                                   int V, uint32_t* __restrict__ mcount) {
  __shared__ uint32_t s_t[16];
  for (int v = 0; v < V; ++v) {
    uint32_t t = 0;
    for (int c = threadIdx.x; c < nmb; c += blockDim.x) t += mpart[(size_t)v * nmb + c];
    t = wave_sum_u32(t);
    if ((threadIdx.x & 63) == 0) s_t[threadIdx.x >> 6] = t;
    __syncthreads();
    if (threadIdx.x == 0) {
      uint32_t a = 0;
      for (int w = 0; w < (int)(blockDim.x >> 6); ++w) a += s_t[w];
      mcount[v] = a;
    }
    __syncthreads();
  }
}

// ... or one 64-lane block per view (view v's count).
__device__ __forceinline__ void sum_mask_parts(const uint32_t* __restrict__ mpart, int nmb, int v,
                                               uint32_t* __restrict__ mcount) {
  uint32_t t = 0;
  for (int c = threadIdx.x; c < nmb; c += 64) t += mpart[(size_t)v * nmb + c];
  t = wave_sum_u32(t);
  if (threadIdx.x == 0) mcount[v] = t;
}

// ------------------------------------------------------------ generic scan

__device__ __forceinline__ int64_t scan_count(const uint32_t* n_dev, int64_t n) {
  if (!n_dev) return n;
  const int64_t d = (int64_t)(*n_dev);
  return d < n ? d : n;
}

// The three passes of the multi-block scan as block bodies: the single-table
// kernels below and the paired ones (both projection count tables in one set
// of launches) share them.
__device__ __forceinline__ void scan_reduce_block(const uint32_t* __restrict__ in, int64_t n,
                                                  uint32_t* __restrict__ sums) {
  __shared__ uint32_t s_w[4];
  const int64_t base = (int64_t)blockIdx.x * kScanChunk;
  uint32_t acc = 0;
  for (int k = threadIdx.x; k < kScanChunk; k += 256) {
    int64_t j = base + k;
    if (j < n) acc += in[j];
  }
  acc = wave_sum_u32(acc);
  if ((threadIdx.x & 63) == 0) s_w[threadIdx.x >> 6] = acc;
  __syncthreads();
  if (threadIdx.x == 0) sums[blockIdx.x] = s_w[0] + s_w[1] + s_w[2] + s_w[3];
}

__global__ __launch_bounds__(256) void k_scan_reduce(const uint32_t* __restrict__ in, int64_t n_cap,
                                                     const uint32_t* __restrict__ n_dev,
                                                     uint32_t* __restrict__ sums) {
  scan_reduce_block(in, scan_count(n_dev, n_cap), sums);
}

// Exclusive scan in place of m values with one block of 1024 threads.
__device__ __forceinline__ void scan_top_block(uint32_t* __restrict__ sums, int64_t m,
                                               uint32_t* __restrict__ total) {
  __shared__ uint32_t s_w[16];
  const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
  const int64_t per = (m + 1023) / 1024;
  const int64_t b = t * per, e = (b + per < m) ? b + per : m;
  uint32_t loc = 0;
  for (int64_t j = b; j < e; ++j) loc += sums[j];
  uint32_t inc = wave_incl_scan(loc, lane);
  if (lane == 63) s_w[wv] = inc;
  __syncthreads();
  uint32_t pre = 0, tot = 0;
  for (int w = 0; w < 16; ++w) {
    pre += (w < wv) ? s_w[w] : 0u;
    tot += s_w[w];
  }
  uint32_t run = pre + inc - loc;
  for (int64_t j = b; j < e; ++j) {
    uint32_t x = sums[j];
    sums[j] = run;
    run += x;
  }
  if (t == 0 && total) *total = tot;
}

__global__ __launch_bounds__(1024) void k_scan_top(uint32_t* __restrict__ sums, int64_t m,
                                                   uint32_t* __restrict__ total) {
  scan_top_block(sums, m, total);
}

// in and out may be the same array (each block reads its chunk before writing it).
__device__ __forceinline__ void scan_down_block(const uint32_t* in, uint32_t* out, int64_t n,
                                                const uint32_t* __restrict__ sums) {
  __shared__ uint32_t s_v[kScanChunk];
  __shared__ uint32_t s_w[4];
  const int64_t base = (int64_t)blockIdx.x * kScanChunk;
  if (base >= n) return;
  for (int k = threadIdx.x; k < kScanChunk; k += 256) {
    int64_t j = base + k;
    s_v[k] = (j < n) ? in[j] : 0u;
  }
  __syncthreads();
  constexpr int per = kScanChunk / 256;
  const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
  uint32_t loc = 0;
  for (int k = 0; k < per; ++k) loc += s_v[t * per + k];
  uint32_t inc = wave_incl_scan(loc, lane);
  if (lane == 63) s_w[wv] = inc;
  __syncthreads();
  uint32_t pre = sums[blockIdx.x];
  for (int w = 0; w < 4; ++w) pre += (w < wv) ? s_w[w] : 0u;
  uint32_t run = pre + inc - loc;
  for (int k = 0; k < per; ++k) {
    uint32_t x = s_v[t * per + k];
    s_v[t * per + k] = run;
    run += x;
  }
  __syncthreads();
  for (int k = threadIdx.x; k < kScanChunk; k += 256) {
    int64_t j = base + k;
    if (j < n) out[j] = s_v[k];
  }
}

__global__ __launch_bounds__(256) void k_scan_down(const uint32_t* in, uint32_t* out, int64_t n_cap,
                                                   const uint32_t* __restrict__ n_dev,
                                                   const uint32_t* __restrict__ sums) {
  scan_down_block(in, out, scan_count(n_dev, n_cap), sums);
}

// Both projection count tables (pairs, visible slots; n values each, scanned
// in place): table blockIdx.y of the reduce and down passes, block b of the
// top pass; the sums of table a at sums + a * ms.
__global__ __launch_bounds__(256) void k_scan2_reduce(uint32_t* t0, uint32_t* t1, int64_t n,
                                                      uint32_t* __restrict__ sums, int64_t ms) {
  scan_reduce_block(blockIdx.y ? t1 : t0, n, sums + blockIdx.y * ms);
}

__global__ __launch_bounds__(1024) void k_scan2_top(uint32_t* __restrict__ sums, int64_t ms,
                                                    int64_t m, uint32_t* __restrict__ total0,
                                                    uint32_t* __restrict__ total1) {
  scan_top_block(sums + blockIdx.x * ms, m, blockIdx.x ? total1 : total0);
}

// A third row of blocks (blockIdx.y == 2) runs once the totals are known:
// block 0 sets the overflow flag, and with mpart block x sums view x's mask
// count.
__global__ __launch_bounds__(256) void k_scan2_down(uint32_t* t0, uint32_t* t1, int64_t n,
                                                    const uint32_t* __restrict__ sums,
                                                    int64_t ms, uint32_t* misc, int64_t cap,
                                                    int64_t scap,
                                                    const uint32_t* __restrict__ mpart, int nmb,
                                                    int V, uint32_t* __restrict__ mcount) {
  if (blockIdx.y == 2) {
    if (threadIdx.x == 0 && blockIdx.x == 0)
      misc[kMiscOverflow] =
          ((int64_t)misc[kMiscPairs] > cap || (int64_t)misc[kMiscVisible] > scap) ? 1u : 0u;
    // one wave per view
    if (mpart && (int)blockIdx.x < V && threadIdx.x < 64)
      sum_mask_parts(mpart, nmb, (int)blockIdx.x, mcount);
    return;
  }
  uint32_t* t = blockIdx.y ? t1 : t0;
  scan_down_block(t, t, n, sums + blockIdx.y * ms);
}

// Exclusive scan of at most kSmallScan values in one block of 1024 threads
// (one launch instead of three for the small tables).  Rounds of kSmallChunk
// values: a coalesced load into LDS (padded by one word per 32 against bank
// conflicts), 8 consecutive values per thread, a block scan of the thread
// sums, the results back through LDS and a coalesced store; a carry links
// the rounds.  Every round reads its values before it writes them, so
// in == out is allowed.
constexpr int kSmallScan = 1024 * 32;
constexpr int kSmallChunk = 1024 * 8;

__device__ __forceinline__ int pad32(int i) { return i + (i >> 5); }

__device__ __forceinline__ void block_scan_small(const uint32_t* in, uint32_t* out, int64_t n,
                                                 uint32_t* __restrict__ total) {
  __shared__ uint32_t s[kSmallChunk + kSmallChunk / 32];
  __shared__ uint32_t s_w[16];
  const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
  uint32_t carry = 0;
  for (int64_t c0 = 0; c0 < n; c0 += kSmallChunk) {
    const int m = (int)((n - c0) < kSmallChunk ? (n - c0) : kSmallChunk);
    for (int i = t; i < kSmallChunk; i += 1024) s[pad32(i)] = (i < m) ? in[c0 + i] : 0u;
    __syncthreads();
    uint32_t v[8];
    uint32_t loc = 0;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      v[j] = s[pad32(8 * t + j)];
      loc += v[j];
    }
    const uint32_t inc = wave_incl_scan(loc, lane);
    if (lane == 63) s_w[wv] = inc;
    __syncthreads();
    uint32_t pre = 0, tot = 0;
    for (int w = 0; w < 16; ++w) {
      pre += (w < wv) ? s_w[w] : 0u;
      tot += s_w[w];
    }
    uint32_t run = carry + pre + inc - loc;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      s[pad32(8 * t + j)] = run;
      run += v[j];
    }
    __syncthreads();
    for (int i = t; i < m; i += 1024) out[c0 + i] = s[pad32(i)];
    carry += tot;
    __syncthreads();
  }
  if (t == 0 && total) *total = carry;
}

__global__ __launch_bounds__(1024) void k_scan_small(const uint32_t* in, uint32_t* out,
                                                     int64_t n_cap,
                                                     const uint32_t* __restrict__ n_dev,
                                                     uint32_t* __restrict__ total) {
  block_scan_small(in, out, scan_count(n_dev, n_cap), total);
}

// Both per-block count tables of the projection (pairs, visible slots) in one
// launch, one block each, and with mpart a third block for the per-view mask
// counts.  (The compaction sets the overflow flag: a last-block test here, with
// its device-wide fence, made 11 us of a 4 us scan.)
__global__ __launch_bounds__(1024) void k_scan_part(uint32_t* part, uint32_t* partv, int64_t n,
                                                    uint32_t* __restrict__ misc,
                                                    const uint32_t* __restrict__ mpart, int nmb,
                                                    int V, uint32_t* __restrict__ mcount) {
  if (blockIdx.x == 2) {
    sum_mask_parts_all(mpart, nmb, V, mcount);
  } else {
    uint32_t* a = blockIdx.x == 0 ? part : partv;
    block_scan_small(a, a, n, misc + (blockIdx.x == 0 ? kMiscPairs : kMiscVisible));
  }
}

// The view table from the host's pinned stage, and the batch's counters cleared
// (one launch; a copy and a fill took two of 4 us each).
__global__ __launch_bounds__(256) void k_upload(const uint32_t* __restrict__ stage,
                                                uint32_t* __restrict__ table, int64_t n,
                                                uint32_t* __restrict__ misc) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i < n) table[i] = stage[i];
  if (i < kMiscCount) misc[i] = 0u;
}

__global__ void k_fill_u32(uint32_t* __restrict__ p, uint32_t value, int64_t n) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (; i < n; i += stride) p[i] = value;
}

}  // namespace

size_t scan_tmp_words(int64_t n) { return (size_t)((n + kScanChunk - 1) / kScanChunk) + 1; }

void scan_u32(const uint32_t* in, uint32_t* out, int64_t n, uint32_t* total, uint32_t* tmp,
              hipStream_t st) {
  if (n <= 0) return;
  if (n <= kSmallScan) {
    hipLaunchKernelGGL(k_scan_small, dim3(1), dim3(1024), 0, st, in, out, n,
                       (const uint32_t*)nullptr, total);
    return;
  }
  int64_t m = (n + kScanChunk - 1) / kScanChunk;
  hipLaunchKernelGGL(k_scan_reduce, dim3((unsigned)m), dim3(256), 0, st, in, n,
                     (const uint32_t*)nullptr, tmp);
  hipLaunchKernelGGL(k_scan_top, dim3(1), dim3(1024), 0, st, tmp, m, total);
  hipLaunchKernelGGL(k_scan_down, dim3((unsigned)m), dim3(256), 0, st, in, out, n,
                     (const uint32_t*)nullptr, tmp);
}

void fill_u32(uint32_t* p, uint32_t value, int64_t n, hipStream_t st) {
  if (n <= 0) return;
  int64_t blocks = (n + 255) / 256;
  if (blocks > 8192) blocks = 8192;
  hipLaunchKernelGGL(k_fill_u32, dim3((unsigned)blocks), dim3(256), 0, st, p, value, n);
}

void launch_upload(const Layout& L, void* ws, const void* stage, size_t bytes, hipStream_t st) {
  const int64_t n = (int64_t)(bytes / 4);
  hipLaunchKernelGGL(k_upload, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st,
                     static_cast<const uint32_t*>(stage), at<uint32_t>(ws, L.o_views), n,
                     at<uint32_t>(ws, L.o_misc));
}

void launch_project(const Layout& L, void* ws, const rogs_surfels* s, hipStream_t st,
                    const uint8_t* mask) {
  if (mask) fill_u32(at<uint32_t>(ws, L.o_misc), 0u, kMiscCount, st);
  const int nmb = mask ? mask_chunks(L) : 0;
  const ViewDev* views = at<const ViewDev>(ws, L.o_views);
  uint32_t* misc = at<uint32_t>(ws, L.o_misc);
  uint32_t* part = at<uint32_t>(ws, L.o_part);
  uint32_t* partv = at<uint32_t>(ws, L.o_partv);
  uint32_t* mpart = mask ? at<uint32_t>(ws, L.o_mpart) : nullptr;
  uint32_t* tcnt = mask ? at<uint32_t>(ws, L.o_tcnt) : nullptr;
  const int64_t n_zero = mask ? L.total_tiles : 0;
  const double r_cut = sqrt((double)L.q_cut) * (1.0 + 1e-9), sqrt_eps = sqrt((double)L.eps2d);
  const bool listed = (int64_t)L.V * L.nb > kProjListMin;
  uint32_t* list = listed ? at<uint32_t>(ws, L.o_pos) : nullptr;   // written by the compaction later
  const int range_blocks = (L.nb + kProjBlock / 64 - 1) / (kProjBlock / 64);
  if (listed)
    launch_bands(range_blocks + (int64_t)nmb * L.V, kProjBlock, [&](int64_t first, unsigned n) {
      hipLaunchKernelGGL(k_project_list, dim3(n), dim3(kProjBlock), 0, st, views, L.V, L.N, L.nb,
                         (int)first, range_blocks, r_cut, sqrt_eps, s->x, s->y, s->z, s->s, part,
                         partv, list, misc, mask, nmb, mpart, tcnt, n_zero);
    });
  const dim3 grid = listed ? dim3((unsigned)std::min<int64_t>((int64_t)L.V * L.nb, kProjListBlocks))
                           : dim3(L.nb + nmb, L.V);
  hipLaunchKernelGGL(listed ? k_project<true> : k_project<false>, grid, dim3(kProjBlock), 0, st,
                     views, L.V, L.N, L.nb, L.eps2d, L.q_cut, r_cut, sqrt_eps, s->x, s->y, s->z, s->q, s->s,
                     at<uint32_t>(ws, L.o_cnt), at<float4>(ws, L.o_rec), at<uint2>(ws, L.o_rect),
                     at<uint16_t>(ws, L.o_rspan), part, partv, list, misc, mask, nmb, mpart, tcnt,
                     n_zero);
}

void launch_pack_feat(const Layout& L, void* ws, const rogs_surfels* s, hipStream_t st) {
  hipLaunchKernelGGL(k_pack_feat, dim3(L.nb), dim3(kProjBlock), 0, st, L.V, L.N, L.nb, L.C, L.FS,
                     at<const uint32_t>(ws, L.o_partv), s->alpha, s->rgb, s->sem,
                     at<float4>(ws, L.o_feat));
}

void launch_scan_part(const Layout& L, void* ws, hipStream_t st, bool mask_parts) {
  uint32_t* misc = at<uint32_t>(ws, L.o_misc);
  const uint32_t* mpart = mask_parts ? at<const uint32_t>(ws, L.o_mpart) : nullptr;
  const int nmb = mask_parts ? mask_chunks(L) : 0;
  uint32_t* mcount = at<uint32_t>(ws, L.o_mcount);
  if ((int64_t)L.V * L.nb <= kSmallScan) {
    hipLaunchKernelGGL(k_scan_part, dim3(mask_parts ? 3 : 2), dim3(1024), 0, st,
                       at<uint32_t>(ws, L.o_part), at<uint32_t>(ws, L.o_partv),
                       (int64_t)L.V * L.nb, misc, mpart, nmb, L.V, mcount);
    return;
  }
  // both tables at once: three launches instead of six
  const int64_t n = (int64_t)L.V * L.nb;
  const int64_t m = (n + kScanChunk - 1) / kScanChunk;
  const int64_t ms = (int64_t)scan_tmp_words(n);   // sums of one table
  uint32_t* sums = at<uint32_t>(ws, L.o_parttmp);
  uint32_t* part = at<uint32_t>(ws, L.o_part);
  uint32_t* partv = at<uint32_t>(ws, L.o_partv);
  hipLaunchKernelGGL(k_scan2_reduce, dim3((unsigned)m, 2), dim3(256), 0, st, part, partv, n, sums,
                     ms);
  hipLaunchKernelGGL(k_scan2_top, dim3(2), dim3(1024), 0, st, sums, ms, m, misc + kMiscPairs,
                     misc + kMiscVisible);
  const int64_t gx = std::max<int64_t>(m, mpart ? L.V : 1);   // the scan's blocks, the views
  hipLaunchKernelGGL(k_scan2_down, dim3((unsigned)gx, 3), dim3(256), 0, st, part, partv, n, sums,
                     ms, misc, L.cap, L.scap, mpart, nmb, L.V, mcount);
}

}  // namespace rogs
