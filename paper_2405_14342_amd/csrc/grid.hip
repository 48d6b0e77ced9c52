// Grid-side terms of the training loss and the surfel grid itself:
//   * elevation smoothness over the four grid neighbours (Eq. 10; the
//     neighbours come from the pixel index of the meshgrid, supp. Sec. 3.3)
//     and the LiDAR elevation loss (Eq. 11), both per surfel;
//   * the LiDAR targets: height of the point nearest to each surfel in the
//     xy-plane (Eq. 11);
//   * the meshgrid layout (Sec. 3.1): vehicle positions on a raster, a disk
//     dilation into the road mask, surfels at its pixels indexed by a running
//     count, neighbour indices from adjacent pixels, and the pose-based
//     initial height and rotation (Eq. 4; supp. Sec. 1).
#include <math.h>

#include <algorithm>
#include <cmath>
#include <mutex>
#include <string>

#include "rogs_internal.h"

namespace rogs {


namespace {

constexpr int kRegBlock = 256;

// Block partial sums of rogs_elev_loss_static: one float per block of the
// largest accepted surfel count (ROGS_ELEV_STATIC_MAX_N).  Each GPU the
// library runs on holds its own copy until the process ends.  Host code uses
// only the per-device address from hipGetSymbolAddress, never this name.
constexpr int64_t kElevStaticFloats = ((int64_t)ROGS_ELEV_STATIC_MAX_N + kRegBlock - 1) / kRegBlock + 1;
static __device__ __align__(256) float scratch[kElevStaticFloats];

// Per surfel i, with r_d = z_i - z_{nbr[d][i]} and a symmetric table (a
// neighbour's opposite neighbour is the surfel itself):
//   loss_i = lambda_s / 4 * sum_d r_d^2 + lambda_z * (z_i - zbar_i)^2
//   dL/dz_i = lambda_s * sum_d r_d + 2 lambda_z (z_i - zbar_i)
// (each edge enters the loss from both ends, hence 2 * 2 / K = 1 for K = 4).
// The gradient goes to out_dz (overwritten) or is added to acc_dz; block sums
// of the loss go to part[blockIdx.x] in a fixed order.
__global__ __launch_bounds__(kRegBlock) void k_elev_reg(int n, const float* __restrict__ z,
                                                        const int32_t* __restrict__ nbr,
                                                        float lam_s, const float* __restrict__ zbar,
                                                        float lam_z, float* __restrict__ out_dz,
                                                        float* __restrict__ acc_dz,
                                                        float* __restrict__ part) {
  __shared__ float s_w[kRegBlock / 64];
  const int i = blockIdx.x * kRegBlock + threadIdx.x;
  float l = 0.0f;
  if (i < n) {
    const float zi = z[i];
    float g = 0.0f;
    if (nbr) {
      float s = 0.0f, t = 0.0f;
#pragma unroll
      for (int d = 0; d < 4; ++d) {
        const float r = zi - z[nbr[(size_t)d * n + i]];
        s += r * r;
        t += r;
      }
      l = (lam_s * 0.25f) * s;
      g = lam_s * t;
    }
    if (zbar) {
      const float r = zi - zbar[i];
      l += lam_z * (r * r);
      g += (2.0f * lam_z) * r;
    }
    if (out_dz) out_dz[i] = g;
    if (acc_dz) acc_dz[i] += g;
  }
  for (int o = 32; o > 0; o >>= 1) l += __shfl_xor(l, o, 64);
  if ((threadIdx.x & 63) == 0) s_w[threadIdx.x >> 6] = l;
  __syncthreads();
  if (threadIdx.x == 0) {
    float t = 0.0f;
    for (int w = 0; w < kRegBlock / 64; ++w) t += s_w[w];
    part[blockIdx.x] = t;
  }
}

// Sums the block partials in a fixed order: thread-strided, then a tree.  One
// block, bound by the latency of its strided loads: 1024 threads with four
// loads in flight each instead of one wave with one, 43 -> 7 us over the 11719
// partials of 3M surfels.
constexpr int kRegTotal = 1024;

__global__ __launch_bounds__(kRegTotal) void k_reg_total(const float* __restrict__ part, int nb,
                                                         float* __restrict__ total,
                                                         int accumulate) {
  __shared__ float s_w[kRegTotal / 64];
  float t = 0.0f;
  for (int k = threadIdx.x; k < nb; k += 4 * kRegTotal) {
    float a[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) a[u] = k + u * kRegTotal < nb ? part[k + u * kRegTotal] : 0.0f;
    t += (a[0] + a[1]) + (a[2] + a[3]);
  }
  for (int o = 32; o > 0; o >>= 1) t += __shfl_xor(t, o, 64);
  if ((threadIdx.x & 63) == 0) s_w[threadIdx.x >> 6] = t;
  __syncthreads();
  if (threadIdx.x < 64) {
    t = threadIdx.x < kRegTotal / 64 ? s_w[threadIdx.x] : 0.0f;
    for (int o = 32; o > 0; o >>= 1) t += __shfl_xor(t, o, 64);
    if (threadIdx.x == 0) *total = accumulate ? (*total + t) : t;
  }
}

// Nearest point in the xy-plane: squared distance in binary64 of the binary32
// inputs, ties to the lower point index.  The points are bucketed into a
// uniform grid over the bounding box of surfels and points (about 2 m cells,
// m = point count; the cell size is chosen on the device) and sorted into cell
// order by counting, so the points of neighbouring cells of a row are
// contiguous; a bit per block of 8 x 8 cells says whether it holds a point, and
// each such block has its points' bounding box.
// Each surfel first looks through the 5 x 5 cells around its own, which ends
// the search for surfels among the points.  The others go through the rows of
// blocks outward from their own, in a row the blocks with points outward from
// their own column, found by bit scans: once for the block whose box promises
// the nearest point, then for the blocks whose box reaches inside the best
// distance.  A row, block or cell is left out, and the walk in that direction
// ends, only where its nearest edge lies further than the best distance by
// more than 1e-6 m (the rounding of the cell positions), a box where it lies
// further: the result is the brute-force one.
//
// What costs is a surfel beside the points' band: metres from the nearest point
// it looked into every empty cell of every ring on the way (25000 cells at 7
// m).  600k surfels of a +-15 m road, 1M points in a +-8 m band: rings 16430
// us, rows of cells with a bit per cell 2360 us, rows of blocks 1000 us (the
// lanes of a wave, at distances of 0 to 6 m, visit blocks in different rows, and
// each visit is a chain of loads), with the boxes 327 us.
constexpr int kNNBlock = 256;

struct NNGrid {
  double x0, y0, h, inv_h;
  int32_t W, H;
  int32_t pad[2];
};
static_assert(sizeof(NNGrid) == 48, "grid header");

__device__ __forceinline__ void nn_cell(const NNGrid& g, float x, float y, int& cx, int& cy) {
#pragma clang fp contract(off)
  const double fx = floor(((double)x - g.x0) * g.inv_h);
  const double fy = floor(((double)y - g.y0) * g.inv_h);
  cx = fx < 0.0 ? 0 : (fx > (double)(g.W - 1) ? g.W - 1 : (int)fx);
  cy = fy < 0.0 ? 0 : (fy > (double)(g.H - 1) ? g.H - 1 : (int)fy);
}

// Minimum (x, y) and maximum (z, w) over the wave, in every lane.
__device__ __forceinline__ void bbox_wave(float4& b) {
  for (int o = 32; o > 0; o >>= 1) {
    b.x = fminf(b.x, __shfl_xor(b.x, o, 64)); b.y = fminf(b.y, __shfl_xor(b.y, o, 64));
    b.z = fmaxf(b.z, __shfl_xor(b.z, o, 64)); b.w = fmaxf(b.w, __shfl_xor(b.w, o, 64));
  }
}

// Per-block minimum and maximum of x and y over the surfels and the points.
__global__ __launch_bounds__(kNNBlock) void k_nn_bbox(int n, const float* __restrict__ x,
                                                      const float* __restrict__ y, int m,
                                                      const float* __restrict__ px,
                                                      const float* __restrict__ py,
                                                      float4* __restrict__ part) {
  __shared__ float4 s[kNNBlock / 64];
  float4 b = make_float4(INFINITY, INFINITY, -INFINITY, -INFINITY);
  const int64_t tot = (int64_t)n + m;
  for (int64_t k = (int64_t)blockIdx.x * kNNBlock + threadIdx.x; k < tot;
       k += (int64_t)gridDim.x * kNNBlock) {
    const float u = k < n ? x[k] : px[k - n];
    const float v = k < n ? y[k] : py[k - n];
    b.x = fminf(b.x, u); b.y = fminf(b.y, v); b.z = fmaxf(b.z, u); b.w = fmaxf(b.w, v);
  }
  bbox_wave(b);
  if ((threadIdx.x & 63) == 0) s[threadIdx.x >> 6] = b;
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < kNNBlock / 64; ++w) {
      b.x = fminf(b.x, s[w].x); b.y = fminf(b.y, s[w].y);
      b.z = fmaxf(b.z, s[w].z); b.w = fmaxf(b.w, s[w].w);
    }
    part[blockIdx.x] = b;
  }
}

// The grid over the bounding box (block 0): cell size h with about 2m cells,
// enlarged until W * H <= max_cells.  Every block clears its share of the
// max_cells + 1 cell counters.
__global__ __launch_bounds__(256) void k_nn_grid(const float4* __restrict__ part, int nparts,
                                                 int m, int64_t max_cells,
                                                 NNGrid* __restrict__ g,
                                                 uint32_t* __restrict__ cnt) {
  for (int64_t k = (int64_t)blockIdx.x * 256 + threadIdx.x; k <= max_cells;
       k += (int64_t)gridDim.x * 256)
    cnt[k] = 0u;
  if (blockIdx.x != 0) return;
  __shared__ float4 s[256 / 64];
  float4 a = make_float4(INFINITY, INFINITY, -INFINITY, -INFINITY);
  for (int k = threadIdx.x; k < nparts; k += 256) {
    const float4 q = part[k];
    a.x = fminf(a.x, q.x); a.y = fminf(a.y, q.y); a.z = fmaxf(a.z, q.z); a.w = fmaxf(a.w, q.w);
  }
  bbox_wave(a);
  if ((threadIdx.x & 63) == 0) s[threadIdx.x >> 6] = a;
  __syncthreads();
  if (threadIdx.x == 0) {
    float4 b = s[0];
    for (int w = 1; w < 256 / 64; ++w) {
      b.x = fminf(b.x, s[w].x); b.y = fminf(b.y, s[w].y);
      b.z = fmaxf(b.z, s[w].z); b.w = fmaxf(b.w, s[w].w);
    }
    const double ex = (double)b.z - (double)b.x, ey = (double)b.w - (double)b.y;
    double h = sqrt((ex * ey) / (2.0 * (double)m));
    if (!(h > 0.0)) h = fmax(fmax(ex, ey) / (2.0 * (double)m), 1e-3);
    for (int it = 0; it < 200; ++it) {
      const double w = floor(ex / h) + 1.0, hh = floor(ey / h) + 1.0;
      if (w * hh <= (double)max_cells) break;
      h *= 1.25;
    }
    NNGrid gg;
    gg.x0 = (double)b.x;
    gg.y0 = (double)b.y;
    gg.h = h;
    gg.inv_h = 1.0 / h;
    gg.W = (int32_t)(floor(ex / h) + 1.0);
    gg.H = (int32_t)(floor(ey / h) + 1.0);
    gg.pad[0] = gg.pad[1] = 0;
    *g = gg;
  }
}

// Cell of every point and its rank among the points of its cell.
__global__ __launch_bounds__(kNNBlock) void k_nn_count(int m, const float* __restrict__ px,
                                                       const float* __restrict__ py,
                                                       const NNGrid* __restrict__ g,
                                                       uint32_t* __restrict__ cnt,
                                                       uint32_t* __restrict__ rank) {
  const int k = blockIdx.x * kNNBlock + threadIdx.x;
  if (k >= m) return;
  const NNGrid gg = *g;
  int cx, cy;
  nn_cell(gg, px[k], py[k], cx, cy);
  rank[k] = atomicAdd(&cnt[(int64_t)cy * gg.W + cx], 1u);
}

// Points in cell order: index, x, y at their cell's start plus their rank.
__global__ __launch_bounds__(kNNBlock) void k_nn_scatter(int m, const float* __restrict__ px,
                                                         const float* __restrict__ py,
                                                         const NNGrid* __restrict__ g,
                                                         const uint32_t* __restrict__ start,
                                                         const uint32_t* __restrict__ rank,
                                                         int32_t* __restrict__ sidx,
                                                         float2* __restrict__ sxy) {
  const int k = blockIdx.x * kNNBlock + threadIdx.x;
  if (k >= m) return;
  const NNGrid gg = *g;
  int cx, cy;
  const float u = px[k], v = py[k];
  nn_cell(gg, u, v, cx, cy);
  const uint32_t p = start[(int64_t)cy * gg.W + cx] + rank[k];
  sidx[p] = k;
  sxy[p] = make_float2(u, v);
}

// Blocks of kNNBlk x kNNBlk cells, ceil(W / kNNBlk) to a row.
constexpr int kNNBlk = 8;

__host__ __device__ inline int nn_blocks(int cells) { return (cells + kNNBlk - 1) / kNNBlk; }

// Words of the block bits: a grid of W H <= cells cells has at most
// (W + 7)(H + 7) / 64 <= cells / 8 + 2 blocks.
inline int64_t nn_block_words(int64_t cells) { return (cells / 8 + 2 + 63) / 64 + 1; }

// Per block (linear block index) a bit, whether it holds a point, and if so its
// points' bounding box (min x, min y, max x, max y): 8 lanes to a block, one
// per row of cells, a byte of bits per wave.
__global__ __launch_bounds__(256) void k_nn_blocks(const NNGrid* __restrict__ g,
                                                   const uint32_t* __restrict__ start,
                                                   const float2* __restrict__ sxy, int64_t bytes,
                                                   uint8_t* __restrict__ bits,
                                                   float4* __restrict__ box) {
  const int W = g->W, H = g->H;
  const int wb = nn_blocks(W);
  const int64_t nblk = (int64_t)wb * nn_blocks(H);
  const int lane = threadIdx.x & 63;
  const int64_t wave = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  const int64_t t = wave * 8 + (lane >> 3);
  float4 b = make_float4(INFINITY, INFINITY, -INFINITY, -INFINITY);
  bool any = false;
  if (t < nblk) {
    const int bj = (int)(t / wb), bi = (int)(t - (int64_t)bj * wb);
    const int c0 = bi * kNNBlk, c1 = min(c0 + kNNBlk, W);
    const int j = bj * kNNBlk + (lane & 7);
    if (j < H) {
      const uint32_t e = start[(int64_t)j * W + c1];
      for (uint32_t s = start[(int64_t)j * W + c0]; s < e; ++s) {
        const float2 p = sxy[s];
        b.x = fminf(b.x, p.x); b.y = fminf(b.y, p.y);
        b.z = fmaxf(b.z, p.x); b.w = fmaxf(b.w, p.y);
        any = true;
      }
    }
  }
  for (int o = 1; o < 8; o <<= 1) {
    b.x = fminf(b.x, __shfl_xor(b.x, o, 64)); b.y = fminf(b.y, __shfl_xor(b.y, o, 64));
    b.z = fmaxf(b.z, __shfl_xor(b.z, o, 64)); b.w = fmaxf(b.w, __shfl_xor(b.w, o, 64));
  }
  const unsigned long long m = __ballot(any);
  if ((lane & 7) == 0 && t < nblk && ((m >> lane) & 0xffull)) box[t] = b;
  if (lane == 0 && wave < bytes) {
    uint32_t v = 0u;
#pragma unroll
    for (int k = 0; k < 8; ++k) v |= ((m >> (8 * k)) & 0xffull) ? 1u << k : 0u;
    bits[wave] = (uint8_t)v;
  }
}

constexpr int kNNHeld = 8;          // blocks a surfel lists before it visits them

__global__ __launch_bounds__(kNNBlock) void k_nn_search(int n, const float* __restrict__ x,
                                                        const float* __restrict__ y,
                                                        const NNGrid* __restrict__ g,
                                                        const uint32_t* __restrict__ start,
                                                        const unsigned long long* __restrict__ bits,
                                                        const float4* __restrict__ box,
                                                        const int32_t* __restrict__ sidx,
                                                        const float2* __restrict__ sxy,
                                                        const float* __restrict__ pz,
                                                        float* __restrict__ zbar,
                                                        int32_t* __restrict__ idx) {
#pragma clang fp contract(off)
  __shared__ uint32_t s_held[kNNHeld][kNNBlock];
  const int i = blockIdx.x * kNNBlock + threadIdx.x;
  if (i >= n) return;
  const NNGrid gg = *g;
  const float xf = x[i], yf = y[i];
  const double xi = (double)xf, yi = (double)yf;
  int cx, cy;
  nn_cell(gg, xf, yf, cx, cy);
  const double inf = __longlong_as_double(0x7ff0000000000000ll);
  double best = inf;
  int bi = -1;
  // squared lower bound of the distance to an edge `gap` metres away
  auto bound2 = [&](double gap) __attribute__((always_inline)) {
    const double b = gap - 1e-6;
    return b > 0.0 ? b * b : 0.0;
  };
  auto row_gap2 = [&](int j) __attribute__((always_inline)) {
    return j > cy ? bound2((gg.y0 + (double)j * gg.h) - yi)
                  : j < cy ? bound2(yi - (gg.y0 + (double)(j + 1) * gg.h)) : 0.0;
  };
  // the points [s, e), four loads in flight
  auto points = [&](uint32_t s, uint32_t e) __attribute__((always_inline)) {
#pragma clang fp contract(off)
    for (; s < e; s += 4u) {
      float2 p[4];
#pragma unroll
      for (uint32_t u = 0; u < 4u; ++u) p[u] = sxy[min(s + u, e - 1u)];
#pragma unroll
      for (uint32_t u = 0; u < 4u; ++u) {
        const double dx = xi - (double)p[u].x;
        const double dy = yi - (double)p[u].y;
        const double d2 = dx * dx + dy * dy;
        if (d2 <= best) {             // (a clamped repeat of the last point changes nothing)
          const int k = sidx[min(s + u, e - 1u)];
          if (d2 < best || k < bi) {
            best = d2;
            bi = k;
          }
        }
      }
    }
  };
  // columns c0 ... c1 cut to those that can hold a point as near as the best
  auto cut = [&](int& c0, int& c1) __attribute__((always_inline)) {
    if (!(best < inf)) return;
    const double r = sqrt(best) + 1e-6;
    const double a = floor(((xi - r) - gg.x0) * gg.inv_h), b = floor(((xi + r) - gg.x0) * gg.inv_h);
    if (a > (double)c0) c0 = a > (double)c1 ? c1 + 1 : (int)a;
    if (b < (double)c1) c1 = b < (double)c0 ? c0 - 1 : (int)b;
  };
  // cells of rows j0 ... j1, columns c0 ... c1, each row's range requested
  // before the row ahead of it is looked through
  auto cells = [&](int j0, int j1, int c0, int c1) __attribute__((always_inline)) {
    cut(c0, c1);
    if (c0 > c1 || j0 > j1) return;
    const uint32_t* st = start + (int64_t)j0 * gg.W;
    uint32_t s = st[c0], e = st[c1 + 1];
    for (int j = j0; j <= j1; ++j) {
      if (j < j1) st += gg.W;
      const uint32_t s1 = st[c0], e1 = st[c1 + 1];
      if (s < e && row_gap2(j) <= best) points(s, e);
      s = s1;
      e = e1;
    }
  };
  constexpr int kNear = 2;
  {
    // the own row first: what it finds cuts the columns of the others
    const int a = max(cx - kNear, 0), b = min(cx + kNear, gg.W - 1);
    cells(cy, cy, a, b);
    for (int k = 0; k < 2; ++k)
      cells(k ? cy + 1 : max(cy - kNear, 0), k ? min(cy + kNear, gg.H - 1) : cy - 1, a, b);
  }
  // every point outside those cells is further than kNear cells
  if (!(best < bound2((double)kNear * gg.h))) {
    const int wb = nn_blocks(gg.W), hb = nn_blocks(gg.H);
    const int bx = cx / kNNBlk, by = cy / kNNBlk;
    const double H8 = gg.h * (double)kNNBlk;
    auto block = [&](int64_t t) __attribute__((always_inline)) {
      const int bj = (int)(t / wb), c0 = (int)(t - (int64_t)bj * wb) * kNNBlk;
      cells(bj * kNNBlk, min(bj * kNNBlk + kNNBlk, gg.H) - 1, c0, min(c0 + kNNBlk, gg.W) - 1);
    };
    // first block with points of the row from lo at or right of column c, up
    // to column c1 (beyond: none) ...
    auto next = [&](int64_t lo, int64_t c, int64_t c1) __attribute__((always_inline)) -> int64_t {
      while (c <= c1) {
        const unsigned long long w = bits[(lo + c) >> 6] >> ((lo + c) & 63);
        c += w ? __builtin_ctzll(w) : 64 - ((lo + c) & 63);
        if (w) break;
      }
      return c;
    };
    // ... and at or left of column c, down to column c0
    auto prev = [&](int64_t lo, int64_t c, int64_t c0) __attribute__((always_inline)) -> int64_t {
      while (c >= c0) {
        const unsigned long long w = bits[(lo + c) >> 6] << (63 - ((lo + c) & 63));
        c -= w ? __builtin_clzll(w) : ((lo + c) & 63) + 1;
        if (w) break;
      }
      return c;
    };
    // block rows outward while their squared gap is <= lim, with the columns
    // that can be as near as lim
    auto rows = [&](const double& lim, auto each) __attribute__((always_inline)) {
      auto one = [&](int bj) __attribute__((always_inline)) {
        const int64_t reach = lim < inf ? (int64_t)fmin(sqrt(lim) / H8 + 2.0, (double)wb) : wb;
        each(bj, max(bx - (int)reach, 0), min(bx + (int)reach, wb - 1));
      };
      one(by);
      bool up = true, down = true;
      for (int d = 1; up || down; ++d) {
        up = up && by + d < hb && bound2((gg.y0 + (double)(by + d) * H8) - yi) <= lim;
        if (up) one(by + d);
        down = down && by - d >= 0 && bound2(yi - (gg.y0 + (double)(by - d + 1) * H8)) <= lim;
        if (down) one(by - d);
      }
    };
    // squared distances of a block's box: nearest and furthest.  The points
    // inside give the same expression of offsets no smaller (no larger), so
    // rounding keeps the order.
    auto box_near = [&](int64_t t) __attribute__((always_inline)) {
#pragma clang fp contract(off)
      const float4 b = box[t];
      const double dx = fmax(fmax((double)b.x - xi, xi - (double)b.z), 0.0);
      const double dy = fmax(fmax((double)b.y - yi, yi - (double)b.w), 0.0);
      return dx * dx + dy * dy;
    };
    auto box_far = [&](int64_t t) __attribute__((always_inline)) {
#pragma clang fp contract(off)
      const float4 b = box[t];
      const double dx = fmax(xi - (double)b.x, (double)b.z - xi);
      const double dy = fmax(yi - (double)b.y, (double)b.w - yi);
      return dx * dx + dy * dy;
    };
    double ub = best;
    int64_t first = -1;
    rows(ub, [&](int bj, int c0, int c1) __attribute__((always_inline)) {
      const int64_t lo = (int64_t)bj * wb;
      auto bound = [&](int64_t t) __attribute__((always_inline)) {
        const double u = box_far(t);
        if (u < ub) {
          ub = u;
          first = t;
        }
      };
      const int64_t cr = next(lo, bx, c1), cl = prev(lo, bx - 1, c0);
      if (cr <= c1) bound(lo + cr);
      if (cl >= c0) bound(lo + cl);
    });
    if (first >= 0) block(first);
    // the other blocks are listed first and visited afterwards, so that the
    // lanes of a wave, whose blocks lie in different rows, visit theirs together
    int held = 0;
    auto other = [&](int64_t t) __attribute__((always_inline)) {
      if (t == first || !(box_near(t) <= best)) return;
      if (held < kNNHeld) s_held[held++][threadIdx.x] = (uint32_t)t;
      else block(t);
    };
    rows(best, [&](int bj, int c0, int c1) __attribute__((always_inline)) {
      const int64_t lo = (int64_t)bj * wb;
      for (int64_t c = next(lo, bx, c1); c <= c1; c = next(lo, c + 1, c1)) other(lo + c);
      for (int64_t c = prev(lo, bx - 1, c0); c >= c0; c = prev(lo, c - 1, c0)) other(lo + c);
    });
    for (int k = 0; k < held; ++k) {
      const int64_t t = s_held[k][threadIdx.x];
      if (box_near(t) <= best) block(t);
    }
  }
  zbar[i] = bi >= 0 ? pz[bi] : 0.0f;
  if (idx) idx[i] = bi;
}

// ------------------------------------------------------------ meshgrid layout

// The road mask is one bit per raster cell, a row in ceil(W / 64) words, with
// the exclusive running count of road cells before each word (row-major), so a
// cell's surfel is a word's count plus a bit count: at 1 km of road (11M
// cells) 1.4 + 0.7 MB instead of two 44 MB arrays.
__host__ __device__ inline int row_words(int W) { return W / 64 + (W % 64 != 0); }

__device__ __forceinline__ bool road_cell(const unsigned long long* __restrict__ bits, int wr,
                                          int row, int col) {
  return (bits[(int64_t)row * wr + (col >> 6)] >> (col & 63)) & 1ull;
}

__device__ __forceinline__ int32_t surfel_of(const unsigned long long* __restrict__ bits,
                                             const uint32_t* __restrict__ before, int wr, int row,
                                             int col) {
  const int64_t q = (int64_t)row * wr + (col >> 6);
  return (int32_t)(before[q] + (uint32_t)__popcll(bits[q] & ((1ull << (col & 63)) - 1ull)));
}

// Disk dilation of the pose cells: a thread forms one word (64 cells of a row)
// as the union of the poses' chords there, a block 256 rows of one word column;
// the block first picks the poses whose disk can reach its cells.  Also the
// word's count of road cells.  (Stamping each disk into memory took 170 us for
// 2001 poses of radius 150; this 19 us.)
constexpr int kMaxRadius = 4096;     // the entry point's limit

__global__ __launch_bounds__(256) void k_road_mask(int np, const rogs_pose* __restrict__ poses,
                                                   double x0, double y0, float h, int r, int W,
                                                   int H, int word0, int row0,
                                                   unsigned long long* __restrict__ bits,
                                                   uint32_t* __restrict__ cnt) {
#pragma clang fp contract(off)
  __shared__ int s_half[kMaxRadius + 1];     // half chord at |dy|
  __shared__ int s_cx[256], s_cy[256];
  __shared__ uint32_t s_n;
  const int tid = threadIdx.x;
  for (int dy = tid; dy <= r; dy += 256) {
    // the largest w with w^2 <= r^2 - dy^2
    const int rem = r * r - dy * dy;
    int w = (int)sqrtf((float)rem);
    while (w * w > rem) --w;
    while ((w + 1) * (w + 1) <= rem) ++w;
    s_half[dy] = w;
  }
  const int word = word0 + (int)blockIdx.x;
  const int c0 = word * 64, r0 = row0 + (int)blockIdx.y * 256, row = r0 + tid;
  const int c1 = min(c0 + 63, W - 1), r1 = min(r0 + 255, H - 1);
  unsigned long long m = 0ull;
  for (int k0 = 0; k0 < np; k0 += 256) {
    __syncthreads();                         // the table is built, the list is read
    if (tid == 0) s_n = 0u;
    __syncthreads();
    if (k0 + tid < np) {
      const rogs_pose& p = poses[k0 + tid];
      const int cx = (int)floor(((double)p.x - x0) / (double)h + 0.5);
      const int cy = (int)floor(((double)p.y - y0) / (double)h + 0.5);
      if ((int64_t)cx + r >= c0 && (int64_t)cx - r <= c1 && (int64_t)cy + r >= r0 &&
          (int64_t)cy - r <= r1) {
        const uint32_t at = atomicAdd(&s_n, 1u);     // any order: a union
        s_cx[at] = cx;
        s_cy[at] = cy;
      }
    }
    __syncthreads();
    for (uint32_t k = 0; k < s_n; ++k) {
      const int dy = abs(row - s_cy[k]);
      if (dy > r) continue;
      const int w = s_half[dy];
      const int a = max(s_cx[k] - w, c0) - c0, b = min(s_cx[k] + w, c1) - c0;
      if (a <= b) m |= (~0ull << a) & (~0ull >> (63 - b));
    }
  }
  if (row < H) {
    const int64_t q = (int64_t)row * row_words(W) + word;
    bits[q] = m;
    cnt[q] = (uint32_t)__popcll(m);
  }
}

__device__ __forceinline__ void quat_of(const float* R, float q[4]) {
#pragma clang fp contract(off)
  const double m00 = R[0], m01 = R[1], m02 = R[2], m10 = R[3], m11 = R[4], m12 = R[5],
               m20 = R[6], m21 = R[7], m22 = R[8];
  double w, a, b, d;
  const double tr = m00 + m11 + m22;
  if (tr > 0.0) {
    const double s = sqrt(tr + 1.0) * 2.0;
    w = 0.25 * s; a = (m21 - m12) / s; b = (m02 - m20) / s; d = (m10 - m01) / s;
  } else if (m00 > m11 && m00 > m22) {
    const double s = sqrt(1.0 + m00 - m11 - m22) * 2.0;
    w = (m21 - m12) / s; a = 0.25 * s; b = (m01 + m10) / s; d = (m02 + m20) / s;
  } else if (m11 > m22) {
    const double s = sqrt(1.0 + m11 - m00 - m22) * 2.0;
    w = (m02 - m20) / s; a = (m01 + m10) / s; b = 0.25 * s; d = (m12 + m21) / s;
  } else {
    const double s = sqrt(1.0 + m22 - m00 - m11) * 2.0;
    w = (m10 - m01) / s; a = (m02 + m20) / s; b = (m12 + m21) / s; d = 0.25 * s;
  }
  if (w < 0.0) { w = -w; a = -a; b = -b; d = -d; }
  q[0] = (float)w; q[1] = (float)a; q[2] = (float)b; q[3] = (float)d;
}

// Blocks of 32 x 32 raster cells, four to a thread: road cells get their
// surfel (position, neighbours, Eq. 4 height, rotation of the nearest pose);
// idx = -1 off the road.  The nearest pose of a block's cells is among those
// whose distance to the block's centre exceeds the least such distance by at
// most twice the half diagonal (triangle inequality; the margin covers the
// binary32 cell positions), so a block looks through all poses once and its
// cells through the few candidates, in index order.  2001 poses over 1 km of
// road: 2420 us with every cell through every pose, 112 us this way.
constexpr int kFill = 32;           // side of a block
constexpr int kFillCand = 512;      // candidates kept in LDS; more: every pose
constexpr int kFillHeld = 16;       // poses per thread whose distance stays in registers

__global__ __launch_bounds__(256) void k_layout_fill(int W, int H,
                                                     const unsigned long long* __restrict__ bits,
                                                     const uint32_t* __restrict__ before,
                                                     double x0, double y0, float h, int np,
                                                     const rogs_pose* __restrict__ poses, int64_t n,
                                                     int col0, int row0, int32_t* __restrict__ idx,
                                                     float* __restrict__ x, float* __restrict__ y,
                                                     float* __restrict__ z, float* __restrict__ q,
                                                     int32_t* __restrict__ nbr) {
#pragma clang fp contract(off)
  constexpr int kRows = kFill * kFill / 256;         // cells per thread, kFill / kRows rows apart
  __shared__ double s_d[4];
  __shared__ uint32_t s_w[kFillHeld][4];
  __shared__ int32_t s_k[kFillCand];
  __shared__ double s_x[kFillCand], s_y[kFillCand];
  __shared__ float4 s_q[kFillCand];                  // the candidates' rotations
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int wr = row_words(W);
  const int c0 = (col0 + (int)blockIdx.x) * kFill, r0 = row0 + (int)blockIdx.y * kFill;
  const int col = c0 + tid % kFill, rowt = r0 + tid / kFill;
  uint32_t road = 0u;
#pragma unroll
  for (int u = 0; u < kRows; ++u) {
    const int row = rowt + u * (kFill / kRows);
    if (col < W && row < H) {
      if (road_cell(bits, wr, row, col)) road |= 1u << u;
      else idx[(int64_t)row * W + col] = -1;
    }
  }
  if (!__syncthreads_or((int)road)) return;
  // least squared distance of a pose to the block's centre
  const double cxw = x0 + ((double)c0 + 0.5 * (kFill - 1)) * (double)h;
  const double cyw = y0 + ((double)r0 + 0.5 * (kFill - 1)) * (double)h;
  const double inf = __longlong_as_double(0x7ff0000000000000ll);
  auto dist2 = [&](int k) {
#pragma clang fp contract(off)
    const double dx = cxw - (double)poses[k].x, dy = cyw - (double)poses[k].y;
    return dx * dx + dy * dy;
  };
  double held[kFillHeld], dmin = inf;
#pragma unroll
  for (int u = 0; u < kFillHeld; ++u) {
    const int k = tid + 256 * u;
    held[u] = k < np ? dist2(k) : inf;
    if (held[u] < dmin) dmin = held[u];
  }
  for (int k = tid + 256 * kFillHeld; k < np; k += 256) {
    const double d2 = dist2(k);
    if (d2 < dmin) dmin = d2;
  }
  for (int o = 32; o > 0; o >>= 1) dmin = fmin(dmin, __shfl_xor(dmin, o, 64));
  if (lane == 0) s_d[wv] = dmin;
  __syncthreads();
  dmin = fmin(fmin(s_d[0], s_d[1]), fmin(s_d[2], s_d[3]));
  const double half = 0.5 * (double)h * sqrt(2.0 * kFill * kFill);
  const double reach = sqrt(dmin) + 2.0 * half + 1e-3 + 1e-6 * (fabs(cxw) + fabs(cyw));
  const double reach2 = reach * reach;
  // the candidates in index order, kFillHeld rounds of 256 poses at a time
  uint32_t count = 0;
  for (int k0 = 0; k0 < np && count <= (uint32_t)kFillCand; k0 += 256 * kFillHeld) {
    uint32_t in = 0u, below[kFillHeld];
#pragma unroll
    for (int u = 0; u < kFillHeld; ++u) {
      const int k = k0 + tid + 256 * u;
      const double d2 = k0 == 0 ? held[u] : (k < np ? dist2(k) : inf);
      const bool c = k < np && d2 <= reach2;
      const unsigned long long m = __ballot(c);
      below[u] = (uint32_t)__popcll(m & ((1ull << lane) - 1ull));
      if (c) in |= 1u << u;
      if (lane == 0) s_w[u][wv] = (uint32_t)__popcll(m);
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < kFillHeld; ++u) {
      uint32_t at = count + below[u];
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        if (w < wv) at += s_w[u][w];
        count += s_w[u][w];
      }
      if (((in >> u) & 1u) && at < (uint32_t)kFillCand) {
        const int k = k0 + tid + 256 * u;
        s_k[at] = k;
        s_x[at] = (double)poses[k].x;
        s_y[at] = (double)poses[k].y;
      }
    }
    __syncthreads();
  }
  const bool listed = count <= (uint32_t)kFillCand;
  if (listed) {
    for (uint32_t c = (uint32_t)tid; c < count; c += 256u) {
      float qq[4];
      quat_of(poses[s_k[c]].R, qq);
      s_q[c] = make_float4(qq[0], qq[1], qq[2], qq[3]);
    }
    __syncthreads();
  }
  for (int u = 0; u < kRows; ++u) {
    if (!((road >> u) & 1u)) continue;
    const int row = rowt + u * (kFill / kRows);
    const int32_t i = surfel_of(bits, before, wr, row, col);
    idx[(int64_t)row * W + col] = i;
    const float xi = (float)(x0 + (double)col * (double)h);
    const float yi = (float)(y0 + (double)row * (double)h);
    x[i] = xi;
    y[i] = yi;
    auto at = [&](int rr, int cc) -> int32_t {
      if (rr < 0 || rr >= H || cc < 0 || cc >= W) return i;
      return road_cell(bits, wr, rr, cc) ? surfel_of(bits, before, wr, rr, cc) : i;
    };
    nbr[0 * n + i] = at(row - 1, col);
    nbr[1 * n + i] = at(row + 1, col);
    nbr[2 * n + i] = at(row, col - 1);
    nbr[3 * n + i] = at(row, col + 1);
    double best = inf;
    int bk = 0, bc = -1;
    if (listed) {
      for (uint32_t c = 0; c < count; ++c) {
        const double dx = (double)xi - s_x[c];
        const double dy = (double)yi - s_y[c];
        const double d2 = dx * dx + dy * dy;
        if (d2 < best) {
          best = d2;
          bc = (int)c;
        }
      }
    } else {
      for (int k = 0; k < np; ++k) {
        const double dx = (double)xi - (double)poses[k].x;
        const double dy = (double)yi - (double)poses[k].y;
        const double d2 = dx * dx + dy * dy;
        if (d2 < best) {
          best = d2;
          bk = k;
        }
      }
    }
    if (bc >= 0) bk = s_k[bc];
    const rogs_pose& P = poses[bk];
    const double n31 = P.R[2], n32 = P.R[5], n33 = P.R[8];
    const double t = (n31 * ((double)xi - (double)P.x) + n32 * ((double)yi - (double)P.y)) / n33;
    z[i] = (float)((double)P.z - t);
    float qq[4];
    if (bc >= 0) {
      const float4 t4 = s_q[bc];
      qq[0] = t4.x; qq[1] = t4.y; qq[2] = t4.z; qq[3] = t4.w;
    } else {
      quat_of(P.R, qq);
    }
    for (int c = 0; c < 4; ++c) q[(size_t)c * n + i] = qq[c];
  }
}

}  // namespace

int64_t elev_reg_blocks(int n) { return (n + kRegBlock - 1) / kRegBlock; }

void launch_elev_reg(int n, const float* z, const int32_t* nbr, float lam_s, const float* zbar,
                     float lam_z, float* out_dz, float* acc_dz, float* part, float* total,
                     bool accumulate_total, hipStream_t st) {
  const int nb = (int)elev_reg_blocks(n);
  hipLaunchKernelGGL(k_elev_reg, dim3((unsigned)nb), dim3(kRegBlock), 0, st, n, z, nbr, lam_s,
                     zbar, lam_z, out_dz, acc_dz, part);
  hipLaunchKernelGGL(k_reg_total, dim3(1), dim3(kRegTotal), 0, st, part, nb, total,
                     accumulate_total ? 1 : 0);
}

size_t lidar_scratch_bytes(int n, int m) {
  const int64_t cells = 2 * (int64_t)m + 64;
  const int64_t nparts = std::min<int64_t>(((int64_t)n + m + kNNBlock - 1) / kNNBlock, 1024);
  size_t o = 0;
  auto take = [&](size_t b) { size_t r = o; o = (o + b + 255) / 256 * 256; return r; };
  take(sizeof(NNGrid));
  take(16 * (size_t)nparts);
  take(4 * (size_t)(cells + 2));
  take(4 * scan_tmp_words(cells + 1));
  take(4 * (size_t)m);       // rank
  take(4 * (size_t)m);       // sorted index
  take(8 * (size_t)m);       // sorted x, y
  take(8 * (size_t)nn_block_words(cells));   // blocks with points
  take(16 * 64 * (size_t)nn_block_words(cells));   // their boxes
  return o;
}

void launch_lidar_nn(int n, const float* x, const float* y, int m, const float* px,
                     const float* py, const float* pz, float* zbar, int32_t* idx, void* scratch,
                     hipStream_t st) {
  const int64_t cells = 2 * (int64_t)m + 64;
  const int64_t nparts = std::min<int64_t>(((int64_t)n + m + kNNBlock - 1) / kNNBlock, 1024);
  size_t o = 0;
  auto take = [&](size_t b) { size_t r = o; o = (o + b + 255) / 256 * 256; return r; };
  char* base = static_cast<char*>(scratch);
  NNGrid* g = reinterpret_cast<NNGrid*>(base + take(sizeof(NNGrid)));
  float4* part = reinterpret_cast<float4*>(base + take(16 * (size_t)nparts));
  uint32_t* cnt = reinterpret_cast<uint32_t*>(base + take(4 * (size_t)(cells + 2)));
  uint32_t* tmp = reinterpret_cast<uint32_t*>(base + take(4 * scan_tmp_words(cells + 1)));
  uint32_t* rank = reinterpret_cast<uint32_t*>(base + take(4 * (size_t)m));
  int32_t* sidx = reinterpret_cast<int32_t*>(base + take(4 * (size_t)m));
  float2* sxy = reinterpret_cast<float2*>(base + take(8 * (size_t)m));
  unsigned long long* bits =
      reinterpret_cast<unsigned long long*>(base + take(8 * (size_t)nn_block_words(cells)));
  float4* box = reinterpret_cast<float4*>(base + take(16 * 64 * (size_t)nn_block_words(cells)));
  hipLaunchKernelGGL(k_nn_bbox, dim3((unsigned)nparts), dim3(kNNBlock), 0, st, n, x, y, m, px, py,
                     part);
  const unsigned cb = (unsigned)std::min<int64_t>((cells + 1 + 2047) / 2048, 4096);
  hipLaunchKernelGGL(k_nn_grid, dim3(cb), dim3(256), 0, st, part, (int)nparts, m, cells, g, cnt);
  const unsigned pb = (unsigned)((m + kNNBlock - 1) / kNNBlock);
  hipLaunchKernelGGL(k_nn_count, dim3(pb), dim3(kNNBlock), 0, st, m, px, py, g, cnt, rank);
  // cells beyond the grid's W * H hold zeros: the scan runs over the bound
  scan_u32(cnt, cnt, cells + 1, nullptr, tmp, st);
  hipLaunchKernelGGL(k_nn_scatter, dim3(pb), dim3(kNNBlock), 0, st, m, px, py, g, cnt, rank, sidx,
                     sxy);
  const int64_t words = nn_block_words(cells);
  hipLaunchKernelGGL(k_nn_blocks, dim3((unsigned)(2 * words)), dim3(256), 0, st, g, cnt, sxy,
                     8 * words, reinterpret_cast<uint8_t*>(bits), box);
  hipLaunchKernelGGL(k_nn_search, dim3((unsigned)((n + kNNBlock - 1) / kNNBlock)), dim3(kNNBlock),
                     0, st, n, x, y, g, cnt, bits, box, sidx, sxy, pz, zbar, idx);
}

// Scratch of the layout: the mask words, the counts before each, the scan's
// sums and the total (the last 256 bytes).
struct LayoutScratch {
  int64_t words;
  size_t o_bits, o_before, o_tmp, o_total, total;
};

static LayoutScratch layout_scratch(int W, int H) {
  LayoutScratch s{};
  s.words = (int64_t)row_words(W) * H;
  size_t o = 0;
  auto take = [&](size_t b) { size_t r = o; o += (b + 255) / 256 * 256; return r; };
  s.o_bits = take(8 * (size_t)s.words);
  s.o_before = take(4 * (size_t)s.words);
  s.o_tmp = take(4 * scan_tmp_words(s.words));
  s.o_total = take(256);
  s.total = o;
  return s;
}

size_t layout_scratch_bytes(int W, int H, int np) {
  (void)np;
  return layout_scratch(W, H).total;
}

// gx columns of blocks of `side` rows, as parts of at most 65535 rows of blocks
// (the grid's y extent) and fewer than 2^32 threads to a row: launch(grid, first
// column of blocks, first row).
template <typename Launch>
static void bands(int64_t gx, int H, int side, Launch launch) {
  const int64_t gy = ((int64_t)H + side - 1) / side;
  for (int64_t b = 0; b < gy; b += 65535)
    launch_bands(gx, 256, [&](int64_t first, unsigned n) {
      launch(dim3(n, (unsigned)std::min<int64_t>(gy - b, 65535)), (int)first, (int)(b * side));
    });
}

void launch_layout_mask(const rogs_pose* poses, int np, double x0, double y0, float h, int W,
                        int H, int r, void* scratch, uint32_t* n_dev, hipStream_t st) {
  const LayoutScratch s = layout_scratch(W, H);
  uint8_t* base = static_cast<uint8_t*>(scratch);
  uint32_t* before = reinterpret_cast<uint32_t*>(base + s.o_before);
  bands(row_words(W), H, 256, [&](dim3 grid, int word0, int row0) {
    hipLaunchKernelGGL(k_road_mask, grid, dim3(256), 0, st, np, poses, x0, y0, h, r, W, H, word0,
                       row0, reinterpret_cast<unsigned long long*>(base + s.o_bits), before);
  });
  scan_u32(before, before, s.words, n_dev, reinterpret_cast<uint32_t*>(base + s.o_tmp), st);
}

void launch_layout_fill(const rogs_pose* poses, int np, double x0, double y0, float h, int W,
                        int H, void* scratch, int64_t n, int32_t* idx, float* x, float* y,
                        float* z, float* q, int32_t* nbr, hipStream_t st) {
  const LayoutScratch s = layout_scratch(W, H);
  const uint8_t* base = static_cast<const uint8_t*>(scratch);
  bands(((int64_t)W + kFill - 1) / kFill, H, kFill, [&](dim3 grid, int col0, int row0) {
    hipLaunchKernelGGL(k_layout_fill, grid, dim3(256), 0, st, W, H,
                       reinterpret_cast<const unsigned long long*>(base + s.o_bits),
                       reinterpret_cast<const uint32_t*>(base + s.o_before), x0, y0, h, np, poses,
                       n, col0, row0, idx, x, y, z, q, nbr);
  });
}

}  // namespace rogs

extern "C" {

size_t rogs_elev_scratch_bytes(int32_t n) {
  return n < 1 ? 0 : (size_t)(rogs::elev_reg_blocks(n) + 1) * 4;
}

int rogs_elev_loss(rogs_ctx* c, int32_t n, const float* z, const int32_t* nbr, float lambda_smooth,
                   const float* zbar, float lambda_z, float* dz, float* loss_out, void* scratch,
                   size_t scratch_bytes, void* stream) {
  if (!c) return ROGS_EINVAL;
  if (n < 1 || !z || !dz || !loss_out || !scratch)
    return rogs::ctx_fail(c, ROGS_EINVAL, "rogs_elev_loss: null argument or n < 1");
  if (scratch_bytes < rogs_elev_scratch_bytes(n))
    return rogs::ctx_fail(c, ROGS_ENOMEM, "rogs_elev_loss: scratch too small");
  if ((nbr && !std::isfinite(lambda_smooth)) || (zbar && !std::isfinite(lambda_z)))
    return rogs::ctx_fail(c, ROGS_EINVAL, "rogs_elev_loss: weights must be finite");
  if (!nbr && !zbar) return ROGS_OK;
  hipStream_t st = static_cast<hipStream_t>(stream);
  float* part = static_cast<float*>(scratch);
  rogs::launch_elev_reg(n, z, nbr, lambda_smooth, zbar, lambda_z, nullptr, dz, part, loss_out,
                        true, st);
  hipError_t e = hipGetLastError();
  return e == hipSuccess ? ROGS_OK
                         : rogs::ctx_fail(c, ROGS_EHIP, std::string("rogs_elev_loss: ") +
                                                            hipGetErrorString(e));
}

int rogs_elev_loss_static(rogs_ctx* c, int32_t n, const float* z, const int32_t* nbr,
                          float lambda_smooth, const float* zbar, float lambda_z, float* dz,
                          float* loss_out, void* stream) {
  if (!c) return ROGS_EINVAL;
  if (n < 1 || !z || !dz || !loss_out)
    return rogs::ctx_fail(c, ROGS_EINVAL, "rogs_elev_loss_static: null argument or n < 1");
  if (n > ROGS_ELEV_STATIC_MAX_N)
    return rogs::ctx_fail(c, ROGS_EINVAL,
                          "rogs_elev_loss_static: n exceeds ROGS_ELEV_STATIC_MAX_N (" +
                              std::to_string(ROGS_ELEV_STATIC_MAX_N) + ")");
  if ((nbr && !std::isfinite(lambda_smooth)) || (zbar && !std::isfinite(lambda_z)))
    return rogs::ctx_fail(c, ROGS_EINVAL, "rogs_elev_loss_static: weights must be finite");
  // the array's device address, looked up once per device with that device current
  static std::mutex mu;
  static void* addr[64] = {};
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess)
    return rogs::ctx_fail(c, ROGS_EHIP, std::string("rogs_elev_loss_static: hipGetDevice: ") +
                                            hipGetErrorString(e));
  if (dev < 0 || dev >= 64)
    return rogs::ctx_fail(c, ROGS_EINVAL, "rogs_elev_loss_static: device ordinal above 63");
  void* part = nullptr;
  {
    std::lock_guard<std::mutex> lock(mu);
    if (!addr[dev]) {
      void* p = nullptr;
      e = hipGetSymbolAddress(&p, HIP_SYMBOL(rogs::scratch));
      if (e != hipSuccess || !p)
        return rogs::ctx_fail(c, ROGS_EHIP,
                              std::string("rogs_elev_loss_static: hipGetSymbolAddress: ") +
                                  hipGetErrorString(e));
      addr[dev] = p;
    }
    part = addr[dev];
  }
  if (!nbr && !zbar) return ROGS_OK;
  // every block overwrites its own partial before the total reads it: nothing
  // in the array needs clearing between calls
  rogs::launch_elev_reg(n, z, nbr, lambda_smooth, zbar, lambda_z, nullptr, dz,
                        static_cast<float*>(part), loss_out, true,
                        static_cast<hipStream_t>(stream));
  e = hipGetLastError();
  return e == hipSuccess ? ROGS_OK
                         : rogs::ctx_fail(c, ROGS_EHIP, std::string("rogs_elev_loss_static: ") +
                                                            hipGetErrorString(e));
}

size_t rogs_lidar_scratch_bytes(int32_t n, int32_t m) {
  if (n < 1 || m < 1) return 0;
  return rogs::lidar_scratch_bytes(n, m);
}

int rogs_lidar_targets(rogs_ctx* c, int32_t n, const float* x, const float* y, int32_t m,
                       const float* px, const float* py, const float* pz, float* zbar,
                       int32_t* idx, void* scratch, size_t scratch_bytes, void* stream) {
  if (!c) return ROGS_EINVAL;
  if (n < 1 || m < 1 || !x || !y || !px || !py || !pz || !zbar || !scratch)
    return rogs::ctx_fail(c, ROGS_EINVAL, "rogs_lidar_targets: null argument or empty set");
  if (m > (1 << 29))
    return rogs::ctx_fail(c, ROGS_EINVAL, "rogs_lidar_targets: at most 2^29 points");
  if (reinterpret_cast<uintptr_t>(scratch) % 256 != 0)
    return rogs::ctx_fail(c, ROGS_EINVAL, "rogs_lidar_targets: scratch must be 256-byte aligned");
  if (scratch_bytes < rogs_lidar_scratch_bytes(n, m))
    return rogs::ctx_fail(c, ROGS_ENOMEM, "rogs_lidar_targets: scratch too small");
  rogs::launch_lidar_nn(n, x, y, m, px, py, pz, zbar, idx, scratch,
                        static_cast<hipStream_t>(stream));
  hipError_t e = hipGetLastError();
  return e == hipSuccess ? ROGS_OK
                         : rogs::ctx_fail(c, ROGS_EHIP, std::string("rogs_lidar_targets: ") +
                                                            hipGetErrorString(e));
}

size_t rogs_meshgrid_scratch_bytes(int32_t W, int32_t H, int32_t n_poses) {
  if (W < 1 || H < 1 || n_poses < 1) return 0;
  return rogs::layout_scratch_bytes(W, H, n_poses);
}

int rogs_meshgrid_layout(rogs_ctx* c, const rogs_pose* poses, int32_t n_poses, double x0,
                         double y0, float spacing, int32_t W, int32_t H, int32_t radius_px,
                         int32_t* idx, int64_t capacity, float* x, float* y, float* z, float* q,
                         int32_t* nbr, int64_t* n_out, void* scratch, size_t scratch_bytes,
                         void* stream) {
  if (!c) return ROGS_EINVAL;
  if (!poses || n_poses < 1 || W < 1 || H < 1 || (int64_t)W * H >= (int64_t(1) << 31) ||
      radius_px < 0 || radius_px > rogs::kMaxRadius || !(spacing > 0.0f) || !std::isfinite(x0) ||
      !std::isfinite(y0) || !n_out || !scratch || capacity < 0)
    return rogs::ctx_fail(c, ROGS_EINVAL, "rogs_meshgrid_layout: invalid argument");
  const size_t need = rogs::layout_scratch_bytes(W, H, n_poses);
  if (scratch_bytes < need) return rogs::ctx_fail(c, ROGS_ENOMEM, "rogs_meshgrid_layout: scratch too small");
  const bool query = capacity == 0 && !idx && !x && !y && !z && !q && !nbr;
  if (!query && (!idx || !x || !y || !z || !q || !nbr))
    return rogs::ctx_fail(c, ROGS_EINVAL, "rogs_meshgrid_layout: null output array");
  hipStream_t st = static_cast<hipStream_t>(stream);
  uint32_t* n_dev = reinterpret_cast<uint32_t*>(static_cast<uint8_t*>(scratch) + need - 256);
  rogs::launch_layout_mask(poses, n_poses, x0, y0, spacing, W, H, radius_px, scratch, n_dev, st);
  uint32_t n_host = 0;
  hipError_t e = hipMemcpyAsync(&n_host, n_dev, 4, hipMemcpyDeviceToHost, st);
  if (e == hipSuccess) e = hipStreamSynchronize(st);
  if (e != hipSuccess)
    return rogs::ctx_fail(c, ROGS_EHIP, std::string("rogs_meshgrid_layout: ") + hipGetErrorString(e));
  *n_out = (int64_t)n_host;
  if (query) return ROGS_OK;
  if ((int64_t)n_host > capacity)
    return rogs::ctx_fail(c, ROGS_ECAPACITY, "rogs_meshgrid_layout: " + std::to_string(n_host) +
                                                 " road cells exceed the capacity");
  rogs::launch_layout_fill(poses, n_poses, x0, y0, spacing, W, H, scratch, capacity, idx, x, y, z,
                           q, nbr, st);
  e = hipGetLastError();
  return e == hipSuccess ? ROGS_OK
                         : rogs::ctx_fail(c, ROGS_EHIP, std::string("rogs_meshgrid_layout: ") +
                                                            hipGetErrorString(e));
}

}  // extern "C"
