// Front-to-back alpha compositing of the sorted tile lists (Eq. 6) and its
// adjoint.
//
// Mapping: one 64-lane wave per 64 pixels (one pixel per lane), tiles launched
// longest list first.  A tile of 64 pixels is one wave; a tile of 128 or 256
// pixels is a block of 2 or 4 waves, each with a part of tile_w x (64 /
// tile_w) pixels.  A wave starts from one precomputed record (tile, list
// range, view) and reads each entry's slot directly, so the prologue is two
// dependent global loads before the records arrive.  Entries are staged in
// LDS (projection record + the surfel's colour/semantic features), then every
// lane walks them in order.  A pixel stops after the surfel that takes its
// transmittance below t_eps; the wave leaves the list once all of its pixels
// have stopped.
//
// What bounds a large tile is the serial walk of its list: far from the
// camera a 16 x 16 tile lists thousands of sub-pixel footprints, and the
// launch ends with the longest list.  Splitting the tile's pixels over waves
// (instead of 4 pixels per lane) makes an entry four times shorter, and the
// test of each entry against the wave's own pixels (part_reached) leaves out
// the half or more that reach other parts only.  Measured with 16 x 16 tiles,
// 4 pixels per lane in one wave -> four waves with the test: 200k surfels x 6
// views of 1600 x 900, C = 8: forward 563 -> 213 us, backward 666 -> 429 us,
// fused step 918 -> 515 us; a 640 x 360 colour view of 3M surfels, C = 16:
// forward 1029 -> 317 us.  One-wave tiles keep the untested walk in the fused
// step and the backward: there at most 4 % of the entries a wave visits reach
// none of its pixels, less than the test costs.
//
// Depth is composited relative to a reference depth t0 per pixel, the depth
// of the first (nearest) list entry that reaches the pixel: D' = sum w (t_z -
// t0), D = D' + t0 A.  The backward differentiates D' and A, so the FP32
// suffix term below cancels in proportion to the spread of the depths a pixel
// sees instead of the absolute depth (tens of metres).  The entries a pixel
// sees, and so t0, do not depend on the tile shape.
//
// The backward walks the list front to back again, recomputing T exactly as
// the forward did, and uses sum_{j>k} w_j f_j = O - prefix - w_k f_k for the
// suffix term of dO/d(alpha_k).  Per (tile, pair) it writes one record of
// 10 + C gradient values at the pair's emission index: the five moments of
// dL/dq over the pixel offsets and dalpha are summed across the wave with a
// reduce-scatter; the colour, semantic and depth gradients sum_p w_p G_p are
// a small matrix product per 16 entries on the matrix cores.  The projection
// adjoint later sums each surfel's records and applies the conic.  No
// atomics: the result does not depend on timing.
//
// The fused training step runs forward, loss and backward of a tile in one
// kernel (k_render_step): the per-pixel loss gradient, G.O, T_final and n_last
// stay in registers between the two passes instead of going through HBM, and
// a list the forward staged whole is not staged again.
#include <type_traits>
#include <cfloat>

#include "rogs_internal.h"

namespace rogs {

namespace {

__device__ __forceinline__ int find_view(const ViewDev* __restrict__ views, int V, int gt) {
  int lo = 0, hi = V - 1;
  while (lo < hi) {
    int mid = (lo + hi + 1) >> 1;
    if (views[mid].tile_off <= gt) lo = mid; else hi = mid - 1;
  }
  return lo;
}


// List entries staged in LDS at a time: the template parameter KS of the
// compositing kernels, 16, 32 or 64 (rogs_render_opts.stage).

// Per-wave constants of the compositing kernels: the tile and the 64 pixels of
// it that this wave (part `part` of the tile) renders, one per lane.
struct TileGeom {
  int gt, v, W, H, px, py, part;
  float pxc, pyc;
  float xa, xb, ya, yb;      // centres of the part's first and last pixel column and row
  uint32_t rbeg, rend, sbase;
  const ViewDev* vw;
};

__device__ __forceinline__ TileGeom tile_geom(const ViewDev* __restrict__ views, int N,
                                              const uint4* __restrict__ tinfo, int part) {
  TileGeom t;
  const int lane = threadIdx.x & 63;
  // tile, list begin, list end, view | tile row << kViewBits
  const uint4 ti = tinfo[blockIdx.x];
  t.gt = (int)ti.x;
  t.v = (int)(ti.w & ((1u << kViewBits) - 1u));
  t.vw = &views[t.v];
  t.W = t.vw->w;
  t.H = t.vw->h;
  const int lt = t.gt - t.vw->tile_off;
  const int ty = (int)(ti.w >> kViewBits), tx = lt - ty * t.vw->tiles_x;
  const int tw = t.vw->tw, th = t.vw->th;
  const int sh = __builtin_ctz((unsigned)tw);      // tile_w divides 64: a power of two
  const int rows = 64 >> sh;
  const int x0 = tx * tw, y0 = ty * th + part * rows;
  t.part = part;
  t.px = x0 + (lane & (tw - 1));
  t.py = y0 + (lane >> sh);
  t.pxc = (float)t.px + 0.5f;
  t.pyc = (float)t.py + 0.5f;
  t.xa = (float)x0 + 0.5f;
  t.xb = (float)(x0 + tw - 1) + 0.5f;
  t.ya = (float)y0 + 0.5f;
  t.yb = (float)(y0 + rows - 1) + 0.5f;
  t.rbeg = ti.y;
  t.rend = ti.z;
  t.sbase = (uint32_t)t.v * (uint32_t)N;
  return t;
}

// Whether an entry's footprint q <= q_cut can reach the pixel centres of a
// part: false only if no pixel of the part passes the binary32 test, so
// leaving the entry out changes no bit of the part.  The least value of the
// quadratic form over the part's rectangle lies on the side facing the centre
// in x or in y (or is 0 inside), with the other offset at its best value on
// that side.  It is compared with the row spans' inflated cut, four times as
// wide, q_cut (1 + 2^-16 / (1 - rho)): the binary32 rounding of the form,
// here and in the pixel test, is below 2^-19 q / (1 - rho).  Entries whose
// conic is too thin for that bound (1 - rho < 2^-12, axis ratio above ~90) or
// out of its range are kept.
__device__ __forceinline__ bool part_reached(const TileGeom& tg, const float4 r0, const float4 r1,
                                             float qcut) {
  const float A = r1.x, B2 = r1.y, C = r1.z;
  const float lx = pixel_offset(tg.xa, r0.x, r0.z), hx = pixel_offset(tg.xb, r0.x, r0.z);
  const float ly = pixel_offset(tg.ya, r0.y, r0.w), hy = pixel_offset(tg.yb, r0.y, r0.w);
  const float dxn = fminf(fmaxf(lx, 0.0f), hx), dyn = fminf(fmaxf(ly, 0.0f), hy);
  const float nb = -0.5f * B2;
  const float dy1 = fminf(fmaxf(ly, nb * dxn * __builtin_amdgcn_rcpf(C)), hy);
  const float dx2 = fminf(fmaxf(lx, nb * dyn * __builtin_amdgcn_rcpf(A)), hx);
  const float q1 = pixel_q32(A, B2, C, dxn, dy1);
  const float q2 = pixel_q32(A, B2, C, dx2, dyn);
  const float ac = A * C;
  const float gap = 1.0f - fabsf(nb) * __builtin_amdgcn_rsqf(ac);
  const bool sure = gap >= 0x1p-12f && ac > 1e-24f && ac < 1e12f;
  const float thr = qcut * (1.0f + 0x1p-16f * __builtin_amdgcn_rcpf(gap));
  return !sure || !(q1 > thr && q2 > thr);
}

typedef float vec4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ float4 to_float4(const vec4 v) {
  return make_float4(v.x, v.y, v.z, v.w);
}

// Orders this wave's LDS writes before its later LDS reads (a wave-private
// region: no barrier between waves).
__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Stages list entries [base, base + cnt) of the tile in LDS: the projection
// record (with 2B in place of B) and the surfel's feature record, entry j at
// s_r0[j (2 + FS4)], s_r1[j (2 + FS4)] and s_f[j (2 + FS4) + f] of one
// interleaved array (so one address serves all of an entry's reads).  With
// kE, returns this lane's emission index (lane < cnt).
template <int FS4, bool kE>
__device__ __forceinline__ uint32_t stage_entries(uint32_t base, int cnt, uint32_t sbase,
                                                  const uint32_t* __restrict__ vals,
                                                  const uint32_t* __restrict__ spair,
                                                  const float4* __restrict__ rec,
                                                  const float4* __restrict__ feat, float4* s_r0,
                                                  float4* s_r1, float4* s_f) {
  const int lane = threadIdx.x;
  uint32_t e = 0;
  if (lane < cnt) {
    if (kE) e = vals[base + lane];
    const uint32_t slot = spair[base + lane];
    s_r0[lane * (2 + FS4)] = rec[2 * (size_t)slot];
    const float4 r1 = rec[2 * (size_t)slot + 1];
    s_r1[lane * (2 + FS4)] = make_float4(r1.x, 2.0f * r1.y, r1.z, r1.w);   // A, 2B, C, t_z
    const uint32_t i = slot - sbase;
#pragma unroll
    for (int f = 0; f < FS4; ++f) s_f[lane * (2 + FS4) + f] = feat[(size_t)i * FS4 + f];
  }
  return e;
}

// The forward state of a pixel (Eq. 6): acc = sum w f (features, then with kD
// the relative depth sum w (t_z - t0)), the transmittance T and nl = the walked
// entries up to the one that stopped the pixel.  With kD, t0 = the depth of the
// pixel's first contributing entry: the list is in ascending depth, so the
// running minimum of the contributing depths (FLT_MAX while none).
template <int C>
struct Pixel {
  float acc[3 + C + 1];
  float T, t0;
  uint32_t nl;
};

template <int C>
__device__ __forceinline__ void pixel_start(const TileGeom& tg, Pixel<C>& p) {
  // a pixel is live while T >= t_eps (T only falls, and t_eps < 1); a pixel
  // outside the image starts at T = 0, which no update changes
  p.T = (tg.px < tg.W && tg.py < tg.H) ? 1.0f : 0.0f;
  p.nl = 0;
  p.t0 = FLT_MAX;
#pragma unroll
  for (int f = 0; f <= 3 + C; ++f) p.acc[f] = 0.0f;
}

// The quadratic form of an entry (u_hi v_hi u_lo v_lo | A 2B C tz) at a pixel
// and its exponential: the part of the entry that does not wait for the
// entries before it.
__device__ __forceinline__ float entry_weight(const TileGeom& tg, const float4 r0, const float4 r1,
                                              float& q) {
#pragma clang fp contract(off)
  const float dx = pixel_offset(tg.pxc, r0.x, r0.z);
  const float dy = pixel_offset(tg.pyc, r0.y, r0.w);
  q = pixel_q32(r1.x, r1.y, r1.z, dx, dy);
  return gauss_weight(q);
}

// Adds a staged entry with quadratic form q and exponential ge to a pixel;
// returns its footprint weight g.
template <int C, bool kD, bool kSem>
__device__ __forceinline__ float entry_add(const float4* s, float tz, float ge, float q,
                                           float qcut, float amax, float teps, Pixel<C>& p) {
#pragma clang fp contract(off)
  constexpr int F = 3 + C;            // composited features besides depth
  constexpr int FS4 = (F + 4) / 4;    // float4 per feature record (features, alpha)
  float fv[FS4 * 4];
#pragma unroll
  for (int f = 0; f < FS4; ++f) {
    const float4 t4 = s[2 + f];
    fv[4 * f] = t4.x; fv[4 * f + 1] = t4.y; fv[4 * f + 2] = t4.z; fv[4 * f + 3] = t4.w;
  }
  const bool live = p.T >= teps;
  const bool hit = live && q <= qcut;
  const float g = hit ? ge : 0.0f;
  const float a = clamp_alpha(fv[F] * g, amax);
  const float w = a * p.T;
#pragma unroll
  for (int f = 0; f < (kSem ? F : 3); ++f) p.acc[f] = __builtin_fmaf(w, fv[f], p.acc[f]);
  if (kD) {
    p.t0 = hit ? fminf(p.t0, tz) : p.t0;
    p.acc[F] = __builtin_fmaf(w, tz - p.t0, p.acc[F]);
  }
  p.T -= w;                     // T (1 - alpha)
  // entries walked while live: at the entry that stops the pixel, its place
  // among the walked ones plus one
  p.nl += live ? 1u : 0u;
  return g;
}

// One staged list entry for a pixel; returns its footprint weight g.  The
// semantic sums are formed with kSem only, the depth sum with kD; T, nl and
// the order of operations do not depend on it.
// Lanes whose pixel the entry does not reach, or has stopped, run the same
// arithmetic with g = 0: w = 0 leaves T and the sums as they are (T >= 0 and
// every feature is finite), so the result is that of a branch around the
// update without its exec-mask bookkeeping.
template <int C, bool kD, bool kSem>
__device__ __forceinline__ float entry_forward(const TileGeom& tg, const float4* s, float qcut,
                                               float amax, float teps, Pixel<C>& p) {
  // every multiply-add is written out: the forward rounds the same in every
  // kernel it is inlined into
#pragma clang fp contract(off)
  const float4 r1 = s[1];             // A 2B C tz
  float q;
  // the exponential of every lane, then a select (no branch around it)
  const float ge = entry_weight(tg, s[0], r1, q);
  return entry_add<C, kD, kSem>(s, r1.w, ge, q, qcut, amax, teps, p);
}

// Whether every pixel of the wave has stopped (every lane runs this together).
template <int C>
__device__ __forceinline__ bool all_stopped(const Pixel<C>& p, float teps) {
  return __builtin_amdgcn_ballot_w64(p.T >= teps) == 0;
}

constexpr int kFwdUnroll = 4;       // forward entries per stop test

// Forward pass of a one-wave tile (64 pixels) over its list, KS staged entries
// at a time.  e_first = this lane's emission index in the first staged batch.
// With kG (16) the footprint weights g of the list's first kG entries are kept
// in gsave for the backward: gsave[j] is the weight of every entry the forward
// evaluates, which covers each pixel's entries before n_last, the only ones
// the backward reads it for, and 0 for the others (past the list's end or
// after the whole wave has stopped).
template <int C, int KS, int kG>
__device__ __forceinline__ void forward_tile(const TileGeom& tg, float qcut, float amax,
                                             float teps, const uint32_t* __restrict__ vals,
                                             const uint32_t* __restrict__ spair,
                                             const float4* __restrict__ rec,
                                             const float4* __restrict__ feat, float4* s_st,
                                             Pixel<C>& p, uint32_t& e_first,
                                             float* gsave) {
  static_assert(kG == 0 || (kG == 16 && KS >= kG), "kept weights");
  constexpr int FS4 = (3 + C + 4) / 4;
  constexpr int ES = 2 + FS4;
  pixel_start<C>(tg, p);
  bool stop_all = false;
  for (uint32_t base = tg.rbeg; base < tg.rend && !stop_all; base += KS) {
    const int cnt = (int)min((uint32_t)KS, tg.rend - base);
    const uint32_t e = stage_entries<FS4, true>(base, cnt, tg.sbase, vals, spair, rec, feat, s_st,
                                                s_st + 1, s_st + 2);
    if (base == tg.rbeg) e_first = e;
    __syncthreads();
    // groups of kFwdUnroll entries, the stop test after each group: entries
    // past a pixel's stop change nothing for it, so the results are those
    // of a test after every entry.  The first kG entries of the list are
    // unrolled whole, so that their weights land in registers.
    // (a constant trip count without early exits: it unrolls fully)
    int jstart = 0;
    if (kG > 0 && base == tg.rbeg) {
#pragma unroll
      for (int j = 0; j < kG; ++j) {
        if (j < cnt && !stop_all) {
          gsave[j] = entry_forward<C, false, true>(tg, s_st + j * ES, qcut, amax, teps, p);
          if (j % kFwdUnroll == kFwdUnroll - 1 && all_stopped<C>(p, teps)) stop_all = true;
        } else {
          gsave[j] = 0.0f;
        }
      }
      jstart = kG;
    }
    for (int j0 = jstart; j0 < cnt && !stop_all; j0 += kFwdUnroll) {
#pragma unroll
      for (int u = 0; u < kFwdUnroll; ++u) {
        const int j = j0 + u;
        if (j >= cnt) break;
        (void)entry_forward<C, false, true>(tg, s_st + j * ES, qcut, amax, teps, p);
      }
      if (all_stopped<C>(p, teps)) stop_all = true;
    }
    __syncthreads();
  }
}

// Forward pass of one part (wave) of a tile over the tile's list, 64 entries
// at a time: every lane tests one entry against the part (part_reached) and
// the entries that reach it are staged side by side in the wave's own LDS
// region, so the waves of a tile share no barrier and each walks only the
// entries that its own 64 pixels can see.  A launch ends with its longest
// lists, one wave on a SIMD that waits for each load and each result: the
// projection records are requested two batches ahead and the feature records
// one ahead, and the entries are walked in groups of kFwdUnroll whose
// footprints are evaluated side by side before the chain of their
// transmittances.  Measured with the channel test out of the entry loop
// (branches there kept the loads from overlapping, 445 cycles per entry in the
// longest list): a 640 x 360 view of 3M surfels, 16 classes, 318 -> 186 us;
// 12 views of 400k surfels, lists up to 4400 entries, 625 -> 367 us; the four
// chunks of a 1.2M-surfel export 354 -> 317 us.
template <int C, bool kD>
__device__ __forceinline__ void forward_part(const TileGeom& tg, float qcut, float amax,
                                             float teps, const uint32_t* __restrict__ spair,
                                             const float4* __restrict__ rec,
                                             const float4* __restrict__ feat, float4* s_st,
                                             uint32_t* s_pos, Pixel<C>& p, bool sem) {
  constexpr int FS4 = (3 + C + 4) / 4;
  constexpr int ES = 2 + FS4;
  const uint32_t lane = threadIdx.x & 63;
  pixel_start<C>(tg, p);
  if (all_stopped<C>(p, teps)) return;      // a part outside the image
  const uint32_t len = tg.rend - tg.rbeg;
  const uint32_t* sp = spair + tg.rbeg;
  const vec4* rv = reinterpret_cast<const vec4*>(rec);
  const vec4* fv = reinterpret_cast<const vec4*>(feat);
  vec4* st = reinterpret_cast<vec4*>(s_st);
  // the present batch (r0, r1, fr), the next one (n0, n1) and the slots of the
  // next and the one after it
  vec4 r0 = {0.0f, 0.0f, 0.0f, 0.0f}, r1 = r0, n0 = r0, n1 = r0, fr[FS4];
#pragma unroll
  for (int f = 0; f < FS4; ++f) fr[f] = r0;
  uint32_t slot = 0, slot1 = 0, slot2 = 0;
  if (lane < len) {
    slot = sp[lane];
    r0 = rv[2 * (size_t)slot];
    r1 = rv[2 * (size_t)slot + 1];
  }
  if (lane + 64u < len) {
    slot1 = sp[lane + 64u];
    n0 = rv[2 * (size_t)slot1];
    n1 = rv[2 * (size_t)slot1 + 1];
  }
  if (lane + 128u < len) slot2 = sp[lane + 128u];
  r1.y *= 2.0f;                                          // A, 2B, C, t_z
  bool in = lane < len && part_reached(tg, to_float4(r0), to_float4(r1), qcut);
  if (in) {
#pragma unroll
    for (int f = 0; f < FS4; ++f) fr[f] = fv[(size_t)(slot - tg.sbase) * FS4 + f];
  }
  for (uint32_t base = 0; base < len; base += 64u) {
    const unsigned long long m = __builtin_amdgcn_ballot_w64(in);
    const int n = (int)__popcll(m);
    if (in) {
      const int j = (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32),
                                                   __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
      vec4* s = st + j * ES;
      s[0] = r0;
      s[1] = r1;
#pragma unroll
      for (int f = 0; f < FS4; ++f) s[2 + f] = fr[f];
      s_pos[j] = base + lane + 1u;
    }
    if (base + 64u < len) {
      r0 = n0;
      r1 = n1;
      r1.y *= 2.0f;
      in = base + 64u + lane < len && part_reached(tg, to_float4(r0), to_float4(r1), qcut);
      if (in) {
#pragma unroll
        for (int f = 0; f < FS4; ++f) fr[f] = fv[(size_t)(slot1 - tg.sbase) * FS4 + f];
      }
      slot1 = slot2;
      if (base + 128u + lane < len) {
        n0 = rv[2 * (size_t)slot1];
        n1 = rv[2 * (size_t)slot1 + 1];
      }
      if (base + 192u + lane < len) slot2 = sp[base + 192u + lane];
    }
    wave_lds_sync();
    bool stop = false;
    const bool was_live = p.T >= teps;
    const uint32_t nl = p.nl;
    p.nl = 0;
    auto walk = [&](auto with_sem) __attribute__((always_inline)) {
      constexpr bool kSem = decltype(with_sem)::value;
      int j0 = 0;
      for (; j0 + kFwdUnroll <= n && !stop; j0 += kFwdUnroll) {
        const float4* s = s_st + j0 * ES;
        float ge[kFwdUnroll], q[kFwdUnroll], tz[kFwdUnroll];
#pragma unroll
        for (int u = 0; u < kFwdUnroll; ++u) {
          const float4 e1 = s[u * ES + 1];
          tz[u] = e1.w;
          ge[u] = entry_weight(tg, s[u * ES], e1, q[u]);
        }
#pragma unroll
        for (int u = 0; u < kFwdUnroll; ++u)
          (void)entry_add<C, kD, kSem>(s + u * ES, tz[u], ge[u], q[u], qcut, amax, teps, p);
        stop = all_stopped<C>(p, teps);
      }
      for (; j0 < n && !stop; ++j0)
        (void)entry_forward<C, kD, kSem>(tg, s_st + j0 * ES, qcut, amax, teps, p);
      stop = stop || all_stopped<C>(p, teps);
    };
    // (a branch within the entries would keep their loads from overlapping)
    if (sem)
      walk(std::true_type{});
    else
      walk(std::false_type{});
    // a pixel that stopped here: its stopping entry's place in the tile's list
    p.nl = was_live && p.T < teps ? s_pos[p.nl - 1u] : nl;
    wave_lds_sync();
    if (stop) break;
  }
}

typedef float mfma_f4 __attribute__((ext_vector_type(4)));

// Floats of a wave's LDS block for one block of 16 list entries: the
// per-pixel weights w of 16 entries (rows of 64 + 4 floats), also used once
// per tile to transpose the per-pixel gradient vectors, 16 columns at a time
// (rows of 16 + 1 floats).
constexpr int kWRow = 64 + 4;
constexpr int kWFloats = 16 * kWRow;
static_assert(kWFloats >= 64 * 17, "transpose space");

// Column blocks of 16 of the feature and depth gradients.
template <int C>
constexpr int kNFB() { return (3 + C + 1 + 15) / 16; }

// Feature and depth gradients of 16 list entries as one matrix product on the
// matrix cores: D[m][n] = sum over the wave's pixels p of w[m][p] *
// gamma[p][n], where gamma[p] = (dL/dfeatures, dL/dD) of pixel p.
// v_mfma_f32_16x16x4_f32 takes A[m][k] from lane m + 16k, B[k][n] from lane
// n + 16k and returns D[4g + i][n] in lane n + 16g, element i.  The k-th
// step of 4 covers pixels kgrp * 16 + c, so a lane reads its A operands as 16
// contiguous floats of its entry's row.
template <int C>
__device__ __forceinline__ void feature_product(const float* s_w, const float (&bG)[kNFB<C>()][16],
                                                mfma_f4 (&acc)[kNFB<C>()]) {
  const int lane = threadIdx.x & 63;
  const int mrow = lane & 15, kgrp = lane >> 4;
  float a[16];
  const float4* ap = reinterpret_cast<const float4*>(s_w + mrow * kWRow + kgrp * 16);
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const float4 t = ap[q];
    a[4 * q] = t.x; a[4 * q + 1] = t.y; a[4 * q + 2] = t.z; a[4 * q + 3] = t.w;
  }
#pragma unroll
  for (int nb = 0; nb < kNFB<C>(); ++nb) {
    acc[nb] = mfma_f4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int c = 0; c < 16; ++c)
      acc[nb] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[c], bG[nb][c], acc[nb], 0, 0, 0);
  }
}

// The products of a one-wave tile's entries, row m < nrows to its record s_e[m].
template <int C>
__device__ __forceinline__ void feature_gemm(const float* s_w, const uint32_t* s_e, int nrows,
                                             const float (&bG)[kNFB<C>()][16],
                                             float* __restrict__ gpair) {
  constexpr int F = 3 + C;
  constexpr uint32_t GS = grad_stride_c(C);
  const int lane = threadIdx.x & 63;
  const int mrow = lane & 15, kgrp = lane >> 4;
  uint32_t e4[4];
  bool ok[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int m = 4 * kgrp + i;
    ok[i] = m < nrows;
    e4[i] = s_e[m];
  }
  mfma_f4 acc[kNFB<C>()];
  feature_product<C>(s_w, bG, acc);
#pragma unroll
  for (int nb = 0; nb < kNFB<C>(); ++nb) {
    const int n = nb * 16 + mrow;
    if (n <= F) {
      const int col = n < F ? 7 + n : 6;       // record: ..., dt_z (6), features (7 ...)
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if (ok[i]) gpair[(size_t)e4[i] * GS + col] = acc[nb][i];
    }
  }
}

// A part's share of 16 entries' products, row m at s_w[m NF] over the weight
// rows that were read.
template <int C>
__device__ __forceinline__ void feature_share(float* s_w, const float (&bG)[kNFB<C>()][16]) {
  constexpr int NF = 16 * kNFB<C>();
  const int lane = threadIdx.x & 63;
  const int mrow = lane & 15, kgrp = lane >> 4;
  mfma_f4 acc[kNFB<C>()];
  feature_product<C>(s_w, bG, acc);
  wave_lds_sync();
#pragma unroll
  for (int nb = 0; nb < kNFB<C>(); ++nb)
#pragma unroll
    for (int i = 0; i < 4; ++i) s_w[(4 * kgrp + i) * NF + nb * 16 + mrow] = acc[nb][i];
}

// A pixel's inputs of the backward: the output gradient Gv (features, depth,
// alpha), G.O (with the relative depth D'), T_final, n_last and the reference
// depth t0 (used with kDA).
template <int C>
struct PixelGrad {
  float Gv[3 + C + 2];
  float GO, Tf, t0;
  uint32_t nl;
};

// The backward's running state of a pixel: the transmittance and the prefix
// sum of w gf over the entries so far, and the alpha channel's gradient term.
struct PixelBack {
  float T, Spre, GAf;
};

template <int C, bool kDA>
__device__ __forceinline__ PixelBack back_start(const PixelGrad<C>& pg) {
#pragma clang fp contract(off)
  constexpr int F = 3 + C;
  PixelBack b;
  b.T = 1.0f;
  b.Spre = 0.0f;
  // D = D' + t0 A: the alpha channel's gradient carries t0 dL/dD, times
  // T_final for dA/d(alpha_k) = T_final / (1 - alpha_k)
  b.GAf = kDA ? __builtin_fmaf(pg.t0, pg.Gv[F], pg.Gv[F + 1]) * pg.Tf : 0.0f;
  return b;
}

// B operand of feature_gemm: gamma[pixel][n] for pixel kgrp * 16 + c,
// transposed through the wave's LDS block.
template <int C>
__device__ __forceinline__ void transpose_grad(const PixelGrad<C>& pg, float* s_w,
                                               float (&bG)[kNFB<C>()][16]) {
  constexpr int F = 3 + C;
  const int lane = threadIdx.x & 63;
  const int mrow = lane & 15, kgrp = lane >> 4;
#pragma unroll
  for (int nb = 0; nb < kNFB<C>(); ++nb) {
    float* row = s_w + lane * 17;
#pragma unroll
    for (int n = 0; n < 16; ++n) row[n] = 16 * nb + n <= F ? pg.Gv[16 * nb + n] : 0.0f;
    wave_lds_sync();
#pragma unroll
    for (int c = 0; c < 16; ++c) bG[nb][c] = s_w[(kgrp * 16 + c) * 17 + mrow];
    wave_lds_sync();
  }
}

// Backward entries evaluated side by side: what the registers of 4 waves per
// SIMD hold without spilling.
template <int C>
constexpr int kBackUnroll() { return C <= 3 ? 4 : 2; }
constexpr int kReduced = 6;     // gradient values per entry summed across the tile

// What a staged list entry brings to a pixel with footprint weight g whatever
// came before it: alpha, w's gradient gf = G . (features, relative depth), 1 /
// (1 - alpha) and g where alpha depends on it (not clamped).
struct BackEntry {
  float a, gf, inv, g;
};

template <int C, bool kDA>
__device__ __forceinline__ BackEntry back_entry(const float* fv, float tz, float g, float amax,
                                                const PixelGrad<C>& pg) {
  // every multiply-add is written out: the backward rounds the same in the
  // fused step and in the stand-alone backward
#pragma clang fp contract(off)
  constexpr int F = 3 + C;
  BackEntry k;
  const float araw = fv[F] * g;
  k.a = clamp_alpha(araw, amax);
  k.gf = kDA ? pg.Gv[F] * (tz - pg.t0) : 0.0f;
#pragma unroll
  for (int f = 0; f < F; ++f) k.gf = __builtin_fmaf(pg.Gv[f], fv[f], k.gf);
  k.inv = __builtin_amdgcn_rcpf(1.0f - k.a);
  // the clamp cuts alpha's dependence on g: gda = g da is dL/d(alpha)
  // where it does not hold (0 where it does), and dL/dq = -(alpha / 2)
  // gda, the factor -alpha / 2 being applied to the slot's sums by
  // the projection adjoint
  k.g = araw > amax ? 0.0f : g;
  return k;
}

// The entry's weight w and gda = g dL/d(alpha g) after the entries before it.
template <bool kDA>
__device__ __forceinline__ float back_add(const BackEntry& k, PixelBack& b, float GO, float& gda) {
#pragma clang fp contract(off)
  const float w = k.a * b.T;
  // the suffix G.O - sum over entries up to this one of w gf
  b.Spre = __builtin_fmaf(w, k.gf, b.Spre);
  const float suffix = GO - b.Spre;
  float da = __builtin_fmaf(b.T, k.gf, -(suffix * k.inv));
  if (kDA) da = __builtin_fmaf(b.GAf, k.inv, da);
  gda = k.g * da;
  b.T -= w;                       // as in the forward
  return w;
}

// One staged list entry of the backward for a pixel with footprint weight g
// (0 where the entry does not reach it): its weight w and gda = g dL/d(alpha
// g) = alpha dL/d(alpha), so that dL/dq = -(alpha / 2) gda.
// Lanes whose pixel the pair does not reach run the same arithmetic with
// g = 0: alpha = w = 0, T and the prefix unchanged, terms +-0 (a pair that
// reaches no pixel of the wave gets a zero record this way; a branch around
// it would copy T and the prefix on every entry).
template <int C, bool kDA>
__device__ __forceinline__ float entry_backward(const float* fv, float tz, float g, float amax,
                                                const PixelGrad<C>& pg, PixelBack& b, float& gda) {
  return back_add<kDA>(back_entry<C, kDA>(fv, tz, g, amax, pg), b, pg.GO, gda);
}

// Adds a pixel's moments of gda over the pixel offsets and gda itself (pv = 0
// before the first: fma(x, y, 0) rounds as x y); the projection adjoint turns
// a slot's sums into dL/d(u, v, A, B, C) with the pair's conic.
__device__ __forceinline__ void add_moments(float gda, float dx, float dy, float (&pv)[kReduced]) {
#pragma clang fp contract(off)
  const float gx = gda * dx, gy = gda * dy;
  pv[5] += gda;
  pv[0] += gx;
  pv[1] += gy;
  pv[2] = __builtin_fmaf(gx, dx, pv[2]);
  pv[3] = __builtin_fmaf(gx, dy, pv[3]);
  pv[4] = __builtin_fmaf(gy, dy, pv[4]);
}

template <int FS4>
__device__ __forceinline__ void load_features(const float4* s, float* fv) {
#pragma unroll
  for (int f = 0; f < FS4; ++f) {
    const float4 t4 = s[2 + f];
    fv[4 * f] = t4.x; fv[4 * f + 1] = t4.y; fv[4 * f + 2] = t4.z; fv[4 * f + 3] = t4.w;
  }
}

// Backward pass of a one-wave tile (64 pixels) over its list.  Writes one
// record of NV gradient values per pair at its emission index: the five
// moments and dalpha are summed across the wave with a reduce-scatter, the
// feature and depth gradients come from feature_gemm once per 16 entries.
// With kG (16) gsave holds the forward's footprint weights of the list's
// first kG entries, valid for the entries before n_last.
template <int C, int KS, bool kDA, int kG>
__device__ __forceinline__ void backward_tile(const TileGeom& tg, float qcut, float amax,
                                              const uint32_t* __restrict__ vals,
                                              const uint32_t* __restrict__ spair,
                                              const float4* __restrict__ rec,
                                              const float4* __restrict__ feat, float4* s_st,
                                              float* s_w, uint32_t* s_e, const PixelGrad<C>& pg,
                                              float* __restrict__ gpair, bool staged,
                                              uint32_t e_pre, const float* gsave) {
  static_assert(kG == 0 || (kG == 16 && KS >= kG), "kept weights");
  constexpr int F = 3 + C;
  constexpr int FS4 = (F + 4) / 4;
  constexpr int ES = 2 + FS4;
  constexpr int NV = 10 + C;
  constexpr uint32_t GS = grad_stride_c(C);   // floats per record
  constexpr int NR = kReduced;
  const int lane = threadIdx.x;
  const int my_comp = rs_comp(lane, NR);
  const bool writer = my_comp >= 0 && (lane & rs_dup_bits(NR)) == 0;
  PixelBack b = back_start<C, kDA>(pg);
  // every lane holds the maximum: as a scalar the list loop is scalar control
  const uint32_t maxn = (uint32_t)__builtin_amdgcn_readfirstlane((int)wave_max_u32(pg.nl));
  const uint32_t stop = tg.rbeg + min(maxn, tg.rend - tg.rbeg);
  // not needed when no entry is visited
  float bG[kNFB<C>()][16];
  if (stop > tg.rbeg) transpose_grad<C>(pg, s_w, bG);
  // this lane's column of the reduced values in every record: lanes that
  // hold a copy of a component write the same bits to the same address, and
  // where the record has padding, the lanes without a component write
  // theirs into its first padding column, so the store needs no lane mask
  constexpr bool kPadCol = GS > (uint32_t)NV;
  float* const gcol = gpair + (my_comp >= 0 ? my_comp : (kPadCol ? NV : 0));
  for (uint32_t base = tg.rbeg; base < stop; base += KS) {
    const int cnt = __builtin_amdgcn_readfirstlane((int)min((uint32_t)KS, stop - base));
    // a list the forward staged whole is still in LDS
    const uint32_t e_mine =
        staged ? e_pre
               : stage_entries<FS4, true>(base, cnt, tg.sbase, vals, spair, rec, feat, s_st,
                                          s_st + 1, s_st + 2);
    if (lane < KS) s_e[lane] = e_mine;
    __syncthreads();
    // blocks of 16 entries: the per-entry pass, then their feature gradients
    for (int j0 = 0; j0 < cnt; j0 += 16) {
      const int j1 = min(j0 + 16, cnt);
      // two entries per iteration (immediate LDS offsets, half the loop
      // bookkeeping); the second is skipped past the block's end
      // gk: the pixel's kept weight of entry j, or nullptr
      auto entry = [&](const int j, const float* gk) {
#pragma clang fp contract(off)
        const uint32_t idx = base - tg.rbeg + (uint32_t)j;
        const uint32_t e = (uint32_t)__builtin_amdgcn_readlane((int)e_mine, j);
        const float4* s = s_st + j * ES;
        const float4 r0 = s[0], r1 = s[1];
        const float dx = pixel_offset(tg.pxc, r0.x, r0.z);
        const float dy = pixel_offset(tg.pyc, r0.y, r0.w);
        float g;
        if (gk) {
          g = idx < pg.nl ? *gk : 0.0f;
        } else {
          const float q = pixel_q32(r1.x, r1.y, r1.z, dx, dy);
          const float ge = gauss_weight(q);
          g = (idx < pg.nl && q <= qcut) ? ge : 0.0f;
        }
        float fv[FS4 * 4];
        load_features<FS4>(s, fv);
        float gda;
        s_w[(j - j0) * kWRow + lane] = entry_backward<C, kDA>(fv, r1.w, g, amax, pg, b, gda);
        const float gx = gda * dx, gy = gda * dy;
        const float pv[NR] = {gx, gy, gx * dx, gx * dy, gy * dy, gda};
        const float tot = wave_reduce_scatter<NR>(pv, lane);
        if (kPadCol || writer) gcol[(size_t)e * GS] = tot;
      };
      if (kG > 0 && base == tg.rbeg && j0 == 0) {
        // the list's first block, unrolled whole so that the kept weights
        // are read from registers
#pragma unroll
        for (int j = 0; j < kG; ++j)
          if (j < j1) entry(j, gsave + j);
      } else {
        for (int j = j0; j < j1; j += 2) {
          entry(j, nullptr);
          if (j + 1 < j1) entry(j + 1, nullptr);
        }
      }
      __syncthreads();
      feature_gemm<C>(s_w, s_e + j0, j1 - j0, bG, gpair);
      __syncthreads();
    }
    __syncthreads();
  }
  // pairs that no pixel of the tile reached contribute nothing
  for (uint32_t p = stop + lane; p < tg.rend; p += 64) {
    const uint32_t e = vals[p];
    for (int c = 0; c < NV; ++c) gpair[(size_t)e * GS + c] = 0.0f;
  }
}

// LDS of a tile of NW waves (parts) in the backward: the staged entries; per
// wave the weight rows of a block of 16 entries, then its share of their
// feature gradients; the gda of all the tile's pixels for the block; per wave
// which staged entries reach it.  A one-wave tile has its weight rows only.
template <int C, int NW, int KS>
struct alignas(16) BlockLds {
  float4 st[KS * (2 + (3 + C + 4) / 4)];
  float w[NW][kWFloats];
  float g[NW == 1 ? 4 : 16 * 64 * NW];
  unsigned long long mask[NW];
  uint32_t e[KS];
  uint32_t maxn[NW];
};

// Backward pass of a tile of NW waves, in blocks of 16 list entries and two
// phases.  First every wave walks the entries for its own pixels, leaving out
// those that do not reach its part (lane j has tested entry j): it leaves each
// pixel's gda in LDS and forms its part's share of the feature gradients on
// the matrix cores.  Then the waves share the block's records: each takes
// 16 / NW entries and reduces their moments, over the parts first, per lane,
// then across the lanes (the order of one wave with NW pixels per lane), and
// the features' shares are added in part order.  So the reduce-scatter runs
// once per entry, not once per part, and a part that an entry does not reach
// costs nothing.  Like the forward, a launch ends with single blocks whose
// waves wait for every result, so entries are staged one batch ahead and
// evaluated side by side: 12 views of 400k surfels 1220 -> 1034 us, 3 views of
// 40k 273 -> 232 us.  (An entry of one part reduced by its own wave at once,
// with barriers only for shared entries: 1422 us, as the wave with most
// entries is the chain.)
template <int C, int NW, int KS, bool kDA>
__device__ __forceinline__ void backward_block(const TileGeom& tg, float qcut, float amax,
                                               const uint32_t* __restrict__ vals,
                                               const uint32_t* __restrict__ spair,
                                               const float4* __restrict__ rec,
                                               const float4* __restrict__ feat,
                                               BlockLds<C, NW, KS>& L, const PixelGrad<C>& pg,
                                               float* __restrict__ gpair) {
#pragma clang fp contract(off)
  constexpr int F = 3 + C;
  constexpr int FS4 = (F + 4) / 4;
  constexpr int ES = 2 + FS4;
  constexpr int NV = 10 + C;
  constexpr uint32_t GS = grad_stride_c(C);
  constexpr int NR = kReduced;
  constexpr int NT = 64 * NW;
  constexpr int NF = 16 * kNFB<C>();                 // columns of a share of the features
  static_assert(16 * NF <= kWFloats, "feature shares over the weight rows");
  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int my_comp = rs_comp(lane, NR);
  constexpr bool kPadCol = GS > (uint32_t)NV;
  const bool writer = kPadCol || (my_comp >= 0 && (lane & rs_dup_bits(NR)) == 0);
  float* const gcol = gpair + (my_comp >= 0 ? my_comp : (kPadCol ? NV : 0));
  float* const s_w = L.w[wv];
  PixelBack b = back_start<C, kDA>(pg);
  const uint32_t my_max = (uint32_t)__builtin_amdgcn_readfirstlane((int)wave_max_u32(pg.nl));
  if (lane == 0) L.maxn[wv] = my_max;
  __syncthreads();
  uint32_t maxn = 0;
#pragma unroll
  for (int w = 0; w < NW; ++w) maxn = max(maxn, L.maxn[w]);
  const uint32_t stop =
      tg.rbeg + min((uint32_t)__builtin_amdgcn_readfirstlane((int)maxn), tg.rend - tg.rbeg);
  float bG[kNFB<C>()][16];
  if (my_max > 0u) transpose_grad<C>(pg, s_w, bG);
  // rows between a lane's pixels of two parts
  const float drow = (float)(64 >> __builtin_ctz((unsigned)tg.vw->tw));
  const float py0 = tg.pyc - (float)tg.part * drow;      // exact: halves below 2^15
  // the next KS entries and the slots of the KS after them are requested while
  // the present ones are walked: this thread's are float4 tid + k NT of ES each
  constexpr int NP = (KS * ES + NT - 1) / NT;
  vec4 nx[NP];
  uint32_t nslot[NP], ne = 0;
  auto request_slots = [&](uint32_t from) __attribute__((always_inline)) {
#pragma unroll
    for (int k = 0; k < NP; ++k) {
      const uint32_t j = (uint32_t)(tid + k * NT) / ES;
      nslot[k] = j < (uint32_t)KS && from + j < stop ? spair[from + j] : 0u;
    }
  };
  auto request_entries = [&](uint32_t from) __attribute__((always_inline)) {
#pragma unroll
    for (int k = 0; k < NP; ++k) {
      const uint32_t t = (uint32_t)(tid + k * NT), j = t / ES, c = t - j * ES;
      nx[k] = vec4{0.0f, 0.0f, 0.0f, 0.0f};
      if (j < (uint32_t)KS && from + j < stop)
        nx[k] = c < 2 ? reinterpret_cast<const vec4*>(rec)[2 * (size_t)nslot[k] + c]
                      : reinterpret_cast<const vec4*>(feat)[(size_t)(nslot[k] - tg.sbase) * FS4 +
                                                            (c - 2)];
    }
    ne = tid < KS && from + (uint32_t)tid < stop ? vals[from + tid] : 0u;
  };
  if (tg.rbeg < stop) {
    request_slots(tg.rbeg);
    request_entries(tg.rbeg);
    request_slots(tg.rbeg + KS);
  }
  for (uint32_t base = tg.rbeg; base < stop; base += KS) {
    const int cnt = (int)min((uint32_t)KS, stop - base);
    if (tid < KS) L.e[tid] = ne;
#pragma unroll
    for (int k = 0; k < NP; ++k) {
      const int t = tid + k * NT;
      if (t % ES == 1) nx[k].y *= 2.0f;                   // A, 2B, C, t_z
      if (t < KS * ES) reinterpret_cast<vec4*>(L.st)[t] = nx[k];
    }
    request_entries(base + KS);
    request_slots(base + 2 * KS);
    __syncthreads();
    const uint32_t seen = base - tg.rbeg;
    const bool in = lane < cnt && seen + (uint32_t)lane < my_max &&
                    part_reached(tg, L.st[min(lane, KS - 1) * ES], L.st[min(lane, KS - 1) * ES + 1],
                                 qcut);
    const unsigned long long mine = __builtin_amdgcn_ballot_w64(in);
    if (lane == 0) L.mask[wv] = mine;
    for (int j0 = 0; j0 < cnt; j0 += 16) {
      const int n = min(16, cnt - j0);
      const uint32_t m16 = (uint32_t)(mine >> j0) & 0xffffu;
      // groups of K entries: what does not wait for the entries before is
      // evaluated side by side, then the chain of the transmittances
      auto walk = [&](auto kc, uint32_t& m) __attribute__((always_inline)) {
        constexpr int K = decltype(kc)::value;
        int i[K];
        BackEntry be[K];
#pragma unroll
        for (int u = 0; u < K; ++u) {
          i[u] = __builtin_ctz(m);
          m &= m - 1u;
        }
#pragma unroll
        for (int u = 0; u < K; ++u) {
          const float4* s = L.st + (j0 + i[u]) * ES;
          const float4 r1 = s[1];
          float q;
          const float ge = entry_weight(tg, s[0], r1, q);
          const float g = (seen + (uint32_t)(j0 + i[u]) < pg.nl && q <= qcut) ? ge : 0.0f;
          float fv[FS4 * 4];
          load_features<FS4>(s, fv);
          be[u] = back_entry<C, kDA>(fv, r1.w, g, amax, pg);
        }
#pragma unroll
        for (int u = 0; u < K; ++u) {
          float gda;
          s_w[i[u] * kWRow + lane] = back_add<kDA>(be[u], b, pg.GO, gda);
          L.g[i[u] * NT + tid] = gda;
        }
      };
      uint32_t m = m16;
      for (int c = __builtin_popcount(m16); c >= kBackUnroll<C>(); c -= kBackUnroll<C>())
        walk(std::integral_constant<int, kBackUnroll<C>()>{}, m);
      while (m) walk(std::integral_constant<int, 1>{}, m);
      if (m16) {
        wave_lds_sync();
        // (rows of entries that do not reach the part hold leftovers: their
        // results are not read)
        feature_share<C>(s_w, bG);
      }
      __syncthreads();
      // the parts that each entry reaches
      uint32_t part16[NW];
#pragma unroll
      for (int w = 0; w < NW; ++w)
        part16[w] = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(L.mask[w] >> j0)) &
                    0xffffu;
      // kB entries side by side: those of one part each, whose sums are that
      // part's, or general ones, where the parts that an entry does not reach
      // are left out (their rows hold leftovers): their share would be +0, which
      // changes no bit of a sum that starts at +0.  Entries past n add nothing and store nothing.
      constexpr int kB = 4;
      for (int i0 = wv; i0 < n; i0 += kB * NW) {
        float pv[kB][NR], fs[kB], tot[kB];
        int only[kB];                                    // the entry's one part
        bool single = true;
#pragma unroll
        for (int u = 0; u < kB; ++u) {
          const int i = min(i0 + u * NW, 15);
          int parts = 0;
          only[u] = 0;
#pragma unroll
          for (int w = 0; w < NW; ++w) {
            const int on = (int)((part16[w] >> i) & 1u);
            parts += on;
            only[u] = on ? w : only[u];
          }
          single = single && (parts == 1 || i0 + u * NW >= n);
#pragma unroll
          for (int c = 0; c < NR; ++c) pv[u][c] = 0.0f;
        }
        if (single) {
#pragma unroll
          for (int u = 0; u < kB; ++u) {
            const int i = min(i0 + u * NW, 15);
            const float4 r0 = L.st[(j0 + i) * ES];
            const float gda = L.g[i * NT + 64 * only[u] + lane];
            fs[u] = L.w[only[u]][i * NF + min(lane, F)];
            add_moments(gda, pixel_offset(tg.pxc, r0.x, r0.z),
                        pixel_offset(py0 + (float)only[u] * drow, r0.y, r0.w), pv[u]);
          }
        } else {
#pragma unroll
          for (int u = 0; u < kB; ++u) {
            const int i = min(i0 + u * NW, 15);
            const float4 r0 = L.st[(j0 + i) * ES];
            const float dx = pixel_offset(tg.pxc, r0.x, r0.z);
            fs[u] = 0.0f;                                // lane = feature column
#pragma unroll
            for (int w = 0; w < NW; ++w) {
              if (!((part16[w] >> i) & 1u)) continue;
              add_moments(L.g[i * NT + 64 * w + lane], dx,
                          pixel_offset(py0 + (float)w * drow, r0.y, r0.w), pv[u]);
              fs[u] += L.w[w][i * NF + min(lane, F)];
            }
          }
        }
#pragma unroll
        for (int u = 0; u < kB; ++u) tot[u] = wave_reduce_scatter<NR>(pv[u], lane);
#pragma unroll
        for (int u = 0; u < kB; ++u) {
          const int i = i0 + u * NW;
          if (i >= n) break;
          const size_t e = (size_t)L.e[j0 + i] * GS;
          if (writer) gcol[e] = tot[u];
          // record: ..., dt_z (6), features (7 ...)
          if (lane <= F) gpair[e + (lane < F ? 7 + lane : 6)] = fs[u];
        }
      }
      __syncthreads();
    }
  }
  // pairs that no pixel of the tile reached contribute nothing
  constexpr uint32_t Q = GS / 4;
  const uint32_t nz = (tg.rend - stop) * Q;
  for (uint32_t t = (uint32_t)tid; t < nz; t += NT) {
    const uint32_t j = t / Q;
    reinterpret_cast<float4*>(gpair)[(size_t)vals[stop + j] * Q + (t - j * Q)] =
        make_float4(0.0f, 0.0f, 0.0f, 0.0f);
  }
}

// Forward compositing of the batch: of the 5 + C output planes per view the
// ones selected by mask and the view's own channel set, and, when all are
// selected and tfin is given, per pixel T_final, n_last, the relative depth D'
// and its reference t0 for the backward.  out = nullptr: each view's planes go
// straight into the view's own output, with the elevation if selected (copied
// there from images in the arena, 8 served views of 1600 x 900 took 489 us
// more, an export of 24 M pixels 66 us).  One wave per 64 pixels; the waves of
// a tile form a block (their records meet in one CU's cache) and are
// independent.
template <int C, int NW>
__global__ __launch_bounds__(64 * NW) void k_render_fwd(
    const ViewDev* __restrict__ views, int V, int N, float qcut, float amax,
    float teps, const uint4* __restrict__ tinfo, const uint32_t* __restrict__ spair,
    const float4* __restrict__ rec, const float4* __restrict__ feat, float* __restrict__ out,
    float* __restrict__ tfin, uint32_t* __restrict__ nlast, float2* __restrict__ drel,
    uint32_t mask, const ViewOutDev* __restrict__ outs, int64_t plane, int64_t row) {
  constexpr int F = 3 + C;
  constexpr int FS4 = (F + 4) / 4;
  constexpr int NO = 5 + C;           // output channels
  // staged entries: projection record, conic, features, one record per entry
  __shared__ float4 s_st[NW][64 * (2 + FS4)];
  __shared__ uint32_t s_pos[NW][64];
  const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const TileGeom tg = tile_geom(views, N, tinfo, wv);
  const uint32_t want = tg.vw->ch & mask;
  // elevation is formed from depth and alpha
  const uint32_t ch = want & ROGS_CH_ELEV ? want | ROGS_CH_D | ROGS_CH_A : want;
  constexpr uint32_t kPlanes = ROGS_CH_RGB | ROGS_CH_SEM | ROGS_CH_D | ROGS_CH_A;
  Pixel<C> p;
  forward_part<C, true>(tg, qcut, amax, teps, spair, rec, feat, s_st[wv], s_pos[wv], p,
                        (ch & ROGS_CH_SEM) != 0u);
  if (!(tg.px < tg.W && tg.py < tg.H)) return;
  const uint32_t len = tg.rend - tg.rbeg;
  const size_t pix = (size_t)tg.py * tg.W + tg.px;
  const float al = 1.0f - p.T;
  const float t0 = p.t0 < FLT_MAX ? p.t0 : 0.0f;           // 0 where nothing contributed
  const float depth = __builtin_fmaf(t0, al, p.acc[F]);    // D = D' + t0 A
  const bool own = out == nullptr;
  const size_t P = plane ? (size_t)plane : (size_t)tg.W * tg.H;
  const ViewOutDev* vo = outs + (tg.vw - views);
  float* o = own ? reinterpret_cast<float*>((uint64_t)vo->lo | (uint64_t)vo->hi << 32) +
                       (size_t)tg.py * (plane ? (size_t)row : (size_t)tg.W) + tg.px
                 : out + (size_t)NO * tg.vw->pix_off + pix;
  const uint32_t wr = own ? want : ch;      // a view's own output has no other planes
  if (wr & ROGS_CH_RGB)
#pragma unroll
    for (int f = 0; f < 3; ++f) o[f * P] = p.acc[f];
  if (!own || (wr & ROGS_CH_RGB)) o += 3 * P;
  if (wr & ROGS_CH_SEM)
#pragma unroll
    for (int f = 3; f < F; ++f) o[(f - 3) * P] = p.acc[f];
  if (!own || (wr & ROGS_CH_SEM)) o += C * P;
  if (wr & ROGS_CH_D) *o = depth;
  if (!own || (wr & ROGS_CH_D)) o += P;
  if (wr & ROGS_CH_A) *o = al;
  if (own && (wr & ROGS_CH_ELEV)) {
    if (wr & ROGS_CH_A) o += P;
    *o = al > 0.0f ? vo->elev_ref - depth / al : __int_as_float(0x7fc00000);
  }
  if (tfin && (ch & kPlanes) == kPlanes) {
    tfin[tg.vw->pix_off + pix] = p.T;
    nlast[tg.vw->pix_off + pix] = (p.T < teps) ? p.nl : len;
    drel[tg.vw->pix_off + pix] = make_float2(p.acc[F], t0);
  }
}

// Register budgets of the backward kernels of one-wave tiles: up to 8 classes,
// 7 waves per SIMD at 16-entry staging (what its LDS block allows) and 5 at 32
// entries (timed slightly faster than 6, the most its LDS block allows); the
// compiler meets them without spilling in the entry loops.  Other instances
// keep the compiler's own budget (1).
template <int C, int NW, int KS>
constexpr int kWavesPerEu() {
  if (NW > 1) return C <= 8 ? 4 : 1;
  return (C <= 8 && KS <= 32) ? (KS <= 16 ? 7 : 5) : 1;
}

// Backward compositing of the batch from the output gradient G (5 + C planes
// per view), the outputs, T_final and n_last.
template <int C, int NW, int KS>
__global__ __launch_bounds__(64 * NW)
__attribute__((amdgpu_waves_per_eu(kWavesPerEu<C, NW, KS>()))) void k_render_bwd(
    const ViewDev* __restrict__ views, int V, int N, float qcut, float amax,
    const uint4* __restrict__ tinfo, const uint32_t* __restrict__ vals,
    const uint32_t* __restrict__ spair,
    const float4* __restrict__ rec, const float4* __restrict__ feat, const float* __restrict__ out,
    const float* __restrict__ G, const float* __restrict__ tfin,
    const uint32_t* __restrict__ nlast, const float2* __restrict__ drel,
    float* __restrict__ gpair) {
  constexpr int F = 3 + C;
  constexpr int NO = 5 + C;
  __shared__ BlockLds<C, NW, KS> L;
  const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const TileGeom tg = tile_geom(views, N, tinfo, wv);
  if (tg.rend == tg.rbeg) return;
  const size_t HW = (size_t)tg.W * tg.H;
  PixelGrad<C> pg;
  pg.GO = 0.0f;
  pg.Tf = 1.0f;
  pg.nl = 0;
  pg.t0 = 0.0f;
#pragma unroll
  for (int f = 0; f < F + 2; ++f) pg.Gv[f] = 0.0f;
  if (tg.px < tg.W && tg.py < tg.H) {
    const size_t p = (size_t)tg.py * tg.W + tg.px;
    const float* g = G + (size_t)NO * tg.vw->pix_off + p;
    const float* o = out + (size_t)NO * tg.vw->pix_off + p;
    float go = 0.0f;
#pragma unroll
    for (int f = 0; f < F + 2; ++f) pg.Gv[f] = g[f * HW];
#pragma unroll
    for (int f = 0; f < F; ++f) go = __builtin_fmaf(pg.Gv[f], o[f * HW], go);
    const float2 dr = drel[tg.vw->pix_off + p];          // D' and t0 of the forward
    go = __builtin_fmaf(pg.Gv[F], dr.x, go);
    pg.GO = go;
    pg.t0 = dr.y;
    pg.Tf = tfin[tg.vw->pix_off + p];
    pg.nl = nlast[tg.vw->pix_off + p];
  }
  if constexpr (NW == 1)
    backward_tile<C, KS, true, 0>(tg, qcut, amax, vals, spair, rec, feat, L.st, L.w[0], L.e, pg,
                                  gpair, false, 0u, nullptr);
  else
    backward_block<C, NW, KS, true>(tg, qcut, amax, vals, spair, rec, feat, L, pg, gpair);
}

// This tile's share of the loss and of dL/d(a, b), summed over its waves in
// wave order.  Every wave of the block calls it.
template <int NW>
__device__ __forceinline__ void tile_loss(const float (&lp)[3], float* s_l, float* part) {
  const int lane = threadIdx.x & 63;
  const float tot = wave_reduce_scatter<3>(lp, lane);
  const int c = rs_comp(lane, 3);
  const bool writer = c >= 0 && (lane & rs_dup_bits(3)) == 0;
  if constexpr (NW == 1) {
    if (writer) part[c] = tot;
  } else {
    if (writer) s_l[3 * (threadIdx.x >> 6) + c] = tot;
    __syncthreads();
    if (threadIdx.x < 3) {
      float t = s_l[threadIdx.x];
#pragma unroll
      for (int w = 1; w < NW; ++w) t += s_l[3 * w + threadIdx.x];
      part[threadIdx.x] = t;
    }
  }
}

// The fused step's compositing: forward, the loss of Eq. 7-9 and 12 per pixel
// (its gradient, G.O, and this tile's share of the loss and of dL/d(a, b)),
// then the backward, in one kernel per tile.
// Register budget as for k_render_bwd.
template <int C, int NW, int KS>
__global__ __launch_bounds__(64 * NW)
__attribute__((amdgpu_waves_per_eu(kWavesPerEu<C, NW, KS>()))) void k_render_step(
    const ViewDev* __restrict__ views, int V, int N, float qcut, float amax,
    float teps, const uint4* __restrict__ tinfo, const uint32_t* __restrict__ vals,
    const uint32_t* __restrict__ spair,
    const float4* __restrict__ rec, const float4* __restrict__ feat, float* __restrict__ gpair,
    FusedLoss fl) {
  constexpr int F = 3 + C;
  constexpr int FS4 = (F + 4) / 4;
  // the forward of several waves stages in regions of their own
  union Lds {
    BlockLds<C, NW, KS> b;
    struct {
      float4 st[NW == 1 ? 1 : NW][NW == 1 ? 1 : 64 * (2 + FS4)];
      uint32_t pos[NW == 1 ? 1 : NW][NW == 1 ? 1 : 64];
    } f;
  };
  __shared__ Lds L;
  __shared__ float s_l[3 * NW];
  const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const TileGeom tg = tile_geom(views, N, tinfo, NW == 1 ? 0 : wv);
  PixelGrad<C> pg;
  const bool in_img = tg.px < tg.W && tg.py < tg.H;
  // the loss inputs of this lane's pixel (mask, target colour and label, in
  // parallel), requested before the forward so that their latency overlaps it
  const LossView lv = loss_view(fl.expo, fl.mcount, tg.v, fl.lam_c, fl.lam_s, fl.scale);
  uint32_t m = 0, lab = 0;
  float tv[3] = {0.0f, 0.0f, 0.0f};
  if (in_img && lv.any) {
    const size_t p = (size_t)tg.py * tg.W + tg.px;
    const size_t pix = tg.vw->pix_off + p;
    const float* t = fl.tgt + 3 * (size_t)tg.vw->pix_off + p;
    const size_t HW = (size_t)tg.W * tg.H;
    m = fl.mask[pix];
    lab = fl.label[pix];
    tv[0] = t[0];
    tv[1] = t[HW];
    tv[2] = t[2 * HW];
  }
  const float wc = m != 0 ? lv.wc : 0.0f, ws = m != 0 ? lv.ws : 0.0f;
  float* const part = fl.part + 3 * (size_t)tg.gt;
  if (tg.rend == tg.rbeg) {
    // a tile without entries: its pixels' outputs are 0 and there is nothing
    // to differentiate, so only its shares of the loss and of dL/db are
    // formed (dL/da is 0 at a zero output)
    float l = 0.0f, dbl = 0.0f;
    pixel_loss_empty<C>(tv, wc, ws, lv.ea, lv.b, l, dbl);
    const float lp[3] = {l, 0.0f, dbl};
    tile_loss<NW>(lp, s_l, part);
    return;
  }
  // the footprint weights of the list's first 16 entries, kept from the
  // forward for the backward where the register budget has room for them
  // (one-wave tiles; up to 8 classes only with 32-entry staging, since
  // at 16 they would spill; with 16 classes the kernel runs 3 waves per
  // SIMD with or without them)
  constexpr int kG = (NW == 1 && (C > 8 || KS == 32)) ? 16 : 0;
  float gsv[16];
  uint32_t e_first = 0;
  Pixel<C> px;
  if constexpr (NW == 1)
    forward_tile<C, KS, kG>(tg, qcut, amax, teps, vals, spair, rec, feat, L.b.st, px, e_first,
                            gsv);
  else
    forward_part<C, false>(tg, qcut, amax, teps, spair, rec, feat, L.f.st[wv], L.f.pos[wv], px,
                           true);
  // loss epilogue: dL/dO and G.O per pixel, this tile's loss partials
  const uint32_t len = tg.rend - tg.rbeg;
  float l = 0.0f, dal = 0.0f, dbl = 0.0f;
  {
    float g[F];
    // every lane evaluates the loss; a pixel outside the mask or the image
    // has zero weights, so its gradient and loss terms are +-0
    pixel_loss<C>(px.acc, tv, lab, wc, ws, lv.ea, lv.b, g, l, dal, dbl);
#pragma unroll
    for (int f = 0; f < F; ++f) pg.Gv[f] = g[f];
    pg.Gv[F] = 0.0f;         // the fused loss has no depth or alpha term
    pg.Gv[F + 1] = 0.0f;
    // G.O over the composited channels, in the same form as the stand-alone
    // backward so that both round alike (its depth term adds 0 * D' = +0)
    float go = 0.0f;
#pragma unroll
    for (int f = 0; f < F; ++f) go = __builtin_fmaf(pg.Gv[f], px.acc[f], go);
    pg.GO = go;
    pg.Tf = in_img ? px.T : 1.0f;
    pg.nl = in_img ? ((px.T < teps) ? px.nl : len) : 0u;
    pg.t0 = 0.0f;            // not used without a depth term
  }
  const float lp[3] = {l, dal, dbl};
  tile_loss<NW>(lp, s_l, part);   // its barrier also ends the forward's use of L
  // the fused loss has no depth or alpha term: their gradient rows are zero
  if constexpr (NW == 1)
    backward_tile<C, KS, false, kG>(tg, qcut, amax, vals, spair, rec, feat, L.b.st, L.b.w[0],
                                    L.b.e, pg, gpair, len <= (uint32_t)KS, e_first, gsv);
  else
    backward_block<C, NW, KS, false>(tg, qcut, amax, vals, spair, rec, feat, L.b, pg, gpair);
}

// Work counts of a rendered batch (diagnostics): per pixel, the list entries
// it visits in front-to-back order up to its termination (n_last) and, of
// those, the ones whose 3-sigma test passes.  Summed over the batch into
// counts[0] (evaluated) and counts[1] (contributing) with 64-bit atomics.
__global__ __launch_bounds__(64) void k_count_work(
    const ViewDev* __restrict__ views, int V, int nw, float qcut,
    const uint2* __restrict__ ranges, const uint32_t* __restrict__ vals,
    const uint32_t* __restrict__ pslot, const float4* __restrict__ rec,
    const uint32_t* __restrict__ nlast, unsigned long long* __restrict__ counts) {
  const int lane = threadIdx.x;
  const int gt = blockIdx.x;
  const int v = find_view(views, V, gt);
  const ViewDev& vw = views[v];
  const int lt = gt - vw.tile_off;
  const int ty = lt / vw.tiles_x, tx = lt - ty * vw.tiles_x;
  const int tw = vw.tw, th = vw.th;
  const int rows = 64 / tw;
  const int px = tx * tw + (lane % tw);
  const float pxc = (float)px + 0.5f;
  uint32_t nl[4];
  float pyc[4];
  uint32_t maxn = 0;
  for (int k = 0; k < 4; ++k) {
    const int py = ty * th + lane / tw + k * rows;
    pyc[k] = (float)py + 0.5f;
    nl[k] = (k < nw && px < vw.w && py < vw.h) ? nlast[vw.pix_off + (size_t)py * vw.w + px] : 0u;
    maxn = max(maxn, nl[k]);
  }
  for (int o = 32; o > 0; o >>= 1) maxn = max(maxn, (uint32_t)__shfl_xor((int)maxn, o, 64));
  const uint2 rg = ranges[gt];
  const uint32_t stop = rg.x + min(maxn, rg.y - rg.x);
  unsigned long long ev = 0, co = 0;
  for (uint32_t p = rg.x; p < stop; ++p) {
    const uint32_t slot = pslot[vals[p]];
    const float4 r0 = rec[2 * (size_t)slot], r1 = rec[2 * (size_t)slot + 1];
    const float dx = pixel_offset(pxc, r0.x, r0.z);
    const uint32_t idx = p - rg.x;
    for (int k = 0; k < 4; ++k) {
      if (idx >= nl[k]) continue;
      ev += 1;
      const float dy = pixel_offset(pyc[k], r0.y, r0.w);
      if (pixel_q32(r1.x, 2.0f * r1.y, r1.z, dx, dy) <= qcut) co += 1;
    }
  }
  for (int o = 32; o > 0; o >>= 1) {
    ev += (unsigned long long)__shfl_xor((long long)ev, o, 64);
    co += (unsigned long long)__shfl_xor((long long)co, o, 64);
  }
  if (lane == 0) {
    atomicAdd(&counts[0], ev);
    atomicAdd(&counts[1], co);
  }
}

template <int C, int NW>
void fwd_launch(const Layout& L, void* ws, float* out, const FwdArgs& fa, hipStream_t st) {
  launch_bands(L.total_tiles, 64 * NW, [&](int64_t first, unsigned n) {
    hipLaunchKernelGGL((k_render_fwd<C, NW>), dim3(n), dim3(64 * NW), 0, st,
                       at<const ViewDev>(ws, L.o_views), L.V, L.N, L.q_cut, L.alpha_max,
                       L.t_eps, at<const uint4>(ws, L.o_tinfo) + first,
                       at<const uint32_t>(ws, L.o_spair),
                       at<const float4>(ws, L.o_rec), at<const float4>(ws, L.o_feat), out,
                       fa.save ? at<float>(ws, L.o_tfin) : nullptr, at<uint32_t>(ws, L.o_nlast),
                       at<float2>(ws, L.o_drel), fa.mask,
                       reinterpret_cast<const ViewOutDev*>(at<int64_t>(ws, L.o_lpart) + L.V + 1),
                       fa.plane, fa.row);
  });
}

template <int C, int NW, int KS>
void bwd_launch(const Layout& L, void* ws, const float* out, const float* G, hipStream_t st) {
  launch_bands(L.total_tiles, 64 * NW, [&](int64_t first, unsigned n) {
    hipLaunchKernelGGL((k_render_bwd<C, NW, KS>), dim3(n), dim3(64 * NW), 0, st,
                       at<const ViewDev>(ws, L.o_views), L.V, L.N, L.q_cut, L.alpha_max,
                       at<const uint4>(ws, L.o_tinfo) + first, at<const uint32_t>(ws, L.o_vals),
                       at<const uint32_t>(ws, L.o_spair),
                       at<const float4>(ws, L.o_rec), at<const float4>(ws, L.o_feat), out, G,
                       at<const float>(ws, L.o_tfin), at<const uint32_t>(ws, L.o_nlast),
                       at<const float2>(ws, L.o_drel), at<float>(ws, L.o_gpair));
  });
}

template <int C, int NW, int KS>
void step_launch(const Layout& L, void* ws, const FusedLoss& fl, hipStream_t st) {
  launch_bands(L.total_tiles, 64 * NW, [&](int64_t first, unsigned n) {
    hipLaunchKernelGGL((k_render_step<C, NW, KS>), dim3(n), dim3(64 * NW), 0, st,
                       at<const ViewDev>(ws, L.o_views), L.V, L.N, L.q_cut, L.alpha_max,
                       L.t_eps, at<const uint4>(ws, L.o_tinfo) + first,
                       at<const uint32_t>(ws, L.o_vals), at<const uint32_t>(ws, L.o_spair),
                       at<const float4>(ws, L.o_rec), at<const float4>(ws, L.o_feat),
                       at<float>(ws, L.o_gpair), fl);
  });
}

// which: 0 forward, 1 backward, 2 fused step
template <int C, int NW, int KS>
void launch_one(const Layout& L, void* ws, const float* out, const float* G, const FusedLoss* fl,
                int which, hipStream_t st) {
  if (which == 1) bwd_launch<C, NW, KS>(L, ws, out, G, st);
  else step_launch<C, NW, KS>(L, ws, *fl, st);
}

template <int C, int NW>
int dispatch_stage(const Layout& L, void* ws, const float* out, const float* G, float* outw,
                   const FusedLoss* fl, int which, const FwdArgs& fa, hipStream_t st) {
  if (which == 0) {
    fwd_launch<C, NW>(L, ws, outw, fa, st);
    return 0;
  }
  switch (L.stage) {
    case 16: launch_one<C, NW, 16>(L, ws, out, G, fl, which, st); return 0;
    case 32: launch_one<C, NW, 32>(L, ws, out, G, fl, which, st); return 0;
    case 64: launch_one<C, NW, 64>(L, ws, out, G, fl, which, st); return 0;
    default: return -1;
  }
}

template <int C>
int dispatch_waves(const Layout& L, void* ws, const float* out, const float* G, float* outw,
                   const FusedLoss* fl, int which, const FwdArgs& fa, hipStream_t st) {
  switch (L.nw) {
    case 1: return dispatch_stage<C, 1>(L, ws, out, G, outw, fl, which, fa, st);
    case 2: return dispatch_stage<C, 2>(L, ws, out, G, outw, fl, which, fa, st);
    case 4: return dispatch_stage<C, 4>(L, ws, out, G, outw, fl, which, fa, st);
    default: return -1;
  }
}

int dispatch(const Layout& L, void* ws, const float* out, const float* G, float* outw,
             const FusedLoss* fl, int which, const FwdArgs& fa, hipStream_t st) {
  switch (L.C) {
    case 1: return dispatch_waves<1>(L, ws, out, G, outw, fl, which, fa, st);
    case 2: return dispatch_waves<2>(L, ws, out, G, outw, fl, which, fa, st);
    case 3: return dispatch_waves<3>(L, ws, out, G, outw, fl, which, fa, st);
    case 4: return dispatch_waves<4>(L, ws, out, G, outw, fl, which, fa, st);
    case 5: return dispatch_waves<5>(L, ws, out, G, outw, fl, which, fa, st);
    case 6: return dispatch_waves<6>(L, ws, out, G, outw, fl, which, fa, st);
    case 7: return dispatch_waves<7>(L, ws, out, G, outw, fl, which, fa, st);
    case 8: return dispatch_waves<8>(L, ws, out, G, outw, fl, which, fa, st);
    case 16: return dispatch_waves<16>(L, ws, out, G, outw, fl, which, fa, st);
    default: return -1;
  }
}

}  // namespace

int launch_render_fwd(const Layout& L, void* ws, const rogs_surfels*, float* out,
                      const FwdArgs& fa, hipStream_t st) {
  if (L.total_tiles <= 0) return 0;
  return dispatch(L, ws, nullptr, nullptr, out, nullptr, 0, fa, st);
}

int launch_render_bwd(const Layout& L, void* ws, const rogs_surfels*, const float* out,
                      const float* G, hipStream_t st) {
  if (L.total_tiles <= 0) return 0;
  return dispatch(L, ws, out, G, nullptr, nullptr, 1, FwdArgs{}, st);
}

void launch_count_work(const Layout& L, void* ws, unsigned long long* counts, hipStream_t st) {
  if (L.total_tiles <= 0) return;
  hipLaunchKernelGGL(k_count_work, dim3((unsigned)L.total_tiles), dim3(64), 0, st,
                     at<const ViewDev>(ws, L.o_views), L.V, L.nw, L.q_cut,
                     at<const uint2>(ws, L.o_ranges), at<const uint32_t>(ws, L.o_vals),
                     at<const uint32_t>(ws, L.o_pslot), at<const float4>(ws, L.o_rec),
                     at<const uint32_t>(ws, L.o_nlast), counts);
}

int launch_render_step(const Layout& L, void* ws, const FusedLoss& fl, hipStream_t st) {
  if (L.total_tiles <= 0) return 0;
  return dispatch(L, ws, nullptr, nullptr, nullptr, &fl, 2, FwdArgs{}, st);
}

}  // namespace rogs
