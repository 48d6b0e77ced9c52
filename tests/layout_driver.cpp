// Host-only checks of the workspace layout (test infrastructure, built by the
// package's build step and run without a GPU).  For batches of mixed view
// sizes in every tile shape, the places that kernels derive from a view's
// index lie inside the region that the layout reserves for them.  Also the parts
// of a launch that one grid cannot hold.  Prints "layout checks: ok".
#include <stdio.h>
#include <stdlib.h>

#include <random>
#include <utility>
#include <vector>

#include "../paper_2405_14342_amd/csrc/rogs_internal.h"

#define CHECK(x)                                                              \
  do {                                                                        \
    if (!(x)) {                                                               \
      fprintf(stderr, "check failed: %s (line %d)\n", #x, __LINE__);          \
      exit(1);                                                                \
    }                                                                         \
  } while (0)

using Sizes = std::vector<std::pair<int, int>>;

static rogs::Layout layout(const Sizes& sizes, int n, int tw, int th) {
  rogs_surfels s{};
  s.n = n;
  s.n_sem = 3;
  std::vector<rogs_camera> cams;
  for (const auto& wh : sizes) {
    rogs_camera c{};
    c.w = wh.first;
    c.h = wh.second;
    c.fx = c.fy = 1.0f;
    c.R_cw[0] = c.R_cw[4] = c.R_cw[8] = 1.0f;
    cams.push_back(c);
  }
  rogs_render_opts o;
  rogs_default_opts(&o);
  o.tile_w = tw;
  o.tile_h = th;
  rogs::Layout L;
  const char* why = nullptr;
  CHECK(rogs::make_layout(&s, cams.data(), (int)cams.size(), &o, 1000, 0, &L, &why, true) == ROGS_OK);
  return L;
}

// The fused step's loss chunk sums: every chunk of every view inside the block
// partials' region, views apart.
static void loss_chunks(const Sizes& sizes, int tw, int th) {
  const rogs::Layout L = layout(sizes, 100, tw, th);
  std::vector<int64_t> first_blk(1, 0);
  for (const auto& wh : sizes)
    first_blk.push_back(first_blk.back() + ((int64_t)wh.first * wh.second + 255) / 256);
  const size_t floats = (L.o_misc - L.o_lpart) / 4 - 2 * (size_t)(L.V + 1);
  int64_t end = 0;
  for (int v = 0; v < L.V; ++v) {
    const int64_t tiles = (int64_t)((sizes[v].first + tw - 1) / tw) * ((sizes[v].second + th - 1) / th);
    for (int64_t c = 0; c < rogs::tile_chunks(tiles); ++c) {
      const int64_t at = rogs::loss_chunk_at(first_blk.data(), v, c);
      CHECK(at >= end);
      end = at + 3;
      CHECK((size_t)end <= floats);
    }
  }
}

// A launch in parts: every block once, in order, and no part of 2^32 threads.
static void bands(int64_t blocks, int threads) {
  int64_t next = 0;
  rogs::launch_bands(blocks, threads, [&](int64_t first, unsigned n) {
    CHECK(first == next && n > 0 && (uint64_t)n * threads < (1ull << 32));
    next = first + n;
  });
  CHECK(next == blocks);
}

int main() {
  for (int threads : {64, 128, 256})
    for (int64_t blocks : {int64_t(0), int64_t(1), (int64_t(1) << 24) - 1, int64_t(1) << 24,
                           (int64_t(1) << 24) + 5, int64_t(1) << 26, (int64_t(1) << 31) - 1})
      bands(blocks, threads);
  const int shapes[][2] = {{16, 4}, {8, 8}, {64, 1}, {1, 64}, {16, 8}, {64, 2}, {1, 128}, {16, 16}, {64, 4}, {1, 256}};
  std::mt19937 rng(5);
  for (const auto& t : shapes) {
    // one large view among many tiny ones, in every place
    for (const auto& big : Sizes{{1920, 1080}, {16384, 16384}, {16384, 1}, {1, 16384}})
      for (int at : {0, 300, 600}) {
        Sizes s(601, {16, 16});
        s[at] = big;
        loss_chunks(s, t[0], t[1]);
      }
    Sizes ones(4096, {1, 1});
    ones[77] = {16384, 16384};
    loss_chunks(ones, t[0], t[1]);
    for (int k = 0; k < 50; ++k) {
      Sizes s;
      for (int v = 0; v < 1 + (int)(rng() % 40); ++v)
        s.push_back({1 + (int)(rng() % (1u << rng() % 13)), 1 + (int)(rng() % (1u << rng() % 13))});
      loss_chunks(s, t[0], t[1]);
    }
  }
  printf("layout checks: ok\n");
  return 0;
}
