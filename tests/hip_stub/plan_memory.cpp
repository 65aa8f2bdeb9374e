// What compiling a long layer and building its table of items ask of the allocator, against what the plan holds in the
// end: lists and image are laid out in memory that is reserved once, not grown and copied over and over.
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <new>
#include <vector>

#include "attn_kernels.h"
#include "plan.h"

namespace {
size_t g_bytes = 0;
}
void* operator new(size_t n) {
  g_bytes += n;
  if (void* p = std::malloc(n)) return p;
  throw std::bad_alloc();
}
void operator delete(void* p) noexcept { std::free(p); }
void operator delete(void* p, size_t) noexcept { std::free(p); }

int main() {
  int failures = 0;
  for (int D : {64, 128}) {
    constexpr int H = 24;
    svd_tensor_desc d{};
    d.B = 1, d.H = H, d.L = 75600, d.D = D;
    d.stride_l = D, d.stride_h = int64_t(d.L) * D, d.stride_b = d.stride_h * H;
    int32_t table[H];
    const std::vector<int32_t> offsets = {-7200, -3600, 0, 3600, 7200};
    std::vector<int32_t> cols;
    for (int c = 0; c < d.L; c += 37) cols.push_back(c);
    svd_head_params pp[H] = {};
    for (int h = 0; h < H; ++h) {
      table[h] = h < 2 ? SVD_DENSE : h < 12 ? SVD_DIAG : h < 18 ? SVD_MULTIDIAG : SVD_VSTRIPE;
      pp[h].half_width = table[h] == SVD_DIAG ? 3600 : 900;
      pp[h].n_offsets = int32_t(offsets.size()), pp[h].offsets = offsets.data();
      pp[h].n_cols = int32_t(cols.size()), pp[h].cols = cols.data();
    }
    for (bool always_large : {false, true}) {
      svd::Plan plan;
      svd::GridTable grid;
      const size_t before = g_bytes;
      if (svd::compile_plan(d, table, pp, 256, D == 64 ? 128 : 64, 0, 128, &plan, always_large) != SVD_OK ||
          !svd::build_grid_table(&plan, 128, 512, false, &grid)) {
        std::printf("D = %d: not compiled\n", D);
        return 2;
      }
      const size_t asked = g_bytes - before;
      size_t held = plan.ws_image.size() * sizeof(int32_t);
      for (const svd::Group& g : plan.groups)
        for (const std::vector<svd::BandList>* lists : {&g.bands, &g.bands_small, &g.bands_large})
          for (const svd::BandList& bl : *lists)
            held += sizeof(int32_t) * (bl.row_ptr.size() + bl.kv_block_idx.size() + bl.flags.size() + bl.run_first.size() + bl.run_count.size());
      // the items are sorted outside the image (as large as the table at most), and a list's room is an upper bound
      std::printf("D = %d: asked for %zu bytes, holds %zu\n", D, asked, held);
      failures += asked > 2 * held;
    }
  }
  return failures ? 1 : 0;
}
