// A table of items that cannot be built leaves the plan as it was: image, list offsets and all.
#include <cstdio>

#include "plan.h"
#include "sparse_vdit.h"

int main() {
  svd_tensor_desc d{};
  d.B = 1, d.H = 2, d.L = 3000, d.D = 64;
  d.stride_l = d.D, d.stride_h = int64_t(d.L) * d.D, d.stride_b = d.stride_h * d.H;
  const int32_t table[2] = {SVD_DIAG, SVD_MULTIDIAG}, offsets[2] = {-900, 900};
  svd_head_params pp[2] = {};
  pp[0].half_width = 30;
  pp[1].half_width = 1000, pp[1].n_offsets = 2, pp[1].offsets = offsets;
  svd::Plan p;
  if (svd::compile_plan(d, table, pp, 256, 128, 0, 128, &p) != SVD_OK) return 2;
  // the narrow group is on the small tile, its lists on the large one beside it; of the other group they are taken away
  if (p.groups[0].block_q != 128 || p.groups[0].bands_large.empty()) return 3;
  p.groups[1].bands.clear();
  p.groups[1].bands_large.clear();
  p.groups[1].block_q = 128;
  const std::vector<int32_t> image = p.ws_image;
  svd::GridTable t;
  if (svd::build_grid_table(&p, 256, 256, true, &t)) return 4;
  const bool same = p.ws_image == image && p.groups[0].ws_list_table_large == 0;
  std::printf("image %zu -> %zu words, list table %zu\n", image.size(), p.ws_image.size(), p.groups[0].ws_list_table_large);
  return same ? 0 : 1;
}
