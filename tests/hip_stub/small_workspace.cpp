// Sanitizer harness of plans whose workspace is smaller than svd_plan_workspace_bytes says.  A long layer runs its FP8 pass
// from a table that is worth a few per cent: a workspace that only lacks the room for it is taken, and the pass runs as a
// launch per group.  A short layer's, and any that lacks more, is refused.
#include <cstdio>
#include <vector>

#include "hip_stub.h"
#include "sparse_vdit.h"

namespace {
int g_failures = 0;
void expect(bool ok, const char* what, int L, long a = 0) {
  if (ok) return;
  std::fprintf(stderr, "small workspace, L = %d: %s (%ld)\n", L, what, a);
  ++g_failures;
}

void run(int D, int L, bool optional) {
  constexpr int H = 10;
  svd_tensor_desc d{};
  d.B = 1, d.H = H, d.L = L, d.D = D;
  d.stride_l = D, d.stride_h = int64_t(L) * D, d.stride_b = d.stride_h * H;
  const std::vector<int32_t> offsets = {-L / 3, 0, L / 3};
  std::vector<int32_t> cols;
  for (int c = 0; c < L; c += 9) cols.push_back(c);
  int32_t table[H] = {SVD_DENSE, SVD_SKIP, SVD_DIAG, SVD_DIAG, SVD_MULTIDIAG, SVD_DIAG, SVD_VSTRIPE, SVD_DIAG, SVD_DENSE, SVD_DIAG};
  svd_head_params pp[H] = {};
  for (svd_head_params& p : pp) {
    p.half_width = L / 6;
    p.n_offsets = 3, p.offsets = offsets.data();
    p.n_cols = int32_t(cols.size()), p.cols = cols.data();
  }
  size_t need = 0, bytes8 = 0;
  svd_plan_workspace_bytes(&d, table, pp, nullptr, &need);
  svd_fp8_workspace_bytes(&d, &bytes8);
  stub::set_tensor_checks(false);
  void* t = stub::device_alloc(256);
  void* ws8_area = stub::device_alloc(512);
  void* ws8 = reinterpret_cast<void*>((reinterpret_cast<uintptr_t>(ws8_area) + 255) / 256 * 256);
  auto create = [&](size_t bytes, void** ws, svd_plan** plan) {
    *ws = stub::device_alloc(bytes);
    const svd_status st = svd_plan_create(plan, &d, table, pp, nullptr, *ws, bytes, nullptr);
    expect((st == SVD_OK) == (*plan != nullptr), "a plan comes with SVD_OK alone", L, st);
    return st;
  };
  auto accepted = [&](size_t bytes) {
    void* ws = nullptr;
    svd_plan* plan = nullptr;
    const svd_status st = create(bytes, &ws, &plan);
    expect(st == SVD_OK || st == SVD_ERR_WORKSPACE, "too small or taken", L, st);
    if (plan) svd_plan_destroy(plan);
    stub::device_free(ws);
    return st == SVD_OK;
  };
  expect(accepted(need), "the workspace that was asked for", L);
  size_t lo = 0, hi = need;   // the smallest that is taken
  while (hi - lo > 1) {
    const size_t mid = lo + (hi - lo) / 2;
    (accepted(mid) ? hi : lo) = mid;
  }
  expect((hi < need) == optional, optional ? "a long layer does without its FP8 table" : "a short layer does not", L, long(need - hi));
  for (size_t bytes : {need, hi}) {
    void* ws = nullptr;
    svd_plan* plan = nullptr;
    if (create(bytes, &ws, &plan) != SVD_OK) continue;
    int32_t waves = -1, waves8 = -1;
    svd_plan_table(plan, &waves, &waves8);
    expect(waves8 == (bytes == need ? 4 : 0), "the FP8 pass has its table with the whole workspace", L, waves8);
    const long before = stub::launches_of("attn_fwd_fp8_kernel"), tables = stub::launches_of("quantise_layer_kernel");
    stub::new_forward();
    expect(svd_attn_forward_planned(plan, t, t, t, t, nullptr) == SVD_OK, "bf16 forward", L);
    expect(svd_attn_forward_fp8(plan, t, t, t, t, ws8, bytes8, nullptr) == SVD_OK, "FP8 forward", L);
    expect((stub::launches_of("quantise_layer_kernel") > tables) == (waves8 == 4), "from the table (its pre-pass covers the whole layer)", L);
    expect((stub::launches_of("attn_fwd_fp8_kernel") > before) == (waves8 == 0), "as a launch per group", L);
    svd_plan_destroy(plan);
    stub::device_free(ws);
  }
  stub::device_free(t);
  stub::device_free(ws8_area);
}
}  // namespace

int main() {
  stub::set_compute_units(8);   // long by its tiles per unit
  for (int D : {64, 128}) {
    run(D, 26000, true);
    run(D, 2600, false);
  }
  std::printf("%d violations, %d failures\n", stub::violations(), g_failures);
  return stub::violations() || g_failures ? 1 : 0;
}
