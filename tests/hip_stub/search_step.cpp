// Sanitizer harness of the search step: its workspace is no larger than its plans need one after the other, and with
// exactly that much every launch finds its lists (the launch models walk them and overwrite what launches write).
#include <algorithm>
#include <cstdio>
#include <vector>

#include "hip_stub.h"
#include "sparse_vdit.h"

namespace {
int g_failures = 0;
void expect(bool ok, const char* what, int L, long a = 0, long b = 0) {
  if (ok) return;
  std::fprintf(stderr, "search step, L = %d: %s (%ld, %ld)\n", L, what, a, b);
  ++g_failures;
}
size_t up(size_t x) { return (x + 255) / 256 * 256; }

// distinct: a list of its own for every head, else one for all
void run(int B, int H, int L, int D, bool distinct) {
  svd_tensor_desc d{};
  d.B = B, d.H = H, d.L = L, d.D = D;
  d.stride_l = D, d.stride_h = int64_t(L) * D, d.stride_b = d.stride_h * H;
  const size_t tensor = size_t(B) * d.stride_b * 2;
  std::vector<std::vector<int32_t>> cols(H), offsets(H);
  std::vector<svd_head_params> diag(H), multi(H), stripe(H), none(H);
  for (int h = 0; h < H; ++h) {
    const int n = distinct ? h : 0;
    for (int c = n % 2; c < L; c += 3 + n % 5) cols[h].push_back(c);
    offsets[h] = {-L / 3, 0, L / 3};   // L >= 3: three of them
    diag[h].half_width = L / 4 + n;
    multi[h].half_width = L / 30 + n, multi[h].n_offsets = 3, multi[h].offsets = offsets[h].data();
    stripe[h].n_cols = int32_t(cols[h].size()), stripe[h].cols = cols[h].data();
  }
  const svd_head_params* by_mode[5] = {nullptr, nullptr, diag.data(), multi.data(), stripe.data()};
  size_t need = 0, mse = 0, plan = 0;
  expect(svd_search_layer_workspace_bytes(&d, by_mode, &need) == SVD_OK, "svd_search_layer_workspace_bytes", L);
  expect(svd_head_mse_workspace_bytes(&d, &mse) == SVD_OK, "svd_head_mse_workspace_bytes", L);
  for (int mode = SVD_SKIP; mode <= SVD_VSTRIPE; ++mode) {
    const std::vector<int32_t> table(H, mode);
    size_t one = 0;
    expect(svd_plan_workspace_bytes(&d, table.data(), mode >= SVD_DIAG ? by_mode[mode] : none.data(), nullptr, &one) == SVD_OK,
           "svd_plan_workspace_bytes", L);
    plan = std::max(plan, one);
  }
  const size_t in_turn = 5 * up(tensor) + up(plan) + up(mse) + up(size_t(4) * H * sizeof(float));
  expect(need <= in_turn, "the workspace holds one plan at a time", L, long(need), long(in_turn));
  void* t[4];
  for (void*& p : t) p = stub::device_alloc(tensor);
  char* ws = static_cast<char*>(stub::device_alloc(need + 256));   // +256: an aligned start
  char* at = ws + (256 - reinterpret_cast<uintptr_t>(ws) % 256) % 256;
  for (size_t i = 0; i < need; ++i) at[i] = 0x7f;
  char* const end = at + need;
  const char behind = *end = 0x5a;
  std::vector<int32_t> table(H, -1);
  for (int round = 0; round < 2; ++round) {
    stub::new_forward();
    const int st = svd_search_layer(t[0], t[1], t[2], &d, by_mode, 0.5, 1.0, table.data(), nullptr, t[3], at, need, nullptr);
    expect(st == SVD_OK, "svd_search_layer", L, st);
    expect(stub::out_rows_written() == size_t(5) * B * H * L, "every row of the five modes is written once", L, long(stub::out_rows_written()));
    expect(*end == behind, "nothing behind the workspace is written", L);
    for (int32_t m : table) expect(m >= SVD_DENSE && m <= SVD_VSTRIPE, "a table of modes", L, m);
  }
  expect(svd_search_layer(t[0], t[1], t[2], &d, by_mode, 0.5, 1.0, table.data(), nullptr, t[3], at, need - 1, nullptr) == SVD_ERR_WORKSPACE,
         "a smaller workspace is refused", L);
  stub::device_free(ws);
  for (void* p : t) stub::device_free(p);
}
}  // namespace

int main() {
  for (int cu : {256, 8}) {
    stub::set_compute_units(cu);
    stub::set_tensor_checks(true);
    for (int D : {64, 128}) {
      run(1, 1, 4, D, false);      // lists longer than an output tensor
      run(1, 3, 20, D, true);
      run(2, 5, 333, D, true);
      run(1, 6, 2000, D, true);
      run(2, 4, 2000, D, false);
    }
  }
  std::printf("%d violations, %d failures\n", stub::violations(), g_failures);
  return stub::violations() || g_failures ? 1 : 0;
}
