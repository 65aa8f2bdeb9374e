// Sanitizer harness of the one-shot entry point: what its calls may rely on between two of them.  The workspace is the
// caller's in between (the harness overwrites it), its address may belong to other data, and the page-locked lists of a
// plan must not change before the copies out of them are made (the model of the runtime checks that).
//
//   one_shot ROUNDS
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <utility>
#include <vector>

#include "hip_stub.h"
#include "sparse_vdit.h"

namespace {
int g_failures = 0;
void expect(bool ok, const char* what, int status = 0) {
  if (ok) return;
  std::fprintf(stderr, "one-shot: %s (status %d)\n", what, status);
  ++g_failures;
}
}  // namespace

int main(int argc, char** argv) {
  const int rounds = argc > 1 ? std::atoi(argv[1]) : 1;
  stub::set_compute_units(256);
  stub::set_tensor_checks(true);
  constexpr int H = 5;
  svd_tensor_desc d{};
  d.B = 2, d.H = H, d.L = 700, d.D = 64;
  d.stride_l = d.D, d.stride_h = int64_t(d.L) * d.D, d.stride_b = d.stride_h * H;
  const size_t tensor = size_t(d.B) * d.stride_b * 2, n_rows = size_t(d.B) * H * d.L;
  void* t[4];
  for (void*& p : t) p = stub::device_alloc(tensor);
  std::vector<int32_t> cols, offsets = {-300, 0, 300};
  for (int c = 3; c < d.L; c += 4) cols.push_back(c);
  svd_head_params pp[H] = {};
  for (svd_head_params& p : pp) {
    p.half_width = 40;
    p.n_offsets = 3, p.offsets = offsets.data();
    p.n_cols = int32_t(cols.size()), p.cols = cols.data();
  }
  const int32_t first[H] = {SVD_DENSE, SVD_SKIP, SVD_DIAG, SVD_MULTIDIAG, SVD_VSTRIPE};
  // the largest workspace that any rotation of the table needs
  size_t bytes = 0;
  for (int r = 0; r < H; ++r) {
    int32_t table[H];
    for (int h = 0; h < H; ++h) table[h] = first[(h + r) % H];
    size_t need = 0;
    expect(svd_plan_workspace_bytes(&d, table, pp, nullptr, &need) == SVD_OK, "svd_plan_workspace_bytes");
    if (need > bytes) bytes = need;
  }
  void* ws[2] = {stub::device_alloc(bytes), stub::device_alloc(bytes)};
  hipStream_t streams[2] = {nullptr, stub::create_stream()};
  auto call = [&](int rot, int w, hipStream_t s, const char* what) {
    int32_t table[H];
    for (int h = 0; h < H; ++h) table[h] = first[(h + rot) % H];
    stub::new_forward();
    const int st = sparse_vdit_attn_forward(t[0], t[1], t[2], table, pp, t[3], &d, ws[w], bytes, s);
    expect(st == SVD_OK, what, st);
    expect(stub::out_rows_written() == n_rows, what);
    return st;
  };
  for (int i = 0; i < rounds; ++i) {
    call(i, 0, nullptr, "a first call");
    call(i, 0, nullptr, "the same call again");
    for (int fill : {0x7f, 0xff, 0x00}) {
      std::memset(ws[0], fill, bytes);   // freed and given to something else, then to the workspace again
      call(i, 0, streams[fill == 0xff], "the same call on a workspace that was used in between");
    }
    for (int k = 0; k < 12; ++k) call(i + k, k & 1, streams[(k / 3) & 1], "tables, workspaces and streams in turn");
    // under capture: the launches of a repeated call are recorded, without a copy; another table is refused
    hipStream_t s = stub::create_stream();
    call(i, 0, s, "the call to be captured");
    long nodes = stub::captured_nodes();
    stub::begin_capture(s);
    call(i, 0, s, "a repeated call under capture");
    expect(stub::captured_nodes() > nodes, "the capture recorded launches");
    expect(stub::end_capture(s) == hipSuccess, "the capture ends");
    nodes = stub::captured_nodes();
    stub::begin_capture(s);
    int32_t dense[H] = {};
    const int st = sparse_vdit_attn_forward(t[0], t[1], t[2], dense, pp, t[3], &d, ws[0], bytes, s);
    expect(st == SVD_ERR_HIP, "a new table under capture is refused", st);
    expect(stub::captured_nodes() == nodes, "a refused call records nothing");
    expect(stub::end_capture(s) == hipSuccess, "the capture ends");
    stub::destroy_stream(s);
    call(i, 0, nullptr, "a call after the capture");
    expect(sparse_vdit_attn_forward(t[0], t[1], t[2], dense, pp, t[3], &d, ws[0], 64, nullptr) == SVD_ERR_WORKSPACE, "a small workspace");
    call(i, 0, nullptr, "a call after a refused one");
  }
  {
    // a plan that forks its groups onto streams of its own is replaced by the next table's only when those are idle
    stub::set_compute_units(3);
    stub::set_tensor_checks(false);
    svd_tensor_desc s{};
    s.B = 1, s.H = 5, s.L = 9300, s.D = 64;
    s.stride_l = s.D, s.stride_h = int64_t(s.L) * s.D, s.stride_b = s.stride_h * s.H;
    svd_head_params sp[5] = {};
    int32_t table[5] = {};
    size_t need = 0;
    for (svd_head_params& p : sp) p.half_width = 60;
    table[4] = SVD_DIAG;
    svd_plan_workspace_bytes(&s, table, sp, nullptr, &need);
    void* w = stub::device_alloc(need);
    const long before = stub::streams_created();
    stub::set_strict_destroy(true);
    for (int i = 0; i < 4; ++i) {
      table[4] = SVD_DIAG, table[0] = SVD_DENSE;
      std::swap(table[4], table[i % 2 ? 0 : 4]);
      const int st = sparse_vdit_attn_forward(t[0], t[1], t[2], table, sp, t[3], &s, w, need, nullptr);
      expect(st == SVD_OK, "a call whose plan forks", st);
    }
    stub::set_strict_destroy(false);
    expect(stub::streams_created() > before, "the plans have streams of their own");
    stub::set_compute_units(256);
  }
  {
    // lists longer than a page-locked area: copied from where they are, and waited for
    stub::set_tensor_checks(false);
    svd_tensor_desc s{};
    s.B = 1, s.H = 6, s.L = 60000, s.D = 64;
    s.stride_l = s.D, s.stride_h = int64_t(s.L) * s.D, s.stride_b = s.stride_h * s.H;
    svd_head_params sp[6] = {};
    int32_t table[6];
    for (int h = 0; h < 6; ++h) table[h] = SVD_DIAG, sp[h].half_width = 20000 + h;
    size_t need = 0;
    svd_plan_workspace_bytes(&s, table, sp, nullptr, &need);
    expect(need > (size_t(8) << 20), "lists of more than 8 MiB");
    void* w = stub::device_alloc(need);
    const long copies = stub::launches_of("copy_lists_kernel");
    for (int i = 0; i < 2; ++i) {
      std::memset(w, 0x7f, need);
      const int st = sparse_vdit_attn_forward(t[0], t[1], t[2], table, sp, t[3], &s, w, need, nullptr);
      expect(st == SVD_OK, "a call with long lists", st);
    }
    expect(stub::launches_of("copy_lists_kernel") == copies, "no page-locked copy of long lists");
  }
  {
    // the library's own buffer: where a layer with its table does not fit it, the launches per group keep the split of
    // the dense heads, if that fits (this layer: 346 us with the split, 481 us without)
    stub::set_tensor_checks(false);
    svd_tensor_desc s{};
    s.B = 1, s.H = 9, s.L = 23000, s.D = 128;
    s.stride_l = s.D, s.stride_h = int64_t(s.L) * s.D, s.stride_b = s.stride_h * s.H;
    int32_t table[9];
    svd_head_params sp[9] = {};
    for (int h = 0; h < 9; ++h) table[h] = h ? SVD_DIAG : SVD_DENSE, sp[h].half_width = 60;
    svd_plan_options opt{};
    size_t need = 0, grouped = 0;
    svd_plan_workspace_bytes(&s, table, sp, &opt, &need);
    opt.single_launch = 2;
    svd_plan_workspace_bytes(&s, table, sp, &opt, &grouped);
    expect(need > SVD_STATIC_SCRATCH_BYTES && grouped <= SVD_STATIC_SCRATCH_BYTES, "the layer's table does not fit the buffer, its launches do");
    const long merges = stub::launches_of("combine_partials_kernel"), tables = stub::launches_of("attn_grid_kernel");
    stub::new_forward();
    const int st = sparse_vdit_attn_forward_static(t[0], t[1], t[2], table, sp, t[3], &s, nullptr);
    expect(st == SVD_OK, "static one-shot call", st);
    expect(stub::launches_of("combine_partials_kernel") > merges && stub::launches_of("attn_grid_kernel") == tables, "the dense head runs split");
  }
  {
    // nothing of an FP8 pass, which these calls do not have, counts against that buffer: a layer that fits it with its own
    // table and would not fit it with a second one for FP8 keeps its table
    stub::set_tensor_checks(false);
    constexpr int N = 27;
    svd_tensor_desc s{};
    s.B = 1, s.H = N, s.L = 40000, s.D = 64;
    s.stride_l = s.D, s.stride_h = int64_t(s.L) * s.D, s.stride_b = s.stride_h * s.H;
    int32_t table[N];
    std::vector<int32_t> many(s.L);
    for (int c = 0; c < s.L; ++c) many[c] = c;
    svd_head_params sp[N] = {};
    for (int h = 0; h < N; ++h) table[h] = h < 7 ? SVD_VSTRIPE : SVD_DIAG, sp[h].half_width = 60, sp[h].cols = many.data();
    size_t need = 0;
    for (int n = 128 * 280; need <= SVD_STATIC_SCRATCH_BYTES && n <= s.L; n += 128) {   // the shortest lists that are too long with both
      for (int h = 0; h < 7; ++h) sp[h].n_cols = n;
      expect(svd_plan_workspace_bytes(&s, table, sp, nullptr, &need) == SVD_OK, "svd_plan_workspace_bytes");
    }
    expect(need > SVD_STATIC_SCRATCH_BYTES, "a layer that does not fit with both tables");
    const long tables = stub::launches_of("attn_grid_kernel");
    stub::new_forward();
    const int st = sparse_vdit_attn_forward_static(t[0], t[1], t[2], table, sp, t[3], &s, nullptr);
    expect(st == SVD_OK, "static one-shot call near the buffer's limit", st);
    expect(stub::launches_of("attn_grid_kernel") > tables, "the layer runs from its table");
  }
  std::printf("%d violations, %d failures\n", stub::violations(), g_failures);
  return stub::violations() || g_failures ? 1 : 0;
}
