// Host model of the launch of a whole layer from a table of items (launch_grid of attn_kernels.h):
// walks the records, touches what the kernels would address, and checks that the chunks of a cut
// item lie in consecutive slots, follow one another and are merged once.
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <tuple>
#include <vector>

#include "attn_kernels.h"
#include "fp8_kernels.h"
#include "hip_stub.h"

namespace svd {
namespace {

void need(const void* p, size_t bytes, const char* what) {
  if (!stub::in_device(p, bytes)) stub::violation("grid: %s (%zu bytes) outside every device allocation", what, bytes);
}

void rows(const GridLaunch& g, int b, int head, int row0, int n) {
  if (!stub::tensor_checks()) return;
  for (int r = row0; r < row0 + n && r < g.a.L; ++r) {
    __bf16* row = g.a.out + b * g.a.stride_b + head * g.a.stride_h + (int64_t)r * g.a.stride_l;
    need(row, (size_t)g.a.D * 2, "output row");
    stub::note_out_row(row);
  }
}

}  // namespace

static void walk(const GridLaunch& g, const Fp8Launch* f8, hipStream_t stream);

hipError_t launch_grid(const GridLaunch& g, hipStream_t stream) {
  walk(g, nullptr, stream);
  return hipSuccess;
}

// The pre-pass writes the arrays of every head that computes; the text rows of stripe heads are not in the table.
hipError_t launch_grid_fp8(const Fp8Launch& f, const GridLaunch& g, hipStream_t stream) {
  stub::note_launch(stream, "quantise_layer_kernel");
  if (g.waves != 4 || f.a.partial != g.partial) stub::violation("grid fp8: waves %d", g.waves);
  for (int h = 0; h < g.n_heads; ++h) {
    const int* r = g.a.ws + g.head_table + h * kGridHeadWords;
    need(r, kGridHeadWords * 4, "head record");
    if (r[0] < 0 || r[0] >= g.a.H) stub::violation("grid fp8: head %d", r[0]);
    if (r[1] >= 0) need(g.a.ws + r[1], (size_t)r[2] * 4, "column list or row map");
    if (r[1] >= 0 && (r[2] > f.Lp || r[2] % 64)) stub::violation("grid fp8: list of %d keys", r[2]);
  }
  walk(g, &f, stream);
  return hipSuccess;
}

static void walk(const GridLaunch& g, const Fp8Launch* f8, hipStream_t stream) {
  stub::note_launch(stream, "attn_grid_kernel");
  need(g.a.ws + g.merge_table, (size_t)g.n_merges * kGridWords * 4, "merge records");
  int chunks = 0;
  for (int i = 0; i < g.n_merges; ++i) chunks += g.a.ws[g.merge_table + (size_t)i * kGridWords + 3];
  std::printf("grid: waves %d records %d merges %d fp8 %d chunks %d\n", g.waves, g.n_blocks, g.n_merges, f8 ? 1 : 0, chunks);
  if (g.n_merges > 0) stub::note_launch(stream, "merge_chunks_kernel");
  const int BR = g.waves * 32, BC = g.a.D == 128 ? Tile128::BC : Tile64::BC;
  const size_t slot_floats = grid_slot_floats(g.a.D, g.waves);
  struct Chunk { int head, b, qblk, t0, n, kind; };
  std::map<int, Chunk> slots;
  const int* table = g.a.ws + g.table;
  need(table, (size_t)g.n_blocks * kGridWords * 4, "records");
  if (((uintptr_t)table - (uintptr_t)g.a.ws) % (kGridWords * 4)) stub::violation("grid: records are not aligned");
  for (int i = 0; i < g.n_blocks; ++i) {
    const int* r = table + (size_t)i * kGridWords;
    if (r[0] < 0) continue;
    const int kind = r[0] & 255, t0 = r[0] >> 8, head = r[1], b = r[2], qblk = r[3], n = r[4];
    if (head < 0 || head >= g.a.H || b < 0 || b >= g.a.B || qblk < 0) {
      stub::violation("grid record %d: head %d, batch entry %d, query tile %d", i, head, b, qblk);
      continue;
    }
    if (kind == SEG_ZERO) {
      rows(g, b, head, qblk * kGridZeroRows, kGridZeroRows);
      continue;
    }
    stub::note_tiles(n);
    if (qblk * BR >= g.a.L || n < 1) stub::violation("grid record %d: query tile %d, %d key tiles", i, qblk, n);
    if (kind == SEG_DENSE) {
      if ((t0 + n - 1) * BC >= g.a.L) stub::violation("grid record %d: key tile past the sequence", i);
    } else if (kind == SEG_GATHER) {
      if ((t0 + n - 1) * BC >= r[6] || (f8 && (t0 + n) * BC > f8->Lp)) stub::violation("grid record %d: past the column list", i);
      const int* cols = g.a.ws + r[5] + t0 * BC;
      need(cols, (size_t)n * BC * 4, "column list");
      for (int c = 0; c < n * BC; ++c)
        if (cols[c] >= g.a.L || (cols[c] < 0) != (t0 * BC + c >= r[6])) stub::violation("grid record %d: column %d is %d", i, c, cols[c]);
    } else {
      const int* e = g.a.ws + r[5] + 2 * t0;
      need(e, (size_t)n * 8, "band entries");
      int before = -1;
      for (int t = 0; t < n; ++t) {
        const int meta = e[2 * t + 1];
        if (e[2 * t] <= before || e[2 * t] * BC >= g.a.L) stub::violation("grid record %d: entry %d names key tile %d", i, t, e[2 * t]);
        before = e[2 * t];
        if (!(meta & 1)) need(g.a.ws + r[6] + 2 * ((meta >> 1) & 0x7fff), (size_t)(meta >> 16) * 8, "runs");
      }
      if (kind == SEG_PBAND) {
        need(g.a.ws + r[7], (size_t)(g.a.L + BC - 1) / BC * BC * 4, "row map");
        rows(g, b, head, qblk * BR, BR);   // never cut
        continue;
      }
    }
    if (r[7] < 0) {
      if (t0) stub::violation("grid record %d: starts at key tile %d but is not a chunk", i, t0);
      rows(g, b, head, qblk * BR, BR);
    } else if (!slots.emplace(r[7], Chunk{head, b, qblk, t0, n, kind}).second) {
      stub::violation("grid: slot %d is written twice", r[7]);
    } else {
      need(g.partial + (size_t)r[7] * slot_floats, slot_floats * sizeof(float), "partial results");
      std::memset(g.partial + (size_t)r[7] * slot_floats, 0x22, slot_floats * sizeof(float));
    }
  }
  size_t merged = 0;
  for (int i = 0; i < g.n_merges; ++i) {
    const int* r = g.a.ws + g.merge_table + (size_t)i * kGridWords;
    int t = 0;
    for (int c = 0; c < r[3]; ++c, ++merged) {
      const auto it = slots.find(r[4] + c);
      if (it == slots.end()) {
        stub::violation("grid merge %d: slot %d is not written", i, r[4] + c);
        continue;
      }
      const Chunk& k = it->second;
      if (k.head != r[0] || k.b != r[1] || k.qblk != r[2] || k.t0 != t) stub::violation("grid merge %d: chunk %d is not the next one", i, c);
      t += k.n;
    }
    const Chunk& k = slots[r[4]];
    if (k.kind == SEG_DENSE && t != (g.a.L + BC - 1) / BC) stub::violation("grid merge %d: the chunks end at key tile %d", i, t);
    rows(g, r[1], r[0], r[2] * BR, BR);
  }
  if (merged != slots.size()) stub::violation("grid: %zu slots, %zu merged", slots.size(), merged);
}

}  // namespace svd
