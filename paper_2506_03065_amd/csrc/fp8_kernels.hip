// gfx950 (MI355X, CDNA4) kernels of the FP8 variant of the sparse attention
// forward (Appendix B: the sparse kernels of Section 4.2 with FP8 quantisation).
//
// The paper names neither format nor recipe; this library quantises Q, K, V and P
// to OCP E4M3 with fixed power-of-two scales:
//   Q8 = e4m3(q * 4 log2(e) / sqrt(D)),  K8 = e4m3(k / 4),  V8 = e4m3(v),
//   P8 = e4m3(2^(Q8.K8 - m)) with the integer reference m = ceil(row max) - 8,
// and accumulates scores, row sums and the output in fp32.
//
// Two kernels:
//   quantise_kv_kernel   pre-pass of a group of heads: K8 row-major, V8 transposed
//                        in groups of 64 keys with the keys of a group in the
//                        order in which a lane's score accumulators hold them.
//                        A vertical-stripe head (M_4) is compacted here: its
//                        arrays hold the listed key columns only.
//   attn_fwd_fp8_kernel  transposed scores and a lane that owns a query column, as
//                        in the bf16 kernel, on the FP8 matrix instructions
//                        v_mfma_f32_32x32x64_f8f6f4 (scores),
//                        v_mfma_scale_f32_32x32x64_f8f6f4 (P V; its block scale
//                        carries the reference of the tile's P) and
//                        v_mfma_f32_16x16x128_f8f6f4 (row sums of P).  Modes:
//                        DENSE, BAND, GATHER = the dense loop over a compacted
//                        head, and PBAND = the banded loop of a multi-diagonal
//                        head in rearranged form (Section 4.1.2): the pre-pass
//                        writes K8 and V8 in the rearranged order, Q rows and O
//                        rows go through the list's row map.
// Operand layout of the 32x32x64 instruction: lane l supplies row (column) l % 32
// with 32 of the 64 contraction indices in its 32 bytes, the same ones in both
// operands (all that the layouts here rely on); the result has the layout of the
// 32x32 bf16 instructions, so masks, maxima and the epilogue are those of the bf16
// kernel.  The reference is an integer: every change
// of units is an exact power of two and the rounding of P does not depend on the
// order of the key tiles (outside the subnormal range).
#include <hip/hip_runtime.h>

#include <cstdint>
#include <type_traits>

#include "fp8_kernels.h"

namespace svd {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x8 __attribute__((ext_vector_type(8)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
typedef short s16x2 __attribute__((ext_vector_type(2)));
typedef int i32x2 __attribute__((ext_vector_type(2)));
typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef int i32x8 __attribute__((ext_vector_type(8)));

constexpr float kNegInf = -__builtin_inff();
constexpr float kE4M3Max = 448.0f;

// Four floats to four E4M3 bytes, first argument in the lowest byte (round to
// nearest even; the caller keeps the values inside +-448).
__device__ __forceinline__ int pack_e4m3(float a, float b, float c, float d) {
  // the first conversion overwrites the low half of its destination and the second
  // the high half: starting from the bits of `a` (dead afterwards) saves a move
  int w = __builtin_bit_cast(int, a);
  w = __builtin_amdgcn_cvt_pk_fp8_f32(a, b, w, false);
  w = __builtin_amdgcn_cvt_pk_fp8_f32(c, d, w, true);
  return w;
}
// The same of a / scale, ...; scale is a power of two.
__device__ __forceinline__ int pack_e4m3(float a, float b, float c, float d, float scale) {
  s16x2 w = __builtin_bit_cast(s16x2, a);
  w = __builtin_amdgcn_cvt_scalef32_pk_fp8_f32(w, a, b, scale, false);
  w = __builtin_amdgcn_cvt_scalef32_pk_fp8_f32(w, c, d, scale, true);
  return __builtin_bit_cast(int, w);
}
__device__ __forceinline__ float sat_e4m3(float x) { return fminf(fmaxf(x, -kE4M3Max), kE4M3Max); }

__device__ __forceinline__ float half_max(float x) {
  const unsigned a = __builtin_bit_cast(unsigned, x);
  const auto r = __builtin_amdgcn_permlane32_swap(a, a, false, false);
  const unsigned r0 = r[0], r1 = r[1];
  return fmaxf(__builtin_bit_cast(float, r0), __builtin_bit_cast(float, r1));
}

// 16-byte chunk swizzle of the K8 tile (row = key, D bytes): a fragment read
// takes 16 bytes per lane with consecutive lanes on consecutive keys.
template <int D>
__device__ __forceinline__ int swz_k8(int row) {
  return D == 128 ? ((row >> 1) & 7) : ((row >> 2) & 3);
}

template <int N>
using Int = std::integral_constant<int, N>;

// ---------------------------------------------------------------------------
// Pre-pass.  Work-group = one group of 64 keys of one head.
// ---------------------------------------------------------------------------
template <int D>
__device__ __forceinline__ void quantise_group(const Fp8Launch& pp, const int G, const int head, const int b,
                                               const int* const cols, const int n_pad) {
  const AttnLaunch& p = pp.a;
  constexpr int SV_STRIDE = D + 8;   // bf16 elements; keeps rows 16-byte aligned
  __shared__ __attribute__((aligned(16))) __bf16 sv[64 * SV_STRIDE];
  if (G * 64 >= n_pad) return;
  const int64_t base = (int64_t)b * p.stride_b + (int64_t)head * p.stride_h;
  const __bf16* __restrict__ K = p.k + base;
  const __bf16* __restrict__ V = p.v + base;
  const size_t base8 = ((size_t)b * p.H + head) * (size_t)pp.Lp * D;
  uint8_t* __restrict__ K8 = pp.k8 + base8;
  uint8_t* __restrict__ V8 = pp.v8t + base8;
  const int tid = threadIdx.x;

  auto source_row = [&](int key) -> int {   // -1: no such key (zeros)
    if (cols) return cols[key];
    return key < p.L ? key : -1;
  };

  // K8: 16 elements per step
  constexpr int KCH = D / 16;
  for (int c = tid; c < 64 * KCH; c += 256) {
    const int row = c / KCH, pc = c % KCH;
    const int src = source_row(G * 64 + row);
    i32x4 outw = {0, 0, 0, 0};
    if (src >= 0) {
      const __bf16* s = K + (int64_t)src * p.stride_l + pc * 16;
      const f32x8 lo = __builtin_convertvector(*reinterpret_cast<const bf16x8*>(s), f32x8);
      const f32x8 hi = __builtin_convertvector(*reinterpret_cast<const bf16x8*>(s + 8), f32x8);
#pragma unroll
      for (int w = 0; w < 2; ++w) {
        outw[w] = pack_e4m3(sat_e4m3(lo[4 * w] * 0.25f), sat_e4m3(lo[4 * w + 1] * 0.25f),
                            sat_e4m3(lo[4 * w + 2] * 0.25f), sat_e4m3(lo[4 * w + 3] * 0.25f));
        outw[2 + w] = pack_e4m3(sat_e4m3(hi[4 * w] * 0.25f), sat_e4m3(hi[4 * w + 1] * 0.25f),
                                sat_e4m3(hi[4 * w + 2] * 0.25f), sat_e4m3(hi[4 * w + 3] * 0.25f));
      }
    }
    *reinterpret_cast<i32x4*>(K8 + ((size_t)(G * 64 + row) * D + pc * 16)) = outw;
  }

  // V: the 64 rows of the group through LDS, then one (d, 16 keys) piece per step
  constexpr int VCH = D / 8;
  for (int c = tid; c < 64 * VCH; c += 256) {
    const int row = c / VCH, pc = c % VCH;
    const int src = source_row(G * 64 + row);
    u32x4 raw = {0u, 0u, 0u, 0u};
    if (src >= 0) raw = *reinterpret_cast<const u32x4*>(V + (int64_t)src * p.stride_l + pc * 8);
    *reinterpret_cast<u32x4*>(&sv[row * SV_STRIDE + pc * 8]) = raw;
  }
  __syncthreads();
  for (int c = tid; c < D * 4; c += 256) {
    const int d = c >> 2, piece = c & 3;
    const int h = piece >> 1, blk = piece & 1;
    i32x4 outw;
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      float x[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) x[r] = sat_e4m3((float)sv[(32 * blk + 8 * g + 4 * h + r) * SV_STRIDE + d]);
      outw[g] = pack_e4m3(x[0], x[1], x[2], x[3]);
    }
    *reinterpret_cast<i32x4*>(V8 + (((size_t)G * D + d) * 64 + piece * 16)) = outw;
  }
}

// One launch per group of heads.
template <int D>
__global__ void __launch_bounds__(256) quantise_kv_kernel(const Fp8Launch pp, const int gather) {
  const AttnLaunch& p = pp.a;
  const int hg = blockIdx.y % p.n_heads;
  const int b = blockIdx.y / p.n_heads;
  const int head = p.heads ? p.heads[hg] : hg;
  const int* cols = nullptr;
  int n_pad = pp.Lp;
  if (gather == 1) {          // vertical-stripe head: its column list
    const int* rec = p.ws + p.list_table + 4 * p.list_id[hg];
    cols = p.ws + rec[0];
    n_pad = rec[1];
  } else if (gather == 2) {   // rearranged head: key j of the arrays is row row_map[j] of the tensors
    const int* rec = p.ws + p.list_table + 4 * p.list_id[hg];
    cols = p.ws + rec[3];
    n_pad = pp.map_len;
  }
  quantise_group<D>(pp, blockIdx.x, head, b, cols, n_pad);
}

// All heads of a layer that compute: head records {head, list word offset or -1, list length}.
template <int D>
__global__ void __launch_bounds__(256) quantise_layer_kernel(const Fp8Launch pp, const int head_table, const int n_heads) {
  typedef const int __attribute__((address_space(4)))* const_int_ptr;
  const const_int_ptr r = (const_int_ptr)(uintptr_t)(pp.a.ws + head_table) + (size_t)(blockIdx.y % n_heads) * kGridHeadWords;
  const int list = r[1];
  quantise_group<D>(pp, blockIdx.x, r[0], blockIdx.y / n_heads, list >= 0 ? pp.a.ws + list : nullptr, list >= 0 ? r[2] : pp.Lp);
}

// ---------------------------------------------------------------------------
// Attention on the quantised arrays.
// ---------------------------------------------------------------------------
typedef const i32x2 __attribute__((address_space(4)))* const_int2_ptr;

// One item: see the bf16 kernels.  Everything in it is uniform.
struct Fp8Item {
  int head, b, qblk;
  int n_tiles;
  int t_base;               // DENSE, GATHER: first key tile
  int n_keys;               // DENSE, GATHER: keys of the head's arrays
  const_int2_ptr entries;   // BAND, PBAND
  const_int2_ptr runs;
  const int* row_map;       // PBAND: row of the tensors for every position of the rearranged order
  float* partial;           // split item: where its unnormalised result goes, else nullptr
};

// Orders a wave's LDS accesses across its lanes: what any lane has written is there for the others.  The LDS serves one wave's
// accesses in order, so this emits nothing; it keeps the compiler, which sees single lanes, from moving one past the other.
__device__ __forceinline__ void wave_lds_order() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// smem: 4 * BC * D bytes of LDS, 16-byte aligned.
template <int D, int NW, int BC, int MODE>
__device__ __forceinline__ void fp8_body(const Fp8Launch& pp, const Fp8Item& it, unsigned char* const smem) {
  const AttnLaunch& p = pp.a;
  constexpr bool kBand = MODE == MODE_BAND || MODE == MODE_PBAND;   // walks a CSR list of key tiles
  constexpr int BR = NW * 32;        // query rows per work-group (one 32-row block per wave)
  constexpr int KB2 = BC / 32;       // 32-key blocks per tile
  constexpr int G64 = BC / 64;       // 64-key contraction steps of the second product
  constexpr int KS = D / 64;         // contraction steps of S^T = K Q^T
  constexpr int DB = D / 32;         // 32-row blocks of O^T
  constexpr int TILE_BYTES = BC * D;
  constexpr int LPT = TILE_BYTES / (NW * 1024);   // load instructions per wave, tile and matrix
  static_assert(TILE_BYTES % (NW * 1024) == 0 && LPT >= 1, "tile must split evenly over the waves");
  static_assert(BC % 64 == 0, "key tiles are whole groups of 64");

  unsigned char* const sK = smem;                    // [2][BC][D] bytes, swizzled
  unsigned char* const sV = smem + 2 * TILE_BYTES;   // [2][G64][DB][2 halves][2][32 d][16 keys]

  const int qblk = it.qblk, b = it.b, head = it.head;
  const int n_tiles = it.n_tiles, t_base = it.t_base, n_keys = it.n_keys;
  const const_int2_ptr entries = it.entries, runs = it.runs;
  const int* __restrict__ row_map = it.row_map;

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31;
  const int half = lane >> 5;

  const int64_t base = (int64_t)b * p.stride_b + (int64_t)head * p.stride_h;
  const __bf16* __restrict__ Q = p.q + base;
  __bf16* __restrict__ O = p.out + base;
  const size_t base8 = ((size_t)b * p.H + head) * (size_t)pp.Lp * D;
  const int L = p.L;

  // ---- Q fragments: B operand of S^T = K Q^T (lane: query l32, d = 64 ks + 32 half + 0..31) ----
  const float c_scale = p.scale_log2e * 4.0f;
  const int q0 = qblk * BR + wave * 32;
  i32x8 qf[KS];
  {
    int row = q0 + l32;
    row = row < L ? row : L - 1;
    if (MODE == MODE_PBAND) row = row_map[row];   // the pre-pass moved K and V; Q and O go through the map
    const __bf16* src = Q + (int64_t)row * p.stride_l + half * 32;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const bf16x8 raw = *reinterpret_cast<const bf16x8*>(src + ks * 64 + j * 8);
        const f32x8 x = __builtin_convertvector(raw, f32x8) * c_scale;
        qf[ks][2 * j] = pack_e4m3(sat_e4m3(x[0]), sat_e4m3(x[1]), sat_e4m3(x[2]), sat_e4m3(x[3]));
        qf[ks][2 * j + 1] = pack_e4m3(sat_e4m3(x[4]), sat_e4m3(x[5]), sat_e4m3(x[6]), sat_e4m3(x[7]));
      }
    }
  }

  // Softmax state.  top: the integer reference ceil(row max so far) - 8 of the lane's
  // query, -inf until the lane has seen its first kept key.  Accumulators and row sums
  // are in units of 2^base; base stays 0 unless a reference leaves +-kReach around it.
  // kReach: 2^(reach + 8) a probability, 2^9 a value, 2^24 keys stay below 2^127, and the smallest product
  // that counts, 2^(-reach - 18), above 2^-126.
  constexpr float kHeadroom = 8.0f, kReach = 80.0f;
  f32x16 o[DB];
  f32x4 l4;
  float top = kNegInf, base_ref = 0.f, tile_ref = kNegInf;
  float l = 0.f, l_scale = 1.f;   // row sum; what l4[0], a tile's sum in the units of its P8, counts in it
  bool based = false;   // some lane of the wave has a base other than 0
#pragma unroll
  for (int i = 0; i < 4; ++i) l4[i] = 0.f;
#pragma unroll
  for (int db = 0; db < DB; ++db)
#pragma unroll
    for (int i = 0; i < 16; ++i) o[db][i] = 0.f;

  // A operand of the row-sum MFMA (16x16x128): fed with a P fragment of the
  // 32x32x64 product (lane: query l32, the 32 keys of half `half`), the unit sees
  // column l % 16 and the quarter l / 16 of its contraction range in lane l.
  // Rows 0 and 8 of A are one over the even quarters, rows 4 and 12 over the odd
  // ones, the other rows are zero: element 0 of the result (row 4 * (l / 16),
  // column l % 16) is the sum over the 64 keys of the lane's own query.
  i32x8 sum_a;
  {
    const int m16 = lane & 15, g16 = lane >> 4;
    const bool on = ((m16 & 7) == 0 && (g16 & 1) == 0) || ((m16 & 7) == 4 && (g16 & 1) == 1);
#pragma unroll
    for (int i = 0; i < 8; ++i) sum_a[i] = on ? 0x38383838 : 0;   // 0x38 = 1.0
  }

  // ---- tile loader: buffer loads straight into LDS, 16 bytes per lane, a wave
  // instruction fills 1 KB of LDS linearly.  K8: the XOR swizzle is applied on the
  // global side.  V8: the lane that fills LDS chunk (group, db, half, j, d) fetches
  // bytes 32 half + 16 j .. of row d of the group. ----
  typedef __attribute__((address_space(3))) void* lds_ptr;
  unsigned g_k[LPT], g_v[LPT];
#pragma unroll
  for (int u = 0; u < LPT; ++u) {
    const int n = (wave * LPT + u) * 64 + lane;   // 16-byte chunk of the tile in LDS
    const int r = n * 16 / D, slot = (n * 16 % D) >> 4;
    g_k[u] = (unsigned)(r * D + ((slot ^ swz_k8<D>(r)) << 4));
    const int dd = n & 31, j = (n >> 5) & 1, hh = (n >> 6) & 1, db = (n >> 7) % DB, g = (n >> 7) / DB;
    g_v[u] = (unsigned)(((g * D + db * 32 + dd) << 6) + ((2 * hh + j) << 4));
  }
  const unsigned head_bytes8 = (unsigned)pp.Lp * (unsigned)D;
  const __amdgpu_buffer_rsrc_t rsrc_k =
      __builtin_amdgcn_make_buffer_rsrc((void*)(pp.k8 + base8), 0, (int)head_bytes8, 0x00020000);
  const __amdgpu_buffer_rsrc_t rsrc_v =
      __builtin_amdgcn_make_buffer_rsrc((void*)(pp.v8t + base8), 0, (int)head_bytes8, 0x00020000);
  auto load_tile = [&](auto is_k_tag, const int buf, const int t) {
    constexpr bool IS_K = decltype(is_k_tag)::value != 0;
    const __amdgpu_buffer_rsrc_t rsrc = IS_K ? rsrc_k : rsrc_v;
    unsigned char* dst = (IS_K ? sK : sV) + buf * TILE_BYTES + wave * (LPT * 1024);
    const int tile = kBand ? entries[t].x : t + t_base;
#pragma unroll
    for (int u = 0; u < LPT; ++u)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (lds_ptr)(dst + u * 1024), 16, (int)(IS_K ? g_k[u] : g_v[u]),
                                               (int)((unsigned)tile * (unsigned)TILE_BYTES), 0, 0);
  };

  // per-lane LDS read offsets (everything else is an immediate)
  int k_off[KS][2];   // K fragment: key l32 of a 32-key block, chunks 4 ks + 2 half + {0, 1}
#pragma unroll
  for (int ks = 0; ks < KS; ++ks)
#pragma unroll
    for (int j = 0; j < 2; ++j) k_off[ks][j] = l32 * D + (((4 * ks + 2 * half + j) ^ swz_k8<D>(l32)) << 4);
  const int v_off = half * 1024 + l32 * 16;   // V fragment: row l32 of a 32-row block of d, half `half`

  // ---- S^T = K Q^T for the tile held in K buffer BUF ----
  auto scores = [&](auto buf_tag, f32x16 (&s)[KB2]) {
    constexpr int BUF = decltype(buf_tag)::value;
    const unsigned char* kbase = sK + BUF * TILE_BYTES;
#pragma unroll
    for (int kb2 = 0; kb2 < KB2; ++kb2)
#pragma unroll
      for (int i = 0; i < 16; ++i) s[kb2][i] = 0.f;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
#pragma unroll
      for (int kb2 = 0; kb2 < KB2; ++kb2) {
        const i32x4 a0 = *reinterpret_cast<const i32x4*>(kbase + kb2 * 32 * D + k_off[ks][0]);
        const i32x4 a1 = *reinterpret_cast<const i32x4*>(kbase + kb2 * 32 * D + k_off[ks][1]);
        const i32x8 a = __builtin_shufflevector(a0, a1, 0, 1, 2, 3, 4, 5, 6, 7);
        s[kb2] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a, qf[ks], s[kb2], 0, 0, 0, 0, 0, 0);
      }
    }
  };

  // ---- masks: element (kb2, i) of a lane is key kb2*32 + (i/4)*8 + half*4 + i%4 ----
  // Returns false when nothing was changed.  Band tiles: a bit per element for the range of
  // elements that each run of kept diagonals keeps, as in the bf16 kernel (against a classification of
  // every 32 x 32 block with a comparison per element, 48 heads x 17,550, D = 64: 397 -> 383 us; 12 heads x 5,805 behind a
  // text prefix, D = 128: 84 -> 70.5; 40 heads x 75,600, D = 128: 7.14 -> 6.86 ms).
  auto apply_mask = [&](f32x16 (&s)[KB2], const int t) -> bool {
    if (kBand) {
      const i32x2 ent = entries[t];
      const int kv0 = ent.x * BC;
      const int r0 = (ent.y >> 1) & 0x7fff, rn = ent.y >> 16;
      const int qw0 = __builtin_amdgcn_readfirstlane(q0);
      i32x2 run = runs[r0];
      const int dmin = kv0 - qw0 - 31, dmax = kv0 + BC - 1 - qw0;   // diagonals the wave's part touches
      if (dmin >= run.x && dmax <= run.y && kv0 + BC <= L) return false;   // kept as a whole
      constexpr int WORDS = KB2 / 2;
      unsigned kept[WORDS];
#pragma unroll
      for (int w = 0; w < WORDS; ++w) kept[w] = 0u;
      const int iq = q0 + l32;
      const int rel = kv0 + half * 4 - iq;   // diagonal of the lane's element 0
      for (int r = r0;;) {
        // elements whose keys lie below x: (x / 8) * 4 + min(x % 8, 4)
        int lo = run.x - rel, hi = (run.y < L - 1 - iq ? run.y : L - 1 - iq) - rel + 1;
        lo = lo < 0 ? 0 : (lo > BC ? BC : lo);
        hi = hi < 0 ? 0 : (hi > BC ? BC : hi);
        lo = (lo >> 3) * 4 + ((lo & 7) < 4 ? (lo & 7) : 4);
        hi = (hi >> 3) * 4 + ((hi & 7) < 4 ? (hi & 7) : 4);
#pragma unroll
        for (int w = 0; w < WORDS; ++w) {
          int nl = lo - 32 * w, nh = hi - 32 * w;
          if (WORDS > 1) {
            nl = nl < 0 ? 0 : (nl > 32 ? 32 : nl);
            nh = nh < 0 ? 0 : (nh > 32 ? 32 : nh);
          }
          kept[w] |= (unsigned)((1ull << nh) - 1) & ~(unsigned)((1ull << nl) - 1);
        }
        if (++r >= r0 + rn) break;
        run = runs[r];
      }
#pragma unroll
      for (int kb2 = 0; kb2 < KB2; ++kb2)
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          const int m = __builtin_amdgcn_sbfe((int)kept[kb2 / 2], (kb2 % 2) * 16 + i, 1);
          const float score = s[kb2][i];   // a scalar first: bit_cast of a vector element misreads element 0
          const int x = __builtin_bit_cast(int, score);
          s[kb2][i] = __builtin_bit_cast(float, (x & m) | (__builtin_bit_cast(int, kNegInf) & ~m));
        }
    } else {
      const int limit = n_keys - (t + t_base) * BC - half * 4;
#pragma unroll
      for (int kb2 = 0; kb2 < KB2; ++kb2)
#pragma unroll
        for (int i = 0; i < 16; ++i)
          s[kb2][i] = kb2 * 32 + (i / 4) * 8 + (i % 4) < limit ? s[kb2][i] : kNegInf;
    }
    return true;
  };

  auto tile_max = [&](const f32x16 (&s)[KB2]) {
    float a = kNegInf, bq = kNegInf;   // two chains of v_max3
#pragma unroll
    for (int kb2 = 0; kb2 < KB2; ++kb2)
#pragma unroll
      for (int i = 0; i < 8; i += 2) {
        a = fmaxf(fmaxf(a, s[kb2][i]), s[kb2][i + 1]);
        bq = fmaxf(fmaxf(bq, s[kb2][8 + i]), s[kb2][8 + i + 1]);
      }
    tile_ref = __builtin_ceilf(half_max(fmaxf(a, bq))) - kHeadroom;
  };

  // ---- reference of a tile's probabilities.  P8 of a tile is taken against the row
  // maximum so far, and the second product puts it back into the units of the
  // accumulators: the conversion divides by 2^e and the matrix instruction multiplies
  // by 2^e (its block scale).  Both run at the rate of the forms without a scale (8.4 and
  // 65 cycles a wave, measured), so a reference that moves costs nothing: neither the scores
  // nor the accumulators are touched.  Moving them instead, 112 vector instructions beside
  // the 64 (D = 128) or 128 (D = 64) of a tile, came with 5 % of the tiles of a list of
  // 1,182 and with 77 to 95 % of lists of 18 to 8 (any of a wave's 32 rows asks for it).
  // Both lanes of a query supply the same scale.  (In the 16x16x128 product a lane's scale does
  // not stay with the lane's own bytes, and its neighbours hold other queries here: the row sums
  // run unscaled, tile by tile, and one multiply-add per tile applies the scale.) ----
  auto fold_sum = [&]() {
    l = fmaf(l4[0], l_scale, l);
    l4[0] = 0.f;
  };
  int pf_scale = 127;   // of the probabilities still to be accumulated
  auto settle = [&](f32x16 (&s)[KB2]) -> int {
    fold_sum();
    top = fmaxf(top, tile_ref);
    float e = top;
    const bool far = fabsf(top - base_ref) > kReach && top != kNegInf;
    if (__builtin_expect(__builtin_amdgcn_ballot_w64(far) != 0, 0)) {
      // Scores beyond what exp2 and the accumulators hold in units of 2^base: the lane moves its base to the reference.
      based = true;
      const float shift = far ? top - base_ref : 0.f;
      base_ref += shift;
      const float alpha = shift > 0.f ? __builtin_amdgcn_exp2f(-shift) : 1.0f;   // shift < 0: the lane's first kept key
      const int moved = pf_scale - (int)shift;
      pf_scale = moved < 0 ? 0 : (moved > 254 ? 254 : moved);
      l *= alpha;
#pragma unroll
      for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int i = 0; i < 16; ++i) o[db][i] *= alpha;
    }
    if (__builtin_expect(based, 0)) {
      // A base that has moved once stays for most tiles, and those pay for this alone.  (40 heads x 75,600, D = 128, logits
      // of up to 140 binary orders: 8.2 ms where they paid for the accumulators too, 7.35 so; of up to 9: 7.1 / 7.1.  A
      // reference in the seed of the scores, 16 registers that all other inputs would pay for, spares them this too where
      // a head's logits share one large offset: all at -150: 7.1 ms so, 6.7 with a seed.)
#pragma unroll
      for (int kb2 = 0; kb2 < KB2; ++kb2)
#pragma unroll
        for (int i = 0; i < 16; ++i) s[kb2][i] -= base_ref;
      e -= base_ref;
    }
    return (int)fmaxf(e, -kReach) + 127;   // the exponent's bits; nothing kept yet: any (P is 0)
  };

  // ---- P = exp2(relative score) as E4M3, in the B-operand layout of the second
  // product: byte 16 blk + i of the lane = element i of block 2 g64 + blk ----
  auto exponentiate = [&](const f32x16 (&s)[KB2], i32x8 (&pf)[G64], const int scale) {
    const float sc = __builtin_bit_cast(float, scale << 23);
#pragma unroll
    for (int g64 = 0; g64 < G64; ++g64)
#pragma unroll
      for (int blk = 0; blk < 2; ++blk)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const f32x16& sv = s[g64 * 2 + blk];
          pf[g64][blk * 4 + g] =
              pack_e4m3(__builtin_amdgcn_exp2f(sv[4 * g]), __builtin_amdgcn_exp2f(sv[4 * g + 1]),
                        __builtin_amdgcn_exp2f(sv[4 * g + 2]), __builtin_amdgcn_exp2f(sv[4 * g + 3]), sc);
        }
  };

  // ---- O^T += V^T P^T and l += rowsum(P) for the tile held in V buffer BUF ----
  auto accumulate = [&](auto buf_tag, const i32x8 (&pf)[G64], const int scale) {
    constexpr int BUF = decltype(buf_tag)::value;
    const unsigned char* vbase = sV + BUF * TILE_BYTES + v_off;
    l_scale = __builtin_bit_cast(float, scale << 23);
#pragma unroll
    for (int g64 = 0; g64 < G64; ++g64) {
#pragma unroll
      for (int db = 0; db < DB; ++db) {
        const unsigned char* src = vbase + (g64 * DB + db) * 2048;
        const i32x4 a0 = *reinterpret_cast<const i32x4*>(src);
        const i32x4 a1 = *reinterpret_cast<const i32x4*>(src + 512);
        const i32x8 a = __builtin_shufflevector(a0, a1, 0, 1, 2, 3, 4, 5, 6, 7);
        o[db] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a, pf[g64], o[db], 0, 0, 0, 127, 0, scale);
      }
      if (g64 == 0)
#pragma unroll
        for (int i = 0; i < 4; ++i) l4[i] = 0.f;
      l4 = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(sum_a, pf[g64], l4, 0, 0, 0, 0, 0, 0);
    }
  };
  // What a stage has computed for later ones is used only there: without these
  // anchors the compiler moves part of the matrix instructions and exponentials past the
  // barrier and the branch that follow, away from what hides them.
  auto keep_here = [&](i32x8 (&pf)[G64]) {
#pragma unroll
    for (int g64 = 0; g64 < G64; ++g64) asm volatile("" : "+v"(pf[g64]));
#pragma unroll
    for (int db = 0; db < DB; ++db) asm volatile("" : "+v"(o[db]));
    asm volatile("" : "+v"(l4));
    asm volatile("" : "+v"(tile_ref));
  };

  // ---- the loop, three tiles deep: a stage computes the scores of tile t + 1, the
  // probabilities of tile t and O += P V of tile t - 1, so that nothing in it waits for
  // anything else in it (the FP8 product takes the probabilities of 64 keys at once: in
  // the stage that produces them it would wait for all of them).  On entry LDS holds
  // K(t+1) and V(t-1); K(t+2) and V(t) are requested.  One barrier a stage: two stages to a
  // barrier on rings of four slots measured 3 to 5 % slower at both head sizes.
  // What bounds it: long lists run at the power limit (40 heads of 75,600 tokens, from the table: 7.0
  // ms on normal inputs, 5.6 on zeros, the same instructions with no bits that toggle); a wave's tile
  // at D = 128 asks for 486 cycles of the vector pipe and 544 of the matrix pipe.  Short lists are
  // bound by the vector pipe and what surrounds the loop.  Against a loop two tiles deep whose
  // reference moved scores and accumulators: 48 heads x 17,550, D = 64: 457 -> 400 us; 24 heads x
  // 8,536, D = 128: 230 -> 199 us; 40 heads x 75,600, D = 128, a launch per group: 7.64 -> 7.11 ms. ----
  f32x16 s_a[KB2], s_b[KB2];
  i32x8 pf_a[G64], pf_b[G64];
  // FIRST: t = 0, nothing to accumulate yet.  NEXT: a tile t + 1 exists, so outside band lists nothing of tile t
  // can be masked.
  auto stage = [&](auto par_tag, auto first_tag, auto next_tag, const int t, f32x16 (&s_cur)[KB2], f32x16 (&s_next)[KB2],
                   i32x8 (&pf_prev)[G64], i32x8 (&pf_cur)[G64]) {
    constexpr int PAR = decltype(par_tag)::value;   // t & 1
    constexpr bool FIRST = decltype(first_tag)::value != 0, NEXT = decltype(next_tag)::value != 0;
    if (NEXT && t + 2 < n_tiles) load_tile(Int<1>{}, PAR, t + 2);   // K(t+2) takes the place of K(t), read in the last stage
    load_tile(Int<0>{}, PAR, t);                                    // V(t) takes the place of V(t-2)
    bool masked;
    if (kBand) masked = !(entries[t].y & 1);
    else masked = !NEXT && (t + t_base + 1) * BC > n_keys;
    if (masked && apply_mask(s_cur, t)) tile_max(s_cur);
    const int scale = settle(s_cur);
    if (NEXT) scores(Int<PAR ^ 1>{}, s_next);
    if (!FIRST) accumulate(Int<PAR ^ 1>{}, pf_prev, pf_scale);
    exponentiate(s_cur, pf_cur, scale);
    pf_scale = scale;
    if (NEXT) tile_max(s_next);
    if (NEXT && !FIRST) {
      // Issue order: the first LDS reads and, under them, a few exponentials; then one
      // MFMA, the LDS reads that feed the MFMAs two steps later, and a share of the
      // vector work (0x008 MFMA, 0x100 DS read, 0x002 VALU, 0x400 TRANS).
      constexpr int N_QK = KS * KB2, N_PV = G64 * DB, N_SUM = G64;
      constexpr int N_RD = (N_QK + N_PV) * 2;
      // per score element: one exp2, half a conversion, half a max3
      constexpr int VALU_PER = (KB2 * 16 * 2 + N_QK + N_PV + N_SUM - 1) / (N_QK + N_PV + N_SUM);
      constexpr int AHEAD = 4;   // reads issued ahead of the MFMA that needs them (two MFMAs' worth)
      __builtin_amdgcn_sched_group_barrier(0x100, AHEAD, 0);
      __builtin_amdgcn_sched_group_barrier(0x402, 8, 0);
#pragma unroll
      for (int i = 0; i < N_QK; ++i) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        if (2 * i + AHEAD < N_RD) __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
        __builtin_amdgcn_sched_group_barrier(0x402, VALU_PER, 0);
      }
#pragma unroll
      for (int g = 0; g < G64; ++g) {
#pragma unroll
        for (int j = 0; j < DB; ++j) {
          __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
          if (2 * (N_QK + g * DB + j) + AHEAD < N_RD) __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
          __builtin_amdgcn_sched_group_barrier(0x402, VALU_PER, 0);
        }
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x402, VALU_PER, 0);
      }
    }
    keep_here(pf_cur);
    __syncthreads();   // what was requested has landed, what was read may be overwritten
  };

  if (n_tiles > 0) {
    load_tile(Int<1>{}, 0, 0);
    if (n_tiles > 1) load_tile(Int<1>{}, 1, 1);
  }
  __syncthreads();
  if (n_tiles > 0) {
    scores(Int<0>{}, s_a);
    tile_max(s_a);
  }
  __syncthreads();   // K(0) has been read by every wave before the first stage requests K(2) into its buffer
  // Tile 0 alone, then two stages per trip (odd tile first) so that buffer indices
  // and register sets stay static; after the last stage the probabilities of the
  // last tile are still to be accumulated.
  constexpr Int<0> even{}, no{};
  constexpr Int<1> odd{}, yes{};
  if (n_tiles > 1) {
    stage(even, yes, yes, 0, s_a, s_b, pf_b, pf_a);
    int t = 1;
    for (; t + 2 < n_tiles; t += 2) {
      stage(odd, no, yes, t, s_b, s_a, pf_a, pf_b);
      stage(even, no, yes, t + 1, s_a, s_b, pf_b, pf_a);
    }
    if (t + 1 < n_tiles) {
      stage(odd, no, yes, t, s_b, s_a, pf_a, pf_b);
      stage(even, no, no, t + 1, s_a, s_b, pf_b, pf_a);
      fold_sum();
      accumulate(even, pf_a, pf_scale);
    } else {
      stage(odd, no, no, t, s_b, s_a, pf_a, pf_b);
      fold_sum();
      accumulate(odd, pf_b, pf_scale);
    }
  } else if (n_tiles == 1) {
    stage(even, yes, no, 0, s_a, s_b, pf_b, pf_a);
    accumulate(even, pf_a, pf_scale);
  }
  fold_sum();

  // ---- split launch: leave the chunk's state for the merge kernel (layout of the bf16 kernel) ----
  if (MODE != MODE_PBAND && it.partial) {
    typedef float __attribute__((address_space(1)))* global_float_ptr;   // global stores, not FLAT ones
    global_float_ptr dst = (global_float_ptr)(uintptr_t)(it.partial + (size_t)wave * ((DB * 16 + 2) * 64) + lane);
    // in units of the row's own reference, an exact power of two away: the units of two chunks that count alike can lie
    // 2^128 apart, and a weight of that size is zero in fp32
    const float to_top = top == kNegInf ? 1.0f : __builtin_amdgcn_exp2f(base_ref - top);
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
      for (int i = 0; i < 16; ++i) dst[(db * 16 + i) * 64] = o[db][i] * to_top;
    dst[(DB * 16) * 64] = top;   // -inf: the row has no finite score in this chunk
    dst[(DB * 16 + 1) * 64] = l * to_top;
    return;
  }

  // ---- epilogue: O = O^T / l, bf16, through LDS so that a wave instruction writes 64 or 128 bytes to a row and not 16
  // (see the bf16 kernel; 48 heads x 17,550, D = 64: 388 -> 381 us; 30 heads x 3,892, D = 128: 66.4 -> 60.3; 40 heads x 75,600:
  // 7.13 -> 7.04 ms).  The K tiles are done with: their last reads lie before the last stage's barrier. ----
  constexpr int PD = 2 * TILE_BYTES / NW / 64 < 64 ? 2 * TILE_BYTES / NW / 64 : 64;   // d of the wave's 32 rows at a time
  static_assert(PD == 32 || PD == 64, "a pass is one or two 32-row blocks of O^T");
  constexpr int PC = PD / 8, PR = 64 / PC;   // 16-byte pieces of a row in a pass, rows of a wave instruction
  unsigned char* const stage_out = sK + wave * (64 * PD);
  const float inv = 1.0f / l;
  int to[32 / PR];   // rows that the lane stores to
#pragma unroll
  for (int j = 0; j < 32 / PR; ++j) {
    to[j] = q0 + j * PR + lane / PC;
    if (MODE == MODE_PBAND && to[j] < L) to[j] = row_map[to[j]];
  }
#pragma unroll
  for (int d0 = 0; d0 < DB; d0 += PD / 32) {
#pragma unroll
    for (int db = d0; db < d0 + PD / 32; ++db) {
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const f32x2 a01 = {o[db][g * 4 + 0] * inv, o[db][g * 4 + 1] * inv};
        const f32x2 a23 = {o[db][g * 4 + 2] * inv, o[db][g * 4 + 3] * inv};
        const bf16x2 b01 = __builtin_convertvector(a01, bf16x2);
        const bf16x2 b23 = __builtin_convertvector(a23, bf16x2);
        const bf16x4 out4 = {b01[0], b01[1], b23[0], b23[1]};
        *reinterpret_cast<bf16x4*>(stage_out + l32 * (2 * PD) + ((((db - d0) * 4 + g) ^ (l32 % PC)) << 4) + half * 8) = out4;
      }
    }
    wave_lds_order();
#pragma unroll
    for (int j = 0; j < 32 / PR; ++j) {
      const int r = j * PR + lane / PC;
      const u32x4 piece = *reinterpret_cast<const u32x4*>(stage_out + r * (2 * PD) + (((lane % PC) ^ (r % PC)) << 4));
      if (q0 + r < L) *reinterpret_cast<u32x4*>(O + (int64_t)to[j] * p.stride_l + d0 * 32 + (lane % PC) * 8) = piece;
    }
    wave_lds_order();
  }
}

// One launch per group: work-group = one item.
template <int D, int NW, int BC, int OCC, int MODE>
__global__ void __launch_bounds__(NW * 64, OCC) attn_fwd_fp8_kernel(const Fp8Launch pp) {
  const AttnLaunch& p = pp.a;
  __shared__ __attribute__((aligned(16))) unsigned char smem[4 * BC * D];
  // which tile of which head (XCD-aware: consecutive items share an XCD)
  const int per_xcd = (p.n_items + 7) >> 3;
  const int item = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
  if (item >= p.n_items) return;
  Fp8Item it{};
  it.qblk = item % p.n_q_blocks;
  const int chunk = (item / p.n_q_blocks) % p.split;
  const int hb = item / p.n_q_blocks / p.split;
  const int hg = hb % p.n_heads;
  it.b = hb / p.n_heads;
  it.head = p.heads ? p.heads[hg] : hg;
  it.n_keys = p.L;
  if (MODE == MODE_DENSE) {
    const int n_all = (p.L + BC - 1) / BC;
    it.t_base = chunk * n_all / p.split;
    it.n_tiles = (chunk + 1) * n_all / p.split - it.t_base;
    if (p.split > 1) it.partial = p.partial + (size_t)item * NW * ((D / 32 * 16 + 2) * 64);
  } else {
    const int* rec = p.ws + p.list_table + 4 * p.list_id[hg];
    if (MODE == MODE_BAND || MODE == MODE_PBAND) {
      const int* row_ptr = p.ws + rec[0];
      const int e0 = row_ptr[it.qblk], e1 = row_ptr[it.qblk + 1];
      it.entries = (const_int2_ptr)(uintptr_t)(p.ws + rec[1]) + e0;
      it.runs = (const_int2_ptr)(uintptr_t)(p.ws + rec[2]);
      it.n_tiles = e1 - e0;
      if (it.n_tiles == 0) return;   // rows that another launch computes (text rows of a layer with a text prefix)
      if (MODE == MODE_PBAND) it.row_map = p.ws + rec[3];
    } else {
      if (it.qblk < p.skip_q_blocks) return;   // text rows: another launch computes them
      it.n_tiles = rec[1] / BC;
      it.n_keys = rec[2];
    }
  }
  fp8_body<D, NW, BC, MODE>(pp, it, smem);
}

// The layer in one launch, work-group = one record of the plan's table of items (see the bf16 kernel).
template <int D, int NW, int BC>
__global__ void __launch_bounds__(NW * 64, 2) attn_grid_fp8_kernel(const Fp8Launch pp, const int table) {
  __shared__ __attribute__((aligned(16))) unsigned char smem[4 * BC * D];
  typedef const int __attribute__((address_space(4)))* const_int_ptr;
  const const_int_ptr r = (const_int_ptr)(uintptr_t)(pp.a.ws + table) + (size_t)blockIdx.x * kGridWords;
  if (r[0] < 0) return;
  const int kind = r[0] & 255, t0 = r[0] >> 8;
  Fp8Item it{};
  it.head = r[1];
  it.b = r[2];
  it.qblk = r[3];
  it.n_tiles = r[4];
  const int list = r[5], more = r[6], last = r[7];
  it.t_base = t0;
  it.n_keys = kind == SEG_GATHER ? more : pp.a.L;
  if (kind == SEG_BAND || kind == SEG_PBAND) {
    it.entries = (const_int2_ptr)(uintptr_t)(pp.a.ws + list) + t0;
    it.runs = (const_int2_ptr)(uintptr_t)(pp.a.ws + more);
  }
  if (kind == SEG_PBAND) it.row_map = pp.a.ws + last;
  else if (last >= 0) it.partial = pp.a.partial + (size_t)last * NW * ((D / 32 * 16 + 2) * 64);
  switch (kind) {
    case SEG_DENSE: fp8_body<D, NW, BC, MODE_DENSE>(pp, it, smem); break;
    case SEG_BAND: fp8_body<D, NW, BC, MODE_BAND>(pp, it, smem); break;
    case SEG_GATHER: fp8_body<D, NW, BC, MODE_GATHER>(pp, it, smem); break;
    case SEG_PBAND: fp8_body<D, NW, BC, MODE_PBAND>(pp, it, smem); break;
    default: {   // zero fill of kGridZeroRows rows of a skipped head
      __bf16* O = pp.a.out + (int64_t)it.b * pp.a.stride_b + (int64_t)it.head * pp.a.stride_h;
      constexpr int CH = D / 8;
      for (int c = threadIdx.x; c < kGridZeroRows * CH; c += NW * 64) {
        const int row = it.qblk * kGridZeroRows + c / CH;
        if (row < pp.a.L) *reinterpret_cast<u32x4*>(O + (int64_t)row * pp.a.stride_l + (c % CH) * 8) = u32x4{0u, 0u, 0u, 0u};
      }
    }
  }
}

template <int D, int NW, int BC, int OCC>
hipError_t launch_mode_fp8(const Fp8Launch& p, int mode, hipStream_t stream) {
  const int per_xcd = (p.a.n_items + 7) / 8;
  const dim3 grid(per_xcd * 8), block(NW * 64);
  switch (mode) {
    case MODE_DENSE:
      hipLaunchKernelGGL((attn_fwd_fp8_kernel<D, NW, BC, OCC, MODE_DENSE>), grid, block, 0, stream, p);
      break;
    case MODE_BAND:
      hipLaunchKernelGGL((attn_fwd_fp8_kernel<D, NW, BC, OCC, MODE_BAND>), grid, block, 0, stream, p);
      break;
    case MODE_GATHER:
      hipLaunchKernelGGL((attn_fwd_fp8_kernel<D, NW, BC, OCC, MODE_GATHER>), grid, block, 0, stream, p);
      break;
    case MODE_PBAND:
      hipLaunchKernelGGL((attn_fwd_fp8_kernel<D, NW, BC, OCC, MODE_PBAND>), grid, block, 0, stream, p);
      break;
    default:
      return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace

hipError_t launch_quantise_kv(const Fp8Launch& p, int mode, hipStream_t stream) {
  if (p.a.n_heads <= 0) return hipSuccess;
  if (!p.k8 || !p.v8t || p.Lp != fp8_padded_len(p.a.L)) return hipErrorInvalidValue;
  const dim3 grid(p.Lp / 64, p.a.n_heads * p.a.B), block(256);
  const int gather = mode == MODE_GATHER ? 1 : mode == MODE_PBAND ? 2 : 0;
  if (gather == 2 && (p.map_len < 1 || p.map_len > p.Lp)) return hipErrorInvalidValue;
  if (p.a.D == 128) hipLaunchKernelGGL(quantise_kv_kernel<128>, grid, block, 0, stream, p, gather);
  else if (p.a.D == 64) hipLaunchKernelGGL(quantise_kv_kernel<64>, grid, block, 0, stream, p, gather);
  else return hipErrorInvalidValue;
  return hipGetLastError();
}

hipError_t launch_attention_fp8(const Fp8Launch& p, int mode, hipStream_t stream, bool small_q) {
  if (p.a.n_items <= 0) return hipSuccess;
  if (!p.k8 || !p.v8t || p.Lp != fp8_padded_len(p.a.L)) return hipErrorInvalidValue;
  if (p.a.split < 1 || (p.a.split > 1 && (mode != MODE_DENSE || !p.a.partial))) return hipErrorInvalidValue;
  if (small_q) {   // small query tile: the band modes, and the compacted stripe heads (no list depends on it)
    if (mode != MODE_BAND && mode != MODE_PBAND && mode != MODE_GATHER) return hipErrorInvalidValue;
    const int per_xcd = (p.a.n_items + 7) / 8;
    const dim3 grid(per_xcd * 8);
    if (p.a.D == 128) {
      using T = Tile128s;
      if (mode == MODE_BAND) hipLaunchKernelGGL((attn_fwd_fp8_kernel<128, T::NW, T::BC, T::OCC, MODE_BAND>), grid, dim3(T::NW * 64), 0, stream, p);
      else if (mode == MODE_PBAND) hipLaunchKernelGGL((attn_fwd_fp8_kernel<128, T::NW, T::BC, T::OCC, MODE_PBAND>), grid, dim3(T::NW * 64), 0, stream, p);
      else hipLaunchKernelGGL((attn_fwd_fp8_kernel<128, T::NW, T::BC, T::OCC, MODE_GATHER>), grid, dim3(T::NW * 64), 0, stream, p);
    } else if (p.a.D == 64) {
      using T = Tile64s;
      if (mode == MODE_BAND) hipLaunchKernelGGL((attn_fwd_fp8_kernel<64, T::NW, T::BC, T::OCC, MODE_BAND>), grid, dim3(T::NW * 64), 0, stream, p);
      else if (mode == MODE_PBAND) hipLaunchKernelGGL((attn_fwd_fp8_kernel<64, T::NW, T::BC, T::OCC, MODE_PBAND>), grid, dim3(T::NW * 64), 0, stream, p);
      else hipLaunchKernelGGL((attn_fwd_fp8_kernel<64, T::NW, T::BC, T::OCC, MODE_GATHER>), grid, dim3(T::NW * 64), 0, stream, p);
    } else {
      return hipErrorInvalidValue;
    }
    return hipGetLastError();
  }
  // the tiles are those of the bf16 kernels, so one plan serves both
  static_assert(Tile128::QB == 1 && Tile64::QB == 1, "the FP8 kernel keeps one 32-row block per wave");
  if (p.a.D == 128) return launch_mode_fp8<128, Tile128::NW, Tile128::BC, Tile128::OCC>(p, mode, stream);
  if (p.a.D == 64) return launch_mode_fp8<64, Tile64::NW, Tile64::BC, Tile64::OCC>(p, mode, stream);
  return hipErrorInvalidValue;
}

template <int D, int BC>
static hipError_t launch_grid_fp8_shape(const Fp8Launch& p, const GridLaunch& g, hipStream_t stream) {
  constexpr int NW = 4;
  const dim3 heads(p.Lp / 64, g.n_heads * p.a.B);
  if (g.n_heads > 0) hipLaunchKernelGGL(quantise_layer_kernel<D>, heads, dim3(256), 0, stream, p, g.head_table, g.n_heads);
  if (hipError_t e = hipGetLastError(); e != hipSuccess) return e;
  hipLaunchKernelGGL((attn_grid_fp8_kernel<D, NW, BC>), dim3(g.n_blocks), dim3(NW * 64), 0, stream, p, g.table);
  return hipGetLastError();
}

hipError_t launch_grid_fp8(const Fp8Launch& p, const GridLaunch& g, hipStream_t stream) {
  if (g.n_blocks < 1) return hipSuccess;
  if (!p.k8 || !p.v8t || p.Lp != fp8_padded_len(p.a.L) || !p.a.ws || g.waves != 4) return hipErrorInvalidValue;
  if (g.n_merges > 0 && !p.a.partial) return hipErrorInvalidValue;
  hipError_t e = hipErrorInvalidValue;
  if (p.a.D == 128) e = launch_grid_fp8_shape<128, Tile128s::BC>(p, g, stream);
  if (p.a.D == 64) e = launch_grid_fp8_shape<64, Tile64s::BC>(p, g, stream);
  return e == hipSuccess ? launch_grid_merge(g, stream) : e;
}

}  // namespace svd
