// gfx950 (MI355X, CDNA4) kernels of the sparse attention forward.
//
// One kernel template serves the three computing modes of Section 4.2:
//   DENSE   M_0, Eq. 1 over every key block
//   BAND    M_2 / M_3 (Section 4.1.2 diagonal and multi-diagonal patterns):
//           key blocks come from a CSR list, partially kept tiles are masked
//           element-wise against the runs of kept diagonals
//   GATHER  M_4 (vertical-stripe pattern): key rows are gathered through the
//           head's sorted column list
// plus a fill kernel for M_1 (skipped heads, zeros).  A launch covers all heads
// of a group (Section 4.2: heads sharing a mode are fused).
//
// Per work-group: one tile of BR query rows of one head.  Online-softmax
// recurrence over the listed key tiles; scores are computed TRANSPOSED,
// S^T = K Q^T with v_mfma_f32_32x32x16_bf16, so that a lane owns one query
// column: the row maximum is a per-lane scalar (one cross-half exchange), and
// the exponentiated scores already sit in the operand layout of the second
// product O^T += V^T P^T.  V^T fragments come from the row-major V tile in LDS
// through the transposing LDS read (ds_read_b64_tr_b16).  Accumulation, scores
// and softmax are fp32; P is rounded to bf16 for the second product, and its
// row sums are taken on the matrix pipe.
//
// K and V tiles travel global -> LDS directly (buffer loads with the LDS bit),
// one tile ahead of their use.  The loop is software-pipelined inside each
// wave: while the VALU turns the scores of tile t into P, the matrix pipe
// already computes the scores of tile t + 1; K therefore runs one tile ahead of
// V through the LDS buffers.  The vector work per score is one exp2, half a
// conversion and half a max3: Q carries log2(e) / sqrt(D), and the score
// accumulators are seeded with minus the reference exponent.
#include <hip/hip_runtime.h>

#include <cstdint>
#include <type_traits>

#include "attn_kernels.h"

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
typedef int i32x2 __attribute__((ext_vector_type(2)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));
typedef __attribute__((address_space(3))) s16x4 lds_s16x4;

constexpr float kNegInf = -__builtin_inff();

// Exchange between the two half-waves (lanes l and l ^ 32) with
// v_permlane32_swap: given (a, b) it returns {a.lower | b.lower moved up,
// a.upper moved down | b.upper}; with a == b == x every lane gets the value of
// the lower-half lane of its pair and that of the upper-half lane.
__device__ __forceinline__ void half_pair(float x, float* own_lo, float* own_hi) {
  const unsigned a = __builtin_bit_cast(unsigned, x);
  const auto r = __builtin_amdgcn_permlane32_swap(a, a, false, false);
  const unsigned r0 = r[0], r1 = r[1];   // scalars first: bit_cast of a vector element misreads lane 0
  *own_lo = __builtin_bit_cast(float, r0);
  *own_hi = __builtin_bit_cast(float, r1);
}
__device__ __forceinline__ float half_max(float x) {
  float lo, hi;
  half_pair(x, &lo, &hi);
  return fmaxf(lo, hi);
}

// 16-byte chunk swizzles of the LDS tiles (row = key, chunk = 8 bf16 of D).
// K is read 16 bytes per lane with consecutive lanes on consecutive keys; V is
// read through the transposing read, 4 keys x 64 bytes per half-wave.  Both
// depend only on row bits that are lane bits at the reading side.
template <int D>
__device__ __forceinline__ int swz_k(int row) {
  return D == 128 ? (row & 15) : ((row >> 1) & 7);
}
template <int D>
__device__ __forceinline__ int swz_v(int row) {
  return D == 128 ? ((row & 3) << 2) : (((row >> 1) & 1) << 2);
}

template <int N>
using Int = std::integral_constant<int, N>;

// Uniform values held in vector registers (arguments of a non-inlined function, words loaded
// through a vector load) moved to scalar registers; a no-op on values that already are scalar.
__device__ __forceinline__ int uni(int x) { return __builtin_amdgcn_readfirstlane(x); }
// (Every pointer that goes through here points into global memory.  Rebuilt from two integers it
// would be a pointer of unknown address space and every access through it a FLAT access, which is
// slower and shares the LDS counter; the detour through the global address space keeps them global.)
template <typename T>
__device__ __forceinline__ T* uni(T* ptr) {
  const unsigned long long u = (unsigned long long)ptr;
  const unsigned lo = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)u);
  const unsigned hi = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)(u >> 32));
  typedef T __attribute__((address_space(1)))* global_ptr;
  return (T*)(global_ptr)(uintptr_t)(((unsigned long long)hi << 32) | lo);
}
__device__ __forceinline__ int64_t uni(int64_t x) {
  const unsigned lo = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)(unsigned long long)x);
  const unsigned hi = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)((unsigned long long)x >> 32));
  return (int64_t)(((unsigned long long)hi << 32) | lo);
}
__device__ __forceinline__ float uni(float x) {
  return __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, x)));
}
// a pointer into the constant address space (the plan's lists), made scalar
template <typename T>
__device__ __forceinline__ const T __attribute__((address_space(4)))* uni_const(const T __attribute__((address_space(4)))* ptr) {
  const unsigned long long u = (unsigned long long)(uintptr_t)ptr;
  const unsigned lo = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)u);
  const unsigned hi = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)(u >> 32));
  return (const T __attribute__((address_space(4)))*)(uintptr_t)(((unsigned long long)hi << 32) | lo);
}

// The band lists are read through the constant address space: the plan's
// workspace is never written by a kernel while lists in it are read, and loads with
// a uniform address from that space are scalar loads, which neither queue behind nor
// wait for the tile loads in flight.
typedef const i32x2 __attribute__((address_space(4)))* const_int2_ptr;

// One item = one tile of BR query rows of one head and the key tiles it walks (for
// a split item: one chunk of them).  Everything in it is uniform.
struct Item {
  int head, b, qblk;
  int n_tiles;
  int t_base;               // DENSE: first key tile
  const_int2_ptr entries;   // BAND, PBAND: the item's part of the CSR list
  const_int2_ptr runs;      // BAND, PBAND
  const int* index;         // PBAND: the row map; COLS: the column list from the item's first tile on
  int n_cols;               // GATHER, COLS: the head's columns from the item's first tile on
  const __bf16* gathered;   // GATHER: the head's gathered K rows from the item's first tile on; V rows follow gather_pad rows later
  float* partial;           // split item: where its unnormalised result goes, else nullptr
};

// LDS of a work-group: two K and two V tiles, and a ring of the key rows of four tiles for the
// modes that reach them through an index list.  Five objects and not one, so that the compiler
// can tell a transposing read of one V tile from the tile loads into the other buffers: out of
// one array every stage waited, before the first of its V reads, after a third of its MFMAs, for the
// loads that it had requested itself.  (42 heads x 32,760, D = 128: 2,596 -> 2,551 us; 40 heads x
// 75,600, 18 of them dense, layer kernel: 43.56 -> 42.90 ms; short layers the same.  Whole dense items two to a
// unit while other units idle, where power is no limit, lose by it: one dense head and ten sparse ones x 30,156, D = 64, 359 ->
// 377; three and six x 15,626, D = 128, 394 -> 402.)
enum { LDS_K0, LDS_K1, LDS_V0, LDS_V1, LDS_INDEX };
template <int D, int BC, int PART>
__device__ __forceinline__ unsigned char* lds_part() {
  __shared__ __attribute__((aligned(16))) unsigned char part[PART == LDS_INDEX ? 4 * BC * 4 : BC * D * 2];
  return part;
}

// Orders a wave's LDS accesses across its lanes: what any lane has written is there for the others.  The LDS serves one wave's
// accesses in order, so this emits nothing; it keeps the compiler, which sees single lanes, from moving one past the other.
__device__ __forceinline__ void wave_lds_order() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Everything a work-group does between picking the item and storing its rows.  K, V: first rows
// of the item's head (or of its gathered arrays).  CALLEE: part of the layer kernel.  Every wave of the work-group calls it
// with the same item; a return leaves no wave behind at a barrier (all returns are
// work-group uniform).
template <int D, int NW, int QB, int BC, int OCC, int MODE, bool CALLEE>
__device__ __forceinline__ void attn_body(const AttnLaunch& p, const Item& it, const __bf16* const K, const __bf16* const V,
                                          unsigned char* const k0, unsigned char* const k1, unsigned char* const v0,
                                          unsigned char* const v1, unsigned char* const sI) {
  constexpr bool kBand = MODE == MODE_BAND || MODE == MODE_PBAND;        // walks a CSR list of key tiles
  constexpr bool kIndirect = MODE == MODE_PBAND || MODE == MODE_COLS;   // key rows come through an index list
  constexpr bool kGathered = MODE == MODE_GATHER;  // K and V are the group's gathered rows: a short dense head
  constexpr int NT = NW * 64;
  constexpr int QW = QB * 32;       // query rows per wave
  constexpr int BR = NW * QW;       // query rows per work-group
  constexpr int CH = D / 8;         // 16-byte chunks per row
  constexpr int KB2 = BC / 32;      // 32-key blocks per tile
  constexpr int KS = D / 16;        // contraction steps of S^T = K Q^T
  constexpr int DB = D / 32;        // 32-row blocks of O^T
  static_assert(BC * CH % NT == 0, "tile must split evenly over the threads");
  constexpr int TILE_BYTES = BC * D * 2;
  constexpr int ROW_BYTES = D * 2;

  unsigned char* const sK[2] = {k0, k1};   // each [BC][D] bf16, swizzled
  unsigned char* const sV[2] = {v0, v1};   // sI: [4][BC] key rows, slot = tile & 3 (kIndirect)

  const int qblk = it.qblk, head = it.head, b = it.b;
  const int n_tiles = it.n_tiles, t_base = it.t_base, n_cols = it.n_cols;
  const const_int2_ptr entries = it.entries, runs = it.runs;
  const int* __restrict__ cols = it.index;

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // uniform: keeps everything derived from it in scalar registers
  const int l32 = lane & 31;
  const int half = lane >> 5;

  const int64_t base = (int64_t)b * p.stride_b + (int64_t)head * p.stride_h;
  const __bf16* __restrict__ Q = p.q + base;
  __bf16* __restrict__ O = p.out + base;
  const int L = p.L;

  // ---- Q fragments: B operand of S^T = K Q^T (lane: query l32, 8 of 16 d) ----
  // Q is multiplied by log2(e) / sqrt(D) here, once, and rounded back to bf16:
  // the scores then come out of the matrix pipe in the exponent domain of exp2
  // and need no per-element scaling.
  const float c_scale = p.scale_log2e;
  const int q0 = qblk * BR + wave * QW;
  bf16x8 qf[QB][KS];
#pragma unroll
  for (int qb = 0; qb < QB; ++qb) {
    int row = q0 + qb * 32 + l32;
    row = row < L ? row : L - 1;
    if (MODE == MODE_PBAND) row = cols[row];   // position of the rearranged order -> row of the tensor
    const __bf16* src = Q + (int64_t)row * p.stride_l + half * 8;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      const bf16x8 raw = *reinterpret_cast<const bf16x8*>(src + ks * 16);
      const f32x8 scaled = __builtin_convertvector(raw, f32x8) * c_scale;
      qf[qb][ks] = __builtin_convertvector(scaled, bf16x8);
    }
  }

  // Softmax state per 32-row block.  Scores are kept RELATIVE to a reference
  // exponent: the score accumulators start from nm = -reference (16 copies, the
  // C operand of the first MFMA of a block), so exp2 applies to the MFMA result
  // as it is.  thr is the excess over the reference that makes the lane move
  // it: -inf until the lane has seen its first kept key, kLazyLog2 afterwards.
  // The row sums accumulate in element 0 of l4 through a small MFMA.
  constexpr float kLazyLog2 = 8.0f;
  f32x16 o[DB][QB], nm[QB];
  f32x4 l4[QB];
  float thr[QB], mx_raw[QB];
#pragma unroll
  for (int qb = 0; qb < QB; ++qb) {
    thr[qb] = kNegInf;
    mx_raw[qb] = kNegInf;
#pragma unroll
    for (int i = 0; i < 4; ++i) l4[qb][i] = 0.f;
#pragma unroll
    for (int i = 0; i < 16; ++i) nm[qb][i] = 0.f;
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
      for (int i = 0; i < 16; ++i) o[db][qb][i] = 0.f;
  }
  // A operand of the row-sum MFMA (16x16x32): fed with a P fragment laid out for
  // the 32x32x16 product (lane: query l32, 8 keys of half `half`), the 16x16x32
  // unit sees query l%16 + 16*((l/16)&1) and keys 8*(l/32).. in lane l.  Rows 0
  // and 8 of A select the lanes of the even 16-lane blocks, rows 4 and 12 those
  // of the odd ones, all other rows are zero: element 0 of the result (row
  // 4*(l/16), column l%16) is then the sum over the 16 keys of the lane's own
  // query, in every lane.
  bf16x8 sum_a;
  {
    const int m16 = lane & 15, g16 = lane >> 4;
    const bool on = ((m16 & 7) == 0 && (g16 & 1) == 0) || ((m16 & 7) == 4 && (g16 & 1) == 1);
    const __bf16 v = on ? (__bf16)1.0f : (__bf16)0.0f;
#pragma unroll
    for (int i = 0; i < 8; ++i) sum_a[i] = v;
  }

  // ---- tile loader: direct global -> LDS loads (buffer_load_dwordx4 with the LDS bit: 16 bytes
  // per lane, a wave instruction fills 1 KB of LDS linearly from a uniform base,
  // no staging registers).  Wave w fills the slabs w*LPT .. w*LPT+LPT-1 of a tile.
  // The XOR swizzle is applied on the global side: the lane that fills chunk
  // slot c' of row r fetches chunk c' ^ swz(r) of that key row, so K and V use
  // different per-lane offsets.  A tile is addressed as a uniform base (scalar
  // register) plus those 32-bit offsets.  Rows past the head's last one lie past the range of
  // its buffer, the uniform base counted in: the hardware delivers zeros (and the scores are
  // masked), so a list's last tiles take the code of the others.  A test for a ragged tile, with
  // rows clamped to L - 1, around every load of the last four stages of a list, one plan run again and again: 12 heads x
  // 1,998 x 2, D = 128: 55.7 us against 53.1 without; 24 heads x 2,352, D = 128: 86.0 / 82.3; 48 x 17,550, D = 64:
  // 530 / 522. ----
  constexpr int LPT = TILE_BYTES / (NW * 1024);   // load instructions per wave, tile and matrix
  static_assert(TILE_BYTES % (NW * 1024) == 0, "tile must split evenly over the waves");
  typedef __attribute__((address_space(3))) void* lds_ptr;
  const unsigned stride_bytes = kGathered ? (unsigned)ROW_BYTES : (unsigned)p.stride_l * 2u;   // of a key row
  unsigned g_k[LPT], g_v[LPT];   // byte offset inside the tile; kIndirect: chunk offset inside the row
  unsigned g_r[LPT];             // kIndirect: 4 * row of the slab's lane inside the tile
#pragma unroll
  for (int u = 0; u < LPT; ++u) {
    const int byte = (wave * LPT + u) * 1024 + lane * 16;
    const int r = byte / ROW_BYTES, slot = (byte % ROW_BYTES) >> 4;
    const unsigned ck = (unsigned)(slot ^ swz_k<D>(r)) * 16u, cv = (unsigned)(slot ^ swz_v<D>(r)) * 16u;
    g_r[u] = (unsigned)r * 4u;
    g_k[u] = kIndirect ? ck : (unsigned)r * stride_bytes + ck;
    g_v[u] = kIndirect ? cv : (unsigned)r * stride_bytes + cv;
  }
  // buffer resources of this head's K and V (raw buffers: base, byte range, no swizzle)
  const unsigned head_bytes = kGathered ? (unsigned)n_tiles * (unsigned)TILE_BYTES
                                        : (unsigned)(L - 1) * stride_bytes + (unsigned)ROW_BYTES;
  const __amdgpu_buffer_rsrc_t rsrc_k = __builtin_amdgcn_make_buffer_rsrc((void*)K, 0, (int)head_bytes, 0x00020000);
  const __amdgpu_buffer_rsrc_t rsrc_v = __builtin_amdgcn_make_buffer_rsrc((void*)V, 0, (int)head_bytes, 0x00020000);
  // Key rows through an index list.  An index read in the loop from memory would hold up
  // the tile load that needs it by a whole trip (and wait, in order, for every load in
  // flight); so the indices of a tile travel to LDS one stage ahead of its K.  -1 =
  // padding (request_rows below).
  // Rearranged window of 8 heads x 75,600, D = 128: 632 us with the indices read from
  // memory, 618 with the ring.  Column lists read this way cost the loop nothing
  // measurable and save the pre-pass that gathers K and V rows (5-8 us ahead of the layer:
  // 24 heads x 2,352, D = 128: 44.9 -> 40.3 us; 4 x 1,024, D = 64: 16.2 -> 13.1).
  const __amdgpu_buffer_rsrc_t rsrc_i = __builtin_amdgcn_make_buffer_rsrc(
      (void*)cols, 0, (MODE == MODE_PBAND ? (L + BC - 1) / BC : n_tiles) * BC * 4, 0x00020000);
  auto index_base = [&](const int t) { return (MODE == MODE_PBAND ? entries[t].x : t) * BC; };
  auto load_index = [&](const int t) {
    if (wave < BC / 64)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc_i, (lds_ptr)(sI + ((t & 3) * BC + wave * 64) * 4), 4,
                                               lane * 4 + wave * 256, index_base(t) * 4, 0, 0);
  };
  // kIndirect: byte offsets of the slabs' rows in the tile whose K was requested last, kept for its V in the next stage (both
  // formed from the ring: 24 heads x 1,998, 200 columns, D = 128: 17.5 -> 16.2 us; window of 8 heads x 75,600: 596 -> 584).
  // V(t + 1) is therefore requested before K(t + 2), or with a copy of them.
  unsigned row_at[LPT];
  // kIndirect: the request of a wave's slabs whose rows start at these offsets, at these of their chunks.  Padding starts at
  // 2^32 - 16, past every head's end, and the sum with the chunk wraps.  For V the larger of the two is taken: zeros (P is 0 there,
  // but the memory may hold infinities).  For K it may read the head's first row: those scores are masked.  (A start 256 bytes
  // lower, without the maximum, lies inside the last row of heads that end there; the maximum for K as well: 24 heads x 1,998, 200
  // columns, D = 128, 15.5 -> 15.9 us.)
  auto request_rows = [&](auto is_k_tag, const __amdgpu_buffer_rsrc_t rsrc, unsigned char* const dst, const unsigned (&rows)[LPT],
                          const unsigned (&chunk)[LPT]) {
#pragma unroll
    for (int u = 0; u < LPT; ++u)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (lds_ptr)(dst + u * 1024), 16, (int)(decltype(is_k_tag)::value ? rows[u] + chunk[u] : max(rows[u], rows[u] + chunk[u])), 0, 0, 0);
  };
  // FIRST: the prologue's loads, whose indices are read from memory
  auto load_tile = [&](auto is_k_tag, const int buf, const int t, auto first_tag) {
    constexpr bool IS_K = decltype(is_k_tag)::value != 0;
    constexpr bool FIRST = decltype(first_tag)::value != 0;
    const __amdgpu_buffer_rsrc_t rsrc = IS_K ? rsrc_k : rsrc_v;
    unsigned char* dst = (IS_K ? sK : sV)[buf] + wave * (LPT * 1024);
    if (kIndirect) {
      if (IS_K) {
        int c[LPT];
#pragma unroll
        for (int u = 0; u < LPT; ++u)
          c[u] = FIRST ? *reinterpret_cast<const int*>(reinterpret_cast<const char*>(cols + index_base(t)) + g_r[u])
                       : *reinterpret_cast<const int*>(sI + (t & 3) * (BC * 4) + g_r[u]);
#pragma unroll
        for (int u = 0; u < LPT; ++u) row_at[u] = c[u] < 0 ? 0xfffffff0u : __umul24((unsigned)c[u], stride_bytes);
      }
      request_rows(is_k_tag, rsrc, dst, row_at, IS_K ? g_k : g_v);
    } else {
      const int row0 = (kBand ? entries[t].x : t + t_base) * BC;
#pragma unroll
      for (int u = 0; u < LPT; ++u)
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (lds_ptr)(dst + u * 1024), 16, (int)(IS_K ? g_k[u] : g_v[u]),
                                                 (int)((unsigned)row0 * stride_bytes), 0, 0);
    }
  };

  // per-lane LDS read offsets (everything else is an immediate)
  int k_off[KS];   // K fragment: key l32 of a 32-key block, chunk 2 * ks + half
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) k_off[ks] = l32 * ROW_BYTES + (((2 * ks + half) ^ swz_k<D>(l32)) << 4);
  const int ti = lane & 15;           // lane inside its block of 16
  const int dsel = (lane >> 4) & 1;   // which 16 of the 32 d rows
  int v_off[DB];   // V^T fragment: key row half*4 + ti/4 of a 16-key step, 4 d from db*32 + dsel*16 + (ti%4)*4
#pragma unroll
  for (int db = 0; db < DB; ++db) {
    const int r = half * 4 + (ti >> 2);
    const int c = db * 4 + 2 * dsel + ((ti & 3) >> 1);
    v_off[db] = r * ROW_BYTES + ((c ^ swz_v<D>(r)) << 4) + ((ti & 1) << 3);
  }

  // ---- S^T = K Q^T for the tile held in K buffer BUF ----
  auto scores = [&](auto buf_tag, f32x16 (&s)[KB2][QB]) {
    constexpr int BUF = decltype(buf_tag)::value;
    const unsigned char* kbase = sK[BUF];
#pragma unroll
    for (int kb2 = 0; kb2 < KB2; ++kb2)
#pragma unroll
      for (int qb = 0; qb < QB; ++qb) s[kb2][qb] = nm[qb];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
#pragma unroll
      for (int kb2 = 0; kb2 < KB2; ++kb2) {
        const bf16x8 a = *reinterpret_cast<const bf16x8*>(kbase + kb2 * 32 * ROW_BYTES + k_off[ks]);
#pragma unroll
        for (int qb = 0; qb < QB; ++qb)
          s[kb2][qb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, qf[qb][ks], s[kb2][qb], 0, 0, 0);
      }
    }
  };

  // ---- masks: element (kb2, i) of a lane is key kb2*32 + (i/4)*8 + half*4 + i%4 ----
  // Returns false when nothing was changed (the wave's part of the tile is kept as a whole).
  // Band tiles: the elements of a lane ascend with their keys, so a run of kept diagonals keeps a
  // range of them: one bit per element in a word or two per lane, then a sign-extended bit and a
  // bitwise select per element, in place, whatever the number of runs and edges.  (A classification
  // of every 32 x 32 block, with a comparison and a conditional move per element in the blocks that
  // an edge crosses, issues no more vector instructions, but its branches cost copies of the
  // scores where they meet: 1,500 cycles a masked tile at D = 128 where a whole tile takes 2,200, and
  // 30 KB of code per mode.  Band heads of 81 diagonals around five offsets, 24 heads x 1,998, D = 128:
  // 50.8 -> 47.6 us; a layer of 12 heads x 1,998 x 2: 46.7 -> 40.0; 4 x 1,024, D = 64: 13.2 -> 11.9.)
  auto apply_mask = [&](f32x16 (&s)[KB2][QB], const int t) -> bool {
    bool changed = false;
    if (kBand) {
      const i32x2 ent = entries[t];
      const int kv0 = ent.x * BC;
      const int r0 = (ent.y >> 1) & 0x7fff, rn = ent.y >> 16;
      const int qw0 = __builtin_amdgcn_readfirstlane(q0);
      const i32x2 first = runs[r0];
#pragma unroll
      for (int qb = 0; qb < QB; ++qb) {
        const int dmin = kv0 - (qw0 + qb * 32) - 31, dmax = kv0 + BC - 1 - (qw0 + qb * 32);   // diagonals the wave's part touches
        if (dmin >= first.x && dmax <= first.y && kv0 + BC <= L) continue;   // kept as a whole
        changed = true;
        constexpr int WORDS = KB2 / 2;
        unsigned kept[WORDS];
#pragma unroll
        for (int w = 0; w < WORDS; ++w) kept[w] = 0u;
        const int iq = q0 + qb * 32 + l32;
        const int rel = kv0 + half * 4 - iq;   // diagonal of the lane's element 0
        i32x2 run = first;
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
            const float score = s[kb2][qb][i];   // a scalar first: bit_cast of a vector element misreads element 0
            const int x = __builtin_bit_cast(int, score);
            s[kb2][qb][i] = __builtin_bit_cast(float, (x & m) | (__builtin_bit_cast(int, kNegInf) & ~m));
          }
      }
    } else {
      // dense: keys past L in the last tile; gather: padding of the column list
      // (the lane-dependent part goes into the limit so that every element is
      // compared with a literal and nothing per element is kept across tiles)
      const int limit = (MODE == MODE_DENSE ? L - (t + t_base) * BC : n_cols - t * BC) - half * 4;
      changed = true;
#pragma unroll
      for (int kb2 = 0; kb2 < KB2; ++kb2)
#pragma unroll
        for (int qb = 0; qb < QB; ++qb)
#pragma unroll
          for (int i = 0; i < 16; ++i)
            s[kb2][qb][i] = kb2 * 32 + (i / 4) * 8 + (i % 4) < limit ? s[kb2][qb][i] : kNegInf;
    }
    return changed;
  };

  // ---- maximum of a tile's relative scores (per lane: the keys of its half) ----
  auto tile_max = [&](const f32x16 (&s)[KB2][QB]) {
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
      float a = kNegInf, b = kNegInf;   // two chains of v_max3
#pragma unroll
      for (int kb2 = 0; kb2 < KB2; ++kb2)
#pragma unroll
        for (int i = 0; i < 8; i += 2) {
          a = fmaxf(fmaxf(a, s[kb2][qb][i]), s[kb2][qb][i + 1]);
          b = fmaxf(fmaxf(b, s[kb2][qb][8 + i]), s[kb2][qb][8 + i + 1]);
        }
      mx_raw[qb] = fmaxf(a, b);
    }
  };

  // ---- lazy reference update.  The reference is only moved when a tile exceeds
  // it by more than kLazyLog2 in the exponent (2^8): until then P keeps the
  // stale reference, which changes no result (any reference cancels in O / l).
  // Moving it shifts the scores already computed and the accumulator seed nm,
  // and rescales l and O; the branch is wave-uniform and rarely taken. ----
  auto settle_max = [&](f32x16 (&s)[KB2][QB]) {
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
      const float mx = half_max(mx_raw[qb]);
      const bool grow = mx > thr[qb];   // false when the lane's tile is fully masked
      if (__builtin_amdgcn_ballot_w64(grow) != 0) {
        const float delta = grow ? mx : 0.f;
        const float alpha = (grow && thr[qb] != kNegInf) ? __builtin_amdgcn_exp2f(-mx) : 1.0f;
        thr[qb] = grow ? kLazyLog2 : thr[qb];
#pragma unroll
        for (int kb2 = 0; kb2 < KB2; ++kb2)
#pragma unroll
          for (int i = 0; i < 16; ++i) s[kb2][qb][i] -= delta;
#pragma unroll
        for (int i = 0; i < 16; ++i) nm[qb][i] -= delta;
        l4[qb][0] *= alpha;
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
          for (int i = 0; i < 16; ++i) o[db][qb][i] *= alpha;
      }
    }
  };

  // ---- P = exp2(relative score), rounded to bf16 in the B-operand layout ----
  auto exponentiate = [&](const f32x16 (&s)[KB2][QB], bf16x8 (&pf)[KB2][2][QB]) {
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
#pragma unroll
      for (int kb2 = 0; kb2 < KB2; ++kb2) {
#pragma unroll
        for (int sub = 0; sub < 2; ++sub) {
          bf16x8 pk;
#pragma unroll
          for (int i = 0; i < 8; i += 2) {
            const float p0 = __builtin_amdgcn_exp2f(s[kb2][qb][sub * 8 + i]);
            const float p1 = __builtin_amdgcn_exp2f(s[kb2][qb][sub * 8 + i + 1]);
            const f32x2 pp = {p0, p1};
            const bf16x2 pb = __builtin_convertvector(pp, bf16x2);
            pk[i] = pb[0];
            pk[i + 1] = pb[1];
          }
          pf[kb2][sub][qb] = pk;
        }
      }
    }
  };

  // ---- O^T += V^T P^T and l += rowsum(P) for the tile held in V buffer BUF ----
  auto accumulate = [&](auto buf_tag, const bf16x8 (&pf)[KB2][2][QB]) {
    constexpr int BUF = decltype(buf_tag)::value;
    const unsigned char* vbase = sV[BUF];
#pragma unroll
    for (int kb2 = 0; kb2 < KB2; ++kb2) {
#pragma unroll
      for (int sub = 0; sub < 2; ++sub) {
#pragma unroll
        for (int db = 0; db < DB; ++db) {
          // a lane supplies the address of (key row, 4 d) and receives 4 keys of one d
          const unsigned char* src = vbase + (kb2 * 32 + sub * 16) * ROW_BYTES + v_off[db];
          const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(src));
          const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(src + 8 * ROW_BYTES));
          const s16x8 both = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
          const bf16x8 a = __builtin_bit_cast(bf16x8, both);
#pragma unroll
          for (int qb = 0; qb < QB; ++qb)
            o[db][qb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, pf[kb2][sub][qb], o[db][qb], 0, 0, 0);
        }
        // row sums of the rounded P (numerator and denominator see the same values)
#pragma unroll
        for (int qb = 0; qb < QB; ++qb)
          l4[qb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(sum_a, pf[kb2][sub][qb], l4[qb], 0, 0, 0);
      }
    }
  };

  // ---- prologue: K(0), V(0), K(1) into LDS, scores of tile 0 ----
  f32x16 s_a[KB2][QB], s_b[KB2][QB];
  if (n_tiles > 0) {
    if (kIndirect && n_tiles > 1) load_index(1);
    if (kIndirect && n_tiles > 2) load_index(2);
    load_tile(Int<1>{}, 0, 0, Int<1>{});
    load_tile(Int<0>{}, 0, 0, Int<1>{});
    if (n_tiles > 1) load_tile(Int<1>{}, 1, 1, Int<1>{});
  }
  __syncthreads();
  if (n_tiles > 0) {
    scores(Int<0>{}, s_a);
    tile_max(s_a);
  }
  // The first stage requests K(2) into the buffer of K(0) at once: every wave must
  // have read K(0) before any wave gets there (the stages end with a barrier, the
  // prologue needs its own).
  __syncthreads();

  // One pipeline stage.  On entry s_cur holds the raw scores of tile t; LDS holds
  // K(t+1) in K buffer (t+1)&1 and V(t) in V buffer t&1, while K(t+2) and V(t+1)
  // travel global -> LDS.  NEXT: 1 = a tile t + 1 is known
  // to exist, 0 = tile t is the last one.  With NEXT the two products and the
  // exponentials sit in one basic block: the matrix pipe computes the scores of
  // tile t + 1 and then O += P V of tile t while the vector pipe turns the
  // scores of tile t into P.
  // Lists are ascending, so only their last tile can reach past L (or hold padding of a column list).
  auto stage = [&](auto par_tag, auto next_tag, auto inner_tag, const int t, f32x16 (&s_cur)[KB2][QB], f32x16 (&s_next)[KB2][QB]) {
    constexpr int PAR = decltype(par_tag)::value;     // t & 1
    constexpr bool has1 = decltype(next_tag)::value != 0;
    constexpr bool INNER = decltype(inner_tag)::value != 0;   // t + 2 exists
    if (kIndirect && t + 3 < n_tiles) load_index(t + 3);
    // The requests cost a wave 470 cycles of issue in a row; four waves spread them over the first MFMAs of the stage
    // (24 heads x 1,998, five bands of 81, D = 128: 47.5 -> 46.2 us; 8 heads x 75,600, one band: 561 -> 557).  With eight waves,
    // half as many requests each, the order that the compiler then finds for the rest loses 10 %.
    constexpr bool kLoadsInside = INNER && !kIndirect && NW == 4;
    // Rows through a row map: those of K(t+2) wait for the index ring, at the top; those of V(t+1) are known (window of 8
    // heads x 75,600, D = 128: 577 -> 560 us; both inside: 637; the same for column lists: 24 heads x 1,998, 200 columns: 15.1 -> 16.7).
    constexpr bool kRowsInside = INNER && MODE == MODE_PBAND && NW == 4;
    auto request = [&]() {
      if (kIndirect && has1) load_tile(Int<0>{}, PAR ^ 1, t + 1, Int<0>{});   // the rows of K(t+1), requested last
      if (INNER || (has1 && t + 2 < n_tiles)) load_tile(Int<1>{}, PAR, t + 2, Int<0>{});       // K(t+2) takes the place of K(t), read in the last stage
      if (!kIndirect && has1) load_tile(Int<0>{}, PAR ^ 1, t + 1, Int<0>{});   // V(t+1) takes the place of V(t-1)
    };
    unsigned v_rows[LPT];
    if (kRowsInside) {
#pragma unroll
      for (int u = 0; u < LPT; ++u) v_rows[u] = row_at[u];
      load_tile(Int<1>{}, PAR, t + 2, Int<0>{});
    } else if (!kLoadsInside) {
      request();
    }
    // partly kept tile?  band lists flag it per entry; the dense and gather loops
    // can only meet one at the very end (keys past L, padding of the column list)
    bool masked;
    if (kBand) masked = !(entries[t].y & 1);
    else if (has1) masked = false;
    else if (MODE == MODE_DENSE) masked = (t + t_base + 1) * BC > L;
    else masked = (t + 1) * BC > n_cols;
    if (masked && apply_mask(s_cur, t)) tile_max(s_cur);   // the maximum taken before masking may belong to a dropped key
    settle_max(s_cur);
    if (kLoadsInside) request();
    if (kRowsInside) {
      request_rows(Int<0>{}, rsrc_v, sV[PAR ^ 1] + wave * (LPT * 1024), v_rows, g_v);
    }
    bf16x8 pf[KB2][2][QB];
    if (has1) scores(Int<PAR ^ 1>{}, s_next);
    exponentiate(s_cur, pf);
    if (has1) tile_max(s_next);
    accumulate(Int<PAR>{}, pf);
    if (has1) {
      // Issue order for the block above: one MFMA, then the LDS reads that feed
      // the MFMAs a few steps later, then a handful of VALU ops that hide behind
      // the MFMA's passes (0x008 MFMA, 0x100 DS read, 0x002 VALU, 0x400 TRANS).
      constexpr int N_QK = KS * KB2 * QB, N_PVG = KB2 * 2, N_PV = N_PVG * DB * QB, N_SUM = N_PVG * QB;
      constexpr int N_KRD = KS * KB2, N_VRD = N_PVG * DB * 2;
      // per score element: one exp2, half a conversion, half a max3
      constexpr int VALU_PER = (KB2 * QB * 16 * 2 + N_QK + N_PV + N_SUM - 1) / (N_QK + N_PV + N_SUM);
      constexpr int K_AHEAD = 4, V_AHEAD = 8;
      __builtin_amdgcn_sched_group_barrier(0x100, K_AHEAD, 0);
#pragma unroll
      for (int i = 0; i < N_QK; ++i) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        if (i < (kLoadsInside ? 2 * LPT : kRowsInside ? LPT : 0)) __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
        if (i * N_KRD / N_QK + K_AHEAD < N_KRD) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
        else if (i >= N_QK - V_AHEAD / 2) __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
        __builtin_amdgcn_sched_group_barrier(0x402, VALU_PER, 0);
      }
#pragma unroll
      for (int g = 0; g < N_PVG; ++g) {
#pragma unroll
        for (int j = 0; j < DB * QB; ++j) {
          __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
          if ((g * DB * QB + j) * 2 + V_AHEAD < N_VRD) __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
          __builtin_amdgcn_sched_group_barrier(0x402, VALU_PER, 0);
        }
#pragma unroll
        for (int j = 0; j < QB; ++j) {
          __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
          __builtin_amdgcn_sched_group_barrier(0x402, VALU_PER, 0);
        }
      }
    }
    // The maximum of the next tile is used only in the next stage: without this
    // anchor at the end of the block the compiler sinks the whole chain out of
    // it, away from the MFMAs that hide it.
    if (has1) {
#pragma unroll
      for (int qb = 0; qb < QB; ++qb) asm volatile("" : "+v"(mx_raw[qb]));
    }
    // the loads that this stage has requested must have landed before anyone reads them
    __syncthreads();
  };

  // Two stages per trip keep buffer indices and the score registers static.  One loop, whose second stage asks whether
  // K(t+3) exists; at D = 128 the bulk of a list runs through a copy that knows it (long lists
  // are 0.5 % faster for it; at D = 64 it brings nothing).
  constexpr bool kLong = D == 128;
  int t = 0;
  for (; kLong && t + 3 < n_tiles; t += 2) {
    stage(Int<0>{}, Int<1>{}, Int<1>{}, t, s_a, s_b);
    stage(Int<1>{}, Int<1>{}, Int<1>{}, t + 1, s_b, s_a);
  }
  for (; t + 2 < n_tiles; t += 2) {
    stage(Int<0>{}, Int<1>{}, Int<1>{}, t, s_a, s_b);
    stage(Int<1>{}, Int<1>{}, Int<0>{}, t + 1, s_b, s_a);
  }
  if (t + 1 < n_tiles) {
    stage(Int<0>{}, Int<1>{}, Int<0>{}, t, s_a, s_b);
    stage(Int<1>{}, Int<0>{}, Int<0>{}, t + 1, s_b, s_a);
  } else if (t < n_tiles) {
    stage(Int<0>{}, Int<0>{}, Int<0>{}, t, s_a, s_b);
  }

  // ---- split launch: leave the chunk's state for the merge kernel, register by
  // register (each a coalesced 256-byte row of the wave) ----
  if (MODE != MODE_PBAND && it.partial) {
    static_assert(QB == 1, "the split path keeps one 32-row block per wave");
    typedef float __attribute__((address_space(1)))* global_float_ptr;   // global stores, not FLAT ones
    global_float_ptr dst = (global_float_ptr)(uintptr_t)(it.partial + (size_t)wave * ((DB * 16 + 2) * 64) + lane);
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
      for (int i = 0; i < 16; ++i) dst[(db * 16 + i) * 64] = o[db][0][i];
    // reference exponent of this chunk; none for a row without a finite logit in it (band chunks without a kept key of
    // the row, chunks of any kind whose keys all have logits of -inf)
    dst[(DB * 16) * 64] = thr[0] == kNegInf ? kNegInf : -nm[0][0];
    dst[(DB * 16 + 1) * 64] = l4[0][0];   // row sum relative to it
    return;
  }

  // ---- epilogue: O = O^T / l, bf16.  A lane owns query l32 and holds 4 consecutive d at a time: stored from there, an
  // instruction writes 16 bytes to each of 32 rows, 5,000 cycles at the end of an item.  Through LDS (the tiles are done
  // with: every stage ends with a barrier), 64 d of the wave's rows at a time, it writes 128 bytes to each of eight.
  // 24 heads x 1,998, D = 128, dense: 57.8 -> 55.9 us, 200 columns: 16.6 -> 15.4; 36 heads x 7,560: 155 -> 149; 42 heads x
  // 32,760: 2,536 -> 2,499.  Eight waves at D = 128 store from the registers in the layer kernel (40 heads x 75,600, 8 dense: 22.31 ms
  // through LDS, 22.13 so; D = 64 the other way: 37 heads x 87,747: 23.74 / 23.89) and in launches of dense heads or gathered columns
  // (10 dense heads x 18,900: 1,491 us through LDS, 1,425 so), but not in those of band lists, which spill four times as many registers
  // then (20 heads x 18,900, bands: 1,007 us through LDS, 1,060 from the registers; with text borders, 16 x 33,016: 1,077 / 1,174; windows
  // of 8 heads x 37,800: 310 / 324). ----
  auto four = [](const f32x16& x, const int g, const float inv) -> bf16x4 {   // d of group g of a 32-row block
    const f32x2 a01 = {x[g * 4 + 0] * inv, x[g * 4 + 1] * inv};
    const f32x2 a23 = {x[g * 4 + 2] * inv, x[g * 4 + 3] * inv};
    const bf16x2 b01 = __builtin_convertvector(a01, bf16x2);
    const bf16x2 b23 = __builtin_convertvector(a23, bf16x2);
    return {b01[0], b01[1], b23[0], b23[1]};
  };
  if constexpr (NW == 8 && D == 128 && (CALLEE || !kBand)) {
    static_assert(QB == 1, "one 32-row block per wave");
    const float inv = 1.0f / l4[0][0];   // every lane holds the complete sum of its query
    const int row = q0 + l32;
    if (row < L) {
      __bf16* dst = O + (int64_t)(MODE == MODE_PBAND ? cols[row] : row) * p.stride_l;
#pragma unroll
      for (int db = 0; db < DB; ++db) {
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          *reinterpret_cast<bf16x4*>(dst + db * 32 + g * 8 + half * 4) = four(o[db][0], g, inv);
        }
      }
    }
    return;
  }
  static_assert(NW * 4096 <= 2 * TILE_BYTES && TILE_BYTES % 4096 == 0, "a wave's 32 rows x 64 d lie inside one K tile");
  unsigned char* const stage_out = (wave * 4096 < TILE_BYTES ? k0 + wave * 4096 : k1 + (wave * 4096 - TILE_BYTES));
#pragma unroll
  for (int qb = 0; qb < QB; ++qb) {
    const float inv = 1.0f / l4[qb][0];   // every lane holds the complete sum of its query
    int to[4];   // rows that the lane stores to
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      to[j] = q0 + qb * 32 + j * 8 + (lane >> 3);
      if (MODE == MODE_PBAND && to[j] < L) to[j] = cols[to[j]];
    }
#pragma unroll
    for (int d0 = 0; d0 < DB; d0 += 2) {
#pragma unroll
      for (int db = d0; db < d0 + 2; ++db) {
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          *reinterpret_cast<bf16x4*>(stage_out + l32 * 128 + ((((db - d0) * 4 + g) ^ (l32 & 7)) << 4) + half * 8) = four(o[db][qb], g, inv);
        }
      }
      wave_lds_order();
      // Read before the first store: with the order behind the stores the table's kernel at D = 128 spills 595 registers in place of
      // 540 (27 heads x 2,560, bands and 5 dense: 57.4 us where the same code without orders took 56.3; so 57.0 where that took 57.3).
      u32x4 piece[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int r = j * 8 + (lane >> 3);
        piece[j] = *reinterpret_cast<const u32x4*>(stage_out + r * 128 + (((lane & 7) ^ (r & 7)) << 4));
      }
      wave_lds_order();
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int r = j * 8 + (lane >> 3);
        if (q0 + qb * 32 + r < L) *reinterpret_cast<u32x4*>(O + (int64_t)to[j] * p.stride_l + d0 * 32 + (lane & 7) * 8) = piece[j];
      }
    }
  }
}

// The same for a function that is not inlined into its kernel, where the compiler does not tell the
// LDS objects apart by themselves: parameters that do not alias say it.
template <int D, int NW, int QB, int BC, int OCC, int MODE>
__device__ __forceinline__ void attn_body_callee(const AttnLaunch& p, const Item& it, const __bf16* __restrict__ const K,
                                                 const __bf16* __restrict__ const V, unsigned char* __restrict__ const k0,
                                                 unsigned char* __restrict__ const k1, unsigned char* __restrict__ const v0,
                                                 unsigned char* __restrict__ const v1, unsigned char* __restrict__ const sI) {
  attn_body<D, NW, QB, BC, OCC, MODE, true>(p, it, K, V, k0, k1, v0, v1, sI);
}

template <int D, int NW, int QB, int BC, int OCC, int MODE, bool CALLEE = false>
__device__ __forceinline__ void attn_run(const AttnLaunch& p, const Item& it) {
  const int64_t base = (int64_t)it.b * p.stride_b + (int64_t)it.head * p.stride_h;
  const __bf16* const K = MODE == MODE_GATHER ? it.gathered : p.k + base;
  const __bf16* const V = MODE == MODE_GATHER ? K + (size_t)p.gather_pad * D : p.v + base;
  unsigned char* const k0 = lds_part<D, BC, LDS_K0>();
  unsigned char* const k1 = lds_part<D, BC, LDS_K1>();
  unsigned char* const v0 = lds_part<D, BC, LDS_V0>();
  unsigned char* const v1 = lds_part<D, BC, LDS_V1>();
  unsigned char* const sI = lds_part<D, BC, LDS_INDEX>();
  if (CALLEE) attn_body_callee<D, NW, QB, BC, OCC, MODE>(p, it, K, V, k0, k1, v0, v1, sI);
  else attn_body<D, NW, QB, BC, OCC, MODE, false>(p, it, K, V, k0, k1, v0, v1, sI);
}

// The item `item` of a launch over one group of heads (or of a segment of the layer
// kernel): its place in the (batch entry, head, chunk, query tile) order and its list.
template <int D, int NW, int QB, int BC, int OCC, int MODE, bool CALLEE = false>
__device__ __forceinline__ void attn_item(const AttnLaunch& p, const int item) {
  constexpr bool kBand = MODE == MODE_BAND || MODE == MODE_PBAND;
  constexpr int DB = D / 32;
  Item it{};
  const int qblk = item % p.n_q_blocks;
  const int chunk = (item / p.n_q_blocks) % p.split;   // key-range chunk (dense launches only)
  const int hb = item / p.n_q_blocks / p.split;
  const int hg = hb % p.n_heads;
  it.qblk = qblk;
  it.b = hb / p.n_heads;
  it.head = uni(p.heads ? p.heads[hg] : hg);   // scalar: the buffer resources of K and V are built from it
  int n_tiles = 0, t_base = 0, n_cols = 0;
  const_int2_ptr entries = nullptr, runs = nullptr;
  const int* row_map = nullptr;
  if (MODE == MODE_DENSE) {
    const int n_all = (p.L + BC - 1) / BC;
    t_base = chunk * n_all / p.split;
    n_tiles = (chunk + 1) * n_all / p.split - t_base;
    if (p.split > 1) it.partial = p.partial + (size_t)item * NW * ((DB * 16 + 2) * 64);
  } else {
    const int* rec = p.ws + p.list_table + 4 * p.list_id[hg];
    if (kBand) {
      const int* row_ptr = p.ws + rec[0];
      const int e0 = row_ptr[qblk], e1 = row_ptr[qblk + 1];
      entries = (const_int2_ptr)(uintptr_t)(p.ws + rec[1]) + e0;
      runs = (const_int2_ptr)(uintptr_t)(p.ws + rec[2]);
      n_tiles = e1 - e0;
      if (n_tiles == 0) return;   // rows that another launch computes (text rows of a layer with a text prefix)
      if (MODE == MODE_PBAND) row_map = p.ws + rec[3];
    } else {
      if (qblk < p.skip_q_blocks) return;   // text rows: another launch computes them
      n_tiles = rec[1] / BC;
      n_cols = rec[2];
      it.gathered = p.gathered + (size_t)hb * 2 * p.gather_pad * D;
    }
  }
  // The list pointers and counts are uniform but may have been loaded through the vector
  // memory path: as scalars, the list reads in the loop are scalar loads, which neither
  // queue behind nor wait for the tile loads in flight.
  it.entries = uni_const(entries);
  it.runs = uni_const(runs);
  it.index = uni(row_map);
  it.n_tiles = uni(n_tiles);
  it.n_cols = uni(n_cols);
  it.t_base = uni(t_base);
  attn_run<D, NW, QB, BC, OCC, MODE, CALLEE>(p, it);
}


// One launch per group: work-group = one item.
template <int D, int NW, int QB, int BC, int OCC, int MODE>
__global__ void __launch_bounds__(NW * 64, OCC) attn_fwd_kernel(const AttnLaunch p) {
  // which tile of which head (XCD-aware: consecutive items share an XCD)
  const int per_xcd = (p.n_items + 7) >> 3;
  const int item = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
  if (item >= p.n_items) return;
  attn_item<D, NW, QB, BC, OCC, MODE>(p, item);
}


// Merge of a split dense launch: work-group = (query tile, head, batch entry,
// slice of RPS accumulator rows), same thread-to-element mapping as
// attn_fwd_kernel.  Chunks are folded one by one with the online-softmax rule:
// O = O * 2^(m - m') + O_c * 2^(m_c - m').  RPS = all rows for the few chunks of
// a dense group; launches with many chunks and few query tiles (the text rows
// of a layer with a text prefix) use slices of four rows, so that the chain over
// the chunks is short per thread and spread over many work-groups.
template <int D, int NW, int RPS>
__global__ void __launch_bounds__(NW * 64) combine_partials_kernel(const AttnLaunch p) {
  constexpr int DB = D / 32;
  constexpr int BR = NW * 32;
  static_assert(RPS % 4 == 0 && (DB * 16) % RPS == 0, "a slice is a whole number of 4-row groups");
  const int qblk = blockIdx.x % p.n_q_blocks;
  const int hb = blockIdx.x / p.n_q_blocks;
  const int hg = hb % p.n_heads;
  const int b = hb / p.n_heads;
  const int head = p.heads ? p.heads[hg] : hg;
  const int r0 = blockIdx.y * RPS;     // first accumulator row of this slice
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int l32 = lane & 31, half = lane >> 5;
  float o[RPS];
#pragma unroll
  for (int r = 0; r < RPS; ++r) o[r] = 0.f;
  float m = kNegInf, l = 0.f;
#pragma unroll 2
  for (int c = 0; c < p.split; ++c) {
    const size_t item = ((size_t)hb * p.split + c) * p.n_q_blocks + qblk;
    const float* src = p.partial + (item * NW + wave) * ((DB * 16 + 2) * 64) + lane;
    const float mc = src[(DB * 16) * 64], lc = src[(DB * 16 + 1) * 64];
    const float m_new = fmaxf(m, mc);
    // a chunk in which the row has no finite logit (mc = -inf) adds nothing
    const float wa = m == kNegInf ? 0.f : __builtin_amdgcn_exp2f(m - m_new), wc = mc == kNegInf ? 0.f : __builtin_amdgcn_exp2f(mc - m_new);
    l = l * wa + lc * wc;
#pragma unroll
    for (int r = 0; r < RPS; ++r) o[r] = o[r] * wa + src[(r0 + r) * 64] * wc;
    m = m_new;
  }
  const float inv = 1.0f / l;
  const int row = qblk * BR + wave * 32 + l32;
  if (row < p.L) {
    __bf16* dst = p.out + (int64_t)b * p.stride_b + (int64_t)head * p.stride_h + (int64_t)row * p.stride_l;
#pragma unroll
    for (int rr = 0; rr < RPS; rr += 4) {
      const int db = (r0 + rr) / 16, g = ((r0 + rr) % 16) / 4;
      const f32x2 a01 = {o[rr + 0] * inv, o[rr + 1] * inv};
      const f32x2 a23 = {o[rr + 2] * inv, o[rr + 3] * inv};
      const bf16x2 b01 = __builtin_convertvector(a01, bf16x2);
      const bf16x2 b23 = __builtin_convertvector(a23, bf16x2);
      const bf16x4 out4 = {b01[0], b01[1], b23[0], b23[1]};
      *reinterpret_cast<bf16x4*>(dst + db * 32 + g * 8 + half * 4) = out4;
    }
  }
}

// Pre-pass of a vertical-stripe group (M_4): work-group = 64 key slots of one (batch entry, head).
// Slot j of the head's gathered arrays takes row cols[j] of K and of V; slots past the padded list
// and padding entries are zero (a masked score times a zero row, never times stale bits).
template <int D>
__global__ void __launch_bounds__(256) gather_kv_kernel(const AttnLaunch p) {
  constexpr int CH = D / 8;
  const int hb = blockIdx.y;
  const int hg = hb % p.n_heads, b = hb / p.n_heads;
  const int head = p.heads[hg];
  const int* rec = p.ws + p.list_table + 4 * p.list_id[hg];
  const int* cols = p.ws + rec[0];
  const int padded = rec[1];
  const int64_t base = (int64_t)b * p.stride_b + (int64_t)head * p.stride_h;
  __bf16* Kg = p.gathered + (size_t)hb * 2 * p.gather_pad * D;
  __bf16* Vg = Kg + (size_t)p.gather_pad * D;
  for (int c = threadIdx.x; c < 64 * CH; c += 256) {
    const int j = blockIdx.x * 64 + c / CH, piece = (c % CH) * 8;
    if (j >= p.gather_pad) continue;
    const int src = j < padded ? cols[j] : -1;
    uint4 kk = make_uint4(0, 0, 0, 0), vv = make_uint4(0, 0, 0, 0);
    if (src >= 0) {
      kk = *reinterpret_cast<const uint4*>(p.k + base + (int64_t)src * p.stride_l + piece);
      vv = *reinterpret_cast<const uint4*>(p.v + base + (int64_t)src * p.stride_l + piece);
    }
    *reinterpret_cast<uint4*>(Kg + (size_t)j * D + piece) = kk;
    *reinterpret_cast<uint4*>(Vg + (size_t)j * D + piece) = vv;
  }
}

// M_1 (Section 4.2): the output of a skipped head is zero.
__global__ void __launch_bounds__(256) zero_heads_kernel(const AttnLaunch p) {
  const int hg = blockIdx.y % p.n_heads;
  const int b = blockIdx.y / p.n_heads;
  const int head = p.heads ? p.heads[hg] : hg;
  __bf16* O = p.out + (int64_t)b * p.stride_b + (int64_t)head * p.stride_h;
  const int chunks = p.D / 8;
  const int64_t total = (int64_t)p.L * chunks;
  for (int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; g < total;
       g += (int64_t)gridDim.x * blockDim.x) {
    const int64_t row = g / chunks;
    const int c = (int)(g % chunks);
    *reinterpret_cast<uint4*>(O + row * p.stride_l + c * 8) = make_uint4(0, 0, 0, 0);
  }
}

// Lists from page-locked host memory to a plan workspace: bound by the reads over the bus, so every thread has one
// 16-byte load in flight and nothing else.  A kernel and not a copy, because a copy between two kernels of a stream waits
// for the copy engine and back: 12 heads x 1,998 x 2 (20 KB of lists), one-shot call repeated: 72 us with the copy, 58 us
// with the kernel, 51 us without either (and wrong results once the memory has held something else).
__global__ void __launch_bounds__(256) copy_lists_kernel(const uint4* __restrict__ src, uint4* __restrict__ dst, const unsigned n16) {
  const unsigned i = blockIdx.x * 256u + threadIdx.x;
  if (i < n16) dst[i] = src[i];
}

// ---- the whole layer in one launch ----

__global__ void __launch_bounds__(128) reset_counters_kernel(int* counters) {
  if (threadIdx.x < kLayerCounterWords) counters[threadIdx.x] = 0;
}

// Waves per work-group of the layer kernel: eight, one work-group per compute unit, every item on the
// 256-row query tile (a K/V tile in LDS then serves twice the rows of the four-wave form, which ran the
// dense items 4-14 % and the wide-band items 4-7 % slower).
constexpr int kLayerWaves = 8;

// Zero fill of one query tile of a skipped head (M_1).
template <int D>
__device__ __forceinline__ void zero_item(const AttnLaunch& p, const int item) {
  constexpr int BR = kLayerWaves * 32, CH = D / 8;
  const int qblk = item % p.n_q_blocks;
  const int hb = item / p.n_q_blocks;
  const int hg = hb % p.n_heads, b = hb / p.n_heads;
  const int head = p.heads[hg];
  __bf16* O = p.out + (int64_t)b * p.stride_b + (int64_t)head * p.stride_h;
  for (int c = threadIdx.x; c < BR * CH; c += blockDim.x) {
    const int row = qblk * BR + c / CH;
    if (row < p.L) *reinterpret_cast<uint4*>(O + (int64_t)row * p.stride_l + (c % CH) * 8) = make_uint4(0, 0, 0, 0);
  }
}

// The segment loops of the layer kernel are real functions, not inlined: inlined
// side by side into one kernel the four loop nests get in each other's way in the
// register allocator; as callees each is allocated like the kernel it also is
// elsewhere in this file.  Arguments of a callee travel in vector registers even
// when they are uniform, so everything is made scalar again on entry.
// One segment of the layer kernel: the work-group pulls items of the segment off the eight
// queues, its own XCD's first, until all are empty.  A real function, called once per segment
// (a call per item would save and restore the callee-saved half of the register file around
// every item: measured as more than a gigabyte of scratch traffic per layer).
// KIND = a MODE_* of attn_item, or kZeroKind for the zero fill of skipped heads.
constexpr int kZeroKind = 100;
template <int D, int BC, int KIND>
__device__ __attribute__((noinline)) void layer_segment(const AttnLaunch av, const int first_item_v, const int n_rest_v,
                                                        int* const counters_v, const int home_v, const unsigned pick_v) {
  AttnLaunch a;
  a.q = uni(av.q);
  a.k = uni(av.k);
  a.v = uni(av.v);
  a.out = uni(av.out);
  a.B = uni(av.B);
  a.H = uni(av.H);
  a.L = uni(av.L);
  a.D = uni(av.D);
  a.stride_b = uni(av.stride_b);
  a.stride_h = uni(av.stride_h);
  a.stride_l = uni(av.stride_l);
  a.n_q_blocks = uni(av.n_q_blocks);
  a.n_heads = uni(av.n_heads);
  a.n_items = uni(av.n_items);
  a.heads = uni(av.heads);
  a.list_id = uni(av.list_id);
  a.ws = uni(av.ws);
  a.list_table = uni(av.list_table);
  a.scale_log2e = uni(av.scale_log2e);
  a.split = 1;
  a.partial = nullptr;
  a.gathered = uni(av.gathered);
  a.gather_pad = uni(av.gather_pad);
  a.skip_q_blocks = uni(av.skip_q_blocks);
  const int first_item = uni(first_item_v), n_rest = uni(n_rest_v), home = uni(home_v);
  int* const counters = uni(counters_v);   // this segment's eight queue positions
  typedef __attribute__((address_space(3))) int* lds_int;
  lds_int const pick = (lds_int)(uintptr_t)uni((int)pick_v);
  const int per = (n_rest + 7) >> 3;
  // Every queue position only grows, so every loop below ends, and all waves of the
  // work-group take the same path (the position is read by all of them after a barrier).
  for (int probe = 0; probe < 8; ++probe) {
    const int x = (home + probe) & 7;
    int cnt = n_rest - x * per;
    cnt = cnt < 0 ? 0 : (cnt > per ? per : cnt);
    if (cnt == 0) continue;
    for (;;) {
      if (threadIdx.x == 0) *pick = atomicAdd(counters + x, 1);
      __syncthreads();
      const int pos = __builtin_amdgcn_readfirstlane(*pick);
      // the next pick overwrites `pick`, the next item the LDS tiles: everyone must be done with both
      if (pos >= cnt) {
        __syncthreads();
        break;
      }
      const int item = first_item + x * per + pos;
      if (KIND == kZeroKind) zero_item<D>(a, item);
      else attn_item<D, kLayerWaves, 1, BC, 2, (KIND == kZeroKind ? MODE_DENSE : KIND), true>(a, item);
      __syncthreads();
    }
  }
}

template <int D, int BC>
__global__ void __launch_bounds__(kLayerWaves * 64, 2) attn_layer_kernel(const LayerLaunch lp) {
  __shared__ int pick;
  typedef __attribute__((address_space(3))) int* lds_int;
  const unsigned pick_addr = (unsigned)(uintptr_t)(lds_int)&pick;
  const int home = blockIdx.x & 7;   // work-groups are dealt to the XCDs in turn
  // Segment after segment, heaviest first; inside a segment a work-group first drains
  // its own XCD's eighth, then the other XCDs' eighths.
  for (int s = 0; s < lp.n_segments; ++s) {
    const LayerSegment sg = lp.seg[s];
    AttnLaunch a = lp.a;
    a.n_q_blocks = sg.n_q_blocks;
    a.n_heads = sg.n_heads;
    a.n_items = sg.n_items + sg.first_item;
    a.heads = lp.a.ws + sg.heads;
    a.list_id = lp.a.ws + sg.list_id;
    a.list_table = sg.list_table;
    int* const counters = lp.counters + s * 8;
    switch (sg.kind) {
      case SEG_DENSE: layer_segment<D, BC, MODE_DENSE>(a, sg.first_item, sg.n_items, counters, home, pick_addr); break;
      case SEG_BAND: layer_segment<D, BC, MODE_BAND>(a, sg.first_item, sg.n_items, counters, home, pick_addr); break;
      case SEG_GATHER: layer_segment<D, BC, MODE_GATHER>(a, sg.first_item, sg.n_items, counters, home, pick_addr); break;
      case SEG_PBAND: layer_segment<D, BC, MODE_PBAND>(a, sg.first_item, sg.n_items, counters, home, pick_addr); break;
      default: layer_segment<D, BC, kZeroKind>(a, sg.first_item, sg.n_items, counters, home, pick_addr); break;
    }
  }
}

// ---- the layer in one launch, work-group = one item of a table ----

// Instantiated for four waves, and at D = 64 for eight (at D = 128 the large tile was never the fastest form).
// The loops are those of attn_fwd_kernel (same registers, no spill inside them: a work-group takes one branch of the
// switch to its end).  What bounds short layers is everything around the loops: here one scalar load brings the item,
// where a group's launch reads head, list record, row pointer and entries one after the other, and one launch
// replaces up to nine.  4 heads x 1,024 tokens, D = 64: 82 us in groups, 16 us with the table.

typedef const int __attribute__((address_space(4)))* const_int_ptr;

template <int D, int NW, int BC>
__global__ void __launch_bounds__(NW * 64, 2) attn_grid_kernel(const GridLaunch g) {
  const const_int_ptr r = (const_int_ptr)(uintptr_t)(g.a.ws + g.table) + (size_t)blockIdx.x * kGridWords;
  if (r[0] < 0) return;
  const int kind = r[0] & 255, t0 = r[0] >> 8;
  Item it{};
  it.head = r[1];
  it.b = r[2];
  it.qblk = r[3];
  it.n_tiles = r[4];
  const int list = r[5], more = r[6], last = r[7];
  if (kind == SEG_DENSE) {
    it.t_base = t0;
  } else if (kind == SEG_GATHER) {
    it.index = g.a.ws + list + t0 * BC;
    it.n_cols = more - t0 * BC;
  } else {
    it.entries = (const_int2_ptr)(uintptr_t)(g.a.ws + list) + t0;
    it.runs = (const_int2_ptr)(uintptr_t)(g.a.ws + more);
  }
  if (kind == SEG_PBAND) it.index = g.a.ws + last;
  else if (last >= 0) it.partial = g.partial + (size_t)last * NW * ((D / 32 * 16 + 2) * 64);
  switch (kind) {
    case SEG_DENSE: attn_run<D, NW, 1, BC, 2, MODE_DENSE>(g.a, it); break;
    case SEG_BAND: attn_run<D, NW, 1, BC, 2, MODE_BAND>(g.a, it); break;
    case SEG_GATHER: attn_run<D, NW, 1, BC, 2, MODE_COLS>(g.a, it); break;
    case SEG_PBAND: attn_run<D, NW, 1, BC, 2, MODE_PBAND>(g.a, it); break;
    default: {   // zero fill of kGridZeroRows rows of a skipped head
      __bf16* O = g.a.out + (int64_t)it.b * g.a.stride_b + (int64_t)it.head * g.a.stride_h;
      constexpr int CH = D / 8;
      for (int c = threadIdx.x; c < kGridZeroRows * CH; c += NW * 64) {
        const int row = it.qblk * kGridZeroRows + c / CH;
        if (row < g.a.L) *reinterpret_cast<uint4*>(O + (int64_t)row * g.a.stride_l + (c % CH) * 8) = make_uint4(0, 0, 0, 0);
      }
    }
  }
}

// Merge of the split items of a grid launch: work-group = (split query tile, slice of
// four accumulator rows); the chunks of a tile lie in consecutive slots.
template <int D, int NW>
__global__ void __launch_bounds__(NW * 64) merge_chunks_kernel(const GridLaunch g) {
  constexpr int DB = D / 32, RPS = 4;
  const const_int_ptr r = (const_int_ptr)(uintptr_t)(g.a.ws + g.merge_table) + (size_t)blockIdx.x * kGridWords;
  const int head = r[0], b = r[1], qblk = r[2], n_chunks = r[3], slot = r[4];
  const int r0 = blockIdx.y * RPS;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int l32 = lane & 31, half = lane >> 5;
  float o[RPS];
#pragma unroll
  for (int i = 0; i < RPS; ++i) o[i] = 0.f;
  float m = kNegInf, l = 0.f;
#pragma unroll 2
  for (int c = 0; c < n_chunks; ++c) {
    const float* src = g.partial + ((size_t)(slot + c) * NW + wave) * ((DB * 16 + 2) * 64) + lane;
    const float mc = src[(DB * 16) * 64], lc = src[(DB * 16 + 1) * 64];
    const float m_new = fmaxf(m, mc);
    // a chunk in which the row has no finite logit (mc = -inf) adds nothing
    const float wa = m == kNegInf ? 0.f : __builtin_amdgcn_exp2f(m - m_new), wc = mc == kNegInf ? 0.f : __builtin_amdgcn_exp2f(mc - m_new);
    l = l * wa + lc * wc;
#pragma unroll
    for (int i = 0; i < RPS; ++i) o[i] = o[i] * wa + src[(r0 + i) * 64] * wc;
    m = m_new;
  }
  const float inv = 1.0f / l;
  const int row = qblk * (NW * 32) + wave * 32 + l32;
  if (row < g.a.L) {
    __bf16* dst = g.a.out + (int64_t)b * g.a.stride_b + (int64_t)head * g.a.stride_h + (int64_t)row * g.a.stride_l;
    const int db = r0 / 16, gg = (r0 % 16) / 4;
    const f32x2 a01 = {o[0] * inv, o[1] * inv}, a23 = {o[2] * inv, o[3] * inv};
    const bf16x2 b01 = __builtin_convertvector(a01, bf16x2), b23 = __builtin_convertvector(a23, bf16x2);
    const bf16x4 out4 = {b01[0], b01[1], b23[0], b23[1]};
    *reinterpret_cast<bf16x4*>(dst + db * 32 + gg * 8 + half * 4) = out4;
  }
}

template <int D, int NW, int QB, int BC, int OCC>
hipError_t launch_mode(const AttnLaunch& p, int mode, hipStream_t stream) {
  const int per_xcd = (p.n_items + 7) / 8;
  const dim3 grid(per_xcd * 8), block(NW * 64);
  switch (mode) {
    case MODE_DENSE:
      hipLaunchKernelGGL((attn_fwd_kernel<D, NW, QB, BC, OCC, MODE_DENSE>), grid, block, 0, stream, p);
      break;
    case MODE_BAND:
      hipLaunchKernelGGL((attn_fwd_kernel<D, NW, QB, BC, OCC, MODE_BAND>), grid, block, 0, stream, p);
      break;
    case MODE_GATHER:
      hipLaunchKernelGGL((attn_fwd_kernel<D, NW, QB, BC, OCC, MODE_GATHER>), grid, block, 0, stream, p);
      break;
    case MODE_PBAND:
      hipLaunchKernelGGL((attn_fwd_kernel<D, NW, QB, BC, OCC, MODE_PBAND>), grid, block, 0, stream, p);
      break;
    default:
      return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

// The dense and band modes on the small query tile.
template <int D, int NW, int QB, int BC, int OCC>
hipError_t launch_small(const AttnLaunch& p, int mode, hipStream_t stream) {
  const int per_xcd = (p.n_items + 7) / 8;
  const dim3 grid(per_xcd * 8), block(NW * 64);
  if (mode == MODE_DENSE && p.split == 1) {   // (a merge of chunks would read them as the large tile's)
    hipLaunchKernelGGL((attn_fwd_kernel<D, NW, QB, BC, OCC, MODE_DENSE>), grid, block, 0, stream, p);
  } else if (mode == MODE_BAND) {
    hipLaunchKernelGGL((attn_fwd_kernel<D, NW, QB, BC, OCC, MODE_BAND>), grid, block, 0, stream, p);
  } else if (mode == MODE_PBAND) {
    hipLaunchKernelGGL((attn_fwd_kernel<D, NW, QB, BC, OCC, MODE_PBAND>), grid, block, 0, stream, p);
  } else {
    return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

template <int D, int NW, int BC>
hipError_t launch_grid_shape(const GridLaunch& p, hipStream_t stream) {
  hipLaunchKernelGGL((attn_grid_kernel<D, NW, BC>), dim3(p.n_blocks), dim3(NW * 64), 0, stream, p);
  if (hipError_t e = hipGetLastError(); e != hipSuccess) return e;
  return launch_grid_merge(p, stream);
}

template <int D, int NW>
hipError_t launch_merge_shape(const GridLaunch& p, hipStream_t stream) {
  hipLaunchKernelGGL((merge_chunks_kernel<D, NW>), dim3(p.n_merges, D / 8), dim3(NW * 64), 0, stream, p);
  return hipGetLastError();
}

}  // namespace

int kernel_small_block_q(int D) {
  return D == 128 ? Tile128s::NW * Tile128s::QB * 32 : Tile64s::NW * Tile64s::QB * 32;
}

void kernel_blocks(int D, int* block_q, int* block_k) {
  if (D == 128) {
    *block_q = Tile128::NW * Tile128::QB * 32;
    *block_k = Tile128::BC;
  } else {
    *block_q = Tile64::NW * Tile64::QB * 32;
    *block_k = Tile64::BC;
  }
}

hipError_t launch_attention(const AttnLaunch& p, int mode, hipStream_t stream, bool small_q) {
  if (p.n_items <= 0) return hipSuccess;
  if (p.split < 1 || (p.split > 1 && (mode != MODE_DENSE || !p.partial))) return hipErrorInvalidValue;
  if (mode == MODE_GATHER && (!p.gathered || p.gather_pad < 1)) return hipErrorInvalidValue;
  if (small_q) {
    if (p.D == 128) return launch_small<128, Tile128s::NW, Tile128s::QB, Tile128s::BC, Tile128s::OCC>(p, mode, stream);
    if (p.D == 64) return launch_small<64, Tile64s::NW, Tile64s::QB, Tile64s::BC, Tile64s::OCC>(p, mode, stream);
    return hipErrorInvalidValue;
  }
  if (p.D == 128)
    return launch_mode<128, Tile128::NW, Tile128::QB, Tile128::BC, Tile128::OCC>(p, mode, stream);
  if (p.D == 64) return launch_mode<64, Tile64::NW, Tile64::QB, Tile64::BC, Tile64::OCC>(p, mode, stream);
  return hipErrorInvalidValue;
}

int layer_block_q(int) { return kLayerWaves * 32; }

hipError_t launch_layer(const LayerLaunch& p, int n_compute_units, hipStream_t stream) {
  if (p.n_segments < 1) return hipSuccess;
  if (p.n_segments > kMaxSegments || !p.counters || n_compute_units < 1) return hipErrorInvalidValue;
  static_assert(Tile128::NW == kLayerWaves && Tile64::NW == kLayerWaves && Tile128::QB == 1 && Tile64::QB == 1,
                "the layer kernel runs the kernels' own query tile: eight waves of 32 rows");
  long long total = 0;
  for (int s = 0; s < p.n_segments; ++s) {
    if (p.seg[s].n_items < 0 || p.seg[s].first_item < 0 || p.seg[s].kind < SEG_DENSE || p.seg[s].kind > SEG_ZERO)
      return hipErrorInvalidValue;
    total += p.seg[s].n_items;
  }
  if (total == 0) return hipSuccess;
  hipLaunchKernelGGL(reset_counters_kernel, dim3(1), dim3(128), 0, stream, p.counters);
  static_assert(kLayerCounterWords <= 128, "one thread per queue position");
  if (hipError_t e = hipGetLastError(); e != hipSuccess) return e;
  // one resident work-group of eight waves per compute unit, a multiple of eight so that every XCD gets its share
  long long groups = static_cast<long long>(8 / kLayerWaves) * n_compute_units;
  if (groups > total) groups = total;
  groups = (groups + 7) / 8 * 8;
  const dim3 grid((unsigned)groups), block(kLayerWaves * 64);
  if (p.a.D == 128) hipLaunchKernelGGL((attn_layer_kernel<128, Tile128::BC>), grid, block, 0, stream, p);
  else if (p.a.D == 64) hipLaunchKernelGGL((attn_layer_kernel<64, Tile64::BC>), grid, block, 0, stream, p);
  else return hipErrorInvalidValue;
  return hipGetLastError();
}

hipError_t launch_grid_merge(const GridLaunch& p, hipStream_t stream) {
  if (p.n_merges < 1) return hipSuccess;
  if (!p.a.ws || !p.partial) return hipErrorInvalidValue;
  if (p.a.D == 128 && p.waves == 4) return launch_merge_shape<128, 4>(p, stream);
  if (p.a.D == 64 && p.waves == 4) return launch_merge_shape<64, 4>(p, stream);
  if (p.a.D == 64 && p.waves == 8) return launch_merge_shape<64, 8>(p, stream);
  return hipErrorInvalidValue;
}

hipError_t launch_grid(const GridLaunch& p, hipStream_t stream) {
  if (p.n_blocks < 1) return hipSuccess;
  if (!p.a.ws || (p.n_merges > 0 && !p.partial)) return hipErrorInvalidValue;
  if (p.a.D == 128 && p.waves == 4) return launch_grid_shape<128, 4, Tile128::BC>(p, stream);
  if (p.a.D == 64 && p.waves == 4) return launch_grid_shape<64, 4, Tile64::BC>(p, stream);
  if (p.a.D == 64 && p.waves == 8) return launch_grid_shape<64, 8, Tile64::BC>(p, stream);
  return hipErrorInvalidValue;
}

size_t partial_floats(int D, int n_items) {
  const int nw = D == 128 ? Tile128::NW : Tile64::NW;
  return (size_t)n_items * nw * ((D / 32 * 16 + 2) * 64);
}

hipError_t launch_combine(const AttnLaunch& p, hipStream_t stream) {
  if (p.split <= 1 || p.n_items <= 0) return hipSuccess;
  if (!p.partial) return hipErrorInvalidValue;
  const int tiles = p.n_items / p.split;
  if (p.D == 128) {
    // always in slices of four accumulator rows (measured: the merge of the Wan2.1-like
    // dense group, three chunks, takes 175 us unsliced and about 70 us sliced)
    hipLaunchKernelGGL((combine_partials_kernel<128, Tile128::NW, 4>), dim3(tiles, 16), dim3(Tile128::NW * 64), 0, stream, p);
  } else if (p.D == 64) {
    // sliced for many chunks only; for the few chunks of a dense group the unsliced form is as fast
    if (p.split > 8)
      hipLaunchKernelGGL((combine_partials_kernel<64, Tile64::NW, 4>), dim3(tiles, 8), dim3(Tile64::NW * 64), 0, stream, p);
    else
      hipLaunchKernelGGL((combine_partials_kernel<64, Tile64::NW, 32>), dim3(tiles, 1), dim3(Tile64::NW * 64), 0, stream, p);
  } else {
    return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_copy_lists(const void* src, void* dst, size_t bytes, hipStream_t stream) {
  if (!src || !dst || bytes == 0 || bytes % 16 || bytes / 16 > 0x7fffffffu) return hipErrorInvalidValue;
  const unsigned n16 = static_cast<unsigned>(bytes / 16);
  hipLaunchKernelGGL(copy_lists_kernel, dim3((n16 + 255) / 256), dim3(256), 0, stream, static_cast<const uint4*>(src),
                     static_cast<uint4*>(dst), n16);
  return hipGetLastError();
}

hipError_t launch_gather_kv(const AttnLaunch& p, hipStream_t stream) {
  if (p.n_heads <= 0) return hipSuccess;
  if (!p.gathered || p.gather_pad < 1 || !p.heads || !p.list_id || !p.ws) return hipErrorInvalidValue;
  const dim3 grid((p.gather_pad + 63) / 64, p.n_heads * p.B), block(256);
  if (p.D == 128) hipLaunchKernelGGL(gather_kv_kernel<128>, grid, block, 0, stream, p);
  else if (p.D == 64) hipLaunchKernelGGL(gather_kv_kernel<64>, grid, block, 0, stream, p);
  else return hipErrorInvalidValue;
  return hipGetLastError();
}

hipError_t launch_zero_heads(const AttnLaunch& p, hipStream_t stream) {
  if (p.n_heads <= 0) return hipSuccess;
  const int64_t total = (int64_t)p.L * (p.D / 8);
  int bx = (int)((total + 255) / 256);
  if (bx > 2048) bx = 2048;
  const dim3 grid(bx, p.n_heads * p.B), block(256);
  hipLaunchKernelGGL(zero_heads_kernel, grid, block, 0, stream, p);
  return hipGetLastError();
}

}  // namespace svd
