// gfx950 (MI355X) kernels of chunk-streamed speculative-verification attention.
//
// Paper Sec. 4.2: every history chunk (K_j, V_j) is read once for the whole
// query group of a request (all n_b candidates x all G query heads sharing a
// KV head); the chunk-local online-softmax state (Eq. 13) is merged into the
// running state with the rescaled update of Eq. 14; the Speculative Frontier
// is attended with the causal candidate mask; O = a / l (Eq. 17).
//
// Layout and precision
//   * scores are kept in the log2 domain: x = sigma * log2(e) * q.k, so every
//     exponential is one v_exp_f32; the state's m is in that domain as well.
//   * all accumulation is fp32.  In the MFMA path the softmax weights P
//     (fp32) are split into bf16 hi + lo parts and both are multiplied with V
//     (two bf16 MFMAs), which keeps P to ~2^-16 relative; rounding P once to
//     bf16 would cost ~1.6e-3 relative L2 error.  The denominator l sums the
//     fp32 weights themselves, which hi + lo carry to that precision.
//   * a running state is split into 32 to 128 slots per query row so that
//     several workgroups can fold disjoint token ranges of one chunk into the
//     same row without atomics; the finalize kernel merges the slots.
#include <hip/hip_runtime.h>

#include "ss_kernels.h"

#include <cstddef>
#include <cstring>

#include <math.h>

#include <mutex>
#include <type_traits>

namespace ss {
namespace {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2_t __attribute__((ext_vector_type(2)));
// Global memory reached through a pointer whose origin the compiler cannot see.
typedef __attribute__((address_space(1))) float GlobalFloat;
typedef __attribute__((address_space(1))) f32x4_t GlobalFloat4;
typedef __attribute__((address_space(1))) u32x4_t GlobalU32x4;

constexpr float kNegInf = -__builtin_huge_valf();
constexpr int kAwPitch = 132;  // floats per row of a wave's partial accumulator
constexpr int kBufferFlags = 0x00020000;   // buffer resource word 3: 32-bit data format, raw offsets
// Cache policy of the history K/V loads: non-temporal.  Every history byte
// is read once per round, so the streaming loads should not displace
// reusable lines; measured on MI355X, this took config 3's round from 378 to
// 354 us and config 4's from 786 to 743 us (means over 40 rounds).
constexpr int kStreamLoad = 2;
constexpr int kMaxDevices = 64;   // devices whose scratch address is cached

__device__ __forceinline__ float exp2_fast(float x) { return __builtin_amdgcn_exp2f(x); }

__device__ __forceinline__ float bf16_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }

// Sum over the 16 lanes of a DPP row; every lane of the row gets the total.
__device__ __forceinline__ float row16_sum(float x) {
  int v;
  v = __builtin_amdgcn_mov_dpp(__float_as_int(x), 0xB1, 0xf, 0xf, false);  // quad_perm [1,0,3,2]
  x += __int_as_float(v);
  v = __builtin_amdgcn_mov_dpp(__float_as_int(x), 0x4E, 0xf, 0xf, false);  // quad_perm [2,3,0,1]
  x += __int_as_float(v);
  v = __builtin_amdgcn_mov_dpp(__float_as_int(x), 0x124, 0xf, 0xf, false); // row_ror:4
  x += __int_as_float(v);
  v = __builtin_amdgcn_mov_dpp(__float_as_int(x), 0x128, 0xf, 0xf, false); // row_ror:8
  x += __int_as_float(v);
  return x;
}

__device__ __forceinline__ float row16_max(float x) {
  int v;
  v = __builtin_amdgcn_mov_dpp(__float_as_int(x), 0xB1, 0xf, 0xf, false);
  x = fmaxf(x, __int_as_float(v));
  v = __builtin_amdgcn_mov_dpp(__float_as_int(x), 0x4E, 0xf, 0xf, false);
  x = fmaxf(x, __int_as_float(v));
  v = __builtin_amdgcn_mov_dpp(__float_as_int(x), 0x124, 0xf, 0xf, false);
  x = fmaxf(x, __int_as_float(v));
  v = __builtin_amdgcn_mov_dpp(__float_as_int(x), 0x128, 0xf, 0xf, false);
  return fmaxf(x, __int_as_float(v));
}
// Sum / max with the lane 16 away (l ^ 16): swapping the odd rows of one copy
// with the even rows of another leaves the pair's two values in the results.
__device__ __forceinline__ float x16_sum(float x) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ __forceinline__ float x16_max(float x) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}

// The same with the lane 32 away (l ^ 32).
__device__ __forceinline__ float x32_sum(float x) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ __forceinline__ float x32_max(float x) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}

// Max / sum across the four 16-lane groups of a wave (lanes l, l^16, l^32, l^48).
__device__ __forceinline__ float xgroup_max(float x) { return x32_max(x16_max(x)); }
__device__ __forceinline__ float xgroup_sum(float x) { return x32_sum(x16_sum(x)); }

// Kernel-argument form of a unit: all that its first loads need, so that they
// wait for one scalar round trip (0.36 us after a workgroup's start).  With the
// item, the chunk table and the header behind one another a workgroup's first
// K/V load went out 0.4 us later.  k, v point at the first item's first token
// of KV head 0.  Rounds back to back, before and after: 1 x 16384 tokens 19.4 ->
// 18.3 us, 24 ragged short requests 26.6 -> 25.5 us, 16 x 32768 tokens by chunk
// (8 launches) 386.5 -> 382.9 us; rounds of one long launch do not change (16 x
// 32768 in one call 308, 32 x 131072 2393 us).
struct UnitArg {
  const uint16_t *k, *v;
  uint64_t hs;           // elements between KV heads
  uint32_t word;         // see UnitRec
  uint32_t ntiles;
  int32_t tok_count;     // of the first item
  int32_t q_row0;
  uint32_t cand_slot;    // n_cand | slot << 8 | flags << 16
  uint32_t pad;
};
static_assert(sizeof(UnitArg) == 48, "UnitArg layout");
__host__ __device__ __forceinline__ uint32_t pack_cand_slot(const Item &it) {
  return (uint32_t)it.n_cand | (uint32_t)it.slot << 8 | (uint32_t)it.flags << 16;
}
__device__ __forceinline__ int unit_cand(const UnitArg &u) { return (int)(u.cand_slot & 0xffu); }
__device__ __forceinline__ uint32_t unit_slot(const UnitArg &u) { return (u.cand_slot >> 8) & 0xffu; }
__device__ __forceinline__ bool unit_fresh(const UnitArg &u) { return (u.cand_slot >> 16) & kSlotFresh; }

// What every unit of a launch needs of its arguments, read once at the start.
struct Ctx {
  const uint16_t *q;
  GlobalFloat *a, *m, *l;   // the state's arrays
  uint32_t R;               // query rows
  int Hq, G;
  uint32_t g_inv;           // ceil(65536 / G): r / G = r * g_inv >> 16 for r < 64, G <= 64
  float sl2;                // sigma log2(e)
  uint32_t stride_b;        // bytes between consecutive tokens of a KV head
};

__device__ __forceinline__ int global_row(const Ctx &c, int q_row0, int g, int r) {
  // local row r of (request, kv head g) -> packed query row (off_b + i) * Hq + h
  const int i = (int)(((uint32_t)r * c.g_inv) >> 16);
  return (q_row0 + i) * c.Hq + g * c.G + (r - i * c.G);
}

// ---------------------------------------------------------------------------
// Workgroup epilogue shared by the chunk kernels: the kWaves waves have left
// their partial states in LDS (aw[w][row][kAwPitch], mw[w][row], lw[w][row],
// all relative to their own maxima); combine them (Eq. 14 over the waves) and
// fold the result into the item's slot of the running state (Eq. 14 again).
// ---------------------------------------------------------------------------
template <int ROWS>
__device__ __forceinline__ void fold_into_slot(const Ctx &c, const UnitArg &u, int g, int M, int tx, const float *aw,
                                               const float *mw, const float *lw) {
  // SEGS threads per row (the largest power of two with SEGS * ROWS <= 256,
  // at most 32); thread seg takes the row's 16-byte pieces seg, seg + SEGS, ...,
  // so that a row's threads read and write neighbouring pieces
  constexpr int SEGS = (256 / ROWS) >= 32 ? 32 : (256 / ROWS) >= 16 ? 16 : (256 / ROWS) >= 8 ? 8 : 4;
  constexpr int PIECES = kHeadDim / 4 / SEGS;
  static_assert(PIECES >= 1 && SEGS * ROWS <= 256, "fold layout");
  const int r = tx / SEGS;
  const int seg = tx % SEGS;
  if (r >= M) return;
  float mwv[kWaves];
  float mstar = kNegInf;
#pragma unroll
  for (int w = 0; w < kWaves; ++w) {
    mwv[w] = mw[w * ROWS + r];
    mstar = fmaxf(mstar, mwv[w]);
  }
  float f[kWaves];
  float lstar = 0.f;
#pragma unroll
  for (int w = 0; w < kWaves; ++w) {
    f[w] = exp2_fast(mwv[w] - mstar);   // a wave without tokens has m = -inf -> 0
    lstar += f[w] * lw[w * ROWS + r];
  }
  f32x4_t a[PIECES];
#pragma unroll
  for (int k = 0; k < PIECES; ++k) a[k] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int w = 0; w < kWaves; ++w) {
    const float *src = aw + (w * ROWS + r) * kAwPitch + 4 * seg;
#pragma unroll
    for (int k = 0; k < PIECES; ++k) a[k] += f[w] * *reinterpret_cast<const f32x4_t *>(src + 4 * SEGS * k);
  }
  const size_t idx = (size_t)unit_slot(u) * c.R + global_row(c, u.q_row0, g, r);
  GlobalFloat *ap = c.a + idx * kHeadDim + 4 * seg;
  if (unit_fresh(u)) {               // first write of this slot in the round: store
#pragma unroll
    for (int k = 0; k < PIECES; ++k) *(GlobalFloat4 *)(ap + 4 * SEGS * k) = a[k];
    if (seg == 0) {
      c.m[idx] = mstar;
      c.l[idx] = lstar;
    }
  } else {
    const float ms = c.m[idx];
    const float mn = fmaxf(ms, mstar);
    const float alpha = exp2_fast(ms - mn);
    const float beta = exp2_fast(mstar - mn);
#pragma unroll
    for (int k = 0; k < PIECES; ++k) {
      GlobalFloat4 *o = (GlobalFloat4 *)(ap + 4 * SEGS * k);
      *o = alpha * *o + beta * a[k];
    }
    if (seg == 0) {
      c.m[idx] = mn;
      c.l[idx] = alpha * c.l[idx] + beta * lstar;
    }
  }
}

// ---------------------------------------------------------------------------
// MFMA chunk body.  Workgroup = (kv head, unit); 4 waves; wave w takes the
// 32-token tiles w, w+4, ... of the unit's chain of items (one request's
// token ranges, possibly from several chunks, attended as one sequence).
// Per tile:
//   K, V tiles -> LDS        coalesced 16-byte loads: one instruction reads 4
//                            whole 256-byte token rows (16 lanes per row)
//   S^T[t][row] = K Q^T      v_mfma_f32_16x16x32_bf16, A = K (16 tokens x 32 d,
//                            one ds_read_b128 per k-step), B = Q^T (from an
//                            LDS copy of the group's query rows)
//   online softmax per row   (row = lane % 16; the four lane groups share it)
//   O^T[d][row] += V^T P^T   A = V^T via the LDS transpose read, B = P^T
//                            straight from the S accumulators (hi and lo parts)
// Lane l: lr = l % 16, lq = l / 16.  In the S tile lane (lr, lq) holds
// tokens 16u + 4*lq + r (u = 0,1; r = 0..3) of row lr; in O it holds
// d = 16*db + 4*lq + r.  The reduction index of both MFMAs is permuted so
// every operand is contiguous: for QK^T lane group lq, k-step s covers the
// d-chunk 4*s + lq (8 values); for PV lane group lq covers tokens
// {4lq..4lq+3, 16+4lq..16+4lq+3}, exactly the S values the lane holds.
//
// LDS tiles are 32 rows of 256 bytes; 16-byte chunk c of token row t is
// stored at chunk position c ^ (t & 15) for K and c ^ 2(t & 7) for V, which
// makes the row-wise stores, the K operand reads (16 rows, same chunk) and
// the transpose reads of V (8 rows, 32 bytes each per half-wave) free of
// bank conflicts.
//
// ds_read_b64_tr_b16: within each 16-lane group, result lane i, element e is
// element (i % 4) of what source lane 4e + i/4 addressed.  Source lane j of
// group lq addresses row 4lq + j/4 (+16 for the second half), columns
// 16db + 4(j%4) .. +3, so result lane i receives V[4lq + e][16db + i].
//
// Each wave keeps the next tile's K and V in flight in registers for the
// whole compute of the current tile: a tile's loads are written to LDS at
// the top of the iteration and the next loads are issued right after.  The
// last tile is peeled so the in-loop prefetch is unconditional (a
// conditional load would make the compiler wait for every outstanding load).
// ---------------------------------------------------------------------------
constexpr int kRowBytes = kHeadDim * 2;          // 256
constexpr int kTileBytes = kTile * kRowBytes;    // 8 KiB per K or V tile

__device__ __forceinline__ int tiles_of(int tokens) { return (tokens + kTile - 1) / kTile; }

// Buffer resource over `tokens` rows from `base` on: loads past the last row
// return zero, so no clamping is needed.  Offsets are 32-bit (the host keeps
// an item below 2^31 bytes).
__device__ __forceinline__ __amdgpu_buffer_rsrc_t rows_rsrc(const Ctx &c, const uint16_t *base, int tokens) {
  const uint32_t nrec = (uint32_t)(tokens - 1) * c.stride_b + kRowBytes;
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t *>(base), (short)0, (int)nrec, kBufferFlags);
}

// Kernel-argument form of an item: what a chain needs past its first.
struct ChainItem {
  uint32_t begin;        // first token
  uint32_t word;         // tokens (below 2^24: a 2^31-byte item of 256-byte rows at most) | chunk << 24
};
// An item in registers, read as whole dwords: a byte-sized read of a kernel
// argument becomes a vector memory load, and the wait for it would also wait
// for every K/V load in flight.
struct ItemWords {
  uint32_t begin, count, chunk, cand_slot;
};
static_assert(sizeof(Item) == 16 && offsetof(Item, n_cand) == 12 && offsetof(Item, chunk) == 13 &&
              offsetof(Item, slot) == 14 && offsetof(Item, flags) == 15, "Item layout");
template <typename P>
__device__ __forceinline__ ItemWords item_at(const P &p, int i) {
  if constexpr (P::kFat) {
    uint32_t begin = p.items[i].begin, word = p.items[i].word;
    asm volatile("" : "+s"(begin), "+s"(word));
    return {begin, word & 0xffffffu, word >> 24, 0u};
  } else {
    uint32_t w[4];
    __builtin_memcpy(w, &p.items[i], sizeof w);
    asm volatile("" : "+s"(w[0]), "+s"(w[1]), "+s"(w[3]));
    return {w[0], w[1], (w[3] >> 8) & 0xffu, (w[3] & 0xffu) | (w[3] >> 16) << 8};
  }
}

// A unit's tiles are numbered across its chain of items (item 0's tiles
// first).  The cursor holds the item of the tile last asked for; it only
// moves forward.
struct Cursor {
  int k, base, end;         // item, its first tile, the tile after its last
  int count;                // its tokens
  __device__ __forceinline__ explicit Cursor(const UnitArg &u)
      : k(0), base(0), end(tiles_of(u.tok_count)), count(u.tok_count) {}
  // Move to tile T (T < the unit's tiles, T >= end); the item moved to.
  template <typename P>
  __device__ __forceinline__ ItemWords seek(const P &p, int i0, int T) {
    ItemWords it;
    do {
      it = item_at(p, i0 + ++k);
      base = end;
      end += tiles_of((int)it.count);
    } while (T >= end);
    count = (int)it.count;
    return it;
  }
};

// Resource of item `it` of KV head g through the launch's chunk table `tab` (p.k or p.v).
template <typename P>
__device__ __forceinline__ __amdgpu_buffer_rsrc_t item_rsrc(const P &p, const Ctx &c, const ItemWords &it, int g,
                                                            const uint16_t *const *tab) {
  const size_t first = (size_t)it.begin * (c.stride_b / 2) + (size_t)g * p.head_stride[it.chunk];
  return rows_rsrc(c, tab[it.chunk] + first, (int)it.count);
}

// Unit u's argument record.  Launches of the largest table class hold units as
// UnitRec and gather the rest here, behind a second round trip.
template <typename P>
__device__ __forceinline__ UnitArg unit_at(const P &p, uint32_t u) {
  UnitArg a;
  if constexpr (P::kFat) {
    a = p.units[u];
  } else {
    const UnitRec r = p.units[u];
    const int c = unit_chunk(r.word);
    const ItemWords it = item_at(p, unit_i0(r.word));
    const size_t first = (size_t)it.begin * p.tok_stride;
    a.k = p.k[c] + first;
    a.v = p.v[c] + first;
    a.hs = p.head_stride[c];
    a.word = r.word;
    a.ntiles = r.ntiles;
    a.tok_count = (int)it.count;
    a.q_row0 = r.q_row0;
    a.cand_slot = it.cand_slot;
  }
  return a;
}

// Resources and item-local token base of the next tile a wave loads.
struct NextTile {
  __amdgpu_buffer_rsrc_t krs, vrs;
  int tb;
};

template <int RB>
struct MfmaLds {
  static constexpr int kQBytes = RB * 16 * kRowBytes;               // Q rows, shared by the waves
  static constexpr int kStageBytes = kQBytes + kWaves * 2 * kTileBytes;
  static constexpr int kMergeBytes = kWaves * RB * 16 * (kAwPitch + 2) * 4;
  static constexpr int kBytes = kStageBytes > kMergeBytes ? kStageBytes : kMergeBytes;
};

typedef short s16x4_t __attribute__((ext_vector_type(4)));

__device__ __forceinline__ s16x4_t lds_read_tr16(const unsigned char *p) {
  return __builtin_amdgcn_ds_read_tr16_b64_v4i16(
      (__attribute__((address_space(3))) s16x4_t *)(reinterpret_cast<uintptr_t>(p)));
}

template <int RB, typename P>
__device__ __forceinline__ void mfma_unit(const P &p, const Ctx &c, unsigned char *smem, const UnitArg &ua, int tx, int g,
                                          int nxt) {
  const int w = __builtin_amdgcn_readfirstlane(tx >> 6);   // wave-uniform
  const int lane = tx & 63;
  const int lr = lane & 15;
  const int lq = lane >> 4;
  const int i0 = unit_i0(ua.word);
  const int M = unit_cand(ua) * c.G;
  const int ntiles = (int)ua.ntiles;

  float m_run[RB], l_run[RB];
  f32x4_t acc[RB][8];
#pragma unroll
  for (int rb = 0; rb < RB; ++rb) {
    m_run[rb] = kNegInf;
    l_run[rb] = 0.f;
#pragma unroll
    for (int db = 0; db < 8; ++db) acc[rb][db] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  }

  const uint32_t stride_b = c.stride_b;
  const uint32_t voff = lq * stride_b + 16 * lr;                     // token lq, chunk lr
  unsigned char *qs = smem;
  unsigned char *ks = smem + MfmaLds<RB>::kQBytes + w * (2 * kTileBytes);
  unsigned char *vs = ks + kTileBytes;
  const float sl2 = c.sl2;

  u32x4_t kr[8], vr[8];
  // coalesced loads: instruction i reads tokens tb + 4i + lq, chunk lr.  The
  // whole offset goes in the VGPR operand: the buffer range check covers the
  // VGPR (and immediate) offset only, not the scalar one, and rows past the
  // item must come back as zeros rather than read beyond the buffer.
  auto load_kv = [&](const NextTile &nx) {
#pragma unroll
    for (int i = 0; i < 8; ++i)
      kr[i] = __builtin_amdgcn_raw_buffer_load_b128(nx.krs, voff + (uint32_t)(nx.tb + 4 * i) * stride_b, 0, kStreamLoad);
#pragma unroll
    for (int i = 0; i < 8; ++i)
      vr[i] = __builtin_amdgcn_raw_buffer_load_b128(nx.vrs, voff + (uint32_t)(nx.tb + 4 * i) * stride_b, 0, kStreamLoad);
  };
  // K operand read: row 16u + lr, chunk 4s + lq at position (4s + lq) ^ lr
  // V transpose read: row 4lq + lr/4 (+16), chunk 2db + (lr&3)/2, half lr&1
  const int vrow = 4 * lq + (lr >> 2);
  const int vrd = vrow * kRowBytes + 8 * (lr & 1);
  const int vsw = 2 * (vrow & 7);
  const int vc0 = (lr & 3) >> 1;

  // one tile: tokens [tb, tb + 32) of an item with `count` tokens, already in
  // kr / vr; `nx` is the tile to load next (unused for a wave's last tile)
  auto tile = [&](int tb, int count, auto prefetch, const NextTile &nx) {
    constexpr bool kPrefetch = decltype(prefetch)::value;
    // stage K(i), V(i) in LDS, then issue the loads of the next tile
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int t = 4 * i + lq;
      *reinterpret_cast<u32x4_t *>(ks + t * kRowBytes + 16 * (lr ^ (t & 15))) = kr[i];
      *reinterpret_cast<u32x4_t *>(vs + t * kRowBytes + 16 * (lr ^ (2 * (t & 7)))) = vr[i];
    }
    if constexpr (kPrefetch) load_kv(nx);
    __builtin_amdgcn_sched_barrier(0);   // keep the prefetch here, ahead of the math

    // S^T = K Q^T
    f32x4_t sacc[2][RB];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      bf16x8_t kop[4];
      const int t = 16 * u + lr;
#pragma unroll
      for (int s = 0; s < 4; ++s)
        kop[s] = *reinterpret_cast<const bf16x8_t *>(ks + t * kRowBytes + 16 * ((4 * s + lq) ^ lr));
#pragma unroll
      for (int rb = 0; rb < RB; ++rb) {
        f32x4_t x = {0.f, 0.f, 0.f, 0.f};
        const unsigned char *qrow = qs + (16 * rb + lr) * kRowBytes;
#pragma unroll
        for (int s = 0; s < 4; ++s) {
          const bf16x8_t qop = *reinterpret_cast<const bf16x8_t *>(qrow + 16 * ((4 * s + lq) ^ lr));
          x = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kop[s], qop, x, 0, 0, 0);
        }
        sacc[u][rb] = x;
      }
    }

    __builtin_amdgcn_sched_barrier(0);   // phases stay apart: bounded register pressure

    // online softmax (Eq. 13 local terms merged per Eq. 14 into the wave's state)
    bf16x8_t phi[RB], plo[RB];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
      // raw scores up to the exponent (sigma log2(e) > 0 commutes with the
      // maximum); only an item's last, partial tile needs the token mask
      float x[8];
      float mx = kNegInf;
      if (tb + kTile <= count) {
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            x[4 * u + r] = sacc[u][rb][r];
            mx = fmaxf(mx, sacc[u][rb][r]);
          }
      } else {
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const int t = tb + 16 * u + 4 * lq + r;
            const float v = t < count ? sacc[u][rb][r] : kNegInf;
            x[4 * u + r] = v;
            mx = fmaxf(mx, v);
          }
      }
      const float mn = fmaxf(m_run[rb], xgroup_max(mx) * sl2);
      // Eq. 14's rescale, only when some row's maximum rose (elsewhere the
      // factor is exactly 1)
      if (__builtin_amdgcn_ballot_w64(mn > m_run[rb])) {
        const float alpha = exp2_fast(m_run[rb] - mn);
        l_run[rb] *= alpha;
#pragma unroll
        for (int db = 0; db < 8; ++db) acc[rb][db] *= alpha;
        m_run[rb] = mn;
      }
      float ls = 0.f;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const float pe = exp2_fast(__builtin_fmaf(x[e], sl2, -mn));
        const __bf16 h = (__bf16)pe;
        const float hf = (float)h;
        const __bf16 lo = (__bf16)(pe - hf);
        phi[rb][e] = h;
        plo[rb][e] = lo;
        ls += pe;
      }
      l_run[rb] += ls;
    }

    __builtin_amdgcn_sched_barrier(0);

    // O^T += V^T P^T  (hi and lo parts of P)
#pragma unroll
    for (int db = 0; db < 8; ++db) {
      const int off = vrd + 16 * ((2 * db + vc0) ^ vsw);
      const s16x4_t v0 = lds_read_tr16(vs + off);
      const s16x4_t v1 = lds_read_tr16(vs + off + 16 * kRowBytes);
      const bf16x8_t vop = __builtin_bit_cast(
          bf16x8_t, __builtin_shufflevector(v0, v1, 0, 1, 2, 3, 4, 5, 6, 7));
#pragma unroll
      for (int rb = 0; rb < RB; ++rb) {
        acc[rb][db] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vop, phi[rb], acc[rb][db], 0, 0, 0);
        acc[rb][db] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vop, plo[rb], acc[rb][db], 0, 0, 0);
      }
    }
  };

  // Q rows of this (request, kv head) -> LDS, chunk c of row r at c ^ (r & 15);
  // rows >= M are zero.  The Q^T operand (B[k = d][j = row]) of lane (lr, lq),
  // k-step s, is row lr's d-chunk 4s + lq.  The query loads are issued first,
  // then the first K/V tile, so staging Q waits only for the query rows.
  // They are buffer loads over the whole Q tensor: a padding row (r >= M)
  // gets an offset past the end and reads zero, so no load sits behind a
  // branch (whose merge with the zero default would force an early wait).
  constexpr int kQPerThread = RB * 16 * 16 / 256;
  const __amdgpu_buffer_rsrc_t qrs = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<uint16_t *>(c.q), (short)0, (int)(c.R * kRowBytes), kBufferFlags);
  u32x4_t qv[kQPerThread];
#pragma unroll
  for (int e = 0; e < kQPerThread; ++e) {
    const int ci = tx + 256 * e, r = ci >> 4, ch = ci & 15;
    const uint32_t qoff = r < M ? (uint32_t)global_row(c, ua.q_row0, g, r) * kRowBytes + 16 * ch : 0x80000000u;
    qv[e] = __builtin_amdgcn_raw_buffer_load_b128(qrs, qoff, 0, 0);
  }
  // wave w takes the chain's tiles T = w, w + 4, ...  The first tile's loads
  // are issued unconditionally (a wave without tiles loads through an empty
  // resource, which reads nothing), so the wait for the query rows below
  // does not have to include them.  A wave whose first tile lies in a later
  // item of the chain rebuilds its resources from that item.
  int T = w;
  Cursor cur(ua);
  NextTile nx;
  const __amdgpu_buffer_rsrc_t empty =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t *>(c.q), (short)0, 0, kBufferFlags);
  const bool has_tile = T < ntiles;
  nx.krs = has_tile ? rows_rsrc(c, ua.k + (size_t)g * ua.hs, ua.tok_count) : empty;
  nx.vrs = has_tile ? rows_rsrc(c, ua.v + (size_t)g * ua.hs, ua.tok_count) : empty;
  if (has_tile && T >= cur.end) {
    const ItemWords ic = cur.seek(p, i0, T);
    nx.krs = item_rsrc(p, c, ic, g, p.k);
    nx.vrs = item_rsrc(p, c, ic, g, p.v);
  }
  nx.tb = (T - cur.base) * kTile;
  __builtin_amdgcn_sched_barrier(0);   // the query loads go out first
  load_kv(nx);
  // The workgroup's next unit of its own list (nxt >= 0): its first item's
  // resources, read now, so that each wave can bring the lines of its first
  // tile of that unit into the L2 cache during its last tile of this one.
  __amdgpu_buffer_rsrc_t wkrs = empty, wvrs = empty;
  if (nxt >= 0) {
    const UnitArg un = unit_at(p, (uint32_t)nxt);
    wkrs = rows_rsrc(c, un.k + (size_t)g * un.hs, un.tok_count);
    wvrs = rows_rsrc(c, un.v + (size_t)g * un.hs, un.tok_count);
  }
#pragma unroll
  for (int e = 0; e < kQPerThread; ++e) {
    const int ci = tx + 256 * e, r = ci >> 4, ch = ci & 15;
    *reinterpret_cast<u32x4_t *>(qs + r * kRowBytes + 16 * (ch ^ (r & 15))) = qv[e];
  }
  __syncthreads();

  if (T < ntiles) {
    for (; T + kWaves < ntiles; T += kWaves) {
      const int tb = nx.tb, count = cur.count;
      if (T + kWaves >= cur.end) {
        const ItemWords in = cur.seek(p, i0, T + kWaves);
        nx.krs = item_rsrc(p, c, in, g, p.k);
        nx.vrs = item_rsrc(p, c, in, g, p.v);
      }
      nx.tb = (T + kWaves - cur.base) * kTile;
      tile(tb, count, std::integral_constant<bool, true>{}, nx);
    }
    // one 4-byte read per 128-byte line of this wave's first tile of the
    // next unit (tokens 32w .. 32w+31 of its first item, K and V; reads
    // past the item return zero without touching memory), at the default
    // cache policy so the lines stay in L2; the values are only kept alive
    // until the last tile is done, where the wait for them is free
    uint32_t warm_k = 0, warm_v = 0;
    if (nxt >= 0) {
      const uint32_t wo = (uint32_t)(kTile * w + (lane >> 1)) * stride_b + 128u * (uint32_t)(lane & 1);
      warm_k = __builtin_amdgcn_raw_buffer_load_b32(wkrs, wo, 0, 0);
      warm_v = __builtin_amdgcn_raw_buffer_load_b32(wvrs, wo, 0, 0);
    }
    tile(nx.tb, cur.count, std::integral_constant<bool, false>{}, nx);
    asm volatile("" ::"v"(warm_k), "v"(warm_v));
  }

  // wave partials -> LDS
#pragma unroll
  for (int rb = 0; rb < RB; ++rb) l_run[rb] = xgroup_sum(l_run[rb]);
  __syncthreads();
  float *aw = reinterpret_cast<float *>(smem);
  float *mw = aw + kWaves * RB * 16 * kAwPitch;
  float *lw = mw + kWaves * RB * 16;
#pragma unroll
  for (int rb = 0; rb < RB; ++rb) {
    float *row = aw + (w * RB * 16 + rb * 16 + lr) * kAwPitch + 4 * lq;
#pragma unroll
    for (int db = 0; db < 8; ++db) *reinterpret_cast<f32x4_t *>(row + 16 * db) = acc[rb][db];
    if (lq == 0) {
      mw[w * RB * 16 + rb * 16 + lr] = m_run[rb];
      lw[w * RB * 16 + rb * 16 + lr] = l_run[rb];
    }
  }
  __syncthreads();
  fold_into_slot<RB * 16>(c, ua, g, M, tx, aw, mw, lw);
}

// ---------------------------------------------------------------------------
// Row-split MFMA body for wide query groups (33..64 rows per KV head).  The
// four waves attend 64 tokens (two 32-token tiles) a step: wave w owns the rows
// from 32 (w / 2) on and the tiles 2k + w % 2 of the unit's chain, and the two
// waves of a row block merge their states once, at the unit's end.  A block is
// 32 rows with v_mfma_f32_32x32x16_bf16; the second block of a unit of at most
// 48 rows is 16 rows with v_mfma_f32_16x16x32_bf16.  Per step and wave: S^T =
// K Q^T (8 MFMAs, Q in registers), the online softmax (a row's 32 scores lie
// in 64 / rows lanes), O^T += V^T P^T with P as hi + lo (16).  What bounds the
// body is the matrix, vector and LDS work that a step puts behind its barrier,
// and the shader clock that sustained work of this kind leaves (1.6-1.7 GHz).
// Every K and V byte is read from LDS by two waves; with 16 rows per wave and
// 32 tokens a step it was read by four, with twice the barriers and row maxima
// per token.  Rounds back to back, that body, this one with 32 rows a wave
// throughout, and this one:
//   16 x 32768 tokens, 64 rows        350.7  337.0  337.1 us
//   16 x 32768, 48 rows               329.8  334.4  322.0
//   16 x 32768, 40 rows               329.5  327.8  318.3
//   16 x 60000, 48 rows               589.8  601.3  574.2
//   4 x 16384, 48 rows                 56.0   54.1   52.2
// (64 rows: LDS busy 0.62 of before, VALU 0.88).  V's second k-step is read
// after the first's products: 339 against 344 us with both read ahead.  Two
// steps of loads in flight instead of one spill 23 to 39 registers and take 380
// us.
//
// Lane l of a wave of n rows: lr = l % n, lh = l / n, G = 64 / n lane groups.
// In the S tile lane (lr, lh) holds tokens 4 G (r / 4) + 4 lh + r % 4 of row lr
// (r = 0 .. 32 / G - 1); in O it holds d = 4 G q + 4 lh .. + 3 as piece q.  The
// reduction index of both MFMAs is permuted so that every operand is
// contiguous: for QK^T k-step s, lane group lh covers the d-chunk G s + lh; for
// PV k-step s it covers tokens 16 s + {4 lh .. +3, 4 G + 4 lh .. +3}, the S
// values the lane holds.  V is read through the LDS transpose (see above): a
// 16-lane group reads 4 tokens x 16 d.  16-byte chunk c of token row t lies at
// c ^ (t & 15) for K, as above, and for V at c ^ (4 (t & 3) + 2 (t / 4 & 1)), so
// that the 32 lanes of a transpose read (4 rows, 64 bytes each, or 8 rows, 32
// bytes each) touch every bank once.
//
// Step k is staged in buffer k % 2 by all waves together (wave w loads tokens
// 16 (w / 2) .. +15 of its tile), with one workgroup barrier; each wave keeps
// the next kRowsAhead steps' loads in flight in registers.  A wave writes
// buffer k % 2 only after the barrier of step k - 1, which every wave reaches
// after attending step k - 2, the buffer's previous contents; the barrier of
// step k then makes the whole step visible.  Every wave runs the same number
// of barriers: the steps run in groups of kRowsGroup, and a step past the
// unit's end stages zeros and attends nothing.  Loads for tiles past the end
// go through an empty buffer resource, which reads zeros without touching
// memory.
// ---------------------------------------------------------------------------
constexpr int kRowsAhead = 1;                          // steps of loads in flight per wave
constexpr int kRowsGroup = 2;                          // steps per loop iteration: even, a multiple of kRowsAhead
constexpr int kRowsStepBytes = 2 * 2 * kTileBytes;     // K and V of two tiles
constexpr int kRowsMergeBytes = kWaves * (8 * 64 * 16 + 2 * 32 * 4);
constexpr int kRowsLdsBytes = 2 * kRowsStepBytes > kRowsMergeBytes ? 2 * kRowsStepBytes : kRowsMergeBytes;
static_assert(kRowsGroup % 2 == 0 && kRowsGroup % kRowsAhead == 0, "step i of a group uses buffer i % 2");

// A wave's part of a unit: rows 32 rb .. 32 rb + ROWS - 1, the tiles of parity w % 2.
template <int ROWS, typename P>
__device__ __forceinline__ void rows_wave(const P &p, const Ctx &cx, unsigned char *smem, const UnitArg &ua, int w, int rb,
                                          int lane, int g) {
  static_assert(ROWS == 32 || ROWS == 16, "v_mfma_f32_32x32x16_bf16 or v_mfma_f32_16x16x32_bf16");
  using Acc = std::conditional_t<ROWS == 32, f32x16_t, f32x4_t>;
  constexpr int kGroups = 64 / ROWS;                       // lane groups that share a row
  constexpr int kQSteps = 16 / kGroups, kPSteps = 2 / (kGroups / 2);
  constexpr int kScores = 32 / kGroups;                    // of a tile, per lane
  constexpr int kBlocks = kHeadDim / ROWS, kPieces = 32 / kGroups;   // accumulators of ROWS d each; 16-byte pieces of them
  const int th = w & 1;                                    // tile parity
  const int lr = lane % ROWS, lh = lane / ROWS;            // row, lane group
  const int i0 = unit_i0(ua.word);
  const int M = unit_cand(ua) * cx.G;
  const int ntiles = (int)ua.ntiles;

  const uint32_t stride_b = cx.stride_b;
  const int sr = lane & 15, sq = lane >> 4;                  // staging: chunk, row within four
  const uint32_t voff = (16 * rb + sq) * stride_b + 16 * sr;
  const float sl2 = cx.sl2;

  // Q^T operand (B[k = d][j = row]) of row 32 rb + lr, k-step s: d-chunk
  // kGroups s + lh.  A padding row (>= M) gets an offset past the end: zeros.
  const int row = 32 * rb + lr;
  const __amdgpu_buffer_rsrc_t qrs = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<uint16_t *>(cx.q), (short)0, (int)(cx.R * kRowBytes), kBufferFlags);
  const uint32_t qoff = row < M ? (uint32_t)global_row(cx, ua.q_row0, g, row) * kRowBytes + 16 * lh : 0x80000000u;
  bf16x8_t qop[kQSteps];
#pragma unroll
  for (int s = 0; s < kQSteps; ++s)
    qop[s] = __builtin_bit_cast(bf16x8_t, __builtin_amdgcn_raw_buffer_load_b128(qrs, qoff + 16 * kGroups * s, 0, 0));
  __builtin_amdgcn_sched_barrier(0);   // the query loads go out first

  // loads of tile t (2k + th): K rows 16 rb + 4j + sq, then the same V rows.
  // Tiles are requested in order; the resources of the current item are
  // kept and rebuilt only when the tile moves on to the next item, so a
  // step issues its loads without a chain of dependent argument reads.
  // The loads themselves are unconditional (a conditional load would make
  // the compiler wait for every outstanding one): past the unit's last tile
  // they go through an empty resource.
  const __amdgpu_buffer_rsrc_t empty =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t *>(cx.q), (short)0, 0, kBufferFlags);
  Cursor lcur(ua);
  __amdgpu_buffer_rsrc_t lkrs = rows_rsrc(cx, ua.k + (size_t)g * ua.hs, ua.tok_count);
  __amdgpu_buffer_rsrc_t lvrs = rows_rsrc(cx, ua.v + (size_t)g * ua.hs, ua.tok_count);
  auto issue = [&](u32x4_t (&d)[8], int t) {
    if (t >= lcur.end && t < ntiles) {
      const ItemWords il = lcur.seek(p, i0, t);
      lkrs = item_rsrc(p, cx, il, g, p.k);
      lvrs = item_rsrc(p, cx, il, g, p.v);
    }
    const bool in = t < ntiles;
    const __amdgpu_buffer_rsrc_t krs = in ? lkrs : empty;
    const __amdgpu_buffer_rsrc_t vrs = in ? lvrs : empty;
    const uint32_t o = voff + (uint32_t)(in ? (t - lcur.base) * kTile : 0) * stride_b;
#pragma unroll
    for (int j = 0; j < 4; ++j) d[j] = __builtin_amdgcn_raw_buffer_load_b128(krs, o + 4 * j * stride_b, 0, kStreamLoad);
#pragma unroll
    for (int j = 0; j < 4; ++j)
      d[4 + j] = __builtin_amdgcn_raw_buffer_load_b128(vrs, o + 4 * j * stride_b, 0, kStreamLoad);
  };
  unsigned char *tile_lds = smem + th * (2 * kTileBytes);   // the wave's tile in buffer 0: K, then V
  auto stage = [&](const u32x4_t (&d)[8], unsigned char *buf) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int t = 16 * rb + 4 * j + sq;
      *reinterpret_cast<u32x4_t *>(buf + t * kRowBytes + 16 * (sr ^ (t & 15))) = d[j];
      *reinterpret_cast<u32x4_t *>(buf + kTileBytes + t * kRowBytes + 16 * (sr ^ (4 * sq + 2 * (j & 1)))) = d[4 + j];
    }
  };

  float m_run = kNegInf, l_run = 0.f;
  Acc acc[kBlocks];
#pragma unroll
  for (int db = 0; db < kBlocks; ++db) acc[db] = Acc{};
  // transpose read of the 16-lane group sq: row 4 lh + j / 4 of the four,
  // columns 4 (j % 4) of its 16 d, j = lane % 16
  const int vrd = (4 * lh + (sr >> 2)) * kRowBytes + 16 * ((sr & 3) >> 1) + 8 * (sr & 1);
  const int vsw = (64 * (sr >> 2) + 32 * (lh & 1)) ^ (ROWS == 32 ? 32 * (sq & 1) : 0);
  const int krd = lr * kRowBytes, ksw = 16 * (lh ^ (lr & 15));
  Cursor cur(ua);   // of the tile being attended

  // attend the wave's staged tile t (tokens [tb, tb + 32) of an item with `count` tokens)
  auto attend = [&](const unsigned char *buf, int t) {
    if (t >= cur.end) cur.seek(p, i0, t);
    const int tb = (t - cur.base) * kTile, count = cur.count;
    const unsigned char *vs = buf + kTileBytes;
    auto k_operand = [&](int s, int t0) {
      return *reinterpret_cast<const bf16x8_t *>(buf + t0 * kRowBytes + krd + (ksw ^ (16 * kGroups * s)));
    };
    float c[kScores];
    if constexpr (ROWS == 32) {
      f32x16_t x = {};
#pragma unroll
      for (int s = 0; s < kQSteps; ++s) x = __builtin_amdgcn_mfma_f32_32x32x16_bf16(k_operand(s, 0), qop[s], x, 0, 0, 0);
#pragma unroll
      for (int r = 0; r < kScores; ++r) c[r] = x[r];
    } else {
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        f32x4_t x = {};
#pragma unroll
        for (int s = 0; s < kQSteps; ++s)
          x = __builtin_amdgcn_mfma_f32_16x16x32_bf16(k_operand(s, 16 * u), qop[s], x, 0, 0, 0);
#pragma unroll
        for (int r = 0; r < 4; ++r) c[4 * u + r] = x[r];
      }
    }
    // the V^T operands of k-step 0 go out now, so their LDS latency hides behind the softmax
    bf16x8_t vop[kBlocks];
    auto load_v = [&](int s) {
#pragma unroll
      for (int db = 0; db < kBlocks; ++db) {
        const unsigned char *a = vs + vrd + ((2 * ROWS * db) ^ vsw) + 16 * s * kRowBytes;
        const s16x4_t v0 = lds_read_tr16(a);
        const s16x4_t v1 = lds_read_tr16(a + 4 * kGroups * kRowBytes);
        vop[db] = __builtin_bit_cast(bf16x8_t, __builtin_shufflevector(v0, v1, 0, 1, 2, 3, 4, 5, 6, 7));
      }
    };
    load_v(0);

    __builtin_amdgcn_sched_barrier(0);

    // Scores stay unscaled up to the exponent: the row maximum of the raw
    // scores times sigma log2(e) (> 0) is the maximum of the scaled ones,
    // and each weight is 2^(x sigma log2(e) - m) with one fma.  Only an
    // item's last, partial tile needs the token mask.
    if (tb + kTile > count) {
#pragma unroll
      for (int r = 0; r < kScores; ++r) c[r] = tb + 4 * kGroups * (r >> 2) + 4 * lh + (r & 3) < count ? c[r] : kNegInf;
    }
    float mx = c[0];
#pragma unroll
    for (int r = 1; r < kScores; ++r) mx = fmaxf(mx, c[r]);
    const float mn = fmaxf(m_run, (ROWS == 32 ? x32_max(mx) : xgroup_max(mx)) * sl2);
    const float mb = mn == kNegInf ? 0.f : mn;   // scores of -inf alone so far: weights 0
    // Eq. 14's rescale, only when some row's maximum rose (elsewhere the
    // factor is exactly 1)
    if (__builtin_amdgcn_ballot_w64(mn > m_run)) {
      const float alpha = exp2_fast(m_run - mb);
      l_run *= alpha;
#pragma unroll
      for (int db = 0; db < kBlocks; ++db) acc[db] *= alpha;
      m_run = mn;
    }
    bf16x8_t phi[kPSteps], plo[kPSteps];
    float ls = 0.f;
#pragma unroll
    for (int r = 0; r < kScores; ++r) {
      const float pe = exp2_fast(__builtin_fmaf(c[r], sl2, -mb));
      const __bf16 h = (__bf16)pe;
      const float hf = (float)h;
      const __bf16 lo = (__bf16)(pe - hf);
      phi[r >> 3][r & 7] = h;
      plo[r >> 3][r & 7] = lo;
      ls += pe;
    }
    l_run += ls;

    __builtin_amdgcn_sched_barrier(0);

    auto weigh = [&](const bf16x8_t &weights) {
#pragma unroll
      for (int db = 0; db < kBlocks; ++db) {
        if constexpr (ROWS == 32)
          acc[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vop[db], weights, acc[db], 0, 0, 0);
        else
          acc[db] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vop[db], weights, acc[db], 0, 0, 0);
      }
    };
#pragma unroll
    for (int s = 0; s < kPSteps; ++s) {
      if (s) load_v(1);
      weigh(phi[s]);
      weigh(plo[s]);
    }
  };

  const int steps = (ntiles + 1) / 2;
  u32x4_t ld[kRowsAhead][8];
#pragma unroll
  for (int i = 0; i < kRowsAhead; ++i) issue(ld[i], 2 * i + th);
  for (int k0 = 0; k0 < steps; k0 += kRowsGroup) {
#pragma unroll
    for (int i = 0; i < kRowsGroup; ++i) {
      const int t = 2 * (k0 + i) + th;
      unsigned char *buf = tile_lds + (i & 1) * kRowsStepBytes;
      stage(ld[i % kRowsAhead], buf);
      issue(ld[i % kRowsAhead], t + 2 * kRowsAhead);
      __syncthreads();
      if (t < ntiles) attend(buf, t);
    }
  }

  // Merge the two waves of a row block (Eq. 14): wave th keeps the pieces of
  // half th of d and hands the others over through LDS.  A wave without
  // tiles has m = -inf, which scales its zeros by 0.  The slot's old m and l
  // are read before the barrier, as the block's first wave replaces them.
  l_run = ROWS == 32 ? x32_sum(l_run) : xgroup_sum(l_run);
  const bool stores = row < M;
  const bool merge_slot = !unit_fresh(ua);
  const size_t idx = (size_t)unit_slot(ua) * cx.R + (stores ? global_row(cx, ua.q_row0, g, row) : 0);
  float ms = kNegInf, lsl = 0.f;
  if (merge_slot && stores) {
    ms = cx.m[idx];
    lsl = cx.l[idx];
  }
  asm volatile("" : "+v"(ms), "+v"(lsl));
  __syncthreads();                       // every wave is done with the tile buffers
  f32x4_t *sh = reinterpret_cast<f32x4_t *>(smem);
  float *m_sh = reinterpret_cast<float *>(smem + kWaves * 8 * 64 * 16), *l_sh = m_sh + kWaves * 32;
  // piece q of the accumulators: d = 4 kGroups q + 4 lh .. + 3 of row lr
  auto piece = [&](int q) {
    f32x4_t a;
#pragma unroll
    for (int e = 0; e < 4; ++e) a[e] = ROWS == 32 ? acc[q >> 2][4 * (q & 3) + e] : acc[q][e];
    return a;
  };
  auto half_piece = [&](int half, int q) {
    const f32x4_t lo = piece(q), hi = piece(kPieces / 2 + q);
    f32x4_t a;
#pragma unroll
    for (int e = 0; e < 4; ++e) a[e] = half ? hi[e] : lo[e];
    return a;
  };
#pragma unroll
  for (int q = 0; q < kPieces / 2; ++q) sh[(w * 8 + q) * 64 + lane] = half_piece(th ^ 1, q);
  if (lh == 0) {
    m_sh[w * 32 + lr] = m_run;
    l_sh[w * 32 + lr] = l_run;
  }
  __syncthreads();
  if (!stores) return;
  const float m2 = m_sh[(w ^ 1) * 32 + lr], l2 = l_sh[(w ^ 1) * 32 + lr];
  const float mn = fmaxf(fmaxf(m_run, m2), ms), mb = mn == kNegInf ? 0.f : mn;
  const float f0 = exp2_fast(m_run - mb), f1 = exp2_fast(m2 - mb), fs = merge_slot ? exp2_fast(ms - mb) : 0.f;
  GlobalFloat *ap = cx.a + idx * kHeadDim + 64 * th + 4 * lh;
#pragma unroll
  for (int q = 0; q < kPieces / 2; ++q) {
    f32x4_t o = f0 * half_piece(th, q) + f1 * sh[((w ^ 1) * 8 + q) * 64 + lane];
    GlobalFloat4 *dst = (GlobalFloat4 *)(ap + 4 * kGroups * q);
    if (merge_slot) o += fs * *dst;
    *dst = o;
  }
  if (th == 0 && lh == 0) {
    cx.m[idx] = mn;
    cx.l[idx] = f0 * l_run + f1 * l2 + fs * lsl;
  }
}

// Every wave runs the same barriers, whatever its rows.
template <typename P>
__device__ __forceinline__ void rows_unit(const P &p, const Ctx &cx, unsigned char *smem, const UnitArg &ua, int tx, int g) {
  const int w = __builtin_amdgcn_readfirstlane(tx >> 6);   // wave-uniform
  const int lane = tx & 63, rb = w >> 1;
  if (rb == 1 && unit_kind(ua.word) == kUnitMfma3)
    rows_wave<16>(p, cx, smem, ua, w, rb, lane, g);
  else
    rows_wave<32>(p, cx, smem, ua, w, rb, lane, g);
}

// ---------------------------------------------------------------------------
// VALU chunk body for sparse query groups (few rows per KV head), used when
// the round's mfma_min_rows asks for it: fp32 dot products on the vector
// ALUs, exact fp32 softmax weights.  Lane l: d-chunk
// c = l % 16 (8 values), token group tg = l / 16; a 32-token tile is 8
// coalesced loads (4 token rows of 256 B each) of K and of V.  Scores are
// reduced over the 16 lanes of a DPP row.
// ---------------------------------------------------------------------------
template <int MAXR, typename P>
__device__ __forceinline__ void valu_unit(const P &p, const Ctx &cx, float *smem, const UnitArg &ua, int tx, int g) {
  const int w = __builtin_amdgcn_readfirstlane(tx >> 6);   // wave-uniform
  const int lane = tx & 63;
  const int c = lane & 15;
  const int tg = lane >> 4;
  const int i0 = unit_i0(ua.word);
  const int M = unit_cand(ua) * cx.G;
  const int ntiles = (int)ua.ntiles;

  float qf[MAXR][8];
#pragma unroll
  for (int r = 0; r < MAXR; ++r) {
    if (r < M) {
      const u32x4_t q4 = ((const GlobalU32x4 *)(cx.q + (size_t)global_row(cx, ua.q_row0, g, r) * kHeadDim))[c];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        qf[r][2 * e] = bf16_lo(q4[e]);
        qf[r][2 * e + 1] = bf16_hi(q4[e]);
      }
    } else {
#pragma unroll
      for (int e = 0; e < 8; ++e) qf[r][e] = 0.f;
    }
  }
  float m_run[MAXR], l_run[MAXR], acc[MAXR][8];
#pragma unroll
  for (int r = 0; r < MAXR; ++r) {
    m_run[r] = kNegInf;
    l_run[r] = 0.f;
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[r][e] = 0.f;
  }
  const uint32_t stride_b = cx.stride_b;
  const uint32_t voff = tg * stride_b + 16 * c;
  const float sl2 = cx.sl2;

  // coalesced loads (4 token rows per instruction); tokens past the item read 0
  u32x4_t kr[8], vr[8];
  // the whole offset goes in the range-checked VGPR operand (see the MFMA kernel)
  auto load_k = [&](const NextTile &nx) {
#pragma unroll
    for (int i = 0; i < 8; ++i)
      kr[i] = __builtin_amdgcn_raw_buffer_load_b128(nx.krs, voff + (uint32_t)(nx.tb + 4 * i) * stride_b, 0, kStreamLoad);
  };
  auto load_v = [&](const NextTile &nx) {
#pragma unroll
    for (int i = 0; i < 8; ++i)
      vr[i] = __builtin_amdgcn_raw_buffer_load_b128(nx.vrs, voff + (uint32_t)(nx.tb + 4 * i) * stride_b, 0, kStreamLoad);
  };
  // one tile per iteration (tokens [tb, tb + 32) of an item with `count`
  // tokens); the next tile's K is issued after the scores, its V after the
  // PV update; the last tile is peeled (unconditional prefetch)
  auto tile = [&](int tb, int count, auto prefetch, const NextTile &nx) {
    constexpr bool more = decltype(prefetch)::value;
    float x[8][MAXR];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      float kf[8];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        kf[2 * e] = bf16_lo(kr[i][e]);
        kf[2 * e + 1] = bf16_hi(kr[i][e]);
      }
      const bool valid = tb + 4 * i + tg < count;
#pragma unroll
      for (int r = 0; r < MAXR; ++r) {
        float d = 0.f;
#pragma unroll
        for (int e = 0; e < 8; ++e) d = fmaf(qf[r][e], kf[e], d);
        d = row16_sum(d);
        x[i][r] = valid ? d * sl2 : kNegInf;
      }
    }
    if constexpr (more) load_k(nx);
#pragma unroll
    for (int r = 0; r < MAXR; ++r) {
      float mx = kNegInf;
#pragma unroll
      for (int i = 0; i < 8; ++i) mx = fmaxf(mx, x[i][r]);
      mx = xgroup_max(mx);
      const float mn = fmaxf(m_run[r], mx);
      const float alpha = exp2_fast(m_run[r] - mn);
      m_run[r] = mn;
      l_run[r] *= alpha;
#pragma unroll
      for (int e = 0; e < 8; ++e) acc[r][e] *= alpha;
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const float pe = exp2_fast(x[i][r] - mn);
        x[i][r] = pe;
        l_run[r] += pe;
      }
    }
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      float vf[8];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        vf[2 * e] = bf16_lo(vr[i][e]);
        vf[2 * e + 1] = bf16_hi(vr[i][e]);
      }
#pragma unroll
      for (int r = 0; r < MAXR; ++r)
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[r][e] = fmaf(x[i][r], vf[e], acc[r][e]);
    }
    if constexpr (more) load_v(nx);
  };
  // wave w takes the chain's tiles T = w, w + 4, ...
  int T = w;
  if (T < ntiles) {
    Cursor cur(ua);
    NextTile nx;
    nx.krs = rows_rsrc(cx, ua.k + (size_t)g * ua.hs, ua.tok_count);
    nx.vrs = rows_rsrc(cx, ua.v + (size_t)g * ua.hs, ua.tok_count);
    if (T >= cur.end) {
      const ItemWords ic = cur.seek(p, i0, T);
      nx.krs = item_rsrc(p, cx, ic, g, p.k);
      nx.vrs = item_rsrc(p, cx, ic, g, p.v);
    }
    nx.tb = (T - cur.base) * kTile;
    load_k(nx);
    load_v(nx);
    for (; T + kWaves < ntiles; T += kWaves) {
      const int tb = nx.tb, count = cur.count;
      if (T + kWaves >= cur.end) {
        const ItemWords in = cur.seek(p, i0, T + kWaves);
        nx.krs = item_rsrc(p, cx, in, g, p.k);
        nx.vrs = item_rsrc(p, cx, in, g, p.v);
      }
      nx.tb = (T + kWaves - cur.base) * kTile;
      tile(tb, count, std::integral_constant<bool, true>{}, nx);
    }
    tile(nx.tb, cur.count, std::integral_constant<bool, false>{}, nx);
  }

  // reduce over the token groups, partials -> LDS
#pragma unroll
  for (int r = 0; r < MAXR; ++r) {
    l_run[r] = xgroup_sum(l_run[r]);
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[r][e] = xgroup_sum(acc[r][e]);
  }
  float *aw = smem;
  float *mw = aw + kWaves * MAXR * kAwPitch;
  float *lw = mw + kWaves * MAXR;
  if (tg == 0) {
#pragma unroll
    for (int r = 0; r < MAXR; ++r) {
      float *row = aw + (w * MAXR + r) * kAwPitch + 8 * c;
      *reinterpret_cast<f32x4_t *>(row) = f32x4_t{acc[r][0], acc[r][1], acc[r][2], acc[r][3]};
      *reinterpret_cast<f32x4_t *>(row + 4) = f32x4_t{acc[r][4], acc[r][5], acc[r][6], acc[r][7]};
      if (c == 0) {
        mw[w * MAXR + r] = m_run[r];
        lw[w * MAXR + r] = l_run[r];
      }
    }
  }
  __syncthreads();
  fold_into_slot<MAXR>(cx, ua, g, M, tx, aw, mw, lw);
}

constexpr int kValuLdsBytes = kWaves * kMaxValuRows * (kAwPitch + 2) * 4;
constexpr int kChunkLdsBytes = MfmaLds<2>::kBytes > kValuLdsBytes ? MfmaLds<2>::kBytes : kValuLdsBytes;
static_assert(MfmaLds<1>::kBytes <= kChunkLdsBytes, "LDS sizes");
static_assert(kRowsLdsBytes <= kChunkLdsBytes && 2 * kChunkLdsBytes <= 160 * 1024, "LDS sizes");

// ---------------------------------------------------------------------------
// History kernel: one launch for every unit of a call.  Workgroup w of KV
// head g first attends the units of its own list in order (the host gives
// every workgroup an equal share of the call's tokens, which may span
// several requests); each unit's kind selects the body: MFMA with two or
// one 16-row blocks, the row-split body for three or four (only on the wide
// instantiation, which a launch with such a unit runs on), or the VALU path
// for <= 4 rows (built for 1, 2 and 4 rows).  The grid is (g, w) with the
// heads as the fast dimension for token-major chunks, where the eight XCDs
// then read the eight heads of the same tokens, and (w, g) for head-major
// chunks, where every XCD then reads every head's plane: on MI355X a
// head-major launch over 16 x 32768 tokens took 354 us with the heads fast
// and 323 us the other way round (the same box; a loads-only copy of the
// kernel 347 against 318 us, and a plain read of the same 2 GiB 301 us).
//
// The XCDs do not stream at the same rate (on MI355X some finish an equal
// share 10% later than others), so the host may hold back the last part of
// every share as a tail of small units, largest first.  A workgroup that has
// finished its own list claims (tail unit, KV head) pairs from a counter
// until none is left, whatever its own head; each tail unit still owns a
// fixed state slot, so the result does not depend on who attends it.  Every
// workgroup makes exactly one claim past the last pair and then stops, so a
// launch makes num_tail * Hkv + (workgroups) claims; the one that receives
// the last number sets the counter back to zero for the next launch.
// Claims are compared without sign: a counter that is not zero at launch
// (garbage, or a broken workspace promise) gives large numbers, which end
// the loop instead of indexing outside the tail.
// ---------------------------------------------------------------------------
template <bool Wide, typename P>
__device__ __forceinline__ void attend_units(const P &p) {
  __shared__ __attribute__((aligned(16))) unsigned char smem[kChunkLdsBytes];
  __shared__ uint32_t claim_sh;
  // Grid (Hkv, workgroups, 1) or (1, workgroups, Hkv): see the launch.
  const uint32_t y = blockIdx.y;                       // workgroup of its KV head
  const int g_own = (int)(blockIdx.x + blockIdx.z);    // KV head of its own units
  // The workgroup's first unit, the range of its further units and what all
  // bodies need of the arguments are read in one scalar round trip and forced
  // into registers here, so that neither the first unit's loads nor its end
  // wait for another.
  UnitArg ua = unit_at(p, y);
  uint32_t more0 = p.more[y], more1 = p.more[y + 1];
  Ctx cx = {p.q, (GlobalFloat *)p.st.a, (GlobalFloat *)p.st.m, (GlobalFloat *)p.st.l, (uint32_t)p.st.R, p.Hq, p.G,
            p.g_inv, p.scale_log2, p.tok_stride * 2};
  asm volatile("" : "+s"(ua.k), "+s"(ua.v), "+s"(ua.hs), "+s"(ua.word), "+s"(ua.ntiles), "+s"(ua.tok_count),
               "+s"(ua.q_row0), "+s"(ua.cand_slot), "+s"(more0), "+s"(more1), "+s"(cx.q), "+s"(cx.a), "+s"(cx.m),
               "+s"(cx.l), "+s"(cx.R), "+s"(cx.Hq), "+s"(cx.G), "+s"(cx.g_inv), "+s"(cx.sl2), "+s"(cx.stride_b));
  const uint32_t nclaims = (uint32_t)p.num_tail * (uint32_t)p.Hkv;
  const uint32_t last_claim = nclaims + (uint32_t)p.Hkv * (uint32_t)p.num_wgs - 1u;
  uint32_t u = more0;
  bool first = true;
  for (;;) {
    int g = g_own;
    if (first) {
      first = false;
      if (unit_nit(ua.word) == 0) continue;   // a workgroup without units of its own
    } else if (u < more1) {
      __syncthreads();   // the previous unit's fold has read the LDS this unit restages
      ua = unit_at(p, u++);
    } else {
      if (nclaims == 0) break;
      __syncthreads();   // ... and every thread has read the previous claim
      if (threadIdx.x == 0) {
        const uint32_t c = atomicAdd(p.claim, 1u);
        if (c == last_claim) __hip_atomic_store(p.claim, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        claim_sh = c;
      }
      __syncthreads();
      const uint32_t c = __builtin_amdgcn_readfirstlane(claim_sh);
      if (c >= nclaims) break;
      uint32_t hkv = (uint32_t)p.Hkv;
      asm volatile("" : "+s"(hkv));   // keeps the division's set-up out of the launch's start
      const uint32_t t = c / hkv;
      ua = unit_at(p, (uint32_t)p.tail_first + t);
      g = (int)(c - t * hkv);
    }
    // The bodies derive their per-lane addresses from tx.  Passing it
    // through an empty asm each unit keeps the compiler from computing
    // them once before the loop and holding all three bodies' worth live
    // across it (that spilled 14 registers and cost 6% on one-unit calls).
    int tx = threadIdx.x;
    asm volatile("" : "+v"(tx));
    const int kind = unit_kind(ua.word);
    if constexpr (Wide) {
      if (kind >= kUnitMfma3) {
        rows_unit(p, cx, smem, ua, tx, g);
        continue;
      }
    }
    const int nxt = u < more1 ? (int)u : -1;   // the next unit of the workgroup's own list
    if (kind == kUnitMfma2)
      mfma_unit<2>(p, cx, smem, ua, tx, g, nxt);
    else if (kind == kUnitMfma1)
      mfma_unit<1>(p, cx, smem, ua, tx, g, nxt);
    else {
      // the VALU body's work grows with the rows it is built for: build it
      // for 1, 2 and 4 rows and take the smallest that holds the unit
      const int rows = unit_cand(ua) * cx.G;
      float *lds = reinterpret_cast<float *>(smem);
      if (rows <= 1)
        valu_unit<1>(p, cx, lds, ua, tx, g);
      else if (rows <= 2)
        valu_unit<2>(p, cx, lds, ua, tx, g);
      else
        valu_unit<kMaxValuRows>(p, cx, lds, ua, tx, g);
    }
  }
}

template <typename P>
__global__ void __launch_bounds__(256, 2) chunk_attn(const P p) {
  attend_units<false>(p);
}
// The wide kernel, of which two workgroups share a CU for the whole of a launch,
// keeps to 248 VGPRs (124 of the attribute's units): the 16 left of a SIMD's 512
// are what a wave of the upload kernel needs.  With 251, a round streamed in 8
// MiB chunks beside rounds of 16 x 32768 tokens and 64 rows took 4774 us, as
// every upload waited for a launch to end; with 248 it takes 2575 us (2514 us
// with the copy engine) and the launches the same time.  The narrow kernel
// leaves half of a CU free as a rule, and at 248 takes 380 us instead of 377 for
// 16 x 32768 tokens by chunk.
template <typename P>
__global__ void __launch_bounds__(256, 2) __attribute__((amdgpu_num_vgpr(124))) chunk_attn_wide(const P p) {
  attend_units<true>(p);
}

__global__ void __launch_bounds__(64) clear_counters_kernel(uint32_t *c, int n) {
  for (int i = threadIdx.x; i < n; i += 64) c[i] = 0u;
}

// ---------------------------------------------------------------------------
// Finalize: for every query row (request b, candidate i, head h)
//   * attend the Speculative Frontier: candidate keys j <= i of the same
//     request, causal by absolute position (Sec. 4.2, GPU-resident pass),
//   * merge the split slots the history calls wrote (Eq. 14; slot count per
//     request from the host, unwritten slots are never read),
//   * write O = a / l and LSE = m ln 2 + ln l (Eq. 17).
//
// The kernel is latency-bound, so a row costs one round trip for the kernel
// arguments, one for memory, and few instructions.  Half a wave takes a row;
// lane t of the half holds d = 4t .. 4t+3, so one load instruction brings a
// slot's values of two rows.  The grid is (block of heads, candidate): a
// candidate's word gives its index within the request and the request's slot
// count, so no lane divides and no workgroup is idle.  Every vector load is
// issued before any use: the query, the candidates' K/V (rows past the causal
// mask lie past the buffer's end and read zero), each slot's m and l (lane s
// loads slot s) and every slot's a values (slots past the count read zero).
// Lane sums and maxima go through DPP and permlane swaps, not LDS.  The
// maximum over the frontier scores and the slot maxima gives each term its
// scale 2^(m_s - m*) once (Eq. 14 applied to all pieces together); the slots'
// scales reach all lanes through LDS.  Against one row per wave, with the row
// found by two divisions after a second round trip for the arguments, 64
// ragged requests (269 candidates x 32 heads, 16 slots) went from 11.4 to 8.3
// us, 128 candidates x 64 heads (4 slots) from 10.6 to 7.5 us.
//
// Split = 1: a workgroup's four waves take four pairs of heads.  Split = 4:
// the four waves take a quarter of the slots and of the candidates of one
// pair, and merge (Eq. 14) through LDS.  A CU's L1 delivers 64 bytes a cycle:
// a pair's 32 slots are 32 KiB, 0.25 us of it, and with four pairs on a CU a
// small round waits 1 us for its loads to go out.  The split also quarters a
// wave's instructions, at the price of a barrier and of four times the waves.
// ---------------------------------------------------------------------------
template <int MS, int Split, bool Huge, typename P>
__global__ void __launch_bounds__(256) finalize_kernel(const P p) {
  constexpr int kSlots = MS / Split, kCand = kMaxCand / Split;   // slots and candidates of a wave
  __shared__ __attribute__((aligned(16))) float scale_sh[kWaves][2][32];
  const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  const int half = lane >> 5, t = lane & 31;
  const uint32_t c = blockIdx.y;
  // every kernel argument, read in one scalar round trip
  uint32_t pair = p.cand[c >> 1], cand0 = (uint32_t)p.cand0, g_magic = p.g_magic, g_mask = p.g_mask;
  uint32_t R = (uint32_t)p.st.R, Hq = (uint32_t)p.Hq, kstep = (uint32_t)p.Hkv * kRowBytes;
  float scale_log2 = p.scale_log2;
  const uint16_t *q_ptr = p.q, *k_ptr = p.kc, *v_ptr = p.vc;
  float *m_ptr = p.st.m, *l_ptr = p.st.l, *a_ptr = p.st.a;
  GlobalFloat *out = (GlobalFloat *)p.out, *lse = (GlobalFloat *)p.lse;
  asm volatile("" : "+s"(pair), "+s"(cand0), "+s"(g_magic), "+s"(g_mask), "+s"(R), "+s"(Hq), "+s"(kstep), "+s"(q_ptr),
               "+s"(k_ptr), "+s"(v_ptr), "+s"(m_ptr), "+s"(l_ptr), "+s"(a_ptr), "+s"(out), "+s"(lse), "+s"(scale_log2));
  const uint32_t word = pair >> (16 * (c & 1));
  const uint32_t i = word & 7u, nslot = (word >> 3) & 0xffu;
  const uint32_t cg = cand0 + c;                                   // packed candidate row
  const uint32_t h = Split == 1 ? 2 * (blockIdx.x * kWaves + w) + half : 2 * blockIdx.x + half;
  const uint32_t hc = h < Hq ? h : Hq - 1;                         // lanes past the heads redo the last one
  const uint32_t g = __umulhi(hc, g_magic) + (hc & g_mask);        // hc / G
  const uint32_t row = cg * Hq + hc;
  const uint32_t s0 = Split == 1 ? 0 : w * kSlots, j0 = Split == 1 ? 0 : w * kCand;   // the wave's first slot, candidate

  auto rsrc = [](const void *base, uint32_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), (short)0, (int)bytes, kBufferFlags);
  };
  // resources over the candidates 0..i of the request and all before it
  const __amdgpu_buffer_rsrc_t krs = rsrc(k_ptr, (cg + 1) * kstep), vrs = rsrc(v_ptr, (cg + 1) * kstep);
  const __amdgpu_buffer_rsrc_t qrs = rsrc(q_ptr, R * kRowBytes);
  const uint32_t koff = (cg - i + j0) * kstep + g * kRowBytes + 8 * t;
  const u32x2_t qw = __builtin_bit_cast(u32x2_t, __builtin_amdgcn_raw_buffer_load_b64(qrs, row * kRowBytes + 8 * t, 0, 0));
  u32x2_t kw[kCand], vw[kCand];
#pragma unroll
  for (int j = 0; j < kCand; ++j)
    kw[j] = __builtin_bit_cast(u32x2_t, __builtin_amdgcn_raw_buffer_load_b64(krs, koff + j * kstep, 0, 0));
  // slot s0 + t's m and l in lane t (slots past the count read zero)
  const __amdgpu_buffer_rsrc_t mrs = rsrc(m_ptr, nslot * R * 4), lrs = rsrc(l_ptr, nslot * R * 4);
  const uint32_t moff = ((s0 + t) * R + row) * 4;
  const float m_lane = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(mrs, moff, 0, 0));
  const float l_lane = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(lrs, moff, 0, 0));
  // the a values of this row in the wave's slots; the launch is built for MS
  // >= every request's slot count.  One resource over the request's slots
  // while all slots lie below 2^32 bytes (Huge: one per slot).
  const uint32_t slot_bytes = R * (kHeadDim * 4);
  const uint32_t aoff = row * (kHeadDim * 4) + 16 * t;
  f32x4_t as[kSlots];
  if constexpr (Huge) {
#pragma unroll
    for (int s = 0; s < kSlots; ++s) {
      const __amdgpu_buffer_rsrc_t ars = rsrc(a_ptr + (size_t)s * R * kHeadDim, (uint32_t)s < nslot ? slot_bytes : 0u);
      as[s] = __builtin_bit_cast(f32x4_t, __builtin_amdgcn_raw_buffer_load_b128(ars, aoff, 0, 0));
    }
  } else {
    const __amdgpu_buffer_rsrc_t ars = rsrc(a_ptr, nslot * slot_bytes);
#pragma unroll
    for (int s = 0; s < kSlots; ++s)
      as[s] = __builtin_bit_cast(f32x4_t,
                                 __builtin_amdgcn_raw_buffer_load_b128(ars, aoff + (s0 + s) * slot_bytes, 0, 0));
  }
#pragma unroll
  for (int j = 0; j < kCand; ++j)
    vw[j] = __builtin_bit_cast(u32x2_t, __builtin_amdgcn_raw_buffer_load_b64(vrs, koff + j * kstep, 0, 0));
  __builtin_amdgcn_sched_barrier(0);   // every load is out before the first use

  // frontier scores: the dot products reduced over the half wave as independent chains
  const float q0 = bf16_lo(qw[0]), q1 = bf16_hi(qw[0]), q2 = bf16_lo(qw[1]), q3 = bf16_hi(qw[1]);
  float x[kCand];
#pragma unroll
  for (int j = 0; j < kCand; ++j) {
    float d = fmaf(q1, bf16_hi(kw[j][0]), q0 * bf16_lo(kw[j][0]));
    d = fmaf(q2, bf16_lo(kw[j][1]), d);
    x[j] = row16_sum(fmaf(q3, bf16_hi(kw[j][1]), d));
  }
#pragma unroll
  for (int j = 0; j < kCand; ++j) x[j] = x16_sum(x[j]);
  float m = kNegInf;
#pragma unroll
  for (int j = 0; j < kCand; ++j) {
    x[j] = j0 + j <= i ? x[j] * scale_log2 : kNegInf;
    m = fmaxf(m, x[j]);
  }
  // m* over the frontier and the slots: finite with Split = 1, where every
  // query sees candidate 0; a wave of a split row may hold neither
  const float ms_lane = t < kSlots && s0 + t < nslot ? m_lane : kNegInf;
  m = fmaxf(m, x16_max(row16_max(ms_lane)));
  const float mb = Split > 1 && m == kNegInf ? 0.f : m;
  const float f_lane = exp2_fast(ms_lane - mb);    // slot scale in lane t; 0 past the count
  scale_sh[w][half][t] = f_lane;
  float l = x16_sum(row16_sum(f_lane * l_lane));
  f32x4_t a = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int j = 0; j < kCand; ++j) {
    // past the mask the weight is 2^-inf = 0 and the value row zero
    const float pj = exp2_fast(x[j] - mb);
    l += pj;
    a[0] = fmaf(pj, bf16_lo(vw[j][0]), a[0]);
    a[1] = fmaf(pj, bf16_hi(vw[j][0]), a[1]);
    a[2] = fmaf(pj, bf16_lo(vw[j][1]), a[2]);
    a[3] = fmaf(pj, bf16_hi(vw[j][1]), a[3]);
  }
#pragma unroll
  for (int s = 0; s < kSlots; ++s) {
    const float f = scale_sh[w][half][s];          // the wave's own writes
#pragma unroll
    for (int k = 0; k < 4; ++k) a[k] = fmaf(f, as[s][k], a[k]);
  }
  if constexpr (Split > 1) {
    __shared__ __attribute__((aligned(16))) f32x4_t a_sh[kWaves][64];
    __shared__ float2 ml_sh[kWaves][2];
    a_sh[w][lane] = a;
    if (t == 0) ml_sh[w][half] = make_float2(m, l);
    __syncthreads();
    if (w != 0) return;
    float2 ml[kWaves];
    m = kNegInf;
#pragma unroll
    for (int v = 0; v < kWaves; ++v) {
      ml[v] = ml_sh[v][half];
      m = fmaxf(m, ml[v].x);                       // finite: wave 0 holds candidate 0
    }
    l = 0.f;
    a = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int v = 0; v < kWaves; ++v) {
      const float f = exp2_fast(ml[v].x - m);
      const f32x4_t av = a_sh[v][lane];
      l = fmaf(f, ml[v].y, l);
#pragma unroll
      for (int k = 0; k < 4; ++k) a[k] = fmaf(f, av[k], a[k]);
    }
  }
  if (h >= Hq) return;
  const float inv = 1.0f / l;
  *(GlobalFloat4 *)(out + (size_t)row * kHeadDim + 4 * t) = a * inv;
  if (lse != nullptr && t == 0) lse[row] = m * 0.69314718055994531f + logf(l);
}

// Read-bandwidth probe: workgroup w XOR-folds the 32-bit words of bytes
// [w * share, min((w + 1) * share, bytes)) of buf and stores the fold to
// sink[w].  The loads are the history kernel's: 16 bytes per lane, non-
// temporal, through a range-checked buffer resource (reads past the slice
// return zero, which the fold ignores), eight per lane in flight.
__global__ void __launch_bounds__(256) read_probe_kernel(const uint8_t *buf, uint64_t bytes, uint64_t share,
                                                         uint32_t *sink) {
  const uint64_t first = (uint64_t)blockIdx.x * share;
  const uint32_t n = first >= bytes ? 0u : (uint32_t)(bytes - first < share ? bytes - first : share);
  const __amdgpu_buffer_rsrc_t rs =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t *>(buf) + (first < bytes ? first : 0), (short)0, (int)n,
                                        kBufferFlags);
  constexpr uint32_t kStep = 256 * 16;   // bytes one load instruction of the workgroup reads
  constexpr int kDepth = 8;
  const uint32_t t = threadIdx.x * 16u;
  u32x4_t acc = {0u, 0u, 0u, 0u};
  uint32_t o = 0;
  for (; o + kDepth * kStep <= n; o += kDepth * kStep) {
    u32x4_t v[kDepth];
#pragma unroll
    for (int i = 0; i < kDepth; ++i)
      v[i] = __builtin_bit_cast(u32x4_t, __builtin_amdgcn_raw_buffer_load_b128(rs, o + i * kStep + t, 0, kStreamLoad));
#pragma unroll
    for (int i = 0; i < kDepth; ++i) acc ^= v[i];
  }
  for (; o < n; o += kStep)
    acc ^= __builtin_bit_cast(u32x4_t, __builtin_amdgcn_raw_buffer_load_b128(rs, o + t, 0, kStreamLoad));
  uint32_t x = acc.x ^ acc.y ^ acc.z ^ acc.w;
#pragma unroll
  for (int m = 32; m >= 1; m >>= 1) x ^= (uint32_t)__shfl_xor((int)x, m, 64);
  __shared__ uint32_t part[4];
  if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = x;
  __syncthreads();
  if (threadIdx.x == 0) sink[blockIdx.x] = part[0] ^ part[1] ^ part[2] ^ part[3];
}

// The library's device scratch (see scratch_address).  Each GPU the library
// runs on holds its own copy until the process ends.
__device__ __align__(256) unsigned char scratch[kScratchBytes];

}  // namespace

namespace {

// Kernel arguments of a launch: the header, the units and items in their
// kernel-argument forms (Fat; as UnitRec and Item in the largest class, whose
// tables would pass 64 KB) and the ranges of the workgroups' further units.
// The runtime's argument pool holds about a megabyte and a full one makes the
// next launch wait, so a launch takes the smallest class that holds it: one
// unit per workgroup (per-chunk calls, small rounds) the first, 16 x 32768
// tokens (92 units, 188 items) the second, 64 ragged requests or 32 x 131072
// tokens (170 and 189 units, 407 and 669 items) the third.
template <int MaxUnits, int MaxItems, int MaxWgs, bool Fat>
struct ChunkArgs : ChunkHeader {
  static constexpr int kUnits = MaxUnits, kItems = MaxItems, kWgs = MaxWgs;
  static constexpr bool kFat = Fat;
  uint32_t g_inv;
  uint32_t more[MaxWgs + 1];
  std::conditional_t<Fat, UnitArg, UnitRec> units[MaxUnits];
  std::conditional_t<Fat, ChainItem, Item> items[MaxItems];
};
using ChunkTiny = ChunkArgs<64, 72, 64, true>;              // 4.8 KB
using ChunkSmall = ChunkArgs<128, 192, 128, true>;          // 9 KB
using ChunkMedium = ChunkArgs<256, 704, 256, true>;         // 20 KB
using ChunkMany = ChunkArgs<512, 1024, 256, true>;          // 35 KB
using ChunkLarge = ChunkArgs<kMaxUnits, kMaxItems, kMaxWgs, false>;   // 54 KB

// Workgroups per KV head.  A share that spans requests is several units, and
// where a share is a few tiles, its workgroup spends more time starting the
// second unit than attending it (the units of 24 requests of 33 to 3000 tokens
// ended within 13 us of the launch's start, those that came second at 22).
// Such a launch, of at most kSpreadTiles tiles per share, gives every unit a
// workgroup, up to kSpreadWgs of them: 512 run at once (two per CU), the others
// start as those end.  Rounds back to back, without and with: those 24 requests
// in one call (7 tiles a share, 688 workgroups) 25.6 -> 23.7 us, by chunk 47.4
// -> 36.5 us.  With 32q/8kv and requests of 33 to 1500 tokens, at a limit of 0,
// 512, 640 and 768: 16 requests 17.7, 15.2, 15.2, 15.4 us, 28 requests 21.1,
// 21.4, 21.5, 18.9, 32 requests 27.4, 27.5, 27.5, 21.3; no cohort of 12 to 128
// requests with 2, 4 or 8 KV heads was slower at 768 than below.  Longer shares
// are balanced as they are, and their units are not: 12 requests of 100 to 20000
// tokens 24.1 us as shares, 26.5 us as units, 16 of 1000 to 16000 53.3 and 62.7.
constexpr long kSpreadTiles = 8;
constexpr long kSpreadWgs = 768;
int launch_wgs(const ChunkParams &p) {
  if (p.num_tail > 0 || (long)p.num_units * p.Hkv > kSpreadWgs) return p.num_wgs;
  long tiles = 0;
  for (int u = 0; u < p.num_units; ++u) tiles += p.units[u].ntiles;
  return tiles <= kSpreadTiles * p.num_wgs ? p.num_units : p.num_wgs;
}

template <bool Wide, typename D>
hipError_t launch_chunk_as(const ChunkParams &p, int wgs, hipStream_t s) {
  static thread_local D d;
  static_cast<ChunkHeader &>(d) = p;
  d.g_inv = (65536u + (uint32_t)p.G - 1) / (uint32_t)p.G;
  if constexpr (D::kFat) {
    for (int u = 0; u < p.num_units; ++u) {
      const UnitRec &r = p.units[u];
      UnitArg &a = d.units[u];
      a.word = r.word;
      if (unit_nit(r.word) == 0) continue;
      const Item &it = p.items[unit_i0(r.word)];
      const size_t first = (size_t)it.tok_begin * p.tok_stride;
      a.k = p.k[it.chunk] + first;
      a.v = p.v[it.chunk] + first;
      a.hs = p.head_stride[it.chunk];
      a.ntiles = r.ntiles;
      a.tok_count = it.tok_count;
      a.q_row0 = r.q_row0;
      a.cand_slot = pack_cand_slot(it);
    }
    for (int i = 0; i < p.num_items; ++i)
      d.items[i] = {(uint32_t)p.items[i].tok_begin, (uint32_t)p.items[i].tok_count | (uint32_t)p.items[i].chunk << 24};
  } else {
    std::memcpy(d.units, p.units, sizeof(UnitRec) * p.num_units);
    std::memcpy(d.items, p.items, sizeof(Item) * p.num_items);
  }
  if (wgs == p.num_wgs) {
    std::memcpy(d.more, p.more, sizeof(uint32_t) * (wgs + 1));
  } else {                            // a workgroup per unit: none has a further one
    for (int w = 0; w <= wgs; ++w) d.more[w] = (uint32_t)p.num_units;
  }
  // the heads are the fast grid dimension, or the workgroups are
  const dim3 grid = p.heads_fast ? dim3(p.Hkv, wgs, 1) : dim3(1, wgs, p.Hkv);
  if constexpr (Wide)
    hipLaunchKernelGGL(chunk_attn_wide<D>, grid, dim3(256), 0, s, d);
  else
    hipLaunchKernelGGL(chunk_attn<D>, grid, dim3(256), 0, s, d);
  return hipGetLastError();
}

template <bool Wide>
hipError_t launch_chunk_sized(const ChunkParams &p, hipStream_t s) {
  const int wgs = launch_wgs(p);
  auto fits = [&](int units, int items, int max_wgs) {
    return p.num_units <= units && p.num_items <= items && wgs <= max_wgs;
  };
  if (fits(ChunkTiny::kUnits, ChunkTiny::kItems, ChunkTiny::kWgs)) return launch_chunk_as<Wide, ChunkTiny>(p, wgs, s);
  if (fits(ChunkSmall::kUnits, ChunkSmall::kItems, ChunkSmall::kWgs)) return launch_chunk_as<Wide, ChunkSmall>(p, wgs, s);
  if (fits(ChunkMedium::kUnits, ChunkMedium::kItems, ChunkMedium::kWgs)) return launch_chunk_as<Wide, ChunkMedium>(p, wgs, s);
  if (fits(ChunkMany::kUnits, ChunkMany::kItems, ChunkMany::kWgs)) return launch_chunk_as<Wide, ChunkMany>(p, wgs, s);
  return launch_chunk_as<Wide, ChunkLarge>(p, wgs, s);
}

}  // namespace

hipError_t launch_chunk(const ChunkParams &p, hipStream_t s) {
  // a launch with any unit of more than two 16-row blocks runs on the wide kernel
  for (int u = 0; u < p.num_units; ++u)
    if (unit_kind(p.units[u].word) >= kUnitMfma3) return launch_chunk_sized<true>(p, s);
  return launch_chunk_sized<false>(p, s);
}

hipError_t launch_clear_counters(uint32_t *counters, int n, hipStream_t s) {
  hipLaunchKernelGGL(clear_counters_kernel, dim3(1), dim3(64), 0, s, counters, n);
  return hipGetLastError();
}
namespace {

// What finalize_kernel reads: candidate c's word holds its index within its
// request (3 bits) and the request's slot count (8 bits), two per dword.
template <int MaxCand>
struct FinalArgs : FinalHeader {
  static constexpr int kCand = MaxCand;
  int32_t cand0;      // packed candidate row of the launch's first candidate
  uint32_t g_magic;   // h / G = mulhi(h, g_magic) + (h & g_mask): ceil(2^32 / G) and 0, or 0 and ~0 for G = 1
  uint32_t g_mask;
  uint32_t cand[MaxCand / 2];
};
using FinalSmall = FinalArgs<128>;
using FinalLarge = FinalArgs<4096>;
static_assert(kMaxCand <= 8 && kNumSlots < 256 && kNumSlots <= 4 * 32 && kBaseSlots == 32, "candidate word fields, a lane per slot of a wave");

template <int MS, int Split, bool Huge, typename D>
hipError_t launch_finalize_as(const D &d, int n, hipStream_t s) {
  constexpr int kHeads = Split == 1 ? 2 * kWaves : 2;   // heads per workgroup
  hipLaunchKernelGGL((finalize_kernel<MS, Split, Huge, D>), dim3((d.Hq + kHeads - 1) / kHeads, n), dim3(256), 0, s, d);
  return hipGetLastError();
}

// Built for 8, 16 or 32 slots: each slot a row may read costs the wave a load
// and four registers, so a launch takes the smallest build that holds every
// request's slot count.
template <int Split, typename D>
hipError_t launch_finalize_split(const D &d, int n, int slots, hipStream_t s) {
  if (slots <= 8) return launch_finalize_as<8, Split, false>(d, n, s);
  if (slots <= 16) return launch_finalize_as<16, Split, false>(d, n, s);
  return launch_finalize_as<kBaseSlots, Split, false>(d, n, s);
}

// Rows are split over a workgroup's waves while that takes at most this many
// workgroups (4 per CU): below, the chip is not full and the shorter chain
// wins; above, four times the waves cost more than it.  Rounds back to back,
// split against not: 1 x 16384 tokens (80 workgroups) 19.6 against 20.8 us,
// 6 candidates x 32 heads (96) 32.3 against 33.3 us, 8 x 8191 (32) 45.5
// against 45.9 us, 4 x 16384 x 48 heads (768) 55.8 against 55.9 us; 24 ragged
// requests (1888) 27.3 against 27.1 us, and 128 candidates x 64 heads (4096)
// 8.9 against 7.5 us for the launch alone.
constexpr long kSplitWgs = 1024;

template <typename D>
hipError_t launch_finalize_cand(const D &d, int n, int slots, hipStream_t s) {
  // more slots than a half wave has lanes are always split; they come with at
  // most 4 requests, so at most 32 candidates, and never with the large table
  if constexpr (D::kCand <= FinalSmall::kCand) {
    if (slots > 64) return launch_finalize_as<kNumSlots, 4, false>(d, n, s);
    if (slots > kBaseSlots) return launch_finalize_as<64, 4, false>(d, n, s);
  }
  if (slots > kBaseSlots) return hipErrorInvalidValue;
  if ((uint64_t)kBaseSlots * (uint32_t)d.st.R * (kHeadDim * 4) >= (uint64_t(1) << 32))
    return launch_finalize_as<kBaseSlots, 1, true>(d, n, s);
  if constexpr (D::kCand <= FinalSmall::kCand)
    if ((long)n * ((d.Hq + 1) / 2) <= kSplitWgs) return launch_finalize_split<4>(d, n, slots, s);
  return launch_finalize_split<1>(d, n, slots, s);
}

}  // namespace

hipError_t launch_finalize(const FinalParams &p, hipStream_t s) {
  // Candidates in packed order, at most FinalLarge::kCand per launch.  The
  // words are gathered here; a launch passes the small table when it fits.
  static thread_local FinalSmall ds;
  static thread_local FinalLarge dl;
  // h * (G ceil(2^32 / G) - 2^32) < 2^23 * 64 < 2^32, so mulhi gives h / G exactly
  const uint32_t magic = p.G > 1 ? (uint32_t)(((uint64_t(1) << 32) + p.G - 1) / p.G) : 0u;
  int n = 0, slots = 0, c0 = p.num_items > 0 ? p.items[0].q_row0 : 0;
  auto flush = [&]() {
    if (n == 0) return hipSuccess;
    hipError_t e;
    if (n <= FinalSmall::kCand) {
      static_cast<FinalHeader &>(ds) = p;
      ds.cand0 = c0;
      ds.g_magic = magic;
      ds.g_mask = p.G > 1 ? 0u : ~0u;
      std::memcpy(ds.cand, dl.cand, sizeof(uint32_t) * ((n + 1) / 2));
      e = launch_finalize_cand(ds, n, slots, s);
    } else {
      static_cast<FinalHeader &>(dl) = p;
      dl.cand0 = c0;
      dl.g_magic = magic;
      dl.g_mask = p.G > 1 ? 0u : ~0u;
      e = launch_finalize_cand(dl, n, slots, s);
    }
    c0 += n;
    n = slots = 0;
    return e;
  };
  for (int b = 0; b < p.num_items; ++b) {
    const Item &it = p.items[b];
    for (int i = 0; i < it.n_cand; ++i) {
      if (n == FinalLarge::kCand) {
        const hipError_t e = flush();
        if (e != hipSuccess) return e;
      }
      const uint32_t word = (uint32_t)i | ((uint32_t)it.tok_count << 3);
      if (n & 1)
        dl.cand[n >> 1] |= word << 16;
      else
        dl.cand[n >> 1] = word;
      ++n;
      slots = slots > it.tok_count ? slots : it.tok_count;
    }
  }
  return flush();
}

hipError_t launch_read_probe(const void *buf, uint64_t bytes, uint64_t share, uint32_t *sink, int workgroups,
                             hipStream_t s) {
  hipLaunchKernelGGL(read_probe_kernel, dim3(workgroups), dim3(256), 0, s, static_cast<const uint8_t *>(buf), bytes,
                     share, sink);
  return hipGetLastError();
}

hipError_t scratch_address(void **ptr) {
  // One lookup per device, with that device current; the array's name is a
  // host-side stand-in, so only the looked-up address may reach a kernel.
  static std::mutex mu;
  static void *addr[kMaxDevices] = {};
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(mu);
  if (addr[dev] == nullptr) {
    void *a = nullptr;
    e = hipGetSymbolAddress(&a, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (a == nullptr) return hipErrorInvalidSymbol;
    addr[dev] = a;
  }
  *ptr = addr[dev];
  return hipSuccess;
}

}  // namespace ss
