// Device helpers shared by the PHSA kernels (gfx950 / CDNA4, wave64).
#pragma once

#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#define PHSA_HD __device__ __forceinline__
#include "unit_map.h"

namespace phsa {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint16_t bf16_t;  // storage type of bfloat16 values
// 16 raw bytes as a native vector: loads and stores of it are single values
// (a uint4 struct copy can be lowered to a memcpy through scratch memory)
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));

constexpr int kWave = 64;
constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;

__device__ __forceinline__ float bf16_to_f32(bf16_t x) {
  return __uint_as_float(static_cast<uint32_t>(x) << 16);
}

// float -> bfloat16, round to nearest even (the gfx950 conversion instruction).
__device__ __forceinline__ bf16_t f32_to_bf16(float f) { return __builtin_bit_cast(bf16_t, (__bf16)f); }

template <typename T> __device__ __forceinline__ float to_f32(T x);
template <> __device__ __forceinline__ float to_f32<float>(float x) { return x; }
template <> __device__ __forceinline__ float to_f32<bf16_t>(bf16_t x) { return bf16_to_f32(x); }

template <typename T> __device__ __forceinline__ T from_f32(float x);
template <> __device__ __forceinline__ float from_f32<float>(float x) { return x; }
template <> __device__ __forceinline__ bf16_t from_f32<bf16_t>(float x) { return f32_to_bf16(x); }

// 16x16x32 bf16 MFMA, fp32 accumulate.  Operand layout used throughout:
//   A (16 x 32, row-major M x K): lane l holds A[l % 16][8 * (l / 16) + 0..7]
//   B (32 x 16, K x N):           lane l holds B[8 * (l / 16) + 0..7][l % 16]
//   C (16 x 16):                  lane l holds C[4 * (l / 16) + 0..3][l % 16]
// A and B always use the same K assignment, so the contraction is exact
// whatever order the unit sums K in.
__device__ __forceinline__ f32x4 mfma16x16x32(const bf16x8 &a, const bf16x8 &b, const f32x4 &c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

// No 64-bit shift here takes its amount from a vector register: one
// (v_lshlrev_b64 / v_lshrrev_b64) whose amount sits in the last register of the
// wave's allocation takes it from v0 instead on this GPU (cache_append pooled
// wrong keys, now and then, when its shift came to lie in v71 of 72), and the
// register is the compiler's choice.  Per-lane bits of wave masks go through the
// helpers below; a test looks for such shifts in the built library.

// Bit j of a 64-bit mask, j differing between lanes.  The empty asm hides that
// the halves are one value, which the compiler would shift by (j & 32) again.
__device__ __forceinline__ bool lane_bit(uint64_t mask, int j) {
  uint32_t hi = (uint32_t)(mask >> 32);
  asm("" : "+v"(hi));
  return ((j & 32 ? hi : (uint32_t)mask) >> (j & 31)) & 1u;
}

// Set bits of a mask below this lane.
__device__ __forceinline__ int bits_below(uint64_t m) {
  return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

// The 16 bits of a wave mask that belong to quarter-wave q4 (this lane's).
__device__ __forceinline__ uint32_t quarter_bits(uint64_t m, int q4) {
  uint32_t hi = (uint32_t)(m >> 32);
  asm("" : "+v"(hi));
  return ((q4 & 2 ? hi : (uint32_t)m) >> (16 * (q4 & 1))) & 0xffffu;
}

// 16-byte load of data that is read once (bypasses cache retention).
__device__ __forceinline__ uint4 ld_stream16(const bf16_t *p) {
  const uint32_t *q = reinterpret_cast<const uint32_t *>(p);
  return make_uint4(__builtin_nontemporal_load(q), __builtin_nontemporal_load(q + 1),
                    __builtin_nontemporal_load(q + 2), __builtin_nontemporal_load(q + 3));
}

typedef float f32x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ bf16x8 load_bf16x8(const bf16_t *p) {  // 16-byte aligned
  return __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4 *>(p));
}

__device__ __forceinline__ float wave_max(float v) {
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) v = fmaxf(v, __shfl_xor(v, o, 64));
  return v;
}

// Cross-row lane exchange with the gfx950 permlane swaps (VALU, no LDS
// round trip).  v_permlane16_swap exchanges the odd 16-lane rows of its first
// operand with the even rows of its second, v_permlane32_swap the upper half of
// the first with the lower half of the second; with x in both operands every
// lane ends up holding x of itself and of lane l ^ 16 (resp. l ^ 32), in an
// order that differs between the two lanes.  Commutative reductions of the
// pair are therefore equal in both lanes.
__device__ __forceinline__ float max_xor16(float x) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __builtin_elementwise_maximum(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float max_xor32(float x) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __builtin_elementwise_maximum(__uint_as_float(r[0]), __uint_as_float(r[1]));
}

typedef short v4i16 __attribute__((ext_vector_type(4)));
typedef short v8i16 __attribute__((ext_vector_type(8)));
typedef __attribute__((address_space(3))) v4i16 lds_v4i16_t;

// Column reads from a row-major bf16 LDS tile X (row pitch `pitch` elements)
// with the gfx950 transposing LDS load (ds_read_b64_tr_b16).  Within each
// 16-lane group the instruction hands lane j element (j % 4) of the 8 bytes
// addressed by lane 4e + j / 4, e = 0..3; giving lane i the address of
// X[r0 + i / 4][c0 + 4 (i % 4)] therefore delivers X[r0 + e][c0 + j] to lane j.
// r0 and c0 may differ between the four groups.  Rows must be 8-byte aligned.
__device__ __forceinline__ v4i16 lds_col4(const bf16_t *X, int pitch, int r0, int c0, int l16) {
  const bf16_t *p = X + (r0 + (l16 >> 2)) * pitch + c0 + 4 * (l16 & 3);
  return __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4i16_t *)p);
}

// 8-element column fragment: lane j gets X[r0 + 0..3][c0 + j] then X[r1 + 0..3][c0 + j].
__device__ __forceinline__ bf16x8 lds_col8(const bf16_t *X, int pitch, int r0, int r1, int c0, int l16) {
  const v4i16 a = lds_col4(X, pitch, r0, c0, l16);
  const v4i16 b = lds_col4(X, pitch, r1, c0, l16);
  const v8i16 c = {a[0], a[1], a[2], a[3], b[0], b[1], b[2], b[3]};
  return __builtin_bit_cast(bf16x8, c);
}

// The partials of one (b, g, query row) for the per-row merges.  Half a wave
// owns a row: lane l32 reads the list positions of slots l32 and l32 + 32
// (-1 marks a slot without a partial).  slots() is a wave-uniform bound on the
// highest used slot of either half, and pos(s) gives each lane its own half's
// position of slot s (every lane must call it, s uniform).
struct RowSlots {
  int pa, pb;
  uint64_t valid;  // this half's slots that hold a partial
  uint32_t lo, hi; // slots < 32 / >= 32 used by either half
  __device__ __forceinline__ RowSlots(const int32_t *pmap, int64_t base, bool row_ok, int ksel, int half, int l32)
      : RowSlots((row_ok && l32 < ksel) ? pmap[base + l32] : -1, (row_ok && l32 + 32 < ksel) ? pmap[base + l32 + 32] : -1,
                 half) {}
  RowSlots() = default;
  // from the two positions this lane loaded (-1 for none), e.g. one row ahead
  __device__ __forceinline__ RowSlots(int pa_, int pb_, int half) : pa(pa_), pb(pb_) {
    const uint64_t ba = __ballot(pa >= 0), bb = __ballot(pb >= 0);
    valid = ((ba >> (32 * half)) & 0xffffffffull) | (((bb >> (32 * half)) & 0xffffffffull) << 32);
    lo = (uint32_t)ba | (uint32_t)(ba >> 32);
    hi = (uint32_t)bb | (uint32_t)(bb >> 32);
  }
  __device__ __forceinline__ int slots() const { return hi ? 64 - __clz(hi) : 32 - __clz(lo); }
  __device__ __forceinline__ int pos(int s, int half) const {
    const int src = half * 32 + (s & 31);
    return s < 32 ? __shfl(pa, src, 64) : __shfl(pb, src, 64);
  }
};

// Folds one partial of a row into a running merge (M, L, a) of Eq. 10-11:
// q = (m, l) in log2 units, raw = 8 bf16 features of its unnormalised O.  The
// maximum moves to the larger m and both sides are rescaled; a partial with
// m = -inf (no key) is skipped.
__device__ __forceinline__ void fold_partial(float &M, float &L, float (&a)[8], float2 q, const uint4 &raw) {
  if (q.x == -INFINITY) return;
  const float mn = fmaxf(M, q.x);
  const float sc = __builtin_amdgcn_exp2f(M - mn), w = __builtin_amdgcn_exp2f(q.x - mn);
  L = fmaf(w, q.y, L * sc);
  const bf16_t *pv = reinterpret_cast<const bf16_t *>(&raw);
#pragma unroll
  for (int j = 0; j < 8; ++j) a[j] = fmaf(w, bf16_to_f32(pv[j]), a[j] * sc);
  M = mn;
}

// The dispatcher hands workgroups to the 8 XCDs (each with its own L2) in
// turn by linear id.  Returns the work item of linear id `lin` (of n) such that
// each XCD takes one contiguous run of items: neighbouring items, which read
// the same tiles, then share an L2.  A bijection of 0..n-1.
__device__ __forceinline__ int xcd_item(int lin, int n) {
  const int x = lin & 7, j = lin >> 3;
  int off = 0;
  for (int y = 0; y < x; ++y) off += (n - y + 7) >> 3;  // items of the XCDs before
  return off + j;
}

// The exponentials of the softmax weights use the hardware 2^x instruction
// (__builtin_amdgcn_exp2f): its arguments are <= 0 or a bounded offset, and it
// flushes results below 2^-126, which are negligible against a sum >= 1.

// Workgroup barrier that orders LDS accesses only.  __syncthreads() also
// fences global and private memory, and values held in registers across it
// (loads issued before the barrier, stored to LDS after it) can then be sent
// through scratch memory; this barrier leaves them in registers.
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Orders a wave's LDS writes before its following LDS reads of other lanes'
// data.  A wave's LDS instructions execute in order, so this only has to stop
// the compiler from moving the accesses across it.
__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// 64-row bf16 tiles in LDS without padding.  Row r holds D elements; its
// 16-byte chunk c sits at chunk position c ^ (r mod D / 8), which spreads the
// rows that one 16-lane group reads (row reads of MFMA operands and the
// transposing reads) over the LDS banks.  Element offset of (r, e):
template <int D>
__device__ __forceinline__ int swz(int r, int e) {
  return r * D + ((((e >> 3) ^ r) & (D / 8 - 1)) << 3) + (e & 7);
}

// 8-element column fragment of a swizzled tile (the layout of lds_col8).
template <int D>
__device__ __forceinline__ bf16x8 lds_col8_sw(const bf16_t *X, int r0, int r1, int c0, int l16) {
  const int e = c0 + 4 * (l16 & 3);
  const v4i16 a = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4i16_t *)(X + swz<D>(r0 + (l16 >> 2), e)));
  const v4i16 b = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4i16_t *)(X + swz<D>(r1 + (l16 >> 2), e)));
  const v8i16 c = {a[0], a[1], a[2], a[3], b[0], b[1], b[2], b[3]};
  return __builtin_bit_cast(bf16x8, c);
}

typedef __attribute__((address_space(3))) void lds_void_t;

// Copies a 64-row tile from global memory straight into LDS in the swizzled
// layout (global_load_lds: no registers, no LDS store instructions).  Each of
// the 4 waves issues D / 32 one-kilobyte copies; lane l of a copy lands at
// byte 16 l of it and fetches the chunk that belongs there.  Row r starts at
// element row_off(r) of src.  The copies count in vmcnt: each wave waits for
// vmcnt(0) and the workgroup then passes a barrier before the tile is read.
// wave must be wave-uniform (it selects the LDS destination).
template <int D, typename RowOff>
__device__ __forceinline__ void tile_dma(const bf16_t *src, RowOff row_off, bf16_t *dst, int wave, int lane) {
  constexpr int VPR = D / 8, RPI = 64 / VPR, NI = 64 / RPI / 4;
#pragma unroll
  for (int v = 0; v < NI; ++v) {
    const int blk = wave * NI + v, r = blk * RPI + lane / VPR, c = (lane % VPR) ^ (r & (VPR - 1));
    __builtin_amdgcn_global_load_lds(src + row_off(r) + c * 8, (lds_void_t *)(dst + blk * RPI * D), 16, 0, 0);
  }
}

// The same tile by way of registers, for a caller's tensor that does not start at
// a multiple of 16 bytes, as the copies straight into LDS want it (ordinary loads
// take any start of an element).
template <int D, typename RowOff>
__device__ __forceinline__ void tile_copy(const bf16_t *src, RowOff row_off, bf16_t *dst, int wave, int lane) {
  constexpr int VPR = D / 8, RPI = 64 / VPR, NI = 64 / RPI / 4;
#pragma unroll 1
  for (int v = 0; v < NI; ++v) {
    const int blk = wave * NI + v, r = blk * RPI + lane / VPR, c = (lane % VPR) ^ (r & (VPR - 1));
    *reinterpret_cast<u32x4 *>(dst + blk * RPI * D + lane * 8) = *reinterpret_cast<const u32x4 *>(src + row_off(r) + c * 8);
  }
}

// Waits until this wave's tile_dma copies have landed in LDS (vmcnt(0); the
// other counters are left alone).
__device__ __forceinline__ void dma_wait() { __builtin_amdgcn_s_waitcnt(0x0f70); }

// Waits for this wave's LDS reads and writes (lgkmcnt(0)).
__device__ __forceinline__ void lds_wait() { __builtin_amdgcn_s_waitcnt(0xc07f); }

// Packs two 4-element float groups into a bf16 MFMA operand (elements 0..3,
// then 4..7), rounding to nearest even with the packed conversion instruction.
typedef float f32x8 __attribute__((ext_vector_type(8)));
__device__ __forceinline__ bf16x8 pack_bf16x8(const f32x4 &a, const f32x4 &b) {
  const f32x8 c = {a[0], a[1], a[2], a[3], b[0], b[1], b[2], b[3]};
  return __builtin_convertvector(c, bf16x8);
}

// Eight consecutive features v of one representative (feature 8 (x mod D / 8) of
// representative x / (D / 8)) split into bf16 hi + lo (hi + lo = v to about 2^-17
// relative), with the Euclidean norms of the representative's parts; D / 8
// consecutive lanes hold one representative and all call this (ok: store).
template <int D>
__device__ __forceinline__ void split_row8(const float (&v)[8], int64_t x, bool ok, bf16_t *Mh, bf16_t *Ml,
                                           float2 *Mnorm) {
  constexpr int TPR = D / 8;
  bf16_t hi[8], lo[8];
  float sh = 0.f, sl = 0.f;
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    hi[e] = f32_to_bf16(v[e]);
    const float h = bf16_to_f32(hi[e]);
    lo[e] = f32_to_bf16(v[e] - h);
    const float l = bf16_to_f32(lo[e]);
    sh = fmaf(h, h, sh);
    sl = fmaf(l, l, sl);
  }
#pragma unroll
  for (int o = 1; o < TPR; o <<= 1) {
    sh += __shfl_xor(sh, o, 64);
    sl += __shfl_xor(sl, o, 64);
  }
  if (!ok) return;
  reinterpret_cast<uint4 *>(Mh)[x] = *reinterpret_cast<const uint4 *>(hi);
  reinterpret_cast<uint4 *>(Ml)[x] = *reinterpret_cast<const uint4 *>(lo);
  if (x % TPR == 0) Mnorm[x / TPR] = make_float2(sqrtf(sh), sqrtf(sl));
}

}  // namespace phsa
