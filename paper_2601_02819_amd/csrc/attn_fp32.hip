// Sparse attention forward/backward for float32 tensors (Eq. 10-11).
//
// float32 inputs are held to a 1e-4 tolerance, which bf16 matrix cores cannot
// meet, so everything here is float32: vector ALUs for the row-major kernels,
// the float32 matrix instruction (16x16x4) for dK/dV.
//
//   forward, dQ : one workgroup per (b, g, query row), its waves sharing the
//                 row's slots.  The G heads of the group meet every key
//                 together, so K and V are read once per group.  A wave reads a
//                 block with 16-byte loads (D / 4 lanes per key), the lanes of a
//                 key reduce its dot products with DPP moves, and P V / dS K
//                 need no exchange: a lane keeps its 4 features.
//   dK/dV       : key-block-major over the inverted selection index, one work
//                 unit (block, part of its list) per workgroup, sums in
//                 registers; lists of several units meet in dkv_sum_fp32_kernel.
//                 No atomics: the result does not depend on timing.
//
// The row-major kernels are bound by their key loads from the caches and the
// dot products' VALU work; in small problems every launch is its own latency.
// At 1k tokens, 2 heads of dim 64, 4 blocks (events around each launch) the
// forward takes 14 us (45 when a lane owned a key and read its row alone), the
// backward's index, dK/dV, sums and dQ 24 + 20 + 8 + 15 us (326 with float32
// atomics per (row, key, feature)).
#include <math.h>

#include <algorithm>
#include <type_traits>

#include "common.h"
#include "launch.h"

namespace phsa {

__device__ __forceinline__ bool slot_ok_f(int t, int cur, int T) { return t >= 0 && t <= cur && t < T; }

// Sum over the CPR (16 or 32) consecutive lanes that share a key, every lane
// getting it: DPP moves within the 16-lane rows, a row swap between them.
template <int CTRL>
__device__ __forceinline__ float add_dpp(float a) {
  return a + __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, a), CTRL, 0xF, 0xF, true));
}
template <int CPR>
__device__ __forceinline__ float key_sum(float a) {
  static_assert(CPR == 16 || CPR == 32, "key rows span 16 or 32 lanes");
  a = add_dpp<0xB1>(a);   // quad_perm [1, 0, 3, 2]
  a = add_dpp<0x4E>(a);   // quad_perm [2, 3, 0, 1]
  a = add_dpp<0x141>(a);  // row_half_mirror
  a = add_dpp<0x140>(a);  // row_mirror
  if constexpr (CPR == 32) {
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(a), false, false);
    a = __uint_as_float(r[0]) + __uint_as_float(r[1]);
  }
  return a;
}

// The row of a workgroup and the walk over its slots and keys, shared by the
// forward and dQ.  Wave w takes slots w, w + NW, ...; lane = (sub, ch) holds
// features 4 ch .. 4 ch + 3 of every KPI-th key.  body(ok[], kr[], vr[]) gets NI
// key rows per lane at a time; ok marks keys the row may see.
template <int D, int NI, int NW>
struct RowWalk {
  static constexpr int CPR = D / 4, KPI = 64 / CPR, KG = NI * KPI;
  int i, bg, b, g, lane, wave, ch, sub, pos;
  __device__ __forceinline__ explicit RowWalk(const Geom &gm) {
    i = blockIdx.x;
    bg = blockIdx.y;
    b = bg / gm.Hkv;
    g = bg - b * gm.Hkv;
    lane = threadIdx.x & 63;
    wave = threadIdx.x >> 6;
    ch = lane % CPR;
    sub = lane / CPR;
    pos = gm.q_pos0 + i;
  }
  __device__ __forceinline__ int64_t qrow(const Geom &gm, int h) const {
    return (((int64_t)b * gm.Lq + i) * gm.Hq + g * (gm.Hq / gm.Hkv) + h) * D;
  }
  template <typename F>
  __device__ __forceinline__ void run(const float *K, const float *V, const int32_t *sel, const Geom &gm, F body) const {
    const int cur = pos / gm.m, sj = wave + NW * lane;
    const int tl = sj < gm.ksel ? sel[((int64_t)bg * gm.Lq + i) * gm.ksel + sj] : -1;
    for (uint64_t todo = __ballot(slot_ok_f(tl, cur, gm.T)); todo; todo &= todo - 1) {
      const int t = __builtin_amdgcn_readlane(tl, __builtin_ctzll(todo));
      const int key0 = t * gm.m;
      for (int k0 = 0; k0 < gm.m && key0 + k0 <= pos; k0 += KG) {
        f32x4 kr[NI], vr[NI];
        bool ok[NI];
#pragma unroll
        for (int n = 0; n < NI; ++n) {
          const int k = k0 + n * KPI + sub;
          ok[n] = k < gm.m && key0 + k <= pos;
          const int64_t src = (((int64_t)b * gm.Lk + min(key0 + k, pos)) * gm.Hkv + g) * D + ch * 4;
          kr[n] = *reinterpret_cast<const f32x4 *>(K + src);
          vr[n] = *reinterpret_cast<const f32x4 *>(V + src);
        }
        body(ok, kr, vr);
      }
    }
  }
};

__device__ __forceinline__ float dot4(const f32x4 &a, const f32x4 &b) {
  return fmaf(a[0], b[0], fmaf(a[1], b[1], fmaf(a[2], b[2], a[3] * b[3])));
}

template <int D, int G, int NI, int NW>
__global__ __launch_bounds__(64 * NW) void attn_fwd_fp32_kernel(const float *__restrict__ Q,
                                                                const float *__restrict__ K,
                                                                const float *__restrict__ V,
                                                                const int32_t *__restrict__ sel,
                                                                float *__restrict__ O, float *__restrict__ LSE,
                                                                Geom gm) {
  using W = RowWalk<D, NI, NW>;
  const W w(gm);
  __shared__ float wm[NW][G], wl[NW][G];
  __shared__ __attribute__((aligned(16))) float wo[NW][G][D];
  const float sl2 = gm.scale * kLog2e;
  f32x4 q[G], o[G];
  float mrun[G], lrun[G];
#pragma unroll
  for (int h = 0; h < G; ++h) {
    q[h] = *reinterpret_cast<const f32x4 *>(Q + w.qrow(gm, h) + w.ch * 4);
    o[h] = f32x4{0.f, 0.f, 0.f, 0.f};
    mrun[h] = -INFINITY;
    lrun[h] = 0.f;
  }
  w.run(K, V, sel, gm, [&](const bool (&ok)[NI], const f32x4 (&kr)[NI], const f32x4 (&vr)[NI]) {
#pragma unroll
    for (int h = 0; h < G; ++h) {
      float sc[NI], mn = mrun[h];
#pragma unroll
      for (int n = 0; n < NI; ++n) {
        const float s = key_sum<W::CPR>(dot4(q[h], kr[n])) * sl2;
        sc[n] = ok[n] ? s : -INFINITY;
        mn = fmaxf(mn, sc[n]);
      }
      // each key group of lanes keeps a maximum of its own (mn is the same in
      // the CPR lanes of a key); they meet at the end
      const float f = mn == -INFINITY ? 1.f : __builtin_amdgcn_exp2f(mrun[h] - mn);  // 2^-inf = 0 at the first key
      const float mz = mn == -INFINITY ? 0.f : mn;  // every score -inf so far (an infinite key): weight 0, not NaN
      mrun[h] = mn;
      lrun[h] *= f;
      o[h] *= f;
#pragma unroll
      for (int n = 0; n < NI; ++n) {
        const float p = ok[n] ? __builtin_amdgcn_exp2f(sc[n] - mz) : 0.f;
        lrun[h] += p;
#pragma unroll
        for (int e = 0; e < 4; ++e) o[h][e] = ok[n] ? fmaf(p, vr[n][e], o[h][e]) : o[h][e];
      }
    }
  });
  // the key groups of a wave, then the waves
#pragma unroll
  for (int h = 0; h < G; ++h) {
#pragma unroll
    for (int x = W::CPR; x < 64; x <<= 1) {
      const float om = __shfl_xor(mrun[h], x, 64), ol = __shfl_xor(lrun[h], x, 64);
      const float mn = fmaxf(mrun[h], om);
      const float fa = mn == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(mrun[h] - mn);
      const float fb = mn == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(om - mn);
      lrun[h] = fmaf(lrun[h], fa, ol * fb);
#pragma unroll
      for (int e = 0; e < 4; ++e) o[h][e] = fmaf(o[h][e], fa, __shfl_xor(o[h][e], x, 64) * fb);
      mrun[h] = mn;
    }
    if (w.sub == 0) *reinterpret_cast<f32x4 *>(&wo[w.wave][h][w.ch * 4]) = o[h];
    if (w.lane == 0) {
      wm[w.wave][h] = mrun[h];
      wl[w.wave][h] = lrun[h];
    }
  }
  __syncthreads();
  for (int x = threadIdx.x; x < G * D; x += 64 * NW) {
    const int h = x / D, c = x - h * D;
    float M = -INFINITY, L = 0.f, acc = 0.f;
#pragma unroll
    for (int v = 0; v < NW; ++v) M = fmaxf(M, wm[v][h]);
#pragma unroll
    for (int v = 0; v < NW; ++v) {
      const float f = wm[v][h] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(wm[v][h] - M);
      L = fmaf(f, wl[v][h], L);
      acc = fmaf(f, wo[v][h][c], acc);
    }
    // NaN beside a NaN or +inf score; 0 where no score was a number above -inf
    O[w.qrow(gm, h) + c] = L > 0.f ? acc / L : M == -INFINITY ? 0.f : acc * 0.f;
    if (c == 0)
      LSE[((int64_t)w.b * gm.Hq + w.g * G + h) * gm.Lq + w.i] = L > 0.f ? (M + log2f(L)) * kLn2 : -INFINITY;
  }
}

template <int D, int G, int NI, int NW>
__global__ __launch_bounds__(64 * NW) void attn_dq_fp32_kernel(const float *__restrict__ Q, const float *__restrict__ K,
                                                               const float *__restrict__ V,
                                                               const float *__restrict__ dO,
                                                               const float *__restrict__ LSE,
                                                               const float *__restrict__ Dvec,
                                                               const int32_t *__restrict__ sel,
                                                               float *__restrict__ dQ, Geom gm) {
  using W = RowWalk<D, NI, NW>;
  const W w(gm);
  __shared__ __attribute__((aligned(16))) float wo[NW][G][D];
  const float sl2 = gm.scale * kLog2e;
  f32x4 q[G], dd[G], dq[G];
  float lse[G], dv[G];
#pragma unroll
  for (int h = 0; h < G; ++h) {
    q[h] = *reinterpret_cast<const f32x4 *>(Q + w.qrow(gm, h) + w.ch * 4);
    dd[h] = *reinterpret_cast<const f32x4 *>(dO + w.qrow(gm, h) + w.ch * 4);
    dq[h] = f32x4{0.f, 0.f, 0.f, 0.f};
    lse[h] = LSE[((int64_t)w.b * gm.Hq + w.g * G + h) * gm.Lq + w.i] * kLog2e;
    dv[h] = Dvec[((int64_t)w.b * gm.Lq + w.i) * gm.Hq + w.g * G + h];
  }
  w.run(K, V, sel, gm, [&](const bool (&ok)[NI], const f32x4 (&kr)[NI], const f32x4 (&vr)[NI]) {
#pragma unroll
    for (int h = 0; h < G; ++h)
#pragma unroll
      for (int n = 0; n < NI; ++n) {
        const float s = key_sum<W::CPR>(dot4(q[h], kr[n])), dp = key_sum<W::CPR>(dot4(dd[h], vr[n]));
        const float ds = __builtin_amdgcn_exp2f(fmaf(s, sl2, -lse[h])) * (dp - dv[h]);
#pragma unroll
        for (int e = 0; e < 4; ++e) dq[h][e] = ok[n] ? fmaf(ds, kr[n][e], dq[h][e]) : dq[h][e];
      }
  });
#pragma unroll
  for (int h = 0; h < G; ++h) {
#pragma unroll
    for (int x = W::CPR; x < 64; x <<= 1)
#pragma unroll
      for (int e = 0; e < 4; ++e) dq[h][e] += __shfl_xor(dq[h][e], x, 64);
    if (w.sub == 0) *reinterpret_cast<f32x4 *>(&wo[w.wave][h][w.ch * 4]) = dq[h];
  }
  __syncthreads();
  for (int x = threadIdx.x; x < G * D; x += 64 * NW) {
    const int h = x / D, c = x - h * D;
    float a = 0.f;
#pragma unroll
    for (int v = 0; v < NW; ++v) a += wo[v][h][c];
    dQ[w.qrow(gm, h) + c] = a * gm.scale;
  }
}

// 16x16x4 float32 MFMA: lane l holds A[l % 16][l / 16], B[l / 16][l % 16] and
// C[4 (l / 16) + r][l % 16].
__device__ __forceinline__ f32x4 mfma_f32(float a, float b, const f32x4 &c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// dK, dV of one unit: block t of M keys and n_ent entries of its list, taken in
// chunks of ROWS = 1024 / M rows (entry x head).  The M / 16 key tiles times the
// ROWS / 16 row tiles of a chunk make four wave tiles; wave w has key tile
// w % KT and row tile w / KT.  A chunk's Q and dO rows are staged in LDS (the
// next chunk's in flight); per wave
//   S = Q K^T, dP = dO V^T  (16 rows x 16 keys; K, V fragments in registers,
//                            lane (q, j) contracting features q D/4 .. + D/4 - 1)
//   dV^T += dO^T P, dK^T += Q^T dS: register r of P (rows 4 q + r) is the B
//                            operand of step r, dO^T and Q^T come from LDS.
// A key takes nothing from a row that may not see it: its weight is zero.  An
// infinity or NaN in Q or dO, which a zero weight would not stop in a product, sends
// the unit through a second walk, whose last two sums run row by row and leave such
// rows out.  (As a branch of the one walk these sums held registers that the products
// need, 204 for 140 at d = 64, and a workgroup less per CU: the whole backward at 4k
// tokens, 2 KV heads of 4 x 128, 32-token blocks, took 587 us without them, 677 with
// the branch and 598 with the second walk; 4 KV heads of 2 x 64, 64-token blocks, 423,
// 464 and 439.  The register bound is the workgroups per CU of the walk alone.)
template <int D, int G, int M>
__global__ __launch_bounds__(256, (D == 64 ? (M == 16 ? 2 : 3) : (M == 16 ? 1 : 2))) void attn_dkv_fp32_kernel(const float *__restrict__ Q, const float *__restrict__ K,
                                                            const float *__restrict__ V,
                                                            const float *__restrict__ dO,
                                                            const float *__restrict__ LSE,
                                                            const float *__restrict__ Dvec, Geom gm, IndexWs ix,
                                                            float *__restrict__ part, float *__restrict__ dK,
                                                            float *__restrict__ dV) {
  constexpr int KT = M / 16, RTL = 4 / KT, ROWS = 16 * RTL;
  constexpr int P = D + 4;               // row pitch: a quarter-wave's 16 rows hit different banks
  constexpr int NT = D / 16, F = D / 4;  // feature tiles; features one lane contracts
  constexpr int VPR = D / 4, NV = ROWS * VPR / 256;
  static_assert(NV * 256 == ROWS * VPR, "staging");
  __shared__ __attribute__((aligned(16))) float Qs[ROWS * P], Os[ROWS * P];
  __shared__ float lse_s[ROWS], dd_s[ROWS], times_s[ROWS];  // times: how often the row lists the block
  __shared__ int pos_s[ROWS];
  __shared__ int odd_s[4];               // wave w staged an infinity or NaN
  const int u = blockIdx.x;
  const int4 unit = ix.units[u];
  if (u % ix.units_bg >= ix.ucnt[u / ix.units_bg]) return;
  const int bgt = unit.x, n_rows = unit.y * G;
  const int bg = bgt / gm.T, t = bgt - bg * gm.T, b = bg / gm.Hkv, g = bg - b * gm.Hkv;
  const int32_t *list = ix.tok + unit.z;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, l16 = lane & 15, q4 = lane >> 4;
  const int kt = wave % KT, rt = wave / KT;
  const int key = t * M + kt * 16 + l16;
  const int64_t krow = (((int64_t)b * gm.Lk + key) * gm.Hkv + g) * D;
  float kf[F], vf[F];
#pragma unroll
  for (int f = 0; f < F; f += 4) {
    const f32x4 a = *reinterpret_cast<const f32x4 *>(K + krow + q4 * F + f);
    const f32x4 c = *reinterpret_cast<const f32x4 *>(V + krow + q4 * F + f);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      kf[f + e] = a[e];
      vf[f + e] = c[e];
    }
  }
  f32x4 dk[NT], dv[NT];

  f32x4 pq[NV], po[NV];
  float pl = 0.f, pd = 0.f, pt = 0.f;
  int pp = -1;
  auto fetch = [&](int r0) {  // rows past the unit's end take its last row; they see no key
#pragma unroll
    for (int k = 0; k < NV; ++k) {
      const int x = tid + 256 * k, r = min(r0 + x / VPR, n_rows - 1), c = (x % VPR) * 4;
      const int64_t src = (((int64_t)b * gm.Lq + (list[r / G] >> 10)) * gm.Hq + g * G + r % G) * D + c;
      pq[k] = *reinterpret_cast<const f32x4 *>(Q + src);
      po[k] = *reinterpret_cast<const f32x4 *>(dO + src);
    }
    if (tid < ROWS) {
      const int r = min(r0 + tid, n_rows - 1), e = list[r / G], i = e >> 10, h = g * G + r % G;
      pt = (float)(1 + (e & 63));
      pl = LSE[((int64_t)b * gm.Hq + h) * gm.Lq + i] * kLog2e;
      pd = Dvec[((int64_t)b * gm.Lq + i) * gm.Hq + h];
      pp = r0 + tid < n_rows ? gm.q_pos0 + i : -1;
    }
  };
  const float sl2 = gm.scale * kLog2e;
  // one walk over the unit's chunks; false: it met an infinity or NaN (not ROWWISE)
  auto walk = [&](auto rowwise_c) {
    constexpr bool ROWWISE = decltype(rowwise_c)::value;
#pragma unroll
    for (int n = 0; n < NT; ++n) dk[n] = dv[n] = f32x4{0.f, 0.f, 0.f, 0.f};
    if (!ROWWISE) fetch(0);
#pragma unroll 1
    for (int r0 = 0; r0 < n_rows; r0 += ROWS) {
      if (ROWWISE) fetch(r0);
      __syncthreads();
      f32x4 z = f32x4{0.f, 0.f, 0.f, 0.f};  // 0 x (finite) stays 0
#pragma unroll
      for (int k = 0; k < NV; ++k) {
        const int x = tid + 256 * k, r = x / VPR, c = (x % VPR) * 4;
        *reinterpret_cast<f32x4 *>(&Qs[r * P + c]) = pq[k];
        *reinterpret_cast<f32x4 *>(&Os[r * P + c]) = po[k];
#pragma unroll
        for (int e = 0; e < 4; ++e) z[e] = fmaf(pq[k][e], 0.f, fmaf(po[k][e], 0.f, z[e]));
      }
      const uint64_t odd_m = __ballot(!(z[0] + z[1] + (z[2] + z[3]) == 0.f));
      if (lane == 0) odd_s[wave] = odd_m != 0;
      if (tid < ROWS) {
        lse_s[tid] = pl;
        dd_s[tid] = pd;
        times_s[tid] = pt;
        pos_s[tid] = pp;
      }
      __syncthreads();
      if (!ROWWISE && r0 + ROWS < n_rows) fetch(r0 + ROWS);
      f32x4 s = f32x4{0.f, 0.f, 0.f, 0.f}, dp = s;
      const float *qr = &Qs[(rt * 16 + l16) * P + q4 * F], *orow = &Os[(rt * 16 + l16) * P + q4 * F];
#pragma unroll
      for (int f = 0; f < F; f += 4) {
        const f32x4 a = *reinterpret_cast<const f32x4 *>(qr + f), c = *reinterpret_cast<const f32x4 *>(orow + f);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          s = mfma_f32(a[e], kf[f + e], s);
          dp = mfma_f32(c[e], vf[f + e], dp);
        }
      }
      // lane (q, j): rows 4 q + r of the tile, key j
      float p[4], ds[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int x = rt * 16 + q4 * 4 + r;
        const float w = times_s[x] * __builtin_amdgcn_exp2f(fmaf(s[r], sl2, -lse_s[x]));
        const bool sees = key <= pos_s[x];
        p[r] = sees ? w : 0.f;
        ds[r] = sees ? w * (dp[r] - dd_s[x]) : 0.f;
      }
      if (ROWWISE) {
#pragma unroll 1
        for (int xq = 0; xq < 4; ++xq)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const int x = rt * 16 + xq * 4 + r;
            const float px = __shfl(p[r], xq * 16 + l16, 64), dx = __shfl(ds[r], xq * 16 + l16, 64);
            if (key > pos_s[x]) continue;
#pragma unroll
            for (int n = 0; n < NT; ++n) {
              const f32x4 ov = *reinterpret_cast<const f32x4 *>(&Os[x * P + n * 16 + q4 * 4]);
              const f32x4 qv = *reinterpret_cast<const f32x4 *>(&Qs[x * P + n * 16 + q4 * 4]);
#pragma unroll
              for (int e = 0; e < 4; ++e) {
                dv[n][e] = fmaf(ov[e], px, dv[n][e]);
                dk[n][e] = fmaf(qv[e], dx, dk[n][e]);
              }
              __builtin_amdgcn_sched_barrier(0);  // a feature tile at a time: no more registers than the other walk
            }
          }
        continue;
      }
      if (!ROWWISE && __builtin_amdgcn_readfirstlane(odd_s[0] | odd_s[1] | odd_s[2] | odd_s[3])) return false;
      // features x keys: A = dO^T (lane: feature l16 of the tile, row 4 q + r), B = P
#pragma unroll
      for (int n = 0; n < NT; ++n)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int at = (rt * 16 + q4 * 4 + r) * P + n * 16 + l16;
          dv[n] = mfma_f32(Os[at], p[r], dv[n]);
          dk[n] = mfma_f32(Qs[at], ds[r], dk[n]);
        }
    }
    return true;
  };
  if (__builtin_expect(!walk(std::false_type{}), 0)) walk(std::true_type{});
  // row tiles of one key tile meet in LDS, one after another; lane (q, j) holds
  // features 16 n + 4 q .. + 3 of key j
  if (RTL > 1) {
    float *acc = Qs;  // [KT * 16 keys][P] dK, then dV in Os
    for (int x = 1; x < RTL; ++x) {
      __syncthreads();
      if (rt == x) {
#pragma unroll
        for (int n = 0; n < NT; ++n) {
          *reinterpret_cast<f32x4 *>(&acc[(kt * 16 + l16) * P + n * 16 + q4 * 4]) = dk[n];
          *reinterpret_cast<f32x4 *>(&Os[(kt * 16 + l16) * P + n * 16 + q4 * 4]) = dv[n];
        }
      }
      __syncthreads();
      if (rt == 0) {
#pragma unroll
        for (int n = 0; n < NT; ++n) {
          dk[n] += *reinterpret_cast<const f32x4 *>(&acc[(kt * 16 + l16) * P + n * 16 + q4 * 4]);
          dv[n] += *reinterpret_cast<const f32x4 *>(&Os[(kt * 16 + l16) * P + n * 16 + q4 * 4]);
        }
      }
    }
    if (rt != 0) return;
  }
  float *ok = dK + krow, *ov = dV + krow;
  if (!unit.w) {  // part of a list: [unit][dK, dV][M][D]
    ok = part + ((int64_t)u * 2 * M + kt * 16 + l16) * D;
    ov = ok + M * D;
  }
#pragma unroll
  for (int n = 0; n < NT; ++n) {
    *reinterpret_cast<f32x4 *>(ok + n * 16 + q4 * 4) = dk[n] * gm.scale;
    *reinterpret_cast<f32x4 *>(ov + n * 16 + q4 * 4) = dv[n];
  }
}

// The blocks with several units (their sums, in unit order) or none (zeros).
template <int D>
__global__ __launch_bounds__(256) void dkv_sum_fp32_kernel(const float *__restrict__ part, float *__restrict__ dK,
                                                           float *__restrict__ dV, Geom gm, IndexWs ix) {
  const int R = gm.B * gm.Hkv, bg = blockIdx.x % R;
  const int b = bg / gm.Hkv, g = bg - b * gm.Hkv;
  for (int j = blockIdx.x / R; j < ix.nfin[bg]; j += gridDim.x / R) {
    const int t = ix.fin[bg * gm.T + j] - bg * gm.T;
    const int32_t *uo = ix.uoff + (int64_t)bg * (gm.T + 1) + t;
    const int u0 = bg * ix.units_bg + uo[0], u1 = bg * ix.units_bg + uo[1];
    for (int x = (blockIdx.y * 256 + threadIdx.x) * 4; x < gm.m * D; x += gridDim.y * 256 * 4) {
      f32x4 sk = f32x4{0.f, 0.f, 0.f, 0.f}, sv = sk;
#pragma unroll 4
      for (int u = u0; u < u1; ++u) {
        sk += *reinterpret_cast<const f32x4 *>(part + (int64_t)u * 2 * gm.m * D + x);
        sv += *reinterpret_cast<const f32x4 *>(part + ((int64_t)u * 2 + 1) * gm.m * D + x);
      }
      const int kk = x / D, c = x - kk * D;
      const int64_t dst = (((int64_t)b * gm.Lk + t * gm.m + kk) * gm.Hkv + g) * D + c;
      *reinterpret_cast<f32x4 *>(dK + dst) = sk;
      *reinterpret_cast<f32x4 *>(dV + dst) = sv;
    }
  }
}

namespace {

// Key rows a lane has in flight: a 16-token block holds 4 (d = 64) or 8 (d =
// 128) per lane; with 8 heads' accumulators beside them 4 is what fits.
template <int D, int G> hipError_t fwd_g(const Geom &g, const float *Q, const float *K, const float *V,
                                         const int32_t *sel, float *O, float *LSE, hipStream_t s) {
  constexpr int NI = G >= 8 ? 4 : 8;
  const dim3 grid(g.Lq, g.B * g.Hkv);
  timing_begin("phsa_attn_fwd_fp32", s);
  if (g.m * D / 256 < NI)
    hipLaunchKernelGGL((attn_fwd_fp32_kernel<D, G, 4, 4>), grid, dim3(256), 0, s, Q, K, V, sel, O, LSE, g);
  else
    hipLaunchKernelGGL((attn_fwd_fp32_kernel<D, G, NI, 4>), grid, dim3(256), 0, s, Q, K, V, sel, O, LSE, g);
  timing_end(s);
  return hipGetLastError();
}

template <int D, int G, int M> hipError_t dkv_m(const Geom &g, const float *Q, const float *K, const float *V,
                                                const float *dO, const float *LSE, const float *Dvec,
                                                const IndexWs &ix, float *part, float *dK, float *dV, hipStream_t s) {
  timing_begin("phsa_attn_bwd_fp32_dkv", s);
  hipLaunchKernelGGL((attn_dkv_fp32_kernel<D, G, M>), dim3((unsigned)(g.B * g.Hkv * ix.units_bg)), dim3(256), 0, s, Q,
                     K, V, dO, LSE, Dvec, g, ix, part, dK, dV);
  timing_end(s);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const int R = g.B * g.Hkv;
  timing_begin("phsa_attn_bwd_dkv_finalize", s);
  hipLaunchKernelGGL((dkv_sum_fp32_kernel<D>), dim3((unsigned)(R * std::min(g.T, std::max(1, 512 / R))), M * D / 1024),
                     dim3(256), 0, s, part, dK, dV, g, ix);
  timing_end(s);
  return hipGetLastError();
}

template <int D, int G> hipError_t bwd_g(const Geom &g, const float *Q, const float *K, const float *V, const float *dO,
                                         const float *LSE, const int32_t *sel, float *dQ, float *dK, float *dV,
                                         const float *Dvec, const IndexWs &ix, float *part, hipStream_t s) {
  hipError_t e = g.m == 64   ? dkv_m<D, G, 64>(g, Q, K, V, dO, LSE, Dvec, ix, part, dK, dV, s)
                 : g.m == 32 ? dkv_m<D, G, 32>(g, Q, K, V, dO, LSE, Dvec, ix, part, dK, dV, s)
                             : dkv_m<D, G, 16>(g, Q, K, V, dO, LSE, Dvec, ix, part, dK, dV, s);
  if (e != hipSuccess) return e;
  timing_begin("phsa_attn_bwd_fp32_dq", s);
  hipLaunchKernelGGL((attn_dq_fp32_kernel<D, G, 4, 4>), dim3(g.Lq, g.B * g.Hkv), dim3(256), 0, s, Q, K, V, dO, LSE,
                     Dvec, sel, dQ, g);
  timing_end(s);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_attn_fwd_fp32(const Geom &g, const float *Q, const float *K, const float *V, const int32_t *sel,
                                float *O, float *LSE, hipStream_t s) {
#define PHSA_FWD(G) \
  case G: return g.d == 128 ? fwd_g<128, G>(g, Q, K, V, sel, O, LSE, s) : fwd_g<64, G>(g, Q, K, V, sel, O, LSE, s);
  switch (g.G) {
    PHSA_FWD(1)
    PHSA_FWD(2)
    PHSA_FWD(4)
    PHSA_FWD(8)
  }
#undef PHSA_FWD
  return hipErrorInvalidValue;
}

hipError_t launch_attn_bwd_fp32(const Geom &g, const float *Q, const float *K, const float *V, const float *O,
                                const float *dO, const float *LSE, const int32_t *sel, float *dQ, float *dK, float *dV,
                                float *ws, hipStream_t s) {
  Fp32BwdWs w;
  fp32_bwd_layout(g, reinterpret_cast<char *>(ws), &w);
  const IndexWs &ix = w.ix;
  float *Dvec = w.Dvec, *part = w.part;
  hipError_t e = launch_bwd_pre(g, O, dO, Dvec, s);
  if (e != hipSuccess) return e;
  e = launch_build_index(g, sel, ix, s);
  if (e != hipSuccess) return e;
#define PHSA_BWD(G)                                                                                      \
  case G:                                                                                                \
    return g.d == 128 ? bwd_g<128, G>(g, Q, K, V, dO, LSE, sel, dQ, dK, dV, Dvec, ix, part, s)          \
                      : bwd_g<64, G>(g, Q, K, V, dO, LSE, sel, dQ, dK, dV, Dvec, ix, part, s);
  switch (g.G) {
    PHSA_BWD(1)
    PHSA_BWD(2)
    PHSA_BWD(4)
    PHSA_BWD(8)
  }
#undef PHSA_BWD
  return hipErrorInvalidValue;
}

}  // namespace phsa
