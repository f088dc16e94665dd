// One decode step with a block KV cache: each of B sequences has one new
// query at position Lk - 1 (its key/value are already in the cache), scores
// the cache's T block representatives, selects, and attends over the chosen
// blocks (Eq. 8, Algorithm 1 selection, Eq. 10-11): one kernel, one workgroup
// per (b, g).
//
//   scores : lanes read K_comp rows as float4 (D / 4 lanes per row, U loads in
//            flight each) and reduce a row's dot product with DPP moves; the
//            scores stay in LDS.
//   top-k  : one wave holds all scores in registers and takes the best one
//            (score desc, block asc) top_k times, a wave maximum each; then it
//            writes the sel row and leaves the slot list in LDS.
//   attend : the selected keys, slot after slot, are dealt to the waves, 32 at a
//            time on the matrix cores (bf16) or NI 16-byte loads of K and of V per
//            lane (float32); a running softmax per wave, merged in LDS into O and
//            LSE.
//
// Both reads are bound by HBM when there are sequences enough to fill the chip
// (64 x 32k: 370 MB in 60 us, 6.2 TB/s; 75 us as a selection and an attention
// kernel) and by what one CU can have in flight when there are few (1 x 8k:
// about 18 bytes a cycle; 27 -> 17 us).  Up to 256 workgroups take 16 waves (one
// per CU), more of them 8, so that two share a CU and one's top-k runs beside
// the other's loads (64 x 32k with 16 waves: 88 against 81 us in the vector
// version).  Long caches of few sequences score in slices (decode_scan_kernel; 6 x
// 32k in 2048 blocks: 70 us with two kernels, 32 with one, 28 in slices).
//
// With per-sequence cache lengths (phsa_decode_varlen) sequence b's query sits
// at position len[b] - 1; its own block may be partly written, and keys past
// the query are masked without reading their values.  cache_append adds one
// token per sequence and maintains the block representatives.
#include <float.h>
#include <math.h>

#include <algorithm>

#include "common.h"
#include "launch.h"

namespace phsa {


// Cache length of sequence b: clen[b] clamped to [1, capacity], or the
// uniform Lk when no length array is given.
__device__ __forceinline__ int seq_len(const int32_t *clen, int b, const Geom &gm) {
  return clen ? min(max(clen[b], 1), gm.Lk) : gm.Lk;
}

// Sum over the CPR consecutive lanes that share a key row (CPR = 8, 16 or 32),
// every lane getting the total.  Within a 16-lane row DPP moves do it: lane ^ 1
// and lane ^ 2 (quad permutations), then the mirrored half row and the
// mirrored row, which pair the quad sums as lane ^ 4 and lane ^ 8 would (the
// same additions, so the same result as a shuffle butterfly).  Rows are paired
// by a shuffle.
template <int CTRL>
__device__ __forceinline__ float dpp_move(float a) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, a), CTRL, 0xF, 0xF, true));
}
template <int CPR>
__device__ __forceinline__ float key_row_sum(float a) {
  static_assert(CPR == 8 || CPR == 16 || CPR == 32, "key rows span 8, 16 or 32 lanes");
  a += dpp_move<0xB1>(a);   // quad_perm [1, 0, 3, 2]
  a += dpp_move<0x4E>(a);   // quad_perm [2, 3, 0, 1]
  a += dpp_move<0x141>(a);  // row_half_mirror
  if constexpr (CPR >= 16) a += dpp_move<0x140>(a);  // row_mirror
  if constexpr (CPR >= 32) a += __shfl_xor(a, 16, 64);
  return a;
}

// Largest value over the wave, every lane getting it (DPP moves within the
// 16-lane rows, row swaps between them).
__device__ __forceinline__ float wave_max_dpp(float v) {
  v = fmaxf(v, dpp_move<0xB1>(v));   // quad_perm [1, 0, 3, 2]
  v = fmaxf(v, dpp_move<0x4E>(v));   // quad_perm [2, 3, 0, 1]
  v = fmaxf(v, dpp_move<0x141>(v));  // row_half_mirror
  v = fmaxf(v, dpp_move<0x140>(v));  // row_mirror
  return max_xor32(max_xor16(v));
}

__device__ __forceinline__ float wave_min_dpp(float v) { return -wave_max_dpp(-v); }

// A NaN score (a NaN or two infinities in a representative) ranks last, as -inf:
// it compares with nothing, and its bits would order above every number.
__device__ __forceinline__ float rank_score(float x) { return x == x ? x : -INFINITY; }

// The k best of the nc candidates sc[0 .. nc) (score desc, index asc), by one
// wave, one pick after the other: lane l holds candidates l, l + 64, ..., and
// each round takes the wave's maximum (the lowest index among equals) out of
// its lane.  Lane p < k returns the p-th pick in index order; nc <= 64 PER.
template <int PER>
__device__ __noinline__ int wave_extract_k(const float *sc, int nc, int k) {
  const int lane = threadIdx.x & 63;
  float v[PER];
  uint32_t taken = 0;  // bit j: candidate j of this lane is out (a score may be -inf itself)
#pragma unroll
  for (int j = 0; j < PER; ++j) {
    v[j] = j * 64 + lane < nc ? rank_score(sc[j * 64 + lane]) : -INFINITY;
    taken |= j * 64 + lane < nc ? 0u : 1u << j;
  }
  int mine = 0x7fffffff;
  for (int p = 0; p < k; ++p) {
    // this lane's best remaining candidate (the lowest j among equals)
    float best = -INFINITY;
    int bj = -1;
#pragma unroll
    for (int j = 0; j < PER; ++j) {
      const bool in = !((taken >> j) & 1) && (bj < 0 || v[j] > best);
      best = in ? v[j] : best;
      bj = in ? j : bj;
    }
    const float top = wave_max_dpp(best);
    const uint64_t m = __ballot(bj >= 0 && best == top);  // not empty: k <= nc, and no score is NaN
    int low = 0x7fffffff;                                 // the lowest index among the equals
    for (uint64_t x = m; x; x &= x - 1) {
      const int l = __builtin_ctzll(x);
      low = min(low, __builtin_amdgcn_readlane(bj, l) * 64 + l);
    }
    if (lane == p) mine = low;
    if (lane == (low & 63)) taken |= 1u << (low >> 6);
  }
  int rank = 0;  // picks below this lane's
  for (int j = 0; j < k; ++j) rank += __builtin_amdgcn_readlane(mine, j) < mine;
  return __builtin_amdgcn_ds_permute((lane < k ? rank : lane) << 2, mine);
}

// The k best of the n <= 64 entries list[0 .. n) (score, index), which stand in
// index order, so that an equal score ranks higher the earlier it stands; an
// index below 0 marks no entry.  Lane p returns the index of the p-th of them in
// index order (0x7fffffff past the last) and its score.
__device__ __forceinline__ int wave_rank_k(float2 *list, int n, int k, int lane, float &score) {
  const float2 me = lane < n ? list[lane] : make_float2(0.f, __int_as_float(-1));
  const bool have = __float_as_int(me.y) >= 0;
  // the score's bits in unsigned order (-0 as +0), 0 for no entry: below -inf
  const uint32_t fb = __float_as_uint(me.x + 0.f);
  const uint32_t key = have ? ((fb & 0x80000000u) ? ~fb : (fb | 0x80000000u)) : 0u;
  int rank = 0;
  for (int l0 = 0; l0 < n; l0 += 8)  // lanes past n hold no entry
#pragma unroll
    for (int l = l0; l < l0 + 8; ++l) rank += __builtin_amdgcn_readlane(key, l) > key;
  uint64_t m = __ballot(have && rank < k);
  if (__popcll(m) > k) {  // equal scores across the k-th place: the earlier ones
    for (int l = 0; l < n; ++l) rank += (l < lane) & (__builtin_amdgcn_readlane(key, l) == key);
    m = __ballot(have && rank < k);
  }
  const int at = bits_below(m);
  wave_lds_sync();
  if (__builtin_amdgcn_inverse_ballot_w64(m)) list[at] = me;
  wave_lds_sync();
  const bool got = lane < __popcll(m);
  const float2 r = list[lane];
  score = got ? r.x : -INFINITY;
  return got ? __float_as_int(r.y) : 0x7fffffff;
}

// The picks of wave_extract_k without a serial chain per pick.  Every lane's
// best is one candidate; the bar is the k-th largest of these 64 (at least k
// candidates reach it, so the k best all do), and the candidates that reach it,
// on random scores a few more than k, are ranked against each other.  Should
// more than 64 reach it (many equal scores, or all the best in few lanes), the
// picks are extracted one by one.  list: 64 entries of LDS.  (Extraction alone
// took 8000 cycles for 14 of 128 candidates, this 4200.)
template <int PER>
__device__ __forceinline__ int wave_top_k(const float *sc, int nc, int k, int lane, float2 *list, float &score) {
  float v[PER], best = -INFINITY;
#pragma unroll
  for (int j = 0; j < PER; ++j) {
    v[j] = j * 64 + lane < nc ? sc[j * 64 + lane] : -INFINITY;
    best = fmaxf(best, v[j]);
  }
  int above = 0;  // lanes whose best is larger
#pragma unroll
  for (int l = 0; l < 64; ++l)
    above += __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(best), l)) > best;
  const float bar = wave_min_dpp(above < k ? best : INFINITY);
  int n = 0;
#pragma unroll
  for (int j = 0; j < PER; ++j) {
    const bool in = j * 64 + lane < nc && v[j] >= bar;
    const uint64_t m = __ballot(in);
    const int at = n + bits_below(m);
    if (in && at < 64) list[at] = make_float2(v[j], __int_as_float(j * 64 + lane));
    n += __popcll(m);
  }
  if (n > 64 || n < k) {  // n < k: NaN scores
    const int c = wave_extract_k<PER>(sc, nc, k);
    score = lane < k ? sc[c] : -INFINITY;
    return c;
  }
  wave_lds_sync();
  return wave_rank_k(list, n, k, lane, score);
}

// top_k by the size of the candidate list (one wave; nc <= 2048)
__device__ __forceinline__ int top_k_of(const float *sc, int nc, int k, int lane, float2 *list, float &score) {
  return nc <= 128   ? wave_top_k<2>(sc, nc, k, lane, list, score)
         : nc <= 512 ? wave_top_k<8>(sc, nc, k, lane, list, score)
                     : wave_top_k<32>(sc, nc, k, lane, list, score);
}

// Scores of blocks s0 <= t < s1 of one (b, g) into sc[h * T + t], by NW waves:
// GM = 1 sums the group's heads before the product (scaled logits), GM = G
// keeps them apart (log2 units).
template <typename T, int D, int G, int GM, int NW>
__device__ __forceinline__ void score_blocks(const T *Qg, const float *kc, int s0, int s1, float *sc, const Geom &gm) {
  constexpr int LPR = D / 4;      // lanes per representative row (one float4 each)
  constexpr int RPW = 64 / LPR;   // rows per wave load instruction
  constexpr int U = 8;            // load instructions in flight per lane
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int sub = lane / LPR, c4 = (lane % LPR) * 4;
  float q[GM][4];
#pragma unroll
  for (int h = 0; h < GM; ++h)
#pragma unroll
    for (int e = 0; e < 4; ++e) q[h][e] = 0.f;
#pragma unroll
  for (int hh = 0; hh < G; ++hh)
#pragma unroll
    for (int e = 0; e < 4; ++e)
      q[GM > 1 ? hh : 0][e] += to_f32<T>(Qg[hh * D + c4 + e]) * (GM > 1 || gm.sel_mode == 1 ? gm.scale * kLog2e : 1.f);
  for (int t0 = s0 + wave * RPW * U; t0 < s1; t0 += NW * RPW * U) {
    float4 v[U];
#pragma unroll
    for (int u = 0; u < U; ++u)
      v[u] = *reinterpret_cast<const float4 *>(kc + (int64_t)min(t0 + u * RPW + sub, s1 - 1) * D + c4);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int t = t0 + u * RPW + sub;
#pragma unroll
      for (int h = 0; h < GM; ++h) {
        float a = fmaf(q[h][0], v[u].x, fmaf(q[h][1], v[u].y, fmaf(q[h][2], v[u].z, q[h][3] * v[u].w)));
        a = key_row_sum<LPR>(a);
        if (lane % LPR == 0 && t < s1) sc[h * gm.T + t] = gm.sel_mode == 1 ? a : a * gm.scale;
      }
    }
  }
}

// Long caches with few sequences: the candidate range of a (b, g) is scored by
// `slices` workgroups, one CU's loads being what bounds it (1 MB of
// representatives per (b, g) at T = 2048).  Each leaves the k best of its slice,
// in index order, as (score, block) at entry slice * k of the group's own O
// rows, which decode_kernel reads before it writes them.
template <typename T, int D, int G>
__global__ __launch_bounds__(512) void decode_scan_kernel(const T *__restrict__ Q, const float *__restrict__ Kc,
                                                          const int32_t *__restrict__ clen, T *__restrict__ O,
                                                          Geom gm) {
  extern __shared__ __attribute__((aligned(16))) float sc[];  // [T]
  __shared__ float2 list_s[64];
  const int bg = blockIdx.y, b = bg / gm.Hkv, g = bg - b * gm.Hkv, lane = threadIdx.x & 63;
  const int cur = (seq_len(clen, b, gm) - 1) / gm.m, lo = max(0, cur - gm.window / gm.m);
  const int nc = max(0, lo - gm.n_init), per = (nc + gridDim.x - 1) / gridDim.x;
  const int c0 = min(per * (int)blockIdx.x, nc), n = min(per, nc - c0), k = min(gm.top_k, n);
  const int64_t q0 = ((int64_t)b * gm.Hq + g * G) * D;
  score_blocks<T, D, G, 1, 8>(Q + q0, Kc + (int64_t)bg * gm.T * D, gm.n_init + c0, gm.n_init + c0 + n, sc, gm);
  __syncthreads();
  if (threadIdx.x >= 64) return;
  float score = -INFINITY;
  int c = 0x7fffffff;
  if (k > 0) c = top_k_of(sc + gm.n_init + c0, n, k, lane, list_s, score);
  if (lane < gm.top_k)
    reinterpret_cast<float2 *>(O + q0)[blockIdx.x * gm.top_k + lane] =
        make_float2(rank_score(score), __int_as_float(lane < k ? gm.n_init + c0 + c : -1));
}

// LDS of one wave in the attention: its V tile (bf16: 32 keys), later its sums.
template <typename T, int D, int G> constexpr int decode_wave_bytes() {
  return sizeof(T) == 2 && 32 * D * 2 > G * D * 4 ? 32 * D * 2 : G * D * 4;
}

// Copies the values of keys key0[0] .. + 15 and key0[1] .. + 15 (keys past pos:
// those of pos) into rows 0 .. 31 of a swizzled LDS tile, by one wave (copies
// straight into LDS, counted in vmcnt).
template <int D>
__device__ __forceinline__ void copy_values(const bf16_t *Vb, int64_t kstep, const int (&key0)[2], int pos, bf16_t *Vs,
                                            int lane) {
  constexpr int VPR = D / 8, RPI = 64 / VPR;
#pragma unroll
  for (int v = 0; v < 32 / RPI; ++v) {
    const int r = v * RPI + lane / VPR, c = (lane % VPR) ^ (r & (VPR - 1));
    const int key = min(key0[(v * RPI) >> 4] + (r & 15), pos);
    __builtin_amdgcn_global_load_lds(Vb + key * kstep + c * 8, (lds_void_t *)(Vs + v * RPI * D), 16, 0, 0);
  }
}

// copy_values by way of registers, for caches that do not start at a multiple of
// 16 bytes.
template <int D>
__device__ __forceinline__ void copy_values_reg(const bf16_t *Vb, int64_t kstep, const int (&key0)[2], int pos,
                                                bf16_t *Vs, int lane) {
  constexpr int VPR = D / 8, RPI = 64 / VPR;
#pragma unroll
  for (int v = 0; v < 32 / RPI; ++v) {
    const int r = v * RPI + lane / VPR, c = (lane % VPR) ^ (r & (VPR - 1));
    const int key = min(key0[(v * RPI) >> 4] + (r & 15), pos);
    *reinterpret_cast<u32x4 *>(Vs + v * RPI * D + lane * 8) = *reinterpret_cast<const u32x4 *>(Vb + key * kstep + c * 8);
  }
}

// MODE 0 ranks on the summed logits of the group's heads.  MODE 1
// (PHSA_FLAG_SELECT_SOFTMAX_SUM) keeps every head's log2 logits of the
// complete blocks 0..cur-1 in LDS, reduces each head's log2 normaliser over
// the workgroup, and scores a candidate by log2 sum_h 2^(x_h - lse_h).  MODE 2
// takes the best of decode_scan_kernel's slices (summed logits).
// The registers of 16 waves (128 each) hold up to two heads, and any group in
// bf16 where the heads are not scored apart; the others take 8 waves with 256.
template <typename T, int G, int MODE> constexpr bool kDecodeSmall = G <= 2 || (sizeof(T) == 2 && MODE != 1);

// ANY: V starts anywhere (bf16; float32 reads it into registers as it is).
template <typename T, int D, int G, int MODE, int NW, bool ANY>
__global__ __launch_bounds__(NW * 64, (kDecodeSmall<T, G, MODE> ? 4 : 2)) void decode_kernel(const T *__restrict__ Q, const T *__restrict__ K,
                                                           const T *__restrict__ V, const float *__restrict__ Kc,
                                                           const int32_t *__restrict__ clen,
                                                           int32_t *__restrict__ sel, T *O,
                                                           float *__restrict__ LSE, Geom gm, int slices) {
  constexpr int GM = MODE == 1 ? G : 1;   // heads scored apart
  constexpr int NTHR = NW * 64;
  constexpr int AREA = decode_wave_bytes<T, D, G>() / 4;  // floats of a wave's area
  // MODE 0: [T] scores; MODE 1: [G][T] head logits, then scores in row 0.  Dead
  // after the top-k: the attention's per-wave areas take the same bytes.
  extern __shared__ __attribute__((aligned(16))) float sc[];
  __shared__ float red_m[NW][GM], red_l[NW][GM];
  __shared__ float2 list_s[64];
  __shared__ int slot_s[64];
  __shared__ int nslot_s;
  __shared__ float wm[NW][G], wl[NW][G], wf[NW][G], lsum[G];
  const int bg = blockIdx.x, b = bg / gm.Hkv, g = bg - b * gm.Hkv;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int pos = seq_len(clen, b, gm) - 1, cur = pos / gm.m;  // the query's position and own block
  const int lo = max(0, cur - gm.window / gm.m);
  const int nc = gm.top_k > 0 ? max(0, lo - gm.n_init) : 0;  // candidates n_init .. lo - 1
  const T *Qg = Q + ((int64_t)b * gm.Hq + g * G) * D;
  if (MODE != 2 && nc > 0) {
    // MODE 0 scores the candidates n_init <= t < lo; MODE 1 every complete block t < cur
    score_blocks<T, D, G, GM, NW>(Qg, Kc + (int64_t)bg * gm.T * D, MODE == 1 ? 0 : gm.n_init, MODE == 1 ? cur : lo, sc, gm);
    __syncthreads();
    if (MODE == 1) {
      // per-head log2 normaliser over t < cur: thread-local running (max, sum),
      // merged across the wave by shuffles and across the waves through LDS
      float lse[GM];
#pragma unroll
      for (int h = 0; h < GM; ++h) {
        float mx = -INFINITY, sm = 0.f;
        for (int t = tid; t < cur; t += NTHR) {
          const float x = sc[h * gm.T + t];
          if (x > mx) {
            sm = sm * exp2f(mx - x) + 1.f;
            mx = x;
          } else {
            sm += exp2f(x - mx);
          }
        }
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
          const float om = __shfl_xor(mx, o, 64), os = __shfl_xor(sm, o, 64);
          const float nm = fmaxf(mx, om);
          sm = (sm > 0.f ? sm * exp2f(mx - nm) : 0.f) + (os > 0.f ? os * exp2f(om - nm) : 0.f);
          mx = nm;
        }
        if (lane == 0) {
          red_m[wave][h] = mx;
          red_l[wave][h] = sm;
        }
      }
      __syncthreads();
#pragma unroll
      for (int h = 0; h < GM; ++h) {
        float M = -INFINITY, L = 0.f;
#pragma unroll
        for (int w = 0; w < NW; ++w) M = fmaxf(M, red_m[w][h]);
#pragma unroll
        for (int w = 0; w < NW; ++w)
          if (red_l[w][h] > 0.f) L += red_l[w][h] * exp2f(red_m[w][h] - M);
        lse[h] = L > 0.f ? M + log2f(L) : 0.f;
      }
      // candidates: the group score replaces head 0's logit in place (one thread per block)
      for (int t = gm.n_init + tid; t < lo; t += NTHR) {
        float y[GM], ym = -INFINITY;
#pragma unroll
        for (int h = 0; h < GM; ++h) {
          y[h] = sc[h * gm.T + t] - lse[h];
          ym = fmaxf(ym, y[h]);
        }
        float e = 0.f;
#pragma unroll
        for (int h = 0; h < GM; ++h) e += exp2f(y[h] - ym);
        sc[t] = ym + log2f(e);
      }
      __syncthreads();
    }
  }
  if (wave == 0) {
    const int npick = min(gm.top_k, nc);
    int mine = 0x7fffffff;  // lanes 0..npick-1: the picks, ascending
    float score;
    if (MODE == 2) {
      list_s[lane] = lane < slices * gm.top_k ? reinterpret_cast<const float2 *>(O + (Qg - Q))[lane]
                                              : make_float2(0.f, __int_as_float(-1));
      wave_lds_sync();
      mine = wave_rank_k(list_s, slices * gm.top_k, npick, lane, score);
    } else if (npick > 0) {
      mine = gm.n_init + top_k_of(sc + gm.n_init, nc, npick, lane, list_s, score);
    }
    int32_t *out = sel + (int64_t)bg * gm.ksel;
    const int ni = min(gm.n_init, cur + 1);
    const int lstart = max(lo, ni);
    const int nlocal = cur - lstart + 1;
    auto put = [&](int slot, int t) {
      out[slot] = t;
      slot_s[slot] = t;
    };
    if (lane < ni) put(lane, lane);
    if (lane < npick) put(ni + lane, mine);
    if (lane < nlocal) put(ni + npick + lane, lstart + lane);
    for (int x = ni + npick + nlocal + lane; x < gm.ksel; x += 64) out[x] = -1;
    if (lane == 0) nslot_s = ni + npick + nlocal;
  }

  // ---- attention over the selected keys, slot after slot
  __syncthreads();
  const int msh = __builtin_ctz((unsigned)gm.m);
  const int nkeys = nslot_s << msh;
  const T *Kb = K + ((int64_t)b * gm.Lk * gm.Hkv + g) * D, *Vb = V + (Kb - K);
  const int64_t kstep = (int64_t)gm.Hkv * D;
  const float sl2 = gm.scale * kLog2e;
  float *wo = sc + wave * AREA;  // this wave's [G][D] sums, in the end
  if constexpr (sizeof(T) == 2) {
    // Matrix cores: 32 keys at a time, S^T = K Q^T (keys x heads; the G heads
    // fill G of 16 columns) with K straight from memory as the A operand, and
    // O^T = V^T P^T with V copied into the wave's LDS area and read transposed.
    // P is split into three bf16 parts, three products: 8 + 8 + 8 bits hold its
    // float32 mantissa, so O is the sum of the weights that LSE counts.  (On the vector
    // ALUs, lane = feature, the products of one workgroup took 14000 of 25000
    // cycles at 1 x 8k.)
    constexpr int KB = D / 32, NT = D / 16;
    bf16_t *Vs = reinterpret_cast<bf16_t *>(wo);  // [32][D], swizzled
    const int l16 = lane & 15, q4 = lane >> 4;
    bf16x8 q[KB];
#pragma unroll
    for (int kb = 0; kb < KB; ++kb) {
      const u32x4 z = {0u, 0u, 0u, 0u};
      q[kb] = __builtin_bit_cast(
          bf16x8, l16 < G ? *reinterpret_cast<const u32x4 *>(Q + ((int64_t)b * gm.Hq + g * G + l16) * D + kb * 32 + q4 * 8)
                          : z);
    }
    f32x4 o[NT];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) o[nt] = f32x4{0.f, 0.f, 0.f, 0.f};
    float mrun = -INFINITY, lrun = 0.f;
    for (int x0 = wave * 32; x0 < nkeys; x0 += NW * 32) {
      int key0[2];  // first key of each 16-key tile (past the last slot: the last tile again, masked)
#pragma unroll
      for (int kt = 0; kt < 2; ++kt) {
        const int x = min(x0 + kt * 16, nkeys - 16);
        key0[kt] = (__builtin_amdgcn_readfirstlane(slot_s[x >> msh]) << msh) + (x & (gm.m - 1));
      }
      bf16x8 kf[2][KB];
#pragma unroll
      for (int kt = 0; kt < 2; ++kt)
#pragma unroll
        for (int kb = 0; kb < KB; ++kb)
          kf[kt][kb] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4 *>(
                                                      Kb + min(key0[kt] + l16, pos) * kstep + kb * 32 + q4 * 8));
      // the previous tile's transposed reads have returned: the copies reach LDS
      // by another path, which the order of LDS instructions does not cover
      wave_lds_sync();
      lds_wait();
      if constexpr (!ANY) copy_values<D>(Vb, kstep, key0, pos, Vs, lane);
      else copy_values_reg<D>(Vb, kstep, key0, pos, Vs, lane);
      f32x4 st[2];
      float mn = mrun;
#pragma unroll
      for (int kt = 0; kt < 2; ++kt) {
        st[kt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int kb = 0; kb < KB; ++kb) st[kt] = mfma16x16x32(kf[kt][kb], q[kb], st[kt]);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const bool ok = x0 + kt * 16 < nkeys && key0[kt] + q4 * 4 + r <= pos;
          st[kt][r] = ok ? st[kt][r] * sl2 : -INFINITY;
          mn = fmaxf(mn, st[kt][r]);
        }
      }
      mn = max_xor32(max_xor16(mn));
      // mn stays -inf only while every key so far was masked
      const float f = mn == -INFINITY ? 1.f : __builtin_amdgcn_exp2f(mrun - mn);
      const float mz = mn == -INFINITY ? 0.f : mn;
      mrun = mn;
      lrun *= f;
      f32x4 mid[2], lo[2];
#pragma unroll
      for (int kt = 0; kt < 2; ++kt)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const float p = __builtin_amdgcn_exp2f(st[kt][r] - mz);
          lrun += p;
          const float h = bf16_to_f32(f32_to_bf16(p)), d1 = p - h, h1 = bf16_to_f32(f32_to_bf16(d1));
          st[kt][r] = h;
          mid[kt][r] = h1;
          lo[kt][r] = d1 - h1;
        }
      const bf16x8 ph = pack_bf16x8(st[0], st[1]), pm = pack_bf16x8(mid[0], mid[1]), pl = pack_bf16x8(lo[0], lo[1]);
      dma_wait();
      wave_lds_sync();
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) {
        const bf16x8 vt = lds_col8_sw<D>(Vs, q4 * 4, 16 + q4 * 4, nt * 16, l16);
        o[nt] *= f;
        o[nt] = mfma16x16x32(vt, pl, o[nt]);
        o[nt] = mfma16x16x32(vt, pm, o[nt]);
        o[nt] = mfma16x16x32(vt, ph, o[nt]);
      }
    }
    lrun += __shfl_xor(lrun, 16, 64);
    lrun += __shfl_xor(lrun, 32, 64);
    wave_lds_sync();
    bool odd = false;
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
      for (int r = 0; r < 4; ++r) odd |= !(o[nt][r] == o[nt][r]);
    if (__builtin_expect(__ballot(odd && l16 < G) != 0, 0)) {
      // An infinite value met a zero part or a masked key in the products
      // (0 x inf): this wave's keys again, one after another.
      constexpr int E = D / 64;  // features lane E .. + E - 1 of every head
      float acc[G][E];
#pragma unroll
      for (int h = 0; h < G; ++h)
#pragma unroll
        for (int e = 0; e < E; ++e) acc[h][e] = 0.f;
#pragma unroll 1
      for (int x0 = wave * 32; x0 < nkeys; x0 += NW * 32)
#pragma unroll 1
        for (int x = x0; x < min(x0 + 32, nkeys); ++x) {
          const int key = (__builtin_amdgcn_readfirstlane(slot_s[x >> msh]) << msh) + (x & (gm.m - 1));
          if (key > pos) break;
#pragma unroll
          for (int h = 0; h < G; ++h) {
            float a = 0.f;
#pragma unroll
            for (int e = 0; e < E; ++e) a = fmaf(to_f32<T>(Qg[h * D + lane * E + e]), to_f32<T>(Kb[key * kstep + lane * E + e]), a);
#pragma unroll
            for (int y = 1; y < 64; y <<= 1) a += __shfl_xor(a, y, 64);
            const float mh = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(mrun), h));
            const float p = __builtin_amdgcn_exp2f(a * sl2 - (mh == -INFINITY ? 0.f : mh));
#pragma unroll
            for (int e = 0; e < E; ++e) acc[h][e] = fmaf(p, to_f32<T>(Vb[key * kstep + lane * E + e]), acc[h][e]);
          }
        }
#pragma unroll
      for (int h = 0; h < G; ++h)
#pragma unroll
        for (int e = 0; e < E; ++e) wo[h * D + lane * E + e] = acc[h][e];
    } else if (l16 < G) {  // lane (q, j) holds features 16 nt + 4 q .. + 3 of head j
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) *reinterpret_cast<f32x4 *>(wo + l16 * D + nt * 16 + q4 * 4) = o[nt];
    }
    if (l16 < G && q4 == 0) {
      wm[wave][l16] = mrun;
      wl[wave][l16] = lrun;
    }
  } else {
    // float32: load unit u covers KPI keys (blocks are multiples of 16 keys, so a
    // unit lies in one block); lane = (sub, ch) holds VEC features of every
    // KPI-th key and the CPR lanes of a key reduce its dot products.
    constexpr int VEC = 16 / sizeof(T), CPR = D / VEC, KPI = 64 / CPR, NI = 8;
    const int ch = lane % CPR, sub = lane / CPR;
    f32x4 qv[G], o[G];
    float mrun[G], lrun[G];
#pragma unroll
    for (int h = 0; h < G; ++h) {
      qv[h] = *reinterpret_cast<const f32x4 *>(Q + ((int64_t)b * gm.Hq + g * G + h) * D + ch * VEC) * sl2;
      o[h] = f32x4{0.f, 0.f, 0.f, 0.f};
      mrun[h] = -INFINITY;
      lrun[h] = 0.f;
    }
    const int nunits = nkeys / KPI;
    for (int u0 = wave * NI; u0 < nunits; u0 += NW * NI) {
      f32x4 kr[NI], vr[NI];
      uint32_t okm = 0;      // bit i: this lane's key of load i counts
#pragma unroll
      for (int i = 0; i < NI; ++i) {
        const int x = min(u0 + i, nunits - 1) * KPI;  // units past the end are masked
        const int key = (__builtin_amdgcn_readfirstlane(slot_s[x >> msh]) << msh) + (x & (gm.m - 1)) + sub;
        okm |= u0 + i < nunits && key <= pos ? 1u << i : 0u;
        const int64_t src = min(key, pos) * kstep + ch * VEC;
        kr[i] = *reinterpret_cast<const f32x4 *>(Kb + src);
        vr[i] = *reinterpret_cast<const f32x4 *>(Vb + src);
      }
#pragma unroll
      for (int h = 0; h < G; ++h) {
        float s[NI], mn = mrun[h];
#pragma unroll
        for (int i = 0; i < NI; ++i) {
          float a = 0.f;
#pragma unroll
          for (int e = 0; e < VEC; ++e) a = fmaf(qv[h][e], kr[i][e], a);
          a = key_row_sum<CPR>(a);
          s[i] = (okm >> i) & 1 ? a : -INFINITY;
          mn = fmaxf(mn, s[i]);
        }
        // every key group of lanes keeps a maximum of its own (equal in the CPR
        // lanes of a key); they meet at the end.  mn stays -inf only while every
        // key so far was masked or scored -inf (an infinite key): weights 0.
        const float f = mn == -INFINITY ? 1.f : __builtin_amdgcn_exp2f(mrun[h] - mn);
        const float mz = mn == -INFINITY ? 0.f : mn;
        mrun[h] = mn;
        lrun[h] *= f;
        o[h] *= f;
        // keys past the query (the unwritten tail of its own block) add nothing;
        // their loads repeat the query's own value, which may be infinite
#pragma unroll
        for (int i = 0; i < NI; ++i) {
          const bool ok = (okm >> i) & 1;
          const float p = ok ? __builtin_amdgcn_exp2f(s[i] - mz) : 0.f;
          lrun[h] += p;
#pragma unroll
          for (int e = 0; e < VEC; ++e) o[h][e] = ok ? fmaf(p, vr[i][e], o[h][e]) : o[h][e];
        }
      }
    }
    // the key groups of the wave (lanes with the same chunk)
#pragma unroll
    for (int h = 0; h < G; ++h) {
      float M = mrun[h];
#pragma unroll
      for (int x = CPR; x < 64; x <<= 1) M = fmaxf(M, __shfl_xor(M, x, 64));
      const float f = mrun[h] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(mrun[h] - M);
      lrun[h] *= f;
      o[h] *= f;
#pragma unroll
      for (int x = CPR; x < 64; x <<= 1) {
        lrun[h] += __shfl_xor(lrun[h], x, 64);
#pragma unroll
        for (int e = 0; e < VEC; ++e) o[h][e] += __shfl_xor(o[h][e], x, 64);
      }
      if (lane == 0) {
        wm[wave][h] = M;
        wl[wave][h] = lrun[h];
      }
      if (sub == 0) *reinterpret_cast<f32x4 *>(wo + h * D + ch * VEC) = o[h];
    }
  }
  // ---- the waves' sums: their factors first (one thread per wave and head), then the features
  __syncthreads();
  if (tid < NW * G) {
    const int w = tid / G, h = tid - w * G;
    float M = -INFINITY, L = 0.f;
#pragma unroll
    for (int v = 0; v < NW; ++v) M = fmaxf(M, wm[v][h]);
#pragma unroll
    for (int v = 0; v < NW; ++v) L += wm[v][h] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(wm[v][h] - M) * wl[v][h];
    wf[w][h] = wm[w][h] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(wm[w][h] - M);
    if (w == 0) {
      lsum[h] = L;
      LSE[(int64_t)b * gm.Hq + g * G + h] = L > 0.f ? (M + log2f(L)) * kLn2 : -INFINITY;
    }
  }
  __syncthreads();
  for (int x = tid; x < G * D; x += NTHR) {
    const int h = x / D, c = x - h * D;
    float acc = 0.f;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      // every wave has stored its sums, zeros where it had no keys (factor 0)
      const float f = wf[w][h];
      acc = fmaf(f, sc[w * AREA + h * D + c], acc);
    }
    O[((int64_t)b * gm.Hq + g * G + h) * D + c] = from_f32<T>(lsum[h] > 0.f ? acc / lsum[h] : 0.f);
  }
}

struct DecodeArgs {
  const void *Q, *K, *V;
  const float *Kc;
  const int32_t *clen;
  int32_t *sel;
  void *O;
  float *LSE;
};

template <typename T, int D, int G, int MODE, int NW, bool ANY = false>
static hipError_t launch_decode_w(const Geom &g, const DecodeArgs &a, int slices, hipStream_t s) {
  timing_begin("phsa_decode", s);
  hipLaunchKernelGGL((decode_kernel<T, D, G, MODE, NW, ANY>), dim3(g.B * g.Hkv), dim3(NW * 64),
                     std::max(MODE == 2 ? 0 : (size_t)(MODE == 1 ? G : 1) * g.T * sizeof(float),
                              (size_t)NW * decode_wave_bytes<T, D, G>()),
                     s, static_cast<const T *>(a.Q), static_cast<const T *>(a.K), static_cast<const T *>(a.V), a.Kc,
                     a.clen, a.sel, static_cast<T *>(a.O), a.LSE, g, slices);
  timing_end(s);
  return hipGetLastError();
}

// Up to one workgroup per CU they take 16 waves, beyond that 8 (two share a CU).
template <typename T, int D, int G, int MODE, bool ANY = false>
static hipError_t launch_decode_m(const Geom &g, const DecodeArgs &a, int slices, hipStream_t s) {
  if constexpr (kDecodeSmall<T, G, MODE>)
    if (g.B * g.Hkv <= 256) return launch_decode_w<T, D, G, MODE, 16, ANY>(g, a, slices, s);
  return launch_decode_w<T, D, G, MODE, 8, ANY>(g, a, slices, s);
}

template <typename T, int D, int G>
static hipError_t launch_decode_g(const Geom &g, const DecodeArgs &a, hipStream_t s) {
  if constexpr (sizeof(T) == 2)
    if (!starts_at_16(a.V))  // a check inside the kernel took 1.1 us of 69 (64 x 32k)
      return g.sel_mode == 1 ? launch_decode_m<T, D, G, 1, true>(g, a, 0, s) : launch_decode_m<T, D, G, 0, true>(g, a, 0, s);
  if (g.sel_mode == 1) return launch_decode_m<T, D, G, 1>(g, a, 0, s);
  // Slices of the candidate range: as many as the group's O rows hold lists of
  // (one wave ranks at most 64 entries), while the workgroups fit the CUs and a
  // slice keeps 256 blocks.  Below that the second launch costs what it gains.
  // O is scratch until the second kernel: not where it is Q, or not aligned.
  int slices = g.top_k > 0 ? std::min({(int)(G * D * sizeof(T) / 8), 64}) / g.top_k : 0;
  slices = std::min({slices, 256 / (g.B * g.Hkv), g.T / 256});
  if (slices < 2 || a.O == a.Q || reinterpret_cast<uintptr_t>(a.O) % 8 != 0)
    return launch_decode_m<T, D, G, 0>(g, a, 0, s);
  timing_begin("phsa_decode_scan", s);
  hipLaunchKernelGGL((decode_scan_kernel<T, D, G>), dim3(slices, g.B * g.Hkv), dim3(512), g.T * sizeof(float), s,
                     static_cast<const T *>(a.Q), a.Kc, a.clen, static_cast<T *>(a.O), g);
  timing_end(s);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  return launch_decode_m<T, D, G, 2>(g, a, slices, s);
}

template <typename T, int D>
static hipError_t launch_decode_t(const Geom &g, const DecodeArgs &a, hipStream_t s) {
  switch (g.G) {
    case 1: return launch_decode_g<T, D, 1>(g, a, s);
    case 2: return launch_decode_g<T, D, 2>(g, a, s);
    case 4: return launch_decode_g<T, D, 4>(g, a, s);
    default: return launch_decode_g<T, D, 8>(g, a, s);
  }
}

// ---------------------------------------------------------------- cache append
// One token per sequence joins the cache at position len[b]; the length grows
// by one.  When the token completes block t, that block's representative is
// computed from the cache (Eq. 6-8, the same pooling as phsa_compress) and
// written to K_comp[b, :, t].  One workgroup per sequence; a sequence whose
// cache is full is left unchanged.  Rows move in 16-byte chunks; for the
// pooling, the Hkv*d elements are split into 16-byte chunks and the block's m
// keys into NTHR / #chunks slices (at most m), U rows in flight per thread, whose
// partial sums meet in LDS, a thread per element.  A chain of memory round trips
// bounds it (length, row, block), so the block's punctuation flags are one load
// and a ballot per wave (one thread counting them a byte at a time took the call
// from 7 to 30 us).  When one thread per chunk added the slices' sums, those of
// a narrow cache (2 heads of 64: 16 threads, 64 slices) took the kernel to 28 us.
template <typename T, int D, int NTHR>
__global__ __launch_bounds__(NTHR) void cache_append_kernel(const T *__restrict__ Kn, const T *__restrict__ Vn,
                                                            const uint8_t *__restrict__ pn, T *__restrict__ Kcache,
                                                            T *__restrict__ Vcache, uint8_t *__restrict__ pcache,
                                                            int32_t *__restrict__ clen, float *__restrict__ Kc,
                                                            Geom gm) {
  constexpr int VEC = 16 / sizeof(T), U = 8;
  __shared__ float red[2][NTHR][VEC];
  const int b = blockIdx.x, tid = threadIdx.x, lane = tid & 63;
  const int pos = clen[b];
  if (pos < 0 || pos >= gm.Lk) return;  // full (or invalid): nothing changes
  const int HD = gm.Hkv * D, NCH = HD / VEC;
  const bool newp = pn[b] != 0;
  for (int x = tid; x < NCH; x += NTHR) {
    const int64_t dst = ((int64_t)b * gm.Lk + pos) * HD + x * VEC;
    *reinterpret_cast<uint4 *>(Kcache + dst) = *reinterpret_cast<const uint4 *>(Kn + (int64_t)b * HD + x * VEC);
    *reinterpret_cast<uint4 *>(Vcache + dst) = *reinterpret_cast<const uint4 *>(Vn + (int64_t)b * HD + x * VEC);
  }
  if (tid == 0) pcache[(int64_t)b * gm.Lk + pos] = pn[b];
  if ((pos + 1) % gm.m == 0) {
    // the block is complete: pool its m keys (the newest one from the input,
    // the others from the cache, which this launch does not write)
    const int t = pos / gm.m, j0 = t * gm.m;
    // flags of the block's keys, in every wave (attention blocks hold at most 64)
    const bool flag = lane < gm.m && (j0 + lane == pos ? newp : pcache[(int64_t)b * gm.Lk + j0 + min(lane, gm.m - 1)] != 0);
    const uint64_t pmask = __ballot(flag);
    const int np = __popcll(pmask);
    for (int x0 = 0; x0 < NCH; x0 += NTHR) {
      const int nch = min(NTHR, NCH - x0);      // chunks handled in this pass
      const int slices = min(NTHR / nch, gm.m); // key slices
      const int ch = tid % nch, sl = tid / nch;
      float sum[VEC], psum[VEC];
#pragma unroll
      for (int e = 0; e < VEC; ++e) sum[e] = psum[e] = 0.f;
      if (sl < slices) {
        for (int ja = sl; ja < gm.m; ja += U * slices) {
          u32x4 raw[U];
#pragma unroll
          for (int u = 0; u < U; ++u) {
            const int j = j0 + min(ja + u * slices, gm.m - 1);
            raw[u] = *reinterpret_cast<const u32x4 *>(
                j == pos ? Kn + (int64_t)b * HD + (x0 + ch) * VEC : Kcache + ((int64_t)b * gm.Lk + j) * HD + (x0 + ch) * VEC);
          }
#pragma unroll
          for (int u = 0; u < U; ++u) {
            const int j = ja + u * slices;
            if (j >= gm.m) break;
            const bool pj = lane_bit(pmask, j);
            const T *pv = reinterpret_cast<const T *>(&raw[u]);
#pragma unroll
            for (int e = 0; e < VEC; ++e) {
              const float k = to_f32<T>(pv[e]);
              sum[e] += k;
              psum[e] += pj ? k : 0.f;
            }
          }
        }
      }
#pragma unroll
      for (int e = 0; e < VEC; ++e) {
        red[0][tid][e] = sum[e];
        red[1][tid][e] = psum[e];
      }
      __syncthreads();
      // one thread per element: slice q's sums start at q * nch * VEC
      const float *r0 = &red[0][0][0], *r1 = &red[1][0][0];
      for (int x = tid; x < nch * VEC; x += NTHR) {
        float s0 = 0.f, s1 = 0.f;
        for (int q = 0; q < slices; ++q) {
          s0 += r0[q * nch * VEC + x];
          s1 += r1[q * nch * VEC + x];
        }
        const float m0 = s0 / (float)gm.m;
        const int at = x0 * VEC + x, g = at / D, c = at - g * D;
        Kc[(((int64_t)b * gm.Hkv + g) * gm.T + t) * D + c] =
            np > 0 ? gm.lambda * m0 + (1.f - gm.lambda) * (s1 / (float)np) : m0;
      }
      __syncthreads();
    }
  }
  __syncthreads();
  if (tid == 0) clen[b] = pos + 1;
}

template <typename T, int D, int NTHR>
static hipError_t launch_cache_append_n(const Geom &g, const void *Kn, const void *Vn, const uint8_t *pn, void *Kcache,
                                        void *Vcache, uint8_t *pcache, int32_t *clen, float *Kc, hipStream_t s) {
  timing_begin("phsa_cache_append", s);
  hipLaunchKernelGGL((cache_append_kernel<T, D, NTHR>), dim3(g.B), dim3(NTHR), 0, s, static_cast<const T *>(Kn),
                     static_cast<const T *>(Vn), pn, static_cast<T *>(Kcache), static_cast<T *>(Vcache), pcache, clen,
                     Kc, g);
  timing_end(s);
  return hipGetLastError();
}

template <typename T, int D>
static hipError_t launch_cache_append_t(const Geom &g, const void *Kn, const void *Vn, const uint8_t *pn, void *Kcache,
                                        void *Vcache, uint8_t *pcache, int32_t *clen, float *Kc, hipStream_t s) {
  // 1024 threads up to one workgroup per CU, where a completed block's chain is the
  // call; more workgroups wait for each other's waves and LDS (64 KB at 1024
  // threads), and most of them only copy a row.  1024 | 512 | 256 threads, 8 heads
  // of 128 in 64-token blocks, no block completed / ragged lengths / every block
  // completed: 256 sequences 4.3 / 7.8 / 9.0 | 4.3 / 7.7 / 9.0 | 4.1 / 9.8 / 11.1 us
  // (32 heads: 15.3 | 16.6 | 26.1 ragged), 512 5.2 / 9.0 / 18.5 | 4.7 / 8.1 / 15.8 |
  // 4.6 / 9.9 / 16.0, 2048 10.3 / 14.1 / 60 | 7.1 / 11.3 / 48 | 5.9 / 11.8 / 48; 2 heads
  // of 64, 4096 sequences 15.3 / 20.5 / 89.5 | 8.8 / 11.2 / 28.2 | 6.4 / 8.1 / 17.4.
  if (g.B <= 256) return launch_cache_append_n<T, D, 1024>(g, Kn, Vn, pn, Kcache, Vcache, pcache, clen, Kc, s);
  if (g.B <= 512) return launch_cache_append_n<T, D, 512>(g, Kn, Vn, pn, Kcache, Vcache, pcache, clen, Kc, s);
  return launch_cache_append_n<T, D, 256>(g, Kn, Vn, pn, Kcache, Vcache, pcache, clen, Kc, s);
}

hipError_t launch_cache_append(const Geom &g, const void *Kn, const void *Vn, const uint8_t *pn, void *Kcache,
                               void *Vcache, uint8_t *pcache, int32_t *clen, float *Kc, hipStream_t s) {
  if (g.dtype == 0)
    return g.d == 128 ? launch_cache_append_t<bf16_t, 128>(g, Kn, Vn, pn, Kcache, Vcache, pcache, clen, Kc, s)
                      : launch_cache_append_t<bf16_t, 64>(g, Kn, Vn, pn, Kcache, Vcache, pcache, clen, Kc, s);
  return g.d == 128 ? launch_cache_append_t<float, 128>(g, Kn, Vn, pn, Kcache, Vcache, pcache, clen, Kc, s)
                    : launch_cache_append_t<float, 64>(g, Kn, Vn, pn, Kcache, Vcache, pcache, clen, Kc, s);
}

hipError_t launch_decode(const Geom &g, const void *Q, const void *K, const void *V, const float *Kc,
                         const int32_t *clen, int32_t *sel, void *O, float *LSE, hipStream_t s) {
  const DecodeArgs a{Q, K, V, Kc, clen, sel, O, LSE};
  if (g.dtype == 0) return g.d == 128 ? launch_decode_t<bf16_t, 128>(g, a, s) : launch_decode_t<bf16_t, 64>(g, a, s);
  return g.d == 128 ? launch_decode_t<float, 128>(g, a, s) : launch_decode_t<float, 64>(g, a, s);
}

}  // namespace phsa
