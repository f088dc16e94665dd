// Inverted selection index: for every (b, g, block t) the ascending list of
// query rows whose selection contains t (the transpose of sel), plus a table
// of attention work units (a unit = one block and up to unit_tokens entries of
// its list).  This lets the attention kernels run key-block-major: one K/V
// tile is loaded once and meets every query row that selected it.
//
// Entries are (row << 10) | (quarters << 6) | slot, where slot is the
// position of t among the row's entries (its sel vector, for 64-token blocks)
// and quarters is a 4-bit mask of the 16-key quarters of t the row attends
// to (all four for 64-token blocks).  The attention kernels store per-entry
// partial results in list order (contiguous per work unit); pmap[(row, slot)]
// = list position lets the per-row merges find them.
//
// Selections of m = 16 or 32 tokens, and rows whose local window goes to the
// band kernels, are indexed on 64-key tiles: the m-token blocks a row selected
// are grouped by the tile that holds them (tile = block / (64 / m)), and each
// tile entry carries the mask of the 16-key quarters its blocks cover.  The
// regrouping happens as the rows are read (row_entries), so the index is
// keyed by the tile geometry gm (m = 64, T = Lk / 64, ksel = min(Ksel, T) plus
// the band slot) while sel keeps its own width (the selection's Ksel).
//
// Integer-only passes, all deterministic (no order depends on timing):
//   count : per 256-row tile, an LDS bitmap [8 words][T] of who selected
//           what; popcounts give per-tile counts cntw[bg][w][t].
//   scan  : one workgroup per bg: per t the exclusive prefix over tiles -> toff,
//           over t the list and unit offsets and the unit tables (with few
//           counts the fill's workgroups do this themselves).
//   fill  : rebuilds the tile bitmap; an entry's place in its list is
//           tile offset + number of lower rows in the tile that chose t.
#include <type_traits>

#include "common.h"
#include "launch.h"

namespace phsa {

__device__ __forceinline__ bool slot_valid(int t, int cur, int T) { return t >= 0 && t <= cur && t < T; }

// Width of a sel row: the selection's own Ksel (in its block units).
__device__ __forceinline__ int sel_width(const Geom &gm) { return gm.n_init + gm.window / gm.sm + 1 + gm.top_k; }

// A selection whose blocks are the index's own: a row's entries are the valid
// prefix of its sel row (ascending causal blocks, ended by -1 or a block past
// the query's own), less its forced blocks when the band takes them (then one
// thread per row; without a band by (row, slot) pairs).
__device__ __forceinline__ bool plain_rows(const Geom &gm) { return gm.sm == gm.m; }

// The forced blocks of Algorithm 1 for the query in block cur: the init blocks
// 0 .. ninit - 1 and the local window a_blk .. cur (a_blk >= ninit, so the
// two ranges are disjoint; both in selection blocks).  With the band, a row
// that holds all of them leaves them to the band kernels.
struct Forced {
  int ninit, a_blk, count;
  // wblk: the window in selection blocks (gm.window / gm.sm)
  __device__ __forceinline__ Forced(const Geom &gm, int cur, int wblk) {
    ninit = min(gm.n_init, cur + 1);
    a_blk = max(max(0, cur - wblk), ninit);
    count = ninit + cur - a_blk + 1;
  }
  __device__ __forceinline__ Forced(const Geom &gm, int cur) : Forced(gm, cur, gm.window / gm.sm) {}
  __device__ __forceinline__ bool has(int t) const { return t < ninit || t >= a_blk; }
};

// Selection block sizes of the attention entry points are 16, 32 or 64
// tokens, so the regrouping divides by shifts: sh = log2(sm), and a 64-key
// tile holds 64 >> sh blocks.  All fields are wave-uniform.
struct BlockShift {
  int sh, per_sh, qpb, wblk, nblk;
  __device__ __forceinline__ explicit BlockShift(const Geom &gm) {
    sh = __builtin_ctz((unsigned)gm.sm);
    per_sh = 6 - sh;
    qpb = gm.sm >> 4;
    wblk = gm.window >> sh;
    nblk = gm.Lk >> sh;
  }
};

// The regrouped entries of one row, one wave per row with lane s holding slot
// s of sel (t = that slot's block, -1 past the row's width).  A row's blocks
// are ascending, so a tile's blocks sit in adjacent lanes; a tile's first lane
// takes its slot by a ballot prefix count and ORs the quarters of the (at most
// 64 / m) lanes of its group.  With gm.band, a row holding every local block
// outside the init blocks (a_blk .. cur) leaves them to the band kernels
// (band_ok) together with its init blocks; other rows keep all their blocks.  A lane with `mine` set holds
// entry `pos` of the row: tile `tile` with quarter mask `qm`; n entries in all.
struct RowEntries {
  int tile;
  unsigned qm;
  int pos;
  int n;
  bool mine;
  bool band_ok;
};

// Whole-wave DPP shifts by one lane: lane i reads lane i - 1 (wave_shr:1) or
// lane i + 1 (wave_shl:1); a lane whose source is outside the wave reads 0.
__device__ __forceinline__ int from_lane_below(int v) {
  return __builtin_amdgcn_update_dpp(0, v, 0x138, 0xF, 0xF, true);
}
__device__ __forceinline__ int from_lane_above(int v) {
  return __builtin_amdgcn_update_dpp(0, v, 0x130, 0xF, 0xF, true);
}

// i: the row (wave-uniform).
__device__ __forceinline__ RowEntries row_entries(int t, int i, const Geom &gm, const BlockShift &bs) {
  const int lane = threadIdx.x & 63;
  RowEntries e;
  e.band_ok = false;
  const int cur = (gm.q_pos0 + i) >> bs.sh;
  const int per = 1 << bs.per_sh, qpb = bs.qpb;
  const bool in_range = t >= 0 && t <= cur && t < bs.nblk;
  const Forced f(gm, cur, bs.wblk);
  if (gm.band) e.band_ok = __popcll(__ballot(in_range && f.has(t))) == f.count;
  const bool valid = in_range && !(e.band_ok && f.has(t));
  const int tc = valid ? t >> bs.per_sh : -1;
  const unsigned qb = valid ? ((1u << qpb) - 1u) << ((t & (per - 1)) * qpb) : 0u;
  const int prev = from_lane_below(tc);
  const bool first = valid && (lane == 0 || prev != tc);
  const uint64_t heads = __ballot(first);
  e.pos = bits_below(heads);
  e.n = __popcll(heads);
  unsigned acc = qb;
  int oq = (int)qb, otc = tc;  // the values of lane + dd
  for (int dd = 1; dd < per; ++dd) {
    oq = from_lane_above(oq);
    otc = from_lane_above(otc);
    if (lane + dd < 64 && otc == tc) acc |= (unsigned)oq;
  }
  e.mine = first && e.pos < gm.ksel - gm.band;
  e.tile = tc;
  e.qm = acc;
  return e;
}

// Sel rows a wave loads at once (regrouped rows), waited for together.  The
// fill stores as it goes, and loads and stores share one wait counter, so a
// load issued after a store cannot be waited for alone: each batch waits once
// for the previous batch's stores, not once per row.
constexpr int kRowBatch = 16;

// A plain row (one thread, its sel row staged at row[0 .. ks)) with the band:
// does it hold every forced block?
__device__ __forceinline__ bool plain_band_ok(const int32_t *row, int ks, int cur, const Geom &gm) {
  if (!gm.band) return false;
  const Forced f(gm, cur);
  int have = 0;
  for (int s = 0; s < ks; ++s) {
    const int t = row[s];
    if (!slot_valid(t, cur, gm.T)) break;
    have += f.has(t);
  }
  return have == f.count;
}

// The bitmap bm [8][T] of the 256-row tile w of (b, g) = bg: bit r % 32 of
// bm[r / 32][t] is set when row r has an entry for t.  Plain rows: the tile's
// sel rows, one contiguous run, are staged into rows_s ([kIndexTile][Ksel])
// with coalesced loads and each thread walks its row.  Regrouped rows: wave v
// takes rows 64v .. 64v + 63, one row per pass with its slots across the
// lanes (word-major bm, so a row's lanes, each on another t, hit different
// banks).  Every thread calls this (it holds barriers).
__device__ void build_tile_bitmap(uint32_t *bm, int32_t *rows_s, const int32_t *__restrict__ sel, const Geom &gm,
                                  int bg, int w) {
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int ks = sel_width(gm);
  const int nrow = min(kIndexTile, gm.Lq - w * kIndexTile);
  const int64_t row0 = (int64_t)bg * gm.Lq + (int64_t)w * kIndexTile;
  for (int x = tid; x < gm.T * 8; x += 256) bm[x] = 0u;
  if (plain_rows(gm)) {
    const int32_t *src = sel + row0 * ks;
    for (int x = tid; x < nrow * ks; x += 256) rows_s[x] = src[x];
    __syncthreads();
    if (tid < nrow) {
      const int cur = (gm.q_pos0 + w * kIndexTile + tid) / gm.m;
      const bool bok = plain_band_ok(rows_s + tid * ks, ks, cur, gm);
      const Forced f(gm, cur);
      for (int s = 0; s < ks; ++s) {
        const int t = rows_s[tid * ks + s];
        if (!slot_valid(t, cur, gm.T)) break;
        if (!(bok && f.has(t))) atomicOr(&bm[(tid >> 5) * gm.T + t], 1u << (tid & 31));
      }
    }
    __syncthreads();
    return;
  }
  __syncthreads();
  const BlockShift bs(gm);
  for (int j0 = 0; j0 < 64; j0 += kRowBatch) {
    int t[kRowBatch];
#pragma unroll
    for (int u = 0; u < kRowBatch; ++u) {
      const int r = wave * 64 + j0 + u;
      t[u] = (r < nrow && lane < ks) ? sel[(row0 + r) * ks + lane] : -1;
    }
#pragma unroll
    for (int u = 0; u < kRowBatch; ++u) {
      const int r = wave * 64 + j0 + u;
      if (r < nrow) {  // wave-uniform
        const RowEntries e = row_entries(t[u], w * kIndexTile + r, gm, bs);
        if (e.mine) atomicOr(&bm[(r >> 5) * gm.T + e.tile], 1u << (r & 31));
      }
    }
  }
  __syncthreads();
}

// LDS of the count kernel (the fill kernel adds one list position per t).
// Plain rows stage their sel rows (width Ksel, in selection blocks) and, in
// the fill kernel, one band flag per row after them.
inline size_t index_lds_bytes(const Geom &g) {
  const bool plain = g.sm == g.m;
  const int ks = g.n_init + g.window / g.sm + 1 + g.top_k;
  return (size_t)g.T * 8 * sizeof(uint32_t) + (plain ? (size_t)kIndexTile * (ks + 1) * sizeof(int32_t) : 0);
}

__global__ __launch_bounds__(256) void index_count_kernel(const int32_t *__restrict__ sel, Geom gm, IndexWs ix) {
  extern __shared__ uint32_t bm[];
  const int w = blockIdx.x, bg = blockIdx.y;
  build_tile_bitmap(bm, reinterpret_cast<int32_t *>(bm + 8 * gm.T), sel, gm, bg, w);
  int32_t *dst = ix.cntw + ((int64_t)bg * ix.W + w) * gm.T;
  for (int t = threadIdx.x; t < gm.T; t += 256) {
    int c = 0;
#pragma unroll
    for (int k = 0; k < 8; ++k) c += __popc(bm[k * gm.T + t]);
    dst[t] = c;
  }
}

// The scans over t.  For a list of c entries: nu = ceil(c / unit_tokens)
// backward units, the flag f = (nu != 1) of the blocks whose dK/dV the
// finalize writes (from partial sums, or zeros for an empty list), and nf
// forward units.
struct ListCounts {
  int c, nu, f, nf;
  __device__ __forceinline__ void add(const ListCounts &o) {
    c += o.c;
    nu += o.nu;
    f += o.f;
    nf += o.nf;
  }
};

constexpr int kScanThreads = 512;

// Exclusive scan of v over a workgroup of kScanThreads (each field on its own);
// tot receives the workgroup's sums.  Holds barriers.
__device__ __forceinline__ ListCounts block_scan(ListCounts v, ListCounts &tot) {
  constexpr int NW = kScanThreads / 64;
  __shared__ ListCounts wsum_s[NW];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  ListCounts inc = v;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const ListCounts o{__shfl_up(inc.c, d, 64), __shfl_up(inc.nu, d, 64), __shfl_up(inc.f, d, 64),
                       __shfl_up(inc.nf, d, 64)};
    if (lane >= d) inc.add(o);
  }
  if (lane == 63) wsum_s[wave] = inc;
  __syncthreads();
  ListCounts pre{0, 0, 0, 0};
  tot = ListCounts{0, 0, 0, 0};
#pragma unroll
  for (int w = 0; w < NW; ++w) {
    const ListCounts s = wsum_s[w];
    if (w < wave) pre.add(s);
    tot.add(s);
  }
  __syncthreads();  // wsum_s may be reused by the caller's next scan
  return ListCounts{pre.c + inc.c - v.c, pre.nu + inc.nu - v.nu, pre.f + inc.f - v.f, pre.nf + inc.nf - v.nf};
}

// The lists of one bg, by a workgroup: per t the exclusive prefix of the tile
// counts, then over t the list offsets, the unit tables and the finalize list.
// Every bg keeps its lists and units in regions of its own, so no prefix crosses
// bg.  tp (a power of two) threads cover the blocks; with few blocks the
// kScanThreads / tp thread groups share the tiles.
//   base_s null: writes the tile prefixes (toff), the list offsets and the tables.
//   base_s given: base_s[t] = list position of the first entry of tile w_own; the
//                 tables are written by the workgroup of tile 0 alone.
__device__ __forceinline__ void scan_lists(const Geom &gm, const IndexWs &ix, int bg, int tp, int w_own, int32_t *base_s) {
  __shared__ int part_s[kScanThreads];
  const int tid = threadIdx.x;
  const bool tables = !base_s || w_own == 0;
  const int32_t *cw = ix.cntw + (int64_t)bg * ix.W * gm.T;
  int32_t *to = ix.toff + (int64_t)bg * ix.W * gm.T;
  int2 *fu = ix.funits + (int64_t)bg * ix.funits_bg;
  int4 *un = ix.units + (int64_t)bg * ix.units_bg;
  const int ng = kScanThreads / tp, grp = tid / tp;  // tile groups, this thread's
  const int wper = (ix.W + ng - 1) / ng, w0 = min(grp * wper, ix.W), w1 = min(w0 + wper, ix.W);
  ListCounts carry{(int)((int64_t)bg * gm.Lq * (gm.ksel - gm.band)), 0, 0, 0};  // first list position of this bg
  constexpr int U = 32;
  for (int t0 = 0; t0 < gm.T; t0 += tp) {
    const int t = t0 + tid % tp;
    const int tc = min(t, gm.T - 1);
    // counts of the group's tiles; a batch is loaded before its prefixes are
    // stored (a load behind a store waits for the store too)
    int run = 0;
    if (ng > 1) {
      for (int w = w0; w < w1; w += U) {
        int c[U];
#pragma unroll
        for (int u = 0; u < U; ++u) c[u] = cw[(int64_t)min(w + u, w1 - 1) * gm.T + tc];
#pragma unroll
        for (int u = 0; u < U; ++u) run += w + u < w1 ? c[u] : 0;
      }
      __syncthreads();
      part_s[tid] = run;
      __syncthreads();
      run = 0;
      for (int x = 0; x < grp; ++x) run += part_s[x * tp + tid % tp];
    }
    for (int w = w0; w < w1; w += U) {
      int c[U];
#pragma unroll
      for (int u = 0; u < U; ++u) c[u] = cw[(int64_t)min(w + u, w1 - 1) * gm.T + tc];
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (w + u < w1) {
          if (t < gm.T) {
            if (!base_s) to[(int64_t)(w + u) * gm.T + t] = run;
            else if (w + u == w_own) base_s[t] = run;
          }
          run += c[u];
        }
    }
    // list lengths: the last group's running sums, taken by the first tp threads
    if (ng > 1) {
      __syncthreads();
      if (grp == ng - 1) part_s[tid % tp] = run;
      __syncthreads();
      run = part_s[tid % tp];
    }
    const bool live = grp == 0 && t < gm.T;
    if (!live) run = 0;
    const int nu = (run + ix.unit_tokens - 1) / ix.unit_tokens, nf = (run + ix.fpart - 1) / ix.fpart;
    const ListCounts v{run, nu, live && nu != 1 ? 1 : 0, nf};
    ListCounts tot, at = block_scan(v, tot);
    at.add(carry);
    if (live) {
      const int x = bg * gm.T + t;
      if (base_s) base_s[t] += at.c;  // written above by another group: the scan's barriers lie between
      else ix.off[x] = at.c;
      if (tables) {
        ix.uoff[(int64_t)bg * (gm.T + 1) + t] = at.nu;
        for (int u = 0; u < nu; ++u)
          un[at.nu + u] =
              make_int4(x, min(ix.unit_tokens, run - u * ix.unit_tokens), at.c + u * ix.unit_tokens, nu == 1 ? 1 : 0);
        if (v.f) ix.fin[(int64_t)bg * gm.T + at.f] = x;
        for (int u = 0; u < nf; ++u)
          fu[at.nf + u] = make_int2((t << 16) | min(ix.fpart, run - u * ix.fpart), at.c + u * ix.fpart);
      }
    }
    carry.add(tot);
  }
  if (tid == 0 && tables) {
    ix.uoff[(int64_t)bg * (gm.T + 1) + gm.T] = carry.nu;
    ix.ucnt[bg] = carry.nu;
    ix.nfin[bg] = carry.f;
    ix.fcnt[bg] = carry.nf;
  }
}

__global__ __launch_bounds__(kScanThreads) void index_scan_kernel(Geom gm, IndexWs ix, int tp) {
  scan_lists(gm, ix, blockIdx.x, tp, 0, nullptr);
}

// ---- selections whose blocks are the index's own (64-token blocks without a
// band, float32): kScanThreads threads per 256-row tile take the tile's (row,
// slot) pairs, each pair on its own.  A row's entries are the valid prefix of
// its sel row; bad_s[r] is the first slot past it.  float32 rows (EVERY) keep
// each valid slot, as the row-major float32 kernels do; a block listed more than
// once is one entry that counts its copies.  (One thread per row walking
// its slots took 12 + 20 us for count and fill at 8k tokens and 49 + 85 at 4 x 32k,
// against 8.5 + 13.7 and 31 + 76; events.)

// The row of pair x (x / ks, by the reciprocal inv = ceil(2^32 / ks); x < 2^14).
__device__ __forceinline__ int pair_row(int x, int ks, uint32_t inv) { return ks == 1 ? x : (int)__umulhi((uint32_t)x, inv); }

// Stages the tile's sel rows, finds bad_s and sets the tile's bitmap bm [8][T].
// EVERY (float32): an invalid slot is staged as -1 and bad_s stays ks; *twice_s is
// set when a row lists a block more than once.  (Chosen at run time it cost the
// fill of a small bf16 call 0.8 of 12 us.)
template <bool EVERY>
__device__ __forceinline__ void pair_bitmap(uint32_t *bm, int32_t *rows_s, int *bad_s, int *twice_s,
                                            const int32_t *__restrict__ sel, const Geom &gm, int ks, uint32_t inv,
                                            int bg, int w) {
  const int tid = threadIdx.x, msh = __builtin_ctz((unsigned)gm.m);
  const int nrow = min(kIndexTile, gm.Lq - w * kIndexTile), n = nrow * ks;
  const int32_t *src = sel + ((int64_t)bg * gm.Lq + (int64_t)w * kIndexTile) * ks;
  for (int x = tid; x < gm.T * 8; x += kScanThreads) bm[x] = 0u;
  if (tid < kIndexTile) bad_s[tid] = ks;
  if (EVERY && tid == 0) *twice_s = 0;
  __syncthreads();
  for (int x = tid; x < n; x += kScanThreads) {
    const int r = pair_row(x, ks, inv), t = src[x];
    const bool ok = slot_valid(t, (gm.q_pos0 + w * kIndexTile + r) >> msh, gm.T);
    rows_s[x] = ok || !EVERY ? t : -1;
    if (!ok && !EVERY) atomicMin(&bad_s[r], x - r * ks);
  }
  __syncthreads();
  for (int x = tid; x < n; x += kScanThreads) {
    const int r = pair_row(x, ks, inv), t = rows_s[x];
    if (EVERY ? t < 0 : x - r * ks >= bad_s[r]) continue;
    uint32_t *word = &bm[(r >> 5) * gm.T + t];
    if (!EVERY) atomicOr(word, 1u << (r & 31));
    else if (atomicOr(word, 1u << (r & 31)) >> (r & 31) & 1u) *twice_s = 1;
  }
  __syncthreads();
}

template <bool EVERY>
__global__ __launch_bounds__(kScanThreads) void index_count_pairs_kernel(const int32_t *__restrict__ sel, Geom gm,
                                                                         IndexWs ix, uint32_t inv) {
  extern __shared__ uint32_t bm[];
  __shared__ int bad_s[kIndexTile], twice_s;
  const int w = blockIdx.x, bg = blockIdx.y;
  pair_bitmap<EVERY>(bm, reinterpret_cast<int32_t *>(bm + 8 * gm.T), bad_s, &twice_s, sel, gm, gm.ksel, inv, bg, w);
  int32_t *dst = ix.cntw + ((int64_t)bg * ix.W + w) * gm.T;
  for (int t = threadIdx.x; t < gm.T; t += kScanThreads) {
    int c = 0;
#pragma unroll
    for (int k = 0; k < 8; ++k) c += __popc(bm[k * gm.T + t]);
    dst[t] = c;
  }
}

// SCAN: every workgroup sums the tile counts itself instead of reading a scan
// kernel's prefixes (one launch less; launch_build_index has the rule).
template <bool SCAN, bool EVERY>
__global__ __launch_bounds__(kScanThreads) void index_fill_pairs_kernel(const int32_t *__restrict__ sel, Geom gm,
                                                                        IndexWs ix, uint32_t inv, int tp) {
  extern __shared__ uint32_t bm[];
  __shared__ int bad_s[kIndexTile], twice_s;
  uint64_t *pre_s = reinterpret_cast<uint64_t *>(bm + 8 * gm.T);
  int32_t *base_s = reinterpret_cast<int32_t *>(pre_s + gm.T);
  int32_t *rows_s = base_s + gm.T;
  // neighbouring tiles write adjacent runs of the same lists: one XCD takes a
  // contiguous range of (bg, w), so a list's cache lines go through one L2
  const int logical = xcd_item(blockIdx.x + blockIdx.y * gridDim.x, gridDim.x * gridDim.y);
  const int w = logical % gridDim.x, bg = logical / gridDim.x, tid = threadIdx.x, ks = gm.ksel;
  if (SCAN) {
    scan_lists(gm, ix, bg, tp, w, base_s);
  } else {
    const int32_t *tile_off = ix.toff + ((int64_t)bg * ix.W + w) * gm.T;
    const int32_t *list_off = ix.off + (int64_t)bg * gm.T;
    for (int t = tid; t < gm.T; t += kScanThreads) base_s[t] = list_off[t] + tile_off[t];
  }
  pair_bitmap<EVERY>(bm, rows_s, bad_s, &twice_s, sel, gm, ks, inv, bg, w);  // its barriers also publish base_s
  for (int t = tid; t < gm.T; t += kScanThreads) {
    uint64_t pre = 0;
    int run = 0;  // at most 7 x 32 = 224 rows below the last word
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      pre |= (uint64_t)run << (8 * k);
      run += __popc(bm[k * gm.T + t]);
    }
    pre_s[t] = pre;
  }
  __syncthreads();
  const int n = min(kIndexTile, gm.Lq - w * kIndexTile) * ks;
  int32_t *pm = ix.pmap + ((int64_t)bg * gm.Lq + (int64_t)w * kIndexTile) * ks;
  for (int x = tid; x < n; x += kScanThreads) {
    const int r = pair_row(x, ks, inv), s = x - r * ks, t = rows_s[x];
    int p = -1;
    if (EVERY ? t >= 0 : s < bad_s[r]) {
      const int word = r >> 5;
      // lower rows of the tile that chose t: those of the lower words (a byte of pre_s) and of its own
      const uint32_t lower = reinterpret_cast<const uint8_t *>(&pre_s[t])[word];
      p = base_s[t] + (int)lower + __popc(bm[word * gm.T + t] & ((1u << (r & 31)) - 1u));
      int low = s;
      if (EVERY) {  // the slot is not used: further copies of the block in the row
        low = 0;
        if (twice_s)
          for (int y = r * ks; y < (r + 1) * ks; ++y) low += y != x && rows_s[y] == t;
      }
      ix.tok[p] = ((w * kIndexTile + r) << 10) | (15 << 6) | low;
    }
    pm[x] = p;
  }
}

// Writes each row's entries into their lists, its position-map row (list
// position per slot, -1 for empty slots, the band partial in the slot after the entries of
// a band row) and, with the band, its band flag.  The tile's first list
// position for each t (list offset + tile offset) is staged in LDS beside the
// bitmap; an entry's position adds the lower rows of the tile that chose t:
// the set bits of its own bitmap word below it plus those of the lower words,
// whose counts are staged per t as eight bytes (byte k: words 0 .. k - 1).
__global__ __launch_bounds__(256) void index_fill_kernel(const int32_t *__restrict__ sel, Geom gm, IndexWs ix) {
  extern __shared__ uint32_t bm[];
  uint64_t *pre_s = reinterpret_cast<uint64_t *>(bm + 8 * gm.T);
  int32_t *base_s = reinterpret_cast<int32_t *>(pre_s + gm.T);
  int32_t *rows_s = base_s + gm.T;  // plain rows: staged sel rows, then their list positions
  // Query tiles w, w + 1 of one (b, g) write adjacent runs of the same lists.
  // Workgroups are dealt to the 8 XCDs in turn (each XCD its own L2), so the
  // grid is renumbered to give each XCD one contiguous range of (bg, w): a
  // list's cache lines are then written through one L2.
  const int logical = xcd_item(blockIdx.x + blockIdx.y * gridDim.x, gridDim.x * gridDim.y);
  const int w = logical % gridDim.x, bg = logical / gridDim.x, tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int32_t *tile_off = ix.toff + ((int64_t)bg * ix.W + w) * gm.T;
  const int32_t *list_off = ix.off + (int64_t)bg * gm.T;
  for (int t = tid; t < gm.T; t += 256) base_s[t] = list_off[t] + tile_off[t];
  build_tile_bitmap(bm, rows_s, sel, gm, bg, w);  // its barriers also publish base_s
  for (int t = tid; t < gm.T; t += 256) {
    uint64_t pre = 0;
    int run = 0;  // at most 7 x 32 = 224 rows below the last word
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      pre |= (uint64_t)run << (8 * k);
      run += __popc(bm[k * gm.T + t]);
    }
    pre_s[t] = pre;
  }
  __syncthreads();
  // rows of the tile below row r (word r / 32, bit r % 32) that chose t
  auto rank_of = [&](int t, int r) {
    const int word = r >> 5;
    return (int)reinterpret_cast<const uint8_t *>(&pre_s[t])[word] + __popc(bm[word * gm.T + t] & ((1u << (r & 31)) - 1u));
  };
  const int ks = sel_width(gm);
  const int nrow = min(kIndexTile, gm.Lq - w * kIndexTile);
  const int64_t row0 = (int64_t)bg * gm.Lq + (int64_t)w * kIndexTile;
  if (plain_rows(gm)) {
    // entries take slots 0 .. n - 1 of the row's position-map row and the band
    // partial of a band row slot n, so that the merges' slot bound stays at the
    // row's own partial count; flag_s holds that slot (-1: no band partial)
    int32_t *flag_s = rows_s + kIndexTile * ks;
    const int i = w * kIndexTile + tid;
    if (tid < nrow) {
      const int cur = (gm.q_pos0 + i) / gm.m;
      const bool bok = plain_band_ok(rows_s + tid * ks, ks, cur, gm);
      const Forced f(gm, cur);
      int n = 0;
      for (int s = 0; s < ks; ++s) {  // the valid prefix, less the band's blocks
        const int t = rows_s[tid * ks + s];
        if (!slot_valid(t, cur, gm.T)) break;
        if (bok && f.has(t)) continue;
        const int32_t p = base_s[t] + rank_of(t, tid);
        ix.tok[p] = (i << 10) | (15 << 6) | n;
        rows_s[tid * ks + n] = p;  // n <= s: the slots still to be read are above
        ++n;
      }
      for (int s = n; s < ks; ++s) rows_s[tid * ks + s] = -1;
      flag_s[tid] = bok ? n : -1;
    }
    __syncthreads();
    // the tile's rows are consecutive, so their position-map rows form one contiguous run
    const int ksel = gm.ksel, nsp = ksel - gm.band;  // nsp <= ks slots for entries
    int32_t *dst = ix.pmap + row0 * ksel;
    for (int x = tid; x < nrow * ksel; x += 256) {
      const int r = x / ksel, s = x - r * ksel;
      dst[x] = s == flag_s[r] ? (int32_t)(ix.band_base + row0 + r) : s < nsp ? rows_s[r * ks + s] : -1;
    }
    if (gm.band && tid < nrow) ix.bflag[row0 + tid] = (uint8_t)(flag_s[tid] >= 0);
    return;
  }
  unsigned flag = 0;  // band flag of row 64 * wave + lane
  const BlockShift bs(gm);
  for (int j0 = 0; j0 < 64; j0 += kRowBatch) {
    int t[kRowBatch];
#pragma unroll
    for (int u = 0; u < kRowBatch; ++u) {
      const int r = wave * 64 + j0 + u;
      t[u] = (r < nrow && lane < ks) ? sel[(row0 + r) * ks + lane] : -1;
    }
    // one wait for the whole batch here, before any branch: an (empty) use of
    // every loaded value, so that no row below waits on the stores again
#pragma unroll
    for (int u = 0; u < kRowBatch; ++u) asm volatile("" ::"v"(t[u]));
#pragma unroll
    for (int u = 0; u < kRowBatch; ++u) {
      const int r = wave * 64 + j0 + u;
      if (r >= nrow) continue;  // wave-uniform
      const int i = w * kIndexTile + r;
      const int64_t x = row0 + r;
      const RowEntries e = row_entries(t[u], i, gm, bs);
      int32_t p = -1;
      if (e.mine) {
        p = base_s[e.tile] + rank_of(e.tile, r);
        ix.tok[p] = (i << 10) | ((int)(e.qm & 15u) << 6) | e.pos;
      }
      // entry pos's list position moves to lane pos (a lane below n has exactly
      // one sender; the others send to lane 63, which is below n only when all
      // 64 lanes are entries), so the row's position-map row is one store
      const int moved = __builtin_amdgcn_ds_permute((e.mine ? e.pos : 63) << 2, p);
      if (lane < gm.ksel)
        ix.pmap[x * gm.ksel + lane] =
            lane < e.n ? moved : (gm.band && e.band_ok && lane == e.n) ? (int32_t)(ix.band_base + x) : -1;
      if (lane == j0 + u) flag = e.band_ok ? 1u : 0u;
    }
  }
  if (gm.band && wave * 64 + lane < nrow) ix.bflag[row0 + wave * 64 + lane] = (uint8_t)flag;
}

hipError_t launch_build_index(const Geom &g, const int32_t *sel, const IndexWs &ix, hipStream_t s) {
  // Each launch's status is taken right after it: the attention kernels gather
  // through these lists, so a failed pass must stop the chain before them.
  hipError_t e;
  int tp = 64;
  while (tp < g.T && tp < kScanThreads) tp *= 2;
  const dim3 tiles(ix.W, g.B * g.Hkv);
  if (g.sm == g.m && !g.band) {  // (row, slot) pairs
    const uint32_t inv = (uint32_t)(((1ull << 32) + g.ksel - 1) / g.ksel);  // pair_row
    const size_t lds = (size_t)g.T * 8 * sizeof(uint32_t) + (size_t)kIndexTile * g.ksel * sizeof(int32_t);
    const size_t lds_fill = lds + (size_t)g.T * (sizeof(int32_t) + sizeof(uint64_t));
    // The fill's workgroups sum the counts themselves while all of them are resident
    // at once (two per CU), so that each does it beside the others; further rounds
    // of them would each wait for theirs.  scan + fill as two launches against one,
    // R (b, g) x W tiles x T blocks: 8 x 64 x 256 (16k) 12 + 18 against 27 us, 16 x 32
    // x 128 28 against 26, 32 x 16 x 64 26 against 24, 4 x 128 x 512 38 against 37;
    // beyond 512 workgroups 32 x 32 x 128 34 against 42, 96 x 8 x 32 26 against 34, 8 x
    // 128 x 512 44 against 62, 96 x 64 x 256 119 against 213.  W * T bounds what a
    // workgroup reads (not measured beyond).
    const bool scan = (int64_t)g.B * g.Hkv * ix.W <= 512 && (int64_t)ix.W * g.T <= 65536;
    timing_begin("phsa_index_count", s);
    if (g.dtype == 0) hipLaunchKernelGGL(index_count_pairs_kernel<false>, tiles, dim3(kScanThreads), lds, s, sel, g, ix, inv);
    else hipLaunchKernelGGL(index_count_pairs_kernel<true>, tiles, dim3(kScanThreads), lds, s, sel, g, ix, inv);
    timing_end(s);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    if (!scan) {
      timing_begin("phsa_index_scan", s);
      hipLaunchKernelGGL(index_scan_kernel, dim3(g.B * g.Hkv), dim3(kScanThreads), 0, s, g, ix, tp);
      timing_end(s);
      if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    timing_begin("phsa_index_fill", s);
    auto fill = [&](auto scan_c, auto every_c) {
      hipLaunchKernelGGL((index_fill_pairs_kernel<decltype(scan_c)::value, decltype(every_c)::value>), tiles,
                         dim3(kScanThreads), lds_fill, s, sel, g, ix, inv, tp);
    };
    using Yes = std::true_type;
    using No = std::false_type;
    if (g.dtype == 0) scan ? fill(Yes{}, No{}) : fill(No{}, No{});
    else scan ? fill(Yes{}, Yes{}) : fill(No{}, Yes{});
    timing_end(s);
    return hipGetLastError();
  }
  const size_t lds = index_lds_bytes(g);
  timing_begin("phsa_index_count", s);
  hipLaunchKernelGGL(index_count_kernel, tiles, dim3(256), lds, s, sel, g, ix);
  timing_end(s);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  timing_begin("phsa_index_scan", s);
  hipLaunchKernelGGL(index_scan_kernel, dim3(g.B * g.Hkv), dim3(kScanThreads), 0, s, g, ix, tp);
  timing_end(s);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  timing_begin("phsa_index_fill", s);
  hipLaunchKernelGGL(index_fill_kernel, tiles, dim3(256), lds + (size_t)g.T * (sizeof(int32_t) + sizeof(uint64_t)), s,
                     sel, g, ix);
  timing_end(s);
  return hipGetLastError();
}

}  // namespace phsa
