// Flash block-sparse attention (paper Eq. (2), §3.3 optimisation (3)) on gfx950.
//
// One workgroup per query block (b, h, i); its kept K/V blocks are walked in list order
// in chunks of 32 keys (attn_walk.h). Work items are dealt to the 8 XCDs so that all XCDs
// share one head at a time; each XCD starts its rows of a head heaviest first
// (heavy_first).
//
// Data movement: each chunk's K and V rows go straight from HBM into LDS with 16-byte
// global_load_lds (no register staging) into a small ring, issued ahead of their use;
// completion is ordered by explicit waits and barriers.
//
// Math, transposed so every softmax statistic is per lane:
//   S^T (32 keys x 32 queries) = K * Q^T        v_mfma_f32_32x32x16_bf16, d/16 steps;
//     lane l then holds query row l%32 and 16 keys of the chunk.
//   O^T (d x 32 queries) += V^T * P^T           P^T straight from the S^T registers
//     (rounded to bf16) as the B operand; the contraction's key order follows the
//     accumulator layout, and ds_read_b64_tr_b16 delivers V^T fragments in that
//     order from row-major V.
// Softmax: logits are scaled into base 2 (one FMA + v_exp_f32 per element); the
// row max pairs lanes l and l^32 with v_permlane32_swap; the running max is only
// raised (and O rescaled) when some row's max grows by more than 2^8, so most
// chunks skip the 64-register rescale; row sums use bf16 dot2 on the same packed
// P that feeds the MFMA.
//
// What bounds it: with long lists the chip's power. At 1.6-1.7 GHz (2.4 when idle) the
// matrix pipes of a dense walk are busy about 60% of the cycles; a mix of just this step's
// MFMAs, vector work and LDS reads, without any loads from memory, ran at 1.3 PFLOP/s on the
// same card, the dense walk's padded rate is 1.05-1.1. Sparse lists stay 10-12% below that:
// busy 51% at 1.88 GHz, with 27% of the wave cycles in waits and barriers (57600 tokens, 24
// heads, a seventh of the pairs). Fewer instructions and LDS bytes per MFMA, and chunks
// without padding, are what helped both.
#include <climits>
#include <mutex>
#include <type_traits>

#include "attn_walk.h"
#include "spade_internal.h"

// Scratch of the allocation-free raster attention call: the head ranking's keys
// and order, 16 bytes per (batch, head) pair for at most spade::kMaxRankedHeads
// pairs (beyond that the launch runs in grid order and needs none). Each GPU holds
// its own copy until the process ends; host code reaches it only through the
// address hipGetSymbolAddress returns on that device.
static __device__ __align__(256) unsigned char scratch[spade::kNoAllocScratchBytes];

namespace spade {
namespace {

struct NoTable {};

// The work item of a workgroup: its geometry, (batch, head) pair, query block i
// (-1 for grid padding) and the source of its kept list.
// Workgroup w runs on XCD w % 8. Every XCD walks the heads in the same order
// and takes one contiguous eighth of each head's query blocks: the XCDs work
// on the same head at a time (its K/V stays in the MALL) and each XCD's L2
// serves spatially adjacent query blocks, whose kept K/V sets overlap.
// MULTI: the heads follow each other in the grid (per batch element), each
// padded to a multiple of 8 items, and are dealt to the XCDs the same way.
struct Item {
  DevGeom g;
  int64_t bh;
  int i;
  int cnt;  // its kept blocks, clamped to [0, NB]
  bool stream;  // its keys may be walked as one stream (WalkCursor)
  const int* list_src;
};

// Row of rank r among the n query blocks c[0..n) of one XCD's share of a head, ordered
// by kept-block count (descending, ties to the lower index) within windows of 64. The
// XCD's CUs then start its rows heaviest first: rows of similar length walk the key
// blocks at a similar pace, so the K/V blocks they share meet in the XCD's L2, and long
// rows do not form the tail. Any order is correct: each row is one work item.
// A radix selection over the window's counts, one ballot per bit: every wave of a workgroup
// does it before its first load, and ranking all 64 against each other took three times
// as long. *count: the row's kept blocks, clamped to [0, NB].
__device__ __forceinline__ int heavy_first(const int* __restrict__ c, int n, int r, int NB,
                                           int* count) {
  const int lane = int(threadIdx.x & 63);
  const int w0 = r & ~63, wn = min(64, n - w0);
  const int cl = min(max(c[w0 + min(lane, wn - 1)], 0), NB);
  uint64_t cand = wn == 64 ? ~uint64_t(0) : (uint64_t(1) << wn) - 1;
  int need = r - w0;  // rank within the candidates
  for (int b = 31 - __builtin_clz(uint32_t(NB)); b >= 0; --b) {
    const uint64_t ones = cand & __ballot((cl >> b) & 1);
    const int n1 = __popcll(ones);
    const bool in = need < n1;
    cand = in ? ones : cand & ~ones;
    need -= in ? 0 : n1;
  }
  // equal counts: the candidate of index `need`
  const int at = __builtin_amdgcn_mbcnt_hi(uint32_t(cand >> 32),
                                           __builtin_amdgcn_mbcnt_lo(uint32_t(cand), 0));
  const uint64_t hit = __ballot(at == need) & cand;
  const int row = __builtin_amdgcn_readfirstlane(int(__builtin_ctzll(hit)));
  *count = __builtin_amdgcn_readlane(cl, row);
  return w0 + row;
}

template <bool MULTI, class Tab>
__device__ __forceinline__ Item work_item(const DevGeom& g_arg, const int* counts,
                                          const int* indices, const int* order, const Tab& tab) {
  Item it;
  it.g = g_arg;
  if constexpr (MULTI) {
    const int b = int(blockIdx.x) / tab.items_per_batch;
    const int w = int(blockIdx.x) - b * tab.items_per_batch;
    int k = 0, start;
    if (order) {
      // ranked: order holds per batch element the launch's heads by rank, then
      // their ascending first items; the item's rank is the number of first
      // items <= w, minus one (one load per lane and a ballot, n_heads <= 64)
      const int n = tab.n_heads;
      const int* ranked = order + int64_t(b) * 2 * n;
      const int ln = int(threadIdx.x & 63);
      const int first = ln < n ? ranked[n + ln] : INT_MAX;
      const int r = __popcll(__ballot(first <= w)) - 1;
      k = __builtin_amdgcn_readfirstlane(ranked[r]);
      start = __builtin_amdgcn_readfirstlane(ranked[n + r]);
    } else {
      while (k + 1 < tab.n_heads && tab.head[k + 1].start <= w) ++k;
      start = tab.head[k].start;
    }
    const MultiHead& mh = tab.head[k];
    it.g = tab.geo[mh.geom];
    it.stream = (tab.streams >> mh.geom) & 1;
    const int local = w - start;  // same residue mod 8 as blockIdx.x
    const int per_xcd = (it.g.NB + 7) / 8;
    const int lo = (local & 7) * per_xcd, r = local >> 3;
    const int rows = min(per_xcd, it.g.NB - lo);
    if (r >= rows) {
      it.i = -1;
      return it;
    }
    const int* hc = mh.counts + int64_t(b) * mh.counts_bstride;
    it.i = lo + heavy_first(hc + lo, rows, r, it.g.NB, &it.cnt);
    it.bh = int64_t(b) * it.g.H + mh.h;
    it.list_src = mh.indices + int64_t(b) * mh.indices_bstride + int64_t(it.i) * it.g.NB;
  } else {
    const DevGeom& g = it.g;
    it.stream = true;  // the launch's own geometry decides
    const int per_xcd = (g.NB + 7) / 8;
    const int64_t slot = int64_t(blockIdx.x) >> 3;
    it.bh = slot / per_xcd;
    if (order) it.bh = order[it.bh];  // heads in the ranked order (heaviest first)
    const int lo = int(blockIdx.x & 7) * per_xcd, r = int(slot % per_xcd);
    const int rows = min(per_xcd, g.NB - lo);
    if (r >= rows) {  // grid padding when NB is not a multiple of 8
      it.i = -1;
      return it;
    }
    it.i = lo + heavy_first(counts + it.bh * g.NB + lo, rows, r, g.NB, &it.cnt);
    it.list_src = indices + (it.bh * g.NB + it.i) * int64_t(g.NB);
  }
  return it;
}

// Workgroups of W waves, wave w on query slots 32 w .. 32 w + 31 for the whole walk, two
// waves per SIMD (three at d = 64: 152..168 registers, and 2 spilled where three waves walk
// raster rows as a stream): 8 / W workgroups share a CU, so barriers of one are filled by
// another. The waves issue the DMA themselves, 1 / W of a chunk's loads each, from inside
// their steps.
// Rings of two K and two V tiles: in step c, after the sync in slot SY, K(c + 1) and
// V(c - 1) have been read by every wave (their reads are in slots <= NS / 2 - 1), so K(c +
// 3) and V(c + 1) are issued into their place; they are waited for at the next sync, a
// step later. Deeper rings were slower: at d = 128 the 4-tile kernel of 120-key blocks
// 27.5 ms with four tiles each against 26.7, 256-slot blocks 3.6 against 3.1 ms, and
// workgroups of one and two waves lose residency (64-token blocks of a small layer 0.57
// against 0.45 ms).
// Against one wave per tile without pipelining (three waves per SIMD, LDS read latency in
// every step): 120-slot blocks of a 75600-token, 40-head layer 29.7 -> 26.7 ms, 128-slot
// blocks 3.0 -> 2.6 ms, 256-slot blocks 3.6 -> 3.1 ms, at d = 64 128-slot blocks 3.1 ->
// 2.7 ms.
template <int D, int W>
struct WalkLayout {
  static constexpr int TILE = KvTile<D>::BYTES;
  static constexpr int V_OFF = 2 * TILE;
  static constexpr int TAB_OFF = 4 * TILE;
  static constexpr int LIST_OFF = TAB_OFF + 4 * W * 32 * 4;
  // kept-list entries staged at a time: few where LDS decides how many workgroups a CU holds
  static constexpr int SEG = W <= 2 ? 256 : 1024;
  static constexpr int BYTES = LIST_OFF + (SEG + 1) * 8;
  static constexpr int P2 = W >= 8 ? 8 : W >= 4 ? 4 : W >= 2 ? 2 : 1;
  static constexpr int PW = KvTile<D>::LOADS > P2 ? KvTile<D>::LOADS / P2 : 1;  // loads per tile, wave
  static constexpr int LW = KvTile<D>::LOADS / PW;                              // waves that load
  static constexpr int ROWS = PW > 1 ? 2 : 1;  // rows of a chunk whose offsets a lane needs
};

template <int D, int W, bool RASTER, bool STREAM>
__device__ __forceinline__ void row_tile_walk(const Item& it, const uint4* __restrict__ qb,
                                              const char* __restrict__ kb,
                                              const char* __restrict__ vb, float scale_log2,
                                              __bf16* __restrict__ ob, float* __restrict__ lse,
                                              char* smem_raw) {
  using KV = KvTile<D>;
  using LY = WalkLayout<D, W>;
  constexpr int NT = 64 * W;
  lds_char* const lds = (lds_char*)smem_raw;
  lds_int* const list = (lds_int*)(smem_raw + LY::LIST_OFF);

  const DevGeom g = it.g;
  const BlockExt e_i = block_ext(g, it.i);
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int q0 = wave * 32;
  const bool rows_live = q0 < e_i.n;
  const int64_t head_row = RASTER ? it.bh * g.N : it.bh * g.NB * int64_t(g.BS);
  const int64_t first_row = head_row + int64_t(it.i) * g.BS;  // blocked layout
  const int cnt = it.cnt;
  const int j0 = tid < min(cnt, LY::SEG) ? it.list_src[tid] : -1;  // in flight beside the tables
  TileState<D> x;
  load_q<D, RASTER>(g, e_i, qb, head_row, first_row, q0, x.qf);
  clear_tile(x);
  slot_tables<D, W, RASTER>(g, (lds_int*)(smem_raw + LY::TAB_OFF), tid, NT);

  const FragAddr fr(lane);
  // this wave's loads of a tile: wave * PW .. + PW - 1
  const bool loads = wave < LY::LW;
  const int first = wave * LY::PW;
  const char* const kbase = kb + head_row * KV::ROW + (first >> 1) * 64;
  const char* const vbase = vb + head_row * KV::ROW + (first >> 1) * 64;
  const uint32_t lds_load = uint32_t(reinterpret_cast<uintptr_t>(lds)) + first * 1024;
  const int lane_row = ((lane >> 2) + (LY::ROWS == 1 ? 16 * (wave & 1) : 0)) * 4;
  const uint32_t kx = k_piece(lane), dvx = v_piece(lane) - k_piece(lane);

  for (int seg = 0; seg < cnt; seg += LY::SEG) {
    const int ns = min(cnt - seg, LY::SEG);
    if (seg) __syncthreads();
    const Staged st = stage_list<D, RASTER, STREAM>(g, it.list_src + seg, ns, seg ? -2 : j0,
                                                    it.stream, list, tid, lane, NT);
    const int n = st.chunks;
    if (n == 0) continue;
    WalkCursor<LY::TAB_OFF, W, STREAM> cur(list, ns, st.stream);
    // a tile's loads of this wave, rows at byte offsets r (K pieces) of the head
    auto issue_k = [&](const uint32_t (&r)[2], int slot) {
      if (loads)
#pragma unroll
        for (int k = 0; k < LY::PW; ++k)
          tile_dma(kbase, r[k & (LY::ROWS - 1)], lds_load + slot * LY::TILE, k);
    };
    auto issue_v = [&](const uint32_t (&r)[2], int slot) {
      if (loads)
#pragma unroll
        for (int k = 0; k < LY::PW; ++k)
          tile_dma(vbase, r[k & (LY::ROWS - 1)] + dvx, lds_load + LY::V_OFF + slot * LY::TILE, k);
    };
    // Past the walk's end the cursor stays on the last chunk: the loads repeat it into
    // slots that are not read again, so the steps need no case for it.
    int t[2];
    uint32_t add[2];  // t + add: rows of the chunk the cursor is on
    auto rows_of = [&](uint32_t (&r)[2]) {
#pragma unroll
      for (int k = 0; k < LY::ROWS; ++k) r[k] = uint32_t(t[k]) + add[k];
    };
    int kv[5];                     // real keys of chunks c .. c + 4
    uint32_t r0[2], rA[2], rB[2], rC[2];  // rows of chunks c + 1, c + 2, c + 3 in step c
    auto fetch = [&](int c) {
      if (c < n) cur.advance(1);
      kv[c] = cur.keys();
      cur.template look_up<LY::ROWS>(lds, lane_row, kx, t, add);
    };
    __builtin_amdgcn_s_waitcnt(0);  // Q and list loads are done: only DMA is counted below
    fetch(0);
    rows_of(r0);
    issue_k(r0, 0);
    fetch(1);
    rows_of(rA);
    issue_k(rA, 1);
    wait_loads<0>();
    __syncthreads();
    f32x16 sA, sB;
    uint32_t pA[8], pB[8];
    if (rows_live) start_walk<D>(x, sA, pA, pB, lds, fr.k, fr.k + LY::TILE);
    // P of "chunk -1" is zero; its V slot must hold finite values
    for (int e = tid; e < LY::TILE / 16; e += NT)
      *(uint4*)(smem_raw + LY::V_OFF + LY::TILE + e * 16) = make_uint4(0, 0, 0, 0);
    fetch(2);
    rows_of(rB);
    __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0)
    __syncthreads();
    issue_k(rB, 0);
    issue_v(r0, 0);
    fetch(3);

    // step c, c of parity `par`
    auto step = [&](int c, int par, f32x16& sc, f32x16& sn, uint32_t (&pp)[8], uint32_t (&pn)[8]) {
      constexpr int SY = D == 128 ? 9 : 4;
      auto mid = [&](int s) {
        if (s == 1) {  // the rows of c + 3 were looked up in the previous step
          rows_of(rC);
          if (c + 4 < n) cur.advance(1);
          kv[4] = cur.keys();
        }
        if (s == SY) {
          asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
          wait_loads<0>();
          __builtin_amdgcn_s_barrier();
          asm volatile("" ::: "memory");
          issue_k(rC, 1 - par);
          issue_v(rA, 1 - par);
        }
        if (s == (D == 128 ? 4 : 2)) cur.template look_up<LY::ROWS>(lds, lane_row, kx, t, add);
      };
      if (rows_live) {
        walk_step<D, SY>(
            x, sc, sn, pp, pn, c, kv[0], scale_log2, lds,
            [&](int d) { return fr.k + (d == c ? par : 1 - par) * LY::TILE; },
            [&](int d) { return fr.v + LY::V_OFF + (d == c ? par : 1 - par) * LY::TILE; }, mid);
      } else {
#pragma unroll
        for (int s = 0; s < 2 * KV::KK; ++s) mid(s);
      }
#pragma unroll
      for (int k = 0; k < LY::ROWS; ++k) {
        rA[k] = rB[k];
        rB[k] = rC[k];
      }
#pragma unroll
      for (int k = 0; k < 4; ++k) kv[k] = kv[k + 1];
    };
    int c = 0;
    if (rows_live) {
#pragma unroll 1
      for (; c + 1 < n; c += 2) {
        step(c, 0, sA, sB, pA, pB);
        step(c + 1, 1, sB, sA, pB, pA);
      }
      if (c < n) {
        step(c, 0, sA, sB, pA, pB);
#pragma unroll
        for (int k = 0; k < 8; ++k) pA[k] = pB[k];
      }
      finish_chunk<D>(x, pA, lds, fr.v + LY::V_OFF + ((n - 1) & 1) * LY::TILE);
    } else {
#pragma unroll 1
      for (; c < n; ++c) step(c, c & 1, sA, sB, pA, pB);
    }
    __builtin_amdgcn_s_waitcnt(0);  // the loads past the walk's end
  }
  store_tile<D, RASTER>(g, e_i, x, q0, head_row, first_row, ob, lse);
}

// Blocks of 5 row tiles (129 .. 160 slots): eight waves, two per SIMD (waves w and w + 4
// share one), one workgroup per CU.
// - wave X_s (s = 0..3) owns query tile s for the whole walk;
// - wave Y_s issues the DMA of every fourth chunk (s, s + 4, ...) and computes tile 4 on
//   those same chunks with its own online-softmax state; the four partial states of tile
//   4 merge by log-sum-exp at the end in a fixed order. So every SIMD carries 1.25 tiles.
// The waves meet at one barrier per window of four chunks: barrier B_v makes window v
// visible. In step c an X wave reads K of c + 2 and V^T of c, so it passes B_v in step 4v -
// 2; then K up to 4v - 1 and V up to 4v - 3 have been read, and Y issues window v + 1: 8 K
// and 10 V tiles are the fewest for which nothing unread is overwritten.
// Against waves that read K of c + 1 and V^T of c in their own step, with whole swizzled
// rows and a 9-chunk ring: 57600-token, 24-head layer of 160-slot blocks 6.40 -> 5.59 ms,
// 32760-token, 12-head layer of 144-slot blocks 1.22 -> 1.00 ms, d = 64 against the
// paired kernel before it 2.23 -> 1.79 ms (two batches of 16 heads, 19890 tokens).
template <int D>
struct FiveTileLayout {
  static constexpr int TILE = KvTile<D>::BYTES, T = 5;
  static constexpr int KRING = 8, VRING = 10;
  static constexpr int V_OFF = KRING * TILE;
  static constexpr int TAB_OFF = V_OFF + VRING * TILE;
  static constexpr int KV_OFF = TAB_OFF + 4 * T * 32 * 4;  // real keys of chunk c at c % 16
  static constexpr int LIST_OFF = KV_OFF + 64;
  static constexpr int SEG = 512;  // kept-list entries staged at a time
  static constexpr int BYTES = LIST_OFF + (SEG + 1) * 8;
  static_assert(BYTES <= 160 * 1024, "one CU's LDS");
};

// Stores accumulators quarter * SH .. of a tile (the merged fifth tile), see store_tile.
template <int D, bool RASTER>
__device__ __forceinline__ void store_quarter(const DevGeom& g, const BlockExt& e, int quarter,
                                              const float* acc, float m, float l, int q0,
                                              int64_t first_row, int64_t head_row, __bf16* ob,
                                              float* lse) {
  constexpr int SH = D / 8;
  const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(l), __float_as_uint(l), false,
                                                   false);
  l = __uint_as_float(sw[0]) + __uint_as_float(sw[1]);
  const int ln = lane_now();
  const int qs = q0 + (ln & 31), half = ln >> 5;
  const bool real = qs < e.n;
  if (RASTER ? real : qs < g.BS) {
    const float inv = (real && l > 0.0f) ? 1.0f / l : 0.0f;
    const int64_t row = RASTER ? head_row + ext_token(g, e, qs) : first_row + qs;
    __bf16* dst = ob + row * D + quarter * (SH * 2) + 4 * half;
#pragma unroll
    for (int r = 0; r < SH; r += 4) {
      bf16x4 v;
#pragma unroll
      for (int k = 0; k < 4; ++k) v[k] = __bf16(acc ? acc[r + k] * inv : 0.0f);
      *reinterpret_cast<bf16x4*>(dst + 2 * r) = v;
    }
    if (lse && real && half == 0 && quarter == 0)
      lse[row] = l > 0.0f ? (m + log2f(l)) * kLn2 : -INFINITY;
  }
}

template <int D, bool RASTER, bool MULTI>
__device__ __forceinline__ void five_tile_walk(const Item& it, const uint4* __restrict__ qb,
                                               const char* __restrict__ kb,
                                               const char* __restrict__ vb, float scale_log2,
                                               __bf16* __restrict__ ob, float* __restrict__ lse,
                                               char* smem_raw) {
  using KV = KvTile<D>;
  using LY = FiveTileLayout<D>;
  constexpr int NT = 512;
  lds_char* const lds = (lds_char*)smem_raw;
  lds_int* const kval = (lds_int*)(smem_raw + LY::KV_OFF);
  lds_int* const list = (lds_int*)(smem_raw + LY::LIST_OFF);

  const DevGeom g = it.g;
  const BlockExt e_i = block_ext(g, it.i);
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int sidx = wave & 3;  // X: tile; Y: chunk residue mod 4
  const int q0 = (wave >= 4 ? 4 : sidx) * 32;
  const bool rows_live = q0 < e_i.n;
  const int64_t head_row = RASTER ? it.bh * g.N : it.bh * g.NB * int64_t(g.BS);
  const int64_t first_row = head_row + int64_t(it.i) * g.BS;  // blocked layout
  const int cnt = it.cnt;
  const int j0 = tid < min(cnt, LY::SEG) ? it.list_src[tid] : -1;  // in flight beside the tables
  slot_tables<D, LY::T, RASTER>(g, (lds_int*)(smem_raw + LY::TAB_OFF), tid, NT);
  const FragAddr fr(lane);

  if (wave < 4) {
    // ---- X ----
    TileState<D> x;
    load_q<D, RASTER>(g, e_i, qb, head_row, first_row, q0, x.qf);
    clear_tile(x);
    for (int seg = 0; seg < cnt; seg += LY::SEG) {
      const int ns = min(cnt - seg, LY::SEG);
      if (seg) __syncthreads();
      const int n = stage_list<D, RASTER, true>(g, it.list_src + seg, ns, seg ? -2 : j0, true,
                                                  list, tid, lane, NT).chunks;
      if (n == 0) continue;
      // P of "chunk -1" is zero; its V slot must hold finite values
      for (int e = tid; e < LY::TILE / 16; e += 256)
        *(uint4*)(smem_raw + LY::V_OFF + (LY::VRING - 1) * LY::TILE + e * 16) =
            make_uint4(0, 0, 0, 0);
      __syncthreads();  // B_0
      if (!rows_live) {  // no query rows here: only the barriers of the walk
#pragma unroll 1
        for (int v = 1; v <= (n + 1) / 4; ++v) __syncthreads();
        continue;
      }
      f32x16 sA, sB;
      uint32_t pA[8], pB[8];
      start_walk<D>(x, sA, pA, pB, lds, fr.k, fr.k + LY::TILE);
      // real keys of chunk c, read a step ahead and moved to a scalar register: a wait for
      // it at the top of a step would also drain the fragment reads just issued
      int kv = __builtin_amdgcn_readfirstlane(kval[0]);
      int vs = LY::V_OFF, vs_prev = LY::V_OFF + (LY::VRING - 1) * LY::TILE;  // V(c), V(c - 1)
      auto step = [&](int c, f32x16& sc, f32x16& sn, uint32_t (&pp)[8], uint32_t (&pn)[8]) {
        constexpr int SY = D == 128 ? 8 : 4;
        int kv_next = 0;
        auto mid = [&](int s) {
          if (s != SY) return;
          if ((c & 3) == 2) {  // B_v, v = (c + 2) / 4
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");
          }
          kv_next = kval[(c + 1) & 15];
        };
        walk_step<D, SY>(
            x, sc, sn, pp, pn, c, kv, scale_log2, lds,
            [&](int d) { return fr.k + ((d + 2) & (LY::KRING - 1)) * LY::TILE; },
            [&](int d) { return fr.v + (d == c ? vs : vs_prev); }, mid);
        kv = __builtin_amdgcn_readfirstlane(kv_next);
        vs_prev = vs;
        vs = vs == LY::V_OFF + (LY::VRING - 1) * LY::TILE ? LY::V_OFF : vs + LY::TILE;
      };
      int c = 0;
#pragma unroll 1
      for (; c + 1 < n; c += 2) {
        step(c, sA, sB, pA, pB);
        step(c + 1, sB, sA, pB, pA);
      }
      if (c < n) {
        step(c, sA, sB, pA, pB);
#pragma unroll
        for (int k = 0; k < 8; ++k) pA[k] = pB[k];
      }
      finish_chunk<D>(x, pA, lds, fr.v + vs_prev);
    }
    __syncthreads();  // every walk is done (the merge overwrites the rings)
    store_tile<D, RASTER>(g, e_i, x, q0, head_row, first_row, ob, lse);
    __syncthreads();
    return;
  }

  // ---- Y ----
  TileState<D> x;
  load_q<D, RASTER>(g, e_i, qb, head_row, first_row, q0, x.qf);
  clear_tile(x);
  const int lane_row = (lane >> 2) * 4;
  const uint32_t kx = k_piece(lane), dvx = v_piece(lane) - k_piece(lane);
  const char* const kbase = kb + head_row * KV::ROW;
  const char* const vbase = vb + head_row * KV::ROW;
  const uint32_t lds_u32 = uint32_t(reinterpret_cast<uintptr_t>(lds));
  for (int seg = 0; seg < cnt; seg += LY::SEG) {
    const int ns = min(cnt - seg, LY::SEG);
    if (seg) __syncthreads();
    const Staged st = stage_list<D, RASTER, true>(g, it.list_src + seg, ns, seg ? -2 : j0, true,
                                                  list, tid, lane, NT);
    const int n = st.chunks;
    if (n == 0) continue;
    __builtin_amdgcn_s_waitcnt(0);  // Q and list loads are done: only DMA is counted below
    WalkCursor<LY::TAB_OFF, LY::T, true> cur(list, ns, st.stream);
    auto next4 = [](int v) { return v + 4 >= LY::VRING ? v + 4 - LY::VRING : v + 4; };
    int c_issue = sidx, v_issue = sidx;  // the next chunk to issue, its V slot
    auto issue = [&]() {
      if (c_issue < n) {
        cur.advance(c_issue == sidx ? sidx + 1 : 4);
        if (lane == 0) kval[c_issue & 15] = cur.keys();
        int t[2];
        uint32_t r[2];
        cur.template look_up<2>(lds, lane_row, kx, t, r);
        r[0] += t[0];
        r[1] += t[1];
        const uint32_t kd = lds_u32 + (c_issue & (LY::KRING - 1)) * LY::TILE;
        const uint32_t vd = lds_u32 + LY::V_OFF + v_issue * LY::TILE;
#pragma unroll
        for (int k = 0; k < KV::LOADS; ++k) tile_dma(kbase, r[k & 1], kd, k);
#pragma unroll
        for (int k = 0; k < KV::LOADS; ++k) tile_dma(vbase, r[k & 1] + dvx, vd, k);
      }
      c_issue += 4;
      v_issue = next4(v_issue);
    };
    int vs = sidx;  // V slot of the next chunk to compute
    auto compute = [&](int c) {
      if (rows_live && c < n)
        lone_chunk<D>(x, kval[c & 15], scale_log2, lds,
                      fr.k + (c & (LY::KRING - 1)) * LY::TILE, fr.v + LY::V_OFF + vs * LY::TILE);
      vs = next4(vs);
    };
    issue();  // window 0
    issue();  // window 1
    if (sidx + 4 < n)
      wait_loads<2 * KV::LOADS>();
    else
      wait_loads<0>();
    __syncthreads();  // B_0: window 0 landed
    const int nb = (n + 1) / 4;  // barriers B_1 .. B_nb of the walk
#pragma unroll 1
    for (int v = 1; v <= nb; ++v) {
      compute(4 * (v - 1) + sidx);
      wait_loads<0>();
      __syncthreads();  // B_v: window v landed
      issue();          // window v + 1
    }
    compute(4 * nb + sidx);
  }

  // tile 4: the Y waves' partial states merge in LDS, each wave a quarter of the columns,
  // summed in the order Y_0 .. Y_3 (one wave merging all of them kept the CU 2k cycles
  // longer)
  constexpr int SH = KV::DT * 16 / 4;  // accumulators per quarter
  float* const ml = reinterpret_cast<float*>(smem_raw);  // [wave][lane][2]
  float* const part = ml + 4 * 128;                      // [quarter][wave][SH][lane]
  __syncthreads();
  if (rows_live) {
    ml[(sidx * 64 + lane) * 2] = x.m;
    ml[(sidx * 64 + lane) * 2 + 1] = x.l;
#pragma unroll
    for (int r = 0; r < KV::DT * 16; ++r)
      part[((r / SH * 4 + sidx) * SH + r % SH) * 64 + lane] = x.o[r / 16][r % 16];
  }
  __syncthreads();
  if (!rows_live) {
    store_quarter<D, RASTER>(g, e_i, sidx, nullptr, 0.0f, 0.0f, q0, first_row, head_row, ob, lse);
    return;
  }
  float f[4], mm = -INFINITY, l = 0.0f;
#pragma unroll
  for (int k = 0; k < 4; ++k) mm = fmaxf(mm, ml[(k * 64 + lane) * 2]);
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    f[k] = mm == -INFINITY ? 0.0f : __builtin_amdgcn_exp2f(ml[(k * 64 + lane) * 2] - mm);
    l += ml[(k * 64 + lane) * 2 + 1] * f[k];
  }
  float acc[SH];
#pragma unroll
  for (int r = 0; r < SH; ++r) {
    acc[r] = 0.0f;
#pragma unroll
    for (int k = 0; k < 4; ++k)
      acc[r] += part[((sidx * 4 + k) * SH + r) * 64 + lane] * f[k];
  }
  store_quarter<D, RASTER>(g, e_i, sidx, acc, mm, l, q0, first_row, head_row, ob, lse);
}

// Kernels. MULTI (raster only): one launch over heads with different blockings; the work
// item picks its head, and with it the geometry and block lists, from `tab`.
#define SPADE_ATTN_ARGS                                                                       \
  DevGeom g_arg, const uint4 *__restrict__ qb, const char *__restrict__ kb,                   \
      const char *__restrict__ vb, const int *__restrict__ counts,                            \
      const int *__restrict__ indices, float scale_log2, __bf16 *__restrict__ ob,             \
      float *__restrict__ lse, const int *__restrict__ order,                                 \
      typename std::conditional<MULTI, MultiTable, NoTable>::type tab
constexpr int kLoaderItems = 4096, kLoaderBlocks = 608;  // blocks of 64..96 slots
constexpr int kLoaderItems64 = 640;                      // wider ones at d = 64

template <int D, int W, bool RASTER, bool MULTI, bool STREAM>
__global__ void __launch_bounds__(64 * W) __attribute__((amdgpu_waves_per_eu(D == 64 ? 3 : 2)))
    attn_kernel(SPADE_ATTN_ARGS) {
  extern __shared__ __align__(16) char smem_raw[];
  const Item it = work_item<MULTI>(g_arg, counts, indices, order, tab);
  if (it.i >= 0)
    row_tile_walk<D, W, RASTER, STREAM>(it, qb, kb, vb, scale_log2, ob, lse, smem_raw);
}

template <int D, bool RASTER, bool MULTI>
__global__ void __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2)))
    attn_sw_kernel(SPADE_ATTN_ARGS) {
  extern __shared__ __align__(16) char smem_raw[];
  const Item it = work_item<MULTI>(g_arg, counts, indices, order, tab);
  if (it.i >= 0) five_tile_walk<D, RASTER, MULTI>(it, qb, kb, vb, scale_log2, ob, lse, smem_raw);
}
#undef SPADE_ATTN_ARGS

// ---- the loader kernel ----

template <int D>
struct Tile {
  static constexpr int NCH = D / 8;                 // 16-byte pieces per row
  static constexpr int ROW_BYTES = D * 2;
  static constexpr int TILE_BYTES = kChunk * ROW_BYTES;
  static constexpr int RPI = 64 / NCH;              // rows per wave-wide 1 KB load
  static constexpr int LOADS = kChunk / RPI;        // wave loads per tile
  static constexpr int BUF_BYTES = 2 * TILE_BYTES;  // K tile then V tile
};

// swizzles: LDS piece c of tile row r holds global piece c ^ f(r)
template <int D>
__device__ __forceinline__ int swz_k(int r) { return r & (Tile<D>::NCH - 1); }
// V: in a transposing read, lanes 0-15 take pieces 4t + {0,1} and lanes 16-31 pieces
// 4t + {2,3} of rows 0-3; an XOR stride of 4 pieces (d = 128) keeps the two groups'
// pieces disjoint, so 32 lanes hit 64 distinct banks (no LDS bank conflicts)
template <int D>
__device__ __forceinline__ int swz_v(int r) { return D >= 128 ? 4 * (r & 3) : 2 * (r & 3); }

// Position in the kept-block walk: list entry jj, its block j and real-key count nj,
// the chunk's first key slot c0, and block j's extent (raster addressing).
struct Cursor {
  int jj, j, nj, c0;
  BlockExt e;
};

// Raster addressing of slot s of the cursor's block, relative to `base`: full
// blocks (every block away from the grid's far edges) share one slot -> token
// offset table `rel` (LDS, built once per workgroup), so a load costs one LDS
// read instead of the division-based map; ragged blocks take the map.
struct RasterRows {
  bool full;
  int64_t base;  // head_row + block origin (full), head_row (ragged)
};

__device__ __forceinline__ RasterRows raster_rows(const DevGeom& g, const Cursor& c,
                                                  int64_t head_row) {
  const bool full = c.e.n == g.BS;
  return {full, head_row + (full ? block_origin(g, c.e) : 0)};
}

__device__ __forceinline__ Cursor next_chunk(const DevGeom& g, const lds_int* list, int cnt,
                                             Cursor c) {
  c.c0 += kChunk;
  while (c.c0 >= c.nj) {
    ++c.jj;
    if (c.jj >= cnt) {
      c.nj = 0;
      c.c0 = 0;
      return c;
    }
    const int j = __builtin_amdgcn_readfirstlane(list[c.jj]);  // uniform: keep in SGPRs
    if (j >= 0 && j < g.NB) {
      c.j = j;
      c.e = block_ext(g, j);
      c.nj = c.e.n;
      c.c0 = 0;
    }
  }
  return c;
}

// The 2*LOADS wave-wide DMA loads of one chunk: K and V rows at base_row + the lane's
// row offsets (bytes), into the chunk's LDS buffer.
template <int D>
__device__ __forceinline__ void loader_issue(const char* kb, const char* vb, int64_t base_row,
                                             const uint32_t (&row_off)[Tile<D>::LOADS],
                                             uint32_t lds_buf, int lane) {
  using TL = Tile<D>;
  const char* kbase = kb + base_row * TL::ROW_BYTES;
  const char* vbase = vb + base_row * TL::ROW_BYTES;
#pragma unroll
  for (int q = 0; q < 2 * TL::LOADS; ++q) {
    const bool is_v = q >= TL::LOADS;
    const int qq = is_v ? q - TL::LOADS : q;
    const int r = qq * TL::RPI + lane / TL::NCH;  // tile row (key slot in chunk)
    const int gp = (lane % TL::NCH) ^ (is_v ? swz_v<D>(r) : swz_k<D>(r));
    const uint32_t off = row_off[qq] + uint32_t(gp * 16);
    const uint32_t dst = lds_buf + (is_v ? TL::TILE_BYTES : 0) + qq * 1024;  // M0
    asm volatile("global_load_lds_dwordx4 %0, %1" ::"v"(off), "s"(is_v ? vbase : kbase),
                 "{m0}"(dst)
                 : "memory");
  }
}

template <int D, bool RASTER>
__device__ __forceinline__ void loader_chunk(const DevGeom& g, const char* kb, const char* vb,
                                             int64_t head_row, const Cursor& c, const lds_int* rel,
                                             uint32_t lds_buf, int lane) {
  using TL = Tile<D>;
  const int last = c.nj - 1 - c.c0;  // last real key slot of the chunk
  uint32_t row_off[TL::LOADS];       // byte offset of this lane's row in load qq
  int64_t base_row;
  auto fill = [&](auto row_of) {
#pragma unroll
    for (int qq = 0; qq < TL::LOADS; ++qq)
      row_off[qq] = uint32_t(row_of(min(qq * TL::RPI + lane / TL::NCH, last)) * TL::ROW_BYTES);
  };
  if (!RASTER) {
    base_row = head_row + int64_t(c.j) * g.BS + c.c0;
    fill([](int sr) { return sr; });
  } else {
    const RasterRows rr = raster_rows(g, c, head_row);
    base_row = rr.base;
    if (rr.full)
      fill([&](int sr) { return rel[c.c0 + sr]; });
    else
      fill([&](int sr) { return int(ext_token(g, c.e, c.c0 + sr)); });
  }
  loader_issue<D>(kb, vb, base_row, row_off, lds_buf, lane);
}

// Single-buffered phases with a loader wave: W compute waves (32 query slots each) and one
// more that issues all loads of the next chunk while this one is computed (two LDS
// buffers, whole rows XOR-swizzled over their 16-byte pieces). Kept for the shapes
// where it beats the pipelined walk (see the dispatch). The same arithmetic in the same order
// as a walk that is not a stream: either gives the same bits.
template <int D, int W, bool RASTER, bool MULTI>
__global__ void __launch_bounds__(64 * (W + 1))
    __attribute__((amdgpu_waves_per_eu(3)))
    attn_loader_kernel(DevGeom g_arg, const uint4* __restrict__ qb, const char* __restrict__ kb,
                const char* __restrict__ vb, const int* __restrict__ counts,
                const int* __restrict__ indices, float scale_log2, __bf16* __restrict__ ob,
                float* __restrict__ lse, const int* __restrict__ order,
                typename std::conditional<MULTI, MultiTable, NoTable>::type tab) {
  using TL = Tile<D>;
  __shared__ __align__(16) char lds_raw[2 * TL::BUF_BYTES];
  __shared__ int rel_raw[RASTER ? kMaxBS : 1];  // full-block slot -> raster token offset
  extern __shared__ int list_raw[];  // kept list of this work item, NB entries
  lds_char* const lds = (lds_char*)lds_raw;
  lds_int* const list = (lds_int*)list_raw;
  lds_int* const rel = (lds_int*)rel_raw;

  const Item it = work_item<MULTI>(g_arg, counts, indices, order, tab);
  if (it.i < 0) return;
  const DevGeom g = it.g;
  const int64_t bh = it.bh;
  const int i = it.i;
  const int* const list_src = it.list_src;
  const BlockExt e_i = block_ext(g, i);
  const int n_i = e_i.n;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // uniform: keep in an SGPR
  const bool loader = wave == W;  // loader wave: q0 = 32 W >= BS, so no query rows
  const int q0 = wave * 32;
  const int half = lane >> 5;  // k-slot group of the MFMA operands
  const int r32 = lane & 31;
  const int64_t head_row = RASTER ? bh * g.N : bh * g.NB * int64_t(g.BS);
  // row of query slot qs < n_i of this item
  auto q_row = [&](int qs) -> int64_t {
    return RASTER ? head_row + ext_token(g, e_i, qs) : head_row + int64_t(i) * g.BS + qs;
  };

  // Q^T fragments (B operand): query row q0 + r32, d = 16*kk + 8*half .. +8
  bf16x8 qf[D / 16];
  {
    const int qs = q0 + r32;
    const uint4* src = qb + q_row(min(qs, n_i - 1)) * TL::NCH + half;
#pragma unroll
    for (int kk = 0; kk < D / 16; ++kk) {
      uint4 v = make_uint4(0, 0, 0, 0);
      if (qs < n_i) v = src[2 * kk];
      qf[kk] = __builtin_bit_cast(bf16x8, v);
    }
  }

  const int cnt = it.cnt;
  for (int e = threadIdx.x; e < cnt; e += 64 * (W + 1)) list[e] = list_src[e];
  if (RASTER) {
    for (int sl = threadIdx.x; sl < g.BS; sl += 64 * (W + 1)) {
      const int q = sl / g.bw;
      rel[sl] = ((q / g.bh) * g.Hs + q % g.bh) * g.Ws + sl % g.bw;
    }
  }
  __syncthreads();  // list and table visible to every wave (also completes the Q loads)

  // per-lane LDS byte offsets that do not depend on the chunk
  // K operand: tile row r32, global piece 2*kk + half
  const int k_off = r32 * TL::ROW_BYTES;
  const int k_sw = swz_k<D>(r32);
  // V^T operand via transposing reads: 16-lane group G, index s
  const int G = lane >> 4, s16 = lane & 15;
  const int v_row0 = 4 * (G >> 1) + (s16 >> 2);     // + 16u + 8h
  const int v_piece0 = 2 * (G & 1) + ((s16 & 3) >> 1);  // + 4t
  const int v_sub = (s16 & 1) * 8;

  f32x16 o[D / 32];
#pragma unroll
  for (int t = 0; t < D / 32; ++t)
#pragma unroll
    for (int r = 0; r < 16; ++r) o[t][r] = 0.0f;
  float m = -INFINITY, l = 0.0f;
  const bool rows_live = q0 < n_i;
  const bf16x2 ones = {__bf16(1.0f), __bf16(1.0f)};

  const uint32_t lds_u32 = uint32_t(reinterpret_cast<uintptr_t>(lds));
  auto issue = [&](const Cursor& c, int b) {  // the loads of chunk c into buffer b
    if (loader)
      loader_chunk<D, RASTER>(g, kb, vb, head_row, c, rel, lds_u32 + b * TL::BUF_BYTES, lane);
  };
  Cursor cur = {-1, 0, 0, -kChunk, e_i};
  cur = next_chunk(g, list, cnt, cur);
  int buf = 0;
  if (cur.jj < cnt) issue(cur, 0);
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();
  while (cur.jj < cnt) {
    const Cursor nxt = next_chunk(g, list, cnt, cur);
    if (nxt.jj < cnt) issue(nxt, buf ^ 1);
    if (rows_live) {
      lds_char* Kt = lds + buf * TL::BUF_BYTES;
      lds_char* Vt = Kt + TL::TILE_BYTES;
      f32x16 s;
#pragma unroll
      for (int r = 0; r < 16; ++r) s[r] = 0.0f;
      {
        bf16x8 kf[D / 16];
#pragma unroll
        for (int kk = 0; kk < D / 16; ++kk)
          kf[kk] = *(lds_bf16x8*)(Kt + k_off + (((2 * kk + half) ^ k_sw) << 4));
#pragma unroll
        for (int kk = 0; kk < D / 16; ++kk)
          s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[kk], qf[kk], s, 0, 0, 0);
        // schedule: two K reads ahead of each pair of MFMAs
#pragma unroll
        for (int gi = 0; gi < D / 32; ++gi) {
          __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);  // LDS reads
          __builtin_amdgcn_sched_group_barrier(0x008, 2, 0);  // MFMAs
        }
      }      // s[r]: key (r/4)*8 + 4*half + r%4 of the chunk, query row r32
      if (cur.c0 + kChunk > cur.nj) {
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int kr = (r >> 2) * 8 + 4 * half + (r & 3);
          if (cur.c0 + kr >= cur.nj) s[r] = -INFINITY;
        }
      }
      float mx = s[0];
#pragma unroll
      for (int r = 1; r < 16; ++r) mx = fmaxf(mx, s[r]);
      {
        const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(mx), __float_as_uint(mx),
                                                         false, false);
        mx = fmaxf(__uint_as_float(sw[0]), __uint_as_float(sw[1])) * scale_log2;
      }
      if (__any(mx > m + kRescaleLog2)) {
        const float mnew = fmaxf(m, mx);
        const float alpha = __builtin_amdgcn_exp2f(m - mnew);
        l *= alpha;
#pragma unroll
        for (int t = 0; t < D / 32; ++t)
#pragma unroll
          for (int r = 0; r < 16; ++r) o[t][r] *= alpha;
        m = mnew;
      }
      bf16x8 p[2];
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const float e = __builtin_amdgcn_exp2f(__builtin_fmaf(s[r], scale_log2, -m));
        p[r >> 3][r & 7] = __bf16(e);
      }
#pragma unroll
      for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const bf16x2 pr = {p[u][2 * e], p[u][2 * e + 1]};
          l = __builtin_amdgcn_fdot2_f32_bf16(pr, ones, l, false);
        }
      {
        bf16x8 vf[D / 32][2];
#pragma unroll
        for (int t = 0; t < D / 32; ++t)
#pragma unroll
          for (int u = 0; u < 2; ++u) {
            bf16x4 h2[2];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
              const int row = 16 * u + 8 * h + v_row0;
              const int piece = (4 * t + v_piece0) ^ swz_v<D>(row);
              h2[h] = __builtin_amdgcn_ds_read_tr16_b64_v4bf16(
                  (lds_bf16x4*)(Vt + row * TL::ROW_BYTES + piece * 16 + v_sub));
            }
            vf[t][u] = __builtin_shufflevector(h2[0], h2[1], 0, 1, 2, 3, 4, 5, 6, 7);
          }
#pragma unroll
        for (int t = 0; t < D / 32; ++t)
#pragma unroll
          for (int u = 0; u < 2; ++u)
            o[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[t][u], p[u], o[t], 0, 0, 0);
        // schedule: the V^T reads of two output tiles ahead of their four MFMAs
#pragma unroll
        for (int gi = 0; gi < D / 64; ++gi) {
          __builtin_amdgcn_sched_group_barrier(0x100, 8, 1);  // LDS reads
          __builtin_amdgcn_sched_group_barrier(0x008, 4, 1);  // MFMAs
        }
      }
    }
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    buf ^= 1;
    cur = nxt;
  }

  // normalise and store: lane holds query row q0 + r32, d = 32t + 8*rq + 4*half + 0..3
  {
    const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(l), __float_as_uint(l),
                                                     false, false);
    l = __uint_as_float(sw[0]) + __uint_as_float(sw[1]);
  }
  const int qs = q0 + r32;
  // blocked output: every slot of the block (padding as zeros); raster: real rows only
  if (RASTER ? qs < n_i : qs < g.BS) {
    const bool real = qs < n_i;
    const float inv = (real && l > 0.0f) ? 1.0f / l : 0.0f;
    const int64_t orow = real ? q_row(qs) : head_row + int64_t(i) * g.BS + qs;
    __bf16* dst = ob + orow * D + 4 * half;
#pragma unroll
    for (int t = 0; t < D / 32; ++t)
#pragma unroll
      for (int rq = 0; rq < 4; ++rq) {
        bf16x4 v;
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = __bf16(o[t][4 * rq + e] * inv);
        *reinterpret_cast<bf16x4*>(dst + 32 * t + 8 * rq) = v;
      }
    if (lse && real && half == 0)
      lse[orow] = l > 0.0f ? (m + log2f(l)) * 0.69314718055994530942f : -INFINITY;
  }
}

// What walking a geometry's keys as one stream does: whether it saves at least 3% of the
// chunks, and whether at least an eighth of the blocks hold fewer than 32 keys, which keep a
// row that lists one of them from being a stream. The look-up of chunks that span two blocks
// costs 2-4% (128-slot blocks whose edge blocks are multiples of 32 keys: 2.67 against
// 2.74 ms; 120-slot blocks: 26.8 ms with the stream against 28.6 without it).
struct StreamGain {
  bool saves, many_small;
};
StreamGain stream_gain(const DevGeom& g) {
  int64_t chunks = 0, keys = 0, small = 0;
  for (int k = 0; k < 8; ++k) {  // full or ragged along each axis
    const int et = (k & 1) ? g.T % g.bt : g.bt, eh = (k & 2) ? g.Hs % g.bh : g.bh;
    const int ew = (k & 4) ? g.Ws % g.bw : g.bw;
    const int64_t n = int64_t(et) * eh * ew;
    if (n == 0) continue;
    const int64_t count = int64_t((k & 1) ? 1 : g.T / g.bt) * ((k & 2) ? 1 : g.Hs / g.bh) *
                          ((k & 4) ? 1 : g.Ws / g.bw);
    const int64_t c = (n + kChunk - 1) / kChunk;
    chunks += count * c;
    keys += count * (n < kChunk ? c * kChunk : n);
    small += n < kChunk ? count : 0;
  }
  return {100 * (chunks * kChunk - keys) >= 3 * chunks * kChunk, 8 * small >= g.NB};
}

// Whether a geometry's rows may be walked as a stream at all: decided by the geometry alone,
// so that a head's rounding does not depend on what else its call holds. Blocks of 64 and 96
// slots at d = 128 are not: their large launches run the loader kernel, which cuts each block
// into chunks of its own, and a walk that does the same gives the same bits. With the 6% that
// a ragged axis leaves to save, the stream was no faster there (960 blocks of 64 slots, 24
// heads: 9.83 ms apart, 9.89 as a stream; 252, 12 heads: 0.380, 0.384; 392 of 96 slots, 8
// heads: 0.902, 0.915). Nor are those of 65..95 slots there with many small blocks, whose
// rows are hardly ever streams: 756 of 90 slots, 23% of them small, 24 heads 10.5 -> 10.2 ms,
// 270 of 72 slots, 33%, 4 heads 0.271 -> 0.259; with 8% small ones the stream is 2..5% ahead.
// Nor those of 161..224 slots at d = 64, whose large launches run the loader kernel too.
bool may_stream(const DevGeom& g) {
  const StreamGain s = stream_gain(g);
  if (!s.saves) return false;
  if (g.d == 128) return g.BS != 64 && g.BS != 96 && !(g.BS > 64 && g.BS < 96 && s.many_small);
  return g.BS <= 160 || g.BS > 224;
}

// Launches `kernel` (one of the above, all with the same arguments) over the work items.
template <bool MULTI, class Kernel>
hipError_t launch_items(Kernel kernel, int threads, size_t lds, int max_lds, const DevGeom& g,
                        const void* qb, const void* kb, const void* vb, const int* counts,
                        const int* indices, float scale_log2, void* ob, float* lse, hipStream_t s,
                        const MultiTable* tab, const int* order) {
  const hipError_t e = ensure_dynamic_lds(reinterpret_cast<const void*>(kernel), max_lds);
  if (e != hipSuccess) return e;
  const uint4* q4 = static_cast<const uint4*>(qb);
  const char* k1 = static_cast<const char*>(kb);
  const char* v1 = static_cast<const char*>(vb);
  __bf16* o2 = static_cast<__bf16*>(ob);
  if constexpr (MULTI) {
    const int64_t items = int64_t(g.B) * tab->items_per_batch;
    kernel<<<dim3(unsigned(items)), threads, lds, s>>>(g, q4, k1, v1, nullptr, nullptr, scale_log2,
                                                       o2, lse, order, *tab);
  } else {
    const int64_t items = int64_t(g.B) * g.H * ((g.NB + 7) / 8) * 8;  // see the XCD mapping
    kernel<<<dim3(unsigned(items)), threads, lds, s>>>(g, q4, k1, v1, counts, indices, scale_log2,
                                                       o2, lse, order, NoTable{});
  }
  return hipGetLastError();
}

template <int D, bool RASTER, bool MULTI = false>
hipError_t launch_d(const DevGeom& g, const void* qb, const void* kb, const void* vb,
                    const int* counts, const int* indices, float scale_log2, void* ob, float* lse,
                    hipStream_t s, const MultiTable* tab = nullptr, const int* order = nullptr) {
  int nb_max = g.NB;
  int64_t items = int64_t(g.B) * g.H * g.NB;
  if constexpr (MULTI) {
    nb_max = 0;
    for (int k = 0; k < tab->n_heads; ++k) nb_max = max(nb_max, tab->geo[tab->head[k].geom].NB);
    items = int64_t(g.B) * tab->items_per_batch;
  }
  auto run = [&](auto kernel, int threads, size_t lds, int max_lds) {
    return launch_items<MULTI>(kernel, threads, lds, max_lds, g, qb, kb, vb, counts, indices,
                               scale_log2, ob, lse, s, tab, order);
  };
  auto loader = [&](auto kernel, int w) {
    return run(kernel, 64 * (w + 1), size_t(nb_max) * sizeof(int), int(kMaxAttnNB * sizeof(int)));
  };
  auto walk = [&](auto kernel, auto layout, int w) {
    return run(kernel, 64 * w, size_t(layout.BYTES), int(layout.BYTES));
  };
  // the walk over concatenated keys where it saves chunks (WalkCursor)
  bool stream = false;
  if constexpr (MULTI)
    stream = tab->streams != 0;
  else
    stream = may_stream(g);
#define SPADE_ATTN_APART(w) walk(attn_kernel<D, w, RASTER, MULTI, false>, WalkLayout<D, w>{}, w)
#define SPADE_ATTN_WALK(w)                                                             \
  (stream ? walk(attn_kernel<D, w, RASTER, MULTI, true>, WalkLayout<D, w>{}, w)        \
          : SPADE_ATTN_APART(w))
  switch ((g.BS + 31) / 32) {
    case 1: return SPADE_ATTN_APART(1);  // a stream needs blocks of more than a chunk
    case 2:
      // Blocks of 64 slots at d = 128 load 16 KB per 64 query rows and chunk. In large
      // launches over long rows a loading wave of its own keeps those loads further ahead;
      // it walks block by block, so it takes rows that are not a stream, and gives the bits of
      // the walk. Loader against walk (Top-P lists, range over two inputs):
      // +3..+6% at 768 to 960 blocks from 4608 items on, +1..+4% at 616 and 720 blocks;
      // -2..-7% at 600 blocks, -7..-17% at 252 to 504; -3% at 960 blocks and 2880 items.
      if constexpr (D == 128) {
        if (g.BS == 64 && !stream && items >= kLoaderItems && nb_max >= kLoaderBlocks)
          return loader(attn_loader_kernel<D, 2, RASTER, MULTI>, 2);
      }
      return SPADE_ATTN_WALK(2);
    case 3:
      // Large launches of rows that are not a stream (same bits either way): with the walk
      // 96-slot blocks took 0..2% longer than with the loading wave (24 heads of 392 blocks,
      // blocked: 3.016 against 2.956 ms; of 720: 7.12, 6.98); at 2016 items and fewer the walk
      // is 1..29% faster. 756 90-slot blocks, 23% of them of fewer than 32 keys, at 3024 items:
      // 1.60 ms walked, 1.63 with the loading wave. At d = 64 the loading wave is ahead in the
      // blocked form only: 576 96-slot blocks, 24 heads 3.85 against 3.97 ms, 8 heads 1.26, 1.31;
      // raster 3.83, 3.78 and 1.22, 1.22, up to 8% behind on other grids.
      if constexpr (D == 128 || !RASTER) {
        if (!stream && items >= kLoaderItems)
          return loader(attn_loader_kernel<D, 3, RASTER, MULTI>, 3);
      }
      return SPADE_ATTN_WALK(3);
    case 4: return SPADE_ATTN_WALK(4);
    case 5:
      return run(attn_sw_kernel<D, RASTER, MULTI>, 512, FiveTileLayout<D>::BYTES,
                 FiveTileLayout<D>::BYTES);
    case 6:
      // At d = 64 four of the loader kernel's waves (101 registers) fit a SIMD, three of the
      // walk's (157). Launches of more than 2.5 items per CU, loader against walk: 1.56, 1.85 ms
      // (224 blocks of 192 slots, 12 heads), 1.09, 1.27 (320, 4 heads); shorter ones are bound
      // by an item's latency: 0.147, 0.126 ms (50, 4 heads).
      if constexpr (D == 64) {
        if (items > kLoaderItems64) return loader(attn_loader_kernel<D, 6, RASTER, MULTI>, 6);
        return SPADE_ATTN_APART(6);
      } else {
        return SPADE_ATTN_WALK(6);
      }
    case 7:
      // at d = 64 seven waves of 101 registers plus a loader leave room for two
      // workgroups per CU, the walk's seven of 157 for one: 3.23 against 3.47 ms (57600
      // tokens, 12 heads)
      if constexpr (D == 64)
        return loader(attn_loader_kernel<D, 7, RASTER, MULTI>, 7);
      else
        return SPADE_ATTN_WALK(7);
    case 8: return SPADE_ATTN_WALK(8);
  }
#undef SPADE_ATTN_WALK
#undef SPADE_ATTN_APART
  return hipErrorInvalidValue;
}

// Ranked work order (§3.3 (3): rows preprocessed into a ranked layout, heads of
// similar density co-scheduled). The dispatch walks the (batch, head) pairs in
// the order of their heaviest row, then their total kept blocks (descending,
// ties to the lower index), so long rows start first instead of forming the
// tail; within a head each XCD takes its rows heaviest first (heavy_first).
constexpr int kRankThreads = 1024;
constexpr int kRankWaves = kRankThreads / 64;
// Counts one workgroup ranks by itself. A call on empty lists, one kernel against two: 19.4,
// 21.5 us at 8640 counts (24 pairs), 30.4, 32.2 at 16384 (4), 33.2, 32.9 at 23040 (24), 50.3,
// 48.3 at 38400 (40), 361, 292 at 262144 (256).
constexpr int64_t kOneRankCounts = 24 << 10;
constexpr int64_t kUnrankedItems = 256;      // work items that all start at once: no order

// A head's key, from its n kept counts (one wave, the result in every lane): its heaviest
// row, then its total.
__device__ __forceinline__ uint64_t head_key(const int* __restrict__ c, int n) {
  const int lane = int(threadIdx.x & 63);
  int mx = 0;
  uint32_t sum = 0;
  for (int i = lane; i < n; i += 64) {
    const int v = min(max(c[i], 0), n);
    mx = max(mx, v);
    sum += uint32_t(v);
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    mx = max(mx, __shfl_xor(mx, off));
    sum += __shfl_xor(sum, off);
  }
  return (uint64_t(uint32_t(mx)) << 32) | sum;
}

// rank of key t among n (descending, ties to the lower index)
__device__ __forceinline__ int key_rank(const uint64_t* keys, int n, int t) {
  const uint64_t kt = keys[t];
  int rank = 0;
  for (int j = 0; j < n; ++j) {
    const uint64_t kj = keys[j];
    rank += (kj > kt || (kj == kt && j < t)) ? 1 : 0;
  }
  return rank;
}

// Keys and order of n <= kRankThreads pairs in one workgroup: a launch less than with the
// two kernels below (24 pairs of 360 counts: 5.3 us against 4.8 + 4.8 and the gap between
// them). Bound by the counts' load latency, so each wave takes whole heads.
__global__ void __launch_bounds__(kRankThreads) head_order_kernel(DevGeom g, int n,
                                                                  const int* __restrict__ counts,
                                                                  int* __restrict__ order) {
  __shared__ uint64_t keys[kRankThreads];
  for (int t = threadIdx.x >> 6; t < n; t += kRankWaves) {
    const uint64_t k = head_key(counts + int64_t(t) * g.NB, g.NB);
    if ((threadIdx.x & 63) == 0) keys[t] = k;
  }
  __syncthreads();
  if (int(threadIdx.x) < n) order[key_rank(keys, n, threadIdx.x)] = threadIdx.x;
}

// The same for more pairs or counts than one workgroup should read: keys, then ranks.
__global__ void __launch_bounds__(64) head_keys_kernel(DevGeom g, const int* __restrict__ counts,
                                                       uint64_t* __restrict__ keys) {
  const uint64_t k = head_key(counts + int64_t(blockIdx.x) * g.NB, g.NB);
  if (threadIdx.x == 0) keys[blockIdx.x] = k;
}

__global__ void __launch_bounds__(kRankThreads) head_rank_kernel(const uint64_t* __restrict__ keys,
                                                                 int n, int* __restrict__ order) {
  for (int t = threadIdx.x; t < n; t += kRankThreads) order[key_rank(keys, n, t)] = t;
}

// The ranking of one multi-scheme launch, one workgroup per batch element over the
// launch's heads; the heads' first items follow as prefix sums of their padded item
// counts in rank order. Layout of `ranked`: per batch element, n head indices by rank,
// then n first items.
__global__ void __launch_bounds__(kRankThreads) multi_order_kernel(MultiTable tab,
                                                                   int* __restrict__ ranked) {
  __shared__ uint64_t keys[kMaxMultiHeads];
  __shared__ int by_rank[kMaxMultiHeads];
  const int n = tab.n_heads, b = blockIdx.x;
  for (int k = threadIdx.x >> 6; k < n; k += kRankWaves) {
    const MultiHead& mh = tab.head[k];
    const uint64_t key = head_key(mh.counts + int64_t(b) * mh.counts_bstride, tab.geo[mh.geom].NB);
    if ((threadIdx.x & 63) == 0) keys[k] = key;
  }
  __syncthreads();
  if (int(threadIdx.x) < n) by_rank[key_rank(keys, n, threadIdx.x)] = threadIdx.x;
  __syncthreads();
  if (threadIdx.x == 0) {
    int* out = ranked + int64_t(b) * 2 * n;
    int first = 0;
    for (int r = 0; r < n; ++r) {
      const int k = by_rank[r];
      out[r] = k;
      out[n + r] = first;
      first += (tab.geo[tab.head[k].geom].NB + 7) / 8 * 8;
    }
  }
}

size_t ranked_pairs(const DevGeom& g) {
  const int64_t n = int64_t(g.B) * g.H;
  return n > 0 && n <= kMaxRankedHeads ? size_t(n) : 0;
}

}  // namespace

hipError_t noalloc_scratch(void** ptr, size_t* bytes) {
  static std::mutex mu;
  static void* by_device[kMaxDevices] = {};
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(mu);
  if (by_device[dev] == nullptr) {  // first call on this device: look the copy up once
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    by_device[dev] = p;
  }
  *ptr = by_device[dev];
  *bytes = kNoAllocScratchBytes;
  return hipSuccess;
}

size_t attn_workspace_bytes(const DevGeom& g) {
  // keys (8 B) of every pair, then the order (4 B; a multi-scheme launch also
  // keeps each head's first item, 4 B more)
  const size_t n = ranked_pairs(g);
  return n ? n * 16 : 0;
}

hipError_t launch_sparse_attn_multi(const DevGeom* geo, int n_geo, const MultiHead* heads,
                                    int n_heads, const void* q, const void* k, const void* v,
                                    float scale, void* o, float* lse, void* ws, hipStream_t s) {
  const float sl2 = scale * 1.44269504088896340736f;
  // each launch ranks its heads in its own part of the workspace (8 B per pair)
  const bool rank = ranked_pairs(geo[0]) > 0;
  char* wsp = static_cast<char*>(ws);
  // one launch per workgroup shape; the launch's geometry carries that shape's BS
  for (int w = 1; w <= kMaxBS / 32; ++w) {
    MultiTable tab = {};
    for (int c = 0; c < n_geo; ++c) tab.geo[c] = geo[c];
    int start = 0, widest = -1;
    for (int hh = 0; hh < n_heads; ++hh) {
      const DevGeom& gh = geo[heads[hh].geom];
      if ((gh.BS + 31) / 32 != w) continue;
      MultiHead mh = heads[hh];
      mh.start = start;
      start += (gh.NB + 7) / 8 * 8;
      tab.head[tab.n_heads++] = mh;
      // Each geometry decides for itself whether its keys are a stream: a head's chunks, and
      // with them the rounding of its output, must not depend on the launch's other heads.
      // Heads that are not streamed run chunk by chunk in a streaming instance as well.
      if (may_stream(gh)) tab.streams |= 1u << mh.geom;
      if (widest < 0 || gh.BS > geo[widest].BS) widest = heads[hh].geom;
    }
    if (tab.n_heads == 0) continue;
    tab.items_per_batch = start;
    const DevGeom& gl = geo[widest];
    const int* order = nullptr;
    if (rank) {
      const int64_t pairs = int64_t(gl.B) * tab.n_heads;
      int* ranked = reinterpret_cast<int*>(wsp);
      wsp += pairs * 8;
      multi_order_kernel<<<dim3(unsigned(gl.B)), kRankThreads, 0, s>>>(tab, ranked);
      const hipError_t e = hipGetLastError();
      if (e != hipSuccess) return e;
      order = ranked;
    }
    const hipError_t e = gl.d == 128
        ? launch_d<128, true, true>(gl, q, k, v, nullptr, nullptr, sl2, o, lse, s, &tab, order)
        : launch_d<64, true, true>(gl, q, k, v, nullptr, nullptr, sl2, o, lse, s, &tab, order);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t launch_block_sparse_attn(const DevGeom& g, const void* qb, const void* kb,
                                    const void* vb, const int* counts, const int* indices,
                                    float scale, void* ob, float* lse, void* ws, bool raster,
                                    hipStream_t s) {
  const float sl2 = scale * 1.44269504088896340736f;
  const int* order = nullptr;
  const int64_t n = int64_t(ranked_pairs(g));
  if (n > 0 && n * g.NB > kUnrankedItems) {
    uint64_t* keys = static_cast<uint64_t*>(ws);
    int* ord = reinterpret_cast<int*>(keys + n);
    if (n <= kRankThreads && n * g.NB <= kOneRankCounts) {
      head_order_kernel<<<1, kRankThreads, 0, s>>>(g, int(n), counts, ord);
    } else {
      head_keys_kernel<<<dim3(unsigned(n)), 64, 0, s>>>(g, counts, keys);
      head_rank_kernel<<<1, kRankThreads, 0, s>>>(keys, int(n), ord);
    }
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    order = ord;
  }
  if (g.d == 128)
    return raster ? launch_d<128, true>(g, qb, kb, vb, counts, indices, sl2, ob, lse, s, nullptr, order)
                  : launch_d<128, false>(g, qb, kb, vb, counts, indices, sl2, ob, lse, s, nullptr, order);
  if (g.d == 64)
    return raster ? launch_d<64, true>(g, qb, kb, vb, counts, indices, sl2, ob, lse, s, nullptr, order)
                  : launch_d<64, false>(g, qb, kb, vb, counts, indices, sl2, ob, lse, s, nullptr, order);
  return hipErrorInvalidValue;
}

}  // namespace spade
