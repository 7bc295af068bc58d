// Building blocks of the attention kernels' chunk walk (gfx950): the LDS tiles of one
// 32-key chunk and their DMA, the walk over a staged kept list, and one wave's
// software-pipelined step. Used by attn.hip.
//
// Tiles. A chunk's K rows and V rows are one LDS tile each: [d / 32 groups of 64 bytes]
// [32 rows][64 bytes], filled by 1 KB wave loads of 16 rows x 64 bytes (whole 64-byte
// sectors). K: the four 16-byte pieces of row r are XORed with (r / 4) & 3, so 16
// consecutive rows' equal pieces hit 16 different bank groups (ds_read_b128 of the K
// operand); V: plain, since 4 rows x 64 bytes are all 64 banks (ds_read_b64_tr_b16 of the
// V^T operand). Every fragment address is a lane constant, the tile's base and an
// instruction offset: 3 address instructions per step, against 12 with whole rows XORed
// over their 16 pieces, and a lane's DMA needs the token offsets of 2 rows per chunk
// instead of 8.
//
// Step. Each of the step's d / 8 slots holds one MFMA and its share of the softmax; a
// wave issues in order, so a slot-by-slot mix keeps the matrix unit fed while the vector
// unit works (two waves per SIMD fill each other's gaps). The order is pinned by
// sched_barrier: left to itself the compiler puts the MFMAs first. A wave's K and V^T
// fragments are re-read in place, half a step or more before their use, so no MFMA waits
// on an LDS round trip; the accumulators, Q^T, the fragments, two S tiles and two P take
// 208 of the 256 registers that two waves per SIMD leave.
#pragma once

#include "spade_internal.h"

namespace spade {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef __attribute__((address_space(3))) void lds_void;
typedef __attribute__((address_space(3))) char lds_char;
typedef __attribute__((address_space(3))) int lds_int;
typedef __attribute__((address_space(3))) bf16x4 lds_bf16x4;
typedef __attribute__((address_space(3))) bf16x8 lds_bf16x8;

constexpr int kChunk = 32;            // key slots per chunk
constexpr float kRescaleLog2 = 8.0f;  // lazy-rescale threshold (base-2 logits)
constexpr float kLn2 = 0.69314718055994530942f;

// Raster token of slot `slot` of a block of any extent (ragged edge blocks).
__device__ __forceinline__ int64_t ext_token(const DevGeom& g, const BlockExt& e, int slot) {
  return block_slot_token(g, e, __builtin_amdgcn_rcpf(float(e.ew)),
                          __builtin_amdgcn_rcpf(float(e.eh)), slot);
}

// Raster token of a block's first slot.
__device__ __forceinline__ int64_t block_origin(const DevGeom& g, const BlockExt& e) {
  return (int64_t(e.t0) * g.Hs + e.y0) * g.Ws + e.x0;
}

// The lane index, computed where it is asked for: keeping what derives from it in
// registers across the chunk walk would spill fragments.
__device__ __forceinline__ int lane_now() {
  int l;
  asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(l));
  return l;
}

// max of three in one instruction (llvm.maximum needs no canonicalisation first; a NaN
// propagates, and makes its row NaN in the end as it does in P)
__device__ __forceinline__ float max3(float a, float b, float c) {
  return __builtin_elementwise_maximum(__builtin_elementwise_maximum(a, b), c);
}

// max over lanes l and l ^ 32 (the two halves of a query row's keys)
__device__ __forceinline__ float row_max(float v) {
  const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false,
                                                   false);
  return __builtin_elementwise_maximum(__uint_as_float(sw[0]), __uint_as_float(sw[1]));
}

// wait until at most N of this wave's vector-memory loads are in flight
template <int N>
__device__ __forceinline__ void wait_loads() {
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

template <int D>
struct KvTile {
  static constexpr int KK = D / 16;  // MFMA steps of an S tile
  static constexpr int DT = D / 32;  // output column tiles
  static constexpr int ROW = D * 2;
  static constexpr int BYTES = kChunk * ROW;
  static constexpr int LOADS = BYTES / 1024;  // wave loads
};

// Lane offsets inside a tile: K fragment kk is at (kk odd ? k ^ 32 : k) + (kk / 2) * 2048
// (row lane % 32, pieces 2 kk + lane / 32); V^T fragment (t, u, h) at v + t * 2048 +
// (16 u + 8 h) * 64 (16-lane group G: rows 4 (G / 2) .. + 3, columns 16 (G & 1) .. + 15).
struct FragAddr {
  int k, v;
  __device__ __forceinline__ explicit FragAddr(int lane) {
    const int r32 = lane & 31, half = lane >> 5;
    k = r32 * 64 + ((half ^ ((r32 >> 2) & 3)) << 4);
    v = (4 * half + ((lane & 15) >> 2)) * 64 +
        (2 * ((lane >> 4) & 1) + ((lane & 3) >> 1)) * 16 + (lane & 1) * 8;
  }
};

__device__ __forceinline__ bf16x8 read_k_frag(lds_char* lds, int k, int kk) {
  return *(lds_bf16x8*)(lds + ((kk & 1) ? k ^ 32 : k) + (kk >> 1) * 2048);
}

__device__ __forceinline__ bf16x8 read_v_frag(lds_char* lds, int v, int t, int u) {
  bf16x4 h2[2];
#pragma unroll
  for (int h = 0; h < 2; ++h)
    h2[h] = __builtin_amdgcn_ds_read_tr16_b64_v4bf16(
        (lds_bf16x4*)(lds + v + t * 2048 + (16 * u + 8 * h) * 64));
  return __builtin_shufflevector(h2[0], h2[1], 0, 1, 2, 3, 4, 5, 6, 7);
}

// Wave load k of a tile: rows 16 (k & 1) .. + 15 of 64-byte group k / 2. `off` is the
// lane's byte offset for group 0; the instruction offset moves the global address one
// group on per 64 bytes and the LDS address with it, which `dst` takes back. Issued from
// asm: the compiler would drain an LDS-DMA builtin before every LDS read.
__device__ __forceinline__ void tile_dma(const char* base, uint32_t off, uint32_t tile, int k) {
  const uint32_t dst = tile + k * 1024 - (k >> 1) * 64;
  switch (k >> 1) {
#define SPADE_DMA(g)                                                                          \
  case g:                                                                                     \
    asm volatile("global_load_lds_dwordx4 %0, %1 offset:%3" ::"v"(off), "s"(base), "{m0}"(dst), \
                 "n"(64 * g)                                                                  \
                 : "memory");                                                                 \
    break;
    SPADE_DMA(0) SPADE_DMA(1) SPADE_DMA(2) SPADE_DMA(3)
#undef SPADE_DMA
  }
}
// a lane's 16-byte piece of its row in a wave load (row 16 (k & 1) + lane / 4)
__device__ __forceinline__ uint32_t k_piece(int lane) {
  return uint32_t(((lane & 3) ^ ((lane >> 4) & 3)) << 4);
}
__device__ __forceinline__ uint32_t v_piece(int lane) { return uint32_t((lane & 3) << 4); }

// Slot -> byte offset from the block's first row, T * 32 entries per table. Raster: one
// table per (y ragged, x ragged) variant, so every block reads its rows from a table (a
// block ragged along t uses the first slots of its table); blocked: one table.
template <int D, int T, bool RASTER>
__device__ __forceinline__ void slot_tables(const DevGeom& g, lds_int* rel, int tid, int nt) {
  if (RASTER) {
    const int eh_r = g.Hs - (g.nH - 1) * g.bh, ew_r = g.Ws - (g.nW - 1) * g.bw;
    for (int e = tid; e < 4 * T * 32; e += nt) {
      const int v = e / (T * 32), sl = e % (T * 32);
      const int ew = (v & 1) ? ew_r : g.bw, eh = (v & 2) ? eh_r : g.bh;
      // float quotients, exact below 2^8 (block_slot_token)
      const int q = int((float(sl) + 0.5f) * __builtin_amdgcn_rcpf(float(ew)));
      const int dt = int((float(q) + 0.5f) * __builtin_amdgcn_rcpf(float(eh)));
      rel[e] = ((dt * g.Hs + q - dt * eh) * g.Ws + sl - q * ew) * KvTile<D>::ROW;
    }
  } else {
    for (int e = tid; e < T * 32; e += nt) rel[e] = e * KvTile<D>::ROW;
  }
}

// block_ext with float quotients, for j < 2^14: (j + 0.5) / d lies 0.5 / d from an
// integer and comes out within 2^-9 / d of it.
__device__ __forceinline__ BlockExt list_block_ext(const DevGeom& g, int j) {
  const int r = int((float(j) + 0.5f) * __builtin_amdgcn_rcpf(float(g.nW)));
  const int tb = int((float(r) + 0.5f) * __builtin_amdgcn_rcpf(float(g.nH)));
  BlockExt e;
  e.t0 = tb * g.bt;
  e.y0 = (r - tb * g.nH) * g.bh;
  e.x0 = (j - r * g.nW) * g.bw;
  e.et = min(g.bt, g.T - e.t0);
  e.eh = min(g.bh, g.Hs - e.y0);
  e.ew = min(g.bw, g.Ws - e.x0);
  e.n = e.et * e.eh * e.ew;
  return e;
}

// Sum over the wave by DPP (quads, half rows, rows) and the four row totals: a tenth of the
// time of six dependent LDS shuffles.
__device__ __forceinline__ int wave_sum(int v) {
  v += __builtin_amdgcn_update_dpp(0, v, 0xB1, 0xf, 0xf, true);   // quad_perm [1,0,3,2]
  v += __builtin_amdgcn_update_dpp(0, v, 0x4E, 0xf, 0xf, true);   // quad_perm [2,3,0,1]
  v += __builtin_amdgcn_update_dpp(0, v, 0x141, 0xf, 0xf, true);  // row_half_mirror
  v += __builtin_amdgcn_update_dpp(0, v, 0x140, 0xf, 0xf, true);  // row_mirror
  return __builtin_amdgcn_readlane(v, 0) + __builtin_amdgcn_readlane(v, 16) +
         __builtin_amdgcn_readlane(v, 32) + __builtin_amdgcn_readlane(v, 48);
}

// A staged part of the kept list: its chunks, and whether they run across block boundaries.
struct Staged {
  int chunks;
  bool stream;  // the blocks' keys form one stream; else each block starts a chunk
};

// Stages ns kept-list entries as {byte offset of the block's first row, real keys |
// table << 16} (malformed indices: no keys). Where some block's keys do not fill its last
// chunk, and every block has at least kChunk keys (so a chunk spans at most two of them),
// the walk runs over the concatenated keys and only the last chunk is partly empty: 10%
// fewer chunks for blocks of 144 keys, 6% for 120 (12 heads of 32760 tokens, every block
// kept: 8.40 -> 7.60 ms); `may` = false (uniform) keeps it from that. j0: the entry of index
// tid, loaded earlier (-2: not loaded). Every wave returns the same result.
template <int D, bool RASTER, bool STREAM>
__device__ __forceinline__ Staged stage_list(const DevGeom& g, const int* src, int ns,
                                             int j0, bool may, lds_int* list, int tid, int lane,
                                             int nt) {
  for (int e = tid; e < ns; e += nt) {
    const int j = e == tid && j0 != -2 ? j0 : src[e];
    int2 ent = make_int2(0, 0);
    if (j >= 0 && j < g.NB) {
      const BlockExt be = list_block_ext(g, j);
      const int var = RASTER ? (be.ew != g.bw ? 1 : 0) | (be.eh != g.bh ? 2 : 0) : 0;
      ent = make_int2((RASTER ? int(block_origin(g, be)) : j * g.BS) * KvTile<D>::ROW,
                      be.n | (var << 16));
    }
    list[2 * e] = ent.x;
    list[2 * e + 1] = ent.y;
  }
  __syncthreads();
  int keys = 0, apart = 0;
  bool small = false, part = false;
  for (int e = lane; e < ns; e += 64) {
    const int n = list[2 * e + 1] & 0xffff;
    keys += n;
    apart += (n + kChunk - 1) / kChunk;
    small = small || n < kChunk;
    part = part || n % kChunk != 0;
  }
  keys = wave_sum(keys);
  apart = wave_sum(apart);
  const bool stream = STREAM && may && __ballot(small) == 0 && __ballot(part) != 0;
  return {stream ? (keys + kChunk - 1) / kChunk : apart, stream};
}

// Position of a chunk in a staged list: it starts at slot c0 of the current entry (n real
// keys, row table at `tab`, first row at byte `org`); entry `next` follows.
// STREAM: whether the walk may be a stream (`pad` 0; 31 where it is not).
template <int TAB_OFF, int T, bool STREAM>
struct WalkCursor {
  lds_int* list;
  int ns, pad;
  int next = 0, c0 = -kChunk, n = 0, len = 0, tab = 0, org = 0;
  int nx, nw;  // the next entry, loaded ahead

  __device__ __forceinline__ WalkCursor(lds_int* l, int count, bool stream)
      : list(l), ns(count), pad(stream ? 0 : kChunk - 1) {
    nx = list[0];
    nw = list[1];
  }
  __device__ __forceinline__ static int table(int w) { return TAB_OFF + (w >> 16) * (T * 128); }
  // moves on by `by` chunks (the caller stays within the walk)
  __device__ __forceinline__ void advance(int by) {
    c0 += by * kChunk;
    while (c0 >= len) {
      c0 -= len;
      org = __builtin_amdgcn_readfirstlane(nx);
      const int w = __builtin_amdgcn_readfirstlane(nw);
      n = w & 0xffff;
      len = STREAM ? (n + pad) & ~pad : (n + kChunk - 1) & ~(kChunk - 1);
      tab = table(w);
      ++next;
      nx = list[2 * next];  // past the last entry: not used
      nw = list[2 * next + 1];
    }
  }
  __device__ __forceinline__ bool spans() const {
    return STREAM && c0 + kChunk > len && next < ns;
  }
  // real keys of the chunk (more than kChunk: all)
  __device__ __forceinline__ int keys() const { return spans() ? kChunk : n - c0; }
  // Rows of this lane in the chunk, `lane_row` (row * 4) and `lane_row` + 64: their table
  // entries and the byte offsets to add. Rows past the walk's last key repeat it.
  template <int ROWS>
  __device__ __forceinline__ void look_up(lds_char* lds, int lane_row, uint32_t piece, int (&t)[2],
                                          uint32_t (&add)[2]) const {
    int at[2];
    if (spans()) {
      const int norg = __builtin_amdgcn_readfirstlane(nx);
      const int ntab = table(__builtin_amdgcn_readfirstlane(nw)) - len * 4;
#pragma unroll
      for (int k = 0; k < ROWS; ++k) {
        const int p = lane_row + 64 * k + c0 * 4;
        const bool here = p < len * 4;
        at[k] = p + (here ? tab : ntab);
        add[k] = uint32_t(here ? org : norg) + piece;
      }
    } else {
      const int last = tab + (n - 1) * 4;
#pragma unroll
      for (int k = 0; k < ROWS; ++k) {
        at[k] = min(lane_row + 64 * k + c0 * 4 + tab, last);
        add[k] = uint32_t(org) + piece;
      }
    }
#pragma unroll
    for (int k = 0; k < ROWS; ++k) t[k] = *(lds_int*)(lds + at[k]);
  }
};

// State of one wave's 32-row query tile. Lane l holds query row l % 32; S^T keeps 16 of
// the chunk's keys per lane (key of register r: 8 (r / 4) + 4 (l / 32) + r % 4).
template <int D>
struct TileState {
  using KV = KvTile<D>;
  bf16x8 qf[KV::KK], kf[KV::KK], vf[KV::DT][2];
  f32x16 o[KV::DT];
  float m, l;   // running max (base 2, scaled) and this half's sum of weights
  float alpha;  // factor O still has to take
  bool rescale;
};

template <int D>
__device__ __forceinline__ void clear_tile(TileState<D>& x) {
#pragma unroll
  for (int t = 0; t < KvTile<D>::DT; ++t) x.o[t] = f32x16{};
  x.m = -INFINITY;
  x.l = 0.0f;
  x.rescale = false;
}

// Loads the Q^T fragments (B operand) of query slots q0 .. q0 + 31; slots past the
// block's last token repeat it, their results are dropped. first_row: the block's first
// row (blocked layout).
template <int D, bool RASTER>
__device__ __forceinline__ void load_q(const DevGeom& g, const BlockExt& e, const uint4* qb,
                                       int64_t head_row, int64_t first_row, int q0,
                                       bf16x8 (&qf)[D / 16]) {
  const int ln = lane_now();
  const int qs = min(q0 + (ln & 31), e.n - 1);
  const int64_t row = RASTER ? head_row + ext_token(g, e, qs) : first_row + qs;
  const uint4* src = qb + row * (D / 8) + (ln >> 5);
#pragma unroll
  for (int kk = 0; kk < D / 16; ++kk) qf[kk] = __builtin_bit_cast(bf16x8, src[2 * kk]);
}

// Normalises and stores a wave's tile: lane holds query slot q0 + lane % 32, columns
// 32 t + 8 rq + 4 (lane / 32) + 0..3. Blocked output: padding slots get zeros.
template <int D, bool RASTER>
__device__ __forceinline__ void store_tile(const DevGeom& g, const BlockExt& e, TileState<D>& x,
                                           int q0, int64_t head_row, int64_t first_row, __bf16* ob,
                                           float* lse) {
  const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(x.l), __float_as_uint(x.l),
                                                   false, false);
  const float l = __uint_as_float(sw[0]) + __uint_as_float(sw[1]);
  const int ln = lane_now();
  const int qs = q0 + (ln & 31), half = ln >> 5;
  const bool real = qs < e.n;
  if (RASTER ? real : qs < g.BS) {
    const float inv = (real && l > 0.0f) ? 1.0f / l : 0.0f;
    const int64_t row = RASTER ? head_row + ext_token(g, e, qs) : first_row + qs;
    __bf16* dst = ob + row * D + 4 * half;
#pragma unroll
    for (int t = 0; t < KvTile<D>::DT; ++t)
#pragma unroll
      for (int rq = 0; rq < 4; ++rq) {
        bf16x4 v;
#pragma unroll
        for (int k = 0; k < 4; ++k) v[k] = __bf16(x.o[t][4 * rq + k] * inv);
        *reinterpret_cast<bf16x4*>(dst + 32 * t + 8 * rq) = v;
      }
    if (lse && real && half == 0) lse[row] = l > 0.0f ? (x.m + log2f(l)) * kLn2 : -INFINITY;
  }
}

template <int D>
__device__ __forceinline__ void apply_rescale(TileState<D>& x) {
  if (x.rescale) {
#pragma unroll
    for (int t = 0; t < KvTile<D>::DT; ++t)
#pragma unroll
      for (int r = 0; r < 16; ++r) x.o[t][r] *= x.alpha;
  }
}

// keys past the chunk's kv real ones get -inf
__device__ __forceinline__ void mask_keys(f32x16& s, int kv) {
  if (kv < kChunk) {
    int kl = kv - ((lane_now() >> 5) << 2);
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      // opaque per group of four: one compare and one select per key, where the compiler
      // would chain all sixteen conditions
      if ((r & 3) == 0) asm volatile("" : "+v"(kl));
      s[r] = (r >> 2) * 8 + (r & 3) >= kl ? -INFINITY : s[r];
    }
  }
}

// Raises the running max when some row's max grows by more than 2^8; O is scaled by
// `alpha` before its next P.V (apply_rescale).
template <int D>
__device__ __forceinline__ void raise_max(TileState<D>& x, float mx) {
  x.rescale = __any(mx > x.m + kRescaleLog2);
  if (x.rescale) {
    const float mnew = fmaxf(x.m, mx);
    x.alpha = __builtin_amdgcn_exp2f(x.m - mnew);
    x.l *= x.alpha;
    x.m = mnew;
  }
}

__device__ __forceinline__ float weight(float s, float scale_log2, float m) {
  return __builtin_amdgcn_exp2f(__builtin_fmaf(s, scale_log2, -m));
}
__device__ __forceinline__ uint32_t pack_weights(float a, float b) {
  const bf16x2 p = {__bf16(a), __bf16(b)};
  return __builtin_bit_cast(uint32_t, p);
}
__device__ __forceinline__ float add_weights(float l, uint32_t p) {
  const bf16x2 ones = {__bf16(1.0f), __bf16(1.0f)};
  return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, p), ones, l, false);
}
__device__ __forceinline__ bf16x8 p_operand(const uint32_t (&p)[8], int u) {
  return __builtin_bit_cast(bf16x8, make_uint4(p[4 * u], p[4 * u + 1], p[4 * u + 2], p[4 * u + 3]));
}

// S of chunk 0 and the first half of chunk 1's K fragments (the first step reads the
// second half), P and V^T of "chunk -1" zero.
template <int D>
__device__ __forceinline__ void start_walk(TileState<D>& x, f32x16& s, uint32_t (&pa)[8],
                                           uint32_t (&pb)[8], lds_char* lds, int k0, int k1) {
  using KV = KvTile<D>;
#pragma unroll
  for (int kk = 0; kk < KV::KK; ++kk) x.kf[kk] = read_k_frag(lds, k0, kk);
  s = f32x16{};
#pragma unroll
  for (int kk = 0; kk < KV::KK; ++kk)
    s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x.kf[kk], x.qf[kk], s, 0, 0, 0);
#pragma unroll
  for (int kk = 0; kk < KV::KK / 2; ++kk) x.kf[kk] = read_k_frag(lds, k1, kk);
#pragma unroll
  for (int k = 0; k < 8; ++k) pa[k] = pb[k] = 0;
#pragma unroll
  for (int t = 0; t < KV::DT; ++t) x.vf[t][0] = x.vf[t][1] = bf16x8{};
  x.rescale = false;
}

// One step of the walk for chunk c: on the matrix unit S of c + 1 (even slots) and P.V of
// c - 1 (odd slots), on the vector unit the softmax of c: row sums of P(c - 1) and the
// row max of S(c) in the first slots, then the weights of c. sc: S of c, sn: S of c + 1;
// pp: P of c - 1, pn: P of c. Past the walk's end S of c + 1 is of stale keys and dropped.
// Slots 0 .. NS / 2 - 1 read the second halves of K(c + 1) and V(c - 1) into the fragments
// that the step's second half uses; the slots after SY read the first halves of K(c + 2)
// and V(c) for the next step. k_at(d) / v_at(d): lane offsets in the tiles of K(d + 2) and
// V(d). mid(s) runs in slot s; where it synchronises, it does so in slot SY (reads of
// slots <= NS / 2 - 1 have returned by then).
template <int D, int SY, class KAt, class VAt, class Mid>
__device__ __forceinline__ void walk_step(TileState<D>& x, f32x16& sc, f32x16& sn,
                                          uint32_t (&pp)[8], uint32_t (&pn)[8], int c, int kv,
                                          float scale_log2, lds_char* lds, KAt k_at, VAt v_at,
                                          Mid mid) {
  using KV = KvTile<D>;
  constexpr int NS = 2 * KV::KK;  // slots
  constexpr int N1 = NS * 5 / 16;  // slots before the branch on the row max
  constexpr int N2 = NS - N1;
  static_assert(SY >= N1 && SY >= NS / 2 && SY < NS - 1, "");
  apply_rescale(x);
  mask_keys(sc, kv);
  __builtin_amdgcn_sched_barrier(0);
  int ka = k_at(c - 1), va = v_at(c - 1);
  auto read_k = [&](int i) { x.kf[i] = read_k_frag(lds, ka, i); };
  auto read_v = [&](int i) { x.vf[i % KV::DT][i / KV::DT] = read_v_frag(lds, va, i % KV::DT, i / KV::DT); };
  auto reads = [&](int s) {
    if (s < NS / 2) {
      const int i = (s + NS / 2) >> 1;
      if ((s & 1) == 0)
        read_k(i);
      else
        read_v(i);
    }
    if (s > SY) {
      constexpr int NR = NS - 1 - SY;
#pragma unroll
      for (int j = 0; j < NS / 2; ++j)
        if (SY + 1 + j * NR / (NS / 2) == s) {
          if ((j & 1) == 0)
            read_k(j >> 1);
          else
            read_v(j >> 1);
        }
    }
  };
  auto mfma = [&](int s) {
    const int i = s >> 1;
    if ((s & 1) == 0) {
      sn = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x.kf[i], x.qf[i], i == 0 ? f32x16{} : sn, 0, 0,
                                                   0);
    } else {
      const int u = i / KV::DT, t = i % KV::DT;
      x.o[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x.vf[t][u], p_operand(pp, u), x.o[t], 0, 0, 0);
    }
  };
  float mx = 0.0f, h3[5];
  auto early = [&](int k) {  // sixteen pieces of the work before the branch
    if (k < 8) {
      x.l = add_weights(x.l, pp[k]);
      if (k == 7) asm volatile("" : "+v"(x.l));  // here, not at its use
    } else if (k < 13) {
      const int a = 3 * (k - 8);
      h3[k - 8] = max3(sc[a], sc[a + 1], sc[a + 2]);
    } else if (k == 13) {
      h3[0] = max3(h3[0], h3[1], sc[15]);
    } else if (k == 14) {
      h3[2] = max3(h3[2], h3[3], h3[4]);
    } else {
      mx = row_max(__builtin_elementwise_maximum(h3[0], h3[2])) * scale_log2;
    }
  };
#pragma unroll
  for (int s = 0; s < N1; ++s) {
    mfma(s);
    reads(s);
#pragma unroll
    for (int k = s * 16 / N1; k < (s + 1) * 16 / N1; ++k) early(k);
    mid(s);
    __builtin_amdgcn_sched_barrier(0);
  }
  raise_max(x, mx);
  __builtin_amdgcn_sched_barrier(0);
  float w[16];
#pragma unroll
  for (int s = N1; s < NS; ++s) {
    mfma(s);
    if (s == SY + 1) {
      ka = k_at(c);
      va = v_at(c);
    }
    reads(s);
    // weight r, and two pieces later the packing of the pair it completes
#pragma unroll
    for (int r = (s - N1) * 18 / N2; r < (s - N1 + 1) * 18 / N2; ++r) {
      if (r < 16) w[r] = weight(sc[r], scale_log2, x.m);
      if (r >= 3 && (r & 1)) {
        const int q = r - 3;
        pn[q >> 1] = pack_weights(w[q], w[q + 1]);
        asm volatile("" : "+v"(pn[q >> 1]));  // in this slot, not at its use
      }
    }
    mid(s);
    __builtin_amdgcn_sched_barrier(0);
  }
}

// P.V of one chunk on its own: the second half of V^T is read here (lane offset v in its
// tile), the first is in the fragments.
template <int D>
__device__ __forceinline__ void finish_chunk(TileState<D>& x, const uint32_t (&p)[8], lds_char* lds,
                                             int v) {
  using KV = KvTile<D>;
#pragma unroll
  for (int i = KV::KK / 2; i < KV::KK; ++i)
    x.vf[i % KV::DT][i / KV::DT] = read_v_frag(lds, v, i % KV::DT, i / KV::DT);
  apply_rescale(x);
#pragma unroll
  for (int u = 0; u < 2; ++u)
#pragma unroll
    for (int t = 0; t < KV::DT; ++t)
      x.o[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x.vf[t][u], p_operand(p, u), x.o[t], 0, 0, 0);
#pragma unroll
  for (int k = 0; k < 8; ++k) x.l = add_weights(x.l, p[k]);
}

// One whole chunk without pipelining: K and V tiles at lane offsets k and v.
template <int D>
__device__ __forceinline__ void lone_chunk(TileState<D>& x, int kv, float scale_log2, lds_char* lds,
                                           int k, int v) {
  using KV = KvTile<D>;
  f32x16 s = {};
#pragma unroll
  for (int kk = 0; kk < KV::KK; ++kk) x.kf[kk] = read_k_frag(lds, k, kk);
#pragma unroll
  for (int kk = 0; kk < KV::KK; ++kk)
    s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x.kf[kk], x.qf[kk], s, 0, 0, 0);
  mask_keys(s, kv);
  float mx = s[0];
#pragma unroll
  for (int r = 1; r < 15; r += 2) mx = max3(mx, s[r], s[r + 1]);
  raise_max(x, row_max(__builtin_elementwise_maximum(mx, s[15])) * scale_log2);
  uint32_t p[8];
#pragma unroll
  for (int q = 0; q < 16; q += 2)
    p[q >> 1] = pack_weights(weight(s[q], scale_log2, x.m), weight(s[q + 1], scale_log2, x.m));
#pragma unroll
  for (int i = 0; i < KV::KK / 2; ++i)
    x.vf[i % KV::DT][i / KV::DT] = read_v_frag(lds, v, i % KV::DT, i / KV::DT);
  finish_chunk<D>(x, p, lds, v);
}

}  // namespace
}  // namespace spade
