// Attention over the vertical-slash pattern of Alg. 5 at token granularity (Sec. 5.1 A(Q,K,V,M) with the mask M
// built from S = S_v U S_s): the kept keys of a head are gathered into packed images of their own, the kept
// offsets are walked as bands of 64-key tiles with a bit mask inside every tile.
#ifndef SP_VS_TOKEN_KERNELS_H
#define SP_VS_TOKEN_KERNELS_H
#include "sp_common.h"
#include "attn_kernel.h"
#include "vertical_slash_kernels.h"
#include "vs_items.h"

namespace {

// Per listed head (hb = b * n_heads + n), all in the caller's workspace (the items in the room of the search, which is done):
//   bits     [hb][2][seq/64] u64   kept keys (bit s) then kept offsets (bit o), written by the vector selection
//   cumv     [hb][nqb+1]           gathered keys with s < x*block (gathered = kept keys outside the forced sink block)
//   gpos     [hb][seq]             token index of gathered key g, ascending
//   bandbits [hb][2][words of 64]  bit x: a kept offset exists / every offset is kept among those that a 64-key tile x tiles
//                              below the row's first can realise (64x - 63 .. 64x + B - 1)
//   hdr      [hb][nqb]         items of row i: how many without a mask (they come first), and all
//   items    [hb][..]          the items of rows row0 .. row1 - 1, VsItem each; row i's start at vs_items_before(i, row0)
//   gimg     [hb][seq/64][2][64*D] packed K and V images of the gathered keys, 64 keys each, zero padded
//   act_pos  [b][n_heads], act_n [b]  the listed positions that take part (role -1, or all without roles), ascending
constexpr int VST_TASK_ROWS = 16;  // consecutive query blocks of a head that one XCD runs side by side
// Most groups of 8 chunks a head that run chunk by chunk: 384 query blocks of a launch, or 768 where the KV heads are not a
// multiple of 8 (see the mapping in vs_token_attn_kernel).
constexpr int VST_BY_LENGTH = 3, VST_BY_LENGTH_UNEVEN = 6;
struct VsTokParams {
  const uint16_t *q, *k, *v;
  const char *kvp;   // packed K/V images of the whole sequence (pack_kv_kernel)
  uint16_t *o;
  int64_t q_sb, q_st, q_sh, kv_sb, kv_st, kv_sh, o_sb, o_st, o_sh;
  int seq, nqb, block, n_kv_heads, group, n_heads, n_q_heads, forced;
  float c;  // softmax scale * log2(e)
  uint64_t *bits;
  int32_t *cumv, *gpos, *act_pos, *act_n;
  uint64_t *bandbits;
  int2 *hdr;
  VsItem *items;
  int64_t item_stride;  // items per listed head
  int row0, row1;       // the query blocks of this launch
  int n_gather;         // 64-key sub-tiles that the gathering launch packs (all, or 0 after the first launch of a call)
  char *gimg;
  int nch8;  // chunks of VST_TASK_ROWS query blocks per head and XCD: ceil(ceil((row1 - row0) / VST_TASK_ROWS) / 8)
  int by_length;  // the chunks run chunk by chunk
  int64_t *pairs;        // optional [b][n]: number of (query, key) pairs of the pattern (statistics)
  const int32_t *role;   // optional [b][n_q_heads]: only heads whose entry is -1 are processed
  int32_t head_ids[SP_MAX_HEADS];
};
__device__ __forceinline__ bool vst_skip(const VsTokParams &p, int b, int n) {
  return p.role != nullptr && p.role[(int64_t)b * p.n_q_heads + p.head_ids[n]] != -1;
}

// exclusive prefix sum of one value per thread over a 1024-thread workgroup; returns the total in `total`
__device__ __forceinline__ int block_scan_1024(int x, int *sh, int &total) {
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  int inc = x;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const int y = __shfl_up(inc, off, 64);
    if (lane >= off) inc += y;
  }
  if (lane == 63) sh[w] = inc;
  __syncthreads();
  int base = 0, tot = 0;
  for (int a = 0; a < 16; ++a) {
    const int s = sh[a];
    if (a < w) base += s;
    tot += s;
  }
  __syncthreads();
  total = tot;
  return base + inc - x;
}

// One workgroup of 1024 threads per listed head: the list of heads that take part, ranks of the kept keys, kept bands.
__global__ __launch_bounds__(1024) void vs_token_prep_kernel(VsTokParams p) {
  __shared__ int sh[16];
  const int n = blockIdx.x, b = blockIdx.y;
  {  // this head's rank among the heads that take part, and their number
    const int a = threadIdx.x;
    const bool on = a < p.n_heads && !vst_skip(p, b, a);
    const int total = __syncthreads_count(on), rank = __syncthreads_count(on && a < n);
    if (threadIdx.x == 0) {
      if (n == 0) p.act_n[b] = total;
      if (!vst_skip(p, b, n)) p.act_pos[(int64_t)b * p.n_heads + rank] = n;
    }
  }
  if (vst_skip(p, b, n)) return;
  const int64_t hb = (int64_t)b * p.n_heads + n;
  const int nw = p.seq / 64, B = p.block, wpb = B / 64;
  const uint64_t *bv = p.bits + hb * 2 * nw, *bs = bv + nw;
  int32_t *cumv = p.cumv + hb * (p.nqb + 1), *gpos = p.gpos + hb * (int64_t)p.seq;
  const int w_lo = p.forced ? wpb : 0;  // the forced sink block is walked as a block: its keys are not gathered
  int carry = 0;
  for (int w0 = 0; w0 < nw; w0 += 1024) {
    const int wd = w0 + threadIdx.x;
    uint64_t word = (wd < nw && wd >= w_lo) ? bv[wd] : 0ull;
    int total;
    int rank = carry + block_scan_1024(__popcll(word), sh, total);
    if (wd < nw && wd % wpb == 0) cumv[wd / wpb] = rank;
    while (word) {
      const int bit = __ffsll((unsigned long long)word) - 1;
      gpos[rank++] = wd * 64 + bit;
      word &= word - 1;
    }
    carry += total;
  }
  if (threadIdx.x == 0) {
    cumv[p.nqb] = carry;
    if (p.pairs) p.pairs[hb] = 0;
  }
  // tiles x >= 1 below a row's first: is any / every offset of theirs kept?
  uint64_t *any = p.bandbits + hb * 2 * ((nw + 63) / 64), *all = any + (nw + 63) / 64;
  for (int x0 = 0; x0 < nw; x0 += 1024) {
    const int x = x0 + threadIdx.x;
    bool some = false, every = false;
    if (x >= 1 && x < nw) {
      const uint64_t lo = bs[x - 1], mid = bs[x], hi = (wpb == 2 && x + 1 < nw) ? bs[x + 1] : 0ull;
      some = ((lo & ~1ull) | mid | hi) != 0ull;
      every = (lo | 1ull) == ~0ull && mid == ~0ull && (wpb == 1 || hi == ~0ull);
    }
    const uint64_t some64 = __ballot(some), every64 = __ballot(every);
    if ((threadIdx.x & 63) == 0 && x < nw) any[x / 64] = some64, all[x / 64] = every64;
  }
}

// The items of one row (query block i of a listed head), by a workgroup of four wavefronts.
// Tiles of 64 keys below the row are either bands, which hold a kept offset of the row's and are walked whole (mask: kept
// offsets | kept keys), or their kept keys are taken from the gathered images; so every allowed pair belongs to one
// item.  A gathered image whose keys all lie in bands is left out.  Items whose masks are all ones come first: they are
// walked without masks.  A row with more items than it has tiles walks all of its tiles as bands.
// With bands of whole key blocks, whose kept keys were taken from the gathered images all the same, the rows of timed
// prompts had 12 % (128K tokens) and 10 % (8K) more items, none of the bands without masks: 32 heads of 128K 44.1 -> 39.0
// ms, of 8K 496 -> 442 us, of 64 heads in dictionary layers of 28K 12.5 -> 10.7 ms (all of it with the scalar reads of
// the offsets in the kernel below).
__device__ void vs_row_items(const VsTokParams &p, int i, int b, int n) {
  __shared__ int cnt_sh[4][2];
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t hb = (int64_t)b * p.n_heads + n;
  const int spb = p.block / KT, nw = p.seq / KT, nx = (nw + 63) / 64;
  const uint64_t *__restrict__ bv = p.bits + hb * 2 * nw;
  const uint64_t *__restrict__ any = p.bandbits + hb * 2 * nx, *__restrict__ all = any + nx;
  const int32_t *__restrict__ gpos = p.gpos + hb * (int64_t)p.seq;
  const int first = i * spb;                          // the row's first tile; tile kt lies first - kt below it
  const int n_sink = (p.forced && i > 0) ? spb : 0;
  const int below = first - n_sink;                   // tiles 1 .. below below the row that are neither sink nor diagonal
  const int G = p.cumv[hb * (p.nqb + 1) + i], ng = (G + KT - 1) / KT;
  const int per = (ng + 2) / 3, g0 = (w - 1) * per, g1 = min(w * per, ng);  // gathered images of wavefronts 1 .. 3
  const uint64_t below_lane = lane == 0 ? 0ull : ~0ull >> (64 - lane);
  // keys of gathered images g .. g + 3 that lie in no band
  auto gathered = [&](int g, uint64_t(&m)[4]) {
    int key[4];
    uint64_t word[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) key[e] = gpos[min((g + e) * KT + lane, G - 1)];
#pragma unroll
    for (int e = 0; e < 4; ++e) word[e] = any[(first - key[e] / KT) / 64];
#pragma unroll
    for (int e = 0; e < 4; ++e)
      m[e] = __ballot(g + e < g1 && (g + e) * KT + lane < G && !((word[e] >> ((first - key[e] / KT) & 63)) & 1));
  };
  // tiles 64c .. 64c + 63 below the row: bands, and those of them whose offsets are all kept
  auto bands = [&](int c, bool walk_all, uint64_t &full) -> uint64_t {
    uint64_t in = ~0ull;  // tiles 1 .. below of this word
    if (c == 0) in &= ~1ull;
    if (below - 64 * c < 63) in &= (2ull << (below - 64 * c)) - 1;
    const uint64_t band = walk_all ? in : any[c] & in;
    full = all[c] & band;
    return band;
  };
  int n_full = 0, n_part = 0;
  if (w == 0) {
    for (int c = lane; 64 * c <= below; c += 64) {
      uint64_t full;
      const uint64_t band = bands(c, false, full);
      n_full += __popcll(full);
      n_part += __popcll(band & ~full);
    }
    n_full = wave_sum_u32(n_full);
    n_part = wave_sum_u32(n_part);
  } else {
    for (int g = g0; g < g1; g += 4) {
      uint64_t m[4];
      gathered(g, m);
#pragma unroll
      for (int e = 0; e < 4; ++e) n_full += m[e] == ~0ull, n_part += m[e] != 0ull && m[e] != ~0ull;
    }
  }
  if (lane == 0) cnt_sh[w][0] = n_full, cnt_sh[w][1] = n_part;
  __syncthreads();
  int all_items = 0;
  for (int x = 0; x < 4; ++x) all_items += cnt_sh[x][0] + cnt_sh[x][1];
  const bool walk_all = all_items > below;
  if (walk_all) {  // rare: bands only, counted again
    if (w == 0) {
      n_full = 0;
      for (int c = lane; 64 * c <= below; c += 64) {
        uint64_t full;
        bands(c, true, full);
        n_full += __popcll(full);
      }
      n_full = wave_sum_u32(n_full);
    }
    __syncthreads();
    if (lane == 0) cnt_sh[w][0] = w == 0 ? n_full : 0, cnt_sh[w][1] = w == 0 ? below - n_full : 0;
    __syncthreads();
  }
  // order: sink, full gathered images, full bands | masked gathered images, masked bands, diagonal
  int U = n_sink, M = 0, at_full = n_sink, at_part = 0;
  for (int x = 1; x <= 4; ++x) {
    if (x == (w == 0 ? 4 : w)) at_full = U, at_part = M;
    U += cnt_sh[x & 3][0];
    M += cnt_sh[x & 3][1];
  }
  at_part += U;
  const int T = U + M + spb;
  VsItem *__restrict__ out =
      p.items + hb * p.item_stride + vs_items_before(i, p.row0, spb);
  if (w == 0) {
    if (lane == 0) p.hdr[hb * p.nqb + i] = make_int2(U, T);
    if (lane < n_sink) out[lane] = VsItem{(uint32_t)lane, 0, ~0ull};
    if (lane < spb) out[U + M + lane] = VsItem{(uint32_t)(first + lane), 0, p.forced ? ~0ull : bv[first + lane]};
    for (int c = 0; 64 * c <= below; ++c) {
      uint64_t full;
      const uint64_t band = bands(c, walk_all, full), part = band & ~full;
      const int kt = first - 64 * c - lane;
      if ((band >> lane) & 1) {
        const bool f = (full >> lane) & 1;
        out[f ? at_full + __popcll(full & below_lane) : at_part + __popcll(part & below_lane)] =
            VsItem{(uint32_t)kt, 0, f ? ~0ull : bv[kt]};
      }
      at_full += __popcll(full);
      at_part += __popcll(part);
    }
  } else if (!walk_all) {
    for (int g = g0; g < g1; g += 4) {
      uint64_t m[4];
      gathered(g, m);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        if (m[e] == 0ull) continue;
        const int at = m[e] == ~0ull ? at_full++ : at_part++;
        if (lane == 0) out[at] = VsItem{VS_GATHERED | (uint32_t)(g + e), 0, m[e]};
      }
    }
  }
}

// Workgroups 0 .. n_gather - 1 of a head pack one gathered 64-key sub-tile each: K image then V image in the operand order
// of pack_kv_kernel, rows taken at the gathered keys' positions (zero rows beyond the last gathered key).  The others make
// the items of one row each.
template <int D>
__global__ __launch_bounds__(256) void vs_gather_items_kernel(VsTokParams p) {
  constexpr int IMG = KT * D * 2, NCH = IMG / 16, DS = D / 16, VROW = D + 8;
  __shared__ __attribute__((aligned(16))) uint16_t vs[KT * VROW];
  __shared__ int32_t pos[KT];
  const int mt = blockIdx.x, n = blockIdx.y, b = blockIdx.z;
  if (vst_skip(p, b, n)) return;
  if (mt >= p.n_gather) {
    vs_row_items(p, p.row1 - 1 - (mt - p.n_gather), b, n);
    return;
  }
  const int64_t hb = (int64_t)b * p.n_heads + n;
  const int nv = p.cumv[hb * (p.nqb + 1) + p.nqb];
  if (mt * KT >= nv) return;
  const int tid = threadIdx.x, kvh = p.head_ids[n] / p.group;
  if (tid < KT) pos[tid] = (mt * KT + tid < nv) ? p.gpos[hb * (int64_t)p.seq + mt * KT + tid] : -1;
  __syncthreads();
  const int64_t base = (int64_t)b * p.kv_sb + (int64_t)kvh * p.kv_sh;
  char *out = p.gimg + (hb * (p.seq / KT) + mt) * (int64_t)(2 * IMG);
  const u32x4 zero = {0u, 0u, 0u, 0u};
  for (int c = tid; c < KT * (D / 8); c += 256) {
    const int key = c / (D / 8), part = c % (D / 8);
    const u32x4 val = pos[key] >= 0 ? *reinterpret_cast<const u32x4 *>(p.v + base + (int64_t)pos[key] * p.kv_st + part * 8) : zero;
    *reinterpret_cast<u32x4 *>(&vs[key * VROW + part * 8]) = val;
  }
  for (int c = tid; c < NCH; c += 256) {
    const int f = c >> 6, lane = c & 63;
    const int rb = f / DS, ds = f % DS;
    const int key = 32 * rb + (lane & 31), dpos = 16 * ds + 8 * (lane >> 5);
    const u32x4 val = pos[key] >= 0 ? *reinterpret_cast<const u32x4 *>(p.k + base + (int64_t)pos[key] * p.kv_st + dpos) : zero;
    *reinterpret_cast<u32x4 *>(out + (int64_t)c * 16) = val;
  }
  __syncthreads();
  for (int c = tid; c < NCH; c += 256) {
    const int f = c >> 6, lane = c & 63;
    const int db = f >> 2, ks = f & 3;
    const int dd = 32 * db + (lane & 31), h = lane >> 5;
    uint32_t w[4];
#pragma unroll
    for (int e2 = 0; e2 < 4; ++e2) {
      const int e = 2 * e2;
      const int key0 = 16 * ks + ((e < 4) ? (4 * h + e) : (8 + 4 * h + (e - 4)));
      const uint32_t lo = vs[key0 * VROW + dd], hi = vs[(key0 + 1) * VROW + dd];
      w[e2] = lo | (hi << 16);
    }
    u32x4 val = {w[0], w[1], w[2], w[3]};
    *reinterpret_cast<u32x4 *>(out + IMG + (int64_t)c * 16) = val;
  }
}

// Wave-uniform part of an item's mask: two words of the kept-offset bitmap around the window the wavefront's 32
// queries see (word wi0 holds offset position start0 of the first query's window; none for gathered keys), the item's own
// keys and, for a diagonal tile, the position of the first query.
struct VsMaskPre {
  uint64_t w0, w1, v;
  int start0, top0;
  bool diag, live;
};

// One workgroup per (query block, listed head): B/32 wavefronts of 32 queries.  The row's work is the list of 64-key items
// that vs_row_items made, each a packed K/V image pair plus a 64-bit mask per query: kept offsets | the item's own keys,
// causal on the diagonal.
// Same software pipeline as attn_kernel: K and V images ride in LDS rings filled two items ahead, one barrier per
// item; while the matrix pipe runs S[t+1] = K[t+1] Q^T and O += V[t]^T P[t]^T the VALU computes P[t], then masks
// S[t+1] and takes its row max (hand-laid groups).  The masks are built one item ahead from wave-uniform words of
// the bitmaps (scalar loads).  In the pipelined steps a wavefront computes every item (an item without an allowed key
// for its 32 queries contributes zeros); the general step of the last items skips such items.  Softmax reference and second
// normaliser sum as in attn_kernel, but for weights that matter (move_reference).
template <int D, int B>
__global__ __launch_bounds__(B * 2, 2) void vs_token_attn_kernel(VsTokParams p) {
  constexpr int NW = B / 32, SPB = B / KT, IMG = KT * D * 2, STAGE = 2 * IMG, DS = D / 16, DB = D / 32;
  constexpr int RK = 2, RV = 3;             // ring slots: K and V are both fetched two items ahead
  constexpr int CH = IMG / 1024 / NW;       // 1 KiB chunks per wavefront per image
  constexpr int VM_KEEP = CH;               // at the top of an item only the V chunks issued last may be in flight
  static_assert(IMG % (1024 * NW) == 0, "image must split evenly over the wavefronts");
  __shared__ __attribute__((aligned(1024))) char smem[(RK + RV) * IMG];
  const uint32_t lds_k = (uint32_t)(size_t)(__attribute__((address_space(3))) char *)smem;
  const uint32_t lds_v = lds_k + RK * IMG;
  // workgroup -> (XCD, head, query block, batch).  Workgroups are dealt round-robin to the 8 XCDs by the hardware.
  // A task is VST_TASK_ROWS consecutive query blocks of one head, chunk c of its rows from the longest; every XCD gets an
  // eighth of every head's chunks (heads differ widely in how much they keep).  The workgroups resident on an XCD at one
  // time are then a few runs of neighbouring rows, which walk nearly the same items at nearly the same time and find each
  // other's images in the XCD's L2.
  // by_length: chunk c of listed head a belongs to XCD (a + c) % 8, which runs them chunk by chunk, all heads: what is
  // dispatched last is short.  (Head by head, a long row of the last head ended alone: 32 heads of 8K 438 -> 411 us, 16 heads
  // d 64 of 2 x 10K 496 -> 456, dictionary layers of 40K 33.0 -> 32.6 ms.)  In launches of more rows chunk c belongs to XCD (KV
  // head + c) % 8, head by head: heads of one KV head run the same rows side by side, whose bands are the same images.  That
  // shares the rows evenly only over KV heads that are a multiple of 8.  Head by head over chunk by chunk, two prompts each:
  //   query / KV heads    256 rows     384 to 400   448 to 512   640 to 768   1024
  //   32 / 8, blocks 128  1.02         1.00 - 1.02  0.98 - 1.00  0.96 - 0.99  0.97 - 0.98
  //   32 / 8, blocks 64   0.99 - 1.03  0.97 - 1.00  0.99         0.97 - 0.99  0.97 - 0.99
  //   24 to 64 / 8 to 32                            0.97 - 1.00  0.96 - 0.99  0.96 - 0.99
  //   28 / 4, both        1.08 - 1.16  1.04 - 1.12  1.04 - 1.09  1.02 - 1.07  0.99 - 1.04
  //   32 / 4                                        1.04 - 1.07  0.98 - 0.99  0.95 - 0.98
  //   8 / 2, both         1.16 - 1.21  1.03 - 1.15  1.05 - 1.13  1.00 - 1.11  1.04 - 1.05
  const int xcd = blockIdx.x & 7, b = blockIdx.y;
  const int n_act = __builtin_amdgcn_readfirstlane(p.act_n[b]);
  const int rr = (blockIdx.x >> 3) % VST_TASK_ROWS, u = (blockIdx.x >> 3) / VST_TASK_ROWS;
  if (n_act <= 0 || u >= n_act * p.nch8) return;
  const int k = (int)((uint32_t)u / (uint32_t)n_act);
  int at = u - k * n_act;  // position among the chunks 8k .. 8k + 7 of this XCD, one of each head
  int r = 0;
  if (p.by_length) {
    for (;; ++r) {
      const int a0 = (xcd - r) & 7;  // a0, + 8, ..: the heads whose chunk 8k + r is this XCD's
      const int cnt = (n_act >> 3) + (a0 < (n_act & 7) ? 1 : 0);
      if (at < cnt || r == 7) {
        at = a0 + 8 * at;
        break;
      }
      at -= cnt;
    }
  }
  const int n = __builtin_amdgcn_readfirstlane(p.act_pos[(int64_t)b * p.n_heads + at]);
  const int head = p.head_ids[n], kvh = head / p.group;
  if (!p.by_length) r = (xcd - kvh) & 7;
  const int c = 8 * k + r;
  const int i = p.row1 - 1 - (c * VST_TASK_ROWS + rr);
  if (i < p.row0) return;  // the last chunks of a head may be short or empty
  const int tid = threadIdx.x, lane = tid & 63, h = lane >> 5, c32 = lane & 31;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int64_t hb = (int64_t)b * p.n_heads + n;
  const int nwords = p.seq / 64;
  // The kept offsets, read as constant memory: scalar loads, counted apart from the ring refills.  As ordinary global loads
  // (which they became beside the kernel's hand-issued ones) every masked step waited for all refills.
  typedef const __attribute__((address_space(4))) uint64_t *ConstWords;
  const ConstWords bs = (ConstWords)(uintptr_t)(p.bits + (hb * 2 + 1) * nwords);
  const int tq = 32 * w + c32;
  bf16x8 qf[DS];
  {
    const uint16_t *qp = p.q + (int64_t)b * p.q_sb + ((int64_t)i * B + tq) * p.q_st + (int64_t)head * p.q_sh + 8 * h;
#pragma unroll
    for (int ds = 0; ds < DS; ++ds) qf[ds] = *reinterpret_cast<const bf16x8 *>(qp + 16 * ds);
  }
  f32x16 oacc[DB];
#pragma unroll
  for (int db = 0; db < DB; ++db)
#pragma unroll
    for (int r = 0; r < 16; ++r) oacc[db][r] = 0.f;
  // m = running reference (-inf until a query has seen an allowed key), mref = m or 0 while m is -inf (so that no
  // inf - inf is ever formed), l = sum of weights, lc = sum of (bf16(p) - p) over the tiles that matter
  float m = -INFINITY, mref = 0.f, l = 0.f, lc = 0.f;
  bool care = true;

  // the row's items, 64 at a time in registers (item t = lane t % 64 of chunk t / 64), the next chunk ahead
  const VsItem *__restrict__ list = p.items + hb * p.item_stride + vs_items_before(i, p.row0, SPB);
  const int2 row_hdr = p.hdr[hb * p.nqb + i];
  const int U = __builtin_amdgcn_readfirstlane(row_hdr.x), T = __builtin_amdgcn_readfirstlane(row_hdr.y);
  const char *kvbase = p.kvp + ((int64_t)b * p.n_kv_heads + kvh) * (int64_t)(p.seq / KT) * STAGE;
  const char *gbase = p.gimg + hb * (int64_t)(p.seq / KT) * STAGE;
  auto load_chunk = [&](int chunk) -> u32x4 {
    const int t = chunk * 64 + lane;
    return *reinterpret_cast<const u32x4 *>(list + (t < T ? t : T - 1));
  };
  u32x4 it_lane = load_chunk(0), it_next = it_lane;
  int it_chunk = 0;
  if (T > 64) it_next = load_chunk(1);
  auto item = [&](int t) -> VsItem {  // asked for in ascending order; beyond the list: the last item again (never used)
    t = t < T ? t : T - 1;
    if (t >= 64 && (t >> 6) != it_chunk) {
      it_lane = it_next;
      ++it_chunk;
      if (T > (it_chunk + 1) * 64) it_next = load_chunk(it_chunk + 1);
    }
    VsItem it;
    it.code = __builtin_amdgcn_readlane(it_lane[0], t & 63);
    it.v = ((uint64_t)(uint32_t)__builtin_amdgcn_readlane(it_lane[3], t & 63) << 32) |
           (uint32_t)__builtin_amdgcn_readlane(it_lane[2], t & 63);
    return it;
  };
  // this wavefront's share of an item's K image (at most 2^16 images, 2^31 bytes)
  const char *const kv_mine = kvbase + w * CH * 1024, *const g_mine = gbase + w * CH * 1024;
  auto item_src = [&](const VsItem &it) -> const char * {
    return ((it.code & VS_GATHERED) ? g_mine : kv_mine) + (it.code & ~VS_GATHERED) * (uint32_t)STAGE;
  };
  // word idx of a bitmap, 0 outside it (idx is wave-uniform)
  auto uword = [&](int idx) -> uint64_t {
    const int ic = idx < 0 ? 0 : (idx >= nwords ? nwords - 1 : idx);
    const uint64_t x = bs[ic];
    return ic == idx ? x : 0ull;
  };
  // The mask of item t for this lane's query: bit kk = key kk of the item is allowed.
  // Offsets of keys kk = 0 .. 63 of a tile x tiles below the row's first: o0 - kk with o0 = 64 x + tq, so the
  // window W[y] = kept(o0 - 63 + y), reversed, is the mask in key order; the window of the wavefront's first
  // query starts at bit start0, query c32's window c32 bits further.
  auto mask_pre = [&](const VsItem &it, int t) -> VsMaskPre {
    VsMaskPre pre;
    const int x = vs_tiles_below(i * SPB, it.code);
    pre.live = t < T;
    pre.diag = t >= T - SPB;
    pre.start0 = 64 * x + 32 * w - 63;
    pre.top0 = 32 * w + 64 * x;
    pre.v = it.v;
    if (it.code < (uint32_t)(i * SPB)) {  // a tile below the row: x >= 1, both words lie in the bitmap
      pre.w0 = bs[pre.start0 >> 6];
      pre.w1 = bs[(pre.start0 >> 6) + 1];
    } else {
      const int wi0 = (it.code & VS_GATHERED) ? -2 : pre.start0 >> 6;  // floor, also for negative positions
      pre.w0 = uword(wi0);
      pre.w1 = uword(wi0 + 1);
    }
    return pre;
  };
  auto mask_lane = [&](const VsMaskPre &pre) -> uint64_t {
    const int x = (pre.start0 & 63) + c32;  // 1 or 33, + c32: at most 64
    const uint64_t win = x >= 64 ? pre.w1 : (pre.w0 >> x) | ((pre.w1 << 1) << (63 - x));
    uint64_t M = __builtin_bitreverse64(win) | pre.v;
    if (pre.diag) {  // causal: key 64 sub + kk <= tq
      const int top = pre.top0 + c32;
      M &= top >= 63 ? ~0ull : (top < 0 ? 0ull : ((2ull << top) - 1));
    }
    return pre.live ? M : 0ull;
  };

  // every wavefront moves CH chunks of an image into a ring slot
  auto issue_chunk = [&](const char *src, uint32_t slot_base, auto nc) __attribute__((always_inline)) {
    constexpr int OFF = decltype(nc)::value * 1024, HI = OFF & ~4095;  // (a share of more than 4 KiB: block 64, d 128)
    lds_dma16<OFF - HI>(src + HI, lane * 16, slot_base + w * CH * 1024 + HI);
  };
  auto issue_img = [&](const VsItem &it, bool is_v, uint32_t slot_base) __attribute__((always_inline)) {
    const char *src = item_src(it) + (is_v ? IMG : 0);
    static_for<0, CH>([&](auto nc) __attribute__((always_inline)) { issue_chunk(src, slot_base, nc); });
  };
  auto qk = [&](const char *kbuf, f32x16(&s)[2]) {
    const char *kb = kbuf + lane * 16;
#pragma unroll
    for (int rb = 0; rb < 2; ++rb)
#pragma unroll
      for (int r = 0; r < 16; ++r) s[rb][r] = 0.f;
    products_read_ahead<2 * DS>(
        [&](int n) { return *reinterpret_cast<const bf16x8 *>(kb + ((n % 2) * DS + n / 2) * 1024); },
        [&](auto nc, bf16x8 a) __attribute__((always_inline)) {
          constexpr int n = decltype(nc)::value;
          s[n % 2] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, qf[n / 2], s[n % 2], 0, 0, 0);
        });
  };
  // score (rb, r) of this lane is key 32 rb + 8 (r / 4) + 4 h + r % 4 of the item: mw = the mask's word rb with the
  // 4 h already shifted out.  A score whose bit is clear becomes -inf (two instructions: bit -> 0 / -1, select).
  auto mask_score = [&](float s, uint32_t mw, int r) -> float {
    const int bit = 8 * (r >> 2) + (r & 3);
    const uint32_t keep = (uint32_t)((int32_t)(mw << (31 - bit)) >> 31);
    return __builtin_bit_cast(float, (__builtin_bit_cast(uint32_t, s) & keep) | (~keep & 0xff800000u));
  };
  auto apply_mask = [&](f32x16(&s)[2], uint64_t M) {
    const uint32_t mw0 = (uint32_t)M >> (4 * h), mw1 = (uint32_t)(M >> 32) >> (4 * h);
#pragma unroll
    for (int rb = 0; rb < 2; ++rb)
#pragma unroll
      for (int r = 0; r < 16; ++r) s[rb][r] = mask_score(s[rb][r], rb ? mw1 : mw0, r);
  };
  // Scaled scores above this weigh more than 1/SP_CARE of the row so far, or outgrow the reference by more than the slack.
  auto matters_above = [&]() -> float { return fminf(m + SP_MAX_SLACK, mref + fast_log2(l * (1.f / SP_CARE))); };
  // mx = raw row max of a fresh (masked) tile, -inf if the query has no allowed key in it; thr = matters_above() after the
  // tiles before.  Returns alpha = 2^(m_old - m_new) for the O accumulators (1 while nothing has been accumulated) and notes
  // in care whether the tile's largest weight matters to the row.  A weight that does becomes the reference, and is then
  // exactly 1 in bf16.  Items come in no order of weight (those without masks first): a reference that only keeps within
  // SP_MAX_SLACK of the max may lag behind the one key that rules a row, whose weight is then rounded.  2-norm of the error
  // against 64 bits, 31 prompts of 1K to 128K tokens x 3 seeds, next to whole key blocks as bands, all gathered keys before
  // them: 0.9992 to 1.0126 of it with these items, 0.913 to 0.998 with this rule.  Times 8K 489.6 -> 493.1 us, 40K 3866 ->
  // 3892, 128K 55.41 -> 55.83 ms, 3.9K in blocks of 64 222.2 -> 226.6 us (3 % more with an exponential in thr's place).
  auto move_reference = [&](float mx, float thr) -> float {
    const float top = mx * p.c;
    const bool matters = top > thr;
    care = any_lane(matters);
    const float m_new = matters ? fmaxf(m, top) : m;
    const float mref_new = (m_new == -INFINITY) ? 0.f : m_new;
    const float alpha = (m == -INFINITY) ? 1.f : fast_exp2(m - mref_new);
    m = m_new;
    mref = mref_new;
    l *= alpha;
    lc *= alpha;
    return alpha;
  };
  auto tile_max = [&](f32x16(&s)[2]) -> float {
    float mx = fmaxf(s[0][0], s[0][1]);
#pragma unroll
    for (int rb = 0; rb < 2; ++rb)
#pragma unroll
      for (int r = (rb == 0 ? 2 : 0); r < 16; r += 2) mx = max3f(mx, s[rb][r], s[rb][r + 1]);
    return move_reference(max_xor32(mx), matters_above());
  };
  auto tile_exp = [&](f32x16(&s)[2], bf16x8(&pb)[4]) {
    float rs0 = 0.f, rs1 = 0.f;
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
      u32x4 tt;
#pragma unroll
      for (int e2 = 0; e2 < 4; ++e2) {
        const int r = 8 * (ks & 1) + 2 * e2;
        const float p0 = fast_exp2(__builtin_fmaf(s[ks >> 1][r], p.c, -mref));
        const float p1 = fast_exp2(__builtin_fmaf(s[ks >> 1][r + 1], p.c, -mref));
        rs0 += p0;
        rs1 += p1;
        tt[e2] = pack_bf16(p0, p1);
      }
      pb[ks] = __builtin_bit_cast(bf16x8, tt);
    }
    const float rs = sum_xor32(rs0 + rs1);
    l += rs;
    lc += sum_xor32(sum_bf16x8(pb[0]) + sum_bf16x8(pb[1]) + sum_bf16x8(pb[2]) + sum_bf16x8(pb[3])) - rs;
  };
  auto rescale = [&](float alpha) {
    if (any_lane(alpha != 1.f)) {
#pragma unroll
      for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int r = 0; r < 16; ++r) oacc[db][r] *= alpha;
    }
  };
  auto pv = [&](const char *vbuf, const bf16x8(&pb)[4]) {
    const char *vb = vbuf + lane * 16;
    products_read_ahead<4 * DB>(
        [&](int n) { return *reinterpret_cast<const bf16x8 *>(vb + ((n % DB) * 4 + n / DB) * 1024); },
        [&](auto nc, bf16x8 a) __attribute__((always_inline)) {
          constexpr int n = decltype(nc)::value;
          oacc[n % DB] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, pb[n / DB], oacc[n % DB], 0, 0, 0);
        });
  };

  // byte offsets of the V slots: of item t's image and of the one before it, which item t + 2 refills (as in attn_kernel)
  uint32_t v_now = 0, v_old = (RV - 1) * IMG;
  auto next_v = [&]() {
    v_old = v_now;
    v_now = v_now == (RV - 1) * IMG ? 0 : v_now + IMG;
  };
  // On entry to step t: s_cur = masked raw S[t] with its max folded into m / l / O (if this wavefront has anything
  // in item t), Mn = the mask of item t+1, it2 / pre2 = item t+2 and the uniform part of its mask.  Every step
  // returns the mask of item t+2.
  // fast step: this wavefront has work in items t and t+1.  One basic block up to the rescale test.
  auto fast_step = [&](int t, const VsItem &it2, const VsMaskPre &pre2, f32x16(&s_cur)[2], f32x16(&s_next)[2],
                       uint64_t Mn, auto masked_tag) __attribute__((always_inline)) -> uint64_t {
    constexpr bool MASKED = decltype(masked_tag)::value;
    wait_vm<VM_KEEP>();
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    const char *ksrc = item_src(it2), *vsrc = ksrc + IMG;
    const uint32_t kslot = lds_k + ((t + 2) % RK) * IMG, vslot = lds_v + v_old;
    const char *kb = smem + ((t + 1) % RK) * IMG + lane * 16;
    const char *vb = smem + RK * IMG + v_now + lane * 16;
    next_v();
    const uint32_t mw0 = (uint32_t)Mn >> (4 * h), mw1 = (uint32_t)(Mn >> 32) >> (4 * h);
    // NM groups, each = one MFMA + half of two LDS reads (PF fragments ahead) + a slice of the VALU work:
    //   groups 0 .. NQ-1   : S[t+1] += K frag * Q frag ; exp / row-sum / bf16 pack of S[t]
    //   groups NQ .. NM-1  : O += V frag * P frag       ; mask and row max of S[t+1], reference update,
    //                                                     the mask of item t+2
    constexpr int NQ = 2 * DS, NP = 4 * DB, NM = NQ + NP;
    // Reads and refills go two at a time with one wait a pair, as in attn_kernel (with three fragments ahead and each wait left
    // to the compiler: n = 3904 d128 block 64 220.8 -> 216.2 us, 40K dictionary layers 31.56 -> 31.29 ms, 8K 412.1 -> 409.5 us,
    // 128K 38.18 -> 37.97 ms).  A wavefront that issues all eight chunks (d128, block 64) keeps single refills.
    constexpr int PF = 4, MAXTAIL = 4;
    constexpr int NF = PF + 2;
    auto frag = [&](int g) -> bf16x8 {
      if (g < NQ) return *reinterpret_cast<const bf16x8 *>(kb + ((g % 2) * DS + g / 2) * 1024);
      const int np = g - NQ;
      return *reinterpret_cast<const bf16x8 *>(vb + ((np % DB) * 4 + np / DB) * 1024);
    };
    bf16x8 fr[NF];
    bf16x8 pb[4];
    u32x4 pt;
    float rs0 = 0.f, rs1 = 0.f, mx = 0.f, mx_odd = 0.f, alpha = 1.f, rs_tile = 0.f, thr = 0.f;
    const bool care_t = care;  // set when this tile's max was taken
    float xa[16], xb[16];
    uint64_t Mnn = 0ull;
#pragma unroll
    for (int g = 0; g < PF; ++g) fr[g] = frag(g);
    __builtin_amdgcn_sched_barrier(0);
    static_for<0, NM>([&](auto gc) __attribute__((always_inline)) {
      constexpr int g = decltype(gc)::value;
      if constexpr (g % 2 == 0) {
        wait_lds<(g + PF <= NM ? PF : NM - g) - 2>();  // fragments g and g + 1 are there
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (g + PF < NM) {
          fr[(g + PF) % NF] = frag(g + PF);
          fr[(g + PF + 1) % NF] = frag(g + PF + 1);
        }
      }
      if (g < NQ) {
        if (g < 2) {
          f32x16 z;
#pragma unroll
          for (int r = 0; r < 16; ++r) z[r] = 0.f;
          s_next[g] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr[g % NF], qf[0], z, 0, 0, 0);
        } else {
          s_next[g % 2] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr[g % NF], qf[g / 2], s_next[g % 2], 0, 0, 0);
        }
      }
      // exp units u (2 scores each), three stages in consecutive groups
#pragma unroll
      for (int u = 0; u < 16; ++u) {
        const int gu = u * NQ / 16;
        const int ks = u / 4, e2 = u % 4, r = 8 * (ks & 1) + 2 * e2;
        if (gu == g) {
          xa[u] = __builtin_fmaf(s_cur[ks >> 1][r], p.c, -mref);
          xb[u] = __builtin_fmaf(s_cur[ks >> 1][r + 1], p.c, -mref);
        }
        if (gu + 1 == g) {
          xa[u] = fast_exp2(xa[u]);
          xb[u] = fast_exp2(xb[u]);
        }
        if (gu + 2 == g) {
          rs0 = u == 0 ? xa[u] : rs0 + xa[u];
          rs1 = u == 0 ? xb[u] : rs1 + xb[u];
          pt[e2] = pack_bf16(xa[u], xb[u]);
          if (e2 == 3) pb[ks] = __builtin_bit_cast(bf16x8, pt);
        }
      }
      if (g == NQ + 2) {
        rs_tile = sum_xor32(rs0 + rs1);
        l += rs_tile;
      }
      if (g == NQ + 4) thr = matters_above();
      {
        constexpr int GAP = NM / (2 * CH);  // groups between two chunk loads
        constexpr int x = g / GAP;
        if constexpr (CH <= 4) {
          if constexpr (g % (2 * GAP) == 1 && x < CH) lds_dma16_pair<x * 1024>(ksrc, lane * 16, kslot + w * CH * 1024);
          if constexpr (g % (2 * GAP) == 1 && x >= CH && x < 2 * CH)
            lds_dma16_pair<(x - CH) * 1024>(vsrc, lane * 16, vslot + w * CH * 1024);
        } else {
          if constexpr (g % GAP == 1 && x < CH) issue_chunk(ksrc, kslot, std::integral_constant<int, x>{});
          if constexpr (g % GAP == 1 && x >= CH && x < 2 * CH) issue_chunk(vsrc, vslot, std::integral_constant<int, x - CH>{});
        }
      }
      if (g >= NQ) {
        const int np = g - NQ;
        oacc[np % DB] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr[g % NF], pb[np / DB], oacc[np % DB], 0, 0, 0);
        // S[t+1]: 16 units of two scores, masked one group before they enter the row max; the reference update
        // MAXTAIL groups before the end
#pragma unroll
        for (int u = 0; u < 16; ++u) {
          const int gm = 2 + u * (NP - 2 - MAXTAIL) / 16;
          const int rb = u / 8, r = 2 * (u % 8);
          if (MASKED && gm - 1 == np) {
            s_next[rb][r] = mask_score(s_next[rb][r], rb ? mw1 : mw0, r);
            s_next[rb][r + 1] = mask_score(s_next[rb][r + 1], rb ? mw1 : mw0, r + 1);
          }
          if (gm == np) {
            const float a0 = s_next[rb][r], a1 = s_next[rb][r + 1];
            float &m2 = u % 2 ? mx_odd : mx;  // two chains
            m2 = (u < 2) ? fmaxf(a0, a1) : max3f(m2, a0, a1);
          }
        }
        if (np == NP - MAXTAIL) alpha = move_reference(max_xor32(fmaxf(mx, mx_odd)), thr);
        if (MASKED && np == NP - 2) Mnn = mask_lane(pre2);
      }
      __builtin_amdgcn_sched_barrier(0);
    });
    if (care_t) {  // rare: the tile summed again as PV saw it (alpha already holds the move after this tile)
      asm volatile("" ::: "memory");  // a real branch: not to be evaluated on every step
      lc += (sum_xor32(sum_bf16x8(pb[0]) + sum_bf16x8(pb[1]) + sum_bf16x8(pb[2]) + sum_bf16x8(pb[3])) - rs_tile) * alpha;
    }
    rescale(alpha);
    return Mnn;
  };
  // general step (the last items of a row): a wavefront whose 32 queries have no allowed key in an item skips its
  // matrix work; optional next item.  Returns whether s_next holds a tile.
  auto slow_step = [&](int t, const VsItem &it2, f32x16(&s_cur)[2], f32x16(&s_next)[2], uint64_t Mn,
                       bool act_cur) __attribute__((always_inline)) -> bool {
    wait_vm<VM_KEEP>();
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    issue_img(it2, false, lds_k + ((t + 2) % RK) * IMG);
    issue_img(it2, true, lds_v + v_old);
    const char *v_cur = smem + RK * IMG + v_now;
    next_v();
    const bool act_next = any_lane(Mn != 0ull);
    if (act_next) qk(smem + ((t + 1) % RK) * IMG, s_next);
    if (act_cur) {
      bf16x8 pb[4];
      tile_exp(s_cur, pb);
      pv(v_cur, pb);
    }
    if (act_next) {
      if (!__all(Mn == ~0ull)) apply_mask(s_next, Mn);
      rescale(tile_max(s_next));
    }
    return act_next;
  };

  // The leading items whose masks are all ones (the sink block, the full gathered items) go through the step
  // without the mask, the others through the step with it, both in pairs (the S tiles swap roles); the last one
  // or two items take the general step.  npairs counts the allowed (query, key) pairs of this lane's query.
  int npairs = 0;  // at most 64 per item
  {
    f32x16 s_a[2], s_b[2];
    const int nfu = (U > 1) ? ((U - 1) & ~1) : 0;   // steps t < nfu: item t+1 is unmasked
    const int nfm = (T - 1 - nfu) & ~1;             // steps nfu <= t < nfu + nfm: the masked step (item t+1 exists)
    const VsItem it0 = item(0);
    VsItem it1 = item(1);
    const uint64_t M0 = mask_lane(mask_pre(it0, 0));
    npairs += __popcll(M0) + KT * nfu;  // items 1 .. nfu are full; the later ones are counted as their masks are built
    // prologue: K and V images of items 0 and 1
    issue_img(it0, true, lds_v);
    issue_img(it0, false, lds_k);
    issue_img(it1, true, lds_v + IMG);
    issue_img(it1, false, lds_k + IMG);
    wait_vm<0>();
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    qk(smem, s_a);
    if (!__all(M0 == ~0ull)) apply_mask(s_a, M0);
    tile_max(s_a);  // O is still zero: nothing to rescale
    int t = 0;
    VsItem it2 = item(2), it3 = item(3);  // it1, it2, it3: items t + 1, t + 2, t + 3
    {
      const VsMaskPre nopre{};
      for (; t < nfu; t += 2) {
        const VsItem it4 = item(t + 4), it5 = item(t + 5);
        fast_step(t, it2, nopre, s_a, s_b, 0ull, std::false_type{});
        fast_step(t + 1, it3, nopre, s_b, s_a, 0ull, std::false_type{});
        it1 = it3;
        it2 = it4;
        it3 = it5;
      }
    }
    uint64_t Mn = mask_lane(mask_pre(it1, t + 1));
    npairs += __popcll(Mn);
    {
      VsMaskPre pre2 = mask_pre(it2, t + 2);
      for (const int tend = t + nfm; t < tend; t += 2) {
        const VsMaskPre pre3 = mask_pre(it3, t + 3);
        const VsItem it4 = item(t + 4);
        const uint64_t Mb = fast_step(t, it2, pre2, s_a, s_b, Mn, std::true_type{});
        const VsMaskPre pre4 = mask_pre(it4, t + 4);
        const VsItem it5 = item(t + 5);
        Mn = fast_step(t + 1, it3, pre3, s_b, s_a, Mb, std::true_type{});
        npairs += __popcll(Mb) + __popcll(Mn);
        it2 = it4;
        pre2 = pre4;
        it3 = it5;
      }
    }
    // one or two items are left (t + 2 >= T: no item t+2, its mask is empty)
    const bool act = slow_step(t, it2, s_a, s_b, Mn, true);
    if (t + 1 < T) slow_step(t + 1, it2, s_b, s_a, 0ull, act);
    wait_vm<0>();  // drain the rings' look-ahead loads before the LDS is released
  }
  {
    const float inv = (l > 0.f) ? 1.f / (l + lc) : 0.f;
    uint16_t *op = p.o + (int64_t)b * p.o_sb + ((int64_t)i * B + tq) * p.o_st + (int64_t)head * p.o_sh;
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
      for (int gq = 0; gq < 4; ++gq) {
        u32x2 tt;
        tt[0] = pack_bf16(oacc[db][4 * gq] * inv, oacc[db][4 * gq + 1] * inv);
        tt[1] = pack_bf16(oacc[db][4 * gq + 2] * inv, oacc[db][4 * gq + 3] * inv);
        *reinterpret_cast<u32x2 *>(op + 32 * db + 8 * gq + 4 * h) = tt;
      }
  }
  if (p.pairs) {  // pairs of the pattern in this row: every query counted once (its two half-lanes hold the same mask)
#pragma unroll
    for (int off = 16; off >= 1; off >>= 1) npairs += __shfl_xor(npairs, off, 64);
    if (lane == 0) atomicAdd(reinterpret_cast<unsigned long long *>(p.pairs + hb), (unsigned long long)(unsigned)npairs);
  }
}

}  // namespace

#endif
