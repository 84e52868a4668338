// Search Vertical Slash Pattern (Alg. 5) and its conversion to key-block lists.
#ifndef SP_VERTICAL_SLASH_KERNELS_H
#define SP_VERTICAL_SLASH_KERNELS_H
#include "sp_common.h"
#include "attn_kernel.h"
#include "mask_kernel.h"
#include "global_select_kernels.h"

namespace {

// ---- Search Vertical Slash Pattern (Alg. 5) ------------------------------------------------------
// Q_hat = the last `block` queries, A_hat = their causal softmax over every key.  Two passes over K form the logits by
// MFMA and keep them on chip: the first leaves row reference and row sum per part of the keys, the second merges those,
// forms the logits again and adds up the normalised vertical sums a_v[s] and slash sums a_s[t - s].  (K is read twice by
// every listed head, 2 x 32 MiB per 128K keys of d 128, from L2 where heads share a KV head; a slab of logits in memory,
// written once and read three times, was 64 MiB per query head.)  The parts follow from the number of key blocks alone,
// and with them the order of every sum: how many parts a workgroup takes depends on the heads of the call, a head's sums
// do not.  The vector selection above keeps the shortest prefixes reaching gamma, and the kept keys / offsets become
// per-row key-block lists.
struct VsParams {
  const uint16_t *q, *k;
  int64_t q_sb, q_st, q_sh, k_sb, k_st, k_sh;
  int seq, group, n_heads, n_q_heads;
  int n_parts, part_blocks;  // the keys in parts of part_blocks key blocks, the last one may be shorter
  int n_chunks, chunk;   // a workgroup's chunk: `chunk` key blocks, whole parts
  float c;               // softmax scale * log2(e)
  float2 *part;          // [b][n][n_parts][B]  row reference (log2 domain) and row sum of a part
  float *sums;           // [b][n][2][seq] a_v then a_s
  float *low;            // [b][n][n_chunks][B] lower diagonals of each chunk's last key block (see VsBorders)
  const int32_t *role;   // optional [b][n_q_heads]: only heads whose entry is -1 are processed
  int32_t head_ids[SP_MAX_HEADS];
};
__device__ __forceinline__ bool vs_skip(const VsParams &p, int b, int n) {
  return p.role != nullptr && p.role[(int64_t)b * p.n_q_heads + p.head_ids[n]] != -1;
}
// (m, l) := (m, l) joined with (m2, l2), sums l relative to 2^m; -inf with 0 is the empty sum
__device__ __forceinline__ void vs_join(float &m, float &l, float m2, float l2) {
  const float mn = fmaxf(m, m2), ref = (mn == -INFINITY) ? 0.f : mn;
  l = l * fast_exp2(m - ref) + l2 * fast_exp2(m2 - ref);
  m = mn;
}

// Pass 1: causal softmax statistics of the B query rows over the parts of one chunk.  Bound by MFMA and the exponentials
// (one per logit); a wavefront owns 32 queries (one per lane, as in attn_kernel, so nothing is exchanged before the end)
// and the wavefronts share 64-key tiles of K in LDS, fetched one tile ahead.  References are whole numbers (the maximum
// rounded up): moving from one to another is then exact, and the weights of pass 2 are the ones that the normaliser added
// up.  With the maximum itself as reference, the slash sums were up to 6 % further from 64 bits than with one global
// maximum per row, now they are 2 to 6 % nearer, at the same speed.
template <int D, int B>
__global__ __launch_bounds__(B * 2) void vs_rowpart_kernel(VsParams p) {
  constexpr int DS = D / 16, NT = B * 2, IMG = KT * D * 2, NP = IMG / 16 / NT;
  __shared__ __attribute__((aligned(16))) char kt_sh[2][IMG];
  const int chunk = blockIdx.x, n = blockIdx.y, b = blockIdx.z;
  if (vs_skip(p, b, n)) return;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, h = lane >> 5, c = lane & 31;
  const int head = p.head_ids[n], nkb = p.seq / B, t0 = p.seq - B;
  const int64_t hb = (int64_t)b * p.n_heads + n;
  const int b0 = chunk * p.chunk, b1 = min(b0 + p.chunk, nkb);
  const int u0 = b0 * (B / KT), u1 = b1 * (B / KT), upart = p.part_blocks * (B / KT);
  const uint16_t *kbase = p.k + (int64_t)b * p.k_sb + (int64_t)(head / p.group) * p.k_sh;
  // piece x of this thread: 16 bytes of fragment f = rb * DS + ds of the tile, in operand order
  u32x4 stage[NP];
  auto fetch = [&](int u) {
#pragma unroll
    for (int x = 0; x < NP; ++x) {
      const int f = (tid + x * NT) >> 6;
      const int key = 32 * (f / DS) + c, dpos = 16 * (f % DS) + 8 * h;
      stage[x] = *reinterpret_cast<const u32x4 *>(kbase + (int64_t)(u * KT + key) * p.k_st + dpos);
    }
  };
  auto put = [&](int buf) {
#pragma unroll
    for (int x = 0; x < NP; ++x) *reinterpret_cast<u32x4 *>(kt_sh[buf] + (tid + x * NT) * 16) = stage[x];
  };
  fetch(u0);
  const int tq = 32 * w + c;
  bf16x8 qf[DS];
  const uint16_t *qp = p.q + (int64_t)b * p.q_sb + (int64_t)(t0 + tq) * p.q_st + (int64_t)head * p.q_sh + 8 * h;
#pragma unroll
  for (int ds = 0; ds < DS; ++ds) qf[ds] = *reinterpret_cast<const bf16x8 *>(qp + 16 * ds);
  put(0);
  __syncthreads();
  float m = -INFINITY, l = 0.f;
  int uend = u0 + upart, part = b0 / p.part_blocks;  // end and number of the part at hand
  for (int u = u0; u < u1; ++u) {
    const int buf = (u - u0) & 1;
    if (u + 1 < u1) fetch(u + 1);
    f32x16 s[2];
#pragma unroll
    for (int rb = 0; rb < 2; ++rb)
#pragma unroll
      for (int r = 0; r < 16; ++r) s[rb][r] = 0.f;
#pragma unroll
    for (int ds = 0; ds < DS; ++ds)
#pragma unroll
      for (int rb = 0; rb < 2; ++rb) {
        const bf16x8 a = *reinterpret_cast<const bf16x8 *>(kt_sh[buf] + (rb * DS + ds) * 1024 + lane * 16);
        s[rb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, qf[ds], s[rb], 0, 0, 0);
      }
    if (u * KT >= t0) {
#pragma unroll
      for (int rb = 0; rb < 2; ++rb)
#pragma unroll
        for (int r = 0; r < 16; ++r)
          if (u * KT + 32 * rb + 8 * (r >> 2) + 4 * h + (r & 3) > t0 + tq) s[rb][r] = -INFINITY;
    }
    float mx = fmaxf(s[0][0], s[1][0]);
#pragma unroll
    for (int r = 1; r < 16; ++r) mx = fmaxf(mx, fmaxf(s[0][r], s[1][r]));
    const float mn = fmaxf(m, ceilf(mx * p.c)), ref = (mn == -INFINITY) ? 0.f : mn;
    float l0 = 0.f, l1 = 0.f;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      l0 += fast_exp2(__builtin_fmaf(s[0][r], p.c, -ref));
      l1 += fast_exp2(__builtin_fmaf(s[1][r], p.c, -ref));
    }
    l = l * fast_exp2(m - ref) + (l0 + l1);
    m = mn;
    if (u + 1 < u1) put(buf ^ 1);
    if (u + 1 == uend || u + 1 == u1) {
      const float m2 = __shfl_xor(m, 32, 64), l2 = __shfl_xor(l, 32, 64);
      vs_join(m, l, m2, l2);
      if (h == 0) p.part[(hb * p.n_parts + part) * B + tq] = make_float2(m, l);
      m = -INFINITY;
      l = 0.f;
      uend += upart;
      ++part;
    }
    __syncthreads();
  }
}

// Pass 2: a_v and a_s of one chunk of key blocks.  Queries are MFMA rows and keys columns (a wavefront owns 32 keys, one
// per lane), so the vertical sums stay in a lane; the weights of 32 queries x B keys go through LDS, double buffered,
// each query's row shifted by its number so that a diagonal is a column (what a row leaves free stays zero): thread q
// adds column q, all reads at fixed distances, into the block's 2B - 1 diagonals, of which the lower half joins the
// upper half of the next key block.  (First written with a row's keys unshifted and two predicated sums per thread:
// 734 us at 128K keys, 75 us at 8K.)  At the ends of a chunk, where the halves belong to two workgroups, both are stored
// and the selection's first kernel adds them up (VsBorders).  Everything is added in a fixed order.
// Both passes, 128K keys, 32 heads of d 128: 2646 -> 588 us; 8K keys: 153 -> 63 us (with the slab -> now).
template <int D, int B>
__global__ __launch_bounds__(B * 2) void vs_sums_kernel(VsParams p) {
  constexpr int DS = D / 16, NT = B * 2, NQ = B / 32;
  constexpr int PS = B + 41;  // one float more than the distance of two writes: 4 (PS - 1) = 32 mod 64 banks
  __shared__ __attribute__((aligned(16))) char q_sh[B * D * 2];
  __shared__ __attribute__((aligned(16))) float pt[2][32 * PS];
  __shared__ __attribute__((aligned(16))) float mx_sh[B], inv_sh[B];
  __shared__ float diag_sh[2 * B + 1];  // [t - key + B], entry 2B stays zero
  const int chunk = blockIdx.x, n = blockIdx.y, b = blockIdx.z;
  if (vs_skip(p, b, n)) return;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, h = lane >> 5, c = lane & 31;
  const int head = p.head_ids[n], nkb = p.seq / B, t0 = p.seq - B;
  const int64_t hb = (int64_t)b * p.n_heads + n;
  const int b0 = chunk * p.chunk, b1 = min(b0 + p.chunk, nkb);
  const uint16_t *kbase =
      p.k + (int64_t)b * p.k_sb + (int64_t)(32 * w + c) * p.k_st + (int64_t)(head / p.group) * p.k_sh + 8 * h;
  bf16x8 kf[DS], kn[DS];
#pragma unroll
  for (int ds = 0; ds < DS; ++ds)
    kn[ds] = *reinterpret_cast<const bf16x8 *>(kbase + (int64_t)b0 * B * p.k_st + 16 * ds);
  const uint16_t *qbase = p.q + (int64_t)b * p.q_sb + (int64_t)t0 * p.q_st + (int64_t)head * p.q_sh;
#pragma unroll
  for (int x = 0; x < NQ * DS * 64 / NT; ++x) {
    const int f = (tid + x * NT) >> 6;
    const u32x4 val =
        *reinterpret_cast<const u32x4 *>(qbase + (int64_t)(32 * (f / DS) + c) * p.q_st + 16 * (f % DS) + 8 * h);
    *reinterpret_cast<u32x4 *>(q_sh + (tid + x * NT) * 16) = val;
  }
  const int d = tid & (B - 1), half = tid / B;
  {
    float m = -INFINITY, l = 0.f;
#pragma unroll 8
    for (int x = half; x < p.n_parts; x += 2) {
      const float2 y = p.part[(hb * p.n_parts + x) * B + d];
      vs_join(m, l, y.x, y.y);
    }
    if (half) diag_sh[d] = m, diag_sh[B + d] = l;
    for (int x = tid; x < 64 * PS; x += NT) (&pt[0][0])[x] = 0.f;
    __syncthreads();
    if (!half) {
      vs_join(m, l, diag_sh[d], diag_sh[B + d]);
      mx_sh[d] = m;
      inv_sh[d] = 1.f / l;
      diag_sh[d] = diag_sh[B + d] = 0.f;
      if (d == 0) diag_sh[2 * B] = 0.f;
    }
    __syncthreads();
  }
  float *sv = p.sums + hb * 2 * p.seq, *ss = sv + p.seq;
  float low = 0.f;  // lower diagonals of the previous key block
  for (int kb = b0; kb < b1; ++kb) {
#pragma unroll
    for (int ds = 0; ds < DS; ++ds) kf[ds] = kn[ds];
    if (kb + 1 < b1) {
#pragma unroll
      for (int ds = 0; ds < DS; ++ds)
        kn[ds] = *reinterpret_cast<const bf16x8 *>(kbase + (int64_t)(kb + 1) * B * p.k_st + 16 * ds);
    }
    const bool last = kb == nkb - 1;
    float av = 0.f;
#pragma unroll
    for (int qt = 0; qt < NQ; ++qt) {
      f32x16 acc;
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[r] = 0.f;
#pragma unroll
      for (int ds = 0; ds < DS; ++ds) {
        const bf16x8 a = *reinterpret_cast<const bf16x8 *>(q_sh + (qt * DS + ds) * 1024 + lane * 16);
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, kf[ds], acc, 0, 0, 0);
      }
      float *put = pt[qt & 1] + 31 + 32 * w + c + 4 * h * (PS - 1);
#pragma unroll
      for (int r4 = 0; r4 < 4; ++r4) {
        const int t = 8 * r4 + 4 * h;
        const float4 mx = *reinterpret_cast<const float4 *>(&mx_sh[32 * qt + t]);
        const float4 inv = *reinterpret_cast<const float4 *>(&inv_sh[32 * qt + t]);
        const float mm[4] = {mx.x, mx.y, mx.z, mx.w}, ii[4] = {inv.x, inv.y, inv.z, inv.w};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          float x = fast_exp2(__builtin_fmaf(acc[4 * r4 + e], p.c, -mm[e])) * ii[e];
          if (last) x = (32 * w + c > 32 * qt + t + e) ? 0.f : x;
          av += x;
          put[(8 * r4 + e) * (PS - 1)] = x;
        }
      }
      __syncthreads();
      if (tid < B + 31) {
        const float *get = pt[qt & 1] + tid;
        float x0 = 0.f, x1 = 0.f;
#pragma unroll
        for (int r = 0; r < 32; r += 2) {
          x0 += get[r * PS];
          x1 += get[(r + 1) * PS];
        }
        diag_sh[32 * qt + 31 - tid + B] += x0 + x1;
      }
    }
    av = sum_xor32(av);
    if (h == 0) sv[kb * B + 32 * w + c] = av * (1.f / B);
    __syncthreads();
    if (!half) {
      const float before = diag_sh[B - d], after = diag_sh[2 * B - d];
      diag_sh[B - d] = 0.f;
      diag_sh[2 * B - d] = 0.f;
      const int o = t0 - kb * B + B - d;  // offset that `after` and the previous block's `before` add up to
      if (kb > b0)
        ss[o] = (low + after) * (1.f / B);
      else if (kb > 0)
        ss[o] = after;  // a border: the previous chunk's `low` and the factor come later
      else if (d > 0)
        ss[o] = after * (1.f / B);
      low = before;
    }
  }
  if (!half) {
    if (b1 < nkb)
      p.low[(hb * p.n_chunks + chunk) * B + d] = low;
    else if (d == 0)
      ss[0] = low * (1.f / B);
  }
}

// Kept keys / offsets -> key-block lists.  flags[b][n][2][nkb] come from the vector selection with rows of
// `block` entries: bit 0 = a kept entry in the row, bit 1 = a kept entry other than the row's first.  Block
// (i, j) holds a kept key iff row j of the vertical flags has bit 0; its token pairs realise the offsets
// (i-j)B - (B-1) .. (i-j)B + (B-1): all of slash row i-j, and slash row i-j-1 without its first entry.
__global__ __launch_bounds__(256) void vs_block_lists_kernel(VsParams p, const int32_t *__restrict__ flags, int nkb,
                                                             int forced, int by_head, int32_t *__restrict__ kb_idx,
                                                             int32_t *__restrict__ kb_cnt) {
  const int lane = threadIdx.x & 63;
  const int i = blockIdx.x * 4 + (threadIdx.x >> 6), n = blockIdx.y, b = blockIdx.z;
  if (i >= nkb || vs_skip(p, b, n)) return;
  const int head = p.head_ids[n], n_heads = p.n_heads, n_q_heads = p.n_q_heads;
  const int32_t *fv = flags + (((int64_t)b * n_heads + n) * 2) * nkb, *fs = fv + nkb;
  // lists are stored per listed position, or per query head when they serve a whole layer
  const int64_t orow = (by_head ? ((int64_t)b * n_q_heads + head) : ((int64_t)b * n_heads + n)) * nkb + i;
  int32_t *out = kb_idx + orow * nkb;
  const uint64_t lt = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
  uint32_t n_out = 0;
  for (int j0 = 0; j0 <= i; j0 += 64) {
    const int j = j0 + lane;
    bool sel = false;
    if (j <= i) {
      const int dlt = i - j;
      sel = (fv[j] & 1) || (fs[dlt] & 1) || (dlt >= 1 && (fs[dlt - 1] & 2)) || (forced && (j == 0 || j == i));
    }
    const uint64_t smask = __ballot(sel);
    if (sel) out[n_out + __popcll(smask & lt)] = j;
    n_out += __popcll(smask);
  }
  for (int pos = n_out + lane; pos < nkb; pos += 64) out[pos] = -1;
  if (lane == 0) kb_cnt[orow] = (int32_t)n_out;
}

}  // namespace

#endif
