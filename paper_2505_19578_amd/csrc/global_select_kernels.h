// Alg. 2 over a flattened map (or over vectors) in exact integers: histogram passes, tie ranking, list emission.
#ifndef SP_GLOBAL_SELECT_KERNELS_H
#define SP_GLOBAL_SELECT_KERNELS_H
#include "sp_common.h"
#include "mask_kernel.h"

namespace {

// ---- Alg. 2 over the flattened map, exact integers -------------------------------------------
// With u = the 24-bit score, T = ceil(gamma_q * total / 2^24): the kept set is every entry above
// a threshold value v* plus the first `need` entries equal to v* in flat (row-major) order, where v*
// is the largest value with sum_{u >= v*} u >= T.  v* is found by two 12-bit histogram passes
// (sums of u per bin), the ties are ranked by a per-row count and a prefix sum over rows.
constexpr int GS_BINS = 4104;  // 4097 used by the first pass (u can equal 2^24), padded
struct GselState {
  uint64_t T, above, need;
  uint32_t bin_hi, vstar;
  uint32_t pad[8];
};
static_assert(sizeof(GselState) == 64, "GselState layout");

struct GselView {
  unsigned long long *hist1, *hist2;
  GselState *state;
  uint32_t *row_ties, *row_before;
};
// Shape of the maps a selection runs over.  A causal block map is n x n with only j <= row present; a plain
// vector of length n_rows * n_cols is a rectangular map whose row-major order is the vector's order.
struct GselGeom {
  int n_rows, n_cols;
  int tri;              // 1: entries j <= row only; 0: all n_cols entries of a row
  const int32_t *role;  // optional [n_maps / per_head]: a map is processed only if its owner's entry is -1
  int per_head;
};
__device__ __forceinline__ int gsel_width(const GselGeom &g, int row) { return g.tri ? row + 1 : g.n_cols; }
__device__ __forceinline__ bool gsel_skip(const GselGeom &g, int map) {
  return g.role != nullptr && g.role[map / g.per_head] != -1;
}
__host__ __device__ inline size_t gsel_map_bytes(int n_rows) {
  return (size_t)2 * GS_BINS * 8 + sizeof(GselState) + (((size_t)n_rows * 8 + 255) / 256) * 256;
}
__device__ __forceinline__ GselView gsel_view(char *scratch, int map, int nqb) {
  char *base = scratch + (size_t)map * gsel_map_bytes(nqb);
  GselView v;
  v.hist1 = reinterpret_cast<unsigned long long *>(base);
  v.hist2 = v.hist1 + GS_BINS;
  v.state = reinterpret_cast<GselState *>(v.hist2 + GS_BINS);
  v.row_ties = reinterpret_cast<uint32_t *>(v.state + 1);
  v.row_before = v.row_ties + nqb;
  return v;
}

// Slash sums at the borders of the search's chunks, of which the search leaves two halves: `low` here and the other one,
// not yet divided by the block, in the vector itself.  They are added up by the kernel that comes before the first
// reading of the vectors, once, always as low + after.  Vectors come in pairs, the slash sums second.
struct VsBorders {
  float *sums;       // [n_maps][seq], or null: nothing to add up
  const float *low;  // [n_maps / 2][n_chunks][block]
  int n_chunks, chunk_keys, block, seq;
};
constexpr int VS_PARTS = 64;  // parts of the keys that the search keeps row statistics of, and chunks, at most

// grid y 0 clears the map's histograms, y > 0 adds up border y of a search's slash sums
__global__ __launch_bounds__(256) void gsel_zero_kernel(char *scratch, GselGeom g, VsBorders e) {
  const int map = blockIdx.x;
  if (blockIdx.y > 0) {
    const int c = blockIdx.y, d = threadIdx.x;
    if ((map & 1) && d < e.block && !gsel_skip(g, map)) {
      float *const at = e.sums + (int64_t)map * e.seq + (e.seq - c * e.chunk_keys - d);
      *at = (e.low[((int64_t)(map >> 1) * e.n_chunks + c - 1) * e.block + d] + *at) * (1.f / e.block);
    }
    return;
  }
  GselView v = gsel_view(scratch, map, g.n_rows);
  for (int x = threadIdx.x; x < 2 * GS_BINS; x += 256) v.hist1[x] = 0ull;
}

template <int PASS>
__global__ __launch_bounds__(256) void gsel_hist_kernel(const float *__restrict__ scores, GselGeom g, char *scratch) {
  __shared__ unsigned long long h[GS_BINS];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int map = blockIdx.y;
  if (gsel_skip(g, map)) return;
  GselView v = gsel_view(scratch, map, g.n_rows);
  for (int x = tid; x < GS_BINS; x += 256) h[x] = 0ull;
  __syncthreads();
  const uint32_t bin_hi = (PASS == 2) ? v.state->bin_hi : 0u;
  unsigned long long low = 0ull;  // first pass: bin 0 holds most of a softmaxed map; keep it out of the LDS atomics
  for (int row = blockIdx.x * 4 + w; row < g.n_rows; row += gridDim.x * 4) {
    const float *src = scores + ((int64_t)map * g.n_rows + row) * g.n_cols;
    const int width = gsel_width(g, row);
    for (int j = lane; j < width; j += 64) {
      const uint32_t u = quantise24(src[j]);
      if (PASS == 1) {
        const uint32_t bin = u >> 12;
        if (bin == 0)
          low += u;
        else
          atomicAdd(&h[bin], (unsigned long long)u);
      } else if (u != 0u && (u >> 12) == bin_hi) {
        atomicAdd(&h[u & 4095u], (unsigned long long)u);
      }
    }
  }
  if (PASS == 1) {
    low = wave_sum_u64(low);
    if (lane == 0 && low) atomicAdd(&h[0], low);
  }
  __syncthreads();
  unsigned long long *gh = (PASS == 1) ? v.hist1 : v.hist2;
  for (int x = tid; x < GS_BINS; x += 256)
    if (h[x]) atomicAdd(&gh[x], h[x]);
}

// One workgroup of 1024 threads per map.  Thread t owns bins [5t, 5t+5); a suffix sum over threads
// locates the bin in which the running sum from the top first reaches the target.  wt: 16 words of LDS.
template <int PASS>
__device__ __forceinline__ void gsel_scan(const unsigned long long *hist, GselState *state, unsigned long long *wt,
                                          uint32_t gq) {
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  constexpr int NB = (PASS == 1) ? 4097 : 4096;
  unsigned long long mine[5], sum = 0ull;
#pragma unroll
  for (int x = 0; x < 5; ++x) {
    const int bin = 5 * t + x;
    mine[x] = (bin < NB) ? hist[bin] : 0ull;
    sum += mine[x];
  }
  unsigned long long incl = sum;  // sum over lanes >= this one
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const unsigned long long y = __shfl_down(incl, off, 64);
    if (lane + off < 64) incl += y;
  }
  if (lane == 0) wt[w] = incl;
  __syncthreads();
  unsigned long long above = incl - sum, tot = 0ull;
  for (int x = 0; x < 16; ++x) {
    tot += wt[x];
    if (x > w) above += wt[x];
  }
  unsigned long long T;
  if (PASS == 1) {
    const unsigned long long th = tot >> 24, tl = tot & 0xFFFFFFull;
    T = (unsigned long long)gq * th + (((unsigned long long)gq * tl + 0xFFFFFFull) >> 24);  // ceil(gq * tot / 2^24)
    if (T < 1) T = 1;
    if (tot == 0ull) {
      if (t == 0) {
        state->T = 0;
        state->above = 0;
        state->need = 0;
        state->bin_hi = 0xFFFFFFFFu;
        state->vstar = 0xFFFFFFFFu;  // nothing reaches it
      }
      return;
    }
  } else {
    if (state->vstar == 0xFFFFFFFFu && state->bin_hi == 0xFFFFFFFFu) return;  // empty map
    T = state->T - state->above;
  }
  if (above < T && T <= above + sum) {  // exactly one thread
    unsigned long long a = above;
    for (int x = 4; x >= 0; --x) {
      if (a + mine[x] >= T) {
        const uint32_t bin = (uint32_t)(5 * t + x);
        if (PASS == 1) {
          state->T = T;
          state->above = a;
          state->bin_hi = bin;
          state->vstar = 0u;
        } else {
          const uint32_t vs = (state->bin_hi << 12) | bin;
          const unsigned long long gt = state->above + a;  // sum of everything above v*
          state->vstar = vs;
          state->need = (state->T - gt + vs - 1) / vs;
        }
        break;
      }
      a += mine[x];
    }
  }
}
template <int PASS>
__global__ __launch_bounds__(1024) void gsel_scan_kernel(char *scratch, GselGeom g, uint32_t gq) {
  __shared__ unsigned long long wt[16];
  if (gsel_skip(g, blockIdx.x)) return;
  GselView v = gsel_view(scratch, blockIdx.x, g.n_rows);
  gsel_scan<PASS>((PASS == 1) ? v.hist1 : v.hist2, v.state, wt, gq);
}

__global__ __launch_bounds__(256) void gsel_row_ties_kernel(const float *__restrict__ scores, GselGeom g, char *scratch) {
  const int lane = threadIdx.x & 63;
  const int row = blockIdx.x * 4 + (threadIdx.x >> 6), map = blockIdx.y;
  if (row >= g.n_rows || gsel_skip(g, map)) return;
  GselView v = gsel_view(scratch, map, g.n_rows);
  const uint32_t vstar = v.state->vstar;
  const float *src = scores + ((int64_t)map * g.n_rows + row) * g.n_cols;
  const int width = gsel_width(g, row);
  uint32_t n = 0;
  for (int j = lane; j < width; j += 64) n += (quantise24(src[j]) == vstar) ? 1u : 0u;
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) n += __shfl_xor(n, off, 64);
  if (lane == 0) v.row_ties[row] = n;
}

// exclusive prefix sum of row_ties over the rows of one map (flat order = row-major)
__global__ __launch_bounds__(1024) void gsel_row_scan_kernel(GselGeom g, char *scratch) {
  __shared__ uint32_t wt[16];
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  if (gsel_skip(g, blockIdx.x)) return;
  const int nqb = g.n_rows;
  GselView v = gsel_view(scratch, blockIdx.x, nqb);
  const int per = (nqb + 1023) / 1024;
  const int r0 = t * per, r1 = min(r0 + per, nqb);
  uint32_t sum = 0;
  for (int r = r0; r < r1; ++r) sum += v.row_ties[r];
  uint32_t incl = sum;  // sum over lanes <= this one
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const uint32_t y = __shfl_up(incl, off, 64);
    if (lane >= off) incl += y;
  }
  if (lane == 63) wt[w] = incl;
  __syncthreads();
  uint32_t before = incl - sum;
  for (int x = 0; x < w; ++x) before += wt[x];
  for (int r = r0; r < r1; ++r) {
    v.row_before[r] = before;
    before += v.row_ties[r];
  }
}

// one wavefront per row: ascending list of the kept key blocks (+ sink and diagonal when forced)
__global__ __launch_bounds__(256) void gsel_emit_kernel(const float *__restrict__ scores, GselGeom g, char *scratch,
                                                        int forced, int32_t *__restrict__ kb_idx,
                                                        int32_t *__restrict__ kb_cnt,
                                                        const int32_t *__restrict__ route) {
  const int lane = threadIdx.x & 63;
  const int nqb = g.n_rows;
  const int i = blockIdx.x * 4 + (threadIdx.x >> 6), map = blockIdx.y;
  if (i >= nqb) return;
  int omap = map;
  if (route) {
    omap = route[map];
    if (omap < 0) return;
  }
  GselView v = gsel_view(scratch, map, nqb);
  const uint32_t vstar = v.state->vstar;
  const uint64_t need = v.state->need;
  const uint64_t before = v.row_before[i];
  const float *src = scores + ((int64_t)map * nqb + i) * nqb;
  int32_t *out = kb_idx + ((int64_t)omap * nqb + i) * nqb;
  const uint64_t lt = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
  uint32_t ties_seen = 0, n_out = 0;
  for (int j0 = 0; j0 <= i; j0 += 64) {
    const int j = j0 + lane;
    const uint32_t x = (j <= i) ? quantise24(src[j]) : 0u;
    const bool tie = (j <= i) && (x == vstar);
    const uint64_t tmask = __ballot(tie);
    const uint64_t trank = before + ties_seen + __popcll(tmask & lt);
    ties_seen += __popcll(tmask);
    const bool sel = (j <= i) && ((x > vstar && vstar != 0xFFFFFFFFu) || (tie && trank < need) ||
                                  (forced && (j == 0 || j == i)));
    const uint64_t smask = __ballot(sel);
    if (sel) out[n_out + __popcll(smask & lt)] = j;
    n_out += __popcll(smask);
  }
  for (int pos = n_out + lane; pos < nqb; pos += 64) out[pos] = -1;
  if (lane == 0) kb_cnt[(int64_t)omap * nqb + i] = (int32_t)n_out;
}

// Selection over plain vectors (rectangular geometry): per (map, row) two flags instead of a list:
// bit 0 = some entry of the row is kept, bit 1 = some entry other than the row's first is kept.  bits (optional,
// n_cols a multiple of 64): the kept set itself, one bit per vector entry, [n_maps][n_rows * n_cols / 64] words.
__global__ __launch_bounds__(256) void gsel_emit_flags_kernel(const float *__restrict__ scores, GselGeom g, char *scratch,
                                                              int32_t *__restrict__ flags,
                                                              uint64_t *__restrict__ bits = nullptr) {
  const int lane = threadIdx.x & 63;
  const int row = blockIdx.x * 4 + (threadIdx.x >> 6), map = blockIdx.y;
  if (row >= g.n_rows || gsel_skip(g, map)) return;
  GselView v = gsel_view(scratch, map, g.n_rows);
  const uint32_t vstar = v.state->vstar;
  const uint64_t need = v.state->need;
  const uint64_t before = v.row_before[row];
  const float *src = scores + ((int64_t)map * g.n_rows + row) * g.n_cols;
  const int width = gsel_width(g, row);
  const uint64_t lt = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
  uint32_t ties_seen = 0;
  int any = 0, any_after_first = 0;
  for (int j0 = 0; j0 < width; j0 += 64) {
    const int j = j0 + lane;
    const uint32_t x = (j < width) ? quantise24(src[j]) : 0u;
    const bool tie = (j < width) && (x == vstar);
    const uint64_t tmask = __ballot(tie);
    const uint64_t trank = before + ties_seen + __popcll(tmask & lt);
    ties_seen += __popcll(tmask);
    const bool sel = (j < width) && ((x > vstar && vstar != 0xFFFFFFFFu) || (tie && trank < need));
    const uint64_t smask = __ballot(sel);
    any |= smask != 0ull;
    any_after_first |= (j0 == 0 ? (smask & ~1ull) : smask) != 0ull;
    if (bits && lane == 0) bits[((int64_t)map * g.n_rows + row) * (g.n_cols / 64) + j0 / 64] = smask;
  }
  if (lane == 0) flags[(int64_t)map * g.n_rows + row] = any | (any_after_first << 1);
}

// The whole selection over one map in one launch, by a workgroup of 1024 threads: rows of at most NC * 64 entries, at most
// GSEL_ROWS of them, histogram, tie counts and threshold in LDS.  load(row, k) gives entry 64 k + lane of a row (any in-range
// entry beyond the map), width(row) how many entries it has; emit(row, u, rank, vstar, need) takes its quantised entries (0
// beyond the row) and the number of ties before it.  The map is read four times (from L2 after the first).  Same integers as
// the launches above, which are latency alone on a small map.
constexpr int GSEL_ROWS = 256;
template <int NC, class Load, class Width, class Emit>
__device__ __forceinline__ void gsel_whole(int n_rows, uint32_t gq, Load load, Width width, Emit emit) {
  __shared__ unsigned long long hist[GS_BINS];
  __shared__ unsigned long long wt[16];
  __shared__ GselState st;
  __shared__ uint32_t ties[GSEL_ROWS];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  // f(row, the row's quantised entries), four rows of a wavefront in flight
  auto each_row = [&](auto f) {
    for (int r0 = w; r0 < n_rows; r0 += 64) {
      float x[4][NC];
#pragma unroll
      for (int k = 0; k < 4; ++k)
#pragma unroll
        for (int e = 0; e < NC; ++e) x[k][e] = load(min(r0 + 16 * k, n_rows - 1), e);
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const int row = r0 + 16 * k;
        if (row >= n_rows) break;
        uint32_t u[NC];
#pragma unroll
        for (int e = 0; e < NC; ++e) u[e] = e * 64 + lane < width(row) ? quantise24(x[k][e]) : 0u;
        f(row, u);
      }
    }
  };
  for (int x = tid; x < GS_BINS; x += 1024) hist[x] = 0ull;
  __syncthreads();
  unsigned long long low = 0ull;
  each_row([&](int, const uint32_t(&u)[NC]) {
#pragma unroll
    for (int e = 0; e < NC; ++e) {
      if (u[e] >> 12)
        atomicAdd(&hist[u[e] >> 12], (unsigned long long)u[e]);
      else
        low += u[e];
    }
  });
  low = wave_sum_u64(low);
  if (lane == 0 && low) atomicAdd(&hist[0], low);
  __syncthreads();
  gsel_scan<1>(hist, &st, wt, gq);
  __syncthreads();
  for (int x = tid; x < GS_BINS; x += 1024) hist[x] = 0ull;
  const uint32_t bin_hi = st.bin_hi;
  __syncthreads();
  each_row([&](int, const uint32_t(&u)[NC]) {
#pragma unroll
    for (int e = 0; e < NC; ++e)
      if (u[e] != 0u && (u[e] >> 12) == bin_hi) atomicAdd(&hist[u[e] & 4095u], (unsigned long long)u[e]);
  });
  __syncthreads();
  gsel_scan<2>(hist, &st, wt, gq);
  __syncthreads();
  const uint32_t vstar = st.vstar;  // never 0
  const uint64_t need = st.need;
  each_row([&](int row, const uint32_t(&u)[NC]) {
    uint32_t n = 0;
#pragma unroll
    for (int e = 0; e < NC; ++e) n += __popcll(__ballot(u[e] == vstar));
    if (lane == 0) ties[row] = n;
  });
  __syncthreads();
  const uint32_t own = tid < n_rows ? ties[tid] : 0u;
  uint32_t incl = own;  // sum over lanes <= this one
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const uint32_t y = __shfl_up(incl, off, 64);
    if (lane >= off) incl += y;
  }
  if (lane == 63) wt[w] = incl;
  __syncthreads();
  uint32_t before_wave = 0;
  for (int x = 0; x < w; ++x) before_wave += (uint32_t)wt[x];
  if (tid < n_rows) ties[tid] = before_wave + incl - own;
  __syncthreads();
  each_row([&](int row, const uint32_t(&u)[NC]) { emit(row, u, (uint64_t)ties[row], vstar, need); });
}

// Plain vectors of at most GSEL_VECTOR_MAX entries, rows of NC * 64.  The borders of the search's slash sums are added up
// first.  The vertical-slash attention of 32 heads (64 vectors) of 8K tokens took 597 us with the launches above, 578 with
// this.
constexpr int GSEL_VECTOR_MAX = 16384;  // (of rows of 64: GSEL_ROWS)
template <int NC>
__global__ __launch_bounds__(1024) void gsel_vector_kernel(VsBorders vs, GselGeom g, uint32_t gq,
                                                           int32_t *__restrict__ flags, uint64_t *__restrict__ bits) {
  const int tid = threadIdx.x, lane = tid & 63, map = blockIdx.x;
  if (gsel_skip(g, map)) return;
  float *const vec = vs.sums + (int64_t)map * vs.seq;
  constexpr int BL = NC * 64, NB = ((VS_PARTS - 1) * BL + 1023) / 1024;
  const int nb = (vs.n_chunks - 1) * BL;
  if ((map & 1) && nb > 0) {  // all loads in flight at once
    const float *low = vs.low + (int64_t)(map >> 1) * vs.n_chunks * BL;
    float a[NB], b[NB];
#pragma unroll
    for (int k = 0; k < NB; ++k) {
      const int x = min(tid + 1024 * k, nb - 1);
      a[k] = low[x];
      b[k] = vec[vs.seq - (x / BL + 1) * vs.chunk_keys - x % BL];
    }
#pragma unroll
    for (int k = 0; k < NB; ++k) {
      const int x = tid + 1024 * k;
      if (x < nb) vec[vs.seq - (x / BL + 1) * vs.chunk_keys - x % BL] = (a[k] + b[k]) * (1.f / BL);
    }
  }
  const float *src = vec + lane;
  const uint64_t lt = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
  gsel_whole<NC>(
      g.n_rows, gq, [&](int row, int e) { return src[(int64_t)row * (NC * 64) + e * 64]; }, [](int) { return NC * 64; },
      [&](int row, const uint32_t(&u)[NC], uint64_t rank, uint32_t vstar, uint64_t need) {
        int any = 0, any_after_first = 0;
#pragma unroll
        for (int e = 0; e < NC; ++e) {
          const bool tie = u[e] == vstar;
          const uint64_t tmask = __ballot(tie);
          const bool sel = (u[e] > vstar && vstar != 0xFFFFFFFFu) || (tie && rank + __popcll(tmask & lt) < need);
          rank += __popcll(tmask);
          const uint64_t smask = __ballot(sel);
          any |= smask != 0ull;
          any_after_first |= (e == 0 ? (smask & ~1ull) : smask) != 0ull;
          if (bits && lane == 0) bits[((int64_t)map * g.n_rows + row) * NC + e] = smask;
        }
        if (lane == 0) flags[(int64_t)map * g.n_rows + row] = any | (any_after_first << 1);
      });
}

// Causal maps of at most GSEL_MAP_ROWS rows, lists as gsel_emit_kernel writes them.  A layer with the printed pattern:
// 9 blocks 99.9 -> 84.2 us, 31 blocks 86.1 -> 71.8, 75 blocks 303 -> 293, 108 blocks 487 -> 477; a workgroup per map is too
// few beyond (165 blocks 1246 -> 1248, 168 blocks 268 -> 273, 193 blocks 1529 -> 1539).
constexpr int GSEL_MAP_ROWS = 128;
template <int NC>
__global__ __launch_bounds__(1024) void gsel_map_kernel(const float *__restrict__ scores, int nqb, uint32_t gq, int forced,
                                                        int32_t *__restrict__ kb_idx, int32_t *__restrict__ kb_cnt,
                                                        const int32_t *__restrict__ route) {
  const int lane = threadIdx.x & 63, map = blockIdx.x;
  const int omap = route ? route[map] : map;
  if (omap < 0) return;
  const float *src = scores + (int64_t)map * nqb * nqb;
  const uint64_t lt = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
  gsel_whole<NC>(
      nqb, gq, [&](int row, int e) { return src[(int64_t)row * nqb + min(e * 64 + lane, row)]; },
      [](int row) { return row + 1; },
      [&](int i, const uint32_t(&u)[NC], uint64_t rank, uint32_t vstar, uint64_t need) {
        int32_t *out = kb_idx + ((int64_t)omap * nqb + i) * nqb;
        uint32_t n_out = 0;
#pragma unroll
        for (int e = 0; e < NC; ++e) {
          const int j = e * 64 + lane;
          const bool tie = u[e] == vstar;
          const uint64_t tmask = __ballot(tie);
          const bool sel = (j <= i) && ((u[e] > vstar && vstar != 0xFFFFFFFFu) ||
                                        (tie && rank + __popcll(tmask & lt) < need) || (forced && (j == 0 || j == i)));
          rank += __popcll(tmask);
          const uint64_t smask = __ballot(sel);
          if (sel) out[n_out + __popcll(smask & lt)] = j;
          n_out += __popcll(smask);
        }
        for (int pos = n_out + lane; pos < nqb; pos += 64) out[pos] = -1;
        if (lane == 0) kb_cnt[(int64_t)omap * nqb + i] = (int32_t)n_out;
      });
}

}  // namespace

#endif
