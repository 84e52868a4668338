// Alg. 2 per query-block row in exact integers.
#ifndef SP_MASK_KERNEL_H
#define SP_MASK_KERNEL_H
#include "sp_common.h"

namespace {

// ---------------------------------------------------------------------------------------------
// mask kernel (Alg. 2 per row, exact integers)
// ---------------------------------------------------------------------------------------------
// Sum over the 64 lanes by lane-to-lane register moves (row shifts inside 16 lanes, then two row broadcasts), returned
// as a wave-uniform value.  The searches below are one chain of these sums: through LDS permutes the chain was the
// whole time of mask_kernel (8 maps of 32 rows: 10.2 us, now 6.3; 2 maps of 16: 9.9, now 5.6).
__device__ __forceinline__ uint32_t wave_sum_u32(uint32_t x) {
  auto add = [&](auto ctrl, auto rows) {
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, decltype(ctrl)::value, decltype(rows)::value, 0xf, false);
  };
  using std::integral_constant;
  add(integral_constant<int, 0x111>{}, integral_constant<int, 0xf>{});  // lane - 1, - 2, - 4, - 8 of the row
  add(integral_constant<int, 0x112>{}, integral_constant<int, 0xf>{});
  add(integral_constant<int, 0x114>{}, integral_constant<int, 0xf>{});
  add(integral_constant<int, 0x118>{}, integral_constant<int, 0xf>{});
  add(integral_constant<int, 0x142>{}, integral_constant<int, 0xa>{});  // last lane of rows 0 and 2 to rows 1 and 3
  add(integral_constant<int, 0x143>{}, integral_constant<int, 0xc>{});  // lane 31 to rows 2 and 3
  return (uint32_t)__builtin_amdgcn_readlane((int)x, 63);
}
__device__ __forceinline__ uint32_t wave_max_u32(uint32_t x) {
  auto join = [&](auto ctrl, auto rows) {
    x = max(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, decltype(ctrl)::value, decltype(rows)::value, 0xf, false));
  };
  using std::integral_constant;
  join(integral_constant<int, 0x111>{}, integral_constant<int, 0xf>{});
  join(integral_constant<int, 0x112>{}, integral_constant<int, 0xf>{});
  join(integral_constant<int, 0x114>{}, integral_constant<int, 0xf>{});
  join(integral_constant<int, 0x118>{}, integral_constant<int, 0xf>{});
  join(integral_constant<int, 0x142>{}, integral_constant<int, 0xa>{});
  join(integral_constant<int, 0x143>{}, integral_constant<int, 0xc>{});
  return (uint32_t)__builtin_amdgcn_readlane((int)x, 63);
}
// Every lane's x below 2^50 (24-bit scores: a lane would have to add 2^26 of them): two halves that cannot overflow.
__device__ __forceinline__ uint64_t wave_sum_u64(uint64_t x) {
  const uint32_t lo = wave_sum_u32((uint32_t)x & 0xFFFFFFu), hi = wave_sum_u32((uint32_t)(x >> 24));
  return ((uint64_t)hi << 24) + lo;
}

__device__ __forceinline__ uint32_t quantise24(float s) {
  // bit tests, so the result does not depend on how the compiler treats NaN comparisons
  const uint32_t bits = __float_as_uint(s);
  if (bits & 0x80000000u) return 0u;         // negative (and -0, -NaN)
  if (bits > 0x7F800000u) return 0u;         // NaN
  if (bits >= 0x3F800000u) return 1u << 24;  // >= 1 (and +inf) clamps to 1
  return (uint32_t)rintf(s * 16777216.f);
}

// The list of row i from its scores src[0 .. i], by one wavefront: out[nkb], *cnt, optionally bits[ceil(nkb / 64)].
// EPL > 0: the row lives in registers (nkb <= 64*EPL); EPL == 0: any nkb, the row is re-read in every pass.
// PASS: rows of up to PASS (64 or 128) blocks find their threshold in one pass over the row.
template <int EPL, int PASS, class Src>
__device__ __forceinline__ void mask_row(Src src, int lane, int i, int nkb, uint32_t gq, int32_t *__restrict__ out,
                                         int32_t *__restrict__ cnt, uint64_t *__restrict__ bits) {
  const int nchunk = (i >> 6) + 1;  // 64-wide chunks that hold valid key blocks
  uint32_t u[EPL > 0 ? EPL : 1];
  auto get = [&](int e) -> uint32_t {
    if (EPL > 0) return u[e];
    const int j = e * 64 + lane;
    return (j <= i) ? quantise24(src[j]) : 0u;
  };
  if (EPL > 0) {
#pragma unroll
    for (int e = 0; e < EPL; ++e) {
      const int j = e * 64 + lane;
      u[e] = (j <= i) ? quantise24(src[j]) : 0u;
    }
  }
  auto sum_ge = [&](uint32_t v) -> uint64_t {
    uint64_t part = 0;
    if (EPL > 0) {
      uint32_t p32 = 0;  // EPL <= 16 scores of at most 2^24
#pragma unroll
      for (int e = 0; e < EPL; ++e) p32 += (u[e] >= v) ? u[e] : 0u;
      part = p32;
    } else {
      for (int e = 0; e < nchunk; ++e) {
        const uint32_t x = get(e);
        part += (x >= v) ? x : 0u;
      }
    }
    return wave_sum_u64(part);
  };
  const uint64_t tot = sum_ge(1u);
  uint32_t vstar = 0xFFFFFFFFu;  // nothing reaches it: only forced blocks when tot == 0
  uint64_t need = 0;
  if (tot > 0) {
    uint64_t T = ((uint64_t)gq * tot + 16777215ull) >> 24;  // least integer prefix sum that reaches gamma
    if (T < 1) T = 1;
    // v* = the largest value with sum_ge(v*) >= T.  It is one of the scores, so a short row takes sum_ge of each of its
    // scores, side by side in the lanes (one pass over the row), and the largest that reaches T.  A longer row halves an
    // interval 24 times: a chain of wave sums, 3 us (a tiny layer 41.1 -> 38.8 us with the pass).  Up to 64 blocks the pass has
    // fewer instructions as well (64 maps of 64 rows 9.0 -> 7.4 us); up to 128 it only has the shorter chain, which counts
    // where a wavefront is alone (64 maps of 128 rows 14.8 us with the search from 64 blocks on, 19.1 with the pass), or where
    // the search adds up 16 registers (64 maps of 512 rows 95.7 and 92.2).
    if (EPL > 0 && i < PASS) {
      uint32_t s0 = 0, s1 = 0;  // at most 128 scores of at most 2^24
      const uint32_t u0 = u[0], u1 = (PASS > 64 && EPL > 1) ? u[EPL > 1 ? 1 : 0] : 0u;
      for (int j0 = 0; j0 <= i; j0 += 8) {
        const uint32_t from = (PASS <= 64 || j0 < 64) ? u0 : u1;
#pragma unroll
        for (int x = 0; x < 8; ++x) {  // (scores beyond the row are zero)
          const uint32_t y = (uint32_t)__builtin_amdgcn_readlane((int)from, (j0 + x) & 63);
          s0 += (u0 <= y) ? y : 0u;
          if (PASS > 64) s1 += (u1 <= y) ? y : 0u;
        }
      }
      const uint32_t t32 = (uint32_t)T;  // T <= tot < 2^32
      vstar = wave_max_u32(max(s0 >= t32 ? u0 : 0u, s1 >= t32 ? u1 : 0u));
    } else {
      uint32_t lo = 1u, hi = 16777217u;  // sum_ge(lo) >= T > sum_ge(hi)
      while (hi - lo > 1u) {
        const uint32_t mid = lo + ((hi - lo) >> 1);
        if (sum_ge(mid) >= T) lo = mid; else hi = mid;
      }
      vstar = lo;
    }
    const uint64_t above = sum_ge(vstar + 1u);
    need = (T - above + vstar - 1) / vstar;  // ties taken, lowest key block first
  }
  const int nwords = (nkb + 63) >> 6;
  const uint64_t lt = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
  uint32_t ties_before = 0, n_out = 0;
  const int nch_all = EPL > 0 ? EPL : nwords;
  for (int e = 0; e < nch_all; ++e) {
    if (e >= nwords) break;
    const int j = e * 64 + lane;
    uint32_t x = 0;
    if (EPL > 0) {
#pragma unroll
      for (int ee = 0; ee < EPL; ++ee)
        if (ee == e) x = u[ee];
    } else {
      x = (e < nchunk) ? get(e) : 0u;
    }
    const bool tie = (j <= i) && (x == vstar);
    const uint64_t tmask = __ballot(tie);
    const uint32_t trank = ties_before + __popcll(tmask & lt);
    ties_before += __popcll(tmask);
    const bool sel = (j <= i) && ((x > vstar && vstar != 0xFFFFFFFFu) || (tie && trank < need) || j == 0 || j == i);
    const uint64_t smask = __ballot(sel);
    if (sel) out[n_out + __popcll(smask & lt)] = j;
    n_out += __popcll(smask);
    if (bits && lane == 0) bits[e] = smask;
  }
  for (int pos = n_out + lane; pos < nkb; pos += 64) out[pos] = -1;
  if (lane == 0) *cnt = (int32_t)n_out;
}

// One wavefront per (map, row).
template <int EPL>
__global__ __launch_bounds__(256) void mask_kernel(const float *__restrict__ scores, int n_rows_total, int nqb,
                                                   int nkb, uint32_t gq, int32_t *__restrict__ kb_idx,
                                                   int32_t *__restrict__ kb_cnt, uint64_t *__restrict__ bitmask,
                                                   const int32_t *__restrict__ route) {
  const int lane = threadIdx.x & 63;
  const int row = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (row >= n_rows_total) return;
  const int i = row % nqb;
  // route (optional, [n_maps]): the map whose lists this map's rows become, negative = leave this map out
  int64_t orow = row;
  if (route) {
    const int dst = route[row / nqb];
    if (dst < 0) return;
    orow = (int64_t)dst * nqb + i;
  }
  const int nwords = (nkb + 63) >> 6;
  mask_row<EPL, EPL <= 4 ? 64 : 128>(scores + (int64_t)row * nkb, lane, i, nkb, gq, kb_idx + orow * nkb, kb_cnt + orow,
                bitmask ? bitmask + orow * nwords : nullptr);
}

}  // namespace

#endif
