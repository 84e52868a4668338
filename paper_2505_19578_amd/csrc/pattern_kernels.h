// Block-mean-logit score map (Sec. 5.2), last-row estimates, the Jensen-Shannon gate of Alg. 3 and pivot election (Alg. 1).
#ifndef SP_PATTERN_KERNELS_H
#define SP_PATTERN_KERNELS_H
#include "sp_common.h"
#include "attn_kernel.h"
#include "mask_kernel.h"

namespace {

// ---------------------------------------------------------------------------------------------
// pattern construction as printed in the paper (Sec. 5.2 "Sparse Attention Computation" and
// "Pivotal Pattern Construction"; Alg. 2): block-mean logits -> row softmax -> one selection over
// the flattened, globally normalised map
// ---------------------------------------------------------------------------------------------
__device__ __forceinline__ float bf16_bits_to_float(uint16_t x) { return __uint_as_float((uint32_t)x << 16); }

struct PoolParams {
  const uint16_t *q, *k;
  int64_t q_sb, q_st, q_sh, k_sb, k_st, k_sh;
  int nqb, group, n_heads, n_kv_heads;
  int row0, n_rows;  // query-block rows row0 .. row0 + n_rows - 1 are wanted
  float *qsum;       // [b][n][n_rows][D]   sum of the block's queries
  float *ksumT;      // [b][kvh][D][nqb]    sum of the block's keys, block index fastest
  float *diag;       // [b][n][n_rows]      sum over the diagonal block's causal entries of q_t . k_s
  float *out;        // [b][n][n_rows][nqb] row softmax of the block-mean logits
  float c_full, c_diag;
  const int32_t *head_dev;  // optional [b][n_heads]: head of listed position n chosen on the device, < 0 = empty
  // optional, one wanted row (n_rows == 1): the row's distances for the pivot election, js[b][n][2] = d_sparse and, if
  // the dictionary has an entry for the head's cluster, d_sim against its representative
  double *js;
  const int32_t *dict_valid;  // [b][n_clusters]
  const float *dict_a_tilde;  // [b][n_clusters][nqb]
  int n_clusters;
  int32_t head_ids[SP_MAX_HEADS];
  int32_t head_cluster[SP_MAX_HEADS];  // with js: dictionary cluster of listed position n, or -1
};
// x ln(x/m) + y ln(y/m), m = (x+y)/2: one entry's contribution to 2*JSD, never negative
__device__ __forceinline__ double js_term(double x, double y) {
  const double m = 0.5 * (x + y);
  double t = 0.0;
  if (x > 0.0) t += x * log(x / m);
  if (y > 0.0) t += y * log(y / m);
  return t;
}
__device__ __forceinline__ int pool_head(const PoolParams &p, int b, int n) {
  return p.head_dev ? p.head_dev[(int64_t)b * p.n_heads + n] : p.head_ids[n];
}

// The average of q_t . k_s over a full block is (sum_t q_t) . (sum_s k_s) / B^2, so the block-mean
// logits need only per-block sums of Q and K.  One thread per head dimension, one block per workgroup.
template <int D, int B>
__device__ __forceinline__ void key_pool(const PoolParams &p, int i, int kvh, int b) {
  const int e = threadIdx.x;
  const uint16_t *kp = p.k + (int64_t)b * p.k_sb + (int64_t)i * B * p.k_st + (int64_t)kvh * p.k_sh + e;
  float run = 0.f;
#pragma unroll 32
  for (int t = 0; t < B; ++t) run += bf16_bits_to_float(kp[(int64_t)t * p.k_st]);
  p.ksumT[(((int64_t)b * p.n_kv_heads + kvh) * D + e) * p.nqb + i] = run;
}

// Query sums of the wanted rows and, for the diagonal block (which keeps s <= t only), the sum
// sum_t q_t . (sum_{s<=t} k_s) from a running key sum walked once.
template <int D, int B>
__device__ __forceinline__ void query_pool(const PoolParams &p, int r, int n, int b) {
  const int e = threadIdx.x;
  const int i = p.row0 + r;
  const int head = pool_head(p, b, n);
  if (head < 0) return;
  const uint16_t *qp = p.q + (int64_t)b * p.q_sb + (int64_t)i * B * p.q_st + (int64_t)head * p.q_sh + e;
  const uint16_t *kp = p.k + (int64_t)b * p.k_sb + (int64_t)i * B * p.k_st + (int64_t)(head / p.group) * p.k_sh + e;
  float run = 0.f, qs = 0.f, acc = 0.f;
#pragma unroll 32
  for (int t = 0; t < B; ++t) {
    const float kk = bf16_bits_to_float(kp[(int64_t)t * p.k_st]);
    const float qq = bf16_bits_to_float(qp[(int64_t)t * p.q_st]);
    run += kk;
    qs += qq;
    acc = fmaf(qq, run, acc);
  }
  const int64_t hr = ((int64_t)b * p.n_heads + n) * p.n_rows + r;
  p.qsum[hr * D + e] = qs;
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) acc += __shfl_xor(acc, off, 64);
  if constexpr (D == 64) {
    if (e == 0) p.diag[hr] = acc;
  } else {
    __shared__ float part[D / 64];
    if ((e & 63) == 0) part[e >> 6] = acc;
    __syncthreads();
    if (e == 0) {
      float s = 0.f;
#pragma unroll
      for (int w = 0; w < D / 64; ++w) s += part[w];
      p.diag[hr] = s;
    }
  }
}

// Both in one launch, neither reads what the other writes: grid x = the key blocks of every KV head, then the wanted rows of
// every listed head; 32 rows of loads in flight, a thread's sum is a chain of its block's loads otherwise.  As two launches of
// 8 rows in flight: four dictionary layers of 1.3K tokens, 32 heads 519 us, as one 495, with 32 rows 482; gated layer of
// 2 x 8128 783 -> 777.
template <int D, int B>
__global__ __launch_bounds__(D) void pool_kernel(PoolParams p) {
  const int x = blockIdx.x, b = blockIdx.y, keys = p.nqb * p.n_kv_heads;
  if (x < keys) {
    key_pool<D, B>(p, x % p.nqb, x / p.nqb, b);
  } else {
    query_pool<D, B>(p, (x - keys) % p.n_rows, (x - keys) / p.n_rows, b);
  }
}

// Four query-block rows per workgroup: thread j forms the four pooled dot products against key block j
// (block index fastest in ksumT, so the loads coalesce), then one wavefront per row applies the row
// softmax in place (Alg. 2, first step; Alg. 3's estimate when only the last row is asked for).
// Entries beyond the diagonal are written as 0.
// With js the workgroup of a head goes on to its Jensen-Shannon distances: about 600 fp64 logarithms per head at 313
// blocks, which elect_kernel's single workgroup took for all heads in turn (two dictionary layers of 32 heads: 2K tokens
// 226.1 -> 216.9 us, 64K 12.08 -> 11.99 ms).
template <int D>
__global__ __launch_bounds__(256) void mean_logit_softmax_kernel(PoolParams p) {
  constexpr int R = 4;
  __shared__ float qs[R][D];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int r0 = blockIdx.x * R;
  const int64_t hb = blockIdx.y;
  const int b = (int)(hb / p.n_heads), n = (int)(hb % p.n_heads);
  const int nqb = p.nqb;
  const int head = pool_head(p, b, n);
  if (head < 0) return;
  for (int x = tid; x < R * D; x += 256) {
    const int r = x / D, e = x % D;
    qs[r][e] = (r0 + r < p.n_rows) ? p.qsum[((hb * p.n_rows) + r0 + r) * D + e] : 0.f;
  }
  __syncthreads();
  const float *kT = p.ksumT + ((int64_t)b * p.n_kv_heads + head / p.group) * D * nqb;
  const int rmax = min(r0 + R - 1, p.n_rows - 1);
  const int imax = p.row0 + rmax;
  for (int j = tid; j <= imax; j += 256) {
    float acc[R] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 8
    for (int e = 0; e < D; ++e) {
      const float kv = kT[(int64_t)e * nqb + j];
#pragma unroll
      for (int r = 0; r < R; ++r) acc[r] = fmaf(qs[r][e], kv, acc[r]);
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const int i = p.row0 + r0 + r;
      if (r0 + r < p.n_rows && j <= i)
        p.out[(hb * p.n_rows + r0 + r) * nqb + j] = (j < i) ? acc[r] * p.c_full : p.diag[hb * p.n_rows + r0 + r] * p.c_diag;
    }
  }
  __syncthreads();
  if (r0 + w < p.n_rows) {
    const int i = p.row0 + r0 + w;
    float *row = p.out + (hb * p.n_rows + r0 + w) * nqb;
    float mx = -INFINITY;
    for (int j = lane; j <= i; j += 64) mx = fmaxf(mx, row[j]);
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) mx = fmaxf(mx, __shfl_xor(mx, off, 64));
    float den = 0.f;
    for (int j = lane; j <= i; j += 64) den += expf(row[j] - mx);
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) den += __shfl_xor(den, off, 64);
    for (int j = lane; j < nqb; j += 64) row[j] = (j <= i) ? expf(row[j] - mx) / den : 0.f;
  }
  if (!p.js) return;
  __shared__ double part[4][2];
  __syncthreads();
  const int c = p.head_cluster[n];
  const float *row = p.out + hb * nqb;
  const float *ref = (c >= 0 && p.dict_valid[(int64_t)b * p.n_clusters + c])
                         ? p.dict_a_tilde + ((int64_t)b * p.n_clusters + c) * nqb
                         : nullptr;
  const double u = 1.0 / (double)nqb;
  double s0 = 0.0, s1 = 0.0;
  for (int j = tid; j < nqb; j += 256) {
    const double a = (double)row[j];
    s0 += js_term(a, u);
    if (ref) s1 += js_term(a, (double)ref[j]);
  }
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) {
    s0 += __shfl_xor(s0, off, 64);
    s1 += __shfl_xor(s1, off, 64);
  }
  if (lane == 0) part[w][0] = s0, part[w][1] = s1;
  __syncthreads();
  if (tid < 2) {
    const double jsd = 0.5 * ((part[0][tid] + part[1][tid]) + (part[2][tid] + part[3][tid]));
    p.js[hb * 2 + tid] = sqrt(jsd > 0.0 ? jsd : 0.0);
  }
}

// ---- Alg. 3 (Determine Sparse Pattern): Jensen-Shannon gate ------------------------------------
struct GateParams {
  const float *a_hat;     // [b][n][nkb] estimates of the listed heads
  float *dist;            // [b][n][2]   d_sparse, d_sim
  int32_t *head_pattern;  // [b][n_q_heads], entry of each listed head written
  int nkb, n_heads, n_q_heads;
  float delta, tau;
  int32_t head_ids[SP_MAX_HEADS];
  int32_t ref_pos[SP_MAX_HEADS];     // position of the head whose estimate is the representative, or -1
  int32_t shared_map[SP_MAX_HEADS];  // value written when the pattern is shared
};

// sqrt(JSD(a || ref)) over n entries, natural logarithm, fp64; ref == nullptr: the uniform distribution.
// Called by a whole wavefront; every lane returns the result.
__device__ __forceinline__ double js_distance_wave(const float *a, const float *ref, int n, int lane) {
  const double u = 1.0 / (double)n;
  double sum = 0.0;
  for (int j = lane; j < n; j += 64) sum += js_term((double)a[j], ref ? (double)ref[j] : u);
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) sum += __shfl_xor(sum, off, 64);
  const double jsd = 0.5 * sum;
  return sqrt(jsd > 0.0 ? jsd : 0.0);
}

// Alg. 3's gate for the listed heads: one wavefront per (head, batch entry).
__global__ __launch_bounds__(64) void js_gate_kernel(GateParams p) {
  const int n = blockIdx.x, b = blockIdx.y, lane = threadIdx.x;
  const float *a = p.a_hat + ((int64_t)b * p.n_heads + n) * p.nkb;
  const int rp = p.ref_pos[n];
  const double d_sparse = js_distance_wave(a, nullptr, p.nkb, lane);
  const double d_sim = (rp >= 0) ? js_distance_wave(a, p.a_hat + ((int64_t)b * p.n_heads + rp) * p.nkb, p.nkb, lane) : 0.0;
  if (lane == 0) {
    const int64_t hb = (int64_t)b * p.n_heads + n;
    p.dist[hb * 2] = (float)d_sparse;
    p.dist[hb * 2 + 1] = (float)d_sim;
    const bool shared = d_sparse < (double)p.delta && d_sim < (double)p.tau;
    p.head_pattern[(int64_t)b * p.n_q_heads + p.head_ids[n]] = shared ? p.shared_map[n] : -1;
  }
}

// ---- dynamic pivotal pattern dictionary (Sec. 5.2; Alg. 1 with Alg. 3 and Alg. 4) ----------------
// Roles written per (batch entry, head): c >= 0 shares cluster c's dictionary pattern, -1 falls back
// (dense, no update), -2 is elected pivot of its cluster in this layer (dense + pattern construction).
struct ElectParams {
  const float *a_hat;   // [b][Hq][nkb] last-row estimates of every head
  const double *js;     // [b][Hq][2] d_sparse; d_sim where the dictionary already has the head's cluster; or null
  float *dist;          // [b][Hq][2]
  int32_t *role;        // [b][Hq]
  int32_t *pivot_head;  // [b][n_slots] head elected for the slot's cluster in this layer, or -1
  int32_t *route;       // [b][n_slots] dictionary map (b * n_clusters + c) the slot's lists go to, or -1
  int32_t *act_n;       // [b] number of slots that elected a pivot
  int32_t *act_pos;     // [b][n_slots] those slots, ascending
  // the heads of the role-driven attention launch, split by weight class so that each class can be spread
  // evenly over the XCDs: positions (in that launch's slot table) of the heads that share a list, and of the
  // heads that fall back
  int32_t *shared_n, *shared_pos, *fallback_n, *fallback_pos;  // [b], [b][n_launch]
  int n_launch;
  int32_t launch_head[SP_MAX_HEADS];  // the launch's slot table: query head of each position
  int32_t *valid;       // dictionary [b][n_clusters]
  float *a_tilde;       // dictionary [b][n_clusters][nkb]
  int nkb, n_q_heads, n_slots, n_clusters;
  float delta, tau;
  int32_t head_cluster[SP_MAX_HEADS];  // global cluster id or -1
  int32_t head_slot[SP_MAX_HEADS];     // slot of the head's cluster, or -1
  int32_t slot_cluster[SP_MAX_HEADS];
};

// Writes the positions 0 .. n-1 for which take() holds to dst, ascending, and returns their number: one wavefront, 64 at a time.
template <typename F>
__device__ __forceinline__ int compact_wave(int n, int32_t *dst, int lane, F take) {
  int cnt = 0;
  for (int base = 0; base < n; base += 64) {
    const bool t = base + lane < n && take(base + lane);
    const uint64_t m = __ballot(t);
    if (t) dst[cnt + __popcll(m & ((1ull << lane) - 1))] = base + lane;
    cnt += __popcll(m);
  }
  return cnt;
}

// Bound by latency: tables are read by all lanes side by side and lists are made from ballots.  (One thread at a time walked
// heads and positions, with the argument tables' loads in a chain: four dictionary layers of 1280
// tokens, 32 heads, 471.4 -> 446.9 us, two of 2 x 2752, 4 heads, 254.3 -> 251.4.)
//
// One workgroup per batch entry.  Heads are taken in ascending order as in Alg. 1: a cluster without a
// dictionary entry elects its first head that passes the sparsity test (there is no representative to
// compare with yet); every other head is tested against the entry's representative, or against the
// estimate of the pivot elected a moment ago.
__global__ __launch_bounds__(1024) void elect_kernel(ElectParams p) {
  __shared__ double ds[SP_MAX_HEADS];
  __shared__ int piv[SP_MAX_HEADS];
  __shared__ int had[SP_MAX_HEADS];
  __shared__ int hc[SP_MAX_HEADS];
  __shared__ int hs[SP_MAX_HEADS];
  __shared__ int role_of[SP_MAX_HEADS];
  const int b = blockIdx.x, tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const float *ah = p.a_hat + (int64_t)b * p.n_q_heads * p.nkb;
  const double *js = p.js + (int64_t)b * p.n_q_heads * 2;
  for (int h = tid; h < p.n_q_heads; h += 1024) {
    hc[h] = p.head_cluster[h];
    hs[h] = p.head_slot[h];
  }
  if (p.js) {
    for (int h = tid; h < p.n_q_heads; h += 1024) ds[h] = js[2 * h];
  } else {
    for (int h = w; h < p.n_q_heads; h += 16) {
      const double d = js_distance_wave(ah + (int64_t)h * p.nkb, nullptr, p.nkb, lane);
      if (lane == 0) ds[h] = d;
    }
  }
  __syncthreads();
  for (int k = w; k < p.n_slots; k += 16) {
    const int c = p.slot_cluster[k];
    const int v = p.valid[(int64_t)b * p.n_clusters + c];
    int first = -1;
    if (!v && 0.0 < (double)p.tau)
      for (int base = 0; base < p.n_q_heads && first < 0; base += 64) {
        const int h = base + lane;
        const uint64_t m = __ballot(h < p.n_q_heads && hc[h] == c && ds[h] < (double)p.delta);
        if (m) first = base + __builtin_ctzll(m);
      }
    if (lane == 0) {
      piv[k] = first;
      had[k] = v;
      p.pivot_head[(int64_t)b * p.n_slots + k] = first;
      p.route[(int64_t)b * p.n_slots + k] = first >= 0 ? b * p.n_clusters + c : -1;
    }
  }
  __syncthreads();
  if (w == 15) {
    const int na = compact_wave(p.n_slots, p.act_pos + (int64_t)b * p.n_slots, lane, [&](int k) { return piv[k] >= 0; });
    if (lane == 0) p.act_n[b] = na;
  }
  for (int h = w; h < p.n_q_heads; h += 16) {
    const int c = hc[h], s = hs[h];
    int role = -1;
    double d_sim = 0.0;
    if (c >= 0) {
      if (piv[s] == h) {
        role = -2;
      } else {
        // heads met before the pivot of a new entry saw an empty dictionary: no representative for them
        const float *ref = had[s] ? p.a_tilde + ((int64_t)b * p.n_clusters + c) * p.nkb
                                  : (piv[s] >= 0 && piv[s] < h ? ah + (int64_t)piv[s] * p.nkb : nullptr);
        if (ref) {
          d_sim = had[s] && p.js ? js[2 * h + 1] : js_distance_wave(ah + (int64_t)h * p.nkb, ref, p.nkb, lane);
          if (ds[h] < (double)p.delta && d_sim < (double)p.tau) role = c;
        }
      }
    }
    if (lane == 0) {
      role_of[h] = role;
      p.role[(int64_t)b * p.n_q_heads + h] = role;
      p.dist[((int64_t)b * p.n_q_heads + h) * 2] = (float)ds[h];
      p.dist[((int64_t)b * p.n_q_heads + h) * 2 + 1] = (float)d_sim;
    }
  }
  __syncthreads();  // every read of the old representatives is done, every role is written
  if (w == 0) {
    const int ns = compact_wave(p.n_launch, p.shared_pos + (int64_t)b * p.n_launch, lane,
                                [&](int pos) { return role_of[p.launch_head[pos]] >= 0; });
    if (lane == 0) p.shared_n[b] = ns;
  } else if (w == 1) {
    const int nf = compact_wave(p.n_launch, p.fallback_pos + (int64_t)b * p.n_launch, lane,
                                [&](int pos) { return role_of[p.launch_head[pos]] == -1; });
    if (lane == 0) p.fallback_n[b] = nf;
  } else {
    for (int k = w - 2; k < p.n_slots; k += 14) {
      if (piv[k] < 0) continue;
      const int c = p.slot_cluster[k];
      float *__restrict__ dst = p.a_tilde + ((int64_t)b * p.n_clusters + c) * p.nkb;
      const float *__restrict__ src = ah + (int64_t)piv[k] * p.nkb;
      for (int j = lane; j < p.nkb; j += 64) dst[j] = src[j];
      if (lane == 0) p.valid[(int64_t)b * p.n_clusters + c] = 1;
    }
  }
}

// Splits the heads of a role-driven attention launch into the two weight classes (sharing a list / falling
// back) so that each class can be spread evenly over the XCDs; positions refer to the launch's slot table.
struct ClassifyParams {
  const int32_t *role;  // [b][n_q_heads]
  int32_t *shared_n, *shared_pos, *fallback_n, *fallback_pos;  // [b], [b][n_launch]
  int n_q_heads, n_launch;
  int32_t launch_head[SP_MAX_HEADS];
};
// One wavefront per class, 64 positions at a time (one thread in turn: gated layer of 2 x 8128 tokens 762.6 -> 758.1 us).
__global__ __launch_bounds__(128) void classify_heads_kernel(ClassifyParams p) {
  const int b = blockIdx.x, lane = threadIdx.x & 63;
  const int32_t *role = p.role + (int64_t)b * p.n_q_heads;
  if (threadIdx.x < 64) {
    const int ns = compact_wave(p.n_launch, p.shared_pos + (int64_t)b * p.n_launch, lane,
                                [&](int pos) { return role[p.launch_head[pos]] >= 0; });
    if (lane == 0) p.shared_n[b] = ns;
  } else {
    const int nf = compact_wave(p.n_launch, p.fallback_pos + (int64_t)b * p.n_launch, lane,
                                [&](int pos) { return role[p.launch_head[pos]] == -1; });
    if (lane == 0) p.fallback_n[b] = nf;
  }
}

}  // namespace

#endif
