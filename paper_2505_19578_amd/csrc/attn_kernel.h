// Dense / block-sparse flash-attention kernel (Sec. 5.1 A(Q,K,V) and A(Q,K,V,M)) with the block-mass score map.
#ifndef SP_ATTN_KERNEL_H
#define SP_ATTN_KERNEL_H
#include "sp_common.h"
#include "mask_kernel.h"

namespace {

// ---------------------------------------------------------------------------------------------
// attention kernel
// ---------------------------------------------------------------------------------------------
constexpr int SP_MAX_SLOTS = SP_MAX_HEADS + 8;
constexpr int SP_MAX_TOGETHER = 16;     // batch entries of a call whose rows are dispatched in one order
constexpr int SP_FUSED_MASK_MAX = 256;  // key blocks of a row whose list the dense kernel makes itself
struct AttnParams {
  const uint16_t *q;
  const char *kvp;  // packed K/V images
  uint16_t *o;
  int64_t q_sb, q_st, q_sh, o_sb, o_st, o_sh;
  int seq, nqb, n_kv_heads, n_heads, n_maps;
  float inv_group;  // 1 / query heads per KV head
  int rgroups;  // ceil(nqb / (8 QB)): workgroups' rows per strand (see the workgroup mapping in attn_kernel)
  int n_together;  // dense: batch entries whose rows are dispatched in one order (1: one after the other, entry blockIdx.y)
  float c;    // softmax scale * log2(e)
  float *lws;     // dense: block-local log2-sum-exp [b][n][nqb(nqb+1)/2][B] (row i, key block j <= i), or null
  float *scores;  // dense: [b][n][nqb][nkb], or null
  // dense with scores, nkb <= SP_FUSED_MASK_MAX, optional: the row's list (Alg. 2) is made where its scores are:
  // [b][n][nqb][nkb] and [b][n][nqb], or the map that route ([b][n], negative = none) names in place of b, n
  int32_t *mask_idx, *mask_cnt;
  const int32_t *route;
  uint32_t mask_gq;  // rint(gamma 2^24)
  const int32_t *kb_idx;  // sparse: [b][n_maps][nqb][nkb]
  const int32_t *kb_cnt;  // sparse: [b][n_maps][nqb]
  // sparse, optional: per (batch entry, query head) pattern chosen on the device (Alg. 3's gate):
  // a list index in [0, n_maps), or < 0 = no shared pattern, the head walks every key block 0..i
  const int32_t *head_pattern;  // [b][n_q_heads]; <= -2 = nothing to do for this head in this launch
  int n_q_heads;
  // optional: private lists per (batch entry, query head), used by a head whose head_pattern entry is -1
  // (its vertical-slash pattern) instead of the dense walk: [b][n_q_heads][nqb][nkb] / [b][n_q_heads][nqb]
  const int32_t *priv_idx, *priv_cnt;
  // optional: the query head of listed position n, chosen on the device (pivot election): [b][n_heads],
  // negative = this position is empty
  const int32_t *head_dev;
  // optional, with head_dev: how many listed positions are occupied per batch entry ([b]) and which ones
  // ([b][n_heads], ascending); the workgroup mapping then spreads just those over the XCDs
  const int32_t *act_n, *act_pos;
  int32_t head_ids[SP_MAX_SLOTS];  // query head of each slot, -1 = padding slot
  int32_t head_map[SP_MAX_SLOTS];  // sparse: which list the slot's head uses
  int32_t head_pos[SP_MAX_SLOTS];  // position of the head in the caller's list (scores / lws index)
};

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }
__device__ __forceinline__ float fast_log2(float x) { return __builtin_amdgcn_logf(x); }

// max / sum of a value with its partner in lane ^ 32 (one v_permlane32_swap, no LDS round trip)
__device__ __forceinline__ float max_xor32(float x) {
  const uint32_t u = __builtin_bit_cast(uint32_t, x);
  const auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
  return fmaxf(__builtin_bit_cast(float, (uint32_t)r[0]), __builtin_bit_cast(float, (uint32_t)r[1]));
}
__device__ __forceinline__ float sum_xor32(float x) {
  const uint32_t u = __builtin_bit_cast(uint32_t, x);
  const auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
  return __builtin_bit_cast(float, (uint32_t)r[0]) + __builtin_bit_cast(float, (uint32_t)r[1]);
}

// Reference point of the online softmax.  The running reference m only has to stay within
// SP_MAX_SLACK (log2 units) of the true running max: P = 2^(x - m) is then at most 2^SP_MAX_SLACK,
// harmless in fp32 / bf16, and m, l, the block sums and O stay mutually consistent whatever m is.
// Moving m only when the max outgrows it by more than the slack makes O rescaling rare (a lane
// triggers it a handful of times per row instead of at every new maximum).
// P is rounded to bf16 for the PV product while the row sum l adds the unrounded values.  With m lagging the
// true max, a row's large weights 2^(x - m) are not exactly representable, so in a row that a few keys
// dominate numerator and normaliser would differ by those weights' rounding errors (up to 2^-9 of |O|).
// The kernel therefore keeps a second sum lc = sum of (bf16(p) - p) over every tile that can hold a weight
// above 1/SP_CARE of the row's running sum (the first tiles of a row, tiles with a sink or a heavy key, and
// all tiles near the diagonal), and normalises O by l + lc: every weight that matters enters the
// normaliser as PV saw it; the weights left out are each below 1/SP_CARE of the row, their rounding
// errors are independent and average out.  The block-mass scores keep using l, so their rows sum to 1.
constexpr float SP_MAX_SLACK = 8.0f;
constexpr float SP_CARE = 32.0f;
__device__ __forceinline__ float lazy_max(float m_ref, float tile_max) {
  return (tile_max > m_ref + SP_MAX_SLACK) ? tile_max : m_ref;
}

__device__ __forceinline__ uint32_t pack_bf16(float a, float b) {
  f32x2 t = {a, b};
  bf16x2 r = __builtin_convertvector(t, bf16x2);
  return __builtin_bit_cast(uint32_t, r);
}

// sum of the eight bf16 values of a packed P fragment, as fp32
__device__ __forceinline__ float sum_bf16x8(bf16x8 v) {
  const u32x4 t = __builtin_bit_cast(u32x4, v);
  float a = 0.f, b = 0.f;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    a += __builtin_bit_cast(float, t[e] << 16);
    b += __builtin_bit_cast(float, t[e] & 0xffff0000u);
  }
  return a + b;
}
// one v_max3_f32 (as inline assembly it was followed by a wait state wherever its result is used)
__device__ __forceinline__ float max3f(float a, float b, float c) { return fmaxf(fmaxf(a, b), c); }
__device__ __forceinline__ bool any_lane(bool x) { return __builtin_amdgcn_ballot_w64(x) != 0ull; }

// One wavefront-wide 1 KiB copy HBM/L2 -> LDS without passing through registers: lane l moves the
// 16 bytes at g_uniform + lane_off to LDS byte address lds_base + 16 l (g_uniform and lds_base are
// wave-uniform).  Issued from inline assembly so that the compiler does not serialise it against
// the kernel's own LDS reads; the kernel counts these loads itself (wait_vm).
// OFF is the instruction's own offset, which moves both addresses: the chunks of one image share their scalar bases.
template <int OFF = 0>
__device__ __forceinline__ void lds_dma16(const void *g_uniform, uint32_t lane_off, uint32_t lds_base) {
  static_assert(OFF >= 0 && OFF < 4096, "13-bit signed immediate");
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2 offset:%3" ::"s"(lds_base),
               "v"(lane_off), "s"(g_uniform), "n"(OFF)
               : "memory", "m0");
}
// The chunks at OFF and OFF + 1024, for one setting of M0.
template <int OFF>
__device__ __forceinline__ void lds_dma16_pair(const void *g_uniform, uint32_t lane_off, uint32_t lds_base) {
  static_assert(OFF >= 0 && OFF + 1024 < 4096, "13-bit signed immediate");
  asm volatile(
      "s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2 offset:%3\n\tglobal_load_lds_dwordx4 %1, %2 offset:%4" ::
          "s"(lds_base),
      "v"(lane_off), "s"(g_uniform), "n"(OFF), "n"(OFF + 1024)
      : "memory", "m0");
}
// wait until at most N LDS reads are in flight (the compiler takes it into account)
template <int N>
__device__ __forceinline__ void wait_lds() {
  static_assert(N >= 0 && N < 16, "4-bit counter");
  __builtin_amdgcn_s_waitcnt(0xC07F | (N << 8));
}
template <int N>
__device__ __forceinline__ void wait_vm() {
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

// N products, product n with the LDS fragment that read(n) names: use(n, fragment) issues it.  AHEAD reads are in flight
// before the first product and one more goes out with each, in this order (the fences): left to itself the compiler keeps
// one fragment at a time, and each product waits for a read of its own (1.5K tokens, 32 heads: 73.5 -> 70.5 us of a layer;
// 2 x 8128 tokens in blocks of 64, gated: 838 -> 823; nothing at 12K and above).
template <int N, class Read, class Use>
__device__ __forceinline__ void products_read_ahead(Read &&read, Use &&use) {
  constexpr int AHEAD = 4;
  bf16x8 fr[AHEAD + 1];
  static_for<0, (AHEAD < N ? AHEAD : N)>([&](auto nc) __attribute__((always_inline)) {
    constexpr int n = decltype(nc)::value;
    fr[n] = read(n);
  });
  __builtin_amdgcn_sched_barrier(0);
  static_for<0, N>([&](auto nc) __attribute__((always_inline)) {
    constexpr int n = decltype(nc)::value;
    if constexpr (n + AHEAD < N) fr[(n + AHEAD) % (AHEAD + 1)] = read(n + AHEAD);
    use(nc, fr[n % (AHEAD + 1)]);
    __builtin_amdgcn_sched_barrier(0);
  });
}

// Flash-attention sweep over 64-key tiles t = 0 .. nsub-1, 32 queries per wavefront.
//
// Software pipeline (per wavefront), step t:
//     MFMA stream   S[t+1] = K[t+1] Q^T          then   O += V[t]^T P[t]^T
//     VALU stream   P[t] = 2^(S[t] c - m)        then   row max of S[t+1], running-max update
//   interleaved instruction by instruction (a hand-laid schedule), so the softmax runs in the
//   shadow of the matrix pipe.  Steps near the diagonal take a general path (causal mask / skip).
// K and V images ride in LDS rings (RK, RV slots) filled by LDS-direct loads issued DK resp. DV
// steps ahead, one chunk at a time from inside the MFMA groups; one workgroup barrier per step.
// One or two query blocks per workgroup (QB B/32 wavefronts); two or three wavefronts per SIMD, of different workgroups, so
// that one's barrier / load-issue time is covered by the others: workgroups of four wavefronts take 80 KiB of LDS at d 128
// (two per CU) and 40 KiB at d 64 (three), those of two wavefronts 40 KiB (four).
// The registers are bounded accordingly (256 or 168 per lane): without a bound the block 64
// kernels spread over accumulation registers and paid moves for it (tiny layer 53.1 -> 50.0 us).
//
// SK: keys of a ring image.  64, except for d 128 / block 64: a workgroup is two wavefronts there and its rings of 64-key
// images take 80 KiB, so only one wavefront per SIMD fits; half images (32 keys) make it two (gated layer of 2 x 8128
// tokens, 32 heads: 980 us with whole images, 856 us with halves).  A step of a half image is half of a tile's step: its
// S, P and PV.  The reference still moves once per 64-key tile, the row sums and O are added up in the same order, so the
// results are the bits that steps of whole images give.  (Tiles of 32 keys had moved the reference twice as often, at
// 886 us, and rounded the weights at other points than the other block size.)
//
// One workgroup walks the whole row, whatever else the launch holds: groups of wavefronts that walked a part of the row
// each and were joined at the end (for launches of at most one wavefront per SIMD: 45 -> 35.5 us of a tiny layer) had
// references of their own, so that a head's output depended on how many heads and batch entries were in the call.
//
// QB: query blocks of a workgroup.  Two where a row is walked densely in blocks of 64: neighbouring rows walk the same
// tiles, so a workgroup of four wavefronts moves every image once for both (the steps of block 128; the block of a wavefront
// decides where its diagonal lies).  Score maps of 2 x 12352 tokens, 16 heads of d 64: 832 -> 788 us; gated layer of 2 x 8128
// tokens, d 128: 794 -> 770.
//
// WAVES: wavefronts per SIMD that the registers are kept to.  Three for d 64 with four wavefronts to a workgroup, where a launch
// is large enough (the launcher's rule).  A step there is bound by its VALU work (exponentials, sums, row maxima), and a third
// wavefront fills what two leave.  168 registers are enough with two LDS fragments ahead instead of four (four: 12 to 20 bytes
// of scratch, up to 30 % slower on short rows).  The same score maps 788 -> 740 us; blocks of 128, score maps of 2 x 12288:
// 805 -> 752; lists of 2 x 15488: 1143 -> 1098.
template <int D, int B, int QB>
constexpr int attn_image_keys() { return (D == 128 && QB * B == 64) ? 32 : 64; }
template <int D, int B, bool DENSE, bool SCORES, int QB, int WAVES>
__global__ __launch_bounds__(QB * B * 2, WAVES) void attn_kernel(AttnParams p) {
  static_assert(QB == 1 || (DENSE && B == KT), "rows share their tiles where every key block is walked");
  static_assert(WAVES == 2 || (D == 64 && QB * B == 128), "three wavefronts per SIMD: 40 KiB of LDS per four wavefronts");
  constexpr int SK = attn_image_keys<D, B, QB>();
  constexpr int KH = KT / SK;       // ring images, and steps, per 64-key tile
  constexpr int WB = B / 32;        // wavefronts per query block, 32 queries each
  constexpr int NW = QB * WB;       // wavefronts per workgroup
  constexpr int SPB = B / KT;       // tiles per key block
  constexpr int NR = SK / 32;       // 32-key row blocks of S^T per step
  constexpr int NKS = SK / 16;      // 16-key parts of the PV product per step
  constexpr int IMG = SK * D * 2;   // bytes of a ring image of K (or V)
  constexpr int PACKED = KT * D * 2;  // bytes of a packed K (or V) image of KT keys, K image then V image
  constexpr int DS = D / 16;        // k-steps of the QK^T product
  constexpr int DB = D / 32;        // 32-row blocks of O^T
  // Step u = KH * tile + part reads K image u + KH and V image u; it fetches K image u + DK and V image u + DV.
  constexpr int DK = KH + 1, DV = 2;
  constexpr int RK = DK - KH + 1, RV = DV + 1;               // ring slots; image u lies in slot u % RK resp. u % RV
  constexpr int CH = IMG / 1024 / NW;                        // 1 KiB chunks per wavefront per image
  // Each step issues its CH chunks of K[u+DK] first, then its CH chunks of V[u+DV].  At the top of the next
  // step its K image (issued a step ago) must have landed; the V chunks issued after it are for a later step and
  // may still be in flight (vmcnt counts in order).
  constexpr int VM_KEEP = CH;
  static_assert(IMG % (1024 * NW) == 0, "image must split evenly over the wavefronts");
  __shared__ __attribute__((aligned(1024))) char smem[(RK + RV) * IMG];
  const uint32_t lds_k = (uint32_t)(size_t)(__attribute__((address_space(3))) char *)smem;
  const uint32_t lds_v = lds_k + RK * IMG;

  const int tid = threadIdx.x, lane = tid & 63, h = lane >> 5, c32 = lane & 31;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);  // wavefront index, kept scalar
  // workgroup -> (XCD, strand, query block, batch).  Workgroups are dealt round-robin to the 8 XCDs by the
  // hardware.  Every listed head is cut into 8 strands (the query blocks i with (nqb-1-i) % 8 == s, all of
  // about equal work and each spanning short and long rows); the 8n strands g = 8*slot + s, in slot-table
  // order, are dealt to the XCDs in contiguous runs of n, so whatever n is every XCD gets the same work and
  // works on at most ceil(n/8)+1 heads (heads that share a KV head sit next to each other and meet in its
  // L2).  Inside an XCD the dispatch order is rows from long to short, then strand number, then head: the
  // heads that walk the same list for the same row are neighbours in time.
  // Up to some size of launch, the rows of several batch entries are dispatched in one order, from long to short over all of
  // them (n_together): one entry after the other, the long rows of the last entry begin when the chip is half empty, which
  // costs the more the fewer and longer-lived the workgroups are (two rows to one, three wavefronts per SIMD).
  const int xcd = blockIdx.x & 7;
  const uint32_t u = blockIdx.x >> 3;
  // number of heads this launch really has for batch entry x (all listed ones unless the device says otherwise)
  auto heads_of = [&](int x) -> int { return p.act_n ? __builtin_amdgcn_readfirstlane(p.act_n[x]) : p.n_heads; };
  const int together = DENSE ? p.n_together : 1;
  int b = blockIdx.y, n_act = heads_of(b), n_all = n_act;
  for (int x = 1; x < together; ++x) n_all += heads_of(x);
  if (n_all <= 0 || (int)u >= n_all * p.rgroups) return;
  const int rest = u / (uint32_t)n_all;
  int strand;
  {
    // Position inside the XCD's run, enumerated strand number first, batch entry second, head third; where the device says
    // which heads there are, entries have runs of their own.
    int kk = u - rest * n_all;
    if (p.act_n)
      while (kk >= n_act && b + 1 < together) {
        kk -= n_act;
        n_act = heads_of(++b);
      }
    const int g0 = xcd * n_act, alike = p.act_n ? 1 : together;
    for (int sn = 0;; ++sn) {
      const int s0 = (sn - g0) & 7;  // g0 + s0, + 8, ..: the strands of the run whose number is sn
      const int cnt = (n_act >> 3) + (s0 < (n_act & 7) ? 1 : 0);
      if (kk < cnt * alike || sn == 7) {
        if (alike > 1) {
          b = (uint32_t)kk / (uint32_t)cnt;
          kk -= b * cnt;
        }
        strand = g0 + s0 + 8 * kk;
        break;
      }
      kk -= cnt * alike;
    }
  }
  int slot = strand >> 3;
  if (p.act_pos) slot = __builtin_amdgcn_readfirstlane(p.act_pos[(int64_t)b * p.n_heads + slot]);
  // the (last) query block of the workgroup, and this wavefront's own (negative: none, the workgroup's first block is 0)
  const int i = p.nqb - 1 - QB * (rest * 8 + (strand & 7));
  if (i < 0) return;  // nqb is not a multiple of 8 QB: this strand has one row fewer
  const int wb = QB > 1 ? w / WB : 0;  // which block is the wavefront's
  const int iw = i - (QB - 1) + wb;
  const bool idle = QB > 1 && iw < 0;
  int head = p.head_ids[slot];
  const int nkb = p.nqb;
  const int hpos = p.head_pos[slot];
  if (p.head_dev) {
    head = __builtin_amdgcn_readfirstlane(p.head_dev[(int64_t)b * p.n_heads + hpos]);
    if (head < 0 || head >= p.n_q_heads) return;
  }
  const int kvh = __builtin_amdgcn_readfirstlane((int)((head + 0.5f) * p.inv_group));  // exact: head < 128

  const int wr = QB > 1 ? w % WB : w, wq = 32 * wr, tq = wq + c32;  // first query of the wavefront, this lane's, inside the block
  f32x16 oacc[DB];
#pragma unroll
  for (int db = 0; db < DB; ++db)
#pragma unroll
    for (int r = 0; r < 16; ++r) oacc[db][r] = 0.f;
  float m = -INFINITY, l = 0.f, bs = 0.f;
  float lc = 0.f;     // sum of bf16(p) - p over the tiles summed twice (see SP_CARE)
  bool care = true;   // the tile whose max was taken last may hold a weight that matters, for any lane

  // A list is read 64 entries at a time into registers, a chunk ahead (entry e of the row = lane e % 64 of chunk e / 64); its
  // first chunk goes out together with the number of entries.  A load per entry inside the loop had every second step wait
  // for all refills (the compiler's own wait counts the loads that the kernel issues by hand), and the first entries were
  // five dependent loads before the first image could be asked for: lists of 98K tokens, 64 heads 19.56 -> 18.84 ms, four
  // dictionary layers of 64K 35.5 -> 34.5 ms, tiny layer 44.8 -> 43.6 us.
  int nblk = 0;
  const int32_t *list = nullptr;
  int lst = 0, lst_next = 0, lst_chunk = 0;
  auto load_chunk = [&](int chunk) -> int {
    const int e = chunk * 64 + lane;
    return list[e < nkb ? e : nkb - 1];
  };
  if (DENSE) {
    nblk = i + 1;
  } else {
    int map = p.head_map[slot];
    if (p.head_pattern) {
      map = __builtin_amdgcn_readfirstlane(p.head_pattern[(int64_t)b * p.n_q_heads + head]);
      map = map >= p.n_maps ? p.n_maps - 1 : map;
      if (map <= -2) return;
    }
    const int32_t *cnt = nullptr;
    if (map < 0 && p.priv_idx) {
      const int64_t lrow_id = ((int64_t)b * p.n_q_heads + head) * p.nqb + i;
      cnt = p.priv_cnt + lrow_id;
      list = p.priv_idx + lrow_id * nkb;
    } else if (map >= 0) {
      const int64_t lrow_id = ((int64_t)b * p.n_maps + map) * p.nqb + i;
      cnt = p.kb_cnt + lrow_id;
      list = p.kb_idx + lrow_id * nkb;
    }
    if (list == nullptr) {
      nblk = i + 1;  // dense walk
    } else {
      lst = load_chunk(0);
      nblk = *cnt;
    }
  }
  bf16x8 qf[DS];
  {
    const uint16_t *qp =
        p.q + (int64_t)b * p.q_sb + ((int64_t)(idle ? 0 : iw) * B + tq) * p.q_st + (int64_t)head * p.q_sh + 8 * h;
#pragma unroll
    for (int ds = 0; ds < DS; ++ds) qf[ds] = *reinterpret_cast<const bf16x8 *>(qp + 16 * ds);
  }

  if (!DENSE && list != nullptr) {
    nblk = __builtin_amdgcn_readfirstlane(nblk);
    nblk = nblk < 0 ? 0 : (nblk > nkb ? nkb : nblk);
    if (nblk > 64) lst_next = load_chunk(1);
  }
  const int nsub = nblk * SPB;
  const char *kvbase = p.kvp + ((int64_t)b * p.n_kv_heads + kvh) * (int64_t)(p.seq / KT) * (2 * PACKED);
  float *lrow = nullptr;
  // block log-sum-exps: causal half, row i of a (batch entry, head) starts at i(i+1)/2 key-block slots
  const int64_t lws_row =
      ((int64_t)b * p.n_heads + hpos) * ((int64_t)p.nqb * (p.nqb + 1) / 2) + (int64_t)iw * (iw + 1) / 2;
  if (SCORES) lrow = p.lws + lws_row * B + tq;

  // key block of tile t (t clamped to the sequence; list entries clamped into [0, i]: memory-safe
  // whatever the list holds).  Asked for in ascending order of t.
  auto block_of = [&](int t) -> int {
    const int e = (t < nsub ? t : nsub - 1) / SPB;
    if (DENSE || list == nullptr) return e;
    if (__builtin_expect(t >= 6 && (e >> 6) != lst_chunk, 0)) {
      lst = lst_next;
      ++lst_chunk;
      if (nblk > (lst_chunk + 1) * 64) lst_next = load_chunk(lst_chunk + 1);
    }
    const int j = __builtin_amdgcn_readlane(lst, e & 63);
    return j < 0 ? 0 : (j > i ? i : j);
  };
  // what this wavefront has to do for tile `sub` of key block j: 0 all of it, 1 causal mask, 2 nothing
  auto mode_of = [&](int j, int sub) -> int {
    if (QB > 1 ? (idle || j > iw) : false) return 2;
    if (j != iw) return 0;
    const int klo = KT * sub, qlo = wq;
    return (klo > qlo + 31) ? 2 : ((klo + KT - 1 <= qlo) ? 0 : 1);
  };
  // every wavefront moves CH chunks of image `part` of tile t (clamped) into ring slot `slot_base`; a half image is one
  // half of a packed K image, and of every 4 KiB (one 32-dim block) of a packed V image
  const char *const k_mine = kvbase + w * CH * 1024;  // the wavefront's share of K and V image 0
  const char *const v_mine = kvbase + PACKED + (KH > 1 ? w * (CH / NKS) * 4096 : w * CH * 1024);
  auto img_src = [&](int t, int part, int j, auto is_v) __attribute__((always_inline)) -> const char * {
    constexpr bool V = decltype(is_v)::value;
    const int tt = t < nsub ? t : nsub - 1;
    // (the compiler loses sight of it being uniform; at most 2^16 tiles, 2^31 bytes)
    const uint32_t tile = __builtin_amdgcn_readfirstlane(DENSE ? tt : j * SPB + tt % SPB);
    return (V ? v_mine : k_mine) + tile * (uint32_t)(2 * PACKED) + (KH == 1 ? 0 : part * (V ? NKS * 1024 : IMG));
  };
  // chunk n (0 .. CH-1) of this wavefront's share of an image.  The chunk number goes into the instruction's offset: with
  // an address computed per chunk, a step of d 128 had 14 scalar instructions more.  That shows where a wavefront is alone
  // on its SIMD, and so bound by the instructions it issues, and where a step is short (tiny layer 45.9 -> 45.2 us, 4K
  // layer 146.7 -> 145.3, d 128 / block 64 811 -> 798), hardly where two wavefronts share the matrix pipe (-0.1 to -0.6 %).
  auto issue_chunk = [&](const char *src, uint32_t slot_base, auto nc, auto is_v) __attribute__((always_inline)) {
    constexpr int n = decltype(nc)::value;
    constexpr bool HALF_V = KH > 1 && decltype(is_v)::value;  // NKS KiB of every 4 KiB of the packed image
    static_assert(!HALF_V || CH % NKS == 0, "a wavefront's share of a half V image starts at a 4 KiB piece");
    lds_dma16<n * 1024>(src + (HALF_V ? n / NKS * (4096 - NKS * 1024) : 0), lane * 16, slot_base + w * CH * 1024);
  };
  auto issue_img = [&](int t, int part, int j, auto is_v, uint32_t slot_base) __attribute__((always_inline)) {
    const char *src = img_src(t, part, j, is_v);
    static_for<0, CH>([&](auto nc) __attribute__((always_inline)) { issue_chunk(src, slot_base, nc, is_v); });
  };
  using IsK = std::false_type;
  using IsV = std::true_type;

  // S rows of image `part` of a tile
  auto qk = [&](auto part, const char *kbuf, f32x16(&s)[2]) {
    constexpr int R0 = decltype(part)::value * NR;
    const char *kb = kbuf + lane * 16;
#pragma unroll
    for (int rb = 0; rb < NR; ++rb)
#pragma unroll
      for (int r = 0; r < 16; ++r) s[R0 + rb][r] = 0.f;
    products_read_ahead<NR * DS>(
        [&](int n) { return *reinterpret_cast<const bf16x8 *>(kb + ((n % NR) * DS + n / NR) * 1024); },
        [&](auto nc, bf16x8 a) __attribute__((always_inline)) {
          constexpr int n = decltype(nc)::value;
          s[R0 + n % NR] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, qf[n / NR], s[R0 + n % NR], 0, 0, 0);
        });
  };
  // move_reference: mx = raw row max of a fresh tile.  Moves the reference if the max outgrew the slack,
  // rescales the running sums, notes whether the tile's largest weight matters to the row (care), returns
  // alpha = 2^(m_old - m_new) for the O accumulators.
  auto move_reference = [&](float mx) -> float {
    const float m_new = lazy_max(m, mx * p.c);
    const float alpha = fast_exp2(m - m_new);
    m = m_new;
    l *= alpha;
    bs *= alpha;
    lc *= alpha;
    care = any_lane(fast_exp2(__builtin_fmaf(mx, p.c, -m_new)) * SP_CARE > l);
    return alpha;
  };
  // Online softmax, split in two halves that sit in different pipeline steps.
  // tile_max: (optionally causal-masked) row max of a freshly computed S tile; moves the running max,
  // rescales the running sums, returns alpha = 2^(m_old - m_new) for the O accumulators.
  auto tile_max = [&](f32x16(&s)[2], int mode, int sub) -> float {
    if (mode == 1) {
#pragma unroll
      for (int rb = 0; rb < 2; ++rb)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int kk = KT * sub + 32 * rb + 8 * (r >> 2) + 4 * h + (r & 3);
          if (kk > tq) s[rb][r] = -INFINITY;
        }
    }
    float mx = fmaxf(s[0][0], s[0][1]);
#pragma unroll
    for (int rb = 0; rb < 2; ++rb)
#pragma unroll
      for (int r = (rb == 0 ? 2 : 0); r < 16; r += 2) mx = fmaxf(mx, fmaxf(s[rb][r], s[rb][r + 1]));
    mx = max_xor32(mx);
    return move_reference(mx);
  };
  // what a tile's steps hand on to one another: two halves of its row sum, the row max of the next tile, the sum of the
  // weights as PV sees them
  float rs0, rs1, mx, mx_odd, psum;
  // QB > 1: the general steps of a workgroup begin at its first block's diagonal.  A wavefront's tiles before twice_from,
  // which it would take by fast steps in a workgroup of its own, are summed as those do: the same bits either way.
  int twice_from = 0;
  float lc_later = 0.f;
  auto add_p = [&](auto part, const bf16x8(&pb)[NKS]) {
    psum = decltype(part)::value == 0 ? sum_bf16x8(pb[0]) : psum + sum_bf16x8(pb[0]);
#pragma unroll
    for (int ks = 1; ks < NKS; ++ks) psum += sum_bf16x8(pb[ks]);
  };
  // tile_exp: P = 2^(S*c - m) for image `part` of a tile whose max is already folded into m, left rounded to bf16 in pb
  // (the B operand of the PV product); the last one adds the tile's row sums
  auto tile_exp = [&](auto part, int t, f32x16(&s)[2], bf16x8(&pb)[NKS]) {
    constexpr int P = decltype(part)::value;
    if (P == 0) rs0 = rs1 = 0.f;
#pragma unroll
    for (int ks = 0; ks < NKS; ++ks) {
      u32x4 t;
#pragma unroll
      for (int e2 = 0; e2 < 4; ++e2) {
        const int r = 8 * (ks & 1) + 2 * e2;
        const float p0 = fast_exp2(__builtin_fmaf(s[P * NR + (ks >> 1)][r], p.c, -m));
        const float p1 = fast_exp2(__builtin_fmaf(s[P * NR + (ks >> 1)][r + 1], p.c, -m));
        rs0 += p0;
        rs1 += p1;
        t[e2] = pack_bf16(p0, p1);
      }
      pb[ks] = __builtin_bit_cast(bf16x8, t);
    }
    add_p(part, pb);
    if (P == KH - 1) {
      const float rs = sum_xor32(rs0 + rs1);
      l += rs;
      bs += rs;
      const float d = sum_xor32(psum) - rs;
      const bool early = QB > 1 && t < twice_from;
      lc += early ? 0.f : d;
      lc_later = early && care ? d : 0.f;
    }
  };
  auto rescale = [&](float alpha) {
    if (any_lane(alpha != 1.f)) {
#pragma unroll
      for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int r = 0; r < 16; ++r) oacc[db][r] *= alpha;
    }
  };
  auto pv = [&](const char *vbuf, const bf16x8(&pb)[NKS]) {
    const char *vb = vbuf + lane * 16;
    products_read_ahead<NKS * DB>(
        [&](int n) { return *reinterpret_cast<const bf16x8 *>(vb + ((n % DB) * NKS + n / DB) * 1024); },
        [&](auto nc, bf16x8 a) __attribute__((always_inline)) {
          constexpr int n = decltype(nc)::value;
          oacc[n % DB] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, pb[n / DB], oacc[n % DB], 0, 0, 0);
        });
  };

  // Byte offsets of the V slots: of the image that this step reads, and of the one before it, which is refilled (DV = RV - 1).
  // Carried along: a remainder by three is eight scalar instructions.  With the image addresses in 32 bits, the row max as
  // fmaxf in two chains and the tests of a lane mask as scalar compares, a step of d 128 went from 378 to 358 instructions
  // (128K layer 52.2 -> 51.4 ms, 32K 3428 -> 3369 us, tiny 38.8 -> 37.7).
  static_assert(DV == RV - 1, "the slot to refill is the previous step's");
  uint32_t v_now = 0, v_old = (RV - 1) * IMG;
  auto next_v = [&]() {
    v_old = v_now;
    v_now = v_now == (RV - 1) * IMG ? 0 : v_now + IMG;
  };
  // On entry to the steps of tile t: s_cur = raw S[t] (masked where needed), m / l / bs / O already moved to the
  // running max that includes tile t.  jt[x] = key block of tile t + x.
  // sync: wait until the images this step reads have landed for every wavefront; the ring slots that the previous step
  // freed may be refilled then.
  auto sync = [&]() {
    wait_vm<VM_KEEP>();
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  };
  // fast step: tiles t and t+1 both off the diagonal.  One basic block up to the rescale test.
  auto fast_step = [&](auto part, int t, const int(&jt)[3], f32x16(&s_cur)[2], f32x16(&s_next)[2]) {
    constexpr int P = decltype(part)::value;
    constexpr bool LAST = P == KH - 1;
    const int u0 = t * KH + P;
    // the ring refills (K, then V) are dropped one chunk at a time into the MFMA groups below instead of going out in a
    // burst after the barrier
    sync();
    const char *ksrc = img_src(t + (P + DK) / KH, (P + DK) % KH, jt[(P + DK) / KH], IsK{});
    const uint32_t kslot = lds_k + ((u0 + DK) % RK) * IMG;
    const char *vsrc = img_src(t + (P + DV) / KH, (P + DV) % KH, jt[(P + DV) / KH], IsV{});
    const uint32_t vslot = lds_v + v_old;
    const char *kb = smem + ((u0 + KH) % RK) * IMG + lane * 16;
    const char *vb = smem + RK * IMG + v_now + lane * 16;
    next_v();
    // Hand-laid schedule: NM groups, each = one MFMA + one LDS read (PF fragments ahead) + a slice
    // of the VALU work; nothing may cross a group boundary (sched_barrier).
    //   groups 0 .. NQ-1   : S[t+1] += K frag * Q frag ; exp / row-sum / bf16 pack of S[t]
    //   groups NQ .. NM-1  : O += V frag * P frag       ; row max of S[t+1], running-max update (a tile's last step)
    // The groups are expanded at compile time (static_for): left to the unroller, the d 128 / block 64 kernels kept
    // a run-time loop over register arrays, i.e. 320 B of scratch per lane (a gated layer of 2 x 8128 tokens, 32
    // heads: 49.2 ms with the loop, 1.07 ms without).
    constexpr int NQ = NR * DS, NP = NKS * DB, NM = NQ + NP, NU = SK / 4;  // NU: exp units (2 scores each)
    constexpr int PF = (WAVES == 3) ? 2 : 4;  // LDS fragments read ahead of the MFMA that uses them
    constexpr int MAXTAIL = LAST ? 4 : 0;  // the running-max update sits this many groups before the end
    auto frag = [&](int n) -> bf16x8 {
      if (n < NQ) return *reinterpret_cast<const bf16x8 *>(kb + ((n % NR) * DS + n / NR) * 1024);
      const int np = n - NQ;
      return *reinterpret_cast<const bf16x8 *>(vb + ((np % DB) * NKS + np / DB) * 1024);
    };
    // Whole images: LDS reads and ring refills two at a time, with one wait and one setting of M0 for both.  Bound by the
    // instructions it issues, a wavefront alone on its SIMD gains (tiny layer 37.6 -> 36.4 us, 7K d 64 145.0 -> 139.8, 4K
    // 135.8 -> 134.8); two on one SIMD do not lose.  The wait is fenced from the products behind it, which otherwise get waits
    // of their own again (4K 134.2 -> 132.0, lists of 98K 19.50 -> 19.24 ms).  Half images: the reads' wait comes too early
    // (gated 776 -> 779).  Three wavefronts per SIMD have no registers for a further fragment.
    constexpr bool READ2 = KH == 1 && WAVES == 2, REFILL2 = KH == 1;
    constexpr int NF = PF + (READ2 ? 2 : 1);
    bf16x8 fr[NF];
    bf16x8 pb[NKS];
    u32x4 pt;
    float lval = 0.f, alpha = 1.f, rs_tile = 0.f;
    const bool care_t = care;  // set when this tile's max was taken
    float xa[NU], xb[NU];
#pragma unroll
    for (int n = 0; n < PF; ++n) fr[n] = frag(n);
    __builtin_amdgcn_sched_barrier(0);  // all PF reads in flight before the first MFMA waits for one of them
    static_for<0, NM>([&](auto nc) __attribute__((always_inline)) {
      constexpr int n = decltype(nc)::value;
      if constexpr (!READ2) {
        if (n + PF < NM) fr[(n + PF) % NF] = frag(n + PF);
      } else if constexpr (n % 2 == 0) {
        static_assert(NM % 2 == 0 && PF % 2 == 0, "fragments come in pairs");
        wait_lds<(n + PF <= NM ? PF : NM - n) - 2>();  // fragments n and n + 1 are there
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (n + PF < NM) {
          fr[(n + PF) % NF] = frag(n + PF);
          fr[(n + PF + 1) % NF] = frag(n + PF + 1);
        }
      }
      if (n < NQ) {
        if (n < NR) {
          f32x16 z;
#pragma unroll
          for (int r = 0; r < 16; ++r) z[r] = 0.f;
          s_next[P * NR + n] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr[n % NF], qf[0], z, 0, 0, 0);
        } else {
          f32x16 &s = s_next[P * NR + n % NR];
          s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr[n % NF], qf[n / NR], s, 0, 0, 0);
        }
      }
      // exp units u (2 scores each), three stages in consecutive groups so that no instruction waits
      // on the one just issued: scale+shift in group g(u), exp2 in g(u)+1, row sum + bf16 pack in g(u)+2
#pragma unroll
      for (int u = 0; u < NU; ++u) {
        const int gu = u * NQ / NU;
        const int ks = u / 4, e2 = u % 4, r = 8 * (ks & 1) + 2 * e2;
        if (gu == n) {
          xa[u] = __builtin_fmaf(s_cur[P * NR + (ks >> 1)][r], p.c, -m);
          xb[u] = __builtin_fmaf(s_cur[P * NR + (ks >> 1)][r + 1], p.c, -m);
        }
        if (gu + 1 == n) {
          xa[u] = fast_exp2(xa[u]);
          xb[u] = fast_exp2(xb[u]);
        }
        if (gu + 2 == n) {
          rs0 = (P == 0 && u == 0) ? xa[u] : rs0 + xa[u];
          rs1 = (P == 0 && u == 0) ? xb[u] : rs1 + xb[u];
          pt[e2] = pack_bf16(xa[u], xb[u]);
          if (e2 == 3) pb[ks] = __builtin_bit_cast(bf16x8, pt);
        }
      }
      if (LAST && n == NQ + 2) {
        const float rs = sum_xor32(rs0 + rs1);
        rs_tile = rs;
        l += rs;
        bs += rs;
        if (SCORES && t % SPB == SPB - 1) {  // end of the key block: log2 of the block's exp-sum
          lval = m + fast_log2(bs);
          bs = 0.f;
        }
      }
      {
        constexpr int GAP = NM / (2 * CH);  // groups between two chunk loads
        constexpr int x = n / GAP;
        if constexpr (REFILL2) {
          static_assert(CH % 2 == 0, "a wavefront's share of an image is pairs of chunks");
          if constexpr (n % (2 * GAP) == 1 && x < CH) lds_dma16_pair<x * 1024>(ksrc, lane * 16, kslot + w * CH * 1024);
          if constexpr (n % (2 * GAP) == 1 && x >= CH && x < 2 * CH)
            lds_dma16_pair<(x - CH) * 1024>(vsrc, lane * 16, vslot + w * CH * 1024);
        } else {
          if constexpr (n % GAP == 1 && x < CH) issue_chunk(ksrc, kslot, std::integral_constant<int, x>{}, IsK{});
          if constexpr (n % GAP == 1 && x >= CH && x < 2 * CH)
            issue_chunk(vsrc, vslot, std::integral_constant<int, x - CH>{}, IsV{});
        }
      }
      if (n >= NQ) {
        const int np = n - NQ;
        oacc[np % DB] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr[n % NF], pb[np / DB], oacc[np % DB], 0, 0, 0);
        // row max of S[t+1]: NU max3 units spread over groups 2 .. NP-1-MAXTAIL, then the running-max
        // update MAXTAIL groups before the end (its dependent chain hides under the last MFMAs)
#pragma unroll
        for (int u = 0; u < NU; ++u) {
          if (2 + u * (NP - 2 - MAXTAIL) / NU != np) continue;
          const f32x16 &s = s_next[P * NR + u / 8];
          const float a0 = s[2 * (u % 8)], a1 = s[2 * (u % 8) + 1];
          float &m2 = u % 2 ? mx_odd : mx;  // two chains
          m2 = (P == 0 && u < 2) ? fmaxf(a0, a1) : max3f(m2, a0, a1);
        }
        if (LAST && np == NP - MAXTAIL) alpha = move_reference(max_xor32(fmaxf(mx, mx_odd)));
      }
      __builtin_amdgcn_sched_barrier(0);
    });
    if (care_t) {  // rare: the tile summed again as PV saw it (alpha already holds the move after this tile)
      add_p(part, pb);
      if (LAST) lc += (sum_xor32(psum) - rs_tile) * alpha;
    }
    if (LAST) {
      rescale(alpha);
      if (SCORES && t % SPB == SPB - 1 && h == 0) lrow[(int64_t)jt[0] * B] = lval;
    }
  };
  // general step: per-wavefront causal mask / skip near the diagonal, optional next tile
  auto slow_step = [&](auto part, int t, const int(&jt)[3], f32x16(&s_cur)[2], f32x16(&s_next)[2]) {
    constexpr int P = decltype(part)::value;
    const int u0 = t * KH + P;
    // the previous step's last LDS reads must be done before others refill their slot (a fast step ends with its MFMAs)
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    sync();
    issue_img(t + (P + DK) / KH, (P + DK) % KH, jt[(P + DK) / KH], IsK{}, lds_k + ((u0 + DK) % RK) * IMG);
    issue_img(t + (P + DV) / KH, (P + DV) % KH, jt[(P + DV) / KH], IsV{}, lds_v + v_old);
    const char *k_next = smem + ((u0 + KH) % RK) * IMG;
    const char *v_cur = smem + RK * IMG + v_now;
    next_v();
    const int sub = t % SPB, sub1 = (t + 1) % SPB;
    const int mode0 = mode_of(jt[0], sub);
    const int mode1 = (t + 1 < nsub) ? mode_of(jt[1], sub1) : 2;
    if (mode1 != 2) qk(part, k_next, s_next);
    if (mode0 != 2) {
      bf16x8 pb[NKS];
      tile_exp(part, t, s_cur, pb);
      pv(v_cur, pb);
    }
    if (P < KH - 1) return;
    if (SCORES && sub == SPB - 1 && mode_of(jt[0], 0) != 2) {
      if (h == 0) lrow[(int64_t)jt[0] * B] = m + fast_log2(bs);
      bs = 0.f;
    }
    if (mode1 != 2) {
      const float alpha = tile_max(s_next, mode1, sub1);
      rescale(alpha);
      if (QB > 1) lc += lc_later * alpha;
    }
  };
  auto fast_tile = [&](int t, int j0, int j1, int j2, f32x16(&s_cur)[2], f32x16(&s_next)[2]) {
    const int jt[3] = {j0, j1, j2};
    static_for<0, KH>([&](auto part) __attribute__((always_inline)) { fast_step(part, t, jt, s_cur, s_next); });
  };
  auto slow_tile = [&](int t, int j0, int j1, int j2, f32x16(&s_cur)[2], f32x16(&s_next)[2]) {
    const int jt[3] = {j0, j1, j2};
    static_for<0, KH>([&](auto part) __attribute__((always_inline)) { slow_step(part, t, jt, s_cur, s_next); });
  };

  if (nsub > 0) {
    f32x16 s_a[2], s_b[2];
    // jw[n] = key block of tile t + n
    int jw[6];
#pragma unroll
    for (int n = 0; n < 6; ++n) jw[n] = block_of(n);
    // prologue: V images 0 .. DV-1, K images 0 .. DK-1.  Those of K are one more than the ring has slots for where a tile
    // is two images: the first waits in the V slot that the first step will fill.
    const uint32_t k_first = (DK > RK) ? lds_v + DV * IMG : lds_k;
    static_for<0, (DK > DV ? DK : DV)>([&](auto nc) __attribute__((always_inline)) {
      constexpr int n = decltype(nc)::value;
      if (n / KH < nsub) {
        if (n < DV) issue_img(n / KH, n % KH, jw[n / KH], IsV{}, lds_v + n * IMG);
        if (n < DK) issue_img(n / KH, n % KH, jw[n / KH], IsK{}, n == 0 ? k_first : lds_k + (n % RK) * IMG);
      }
    });
    // leading run of tiles that lie before the first diagonal entry of the list
    int nfast;
    if (DENSE || list == nullptr) {
      nfast = (i - (QB - 1)) * SPB;
    } else {
      int first = nblk;
      for (int e0 = 0; e0 < nblk && first == nblk; e0 += 256) {
        int at[4];
#pragma unroll
        for (int x = 0; x < 4; ++x) {
          const int e = e0 + 64 * x + lane;
          at[x] = (e0 == 0 && x == 0) ? lst : list[e < nkb ? e : nkb - 1];
        }
#pragma unroll
        for (int x = 3; x >= 0; --x) {
          const int e = e0 + 64 * x + lane;
          const uint64_t hit = __ballot(e < nblk && at[x] >= i);
          if (hit) first = e0 + 64 * x + __builtin_ctzll(hit);
        }
      }
      nfast = first * SPB;
    }
    if (QB > 1) twice_from = (iw * SPB - 1) & ~1;
    // fast steps need tile t+1 off the diagonal too; keep their count even (tail starts on even parity)
    nfast = nfast > 0 ? ((nfast - 1) & ~1) : 0;

    wait_vm<0>();
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    {
      const int mode = mode_of(jw[0], 0);
      if (mode != 2) {
        static_for<0, KH>([&](auto part) __attribute__((always_inline)) {
          constexpr int n = decltype(part)::value;
          qk(part, smem + ((n == 0 && DK > RK) ? RK + DV : n % RK) * IMG, s_a);
        });
        tile_max(s_a, mode, 0);  // O is still zero: nothing to rescale
      }
    }
    int t = 0;
    for (; t < nfast; t += 2) {
      const int jn0 = block_of(t + 6), jn1 = block_of(t + 7);
      fast_tile(t, jw[0], jw[1], jw[2], s_a, s_b);
      fast_tile(t + 1, jw[1], jw[2], jw[3], s_b, s_a);
#pragma unroll
      for (int n = 0; n < 4; ++n) jw[n] = jw[n + 2];
      jw[4] = jn0;
      jw[5] = jn1;
    }
    for (; t < nsub; t += 2) {
      const int jn0 = block_of(t + 6), jn1 = block_of(t + 7);
      slow_tile(t, jw[0], jw[1], jw[2], s_a, s_b);
      if (t + 1 < nsub) slow_tile(t + 1, jw[1], jw[2], jw[3], s_b, s_a);
#pragma unroll
      for (int n = 0; n < 4; ++n) jw[n] = jw[n + 2];
      jw[4] = jn0;
      jw[5] = jn1;
    }
    wait_vm<0>();  // drain the ring's look-ahead loads before the LDS is reused or released
  }

  // ---- output: O = O^T accumulators / l, rounded to bf16 ----
  if (!idle) {
    const float inv = (l > 0.f) ? 1.f / (l + lc) : 0.f;
    uint16_t *op = p.o + (int64_t)b * p.o_sb + ((int64_t)iw * B + tq) * p.o_st + (int64_t)head * p.o_sh;
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
      for (int gq = 0; gq < 4; ++gq) {
        u32x2 t;
        t[0] = pack_bf16(oacc[db][4 * gq] * inv, oacc[db][4 * gq + 1] * inv);
        t[1] = pack_bf16(oacc[db][4 * gq + 2] * inv, oacc[db][4 * gq + 3] * inv);
        *reinterpret_cast<u32x2 *>(op + 32 * db + 8 * gq + 4 * h) = t;
      }
  }

  // ---- block-mass scores: S[i][j] = (1/B) sum_t 2^(lws[j][t] - L_t) ----
  // Each wavefront takes 32 key blocks at a time.  Stage 1: lane <-> query, coalesced reads of the block
  // log-sum-exps, one partial per (key block, lane) into a wavefront-private LDS tile (rows padded to 65
  // floats).  Stage 2: lane <-> key block, the tile is read transposed and summed.  No cross-lane reduction
  // chain and several rows of loads in flight: the workspace rows were written long ago and come from HBM.
  // The rows were stored by this workgroup, so the barrier's workgroup-scope ordering is enough to read them back.
  // (A device-scope fence here wrote back and invalidated the XCD's whole L2 once per workgroup, under all others:
  // score maps of 32 heads of 12352 tokens, d 64, block 64: 1200 us with it, 850 us without; 32K layer 3505 -> 3390.)
  if (SCORES) {
    constexpr int TPL = B / 64, PST = 65, JU = 8;
    constexpr int JB = (1024 + NW * 32 * PST * 4 <= (RK + RV) * IMG) ? 32 : 16;  // key blocks per tile
    constexpr int NPART = 64 / JB, PLEN = 64 / NPART;  // stage 2: NPART lanes share a key block, PLEN entries each
    static_assert(1024 + NW * JB * PST * 4 + QB * SP_FUSED_MASK_MAX * 4 <= (RK + RV) * IMG,
                  "score epilogue tiles and rows must fit the idle rings");
    float *lse_sh = reinterpret_cast<float *>(smem) + wb * B;  // [QB][B]; the rings are idle now
    float *part = reinterpret_cast<float *>(smem + 1024) + w * (JB * PST);
    __syncthreads();
    if (h == 0) lse_sh[tq] = m + fast_log2(l);
    __syncthreads();
    float *row_sh = reinterpret_cast<float *>(smem + 1024 + NW * JB * PST * 4) + wb * SP_FUSED_MASK_MAX;
    float lt[TPL];
#pragma unroll
    for (int tt = 0; tt < TPL; ++tt) lt[tt] = lse_sh[lane + 64 * tt];
    const float *lblk = p.lws + lws_row * B;
    float *srow = p.scores + (((int64_t)b * p.n_heads + hpos) * p.nqb + iw) * nkb;
    const int jr = lane % JB, jp = lane / JB;
    for (int j0 = wr * JB; j0 <= iw; j0 += WB * JB) {  // (iw < 0: nothing)
#pragma unroll
      for (int u0 = 0; u0 < JB; u0 += JU) {
        float x[JU][TPL];
#pragma unroll
        for (int u = 0; u < JU; ++u) {
          const int j = (j0 + u0 + u <= iw) ? j0 + u0 + u : iw;
#pragma unroll
          for (int tt = 0; tt < TPL; ++tt) x[u][tt] = lblk[(int64_t)j * B + lane + 64 * tt];
        }
#pragma unroll
        for (int u = 0; u < JU; ++u) {
          float e = 0.f;
#pragma unroll
          for (int tt = 0; tt < TPL; ++tt) e += fast_exp2(x[u][tt] - lt[tt]);
          part[(u0 + u) * PST + lane] = e;
        }
      }
      // the tile is private to this wavefront: order its own LDS writes before its transposed reads
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
      float acc = 0.f;
#pragma unroll
      for (int kq = 0; kq < PLEN; ++kq) acc += part[jr * PST + jp * PLEN + kq];
      acc = sum_xor32(acc);
      if (NPART == 4) acc += __shfl_xor(acc, 16, 64);
      if (jp == 0 && j0 + jr <= iw) {
        srow[j0 + jr] = acc * (1.f / B);
        if (p.mask_idx) row_sh[j0 + jr] = acc * (1.f / B);
      }
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }
    if (!idle)
      for (int j = iw + 1 + wr * 64 + lane; j < nkb; j += WB * 64) srow[j] = 0.f;
    // The row's list, by one wavefront, from the scores in LDS: the same row of mask_kernel, without its launch (5 us behind
    // the sweep of a short prompt, hidden behind other rows' steps here).
    if (p.mask_idx) {
      __syncthreads();
      if (!idle && wr == 0) {
        int64_t map = (int64_t)b * p.n_heads + hpos;
        if (p.route) map = p.route[map];
        if (map >= 0)
          mask_row<SP_FUSED_MASK_MAX / 64, 128>(row_sh, lane, iw, nkb, p.mask_gq, p.mask_idx + (map * p.nqb + iw) * nkb,
                                           p.mask_cnt + map * p.nqb + iw, nullptr);
      }
    }
  }
}

}  // namespace

#endif
