// General-path decode of fused-RoPE paged attention (§3.3.3) on matrix cores, for bf16 and e4m3 pages: both rotary
// pairings, D 64 / 128, pages of 16 / 32 slots, block positions, valid masks; also prefill of so few tokens per request that
// attn_prefill_split.hip would idle. Split precision (split_common.h).
//
// One workgroup of 4 waves serves one (query token, KV head, split of the KV); a wave takes a contiguous run of steps of 32
// slots (two groups of 16, each inside one page) for all G <= 16 heads of the group and the waves' partials are merged
// through LDS. Operands come straight from the pages, as in attn_decode_plain.hip:
//   S^T[16 slots x 16 heads] per group = Khat x Q'^T, three v_mfma_f32_16x16x32_bf16 per 32 dims
//   O  [16 heads x D]       += P x V, two per 16 dims of the output: a lane's k index runs over eight consecutive slots of one group,
//        8 (kg / 2) .. of group kg % 2, so that V comes in pieces of eight slots of a row. A lane's scores are those of slots 4 kg .. 4 kg + 3
//        of either group; one swap instruction a register between neighbouring k-groups brings their probabilities there.
// Rotation without a sine per key: q^.k^ = (R(pos_q - base) q).(R(pos_k - base) k). R(s), s in [0, kTab), is a table in LDS
// (fp32); base is the position of some earlier group, moved - and Q' computed afresh - when a group starts outside
// [base, base + kTab - 16] (or the part of it that short runs build): every fourth (eighth) step along a run of consecutive positions,
// and wherever block positions jump (a step whose groups lie too far apart is taken in two turns). The angles of a set-up are found once
// for the 16 lanes that share them.
// kTerms (D 128, rotate-half, G <= 8): the slow half of the pairs, frequencies 32 .. 63, is not rotated. Over the table's span it turns by x t
// about its middle, |x| <= 0.2, t in [-1, 1], and e^(-i x t) = (J0 + 2 J2) - i (2 J1 + 6 J3) t - 4 J2 t^2 + 8 i J3 t^3 up to 2 J4(x) = 2^-17
// (Jacobi-Anger, Chebyshev polynomials written out). A head has two matrix rows and there are two sets of products: four terms
// of Q', each as head and remainder, meet the keys as stored, exact in bf16, and the scores are their sum by powers of t.
//
// 64 requests of 4.3 K bf16 slots with valid masks and block positions, 32 heads on 8: 382 us (scalar) -> 110 us a call
// (loads with scalar bases in a fixed order, one round of workgroups) -> 84 us (terms, with half the set-ups; eight-slot pieces of V; 636 -> 431
// vector instructions a step, start-up and merge counted in) -> 80 - 84 us from card to card (the two waves of a SIMD by turns). e4m3: 35
// requests of up to 1.6 K slots 41 -> 28 us. Where no page is shared, HBM: 30 requests of up to 20 K bf16 slots on 12 heads 295 -> 222 us.
//
// A NaN or Inf in the merged result sends the workgroup through the scalar body: operand splits make NaN of some infinities, and
// probabilities of up to kMostSum times values near the largest float make Inf of finite ones.
#include <type_traits>

#include <limits.h>

#include "attn_scalar.h"
#include "split_common.h"

namespace mepic {
namespace {


constexpr int kWaves = 4, kThreads = 64 * kWaves;
constexpr float kMostSum = 64.f;      // a lane's probabilities of a step above which the reference maximum is raised

// Keep the stored elements whose bit of `keep` (8 bits) is set, zero the others.
__device__ __forceinline__ void mask_raw8(Raw8<false>& x, uint32_t keep) {
  Frag f;
  f.u = x.r;
  mask8(f, keep);
  x.r = f.u;
}
__device__ __forceinline__ void mask_raw8(Raw8<true>& x, uint32_t keep) {
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    x.r.x &= (keep >> e) & 1u ? ~0u : ~(0xffu << (8 * e));
    x.r.y &= (keep >> (4 + e)) & 1u ? ~0u : ~(0xffu << (8 * e));
  }
}

template <int D>
struct Merge {
  float m[kWaves][16], l[kWaves][16], o[kWaves][16][D];
};
// Dynamic LDS: the rotation table (with kTerms of the fast half only), whose place the merge and the scalar body take afterwards.
template <int D, bool kTerms, int kTab>
constexpr size_t lds_bytes() {
  size_t n = (size_t)D / (kTerms ? 8 : 4) * kTab * sizeof(float4);
  if (n < sizeof(Merge<D>)) n = sizeof(Merge<D>);
  return n < sizeof(ScalarLds<4, kThreads>) ? sizeof(ScalarLds<4, kThreads>) : n;
}

// kLong: calls whose waves have eight steps and more. Their table is whole, its size a constant; with D 128 the two workgroups of a
// compute unit share its SIMDs by turns (take_turns). In the others as much of the table is built as their groups of slots span.
template <bool kFp8, int D, int P, bool kIL, bool kTerms, int kTab, bool kLong>
__global__ __launch_bounds__(kThreads, 2) void decode_split_kernel(const AttnArgs a) {
  constexpr int kKs = D / 32;     // k-steps of 32 dims; granule of k-step j: dims 32 j + 8 kg ..
  constexpr int kNt = D / 16;     // output tiles of 16 dims
  constexpr int kRows = kTerms ? 2 : 1;  // matrix rows a head has
  constexpr bool kShare = D == 128;      // Q' set-up: sines shared by the lanes of a k-group (eight pairs: faster without)
  constexpr float kMiddle = 0.5f * (kTab - 1);  // of the table's span, and half its length
  typedef Merge<D> MergeT;
  static_assert(!kTerms || (D == 128 && !kIL), "the slow half of the pairs has k-steps of its own");
  extern __shared__ uint4 smem[];
  float4(*const tab)[kTab] = reinterpret_cast<float4(*)[kTab]>(smem);  // [frequencies 2 c, 2 c + 1][slot] {c0, s0, c1, s1}
  __shared__ uint4 q_lds[kKs][64];  // un-rotated q, granule j of every lane's head
  __shared__ __align__(16) float2 freq[D / 2];  // {hi, lo}: indexed per lane, which the kernel arguments are too slow for
  __shared__ float2 turn[kShare ? kWaves : 1][4][kRows][16];  // what Q' set-up shares: [wave][kg][row][pair] {cos, sin} times the row's factor
  __shared__ __align__(16) float ratio[2][32];   // [row][pair of the slow half]: the second set in units of the first
  __shared__ __align__(16) int span[kWaves];     // slots that each wave's groups span

  const int tid = threadIdx.x, lane = tid & 63, wave = uni(tid >> 6), n16 = lane & 15, kg = lane >> 4;
  if (tid < D / 2) freq[tid] = make_float2(a.freq_hi[tid], a.freq_lo[tid]);
  const int G = a.G, Hkv = a.Hkv;
  const int head = n16 / kRows, term = n16 % kRows;  // of this lane's matrix row
  // Q' set-up: lane n16 finds the angle of the n16-th of the pairs that its 16 lanes have in common. Rotate-half: pairs (dims i,
  // i + D/2) of granules h and h + kKs/2, i = 32 h + 8 kg + e; interleaved: four pairs inside each granule j, i = 16 j + 4 kg + e.
  const int my_pair = (kIL ? 16 * (n16 >> 2) + 4 * kg + (n16 & 3) : 32 * (n16 >> 3) + 8 * kg + (n16 & 7)) & (D / 2 - 1);
  const bool my_slow = kTerms && n16 >= 8;
  const int hk = (int)(blockIdx.x % (unsigned)Hkv), split = (int)blockIdx.z;
  const int t = (int)(blockIdx.y * (gridDim.x / (unsigned)Hkv) + blockIdx.x / (unsigned)Hkv);
  if (t >= a.n_q) return;

  // ---- the request that owns this query token: largest b with cu[b] <= t (64 probes at a time) ----
  int b = t;
  if (a.cu_q_lens) {
    b = 0;
    int hi = a.B;
    while (hi - b > 1) {
      const int step = (hi - b + 63) / 64, c = b + lane * step;
      const int n = __popcll(__ballot(c < hi && (c == 0 || a.cu_q_lens[c] <= t)));
      b += max(n - 1, 0) * step;
      hi = min(b + step, hi);
    }
    b = uni(b);
  }
  const int L = uni(a.kv_lens[b]), pos_q = uni(a.q_positions[t]);
  const int n_begin = split * a.blocks_per_split * P;
  const int s_end = min(L, (split + 1) * a.blocks_per_split * P);
  int n_end = s_end;
  if (a.causal && !a.block_positions) n_end = min(n_end, max(pos_q, -1) + 1);

  // ---- this wave's steps, and what their groups of 16 slots are: lane i of a window holds group i of 32 steps ----
  const int n_steps = n_end > n_begin ? (n_end - n_begin + 31) / 32 : 0;
  const int per_wave = (n_steps + kWaves - 1) / kWaves;
  const int st0 = wave * per_wave, n_st = max(min(per_wave, n_steps - st0), 0);
  struct Win {
    int page, pos;
    uint32_t vis;
    float ksc, vsc;
  };
  const size_t bt_row = (size_t)b * a.max_blocks;
  auto win_load = [&](Win& w, int win) __attribute__((always_inline)) {
    const int n = n_begin + 32 * st0 + (64 * win + lane) * 16;  // first slot of the group
    const int j = min(n, L - 1) / P, off = n % P;
    w.page = max(min(a.block_tables[bt_row + j], a.num_pages - 1), 0);  // a corrupt id reads a wrong page, never faults
    w.pos = a.block_positions ? a.block_positions[bt_row + j] + off : n;
    uint32_t v = a.block_valid_mask ? (a.block_valid_mask[bt_row + j] >> off) & 0xffffu : 0xffffu;
    const int left = n_end - n;
    if (left < 16) v &= left <= 0 ? 0u : (1u << left) - 1u;
    if (a.causal) {  // one query token: what the causal rule hides is the same for all rows
      const long ahead = (long)pos_q - w.pos;  // the group's slots 0 .. ahead are visible
      if (ahead < 15) v &= ahead < 0 ? 0u : (2u << ahead) - 1u;
    }
    w.vis = v;
    w.ksc = w.vsc = 1.f;
    if constexpr (kFp8) {
      w.ksc = a.k_scales[w.page];
      w.vsc = a.v_scales[w.page];
    }
  };
  Win cur{}, nxt;
  int win = 0;
  if (n_st > 0) {
    win_load(cur, 0);
    nxt = cur;
    if (n_st > 32) win_load(nxt, 1);
  }

  // ---- K and V of a step. K row n16 of product u is slot n16 of group u. ----
  // (addresses: a page's base is uniform and a lane's place in it never changes, so that the loads take a scalar base, a
  // 32-bit lane offset and an immediate - as 64-bit sums per load the addresses alone were 130 vector instructions a step)
  using RawT = decltype(Raw8<kFp8>::r);
  constexpr int kElem = kFp8 ? 1 : 2;
  constexpr size_t kHeadBytes = (size_t)D * P * kElem;       // one KV head of a page, K or V alike
  // V: dim 16 nt + n16, eight slots 8 (kg / 2) .. of group kg % 2 in one load (the time that a load takes to address does not
  // depend on its width: e4m3 pages, 8 requests of 3 - 6 K slots on 12 heads, 44 us in two loads, 33 in one)
  Raw8<kFp8> kf[2][kKs];
  Raw8<kFp8> vf[kNt];
  const uint32_t k_off = kFp8 ? (uint32_t)(((kg >> 1) * P + n16) * 16 + (kg & 1) * 8) : (uint32_t)((kg * P + n16) * 16);
  const uint32_t v_off = (uint32_t)((n16 * P + 8 * (kg >> 1) + (P == 16 ? 0 : 16 * (kg & 1))) * kElem);
  constexpr uint32_t kStepK = (kFp8 ? 2 : 4) * P * 16;        // bytes between a lane's granules of successive k-steps
  auto issue_k = [&](int pg0, int pg1) __attribute__((always_inline)) {
    // steps start at multiples of 32: a page of 32 is a whole step
    const char* b0 = reinterpret_cast<const char*>(a.k_pages) + ((size_t)pg0 * Hkv + hk) * kHeadBytes;
    const char* b1 = reinterpret_cast<const char*>(a.k_pages) + ((size_t)pg1 * Hkv + hk) * kHeadBytes + (P == 16 ? 0 : 16 * 16);
#pragma unroll
    for (int j = 0; j < kKs; ++j) {
      kf[0][j].r = *reinterpret_cast<const RawT*>(b0 + j * kStepK + k_off);
      kf[1][j].r = *reinterpret_cast<const RawT*>(b1 + j * kStepK + k_off);
    }
  };
  auto issue_v = [&](int pg0, int pg1) __attribute__((always_inline)) {
    const char* base = reinterpret_cast<const char*>(a.v_pages) + ((size_t)((kg & 1) ? pg1 : pg0) * Hkv + hk) * kHeadBytes + v_off;
#pragma unroll
    for (int nt = 0; nt < kNt; ++nt) vf[nt].r = *reinterpret_cast<const RawT*>(base + nt * (16 * P * kElem));
  };
  int np0 = 0, np1 = 0;  // pages of the next step
  if (n_st > 0) {
    np0 = __builtin_amdgcn_readlane(cur.page, 0);
    np1 = __builtin_amdgcn_readlane(cur.page, 1);
    issue_k(np0, np1);
    __builtin_amdgcn_sched_barrier(0);  // K before V on every path: the loop's waits count on it
    issue_v(np0, np1);
    __builtin_amdgcn_sched_barrier(0);
  }

  // ---- q of this lane's head, un-rotated: granule j as stored ----
  const bool row_ok = term == 0 && head < G;
  if (wave == 0) {
    const uint4* q4 = reinterpret_cast<const uint4*>(a.q) + ((size_t)t * a.Hq + (size_t)hk * G + (head < G ? head : 0)) * (D / 8);
#pragma unroll
    for (int j = 0; j < kKs; ++j) q_lds[j][lane] = head < G ? q4[4 * j + kg] : make_uint4(0, 0, 0, 0);  // (rows without a head are zeros)
  }

  // ---- rotation table, 32 slots at a time ----
  // Of calls of few steps, building it whole was up to 1.5 us of the start: there it goes as far as the groups of some wave span, gaps of up
  // to half a table included, since every group outside is a new base and a set-up of Q' (longer gaps are that however long the table is: with 200
  // slots left out after every 48, 2 requests of 7 K on 2 heads 14.3 us if they count, 13.8 if not). us a call, whole and
  // so: 1 masked request of 3.9 K slots on 12 heads 13.75 and 12.65, 2 of 7 K on 2 heads 13.45 and 12.1 (with 16 slots left out after
  // every 32 of them 13.4 and 12.2; by the length of the runs alone 13.85), 24 of 0.6 - 1.1 K e4m3 slots in three parts 22.15 and 20.05, 100 of 250
  // 25.45 and 23.3, 2 of 1.2 K, D 64, 9.58 and 9.2. What it adds to calls that need the whole table all the same is within 0.5 % (11 requests
  // of 2.4 - 5 K e4m3 slots, D 64, 20.85 and 20.95), 1 % in one form (e4m3, theta 1e4, 20 requests of 700 slots 17.9 and 18.1).
  constexpr int kChunks = kTab / 32;
  static_assert(kTab % 32 == 0 && kChunks <= 8, "the groups of a run that may need less lie in a row of lanes");
  if constexpr (!kLong) {
    // from the group before (16 groups, a row of lanes, are as many as there are in runs that do not need it whole); written as a sum
    // because the difference, v_subrev_u32_dpp, came out with its sign turned
    const uint32_t up = (uint32_t)cur.pos + (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(0u - (uint32_t)cur.pos), 0x111, 0xf, 0xf, true);  // row_shr:1
    int x = lane > 0 && lane < 2 * n_st && up <= kTab / 2 ? (int)up : 0;
    x += __builtin_amdgcn_update_dpp(0, x, 0x121, 0xf, 0xf, true);  // row_ror:1, 2, 4, 8
    x += __builtin_amdgcn_update_dpp(0, x, 0x122, 0xf, 0xf, true);
    x += __builtin_amdgcn_update_dpp(0, x, 0x124, 0xf, 0xf, true);
    x += __builtin_amdgcn_update_dpp(0, x, 0x128, 0xf, 0xf, true);
    if (lane == 0) span[wave] = x + 16;
  }
  __syncthreads();
  const float my_hi = freq[my_pair].x, my_lo = freq[my_pair].y;
  float my_f0 = a.qk_scale_log2, my_f1 = 0.f;  // factors of the two rows
  if constexpr (kTerms) {
    if (my_slow) {
      const float x = kMiddle * 6.283185307f * my_hi, h = 0.5f * x, y = h * h;  // Bessel functions of x, as far as x <= 0.2 has use for
      const float j0 = 1.f - y * (1.f - 0.25f * y), j2 = 0.5f * y * (1.f - y * (1.f / 3.f));
      // (J1 and J3 in units of h, which is 0 for pairs that do not turn at all: rope_theta infinite)
      const float j1 = 1.f - y * (0.5f - y * (1.f / 12.f)), j3 = y * (1.f / 6.f) * (1.f - 0.25f * y);
      my_f1 = my_f0 * h * (2.f * j1 + 6.f * j3);
      my_f0 *= j0 + 2.f * j2;
      if (wave == 0) {
        ratio[0][my_pair - 32] = -4.f * j2 / (j0 + 2.f * j2);
        ratio[1][my_pair - 32] = -4.f * j3 / (j1 + 3.f * j3);
      }
    }
  }
  constexpr int kPairs2 = D / (kTerms ? 8 : 4);  // pairs in the table, by two
  constexpr int kOwn = kPairs2 * 32 / kThreads;  // a thread's entries of 32 slots: columns tid / 32 + 8 k
  static_assert(kThreads == 8 * 32 && kPairs2 % 8 == 0, "a pass of the threads is 32 slots of eight columns");
  float4 f[kOwn];
#pragma unroll
  for (int k = 0; k < kOwn; ++k) f[k] = *reinterpret_cast<const float4*>(&freq[2 * (tid / 32 + 8 * k)]);
  auto build = [&](int chunk) __attribute__((always_inline)) {
    const int s = 32 * chunk + tid % 32;
#pragma unroll
    for (int k = 0; k < kOwn; ++k) {
      const float t0 = turns_frac((float)s, f[k].x, f[k].y), t1 = turns_frac((float)s, f[k].z, f[k].w);
      tab[tid / 32 + 8 * k][s] = make_float4(__builtin_amdgcn_cosf(t0), __builtin_amdgcn_sinf(t0), __builtin_amdgcn_cosf(t1),
                                             __builtin_amdgcn_sinf(t1));
    }
  };
  build(0);
  int n_chunks = kChunks;
  if constexpr (!kLong) n_chunks = max(1, min(max(per_wave, uni(max(max(span[0], span[1]), max(span[2], span[3])) + 31) / 32), kChunks));
  const int n_tab = 32 * n_chunks;
#pragma unroll 1
  for (int i = 1; i < n_chunks; ++i) build(i);
  __syncthreads();

  // Q' as the B operands. kTerms: qh / ql hold the first set of the slow half (pairs of granules 1 and 3), qh2 / ql2 the second.
  Frag qh[kKs], ql[kKs], qh2[2], ql2[2];
  auto rotate_q = [&](int base) __attribute__((always_inline)) {
    const float delta = (float)(pos_q - base);
    if constexpr (kShare) {
      const float tr = turns_frac(my_slow ? delta - kMiddle : delta, my_hi, my_lo);
      const float c = __builtin_amdgcn_cosf(tr), s = __builtin_amdgcn_sinf(tr);
      turn[wave][kg][0][n16] = make_float2(c * my_f0, s * my_f0);
      if constexpr (kTerms) turn[wave][kg][kRows - 1][n16] = make_float2(s * my_f1, -c * my_f1);  // (times -i)
      __builtin_amdgcn_wave_barrier();  // (the wave's own LDS accesses are served in order)
    }
    int again = 0;
    asm volatile("" : "+v"(again));  // q is fetched anew each time: it must not stay in registers
    auto rot = [&](float x0, float x1, int p, float& y0, float& y1) __attribute__((always_inline)) {
      float2 r;
      if constexpr (kShare) {
        r = turn[wave][kg][term][p + again];
      } else {
        const float2 f = freq[(kIL ? 16 * (p >> 2) + 4 * kg + (p & 3) : 32 * (p >> 3) + 8 * kg + (p & 7)) + again];
        const float tr = turns_frac(delta, f.x, f.y);
        r = make_float2(__builtin_amdgcn_cosf(tr) * my_f0, __builtin_amdgcn_sinf(tr) * my_f0);
      }
      y0 = x0 * r.x - x1 * r.y;
      y1 = x1 * r.x + x0 * r.y;
    };
#pragma unroll
    for (int j = 0; j < (kIL ? kKs : kKs / 2); ++j) {
      Frag qa, qb;
      qa.u = q_lds[j][lane + again];
      if constexpr (!kIL) qb.u = q_lds[j + kKs / 2][lane + again];
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        if constexpr (kIL) {
          float y0, y1;
          rot(__uint_as_float(qa.w[w] << 16), __uint_as_float(qa.w[w] & 0xffff0000u), 4 * j + w, y0, y1);
          split2(y0, y1, qh[j].w[w], ql[j].w[w]);
        } else {
          const int j1 = j + kKs / 2;
          float a0, b0, a1, b1;
          rot(__uint_as_float(qa.w[w] << 16), __uint_as_float(qb.w[w] << 16), 8 * j + 2 * w, a0, b0);
          rot(__uint_as_float(qa.w[w] & 0xffff0000u), __uint_as_float(qb.w[w] & 0xffff0000u), 8 * j + 2 * w + 1, a1, b1);
          split2(a0, a1, qh[j].w[w], ql[j].w[w]);
          split2(b0, b1, qh[j1].w[w], ql[j1].w[w]);
          if (kTerms && j == 1) {
            const float2 r = *reinterpret_cast<const float2*>(&ratio[term][8 * kg + 2 * w + again]);
            split2(a0 * r.x, a1 * r.y, qh2[0].w[w], ql2[0].w[w]);
            split2(b0 * r.x, b1 * r.y, qh2[1].w[w], ql2[1].w[w]);
          }
        }
      }
    }
  };
  floatx4 sc0 = {0.f, 0.f, 0.f, 0.f};  // minus the reference maximum (log2 units): what bf16 score accumulators start from
  // scores of group u (16 slots x 16 rows) relative to the reference (e4m3: before the page's scale), its keys rotated by
  // R(s), s = s0 + n16
  auto score = [&](int u, int s0) __attribute__((always_inline)) {
    floatx4 sc;
    if constexpr (kFp8) sc = floatx4{0.f, 0.f, 0.f, 0.f};
    else sc = sc0;
    const float4* tp = &tab[0][min(max(s0, 0), n_tab - 16) + n16];
    auto three = [&](const Frag& kh, const Frag& kl, int j) __attribute__((always_inline)) {
      sc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kh.v, qh[j].v, sc, 0, 0, 0);
      sc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kh.v, ql[j].v, sc, 0, 0, 0);
      sc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kl.v, qh[j].v, sc, 0, 0, 0);
    };
#pragma unroll
    for (int j = 0; j < (kIL ? kKs : kTerms ? kKs / 4 : kKs / 2); ++j) {
      if constexpr (kIL) {
        float x[8];
        widen8<kFp8>(kf[u][j], x);
        Frag h, l;
#pragma unroll
        for (int w = 0; w < 4; w += 2) {
          const float4 r = tp[(8 * j + 2 * kg + w / 2) * kTab];
          split2(x[2 * w] * r.x - x[2 * w + 1] * r.y, x[2 * w + 1] * r.x + x[2 * w] * r.y, h.w[w], l.w[w]);
          split2(x[2 * w + 2] * r.z - x[2 * w + 3] * r.w, x[2 * w + 3] * r.z + x[2 * w + 2] * r.w, h.w[w + 1], l.w[w + 1]);
        }
        three(h, l, j);
      } else {
        const int j1 = j + kKs / 2;
        float x[8], y[8];
        widen8<kFp8>(kf[u][j], x);
        widen8<kFp8>(kf[u][j1], y);
        Frag h0, l0, h1, l1;
#pragma unroll
        for (int w = 0; w < 4; ++w) {
          const float4 r = tp[(16 * j + 4 * kg + w) * kTab];
          split2(x[2 * w] * r.x - y[2 * w] * r.y, x[2 * w + 1] * r.z - y[2 * w + 1] * r.w, h0.w[w], l0.w[w]);
          split2(y[2 * w] * r.x + x[2 * w] * r.y, y[2 * w + 1] * r.z + x[2 * w + 1] * r.w, h1.w[w], l1.w[w]);
        }
        three(h0, l0, j);
        three(h1, l1, j1);
      }
    }
    if constexpr (kTerms) {  // the slow half: keys as they are, exact in bf16
      const Frag k0 = bf16_of8<kFp8>(kf[u][1]), k1 = bf16_of8<kFp8>(kf[u][3]);
      floatx4 s2 = {0.f, 0.f, 0.f, 0.f};
      sc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(k0.v, qh[1].v, sc, 0, 0, 0);
      s2 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(k0.v, qh2[0].v, s2, 0, 0, 0);
      sc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(k0.v, ql[1].v, sc, 0, 0, 0);
      s2 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(k0.v, ql2[0].v, s2, 0, 0, 0);
      sc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(k1.v, qh[3].v, sc, 0, 0, 0);
      s2 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(k1.v, qh2[1].v, s2, 0, 0, 0);
      sc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(k1.v, ql[3].v, sc, 0, 0, 0);
      s2 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(k1.v, ql2[1].v, s2, 0, 0, 0);
      const float t0 = (float)(s0 + 4 * kg) * (1.f / kMiddle) - 1.f;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float t = t0 + (float)e / kMiddle;
        float x = __builtin_fmaf(lane_up<1>(s2[e]), t, s2[e]);
        x = __builtin_fmaf(x, t, lane_up<1>(sc[e]));
        sc[e] = __builtin_fmaf(x, t, sc[e]);
      }
    }
    return sc;
  };

  floatx4 o[kNt];
#pragma unroll
  for (int nt = 0; nt < kNt; ++nt) o[nt] = floatx4{0.f, 0.f, 0.f, 0.f};
  bool unset = true;  // no reference maximum yet
  float l_part = 0.f;
  int base = 0;
  bool have_base = false;
  auto inside = [&](int ps) __attribute__((always_inline)) {
    return (uint64_t)((long)ps - base) <= (uint64_t)(n_tab - 16);  // (not below 0 either; one comparison)
  };

  // Softmax and output products of one turn; slots of the step outside vis0 / vis1 get no weight.
  auto attend = [&](floatx4 (&sc)[2], uint32_t vis0, uint32_t vis1, int l0) __attribute__((always_inline)) {
    float vs0 = 1.f, vs1 = 1.f;
    if constexpr (kFp8) {
      const float ks0 = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(cur.ksc), l0));
      const float ks1 = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(cur.ksc), l0 + 1));
      vs0 = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(cur.vsc), l0));
      vs1 = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(cur.vsc), l0 + 1));
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        sc[0][e] = __builtin_fmaf(sc[0][e], ks0, sc0[e]);
        sc[1][e] = __builtin_fmaf(sc[1][e], ks1, sc0[e]);
      }
    }
    const bool partial = (vis0 & vis1) != 0xffffu;
    if (partial) {
      asm volatile("");  // a branch, not selects in every step
#pragma unroll
      for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (!(((u ? vis1 : vis0) >> (4 * kg + e)) & 1u)) sc[u][e] = -INFINITY;
    }
    float pf[8], psum;
    auto exps = [&]() __attribute__((always_inline)) {
#pragma unroll
      for (int e = 0; e < 8; ++e) pf[e] = __builtin_amdgcn_exp2f(sc[e >> 2][e & 3]);
      psum = ((pf[0] + pf[1]) + (pf[2] + pf[3])) + ((pf[4] + pf[5]) + (pf[6] + pf[7]));
    };
    exps();
    // the reference maximum only has to keep probabilities bounded (2^6): raised, with everything accumulated so far rescaled,
    // when a lane's sum gets past that
    if (__ballot(row_ok && (unset || !(psum <= kMostSum))) != 0) {
      const float mx = max_over_kgroups(fmaxf(fmaxf(fmaxf(sc[0][0], sc[0][1]), fmaxf(sc[0][2], sc[0][3])),
                                              fmaxf(fmaxf(sc[1][0], sc[1][1]), fmaxf(sc[1][2], sc[1][3]))));
      float up = unset ? mx : fmaxf(mx, 0.f);
      if (!row_ok || up == -INFINITY) up = 0.f;  // (the other terms' rows have no reference)
      const float alpha = unset ? 1.f : __builtin_amdgcn_exp2f(-up);
      sc0 -= up;
      sc[0] -= up;
      sc[1] -= up;
      exps();
      if (__ballot(row_ok && !unset) != 0) {  // (nothing is accumulated before the first step)
        l_part *= alpha;
#pragma unroll
        for (int e = 0; e < 4; ++e) {  // accumulator rows of this lane are matrix rows 4 kg + e; their factors live in lanes 4 kg + e
          const float ar = __shfl(alpha, 4 * kg + e);
#pragma unroll
          for (int nt = 0; nt < kNt; ++nt) o[nt][e] *= ar;
        }
      }
      unset = unset && mx == -INFINITY;
    }
    l_part += psum;
    if constexpr (kFp8) {
#pragma unroll
      for (int e = 0; e < 8; ++e) pf[e] *= e < 4 ? vs0 : vs1;
    }
    if (partial) {  // slots that take no part may hold anything, NaN included, and so may the scale of a page of such
      asm volatile("");
      // (V in place: a group whose turn is yet to come keeps its slots, under probabilities of zero)
      const uint32_t all0 = (uint32_t)__builtin_amdgcn_readlane((int)cur.vis, l0), all1 = (uint32_t)__builtin_amdgcn_readlane((int)cur.vis, l0 + 1);
      const uint32_t keep = (((kg & 1) ? all1 : all0) >> (8 * (kg >> 1))) & 0xffu;
#pragma unroll
      for (int nt = 0; nt < kNt; ++nt) mask_raw8(vf[nt], keep);
      if constexpr (kFp8) {
#pragma unroll
        for (int e = 0; e < 8; ++e)
          if (!(((e < 4 ? vis0 : vis1) >> (4 * kg + (e & 3))) & 1u)) pf[e] = 0.f;
      }
    }
    Frag ph, pl;
#pragma unroll
    for (int w = 0; w < 4; ++w) split2(pf[2 * w], pf[2 * w + 1], ph.w[w], pl.w[w]);
    // A lane has the probabilities of four slots of either group; exchanged between neighbouring k-groups they are those of
    // the eight slots of one group that its V has.
#pragma unroll
    for (int w = 0; w < 2; ++w) {
      const auto x = __builtin_amdgcn_permlane16_swap(ph.w[w], ph.w[w + 2], false, false);
      const auto y = __builtin_amdgcn_permlane16_swap(pl.w[w], pl.w[w + 2], false, false);
      ph.w[w] = x[0]; ph.w[w + 2] = x[1];
      pl.w[w] = y[0]; pl.w[w + 2] = y[1];
    }
#pragma unroll
    for (int nt = 0; nt < kNt; ++nt) {
      const Frag vb = bf16_of8<kFp8>(vf[nt]);
      o[nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ph.v, vb.v, o[nt], 0, 0, 0);
      o[nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(pl.v, vb.v, o[nt], 0, 0, 0);
    }
  };

  // K of the next step is requested as soon as the scores are done with the registers, V after its products; always, so
  // that the waits can count the loads in flight (past the last step the last pages come once more).
  const bool later = kLong && D == 128 && (int)(blockIdx.x + gridDim.x * (blockIdx.y + gridDim.y * blockIdx.z)) >= a.later_wg;
  for (int st = 0; st < n_st; ++st) {
    const int l0 = (2 * st) & 63;
    if (st > 0 && l0 == 0) {
      cur = nxt;
      ++win;
      if (n_st > 32 * (win + 1)) win_load(nxt, win + 1);
    }
    const int cp0 = np0, cp1 = np1;
    if (st + 1 < n_st) {
      const int pages = l0 == 62 ? nxt.page : cur.page, l1 = (l0 + 2) & 63;
      np0 = __builtin_amdgcn_readlane(pages, l1);
      np1 = __builtin_amdgcn_readlane(pages, l1 + 1);
    }
    const int ps0 = __builtin_amdgcn_readlane(cur.pos, l0), ps1 = __builtin_amdgcn_readlane(cur.pos, l0 + 1);
    const uint32_t vis0 = (uint32_t)__builtin_amdgcn_readlane((int)cur.vis, l0), vis1 = (uint32_t)__builtin_amdgcn_readlane((int)cur.vis, l0 + 1);
    if (!have_base || (vis0 && !inside(ps0)) || (!vis0 && vis1 && !inside(ps1))) {
      base = vis0 ? ps0 : ps1;
      have_base = true;
      rotate_q(base);
    }
    const bool both = inside(ps1);  // (a group without visible slots may be rotated by anything)
    floatx4 sc[2];
    sc[0] = score(0, ps0 - base);
    sc[1] = score(1, ps1 - base);
    __builtin_amdgcn_sched_barrier(0);
    issue_k(np0, np1);
    if constexpr (kLong && D == 128) take_turns(later, st);
    __builtin_amdgcn_sched_barrier(0);
    attend(sc, vis0, both ? vis1 : 0u, l0);
    if (!both && vis1) {  // the step's groups lie too far apart for one table: the second one takes a turn of its own
      issue_k(cp0, cp1);
      base = ps1;
      rotate_q(base);
      sc[0] = floatx4{0.f, 0.f, 0.f, 0.f};
      sc[1] = score(1, 0);
      attend(sc, 0u, vis1, l0);
      issue_k(np0, np1);
    }
    __builtin_amdgcn_sched_barrier(0);
    issue_v(np0, np1);
    __builtin_amdgcn_sched_barrier(0);
  }

  // ---- merge the waves (the table's LDS is free now), write the split's partial or, if it is the only one, the rows ----
  __syncthreads();
  MergeT& mg = *reinterpret_cast<MergeT*>(smem);
  {
    const float l_tot = sum_over_kgroups(l_part);
    if (kg == 0) {
      mg.m[wave][n16] = unset ? -INFINITY : -sc0[0];
      mg.l[wave][n16] = l_tot;
    }
#pragma unroll
    for (int nt = 0; nt < kNt; ++nt)
#pragma unroll
      for (int e = 0; e < 4; ++e) mg.o[wave][4 * kg + e][16 * nt + n16] = o[nt][e];
  }
  __syncthreads();
  const bool direct = a.n_splits == 1;
  bool odd = false;
  for (int i = tid; i < G * (D / 4); i += kThreads) {
    const int g = i / (D / 4), dq = i % (D / 4);
    const int r = g * kRows;  // the head's matrix row
    float m = mg.m[0][r];
#pragma unroll
    for (int w = 1; w < kWaves; ++w) m = fmaxf(m, mg.m[w][r]);
    float4 x = make_float4(0.f, 0.f, 0.f, 0.f);
    float l = 0.f;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
      const float f = mg.m[w][r] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(mg.m[w][r] - m);
      const float4 y = *reinterpret_cast<const float4*>(&mg.o[w][r][4 * dq]);
      x.x += f * y.x; x.y += f * y.y; x.z += f * y.z; x.w += f * y.w;
      l += f * mg.l[w][r];
    }
    const float all = (x.x + x.y) + (x.z + x.w) + l;
    odd |= !(fabsf(all) < INFINITY);
    const size_t row = (size_t)t * a.Hq + (size_t)hk * G + g;
    if (direct) {
      const float inv = l != 0.f ? 1.f / l : 0.f;
      uint2 w;
      w.x = pack2_bf16(x.x * inv, x.y * inv);
      w.y = pack2_bf16(x.z * inv, x.w * inv);
      reinterpret_cast<uint2*>(a.out)[row * (D / 4) + dq] = w;
    } else {
      const size_t pr = row * a.n_splits + split;
      reinterpret_cast<float4*>(a.part_o)[pr * (D / 4) + dq] = x;
      if (dq == 0) {
        a.part_ml[2 * pr] = m;
        a.part_ml[2 * pr + 1] = l;
      }
    }
  }
  if (__syncthreads_or(odd ? 1 : 0))
    scalar_attend_all<kFp8 ? MEPIC_F8E4M3 : MEPIC_BF16, kThreads>(a, *reinterpret_cast<ScalarLds<4, kThreads>*>(smem), t, b, hk, 0, G,
                                                                  n_begin, s_end, split, direct);
}

template <bool kFp8, int D, int P, bool kIL, bool kTerms, int kTab, bool kLong = false>
hipError_t launch_one(const AttnArgs& a, hipStream_t s) {
  // From eight steps a wave on turns are worth what they add to the loop (64 requests of 4.2 K slots with masks, 34 steps a wave, 84.0 -> 80.2 us;
  // 2 of 7 K on 2 heads, 7 steps, 13.1 -> 13.3, 2 of 1.2 K, D 64, 9.54 -> 9.75), and every run that is not a request's last needs the whole
  // table: as a constant 56.3 us for 64 requests of 4.2 K slots, D 64, as a number known to the kernel only 56.9.
  if constexpr (!kLong)
    if (a.blocks_per_split * P >= 8 * 32 * kWaves) return launch_one<kFp8, D, P, kIL, kTerms, kTab, true>(a, s);
  constexpr size_t lds = lds_bytes<D, kTerms, kTab>();
  static std::atomic<uint64_t> asked{0};
  const hipError_t status = allow_lds(reinterpret_cast<const void*>(&decode_split_kernel<kFp8, D, P, kIL, kTerms, kTab, kLong>), lds, asked);
  if (status != hipSuccess) return status;
  // KV heads fastest (neighbours go to different dies, which then each keep their own heads' pages); tokens over x and y
  const unsigned per_row = (unsigned)min(a.n_q, max(65536 / a.Hkv, 1));
  const dim3 grid((unsigned)a.Hkv * per_row, ((unsigned)a.n_q + per_row - 1) / per_row, (unsigned)a.n_splits);
  hipLaunchKernelGGL((decode_split_kernel<kFp8, D, P, kIL, kTerms, kTab, kLong>), grid, dim3(kThreads), lds, s, a);
  return hipGetLastError();
}
template <bool kFp8, int D, int P>
hipError_t launch_il(const AttnArgs& a, hipStream_t s) {
  if (a.interleaved) return launch_one<kFp8, D, P, true, false, 128>(a, s);
  if constexpr (D == 128) {
    // Terms where four of them are enough: x = half the table's span times the fastest slow frequency (rope_theta 4.1e5 and up with 256
    // slots, 1.01e5 with 128). 84 us with 256 slots on the call above, 92 with 128.
    const float f = 6.283185307f * a.freq_hi[32];
    if (a.G <= 8 && 127.5f * f <= 0.2f) return launch_one<kFp8, D, P, false, true, 256>(a, s);
    if (a.G <= 8 && 63.5f * f <= 0.2f) return launch_one<kFp8, D, P, false, true, 128>(a, s);
  }
  return launch_one<kFp8, D, P, false, false, 128>(a, s);
}
template <bool kFp8>
hipError_t launch_kv(const AttnArgs& a, hipStream_t s) {
  if (a.D == 128) return a.P == 16 ? launch_il<kFp8, 128, 16>(a, s) : launch_il<kFp8, 128, 32>(a, s);
  return a.P == 16 ? launch_il<kFp8, 64, 16>(a, s) : launch_il<kFp8, 64, 32>(a, s);
}

}  // namespace

hipError_t launch_decode_split(const AttnArgs& args, hipStream_t s) {
  AttnArgs a = args;
  // Turns: up to two workgroups a compute unit in one round; of more, which one is the later changes as they end. Not where the caller says
  // that pages are not shared: HBM sets the time there, and the two workgroups' loads come less evenly (64 private requests of 2.1 and
  // 4.2 K slots 92.5 and 178.6 us, by turns 94.4 and 184.6, as they are where the caller does not say so; shared ones 3 - 8 % faster by turns).
  const long cus = device_compute_units(), n_wg = (long)a.n_q * a.Hkv * a.n_splits;
  a.later_wg = n_wg > cus && n_wg <= 2 * cus && !a.kv_read_once ? (int)cus : INT_MAX;
  return a.kv_dtype == MEPIC_F8E4M3 ? launch_kv<true>(a, s) : launch_kv<false>(a, s);
}

}  // namespace mepic
