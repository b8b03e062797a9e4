// General-path decode of fused-RoPE paged attention (§3.3.3) on matrix cores, for bf16 and e4m3 pages: both rotary
// pairings, D 64 / 128, pages of 16 / 32 slots, block positions, valid masks; also prefill of so few tokens per request that
// attn_prefill_split.hip would idle. Split precision (split_common.h).
//
// One workgroup of 4 waves serves one (query token, KV head, split of the KV); a wave takes a contiguous run of steps of 32
// slots (two groups of 16, each inside one page) for all G <= 16 heads of the group and the waves' partials are merged
// through LDS. Operands come straight from the pages, as in attn_decode_plain.hip:
//   S^T[16 slots x 16 heads] per group = Khat x Q'^T, three v_mfma_f32_16x16x32_bf16 per 32 dims
//   O  [16 heads x D]       += P x V, two per 16 dims of the output: the k index of the product runs over slots 4 kg ..
//        4 kg + 3 of the first and of the second group, which is what a lane's score registers hold.
// Rotation without a sine per key: q^.k^ = (R(pos_q - base) q).(R(pos_k - base) k). R(s), s in [0, 128), is a table in LDS
// (fp32); base is the position of some earlier group, moved - and Q' computed afresh - when a group starts outside
// [base, base + 112]: every fourth step along a run of consecutive positions, and wherever block positions jump (a step
// whose groups lie too far apart is taken in two turns). What bounds it is vector work, two thirds of its clocks, half
// of it on K (widen, rotate, split: six instructions per element); not the products.
//
// 64 requests of 4.3 K bf16 slots with valid masks and block positions, 32 heads on 8: 382 us (scalar) -> 110 us a call
// (146 before the loads got scalar bases and a fixed order, so that a step's waits leave the next step's loads in flight, and
// one round of workgroups); where no page is shared, 64 requests of 4 - 6 K slots, 249 us = 5.4 TB/s: HBM.
//
// A NaN or Inf in the merged result sends the workgroup through the scalar body: operand splits make NaN of some infinities, and
// probabilities of up to 2^kRescaleSlack times values near the largest float make Inf of finite ones.
#include <type_traits>

#include "attn_scalar.h"
#include "split_common.h"

namespace mepic {
namespace {

typedef float floatx4 __attribute__((ext_vector_type(4)));

constexpr int kWaves = 4, kThreads = 64 * kWaves;
constexpr int kTab = 128;             // slots the rotation table covers
constexpr float kRescaleSlack = 6.f;  // the reference maximum may lag the true one by this much (log2 units)

// Keep the elements whose bit of `keep` (4 bits) is set, zero the others.
__device__ __forceinline__ void mask4(uint2& x, uint32_t keep) {
  x.x &= (keep & 1u ? 0x0000ffffu : 0u) | (keep & 2u ? 0xffff0000u : 0u);
  x.y &= (keep & 4u ? 0x0000ffffu : 0u) | (keep & 8u ? 0xffff0000u : 0u);
}
__device__ __forceinline__ void mask4(uint32_t& x, uint32_t keep) {
#pragma unroll
  for (int e = 0; e < 4; ++e) x &= (keep >> e) & 1u ? ~0u : ~(0xffu << (8 * e));
}

template <int D>
struct Merge {
  float m[kWaves][16], l[kWaves][16], o[kWaves][16][D];
};
constexpr size_t table_bytes(int D) { return (size_t)D / 4 * kTab * sizeof(float4); }

template <bool kFp8, int D, int P, bool kIL>
__global__ __launch_bounds__(kThreads, 2) void decode_split_kernel(const AttnArgs a) {
  constexpr int kKs = D / 32;     // k-steps of 32 dims; granule of k-step j: dims 32 j + 8 kg ..
  constexpr int kNt = D / 16;     // output tiles of 16 dims
  typedef typename std::conditional<kFp8, uint32_t, uint2>::type Raw4;  // four stored elements of a V row
  typedef Merge<D> MergeT;
  static_assert(sizeof(MergeT) <= table_bytes(D) && sizeof(ScalarLds<4, kThreads>) <= table_bytes(D), "they share the table's LDS");
  extern __shared__ uint4 smem[];
  float4(*const tab)[kTab] = reinterpret_cast<float4(*)[kTab]>(smem);  // [frequencies 2 c, 2 c + 1][slot] {c0, s0, c1, s1}
  __shared__ uint4 q_lds[kKs][64];  // un-rotated q, granule j of every lane's head
  __shared__ __align__(16) float2 freq[D / 2];  // {hi, lo}: indexed per lane, which the kernel arguments are too slow for

  const int tid = threadIdx.x, lane = tid & 63, wave = uni_i(tid >> 6), n16 = lane & 15, kg = lane >> 4;
  if (tid < D / 2) freq[tid] = make_float2(a.freq_hi[tid], a.freq_lo[tid]);
  const int G = a.G, Hkv = a.Hkv;
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
    b = uni_i(b);
  }
  const int L = uni_i(a.kv_lens[b]), pos_q = uni_i(a.q_positions[t]);
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
  Win cur, nxt;
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
  Raw8<kFp8> kf[2][kKs];
  Raw4 vf[2][kNt];
  const uint32_t k_off = kFp8 ? (uint32_t)(((kg >> 1) * P + n16) * 16 + (kg & 1) * 8) : (uint32_t)((kg * P + n16) * 16);
  const uint32_t v_off = (uint32_t)((n16 * P + 4 * kg) * kElem);
  constexpr uint32_t kStepK = (kFp8 ? 2 : 4) * P * 16;        // bytes between a lane's granules of successive k-steps
  auto issue_k = [&](int pg0, int pg1) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      // steps start at multiples of 32: a page of 32 is a whole step
      const char* base = reinterpret_cast<const char*>(a.k_pages) + ((size_t)(u ? pg1 : pg0) * Hkv + hk) * kHeadBytes +
                         (P == 16 ? 0 : 16 * 16 * u);
#pragma unroll
      for (int j = 0; j < kKs; ++j) kf[u][j].r = *reinterpret_cast<const RawT*>(base + j * kStepK + k_off);
    }
  };
  auto issue_v = [&](int pg0, int pg1) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const char* base = reinterpret_cast<const char*>(a.v_pages) + ((size_t)(u ? pg1 : pg0) * Hkv + hk) * kHeadBytes +
                         (P == 16 ? 0 : 16 * kElem * u);
#pragma unroll
      for (int nt = 0; nt < kNt; ++nt) vf[u][nt] = *reinterpret_cast<const Raw4*>(base + nt * (16 * P * kElem) + v_off);
    }
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
  const bool row_ok = n16 < G;
  if (wave == 0) {
    const uint4* q4 = reinterpret_cast<const uint4*>(a.q) + ((size_t)t * a.Hq + (size_t)hk * G + (row_ok ? n16 : 0)) * (D / 8);
#pragma unroll
    for (int j = 0; j < kKs; ++j) q_lds[j][lane] = q4[4 * j + kg];
  }
  const float qs = row_ok ? a.qk_scale_log2 : 0.f;

  // ---- rotation table ----
  __syncthreads();
  for (int i = tid; i < D / 4 * kTab; i += kThreads) {
    const int c = i / kTab, s = i % kTab;
    const float t0 = turns_frac((float)s, freq[2 * c].x, freq[2 * c].y);
    const float t1 = turns_frac((float)s, freq[2 * c + 1].x, freq[2 * c + 1].y);
    tab[c][s] = make_float4(__builtin_amdgcn_cosf(t0), __builtin_amdgcn_sinf(t0), __builtin_amdgcn_cosf(t1),
                            __builtin_amdgcn_sinf(t1));
  }
  __syncthreads();

  // Rotary pairs of a lane: rotate-half: pairs (dims i, i + D/2) of granules h and h + kKs/2, i = 32 h + 8 kg + e;
  // interleaved: the four pairs inside each granule j, frequencies 16 j + 4 kg + e.
  SplitFrag qh[kKs], ql[kKs];
  auto rotate_q = [&](int base) __attribute__((always_inline)) {
    const float delta = (float)(pos_q - base);
    int again = 0;
    asm volatile("" : "+v"(again));  // q and the frequencies are fetched anew each time: they must not stay in registers
    auto rot = [&](float x0, float x1, int i, float& y0, float& y1) __attribute__((always_inline)) {
      const float2 f = freq[i + again];
      const float tr = turns_frac(delta, f.x, f.y);
      const float c = __builtin_amdgcn_cosf(tr), s = __builtin_amdgcn_sinf(tr);
      y0 = (x0 * c - x1 * s) * qs;
      y1 = (x1 * c + x0 * s) * qs;
    };
#pragma unroll
    for (int j = 0; j < (kIL ? kKs : kKs / 2); ++j) {
      SplitFrag qa, qb;
      qa.u = q_lds[j][lane + again];
      if constexpr (!kIL) qb.u = q_lds[j + kKs / 2][lane + again];
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        if constexpr (kIL) {
          float y0, y1;
          rot(__uint_as_float(qa.w[w] << 16), __uint_as_float(qa.w[w] & 0xffff0000u), 16 * j + 4 * kg + w, y0, y1);
          split2(y0, y1, qh[j].w[w], ql[j].w[w]);
        } else {
          const int i = 32 * j + 8 * kg + 2 * w, j1 = j + kKs / 2;
          float a0, b0, a1, b1;
          rot(__uint_as_float(qa.w[w] << 16), __uint_as_float(qb.w[w] << 16), i, a0, b0);
          rot(__uint_as_float(qa.w[w] & 0xffff0000u), __uint_as_float(qb.w[w] & 0xffff0000u), i + 1, a1, b1);
          split2(a0, a1, qh[j].w[w], ql[j].w[w]);
          split2(b0, b1, qh[j1].w[w], ql[j1].w[w]);
        }
      }
    }
  };
  // scores of group u (16 slots x 16 heads), its keys rotated by R(s), s = s0 + n16
  auto score = [&](int u, int s0) __attribute__((always_inline)) {
    floatx4 sc = {0.f, 0.f, 0.f, 0.f};
    const float4* tp = &tab[0][min(max(s0, 0), kTab - 16) + n16];
    auto three = [&](const SplitFrag& kh, const SplitFrag& kl, int j) __attribute__((always_inline)) {
      sc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kh.v, qh[j].v, sc, 0, 0, 0);
      sc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kh.v, ql[j].v, sc, 0, 0, 0);
      sc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kl.v, qh[j].v, sc, 0, 0, 0);
    };
#pragma unroll
    for (int j = 0; j < (kIL ? kKs : kKs / 2); ++j) {
      if constexpr (kIL) {
        float x[8];
        widen8<kFp8>(kf[u][j], x);
        SplitFrag h, l;
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
        SplitFrag h0, l0, h1, l1;
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
    return sc;
  };

  floatx4 o[kNt];
#pragma unroll
  for (int nt = 0; nt < kNt; ++nt) o[nt] = floatx4{0.f, 0.f, 0.f, 0.f};
  float m_run = -INFINITY, l_part = 0.f;
  int base = 0;
  bool have_base = false;
  auto inside = [&](int ps) __attribute__((always_inline)) {
    const long d = (long)ps - base;
    return d >= 0 && d <= kTab - 16;
  };

  // Softmax and output products of one turn; slots of the step outside vis0 / vis1 get no weight.
  auto attend = [&](floatx4 (&sc)[2], uint32_t vis0, uint32_t vis1, int l0) __attribute__((always_inline)) {
    float vs0 = 1.f, vs1 = 1.f;
    if constexpr (kFp8) {
      sc[0] *= __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(cur.ksc), l0));
      sc[1] *= __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(cur.ksc), l0 + 1));
      vs0 = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(cur.vsc), l0));
      vs1 = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(cur.vsc), l0 + 1));
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
    const float mx = fmaxf(fmaxf(fmaxf(sc[0][0], sc[0][1]), fmaxf(sc[0][2], sc[0][3])),
                           fmaxf(fmaxf(sc[1][0], sc[1][1]), fmaxf(sc[1][2], sc[1][3])));
    if (__any(mx > m_run + kRescaleSlack)) {
      const float m_new = fmaxf(m_run, max_over_kgroups(mx));
      const float alpha = (m_new == -INFINITY) ? 1.f : __builtin_amdgcn_exp2f(m_run - m_new);
      m_run = m_new;
      l_part *= alpha;
#pragma unroll
      for (int e = 0; e < 4; ++e) {  // accumulator rows of this lane are heads 4 kg + e; their factors live in lanes 4 kg + e
        const float ar = __shfl(alpha, 4 * kg + e);
#pragma unroll
        for (int nt = 0; nt < kNt; ++nt) o[nt][e] *= ar;
      }
    }
    const float m_use = (m_run == -INFINITY) ? 0.f : m_run;
    float pf[8];
    float psum = 0.f;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      pf[e] = __builtin_amdgcn_exp2f(sc[e >> 2][e & 3] - m_use);
      psum += pf[e];
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
      const uint32_t keep0 = (all0 >> (4 * kg)) & 0xfu, keep1 = (all1 >> (4 * kg)) & 0xfu;
#pragma unroll
      for (int nt = 0; nt < kNt; ++nt) {
        mask4(vf[0][nt], keep0);
        mask4(vf[1][nt], keep1);
      }
      if constexpr (kFp8) {
#pragma unroll
        for (int e = 0; e < 8; ++e)
          if (!(((e < 4 ? vis0 : vis1) >> (4 * kg + (e & 3))) & 1u)) pf[e] = 0.f;
      }
    }
    SplitFrag ph, pl;
#pragma unroll
    for (int w = 0; w < 4; ++w) split2(pf[2 * w], pf[2 * w + 1], ph.w[w], pl.w[w]);
#pragma unroll
    for (int nt = 0; nt < kNt; ++nt) {
      Raw8<kFp8> both;
      if constexpr (kFp8) both.r = make_uint2(vf[0][nt], vf[1][nt]);
      else both.r = make_uint4(vf[0][nt].x, vf[0][nt].y, vf[1][nt].x, vf[1][nt].y);
      const SplitFrag vb = bf16_of8<kFp8>(both);
      o[nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ph.v, vb.v, o[nt], 0, 0, 0);
      o[nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(pl.v, vb.v, o[nt], 0, 0, 0);
    }
  };

  // K of the next step is requested as soon as the scores are done with the registers, V after its products; always, so
  // that the waits can count the loads in flight (past the last step the last pages come once more).
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
      mg.m[wave][n16] = m_run;
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
    float m = mg.m[0][g];
#pragma unroll
    for (int w = 1; w < kWaves; ++w) m = fmaxf(m, mg.m[w][g]);
    float4 x = make_float4(0.f, 0.f, 0.f, 0.f);
    float l = 0.f;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
      const float f = mg.m[w][g] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(mg.m[w][g] - m);
      const float4 y = *reinterpret_cast<const float4*>(&mg.o[w][g][4 * dq]);
      x.x += f * y.x; x.y += f * y.y; x.z += f * y.z; x.w += f * y.w;
      l += f * mg.l[w][g];
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

template <bool kFp8, int D, int P, bool kIL>
hipError_t launch_one(const AttnArgs& a, hipStream_t s) {
  static std::atomic<uint64_t> asked{0};
  const hipError_t status = allow_lds(reinterpret_cast<const void*>(&decode_split_kernel<kFp8, D, P, kIL>), table_bytes(D), asked);
  if (status != hipSuccess) return status;
  // KV heads fastest (neighbours go to different dies, which then each keep their own heads' pages); tokens over x and y
  const unsigned per_row = (unsigned)min(a.n_q, max(65536 / a.Hkv, 1));
  const dim3 grid((unsigned)a.Hkv * per_row, ((unsigned)a.n_q + per_row - 1) / per_row, (unsigned)a.n_splits);
  hipLaunchKernelGGL((decode_split_kernel<kFp8, D, P, kIL>), grid, dim3(kThreads), table_bytes(D), s, a);
  return hipGetLastError();
}
template <bool kFp8, int D, int P>
hipError_t launch_il(const AttnArgs& a, hipStream_t s) {
  return a.interleaved ? launch_one<kFp8, D, P, true>(a, s) : launch_one<kFp8, D, P, false>(a, s);
}
template <bool kFp8>
hipError_t launch_kv(const AttnArgs& a, hipStream_t s) {
  if (a.D == 128) return a.P == 16 ? launch_il<kFp8, 128, 16>(a, s) : launch_il<kFp8, 128, 32>(a, s);
  return a.P == 16 ? launch_il<kFp8, 64, 16>(a, s) : launch_il<kFp8, 64, 32>(a, s);
}

}  // namespace

hipError_t launch_decode_split(const AttnArgs& a, hipStream_t s) {
  return a.kv_dtype == MEPIC_F8E4M3 ? launch_kv<true>(a, s) : launch_kv<false>(a, s);
}

}  // namespace mepic
