// General path of fused-RoPE paged attention (§3.3.3) for fp32 pages on the fp32 matrix instruction: decode and prefill, both
// rotary pairings, D 64 / 128, pages of 16 / 32 slots, block positions, valid masks. The arithmetic is fp32 throughout.
//
// One workgroup of 8 waves serves one (query token, KV head, split of the KV) for all G <= 16 heads of the group; a wave takes
// a contiguous run of groups of 16 slots (each inside one page), and the waves' partials are merged through LDS. Operands
// come straight from the pages: the 16-byte granules of the layouts are four k-steps of v_mfma_f32_16x16x4_f32 each,
//   S^T[16 slots x 16 heads] += Khat x Q'^T      step (j, e): dims 16 j + 4 kg + e of the lane's granule j
//   O  [16 heads x D]        += P x V            step e: slots 4 kg + e, which is what a lane's score registers hold.
// Keys are rotated with a table of slot rotations R(s), s in [0, 128), in LDS, queries by R(pos_q - base), as in
// attn_decode_split.hip (base moves when a group lies outside [base, base + 112]).
//
// Small calls are what fp32 pages are used for (bring-up, verification): the kernel is arranged for latency. K and V of the
// first groups are on their way while the table is built, eight waves share a split, and contexts too short for a
// second split need no merge kernel. 1 request of 289 slots, 8 heads of 64 dims: 17.4 us (scalar body) -> 8.9 us a call; 1 of
// 1 K slots, 32 heads on 8, 128 dims: 57 -> 14.3 us; 16 of 2.5 - 10 K private slots 153 -> 135 us (4.9 K in the mean). The error
// against 64 bits is a tenth of the scalar kernel's (2.4e-7 and 2.4e-6 on the first): shorter chains of sums, phases.
//
// A NaN or Inf in the merged result sends the workgroup through the scalar body (values near the largest float, times
// probabilities of up to 2^kRescaleSlack, make Inf of what plain arithmetic keeps finite).
#include "attn_scalar.h"
#include "split_common.h"

namespace mepic {
namespace {


constexpr int kWaves = 8, kThreads = 64 * kWaves;
constexpr int kTab = 128;             // slots the rotation table covers
constexpr float kRescaleSlack = 6.f;  // the reference maximum may lag the true one by this much (log2 units)

template <int D>
struct Merge {
  float m[kWaves][16], l[kWaves][16], o[kWaves][16][D];
};
constexpr size_t table_bytes(int D) { return (size_t)D / 4 * kTab * sizeof(float4); }
template <int D>
constexpr size_t lds_bytes() {
  return sizeof(Merge<D>) > table_bytes(D) ? sizeof(Merge<D>) : table_bytes(D);
}

// kTurns: the two waves of a SIMD share it by turns (take_turns).
template <int D, int P, bool kIL, bool kTurns>
__global__ __launch_bounds__(kThreads, 2) void decode_f32_kernel(const AttnArgs a) {
  constexpr int kGr = D / 16;  // granules (4 dims) of a K row a lane owns: j-th = dims 16 j + 4 kg ..
  constexpr int kNt = D / 16;  // output tiles of 16 dims
  static_assert(sizeof(ScalarLds<4, kThreads>) <= table_bytes(D), "they share the table's LDS");
  extern __shared__ uint4 smem[];
  float4(*const tab)[kTab] = reinterpret_cast<float4(*)[kTab]>(smem);  // [frequencies 2 c, 2 c + 1][slot] {c0, s0, c1, s1}
  __shared__ float4 q_lds[kGr][64];             // un-rotated q, granule j of every lane's head
  __shared__ __align__(16) float2 freq[D / 2];  // {hi, lo}: indexed per lane, which the kernel arguments are too slow for

  const int tid = threadIdx.x, lane = tid & 63, wave = uni(tid >> 6), n16 = lane & 15, kg = lane >> 4;
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
    b = uni(b);
  }
  const int L = uni(a.kv_lens[b]), pos_q = uni(a.q_positions[t]);
  const int n_begin = split * a.blocks_per_split * P;
  const int s_end = min(L, (split + 1) * a.blocks_per_split * P);
  int n_end = s_end;
  if (a.causal && !a.block_positions) n_end = min(n_end, max(pos_q, -1) + 1);

  // ---- this wave's groups of 16 slots: lane i of a window holds group i of 64 ----
  const int n_groups = n_end > n_begin ? (n_end - n_begin + 15) / 16 : 0;
  const int per_wave = (n_groups + kWaves - 1) / kWaves;
  const int g_first = wave * per_wave, n_st = max(min(per_wave, n_groups - g_first), 0);
  struct Win {
    int page, pos;
    uint32_t vis;
  };
  const size_t bt_row = (size_t)b * a.max_blocks;
  auto win_load = [&](Win& w, int win) __attribute__((always_inline)) {
    const int n = n_begin + 16 * (g_first + 64 * win + lane);  // first slot of the group
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
  };
  Win cur, nxt;
  int win = 0;
  if (n_st > 0) {
    win_load(cur, 0);
    nxt = cur;
    if (n_st > 64) win_load(nxt, 1);
  }

  // ---- K and V of a group. K row n16 is slot n16. Scalar base, 32-bit lane offset, immediate. ----
  constexpr size_t kHeadBytes = (size_t)D * P * 4;
  float4 kf[kGr], vf[kNt];
  const uint32_t k_off = (uint32_t)((kg * P + n16) * 16), v_off = (uint32_t)((n16 * P + 4 * kg) * 4);
  auto place = [&](int pg) __attribute__((always_inline)) {
    return ((size_t)pg * Hkv + hk) * kHeadBytes;
  };
  auto half = [&](int st) __attribute__((always_inline)) { return P == 16 ? 0 : ((n_begin / 16 + g_first + st) & 1) * 16; };
  auto issue_k = [&](int pg, int st) __attribute__((always_inline)) {
    const char* base = reinterpret_cast<const char*>(a.k_pages) + place(pg) + half(st) * 16;
#pragma unroll
    for (int j = 0; j < kGr; ++j) kf[j] = *reinterpret_cast<const float4*>(base + j * (4 * P * 16) + k_off);
  };
  auto issue_v = [&](int pg, int st) __attribute__((always_inline)) {
    const char* base = reinterpret_cast<const char*>(a.v_pages) + place(pg) + half(st) * 4;
#pragma unroll
    for (int nt = 0; nt < kNt; ++nt) vf[nt] = *reinterpret_cast<const float4*>(base + nt * (16 * P * 4) + v_off);
  };
  int np = 0;  // page of the next group
  if (n_st > 0) {
    np = __builtin_amdgcn_readlane(cur.page, 0);
    issue_k(np, 0);
    __builtin_amdgcn_sched_barrier(0);  // K before V on every path: the loop's waits count on it
    issue_v(np, 0);
    __builtin_amdgcn_sched_barrier(0);
  }

  // ---- q of this lane's head, un-rotated ----
  const bool row_ok = n16 < G;
  if (wave == kWaves - 1) {
    const float4* q4 = reinterpret_cast<const float4*>(a.q) + ((size_t)t * a.Hq + (size_t)hk * G + (row_ok ? n16 : 0)) * (D / 4);
#pragma unroll
    for (int j = 0; j < kGr; ++j) q_lds[j][lane] = q4[4 * j + kg];
  }
  const float qs = row_ok ? a.qk_scale_log2 : 0.f;

  // ---- rotation table, as far as a wave's run of slots can need it ----
  // (to a power of two: 1 request of 289 slots 9.1 -> 8.9 us, 3 of 1.3 K, 12 heads of 64, 12.1 -> 11.7, against as many slots in a loop over all)
  const int tab_bits = min(7, 4 + (per_wave > 1 ? 32 - __builtin_clz(per_wave - 1) : 0)), n_tab = 1 << tab_bits;
  static_assert(kTab == 1 << 7, "");
  __syncthreads();
  auto entry = [&](int c, int s) __attribute__((always_inline)) {
    const float t0 = turns_frac((float)s, freq[2 * c].x, freq[2 * c].y);
    const float t1 = turns_frac((float)s, freq[2 * c + 1].x, freq[2 * c + 1].y);
    tab[c][s] = make_float4(__builtin_amdgcn_cosf(t0), __builtin_amdgcn_sinf(t0), __builtin_amdgcn_cosf(t1),
                            __builtin_amdgcn_sinf(t1));
  };
  if (n_tab == kTab) {  // (a number of turns that the compiler knows)
    for (int i = tid; i < D / 4 * kTab; i += kThreads) entry(i / kTab, i % kTab);
  } else {
    for (int i = tid; i < D / 4 << tab_bits; i += kThreads) entry(i >> tab_bits, i & (n_tab - 1));
  }
  __syncthreads();

  // Rotary pairs of a lane: rotate-half: element e of granules j and j + kGr/2, frequency 16 j + 4 kg + e;
  // interleaved: the two pairs inside each granule j, frequencies 8 j + 2 kg and the next.
  float q[kGr][4];
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
    for (int j = 0; j < (kIL ? kGr : kGr / 2); ++j) {
      const float4 x = q_lds[j][lane + again];
      if constexpr (kIL) {
        rot(x.x, x.y, 8 * j + 2 * kg, q[j][0], q[j][1]);
        rot(x.z, x.w, 8 * j + 2 * kg + 1, q[j][2], q[j][3]);
      } else {
        const int j1 = j + kGr / 2, i = 16 * j + 4 * kg;
        const float4 y = q_lds[j1][lane + again];
        rot(x.x, y.x, i, q[j][0], q[j1][0]);
        rot(x.y, y.y, i + 1, q[j][1], q[j1][1]);
        rot(x.z, y.z, i + 2, q[j][2], q[j1][2]);
        rot(x.w, y.w, i + 3, q[j][3], q[j1][3]);
      }
    }
  };
  auto score = [&](int s0) __attribute__((always_inline)) {  // 16 slots x 16 heads, keys rotated by R(s0 + n16)
    floatx4 sa = {0.f, 0.f, 0.f, 0.f}, sb = {0.f, 0.f, 0.f, 0.f};  // two chains: the products depend on each other
    const float4* tp = &tab[0][min(max(s0, 0), n_tab - 16) + n16];
    auto four = [&](floatx4& s, const float (&k)[4], int j) __attribute__((always_inline)) {
#pragma unroll
      for (int e = 0; e < 4; ++e) s = __builtin_amdgcn_mfma_f32_16x16x4f32(k[e], q[j][e], s, 0, 0, 0);
    };
#pragma unroll
    for (int j = 0; j < (kIL ? kGr : kGr / 2); ++j) {
      const float4 x = kf[j];
      if constexpr (kIL) {
        const float4 r = tp[(4 * j + kg) * kTab];
        const float k[4] = {x.x * r.x - x.y * r.y, x.y * r.x + x.x * r.y, x.z * r.z - x.w * r.w, x.w * r.z + x.z * r.w};
        four(j & 1 ? sb : sa, k, j);
      } else {
        const float4 y = kf[j + kGr / 2];
        const float4 r0 = tp[(8 * j + 2 * kg) * kTab], r1 = tp[(8 * j + 2 * kg + 1) * kTab];
        const float k0[4] = {x.x * r0.x - y.x * r0.y, x.y * r0.z - y.y * r0.w, x.z * r1.x - y.z * r1.y, x.w * r1.z - y.w * r1.w};
        const float k1[4] = {y.x * r0.x + x.x * r0.y, y.y * r0.z + x.y * r0.w, y.z * r1.x + x.z * r1.y, y.w * r1.z + x.w * r1.w};
        four(sa, k0, j);
        four(sb, k1, j + kGr / 2);
      }
    }
    return sa + sb;
  };

  floatx4 o[kNt];
#pragma unroll
  for (int nt = 0; nt < kNt; ++nt) o[nt] = floatx4{0.f, 0.f, 0.f, 0.f};
  float m_run = -INFINITY, l_part = 0.f;
  int base = 0;
  bool have_base = false;

  // K of the next group is requested as soon as the scores are done with the registers, V after its products; always, so
  // that the waits can count the loads in flight (past the last group the last page comes once more).
  for (int st = 0; st < n_st; ++st) {
    if constexpr (kTurns) take_turns(wave >= kWaves / 2, st);
    const int l0 = st & 63;
    if (st > 0 && l0 == 0) {
      cur = nxt;
      ++win;
      if (n_st > 64 * (win + 1)) win_load(nxt, win + 1);
    }
    if (st + 1 < n_st) np = __builtin_amdgcn_readlane(l0 == 63 ? nxt.page : cur.page, (l0 + 1) & 63);
    const int ps = __builtin_amdgcn_readlane(cur.pos, l0);
    const uint32_t vis = (uint32_t)__builtin_amdgcn_readlane((int)cur.vis, l0);
    const long ahead = (long)ps - base;
    if (!have_base || (vis && (ahead < 0 || ahead > n_tab - 16))) {
      base = ps;
      have_base = true;
      rotate_q(base);
    }
    floatx4 sc = score(ps - base);
    __builtin_amdgcn_sched_barrier(0);
    issue_k(np, min(st + 1, n_st - 1));
    __builtin_amdgcn_sched_barrier(0);
    if (vis != 0xffffu) {  // slots that take no part may hold anything, NaN included
      asm volatile("");  // a branch, not selects in every step
      const uint32_t mine = vis >> (4 * kg);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const bool keep = (mine >> e) & 1u;
        if (!keep) sc[e] = -INFINITY;
#pragma unroll
        for (int nt = 0; nt < kNt; ++nt) {
          float& v = e == 0 ? vf[nt].x : e == 1 ? vf[nt].y : e == 2 ? vf[nt].z : vf[nt].w;
          v = keep ? v : 0.f;
        }
      }
    }
    const float mx = fmaxf(fmaxf(sc[0], sc[1]), fmaxf(sc[2], sc[3]));
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
    float p[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) p[e] = __builtin_amdgcn_exp2f(sc[e] - m_use);
    l_part += (p[0] + p[1]) + (p[2] + p[3]);
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
      for (int nt = 0; nt < kNt; ++nt)
        o[nt] = __builtin_amdgcn_mfma_f32_16x16x4f32(p[e], e == 0 ? vf[nt].x : e == 1 ? vf[nt].y : e == 2 ? vf[nt].z : vf[nt].w,
                                                     o[nt], 0, 0, 0);
    __builtin_amdgcn_sched_barrier(0);
    issue_v(np, min(st + 1, n_st - 1));
    __builtin_amdgcn_sched_barrier(0);
  }

  // ---- merge the waves (the table's LDS is free now), write the split's partial or, if it is the only one, the rows ----
  __syncthreads();
  Merge<D>& mg = *reinterpret_cast<Merge<D>*>(smem);
  {
    const float l_tot = sum_over_kgroups(l_part);
    if (kg == 0) {
      mg.m[wave][n16] = m_run;
      mg.l[wave][n16] = l_tot;
    }
#pragma unroll
    for (int nt = 0; nt < kNt; ++nt)
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (4 * kg + e < G) mg.o[wave][4 * kg + e][16 * nt + n16] = o[nt][e];
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
      const bool some = l != 0.f;
      reinterpret_cast<float4*>(a.out)[row * (D / 4) + dq] =
          make_float4(some ? x.x / l : 0.f, some ? x.y / l : 0.f, some ? x.z / l : 0.f, some ? x.w / l : 0.f);
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
    scalar_attend_all<MEPIC_F32, kThreads>(a, *reinterpret_cast<ScalarLds<4, kThreads>*>(smem), t, b, hk, 0, G, n_begin, s_end,
                                           split, direct);
}

template <int D, int P, bool kIL, bool kTurns = false>
hipError_t launch_one(const AttnArgs& a, hipStream_t s) {
  // Turns pay where waves have many groups; with few, what they add to the loop is more than they give. us a call without and with them, by
  // groups of 16 slots a wave (of the bound on lengths): 4 requests of 32 K slots, 8 KV heads (32) 197.4 and 188.9, 16 of 2.5 - 10 K (38) 136.9
  // and 134.5, prefill of 792 tokens, 12 KV heads (30) 2663 and 2645; 4 of 16 K (16) 98.5 and 97.2, but 16 of 4 K (16) 96.2 and 97.4, 14 of 6 K
  // (24) 172.8 and 174.7, 16 of 2 K (8) 53.5 and 54.2, 4 of 2 K (2) 18.65 and 18.9. Of those with more than 28 one lost: 8 of up to 16 K on 12 heads
  // (44, 288 workgroups) 143.2 and 146.5.
  if constexpr (D == 128 && !kTurns)
    if (a.blocks_per_split * P >= 28 * 16 * kWaves) return launch_one<D, P, kIL, true>(a, s);
  static std::atomic<uint64_t> asked{0};
  const hipError_t status = allow_lds(reinterpret_cast<const void*>(&decode_f32_kernel<D, P, kIL, kTurns>), lds_bytes<D>(), asked);
  if (status != hipSuccess) return status;
  // KV heads fastest (neighbours go to different dies, which then each keep their own heads' pages); tokens over x and y
  const unsigned per_row = (unsigned)min(a.n_q, max(65536 / a.Hkv, 1));
  const dim3 grid((unsigned)a.Hkv * per_row, ((unsigned)a.n_q + per_row - 1) / per_row, (unsigned)a.n_splits);
  hipLaunchKernelGGL((decode_f32_kernel<D, P, kIL, kTurns>), grid, dim3(kThreads), lds_bytes<D>(), s, a);
  return hipGetLastError();
}
template <int D, int P>
hipError_t launch_il(const AttnArgs& a, hipStream_t s) {
  return a.interleaved ? launch_one<D, P, true>(a, s) : launch_one<D, P, false>(a, s);
}

}  // namespace

hipError_t launch_decode_f32(const AttnArgs& a, hipStream_t s) {
  if (a.D == 128) return a.P == 16 ? launch_il<128, 16>(a, s) : launch_il<128, 32>(a, s);
  return a.P == 16 ? launch_il<64, 16>(a, s) : launch_il<64, 32>(a, s);
}

}  // namespace mepic
