// Plain decode of fused-RoPE paged attention (§3.3.3) on matrix cores, every request for itself. D = 128:
//   bf16 K/V pages of 16 slots (a step of 32 slots = two pages), and
//   fp8 e4m3 K/V pages of 32 slots with one fp32 scale per page for K and for V (a step = one page).
//
// Persistent waves, stream-K over pages. The grid is one workgroup of eight waves (two a SIMD) per compute unit; workgroup g serves KV
// head g % Hkv (consecutive workgroups land on consecutive XCDs, so one KV head's pages stay in one XCD's L2). For one KV head
// the steps of all requests form one sequence of length T; the waves of that head cut it into equal contiguous chunks, at
// request boundaries where that comes out even enough (up to 64 requests), regardless of them otherwise. A wave writes one partial (max, sum,
// un-normalised output) per request it touched; a second kernel merges the partials of each (request, head). Consecutive chunks
// go to different workgroups: a call too small for all waves is spread over all compute units (6 requests of up to 430 bf16 slots 10.6
// -> 9.2 us), and the streams that a compute unit reads lie far apart (8 requests of 65 537 slots 332 -> 320 us).
//
// Everything a step needs comes straight from the pages into registers as 16-byte loads that (nearly) are matrix operands:
//
//   S^T[32 slots x 16 rows] = Khat[32 x 128] * Q'^T[128 x 16]     v_mfma_f32_16x16x32_bf16 (fp8: _f16)
//   O  [16 rows x 128]     += P[16 x 32 slots] * V[32 x 128]      v_mfma_f32_16x16x32_bf16 (fp8: _fp8_fp8)
//
// A K load covers sixteen consecutive slots (whole lines); a lane then has the scores of four slots of either product. One
// lane-swap instruction a register (neighbouring k-groups) turns their probabilities into those of eight consecutive slots,
// which is what a 16-byte piece of a bf16 V row is. fp8 V rows come in 16-byte pieces of 16 slots - half the load instructions of
// 8-byte pieces - and a lane swap makes the operands of two column tiles of each.
//
// Rotation without per-key trigonometry. A key at position n0 + s (n0: where Q' stands) has q^.k^ = (R(pos_q - n0) q) . (R(s) k).
// R(s) is a per-lane constant read from LDS (a lane always handles the same slot offsets and 16 frequencies), kept for the 32 kNV
// slots (64 kNV for two steps a turn) between two advances of Q' by a constant rotation.
// * bf16 keys are rotated by two-term dot products (v_dot2_f32_bf16) on words that v_perm_b32 assembles from the pair's two
//   granules; fp8 codes are widened to packed fp16 (exact) and rotated in packed fp16 arithmetic, two pairs an instruction.
// * bf16, idle matrix rows instead of rotations. A group of G <= 8 query heads uses G of 16 rows. The slow half of the pairs (frequencies
//   32 .. 63) turns by x t, |x| <= 0.1 (0.35), about the middle of that span, t in [-1, 1], and e^(-i x t) = J0(x) - 2 i J1(x) T1(t) -
//   2 J2(x) T2(t) + ... (Jacobi-Anger): with a row for each of two (three) terms, Q' times the term's coefficient, their keys
//   go into the products as they are, and the scores of a head are the sum of its rows' weighted by T_m(t) of the slot: one multiply-add a
//   score and term. 292 -> 183 vector instructions a step (start-up and run ends counted in), and these keys lose no bits to a rotation.
//   Infinite keys, and scores past the largest float, have no such series (0 x Inf, Inf - Inf between the terms): a run that met any
//   is computed again by plain_run.
// * fp8, two steps a turn. With G <= 8 rows 0-7 belong to the turn's first step and 8-15 to its second, Q' of the latter standing 32
//   slots on: both use the same constants, and softmax, the split of the probabilities and their scaling happen once for both.
//   260 -> 205 vector instructions a step. Either half of the rows keeps a reference maximum and a reference V scale of its own, as two
//   waves would, and they are brought together at the run's end.
// fp8: the page's K scale multiplies the scores. V is never widened: PV takes the bytes as loaded and the probabilities split
// into two e4m3 terms (p*16 = hi + lo, 8 significant bits together down to p = 2^-7); the page's V scale rides on the probabilities, O
// being kept in units of a reference scale that is raised (with a rescale of O) only when a page's scale exceeds it by 1.75 x.
//
// What bounds it. Where pages are read once, HBM: 8 requests of 65 537 bf16 slots with the read-once hint 315 us = 6.8 TB/s (320 before a
// SIMD's waves took turns, 332 with two requests' worth of waves side by side on a unit). Where requests share pages, what misses L2: 64
// requests of 4.3 K slots ask L1 for 1.13 GB (33 us at a line a two clocks on every unit), of which 0.36 GB miss L2, and those come at 6 - 7
// TB/s whether from HBM or the Infinity Cache: 81.5 -> 69 us a call (47 with every page in L2); 128 requests of 2 - 33 K fp8 slots 212 ->
// 172 - 182 us from card to card. Measured and of no use there: requesting two or
// three steps ahead by touching a word of every line (the lines are gone from the 32 KB of L1 again: 102 - 112 us), the
// non-temporal hint for pages of few readers (misses 0.36 -> 0.30 GB, but those then always come from HBM: 78 - 94 us).
#include "decode_common.h"
#include "merge_partials.h"

namespace mepic {
namespace {

constexpr int kD = 128;
constexpr int kWaves = 8;
// A lane's probabilities of a step (so at most that each) above which the reference maximum is raised. fp8: what e4m3 has room for,
// 448, is their largest times the factor that they are split with and 1.75. A larger factor under a smaller sum puts the
// split's absolute step (2^-10) lower beside probabilities of 1: error of 128 requests of 2 - 33 K slots against 64 bits, 4 under 64
// 1.78e-3, 8 under 32 1.75e-3, 16 under 16 1.745e-3 (the result's own rounding 1.66e-3), all at the same time a call.
__host__ __device__ constexpr float most_sum(bool fp8) { return fp8 ? 16.f : 64.f; }
constexpr float kPScale = 256.f / most_sum(true);

// Inclusive prefix sum over the wave.
__device__ __forceinline__ int wave_scan(int x) {
  x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, true);  // row_shr:1, 2, 4, 8
  x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, true);
  x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, true);
  x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, true);
  x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false);  // row_bcast:15 into rows 1 and 3
  x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false);  // row_bcast:31 into rows 2 and 3
  return x;
}

// Slot-rotation tables: step j of a run uses table j mod n, Q' advances every n steps.
constexpr int n_tables(bool fp8, int terms) { return fp8 || terms == 2 ? 4 : 2; }

// A run of a bf16 request - slots [n_begin, n_end) below its length, n_begin a multiple of 32 - for KV head hk by plain arithmetic, one
// wave: every key rotated at its own position. A run that met a score without a finite value is computed again by it, at the end of a
// wave's work and in few instructions: a second way through the walker's loop cost calls of few requests 0.7 - 2 us by its length alone.
__device__ __forceinline__ void plain_run(const AttnArgs& a, const float2* freq, int b, int hk, int n_begin, int n_end, size_t row0) {
  const int lane = threadIdx.x & 63;
  const uint16_t* const q = reinterpret_cast<const uint16_t*>(a.q);
  const uint4* const k4 = reinterpret_cast<const uint4*>(a.k_pages);
  const uint4* const v4 = reinterpret_cast<const uint4*>(a.v_pages);
  auto turns = [&](int pos, int i) {  // of pair i
    const float2 f = freq[((i >> 3) & 3) * 16 + (i >> 5) * 8 + (i & 7)];
    return turns_frac((float)pos, f.x, f.y);
  };
  auto element = [](const Frag& x, int e) { return __uint_as_float(e & 1 ? x.w[e >> 1] & 0xffff0000u : x.w[e >> 1] << 16); };
  auto of_lane = [](float x, int i) { return __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(x), i)); };
#pragma unroll 1
  for (int g = 0; g < a.G; ++g) {
    const size_t q_row = ((size_t)b * a.Hq + (size_t)hk * a.G + g) * kD + lane;
    const float x0 = bf16_bits_to_f32(q[q_row]) * a.qk_scale_log2, x1 = bf16_bits_to_f32(q[q_row + 64]) * a.qk_scale_log2;
    const float tq = turns(a.q_positions[b], lane), cq = __builtin_amdgcn_cosf(tq), sq = __builtin_amdgcn_sinf(tq);
    const float q0 = x0 * cq - x1 * sq, q1 = x1 * cq + x0 * sq;  // of pair `lane`
    float m = -INFINITY, l = 0.f, o0 = 0.f, o1 = 0.f;            // o: of dims lane and lane + 64
#pragma unroll 1
    for (int n0 = n_begin; n0 < n_end; n0 += 64) {
      const int n = n0 + lane, last = min(n, n_end - 1);
      const int page = safe_page(a.block_tables[(size_t)b * a.max_blocks + last / 16], a.num_pages);
      const size_t key = ((size_t)page * a.Hkv + hk) * (2 * kD) + last % 16;
      float sc = 0.f;
#pragma unroll 1
      for (int j = 0; j < 8; ++j) {  // pairs 8 j ..
        Frag lo, hi;
        lo.u = k4[key + 16 * j];
        hi.u = k4[key + 16 * (8 + j)];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const float t = turns(n, 8 * j + e), c = __builtin_amdgcn_cosf(t), sn = __builtin_amdgcn_sinf(t);
          const float y0 = element(lo, e), y1 = element(hi, e);
          sc += (y0 * c - y1 * sn) * of_lane(q0, 8 * j + e);
          sc += (y1 * c + y0 * sn) * of_lane(q1, 8 * j + e);
        }
      }
      if (n >= n_end) sc = -INFINITY;
      const float most = fmaxf(m, wave_reduce(sc, [](float x, float y) { return fmaxf(x, y); }));
      const float alpha = most == -INFINITY ? 1.f : __builtin_amdgcn_exp2f(m - most);
      const float p = __builtin_amdgcn_exp2f(sc - (most == -INFINITY ? 0.f : most));
      m = most;
      l = l * alpha + wave_reduce(p, [](float x, float y) { return x + y; });
      o0 *= alpha;
      o1 *= alpha;
#pragma unroll 1
      for (int i = 0; i < min(64, n_end - n0); i += 8) {  // eight slots of one page
        const size_t value = ((size_t)(uint32_t)__builtin_amdgcn_readlane(page, i) * a.Hkv + hk) * (2 * kD) + 2 * lane + (i >> 3 & 1);
        Frag lo, hi;
        lo.u = v4[value];
        hi.u = v4[value + 128];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const bool in = n0 + i + e < n_end;  // (slots past the end may hold anything)
          const float w = of_lane(p, i + e);
          o0 += w * (in ? element(lo, e) : 0.f);
          o1 += w * (in ? element(hi, e) : 0.f);
        }
      }
    }
    const size_t part = row0 + (size_t)g * a.n_splits;
    if (lane == 0) {
      a.part_ml[part * 2] = l == 0.f ? -INFINITY : m;
      a.part_ml[part * 2 + 1] = l;
    }
    a.part_o[part * kD + lane] = o0;
    a.part_o[part * kD + lane + 64] = o1;
  }
}

// kTerms: matrix rows a head has in the products with the slow half of the pairs (1: all pairs are rotated). kPack: steps a turn
// of the loop takes together, each with matrix rows of its own for every head. kFull: with terms, every matrix row belongs to a head (as a
// branch in the loop this cost a decode step's call of 16 requests 0.15 us, whether taken or not).
template <bool kFp8, int kTerms, int kPack, bool kFull, bool kReadOnce>
__global__ __launch_bounds__(64 * kWaves, 2) void decode_plain_kernel(const AttnArgs a) {
  static_assert(kFp8 ? kTerms == 1 : kPack == 1, "bf16 uses idle rows for terms, e4m3 for steps");
  static_assert(!kFull || kTerms == 2, "eight heads of two rows; three rows a head leave one over");
  constexpr int kP = kFp8 ? 32 : 16;          // slots per page
  constexpr int kBps = kFp8 ? 1 : 2;          // pages per step of 32 slots
  constexpr int kNK = kFp8 ? 2 : 4;           // 16-byte K fragments per lane and product
  constexpr int kNVec = kFp8 ? 4 : 8;         // 16-byte V fragments per lane
  constexpr int kNV = n_tables(kFp8, kTerms);
  constexpr int kRot = kTerms == 1 ? 2 : 1;   // halves of a lane's pairs whose keys are rotated
  constexpr int kRotK = kNV * 2 * kRot * 4;
  constexpr int kTurn = 32 * kPack;           // slots a turn
  constexpr float kCentre = 16.f * kNV - 0.5f;  // middle of the 32 kNV slots between two advances, and half their span
  constexpr uint32_t kHeadBytes = kD * kP * (kFp8 ? 1 : 2);  // one KV head of a page, K or V alike
  typedef typename std::conditional<kFp8, float2, float4>::type RotK;
  __shared__ RotK rotK[kRotK][64];     // index ((table * 2 + product) * kRot + half) * 4 + w, pairs 2 w and 2 w + 1 of the half
  __shared__ float4 rotS[8][64];       // R(-kTurn kNV), index half * 4 + w
  __shared__ float2 freq_lds[64];      // {hi, lo}, index kg * 16 + pair (per-lane reads of the kernel arguments are slow)
  __shared__ float2 coef[kTerms][64];  // term m of Q' is coef.x Q' - i coef.y Q', index [m][kg * 16 + pair]
  __shared__ float4 weight[kTerms > 1 ? kTerms - 1 : 1][kNV][2][4];  // T_{m + 1} at the slots of [table][product][kg]
  extern __shared__ int cum[];         // more than 64 requests: steps of the requests before b; B + 1 entries

  const int tid = threadIdx.x, lane = tid & 63, wave = uni(tid >> 6), n16 = lane & 15, kg = lane >> 4;
  const int G = a.G, Hkv = a.Hkv;
  // of this lane's matrix row: which step of the turn, which head, which term
  const int part = kPack == 2 ? n16 >> 3 : 0, head = (kPack == 2 ? n16 & 7 : n16) / kTerms, term = n16 % kTerms;
  const bool row_ok = term == 0 && head < G;

  // ---- steps of every request. Up to 64 requests: each wave scans the lengths itself and keeps them in its lanes (lane b:
  // request b's length and the steps up to its end), so that its first page ids are on their way before the tables are built. ----
  const bool in_lanes = a.B <= 64;
  int len_lane = 0, cum_lane = 0;
  auto steps_of = [](int len) { return ((len + kP - 1) / kP + kBps - 1) / kBps; };
  if (in_lanes) {
    len_lane = lane < a.B ? a.kv_lens[lane] : 0;
    cum_lane = wave_scan(steps_of(len_lane));
  } else if (wave == 0) {
    int carry = 0;
    for (int base = 0; base < a.B; base += 64) {
      const int b = base + lane;
      const int x = wave_scan(b < a.B ? steps_of(a.kv_lens[b]) : 0);
      if (b < a.B) cum[b + 1] = carry + x;
      carry += __builtin_amdgcn_readlane(x, 63);
    }
    if (lane == 0) cum[0] = 0;
  }
  auto cum_at = [&](int i) __attribute__((always_inline)) {  // i wave-uniform
    if (in_lanes) return i == 0 ? 0 : __builtin_amdgcn_readlane(cum_lane, i - 1);
    return uni(cum[i]);
  };

  // ---- frequencies of a lane's 16 rotary pairs p = 8 h + e: i(p) = 32 h + 8 kg + e for bf16 (dims i and i + 64 sit in k-steps
  // h and h + 2), 16 kg + p for fp8; and what the terms are made of ----
  if (wave == kWaves - 1) {
    const int i = kFp8 ? lane : 32 * (n16 >> 3) + 8 * kg + (n16 & 7);  // lane (kg, n16) fills entry kg * 16 + n16
    const float hi = a.freq_hi[i];
    freq_lds[lane] = make_float2(hi, a.freq_lo[i]);
    if constexpr (kTerms > 1) {
      const bool low = n16 >= 8;  // the rotated half has the one term that it always had
      const float x = low ? kCentre * 6.283185307f * hi : 0.f, y = 0.25f * x * x;  // y = (x / 2)^2
      coef[0][lane] = make_float2(1.f - y + 0.25f * y * y, 0.f);                                    // J0(x)
      coef[1][lane] = make_float2(0.f, x * (1.f - 0.5f * y));                                       // 2 J1(x)
      if constexpr (kTerms > 2) coef[2][lane] = make_float2(-y * (1.f - y * (1.f / 3.f)), 0.f);     // -2 J2(x)
    }
  }
  if constexpr (kTerms > 1) {
    if (wave == kWaves - 2 && lane < kNV * 8) {
      const int k = lane & 3, u = (lane >> 2) & 1, v = lane >> 3;
      float t[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) t[e] = ((float)(32 * v + 16 * u + 4 * k + e) - kCentre) * (1.f / kCentre);
      weight[0][v][u][k] = make_float4(t[0], t[1], t[2], t[3]);
      if constexpr (kTerms > 2)
        weight[1][v][u][k] = make_float4(2.f * t[0] * t[0] - 1.f, 2.f * t[1] * t[1] - 1.f, 2.f * t[2] * t[2] - 1.f,
                                         2.f * t[3] * t[3] - 1.f);
    }
  }

  const int hk = (int)blockIdx.x % Hkv;
  // (waves of one workgroup take parts far from each other: a call too small for all waves still uses all compute units)
  const int n_wg = (int)gridDim.x / Hkv, wk = wave * n_wg + (int)blockIdx.x / Hkv, n_k = n_wg * kWaves;
  int chunk = 0, pos_begin = 0, pos_end = 0;
  int most_steps = 0;          // of a wave's run, in the whole call
  bool whole = false;          // every wave has one run: requests are cut into pieces of their own
  int upto = 0, piece = 0;     // whole: lane b: pieces of the requests up to b; the wave's piece of its request
  auto cut = [&]() __attribute__((always_inline)) {  // this wave's part of the sequence
    const int T = cum_at(a.B);
    // (blocks_per_split carries the minimum chunk, of lengths up to what the caller calls their bound; past T it makes no difference)
    chunk = uni(max(max((T + n_k - 1) / n_k, min(a.blocks_per_split, T)), 1));
    // Where a wave's part runs from one request into the next, it pays for a second start (page ids, Q') and a second partial:
    // some 2 - 3 us. So requests are cut into equal pieces of their own, one a wave, if there are waves enough for pieces at most a step (turn)
    // and a sixteenth longer than parts of the sequence would be. us a call without and with: 60 requests of up to 407 e4m3 slots 18.6 -> 15.8, 19
    // of up to 4 K 25.2 -> 20.8; 64 of 4.3 K bf16 74.5 -> 71.2, 56 of up to 2.9 K 43.5 -> 41.3; the worst of fifty mixes lost 3 %.
    if (in_lanes && a.B > 1 && chunk + kPack > 2 && T < 1 << 20) {
      const int steps = steps_of(len_lane);
      auto pieces_of = [](int n, int c) __attribute__((always_inline)) {  // n / c rounded up (exact: n <= T < 2^20, c < 1.1 T)
        return (int)(((float)(n + c) - 0.5f) * __builtin_amdgcn_rcpf((float)c));
      };
      const int c0 = (chunk + kPack - 1) / kPack * kPack, by = kPack * (1 + chunk / 64), most = c0 + kPack + chunk / 16;
      int c = c0, pieces = 0;
      for (; c <= most; c += by) {
        pieces = pieces_of(steps, c);
        upto = wave_scan(pieces);
        whole = __builtin_amdgcn_readlane(upto, 63) <= n_k;
        if (whole) break;
      }
      if (whole) {
        most_steps = uni(c);
        const int b = (int)__popcll(__ballot(upto <= wk));
        if (b < a.B) {
          const int k = __builtin_amdgcn_readlane(pieces, b), n = __builtin_amdgcn_readlane(steps, b);
          piece = wk - (__builtin_amdgcn_readlane(upto, b) - k);
          const int len = uni((pieces_of(n, k) + kPack - 1) / kPack * kPack);  // as even as whole turns allow
          const int first = cum_at(b);
          pos_begin = first + min(piece * len, n);
          pos_end = first + min(piece * len + len, n);
        }
      }
    }
    if (!whole) {
      most_steps = chunk;
      pos_begin = wk * chunk;
      pos_end = min(pos_begin + chunk, T);
    }
    if (blockIdx.x == 0 && wave == 0) {  // what the merge kernel needs to find each request's partials
      for (int i = lane; i <= a.B; i += 64) {
        if (in_lanes) {
          if (i < a.B) a.part_meta[i + 1] = whole ? upto : cum_lane;
        } else {
          a.part_meta[i] = cum[i];
        }
      }
      if (lane == 0) {
        a.part_meta[0] = 0;
        a.part_meta[a.B + 1] = whole ? 1 : chunk;
      }
    }
  };

  // ---- a run of steps of one request, and what its start waits for (page ids, q): requested for the first run before the
  // tables are built, for every other one while the run before it is computed ----
  const uint4* q4 = reinterpret_cast<const uint4*>(a.q);
  struct Seg {
    int b, c0, seg_end, n_st, step_first, L;
    int bt0, bt1, posq;  // lane i: page of block i (64 + i) of the run, as stored; position of the query token
    Frag qf[4];          // q of the lane's head: pairs 8 h .. of the low dims in qf[h], of the high dims in qf[h + 2]
  };
  auto seg_load = [&](Seg& sg, int pos, int b) __attribute__((always_inline)) {
    int c0 = cum_at(b), c1 = cum_at(b + 1);
    while (c1 <= pos) {  // skip requests without steps
      ++b;
      c0 = c1;
      c1 = cum_at(b + 1);
    }
    sg.b = b; sg.c0 = c0; sg.seg_end = min(pos_end, c1); sg.n_st = sg.seg_end - pos; sg.step_first = pos - c0;
    sg.L = in_lanes ? __builtin_amdgcn_readlane(len_lane, b) : sload(a.kv_lens, b);
    const int j0 = kBps * sg.step_first, jl = min((sg.L + kP - 1) / kP, j0 + kBps * sg.n_st) - 1;  // first and last block
    const size_t row = (size_t)b * a.max_blocks;
    sg.bt0 = a.block_tables[row + min(j0 + lane, jl)];
    sg.bt1 = a.block_tables[row + min(j0 + 64 + lane, jl)];
    sg.posq = a.q_positions[b];
    const size_t qrow = ((size_t)b * a.Hq + (size_t)hk * G + (head < G ? head : 0)) * (kD / 8);
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int glo = kFp8 ? 2 * kg + h : 4 * h + kg;
      sg.qf[h].u = q4[qrow + glo];
      sg.qf[h + 2].u = q4[qrow + 8 + glo];
    }
  };
  Seg seg;
  auto first_seg = [&]() __attribute__((always_inline)) {
    if (pos_begin >= pos_end) return;
    int lo = 0;  // request that owns the first step: largest b with cum[b] <= pos_begin
    if (in_lanes) {
      lo = min((int)__popcll(__ballot(lane < a.B && cum_lane <= pos_begin)), a.B - 1);
    } else {
      int hi = a.B - 1;
      while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (uni(cum[mid]) <= pos_begin) lo = mid; else hi = mid - 1;
      }
    }
    seg_load(seg, pos_begin, uni(lo));
  };
  if (in_lanes) {
    cut();
    first_seg();
  }
  __syncthreads();
  if (!in_lanes) {
    cut();
    first_seg();
  }
  // ---- K and V of a step, one register buffer of either ----
  // K row n16 of product u is slot 16 u + n16 of the step: whole lines per load, a uniform base and a lane offset that never
  // changes. bf16: kf[u][j] = granule 4 j + kg of page u; fp8: granules kg and kg + 4 of the page.
  // V. bf16: dim 16 nt + n16, eight slots 8 (kg / 2) .. of page kg % 2. fp8: sixteen slots 16 (kg % 2) .. of dim
  // 32 i + 16 (kg / 2) + n16; attend() makes two operands of it.
  const char* const kbase = reinterpret_cast<const char*>(a.k_pages) + (size_t)hk * kHeadBytes;
  const char* const vbase = reinterpret_cast<const char*>(a.v_pages) + (size_t)hk * kHeadBytes +
                            (kFp8 ? ((kg >> 1) * 16 + n16) * 32 + (kg & 1) * 16 : n16 * 32 + (kg >> 1) * 16);
  const uint32_t k_off = (uint32_t)(kg * kP + n16) * 16;
  const uint64_t page_bytes = (uint64_t)Hkv * kHeadBytes;
  // (p0, p1: the two pages of a bf16 step; the pages of the one or two steps of a fp8 turn)
  Frag kf[kPack][2][kNK];
  uint4 vf[kPack][kNVec];
  auto issue_k = [&](int p0, int p1) __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < kNK; ++j)  // (pages in turn: 333.7 -> 331.8 us on 8 requests of 65 537 bf16 slots)
#pragma unroll
      for (int s = 0; s < kPack; ++s)
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          const char* p = kbase + (uint64_t)(uint32_t)((kFp8 ? s : u) ? p1 : p0) * page_bytes + (kFp8 ? 256 * u : 0);
          kf[s][u][j].u = load_page<kReadOnce>(reinterpret_cast<const uint4*>(p + j * (4 * kP * 16) + k_off));
        }
  };
  auto issue_v = [&](int p0, int p1) __attribute__((always_inline)) {
#pragma unroll
    for (int s = 0; s < kPack; ++s) {
      const char* p = vbase + (uint64_t)(uint32_t)((kFp8 ? s : kg & 1) ? p1 : p0) * page_bytes;
#pragma unroll
      for (int i = 0; i < kNVec; ++i) vf[s][i] = load_page<kReadOnce>(reinterpret_cast<const uint4*>(p + i * (kFp8 ? 1024 : 512)));
    }
  };

  auto clean = [&](int id) { return safe_page(id, a.num_pages); };
  float ks_cur = 1.f, vs_cur = 1.f, ks_nxt = 1.f, vs_nxt = 1.f;  // fp8: lane i: scales of the page of block i of the window
  auto issue_first = [&]() __attribute__((always_inline)) {  // the run's first step
    const int ids = clean(seg.bt0);
    const int p0 = __builtin_amdgcn_readlane(ids, 0), p1 = kPack == 2 && seg.n_st == 1 ? p0 : __builtin_amdgcn_readlane(ids, kBps * kPack - 1);
    if constexpr (kFp8) {
      ks_cur = a.k_scales[ids];
      vs_cur = a.v_scales[ids];
    }
    issue_k(p0, p1);
    __builtin_amdgcn_sched_barrier(0);  // K before V on every path: the loop's waits count on it
    issue_v(p0, p1);
    __builtin_amdgcn_sched_barrier(0);
  };
  // ---- tables, as far as the call's longest run of a wave needs them: most_steps is the same for every wave. Where that is a step or
  // two, building all of them was 1 us of the 7.5 before the merge: 4 requests of 1.7 K slots 11.8 -> 11.0 us a call, 30 of 800 e4m3
  // slots 18.6 -> 16.9, a commit and 16 of 2.2 K (5 steps) 20.9 -> 20.7. (The first loads ahead of the tables: 11.6 and 21.7.) ----
  const int turns = uni((most_steps + kPack - 1) / kPack);
  auto entry = [&](float pos, int h, int w) __attribute__((always_inline)) {  // R(pos) of pairs 2 w and 2 w + 1 of half h
    const float2 f0 = freq_lds[kg * 16 + 8 * h + 2 * w], f1 = freq_lds[kg * 16 + 8 * h + 2 * w + 1];
    const float t0 = turns_frac(pos, f0.x, f0.y);
    const float t1 = turns_frac(pos, f1.x, f1.y);
    return make_float4(__builtin_amdgcn_cosf(t0), __builtin_amdgcn_sinf(t0), __builtin_amdgcn_cosf(t1), __builtin_amdgcn_sinf(t1));
  };
  constexpr int kPerTable = 2 * kRot * 4;
  static_assert(kWaves == 8 && kPerTable % kWaves == 0 && kRotK % kPerTable == 0, "a pass of the waves stays in one table, and is all of rotS");
#pragma unroll
  for (int base = 0; base < kRotK; base += kWaves) {
    if (base / kPerTable >= turns) break;
    const int i = base + wave, uv = i / (4 * kRot);
    const float4 r = entry((float)(n16 + 16 * (uv & 1) + kTurn * (uv >> 1)), kRot == 2 ? (i >> 2) & 1 : 0, i & 3);
    if constexpr (kFp8) {  // {cos pair, sin pair} as packed fp16
      rotK[i][lane] = make_float2(__uint_as_float(pack_f16x2(r.x, r.z)), __uint_as_float(pack_f16x2(r.y, r.w)));
    } else {  // per pair the two constant words (cos, -sin) and (sin, cos) as packed bf16
      rotK[i][lane] = make_float4(__uint_as_float(pack2_bf16(r.x, -r.y)), __uint_as_float(pack2_bf16(r.y, r.x)),
                                  __uint_as_float(pack2_bf16(r.z, -r.w)), __uint_as_float(pack2_bf16(r.w, r.z)));
    }
  }
  if (turns > kNV) rotS[wave][lane] = entry(-(float)(kTurn * kNV), wave >> 2, wave & 3);
  __syncthreads();
  if (pos_begin >= pos_end) return;

  floatx4 o[8];
  floatx4 sc0;                 // minus the reference maximum (log2 units): what bf16 score accumulators start from
  float l_part;
  float v_ref = 0.f;           // fp8: O is kept in units of this reference V scale (one for each part), raised lazily
  float v_lim = 0.f, v_inv = 0.f;  // 1.75 v_ref, 1 / v_ref
  float qlo[2][8], qhi[2][8];  // Q' of this lane's matrix row for its 16 rotary pairs [h][e], in log2 units
  Frag bq[4];                  // the same as matrix operands
  auto pack_q = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int e = 0; e < 8; e += 2) {
        bq[h].w[e / 2] = kFp8 ? pack_f16x2(qlo[h][e], qlo[h][e + 1]) : pack2_bf16(qlo[h][e], qlo[h][e + 1]);
        bq[h + 2].w[e / 2] = kFp8 ? pack_f16x2(qhi[h][e], qhi[h][e + 1]) : pack2_bf16(qhi[h][e], qhi[h][e + 1]);
      }
  };
  auto advance_q = [&]() __attribute__((always_inline)) {  // by R(-kTurn kNV)
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        const float4 r = rotS[h * 4 + w][lane];
        const float a0 = qlo[h][2 * w], b0 = qhi[h][2 * w], a1 = qlo[h][2 * w + 1], b1 = qhi[h][2 * w + 1];
        qlo[h][2 * w] = a0 * r.x - b0 * r.y;
        qhi[h][2 * w] = b0 * r.x + a0 * r.y;
        qlo[h][2 * w + 1] = a1 * r.z - b1 * r.w;
        qhi[h][2 * w + 1] = b1 * r.z + a1 * r.w;
      }
    pack_q();
  };

  // Rotate the eight pairs of half h of product u's rows, and multiply.
  auto rotated = [&](floatx4& sc, const Frag (&k)[2][kNK], int u, int h, const RotK (&r)[4]) __attribute__((always_inline)) {
    Frag klo, khi;
    if constexpr (kFp8) {
      // e4m3 codes -> packed fp16 (exact), rotated with packed fp16 arithmetic (two pairs per instruction; fp16 keeps 11
      // significant bits, more than the bf16 operands of the bf16 path), fp16 products
#pragma unroll
      for (int w = 0; w < 4; ++w) {  // pairs 8h + 2w and 8h + 2w + 1
        const uint32_t wl = k[u][0].w[2 * h + (w >> 1)], wh = k[u][1].w[2 * h + (w >> 1)];
        const f16x2 lo = (w & 1) ? __builtin_amdgcn_cvt_scalef32_pk_f16_fp8(wl, 1.0f, true)
                                 : __builtin_amdgcn_cvt_scalef32_pk_f16_fp8(wl, 1.0f, false);
        const f16x2 hi = (w & 1) ? __builtin_amdgcn_cvt_scalef32_pk_f16_fp8(wh, 1.0f, true)
                                 : __builtin_amdgcn_cvt_scalef32_pk_f16_fp8(wh, 1.0f, false);
        const f16x2 c2 = __builtin_bit_cast(f16x2, __float_as_uint(r[w].x));
        const f16x2 s2 = __builtin_bit_cast(f16x2, __float_as_uint(r[w].y));
        klo.w[w] = __builtin_bit_cast(uint32_t, lo * c2 - hi * s2);
        khi.w[w] = __builtin_bit_cast(uint32_t, hi * c2 + lo * s2);
      }
      sc = __builtin_amdgcn_mfma_f32_16x16x32_f16(klo.hv, bq[h].hv, sc, 0, 0, 0);
      sc = __builtin_amdgcn_mfma_f32_16x16x32_f16(khi.hv, bq[h + 2].hv, sc, 0, 0, 0);
    } else {
#pragma unroll
      for (int w = 0; w < 4; w += 2) {  // pairs 8h + 2w .. 8h + 2w + 3
        // Bring the low and the high element of a pair into one word (v_perm_b32); each rotated element is then
        // one two-term dot product with a constant word, (cos, -sin) or (sin, cos), accumulated in fp32.
        const uint32_t la = k[u][h].w[w], ha = k[u][h + 2].w[w], lb = k[u][h].w[w + 1], hb = k[u][h + 2].w[w + 1];
        const uint32_t e0 = __builtin_amdgcn_perm(ha, la, 0x05040100u), e1 = __builtin_amdgcn_perm(ha, la, 0x07060302u);
        const uint32_t e2 = __builtin_amdgcn_perm(hb, lb, 0x05040100u), e3 = __builtin_amdgcn_perm(hb, lb, 0x07060302u);
        float l0, l1, l2, l3, h0, h1, h2, h3;
        dot_rotate_block(e0, e1, e2, e3, __float_as_uint(r[w].x), __float_as_uint(r[w].y), __float_as_uint(r[w].z),
                         __float_as_uint(r[w].w), __float_as_uint(r[w + 1].x), __float_as_uint(r[w + 1].y),
                         __float_as_uint(r[w + 1].z), __float_as_uint(r[w + 1].w), l0, l1, l2, l3, h0, h1, h2, h3);
        klo.w[w] = pack2_bf16(l0, l1);
        klo.w[w + 1] = pack2_bf16(l2, l3);
        khi.w[w] = pack2_bf16(h0, h1);
        khi.w[w + 1] = pack2_bf16(h2, h3);
      }
      sc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(klo.v, bq[h].v, sc, 0, 0, 0);
      sc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(khi.v, bq[h + 2].v, sc, 0, 0, 0);
    }
  };
  // Scores of a turn relative to the reference maximum, log2 units: lane (part, head, kg) has slots 16 u + 4 kg + e of its step.
  // ksc: its page's K scale (fp8).
  auto scores = [&](floatx4 (&sc)[2], int v, float ksc) __attribute__((always_inline)) {
    floatx4 x[kPack][2];
#pragma unroll
    for (int s = 0; s < kPack; ++s)
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        if constexpr (kFp8) x[s][u] = floatx4{0.f, 0.f, 0.f, 0.f};
        else x[s][u] = sc0;
      }
    if constexpr (kTerms > 1) {
      if constexpr (kFull) {  // (no row is left whose zeros would tell of an infinite key)
        const Frag none = {make_uint4(0, 0, 0, 0)};
#pragma unroll
        for (int j = 1; j < 4; j += 2)
#pragma unroll
          for (int u = 0; u < 2; ++u) x[0][u] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[0][u][j].v, none.v, x[0][u], 0, 0, 0);
      }
#pragma unroll
      for (int u = 0; u < 2; ++u) {  // the slow half: keys as they are
        x[0][u] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[0][u][1].v, bq[1].v, x[0][u], 0, 0, 0);
        x[0][u] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[0][u][3].v, bq[3].v, x[0][u], 0, 0, 0);
      }
    }
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int h = 0; h < kRot; ++h) {
        RotK r[4];
#pragma unroll
        for (int w = 0; w < 4; ++w) r[w] = rotK[((v * 2 + u) * kRot + h) * 4 + w][lane];
#pragma unroll
        for (int s = 0; s < kPack; ++s) rotated(x[s][u], kf[s], u, h, r);
        __builtin_amdgcn_sched_barrier(0);  // (two sets of constants live at most)
      }
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      if constexpr (kPack == 2) {
#pragma unroll
        for (int e = 0; e < 4; ++e) sc[u][e] = part ? x[kPack - 1][u][e] : x[0][u][e];
      } else {
        sc[u] = x[0][u];
      }
      if constexpr (kFp8) {
#pragma unroll
        for (int e = 0; e < 4; ++e) sc[u][e] = __builtin_fmaf(sc[u][e], ksc, sc0[0]);
      }
    }
    if constexpr (kTerms > 1) {
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const floatx4 x = sc[u];
        const float4 t = weight[0][v][u][kg];
        sc[u][0] = __builtin_fmaf(lane_up<1>(x[0]), t.x, sc[u][0]);
        sc[u][1] = __builtin_fmaf(lane_up<1>(x[1]), t.y, sc[u][1]);
        sc[u][2] = __builtin_fmaf(lane_up<1>(x[2]), t.z, sc[u][2]);
        sc[u][3] = __builtin_fmaf(lane_up<1>(x[3]), t.w, sc[u][3]);
        if constexpr (kTerms > 2) {
          const float4 t2 = weight[kTerms > 2 ? 1 : 0][v][u][kg];
          sc[u][0] = __builtin_fmaf(lane_up<2>(x[0]), t2.x, sc[u][0]);
          sc[u][1] = __builtin_fmaf(lane_up<2>(x[1]), t2.y, sc[u][1]);
          sc[u][2] = __builtin_fmaf(lane_up<2>(x[2]), t2.z, sc[u][2]);
          sc[u][3] = __builtin_fmaf(lane_up<2>(x[3]), t2.w, sc[u][3]);
        }
      }
    }
  };

  // Softmax of the turn's scores and the output products.
  // vs0, vs1: the V scales of the turn's pages (fp8).
  bool unset = true;  // no reference maximum yet
  auto attend = [&](floatx4 (&sc)[2], float vs0, float vs1) __attribute__((always_inline)) {
    float pf[8], psum;
    auto exps = [&]() __attribute__((always_inline)) {
#pragma unroll
      for (int e = 0; e < 8; ++e) pf[e] = __builtin_amdgcn_exp2f(sc[e >> 2][e & 3]);
      psum = ((pf[0] + pf[1]) + (pf[2] + pf[3])) + ((pf[4] + pf[5]) + (pf[6] + pf[7]));
    };
    exps();
    // The reference maximum only has to keep probabilities bounded; it is raised, and everything accumulated so far
    // rescaled, only when a lane's sum gets past the bound. Rare after the first step, so the cross-lane work sits in the branch.
    if (__ballot(row_ok && (unset || !(psum <= most_sum(kFp8)))) != 0) {
      const float mx = max_over_kgroups(fmaxf(fmaxf(fmaxf(sc[0][0], sc[0][1]), fmaxf(sc[0][2], sc[0][3])),
                                              fmaxf(fmaxf(sc[1][0], sc[1][1]), fmaxf(sc[1][2], sc[1][3]))));
      float up = unset ? mx : fmaxf(mx, 0.f);
      if (!row_ok || up == -INFINITY) up = 0.f;  // (the other terms' rows have no reference)
      sc0 -= up;
      sc[0] -= up;
      sc[1] -= up;
      exps();
      const float alpha = unset ? 1.f : __builtin_amdgcn_exp2f(-up);
      if (__ballot(row_ok && !unset) != 0) {  // (nothing is accumulated before the first step)
        l_part *= alpha;
        // accumulator rows of this lane are matrix rows 4 kg + e; their factors live in lanes 4 kg + e
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float ar = __shfl(alpha, 4 * kg + e);
#pragma unroll
          for (int nt = 0; nt < 8; ++nt) o[nt][e] *= ar;
        }
      }
      unset = unset && mx == -INFINITY;
    }
    l_part += psum;
    // A lane has the probabilities of four slots of either product. Exchanged between neighbouring k-groups they are those of
    // eight consecutive slots, in the order that V is loaded in: k-groups 0 .. 3 have slots 0-7, 16-23, 8-15, 24-31.
    if constexpr (kFp8) {
      // The page's V scale rides on the probabilities: O accumulates in units of a reference scale v_ref that is
      // at least vsc / 1.75, raised (with a rescale of O) only when a page's scale exceeds that; then
      // p * 16 * vsc / v_ref = hi + lo, both e4m3: p <= 16, so the product stays below 448, the largest
      // e4m3 value. Pages with a much smaller scale lose relative precision in proportion to how little they add.
      const float vsc = kPack == 2 && part ? vs1 : vs0;
      if (__ballot(vsc > v_lim) != 0) {
        const bool raise = vsc > v_lim;
        const float f = __shfl(raise ? v_ref / vsc : 1.f, kPack == 2 ? 8 * (kg >> 1) : 0);  // of the accumulator's rows; 0 on the first page
#pragma unroll
        for (int nt = 0; nt < 8; ++nt) o[nt] *= f;
        v_ref = raise ? vsc : v_ref;
        v_lim = 1.75f * v_ref;
        v_inv = v_ref > 0.f ? __builtin_amdgcn_rcpf(v_ref) : 0.f;  // a zero scale means an all-zero page
      }
      const float ps = kPScale * (vsc * v_inv);
      uint32_t hi[2], lo[2];
#pragma unroll
      for (int w = 0; w < 2; ++w) {
        float x[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) x[e] = pf[4 * w + e] * ps;
        int hw = __builtin_amdgcn_cvt_pk_fp8_f32(x[0], x[1], 0, false);
        hw = __builtin_amdgcn_cvt_pk_fp8_f32(x[2], x[3], hw, true);
        const f32x2 b0 = __builtin_amdgcn_cvt_pk_f32_fp8(hw, false), b1 = __builtin_amdgcn_cvt_pk_f32_fp8(hw, true);
        int lw = __builtin_amdgcn_cvt_pk_fp8_f32(x[0] - b0[0], x[1] - b0[1], 0, false);
        lw = __builtin_amdgcn_cvt_pk_fp8_f32(x[2] - b1[0], x[3] - b1[1], lw, true);
        hi[w] = (uint32_t)hw;
        lo[w] = (uint32_t)lw;
      }
      const auto ah = __builtin_amdgcn_permlane16_swap(hi[0], hi[1], false, false);
      const auto al = __builtin_amdgcn_permlane16_swap(lo[0], lo[1], false, false);
      const long a_hi = (long)(((uint64_t)ah[1] << 32) | ah[0]), a_lo = (long)(((uint64_t)al[1] << 32) | al[0]);
#pragma unroll
      for (int s = 0; s < kPack; ++s) {
        // (rows of the turn's other step take no part)
        const long p_hi = kPack == 2 && part != s ? 0 : a_hi, p_lo = kPack == 2 && part != s ? 0 : a_lo;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          // slots 0-7 | 8-15 (k-groups 0, 2) and 16-23 | 24-31 (1, 3) of dims 32 i (k-groups 0, 1) and 32 i + 16 (2, 3): the
          // upper half of the one register against the lower half of the other makes the operand of either tile
          const auto x = __builtin_amdgcn_permlane32_swap(vf[s][i].x, vf[s][i].z, false, false);
          const auto y = __builtin_amdgcn_permlane32_swap(vf[s][i].y, vf[s][i].w, false, false);
          const long v0 = (long)(((uint64_t)y[0] << 32) | x[0]), v1 = (long)(((uint64_t)y[1] << 32) | x[1]);
          o[2 * i] = __builtin_amdgcn_mfma_f32_16x16x32_fp8_fp8(p_hi, v0, o[2 * i], 0, 0, 0);
          o[2 * i + 1] = __builtin_amdgcn_mfma_f32_16x16x32_fp8_fp8(p_hi, v1, o[2 * i + 1], 0, 0, 0);
          o[2 * i] = __builtin_amdgcn_mfma_f32_16x16x32_fp8_fp8(p_lo, v0, o[2 * i], 0, 0, 0);
          o[2 * i + 1] = __builtin_amdgcn_mfma_f32_16x16x32_fp8_fp8(p_lo, v1, o[2 * i + 1], 0, 0, 0);
        }
      }
    } else {
      Frag pa;
#pragma unroll
      for (int w = 0; w < 2; ++w) {
        const auto x = __builtin_amdgcn_permlane16_swap(pack2_bf16(pf[2 * w], pf[2 * w + 1]),
                                                        pack2_bf16(pf[4 + 2 * w], pf[5 + 2 * w]), false, false);
        pa.w[w] = x[0];
        pa.w[w + 2] = x[1];
      }
#pragma unroll
      for (int nt = 0; nt < 8; ++nt) {
        Frag vb;
        vb.u = vf[0][nt];
        o[nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(pa.v, vb.v, o[nt], 0, 0, 0);
      }
    }
  };

  // ---- walk the wave's chunk request by request ----
  auto of_lane = [](float x, int i) { return __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(x), i)); };
  uint64_t again = 0;  // terms: bit i: the wave's run i is to be computed again (63: every run from there on)
  int run = 0, turn = 0;
  const bool later = wave >= kWaves / 2;
  issue_first();
  for (;;) {
    const int b = seg.b, c0 = seg.c0, n_st = seg.n_st, step_first = seg.step_first, L = seg.L;
    const int j0 = kBps * step_first, jend = min((L + kP - 1) / kP, j0 + kBps * n_st);
    const size_t bt_row = (size_t)b * a.max_blocks;
    // Page ids of the run: lane i of bt_cur holds the page of block 64 k + i of the run (clamped to its last block), bt_nxt the 64 after those
    // as stored; a step reads its ids with v_readlane. Vector loads on purpose: scalar loads share a counter with the LDS reads, so every
    // wait for a rotation constant would also wait for them.
    int bt_cur = clean(seg.bt0), bt_nxt = seg.bt1;

    // Q' = R(pos_q - n0) q, scaled into log2 units; reset the accumulators
#pragma unroll
    for (int nt = 0; nt < 8; ++nt) o[nt] = floatx4{0.f, 0.f, 0.f, 0.f};
    sc0 = floatx4{0.f, 0.f, 0.f, 0.f};
    l_part = 0.f;
    v_ref = v_lim = v_inv = 0.f;
    unset = true;
    {
      const float delta = (float)(uni(seg.posq) - step_first * 32 - 32 * part);
      const float qs = head < G ? a.qk_scale_log2 : 0.f;  // (rows without a head are zeros)
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const float2 f = freq_lds[kg * 16 + 8 * h + e];
          const uint32_t wl = seg.qf[h].w[e >> 1], wh = seg.qf[h + 2].w[e >> 1];
          const float x0 = qs * ((e & 1) ? __uint_as_float(wl & 0xffff0000u) : bf16_bits_to_f32(wl & 0xffffu));
          const float x1 = qs * ((e & 1) ? __uint_as_float(wh & 0xffff0000u) : bf16_bits_to_f32(wh & 0xffffu));
          const float t = turns_frac(kTerms > 1 && h == 1 ? delta - kCentre : delta, f.x, f.y);
          const float c = __builtin_amdgcn_cosf(t), sn = __builtin_amdgcn_sinf(t);
          qlo[h][e] = x0 * c - x1 * sn;
          qhi[h][e] = x1 * c + x0 * sn;
          if constexpr (kTerms > 1) {
            const float2 k = coef[term][kg * 16 + 8 * h + e];
            const float y0 = qlo[h][e], y1 = qhi[h][e];
            qlo[h][e] = y0 * k.x + y1 * k.y;
            qhi[h][e] = y1 * k.x - y0 * k.y;
          }
        }
      pack_q();
    }

    const bool more = seg.seg_end < pos_end;
    if (more) seg_load(seg, seg.seg_end, b);  // the next run: in flight while this one is computed

    constexpr int kBpt = kBps * kPack;                // pages a turn
    const int n_turns = (n_st + kPack - 1) / kPack;
    int v = 0;
    for (int t = 0; t < n_turns - 1; ++t) {
      take_turns(later, turn++);
      const int here = (kBpt * t) & 63, rel = (kBpt * (t + 1)) & 63;  // blocks of this and the next turn in their windows
      float ksc = 1.f, vs0 = 1.f, vs1 = 1.f;
      if constexpr (kFp8) {
        ksc = of_lane(ks_cur, here);
        vs0 = of_lane(vs_cur, here);
        if constexpr (kPack == 2) {
          const float k1 = of_lane(ks_cur, here + 1);
          ksc = part ? k1 : ksc;
          vs1 = of_lane(vs_cur, here + 1);
        }
      }
      if (rel == 0) {
        bt_cur = clean(bt_nxt);
        bt_nxt = a.block_tables[bt_row + min(j0 + kBpt * (t + 1) + 64 + lane, jend - 1)];
        if constexpr (kFp8) {
          ks_cur = ks_nxt;
          vs_cur = vs_nxt;
        }
      }
      if (kFp8 && here == 32) {
        const int ids = clean(bt_nxt);
        ks_nxt = a.k_scales[ids];
        vs_nxt = a.v_scales[ids];
      }
      const int p0 = __builtin_amdgcn_readlane(bt_cur, rel);
      const int p1 = kPack == 2 && 2 * t + 3 >= n_st ? p0 : __builtin_amdgcn_readlane(bt_cur, rel + kBpt - 1);
      floatx4 sc[2];
      scores(sc, v, ksc);
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (!kReadOnce) issue_k(p0, p1);
      __builtin_amdgcn_sched_barrier(0);
      attend(sc, vs0, vs1);
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (kReadOnce) issue_k(p0, p1);
      issue_v(p0, p1);
      __builtin_amdgcn_sched_barrier(0);
      if (++v == kNV) {
        v = 0;
        advance_q();
      }
    }
    {  // the run's last turn
      const int here = (kBpt * (n_turns - 1)) & 63;
      const int n0 = (step_first + kPack * (n_turns - 1)) * 32, end = min(L, (step_first + n_st) * 32);
      float ksc = 1.f, vs0 = 1.f, vs1 = 1.f;
      if constexpr (kFp8) {
        ksc = of_lane(ks_cur, here);
        vs1 = vs0 = of_lane(vs_cur, here);
        if (kPack == 2 && n0 + 32 < end) {
          const float k1 = of_lane(ks_cur, here + 1);
          ksc = part ? k1 : ksc;
          vs1 = of_lane(vs_cur, here + 1);
        }
      }
      floatx4 sc[2];
      scores(sc, v, ksc);
      if (n0 + kTurn > end) {
        // slots at or past kv_len take no part and may hold anything (even NaN): masked here, zeroed in V; so are those of a
        // step that is not the run's
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (n0 + 32 * part + 16 * u + 4 * kg + e >= end) sc[u][e] = -INFINITY;
#pragma unroll
        for (int s = 0; s < kPack; ++s) {
          const int left = end - (n0 + 32 * s + 16 * (kg & 1) + (kFp8 ? 0 : 8 * (kg >> 1)));  // of the slots in the lane's V
#pragma unroll
          for (int w = 0; w < 4; ++w) {
            uint32_t keep = 0;
            if constexpr (kFp8) {
#pragma unroll
              for (int e = 0; e < 4; ++e) keep |= 4 * w + e < left ? 0xffu << (8 * e) : 0u;
            } else {
              keep = (2 * w < left ? 0x0000ffffu : 0u) | (2 * w + 1 < left ? 0xffff0000u : 0u);
            }
#pragma unroll
            for (int i = 0; i < kNVec; ++i) reinterpret_cast<uint32_t*>(&vf[s][i])[w] &= keep;
          }
        }
      }
      attend(sc, vs0, vs1);
    }
    if (more) issue_first();

    // the partial of this (request, wave): un-normalised rows, reference max (log2 units), sum
    {
      const int split = whole ? piece : wk - c0 / chunk;
      const size_t row0 = ((size_t)b * a.Hq + (size_t)hk * G) * a.n_splits + split;  // + g * n_splits
      float l_tot = sum_over_kgroups(l_part), m = l_tot == 0.f ? -INFINITY : -sc0[0], f = 1.f;
      if constexpr (kPack == 2) {  // rows 8 .. 15 are the same heads', relative to a maximum of their own
        const float most = fmaxf(m, row_ror<8>(m));
        f = m == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m - most);
        l_tot *= f;
        l_tot += row_ror<8>(l_tot);
        m = most;
      }
      if (kg == 0 && row_ok && part == 0) {
        a.part_ml[(row0 + (size_t)head * a.n_splits) * 2] = m;
        a.part_ml[(row0 + (size_t)head * a.n_splits) * 2 + 1] = l_tot;
      }
      const float unit = kFp8 ? __shfl(v_ref, kPack == 2 ? 8 * (kg >> 1) : 0) * (1.f / kPScale) : 1.f;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int r = 4 * kg + e, g = r / kTerms;
        const float scale = kPack == 2 ? unit * __shfl(f, r) : unit;
        float x[8];
#pragma unroll
        for (int nt = 0; nt < 8; ++nt) {
          x[nt] = kFp8 ? o[nt][e] * scale : o[nt][e];
          if constexpr (kPack == 2) {
            const auto y = __builtin_amdgcn_permlane32_swap(__float_as_uint(x[nt]), __float_as_uint(x[nt]), false, false);
            x[nt] = __uint_as_float(y[0]) + __uint_as_float(y[1]);
          }
        }
        if (g < G && r % kTerms == 0 && (kPack == 1 || kg < 2)) {
          float* dst = a.part_o + (row0 + (size_t)g * a.n_splits) * kD + n16;
#pragma unroll
          for (int nt = 0; nt < 8; ++nt) dst[16 * nt] = x[nt];
        }
      }
    }
    if constexpr (kTerms > 1) {
      // An infinite key, or terms past the largest float, made NaN of a probability: of its row, or of a row without a head, all
      // of whose products are 0 x key (the sums of the lanes of such rows are looked at for nothing else).
      if (__ballot(l_part != l_part) != 0) again |= 1ull << min(run, 63);
      ++run;
    }
    if (!more) break;
  }
  if (kTerms > 1 && again != 0) {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");  // the partials written above come first, also those of other lanes
    int b = 0, pos = pos_begin;
    for (run = 0; pos < pos_end; ++run) {
      while (cum_at(b + 1) <= pos) ++b;
      const int c0 = cum_at(b), end = min(pos_end, cum_at(b + 1)), L = in_lanes ? __builtin_amdgcn_readlane(len_lane, b) : sload(a.kv_lens, b);
      if ((again >> min(run, 63)) & 1)
        plain_run(a, freq_lds, b, hk, 32 * (pos - c0), min(L, 32 * (end - c0)),
                  ((size_t)b * a.Hq + (size_t)hk * G) * a.n_splits + (whole ? piece : wk - c0 / chunk));
      pos = end;
    }
  }
}

template <bool kFp8, int kTerms, int kPack, bool kFull = false>
void launch_one(const AttnArgs& a, int n_wg, hipStream_t s) {
  const size_t lds = a.B <= 64 ? 0 : (size_t)(a.B + 1) * sizeof(int);
  if (a.kv_read_once) hipLaunchKernelGGL((decode_plain_kernel<kFp8, kTerms, kPack, kFull, true>), dim3(n_wg), dim3(64 * kWaves), lds, s, a);
  else hipLaunchKernelGGL((decode_plain_kernel<kFp8, kTerms, kPack, kFull, false>), dim3(n_wg), dim3(64 * kWaves), lds, s, a);
}

// Merge the partials of one (request, query head). Request b owns steps [cum[b], cum[b+1]) of its KV
// head's sequence; the waves that cut that range wrote partials 0 .. (cum[b+1]-1)/chunk - cum[b]/chunk.
template <int kThreads>
__global__ __launch_bounds__(kThreads) void combine_streamk_kernel(const AttnArgs a) {
  const int row = blockIdx.x;
  const int b = row / a.Hq;
  const int c0 = a.part_meta[b], c1 = a.part_meta[b + 1], chunk = a.part_meta[a.B + 1];
  const int ns = c1 > c0 ? (c1 - 1) / chunk - c0 / chunk + 1 : 0;
  merge_row<kD, kThreads>(a.part_ml + (size_t)row * a.n_splits * 2, a.part_o + (size_t)row * a.n_splits * kD, a.n_splits, ns,
                          reinterpret_cast<uint16_t*>(a.out) + (size_t)row * kD);
}

// Self-test of dot_rotate_block: words[i] = {e0..e3, ca0, cb0, ca1, cb1, ca2, cb2, ca3, cb3}; out[i] = {l0..l3, h0..h3}.
__global__ __launch_bounds__(256) void dot_rotate_selftest_kernel(const uint32_t* words, float* out, int n) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i >= n) return;
  const uint32_t* w = words + (size_t)i * 12;
  float r[8];
  dot_rotate_block(w[0], w[1], w[2], w[3], w[4], w[5], w[6], w[7], w[8], w[9], w[10], w[11], r[0], r[1], r[2], r[3], r[4],
                   r[5], r[6], r[7]);
#pragma unroll
  for (int k = 0; k < 8; ++k) out[(size_t)i * 8 + k] = r[k];
}

int compute_units() {
  static const int cus = [] {  // initialised once, thread-safely (function-local static)
    int dev = 0, n = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0)
      n = 256;
    return n;
  }();
  return cus;
}

}  // namespace

hipError_t launch_decode_plain(const AttnArgs& a, hipStream_t s) {
  const int n_wg = max(compute_units() / a.Hkv, 1) * a.Hkv;  // a whole number of workgroups per KV head
  if (a.timing_start) (void)hipEventRecord(reinterpret_cast<hipEvent_t>(a.timing_start), s);
  // bf16: idle matrix rows take the place of the slow half's rotation where two (three) terms of the expansion are enough and a
  // head has as many rows: f radians a position, of the fastest pair of that half, times the half span between two advances of Q'. The
  // first term left out is at most x^2 / 4 (x^3 / 24), 2.5e-3 (1.8e-3) of that one pair's part of a score where the lines lie, and
  // falls with the square (cube) of the frequency from there: 4e-4 (3e-4) of a score in the root mean square over the pairs,
  // against the 1.1e-3 that rounding every rotated key to bf16 cost and that these pairs no longer have. rope_theta 5e5: x = 0.09,
  // two terms; 1e4: x = 0.32, three. 64 requests of 4.3 K slots, us a call: 73.3 with two terms, 74.2 with three, 75.4 with all
  // pairs rotated; a commit and 16 requests of 2.2 K slots 23.2, 23.7, 25.0.
  const float f = 6.283185307f * a.freq_hi[32];
  if (a.kv_dtype == MEPIC_F8E4M3) {
    // Two steps a turn where a KV head's query heads fit half the matrix rows and waves have steps enough (by the bound on the lengths):
    // 128 requests of 2 - 33 K slots, 7 heads each, 257 steps a wave, 182 us a call against 193; 130 requests of 2 K, 8 heads, 36 a wave, 104
    // against 106. With fewer, requests and parts of an odd number of steps leave too many turns half empty: us with two and one steps
    // a turn 130 of 1.1 K (19 a wave) 61.0 and 59.4, 130 of up to 328 slots (5.6) 28.7 and 24.4, 1 of 200 11.1 and 9.8.
    // Between half a step and one a wave, where up to 64 requests are cut into pieces of their own, it is turns that make
    // pieces, and so partials: 4 of 5.7 K slots on 2 heads 14.8 and 18.0, 20 of 1.1 K 12.9 and 13.5, 64 of 200 13.2 and 13.1.
    const long steps = (long)a.B * a.kv_tiles, waves = (long)(n_wg / a.Hkv) * kWaves;
    if (a.G <= 8 && (steps >= 32 * waves || (a.B > 1 && a.B <= 64 && 2 * steps > waves && steps <= waves))) launch_one<true, 1, 2>(a, n_wg, s);
    else launch_one<true, 1, 1>(a, n_wg, s);
  } else if (63.5f * f <= 0.1f && a.G <= 8) {
    if (a.G == 8) launch_one<false, 2, 1, true>(a, n_wg, s);
    else launch_one<false, 2, 1>(a, n_wg, s);
  } else if (31.5f * f <= 0.35f && a.G <= 5) {
    launch_one<false, 3, 1>(a, n_wg, s);
  } else {
    launch_one<false, 1, 1>(a, n_wg, s);
  }
  const hipError_t e = hipGetLastError();
  if (a.timing_stop) (void)hipEventRecord(reinterpret_cast<hipEvent_t>(a.timing_stop), s);
  if (e != hipSuccess) return e;
  const int rows = a.n_q * a.Hq;
  if (rows <= kMergeFewRows)
    hipLaunchKernelGGL((combine_streamk_kernel<kMergeThreadsFew>), dim3(rows), dim3(kMergeThreadsFew), 0, s, a);
  else
    hipLaunchKernelGGL((combine_streamk_kernel<kMergeThreads>), dim3(rows), dim3(kMergeThreads), 0, s, a);
  return hipGetLastError();
}

// Requests one plain decode call can take: the per-request step counts (B + 1 ints of dynamic LDS) must fit beside the
// kernel's static tables in the 64 KB a workgroup gets without asking for more.
int decode_plain_max_requests() { return (64 * 1024 - 44 * 1024) / (int)sizeof(int) - 1; }

int device_compute_units() { return compute_units(); }

hipError_t launch_dot_rotate_selftest(const uint32_t* words, float* out, int n, hipStream_t s) {
  hipLaunchKernelGGL(dot_rotate_selftest_kernel, dim3((n + 255) / 256), dim3(256), 0, s, words, out, n);
  return hipGetLastError();
}

// Upper bound on the partials per request and the matching minimum chunk (in steps of 32 slots), from
// host-known sizes only: with W waves per KV head and B requests a request needs about W/B pieces for an even
// cut; allow four times that for skewed length mixes, never more than W. (W counts half compute units of four waves, so that for head
// counts that do not divide the units it is a few more or fewer than the kernel's waves. It sets the size of the workspace, which callers have
// laid out; the kernel keeps to the minimum chunk, and so to the partials there is room for.)
void decode_plain_plan(int B, int Hkv, int max_kv_len, int* max_splits, int* min_chunk) {
  const int W = max(2 * compute_units() / Hkv, 1) * 4;
  const int max_steps = max((max_kv_len + 31) / 32, 1);
  int pieces = 4 * ((W + max(B, 1) - 1) / max(B, 1));
  if (pieces > W) pieces = W;
  if (pieces > max_steps) pieces = max_steps;
  *min_chunk = (max_steps + pieces - 1) / pieces;
  *max_splits = (max_steps + *min_chunk - 1) / *min_chunk + 1;
}

}  // namespace mepic
