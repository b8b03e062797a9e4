// General-path prefill of fused-RoPE paged attention (§3.3.3) on matrix cores, for bf16 and e4m3 pages: both rotary
// pairings, D 64 / 128, pages of 16 / 32 slots, any number of query heads per KV head, block positions, valid masks.
// Split precision throughout (split_common.h). For more than a few query tokens per request.
//
// One workgroup of 8 waves serves 256 query rows (row = query token x head of the KV head's group, counted through
// token boundaries so that no group size leaves rows idle) of one (request, KV head) and walks the KV in tiles of 64 slots.
// A workgroup fills a compute unit, so there is exactly one for each, and the work of a KV head - all its (row tile,
// KV tile) pairs in one sequence - is cut into equal runs, however the lengths differ as long as a run is at least the longest
// request over the pieces a row has room for (prefill_split_plan); rows of a row tile that is cut are merged by a second kernel. (Workgroups per (row tile, split) ran in rounds with idle units at the end, and empty ones among them,
// for requests with fewer row tiles than the grid allows, put two full ones on the same unit: 1.6 times the time.)
//   stage   a thread rotates one slot's share of K (8 rotary pairs) in fp32 at the slot's own position - hardware
//           sin/cos of a phase reduced with the two-float frequency - and writes head and remainder to LDS in operand
//           order; V goes there as bf16 (e4m3 codes widen exactly; the page's V scale rides on the probabilities).
//   QK      S^T[32 slots x 32 rows] per wave, three v_mfma_f32_32x32x16_bf16 per 16 dims.
//   softmax fp32, reference maximum raised lazily, as in attn_prefill_mfma.hip.
//   PV      O^T[D x 32 rows] += V^T x P^T, two products (head and remainder of P) per operand read.
// The rotation is shared by 256 rows and every K/V operand read from LDS feeds 1.5 (K) or 2 (V) products; 80 products per wave
// and tile where the bf16 kernel has 32. Neither pipe bounds the loop alone: on the fp8 call below vector instructions issue
// for 269 K of 580 K clocks (each row tile rotates its keys anew, with a sine and a cosine a pair), the matrix pipe is busy for
// 222 K, and the two groups of waves overlap them only in part. Measured against the scalar kernel:
// 8 requests of 2 - 12 K fp8 slots, 128 question tokens, 28 heads on 4: 10 772 -> 251 us a call (335 with workgroups per row
// tile and split); 4 of 4.2 K bf16 slots with masks and positions, 121 tokens, 32 heads on 8: 2 684 -> 108 us (128); 16 of
// 17 K bf16 slots in pages of 32, 256 tokens: 480 TFLOP/s of attention, 1.2 PFLOP/s of products.
//
// Slots that do not take part for any row (pads, past kv_len) are zeroed in V when staged. A slot that only some rows
// see (causal edge) may hold Inf or NaN, infinities anywhere may turn into NaN between the terms of a split, and probabilities of up
// to kBig times values of 2^88 and more make Inf of finite ones: the tokens of rows that come out NaN or Inf are computed again
// by the scalar body at the end (attn_scalar.h).
#include "attn_scalar.h"
#include "merge_partials.h"
#include "split_common.h"

namespace mepic {
namespace {

typedef float floatx16 __attribute__((ext_vector_type(16)));

constexpr int kThreads = 512;
constexpr int kRows = 256;   // query rows per workgroup, 32 per wave
constexpr int kTile = 64;    // KV slots per tile
constexpr int kNBuf = 3;     // LDS tile buffers
constexpr float kBig = 0x1p40f;  // row sum of a block that makes the reference maximum move

template <int D>
struct __align__(16) Tile {
  uint4 khi[D / 8 * kTile];  // [chunk of 8 dims][slot], rotated
  uint4 klo[D / 8 * kTile];
  uint4 v[4 * D * 2];        // [group of 16 slots][dim][half], halves swapped where bit 3 of the dim is set
  int pos[4];                // position of each group's first slot
  uint32_t valid[4];         // which of its 16 slots take part
  float vsc[4];              // V scale of its page
};

// Workgroup barrier that orders LDS traffic only: global loads issued before it stay in flight across it.
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

constexpr int kMaxRedo = 32;
constexpr int kMaxRequests = 2048;  // of one call: their work's prefix sums live in LDS

template <bool kFp8, int D, int P, bool kIL>
__global__ __launch_bounds__(kThreads, 1) void prefill_split_kernel(const AttnArgs a) {
  constexpr int kCh = D / 16;     // chunks of 8 rotary pairs = waves that stage K
  constexpr int kKs = D / 16;     // k-steps of 16 dims
  constexpr int kDb = D / 32;     // output blocks of 32 dims
  constexpr int kNv = D / 64;     // V units (8 slots of one dim) a thread stages per tile
  extern __shared__ uint4 lds_all[];
  Tile<D>* const tiles = reinterpret_cast<Tile<D>*>(lds_all);
  // Runs of rows whose result holds NaN or Inf, for the scalar body at the end: where in the sequence, and which rows. (With more
  // of them than there is room for, everything the workgroup did is done again.)
  __shared__ int n_redo, redo_at[kMaxRedo];
  __shared__ uint32_t redo_rows[kMaxRedo][kRows / 32];
  const int tid = threadIdx.x, lane = tid & 63, wave = uni(tid >> 6);
  __shared__ float2 freq[D / 2];  // {hi, lo}: indexed per lane, which the kernel arguments are too slow for
  if (tid < D / 2) freq[tid] = make_float2(a.freq_hi[tid], a.freq_lo[tid]);
  const int l32 = lane & 31, half = lane >> 5;
  const int G = a.G, Hkv = a.Hkv;
  const int hk = (int)(blockIdx.x % (unsigned)Hkv), w = (int)(blockIdx.x / (unsigned)Hkv), n_w = (int)(gridDim.x / (unsigned)Hkv);

  // ---- the head's work: for every request its row tiles, for each of those its KV tiles (at least one), in this order;
  // cum[b] = KV tiles before request b. The workgroups of the head cut the sequence into equal runs. ----
  __shared__ int cum[kMaxRequests + 1];
  auto q_first = [&](int r) { return r <= 0 ? 0 : r >= a.B ? a.n_q : min(max(a.cu_q_lens[r], 0), a.n_q); };
  auto kv_tiles = [&](int len) { return max((min(len, a.kv_tiles * kTile) + kTile - 1) / kTile, 1); };
  if (wave == 0) {
    int carry = 0;
    for (int r0 = 0; r0 < a.B; r0 += 64) {
      const int r = r0 + lane;
      int x = 0;
      if (r < a.B) x = (int)(((long)max(q_first(r + 1) - q_first(r), 0) * G + kRows - 1) / kRows) * kv_tiles(a.kv_lens[r]);
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const int y = __shfl_up(x, o);
        if (lane >= o) x += y;
      }
      if (r < a.B) cum[r + 1] = carry + x;
      carry += __shfl(x, 63);
    }
    if (lane == 0) cum[0] = 0;
  }
  __syncthreads();
  const int total = uni(cum[a.B]);
  const int chunk = max((total + n_w - 1) / n_w, a.blocks_per_split);  // (blocks_per_split: the least run, in tiles)
  const int run_end = min((w + 1) * chunk, total);
  int at = w * chunk, b = 0;
  {  // largest b with cum[b] <= at
    int hi = a.B;
    while (hi - b > 1) {
      const int mid = (b + hi) >> 1;
      if (uni(cum[mid]) <= at) b = mid; else hi = mid;
    }
  }
  struct Segment {
    int L, q_begin, t_first, n_seg, split, n_parts;
    long n_rows, row0;
  };
  auto segment = [&](int pos, int& r) __attribute__((always_inline)) {  // what lies at `pos` of the sequence; r: request at or before it
    while (uni(cum[r + 1]) <= pos) ++r;
    Segment s;
    s.L = uni(a.kv_lens[r]);
    s.q_begin = uni(q_first(r));
    s.n_rows = (long)(uni(q_first(r + 1)) - s.q_begin) * G;
    const int T = kv_tiles(s.L), seq0 = uni(cum[r]), rt = (pos - seq0) / T;
    s.t_first = pos - seq0 - rt * T;
    s.n_seg = min(run_end - pos, T - s.t_first);
    s.row0 = (long)rt * kRows;
    const int p0 = seq0 + rt * T;                        // the row tile's first place in the sequence
    s.split = w - p0 / chunk;                            // this piece of the row tile,
    s.n_parts = (p0 + T - 1) / chunk - p0 / chunk + 1;   // of how many
    return s;
  };
  if (tid == 0) n_redo = 0;
  while (at < run_end) {
    const Segment sg = segment(at, b);
    const int L = sg.L, q_begin = sg.q_begin, split = sg.split, n_parts = sg.n_parts, at_now = at;
    const long n_rows = sg.n_rows, row0 = sg.row0;
    at += sg.n_seg;

    // ---- this lane's query row and its rotated query: B operands, k-step ks: dims 16 ks + 8 half + e ----
    const long row = row0 + wave * 32 + l32;
    const bool row_ok = row < n_rows;
    const int tok = q_begin + (int)((row_ok ? row : row0) / G), g = (int)((row_ok ? row : row0) % G);
    const int pos_q = a.q_positions[tok];
    const size_t out_row = (size_t)tok * a.Hq + (size_t)hk * G + g;
    Frag qh[kKs], ql[kKs];
    {
      const uint4* q4 = reinterpret_cast<const uint4*>(a.q) + out_row * (D / 8);
      const float qs = row_ok ? a.qk_scale_log2 : 0.f;
      auto rotate = [&](float x0, float x1, int i, float& y0, float& y1) __attribute__((always_inline)) {
        const float t = turns_frac((float)pos_q, freq[i].x, freq[i].y);
        const float c = __builtin_amdgcn_cosf(t), s = __builtin_amdgcn_sinf(t);
        y0 = (x0 * c - x1 * s) * qs;
        y1 = (x1 * c + x0 * s) * qs;
      };
      if constexpr (!kIL) {
#pragma unroll
        for (int ks = 0; ks < kKs / 2; ++ks) {
          Raw8<false> r0, r1;
          r0.r = q4[2 * ks + half];
          r1.r = q4[2 * (ks + kKs / 2) + half];
          float x0[8], x1[8];
          widen8<false>(r0, x0);
          widen8<false>(r1, x1);
#pragma unroll
          for (int e = 0; e < 8; ++e) rotate(x0[e], x1[e], 16 * ks + 8 * half + e, x0[e], x1[e]);
#pragma unroll
          for (int w = 0; w < 4; ++w) {
            split2(x0[2 * w], x0[2 * w + 1], qh[ks].w[w], ql[ks].w[w]);
            split2(x1[2 * w], x1[2 * w + 1], qh[ks + kKs / 2].w[w], ql[ks + kKs / 2].w[w]);
          }
        }
      } else {
#pragma unroll
        for (int ks = 0; ks < kKs; ++ks) {
          Raw8<false> r;
          r.r = q4[2 * ks + half];
          float x[8];
          widen8<false>(r, x);
#pragma unroll
          for (int w = 0; w < 4; ++w) {
            float y0, y1;
            rotate(x[2 * w], x[2 * w + 1], 8 * ks + 4 * half + w, y0, y1);
            split2(y0, y1, qh[ks].w[w], ql[ks].w[w]);
          }
        }
      }
    }

    // ---- positions of the wave's rows, KV range of the workgroup ----
    int wpos_min = row_ok ? pos_q : 0x7fffffff, wpos_max = row_ok ? pos_q : (int)0x80000000;
#pragma unroll
    for (int o = 16; o; o >>= 1) {
      wpos_min = min(wpos_min, __shfl_xor(wpos_min, o));
      wpos_max = max(wpos_max, __shfl_xor(wpos_max, o));
    }
    wpos_min = uni(wpos_min);
    wpos_max = uni(wpos_max);
    const int n_begin = sg.t_first * kTile;
    int n_end = min(L, (sg.t_first + sg.n_seg) * kTile);
    if (!a.block_positions) {  // slots are their own positions: nothing past the last query token is visible
      int pmax = (int)0x80000000;
      const int t_last = q_begin + (int)((min(row0 + kRows, n_rows) - 1) / G);
      for (int t = q_begin + (int)(row0 / G) + lane; t <= t_last; t += 64) pmax = max(pmax, a.q_positions[t]);
#pragma unroll
      for (int o = 32; o; o >>= 1) pmax = max(pmax, __shfl_xor(pmax, o));
      n_end = min(n_end, max(uni(pmax), -1) + 1);
    }
    const int n_tiles = n_end > n_begin ? (n_end - n_begin + kTile - 1) / kTile : 0;

    // ---- what the groups of 16 slots are: lane i of a window holds group 64 win + i of the split ----
    struct Win {
      int page, pos;
      uint32_t valid;
      float ksc, vsc;
    };
    const size_t bt_row = (size_t)b * a.max_blocks;
    auto win_load = [&](Win& w, int win) __attribute__((always_inline)) {
      const int n = n_begin + (64 * win + lane) * 16;      // first slot of the group
      const int j = min(n, L - 1) / P, off = n % P;
      w.page = max(min(a.block_tables[bt_row + j], a.num_pages - 1), 0);  // a corrupt id reads a wrong page, never faults
      w.pos = a.block_positions ? a.block_positions[bt_row + j] + off : n;
      uint32_t v = a.block_valid_mask ? (a.block_valid_mask[bt_row + j] >> off) & 0xffffu : 0xffffu;
      const int left = n_end - n;
      w.valid = left <= 0 ? 0u : left >= 16 ? v : v & ((1u << left) - 1u);
      w.ksc = w.vsc = 1.f;
      if constexpr (kFp8) {
        w.ksc = a.k_scales[w.page];
        w.vsc = a.v_scales[w.page];
      }
    };
    Win cur;
    int win = 0;

    // ---- staging: thread = (slot `lane`, chunk `wave`) of K, and kNv units of V ----
    float fh[8], fl[8];  // wave-uniform
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const int i = min(8 * wave + j, D / 2 - 1);
      fh[j] = a.freq_hi[i];
      fl[j] = a.freq_lo[i];
    }
    struct Staged {
      Raw8<kFp8> k[2], v[kNv];
      int page[4], pos[4];
      uint32_t valid[4];
      float ksc[4], vsc[4];
    } st;
    auto pick = [](int i, auto x0, auto x1, auto x2, auto x3) __attribute__((always_inline)) {
      const auto a01 = i == 0 ? x0 : x1, a23 = i == 2 ? x2 : x3;
      return i < 2 ? a01 : a23;
    };
    const int grp_of_slot = lane >> 4;
    using RawT = decltype(Raw8<kFp8>::r);
    const RawT* kpages = reinterpret_cast<const RawT*>(a.k_pages);
    const RawT* vpages = reinterpret_cast<const RawT*>(a.v_pages);
    const int c0 = kIL ? 2 * wave : wave, c1 = kIL ? 2 * wave + 1 : wave + kCh;
    auto k_unit = [&](int pg, int c) __attribute__((always_inline)) {
      const int s = lane & (P - 1);
      if constexpr (kFp8) return (((size_t)pg * Hkv + hk) * (D / 16 * P) + (size_t)(c >> 1) * P + s) * 2 + (c & 1);
      else return ((size_t)pg * Hkv + hk) * (D / 8 * P) + (size_t)c * P + s;
    };
    // V unit u of a tile: where it lies in its page row, which group and half it is
    constexpr int kUpd = P / 8;  // units per dim of a page
    auto v_place = [&](int i, int& pg_grp, int& rem, int& grp, int& dim, int& hf) __attribute__((always_inline)) {
      const int u = tid + kThreads * i;
      pg_grp = (wave * 64 + kThreads * i) / (D * kUpd) * (P / 16);   // first group of the unit's page (wave-uniform)
      rem = u % (D * kUpd);
      dim = rem / kUpd;
      const int q = rem % kUpd;
      grp = pg_grp + (q >> 1);
      hf = q & 1;
    };
    auto load_tile = [&](int t) __attribute__((always_inline)) {  // non-decreasing t
      if ((t >> 4) != win) {
        ++win;
        win_load(cur, win);  // (a wait every 16 tiles; the window after it in registers as well would spill)
      }
      const int l0 = (4 * t) & 63;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        st.page[i] = __builtin_amdgcn_readlane(cur.page, l0 + i);
        st.pos[i] = __builtin_amdgcn_readlane(cur.pos, l0 + i);
        st.valid[i] = (uint32_t)__builtin_amdgcn_readlane((int)cur.valid, l0 + i);
        if constexpr (kFp8) {
          st.ksc[i] = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(cur.ksc), l0 + i));
          st.vsc[i] = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(cur.vsc), l0 + i));
        }
      }
      if (kCh == 8 || wave < kCh) {
        const int pg = pick(grp_of_slot, st.page[0], st.page[1], st.page[2], st.page[3]);
        st.k[0].r = kpages[k_unit(pg, c0)];
        st.k[1].r = kpages[k_unit(pg, c1)];
      }
#pragma unroll
      for (int i = 0; i < kNv; ++i) {
        int pg_grp, rem, grp, dim, hf;
        v_place(i, pg_grp, rem, grp, dim, hf);
        const int pg = pick(pg_grp, st.page[0], st.page[1], st.page[2], st.page[3]);
        st.v[i].r = vpages[((size_t)pg * Hkv + hk) * (D * kUpd) + rem];
      }
    };
    auto stage_tile = [&](int buf) __attribute__((always_inline)) {
      Tile<D>& T = tiles[buf];
      if (kCh == 8 || wave < kCh) {
        const float pos = (float)(pick(grp_of_slot, st.pos[0], st.pos[1], st.pos[2], st.pos[3]) + (lane & 15));
        const float ksc = kFp8 ? pick(grp_of_slot, st.ksc[0], st.ksc[1], st.ksc[2], st.ksc[3]) : 1.f;
        float x0[8], x1[8];
        widen8<kFp8>(st.k[0], x0);
        widen8<kFp8>(st.k[1], x1);
        Frag h0, l0, h1, l1;
        auto rot = [&](float x, float y, int j, float& u, float& v) __attribute__((always_inline)) {
          const float tr = turns_frac(pos, fh[j], fl[j]);
          float c = __builtin_amdgcn_cosf(tr), s = __builtin_amdgcn_sinf(tr);
          if constexpr (kFp8) {
            c *= ksc;
            s *= ksc;
          }
          u = x * c - y * s;
          v = y * c + x * s;
        };
#pragma unroll
        for (int w = 0; w < 4; ++w) {
          if constexpr (kIL) {
            float u, v;
            rot(x0[2 * w], x0[2 * w + 1], w, u, v);
            split2(u, v, h0.w[w], l0.w[w]);
            rot(x1[2 * w], x1[2 * w + 1], 4 + w, u, v);
            split2(u, v, h1.w[w], l1.w[w]);
          } else {
            float u0, v0, u1, v1;
            rot(x0[2 * w], x1[2 * w], 2 * w, u0, v0);
            rot(x0[2 * w + 1], x1[2 * w + 1], 2 * w + 1, u1, v1);
            split2(u0, u1, h0.w[w], l0.w[w]);
            split2(v0, v1, h1.w[w], l1.w[w]);
          }
        }
        T.khi[c0 * kTile + lane] = h0.u;
        T.klo[c0 * kTile + lane] = l0.u;
        T.khi[c1 * kTile + lane] = h1.u;
        T.klo[c1 * kTile + lane] = l1.u;
      }
#pragma unroll
      for (int i = 0; i < kNv; ++i) {
        int pg_grp, rem, grp, dim, hf;
        v_place(i, pg_grp, rem, grp, dim, hf);
        Frag x = bf16_of8<kFp8>(st.v[i]);
        uint32_t keep = pick(grp, st.valid[0], st.valid[1], st.valid[2], st.valid[3]);
        keep = (keep >> (8 * hf)) & 0xffu;
        if (keep != 0xffu) mask8(x, keep);
        T.v[(grp * D + dim) * 2 + (hf ^ ((dim >> 3) & 1))] = x.u;
      }
      if (tid < 4) {
        T.pos[tid] = pick(tid, st.pos[0], st.pos[1], st.pos[2], st.pos[3]);
        T.valid[tid] = pick(tid, st.valid[0], st.valid[1], st.valid[2], st.valid[3]);
        if constexpr (kFp8) T.vsc[tid] = pick(tid, st.vsc[0], st.vsc[1], st.vsc[2], st.vsc[3]);
      }
    };

    floatx16 o[kDb];
#pragma unroll
    for (int db = 0; db < kDb; ++db)
#pragma unroll
      for (int e = 0; e < 16; ++e) o[db][e] = 0.f;
    // Reference maximum of the row (log2 units), -inf until the row has seen a slot; rows that do not exist (zero query)
    // start at 0 so that they never ask for attention.
    float m_run = row_ok ? -INFINITY : 0.f, l_part = 0.f, negm = 0.f;

    // Matrix row m of a 32-slot block holds slot (m & 16) + 8 * bit2(m) + 4 * bit3(m) + (m & 3): a lane of the score tile then
    // owns, in accumulator order, slots 8 half .. 8 half + 7 of the block's first group of 16 and of its second.
    const int k_read = (l32 & 16) + ((l32 & 4) << 1) + ((l32 & 8) >> 1) + (l32 & 3);
    const bool wave_idle = row0 + wave * 32 >= n_rows;

    auto tile_step = [&](int buf) __attribute__((always_inline)) {
      const Tile<D>& T = tiles[buf];
#pragma unroll 1
      for (int sb = 0; sb < 2; ++sb) {
        const int ps0 = uni(T.pos[2 * sb]), ps1 = uni(T.pos[2 * sb + 1]);
        const uint32_t vd0 = (uint32_t)uni((int)T.valid[2 * sb]), vd1 = (uint32_t)uni((int)T.valid[2 * sb + 1]);
        if ((vd0 | vd1) == 0 || (min(ps0, ps1) > wpos_max)) continue;  // nothing here is visible to any of the wave's rows
        const bool need_mask = (vd0 & vd1) != 0xffffu || max(ps0, ps1) + 15 > wpos_min;
        constexpr int kRing = 4;
        Frag ring[kRing];
        const uint4* kh = T.khi + half * kTile + k_read + 32 * sb;
        const uint4* kl = T.klo + half * kTile + k_read + 32 * sb;
        const uint4* vt = T.v + 4 * sb * D + l32 * 2 + (half ^ ((l32 >> 3) & 1));
        // operands in the order they are used: head and remainder of K for each k-step, then V of the two groups
        auto operand = [&](int j) __attribute__((always_inline)) {
          if (j < 2 * kKs) return (j & 1 ? kl : kh)[2 * (j >> 1) * kTile];
          const int jj = j - 2 * kKs;
          return vt[((jj / kDb) * D + 32 * (jj % kDb)) * 2];
        };
        constexpr int kOps = 2 * kKs + 2 * kDb;
#pragma unroll
        for (int i = 0; i < kRing; ++i) ring[i].u = operand(i);
        floatx16 sc;
        {
          float nm = negm;
          asm volatile("" : "+v"(nm));
#pragma unroll
          for (int e = 0; e < 16; ++e) sc[e] = nm;
        }
#pragma unroll
        for (int j = 0; j < 2 * kKs; ++j) {
          const int ks = j >> 1;
          sc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ring[j % kRing].v, qh[ks].v, sc, 0, 0, 0);
          if (!(j & 1)) sc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ring[j % kRing].v, ql[ks].v, sc, 0, 0, 0);
          ring[j % kRing].u = operand(j + kRing);
        }
        if (need_mask) {
#pragma unroll
          for (int e = 0; e < 16; ++e) {
            const int s = 8 * half + (e & 7);
            const bool see = (((e < 8 ? vd0 : vd1) >> s) & 1u) && (e < 8 ? ps0 : ps1) + s <= pos_q;
            if (!see) sc[e] = -INFINITY;
          }
        }
        float p[16];
        float psum = 0.f;
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          p[e] = __builtin_amdgcn_exp2f(sc[e]);
          psum += p[e];
        }
        if (__any(!(psum <= kBig) || m_run == -INFINITY)) {
          float mx = sc[0];
#pragma unroll
          for (int e = 1; e < 16; ++e) mx = fmaxf(mx, sc[e]);
          const uint32_t u = __float_as_uint(mx);
          const auto sw = __builtin_amdgcn_permlane32_swap(u, u, false, false);
          const float mrow = fmaxf(__uint_as_float(sw[0]), __uint_as_float(sw[1]));  // relative to the old reference
          if (mrow > -INFINITY) {
            const bool first = m_run == -INFINITY;
            const float delta = first ? mrow : fmaxf(mrow, 0.f);
            const float alpha = first ? 1.f : __builtin_amdgcn_exp2f(-delta);
            m_run = (first ? 0.f : m_run) + delta;
            l_part *= alpha;
#pragma unroll
            for (int db = 0; db < kDb; ++db)
#pragma unroll
              for (int e = 0; e < 16; ++e) o[db][e] *= alpha;
            negm = -m_run;
            psum = 0.f;
#pragma unroll
            for (int e = 0; e < 16; ++e) {
              p[e] = __builtin_amdgcn_exp2f(sc[e] - delta);
              psum += p[e];
            }
          }
        }
        l_part += psum;
        if constexpr (kFp8) {
          const float vs0 = uni_f(T.vsc[2 * sb]), vs1 = uni_f(T.vsc[2 * sb + 1]);
#pragma unroll
          for (int e = 0; e < 16; ++e) p[e] *= e < 8 ? vs0 : vs1;
          if (need_mask) {  // the scale of a page that nothing of takes part may be anything
#pragma unroll
            for (int e = 0; e < 16; ++e)
              if (sc[e] == -INFINITY) p[e] = 0.f;
          }
        }
        Frag ph[2], pl[2];  // group gg of the block: k index e -> slot 8 half + e
#pragma unroll
        for (int gg = 0; gg < 2; ++gg)
#pragma unroll
          for (int w = 0; w < 4; ++w) split2(p[8 * gg + 2 * w], p[8 * gg + 2 * w + 1], ph[gg].w[w], pl[gg].w[w]);
#pragma unroll
        for (int i = 0; i < 2 * kDb; ++i) {
          const int j = 2 * kKs + i;
          o[i % kDb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ring[j % kRing].v, ph[i / kDb].v, o[i % kDb], 0, 0, 0);
          o[i % kDb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ring[j % kRing].v, pl[i / kDb].v, o[i % kDb], 0, 0, 0);
          if (j + kRing < kOps) ring[j % kRing].u = operand(j + kRing);
        }
      }
    };

    // Two groups of waves run the same sequence half a turn apart (one stages the next tile before the turn's barrier, the
    // other after it), so that the matrix segments of one fall on the vector segments of the other. Staging is unconditional:
    // past the last tile it repeats the last one into a buffer nobody reads.
    const int grp = wave >> 2, t_last = n_tiles - 1;
    if (n_tiles > 0) {
      win_load(cur, 0);
      load_tile(0);
      stage_tile(0);
      load_tile(min(1, t_last));
      lds_barrier();
      int bi = 0;
      for (int t = 0; t < n_tiles; ++t) {
        const int bn = bi + 1 == kNBuf ? 0 : bi + 1;
        if (grp) lds_barrier();
        stage_tile(bn);
        load_tile(min(t + 2, t_last));
        if (!grp) lds_barrier();
        if (!wave_idle) tile_step(bi);
        bi = bn;
      }
    }

    // ---- normalise and store: lane (row l32, half) holds dims 32 db + 8 blk + 4 half + e of its row ----
    const uint32_t u = __float_as_uint(l_part);
    const auto sw = __builtin_amdgcn_permlane32_swap(u, u, false, false);
    const float l_tot = __uint_as_float(sw[0]) + __uint_as_float(sw[1]);
    float total = l_tot;  // NaN or Inf if the sum or some accumulator is (or if their sum overflows: computed again for nothing)
#pragma unroll
    for (int db = 0; db < kDb; ++db)
#pragma unroll
      for (int e = 0; e < 16; ++e) total += o[db][e];
    const bool odd = row_ok && !(fabsf(total) < INFINITY);
    if (row_ok) {
      if (half == 0 && split == 0) a.part_meta[out_row] = n_parts;  // for the merge
      if (n_parts == 1) {
        const float inv = l_tot != 0.f ? 1.f / l_tot : 0.f;
        uint2* dst = reinterpret_cast<uint2*>(reinterpret_cast<uint16_t*>(a.out) + out_row * D);
#pragma unroll
        for (int db = 0; db < kDb; ++db)
#pragma unroll
          for (int blk = 0; blk < 4; ++blk) {
            uint2 w;
            w.x = pack2_bf16(o[db][4 * blk] * inv, o[db][4 * blk + 1] * inv);
            w.y = pack2_bf16(o[db][4 * blk + 2] * inv, o[db][4 * blk + 3] * inv);
            dst[(32 * db + 8 * blk + 4 * half) / 4] = w;
          }
      } else {
        const size_t r = out_row * a.n_splits + split;
        if (half == 0) {
          a.part_ml[2 * r] = m_run;
          a.part_ml[2 * r + 1] = l_tot;
        }
        float4* dst = reinterpret_cast<float4*>(a.part_o + r * D);
#pragma unroll
        for (int db = 0; db < kDb; ++db)
#pragma unroll
          for (int blk = 0; blk < 4; ++blk)
            dst[(32 * db + 8 * blk + 4 * half) / 4] =
                make_float4(o[db][4 * blk], o[db][4 * blk + 1], o[db][4 * blk + 2], o[db][4 * blk + 3]);
      }
    }

    if (__syncthreads_or(odd ? 1 : 0)) {
      const unsigned long long rows = __ballot(odd);  // both halves of the wave report their share of a row
      if (n_redo < kMaxRedo && lane == 0) redo_rows[n_redo][wave] = (uint32_t)(rows | (rows >> 32));
      __syncthreads();
      if (tid == 0) {
        if (n_redo < kMaxRedo) redo_at[n_redo] = at_now;
        ++n_redo;
      }
      __syncthreads();
    }
  }

  // ---- tokens with such a row once more, scalar (those of a token's heads that the row tile holds) ----
  __syncthreads();
  const int n_list = n_redo;
  if (n_list == 0) return;
  int next = w * chunk;
  b = 0;
  for (int i = 0; n_list <= kMaxRedo ? i < n_list : next < run_end; ++i) {
    const int pos = n_list <= kMaxRedo ? redo_at[i] : next;
    const Segment sg = segment(pos, b);
    next = pos + sg.n_seg;
    const int n_begin = sg.t_first * kTile, n_end = min(sg.L, (sg.t_first + sg.n_seg) * kTile);
    const long row_end = min(sg.row0 + kRows, sg.n_rows);
    for (int t = (int)(sg.row0 / G); t <= (int)((row_end - 1) / G); ++t) {
      const int r0 = (int)max((long)t * G - sg.row0, 0L), r1 = (int)(min((long)(t + 1) * G, row_end) - sg.row0);  // rows of the tile
      bool any = n_list > kMaxRedo;
      for (int r = r0; r < r1 && !any; ++r) any = (redo_rows[i][r >> 5] >> (r & 31)) & 1u;
      if (!any) continue;
      const int g0 = (int)(sg.row0 + r0 - (long)t * G);
      scalar_attend_all<kFp8 ? MEPIC_F8E4M3 : MEPIC_BF16, kThreads>(a, *reinterpret_cast<ScalarLds<4, kThreads>*>(lds_all),
                                                                    sg.q_begin + t, b, hk, g0, g0 + r1 - r0, n_begin, n_end,
                                                                    sg.split, sg.n_parts == 1);
    }
    __syncthreads();
  }
}

int prefill_split_workgroups_per_head(int Hkv) { return max(device_compute_units() / Hkv, 1); }

template <bool kFp8, int D, int P, bool kIL>
hipError_t launch_one(const AttnArgs& a, hipStream_t s) {
  static std::atomic<uint64_t> asked{0};
  const hipError_t status = allow_lds(reinterpret_cast<const void*>(&prefill_split_kernel<kFp8, D, P, kIL>), kNBuf * sizeof(Tile<D>), asked);
  if (status != hipSuccess) return status;
  const unsigned grid = (unsigned)a.Hkv * (unsigned)prefill_split_workgroups_per_head(a.Hkv);
  hipLaunchKernelGGL((prefill_split_kernel<kFp8, D, P, kIL>), dim3(grid), dim3(kThreads), kNBuf * sizeof(Tile<D>), s, a);
  return hipGetLastError();
}

// Merge the pieces of a query row (one piece: the kernel has written the row itself). There are many rows of few pieces, so
// what counts is rows in flight: one wave each (28 672 rows, mostly of two to three pieces: 15.7 us with two waves, 11.5 with one).
template <int D>
__global__ __launch_bounds__(64) void combine_pieces_kernel(const AttnArgs a) {
  const int row = blockIdx.x, ns = a.part_meta[row];
  if (ns <= 1) return;
  merge_row<D, 64>(a.part_ml + (size_t)row * a.n_splits * 2, a.part_o + (size_t)row * a.n_splits * D, ns, ns,
                   reinterpret_cast<uint16_t*>(a.out) + (size_t)row * D);
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

hipError_t launch_prefill_split(const AttnArgs& a, hipStream_t s) {
  const hipError_t e = a.kv_dtype == MEPIC_F8E4M3 ? launch_kv<true>(a, s) : launch_kv<false>(a, s);
  if (e != hipSuccess) return e;
  if (a.timing_stop) (void)hipEventRecord(reinterpret_cast<hipEvent_t>(a.timing_stop), s);
  const dim3 grid(a.n_q * a.Hq), block(64);
  if (a.D == 128) hipLaunchKernelGGL((combine_pieces_kernel<128>), grid, block, 0, s, a);
  else hipLaunchKernelGGL((combine_pieces_kernel<64>), grid, block, 0, s, a);
  return hipGetLastError();
}

// How the call is cut. A row tile is cut where the workgroups' runs meet, so with W workgroups per head and R row tiles into
// about W / R + 1 pieces; there is room for twice that, for requests longer than the mean. The room is a row's (max_pieces partials
// of D + 2 floats each: 8 of them, 119 MB, on the fp8 call above, where most rows come in two or three), and a run is at least
// what keeps the longest request within it: one request of 32 K slots among 63 of 1 K on 4 KV heads makes runs of 171 tiles where
// an even share is 24, and leaves 55 of a head's 64 workgroups idle. B or the work may be too much for the kernel's prefix
// sums: then max_pieces is 0.
void prefill_split_plan(int B, int Hkv, long n_rows, int max_kv_len, int* kv_tiles, int* min_run, int* max_pieces) {
  const int W = prefill_split_workgroups_per_head(Hkv), T = max((max_kv_len + kTile - 1) / kTile, 1);
  const long R = max((n_rows + kRows - 1) / kRows, (long)B);
  int pieces = (int)(2 * ((W + R - 1) / max(R, 1L)) + 1);
  if (pieces > T) pieces = T;
  *kv_tiles = T;
  *min_run = (T + pieces - 1) / pieces;
  *max_pieces = B <= kMaxRequests && (n_rows / kRows + B) * T < (1L << 30) ? (T - 1 + *min_run - 1) / *min_run + 1 : 0;
}

}  // namespace mepic
