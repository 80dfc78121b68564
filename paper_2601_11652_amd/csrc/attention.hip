// Ragged multi-query causal attention over the paged KV cache (the attention inside
// Sec. 4.5's batched one-step verification): request i's (gamma_i + 1) * G query rows of
// kv head h attend to keys 0 .. ctx_len_i + j (row j), read page by page through the
// request's block table.
//
// bf16 path, a work item being (request, kv head, group of 32, 48 or 64 query rows, token
// range) and a wave running one or several of them.  Per 32 tokens (a page pair) the wave
// computes S^T = K Q^T and O^T += V^T P^T with v_mfma_f32_16x16x32_bf16.  Computing the transposed products keeps every query row
// in one lane column (lane % 16), so the online softmax needs only two cross-row steps
// (VALU lane swaps),
// and the probabilities leave the first product in exactly the register order the second
// one consumes.  The token order inside the pair is chosen (through the K and V page
// layouts) so that lane group g = lane / 16 holds tokens 8g .. 8g + 7 of the pair, all in
// one page: the V operand of each lane is then one 16-byte load, and the K operand of
// each product row one 16-byte load.  Partials of a context cut into several ranges are
// combined afterwards in fixed order.
#include <type_traits>

#include "common.h"
#include "kernels.h"

namespace wisp {

// Bound by HBM for decode batches and by its own serial chain (products, softmax, products)
// for prompts.  Wave w of the launch runs items first[w] .. first[w + 1] - 1 one after
// another (item w alone without that list), 4 waves per workgroup.  A SIMD holds two waves of 32
// query rows and one of 48 or 64; at head_dim 64 four, two and one.  The loads run one page pair ahead of the products, across items, so 16 KiB per wave stay in
// flight and what an item costs besides its pairs (descriptor, block ids, query rows) loads
// while the one before is computed; a context that one wave covers alone is written without
// a combine.  Measured per layer, against one wave per item of at most 32 pairs with the query
// rows in registers: 256 requests of 1-8k tokens 692 -> 610 us (6.0 TB/s; random 4 KiB pages
// alone stream at 6.6), 128 requests of 0.25-32k 661 -> 590 us; 32 requests of
// 0.5-2k (one item per wave either way) 30 us in both; a prompt of 4096 rows with its combine
// 511 -> 364 us.
template <int HD, int RB>
__global__ __launch_bounds__(256, RB == 2 ? 2 : 1) void attn_bf16_kernel(StepDesc d, const AttnItem *__restrict__ items,
                                                           const int32_t *__restrict__ first, int n_waves,
                                                           const uint16_t *__restrict__ q,
                                                           const uint16_t *__restrict__ kp,
                                                           const uint16_t *__restrict__ vp,
                                                           float *__restrict__ part_o,
                                                           float *__restrict__ part_ml,
                                                           uint16_t *__restrict__ out, bool packed, int out_K,
                                                           bool q16, int nq, int nkv, float scale) {
  constexpr int ROWS = 16 * RB; // query rows of an item
  constexpr int KC = HD / 32;   // 32-wide chunks of the QK^T contraction
  constexpr int MB = HD / 16;   // 16-wide blocks of the output head dimension
  // everything about an item is wave-uniform: kept in scalar registers, so branches and loop
  // bounds are scalar
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  // workgroups are dealt to the 8 XCDs in turn: consecutive waves on one XCD, whose L2 then
  // holds the one or two kv heads that a prompt's row groups read over and over
  const int per_xcd = (gridDim.x + 7) / 8;
  const int wid = ((int)(blockIdx.x % 8u) * per_xcd + (int)(blockIdx.x / 8u)) * 4 + wave;
  if (wid >= n_waves) return;
  auto uni = [](int x) { return __builtin_amdgcn_readfirstlane(x); };
  int it = first ? uni(first[wid]) : wid;             // no list: one item per wave
  const int it_end = first ? uni(first[wid + 1]) : wid + 1;
  if (it >= it_end) return;
  const int G = nq / nkv;
  const int lc = lane & 15, lg = lane >> 4;
  const int page_elems = kPage * HD;
  // the item's query rows in operand order: in LDS (read back per pair), as in registers they
  // would leave no room for a second wave per SIMD, or for 64 rows.  Each wave uses its own
  // part, one buffer for the item being computed and one for the next.
  __shared__ __attribute__((aligned(1024))) uint4 qs[4][2][RB][KC][64];

  struct Item {   // an AttnItem and its request's figures, in scalar registers
    int req, kvh, rbg, t0, t1, ctx, row0, rows;
    bool whole;
  };
  // two dependent loads: the descriptor, then the request's figures (vector loads, waited for
  // where they are first used: in a wave's later items, pairs after they were issued)
  int4 d0;
  int d_ctx, d_row0, d_nrow;
  auto fetch = [&](int item) __attribute__((always_inline)) {
    d0 = *reinterpret_cast<const int4 *>(items + item);
  };
  auto fetched = [&](Item &a) __attribute__((always_inline)) {
    a.req = uni(d0.x);
    a.kvh = attn_kvh(uni(d0.y));
    a.rbg = attn_rbg(uni(d0.y), uni(d0.z));
    a.t0 = uni(d0.z) & ~kAttnFlags;
    a.whole = uni(d0.z) & kAttnWhole;
    a.t1 = uni(d0.w);
    d_ctx = d.ctx[d0.x];
    d_row0 = d.off[d0.x];
    d_nrow = d.nrow[d0.x];
  };
  auto complete = [&](Item &a) __attribute__((always_inline)) {
    a.ctx = uni(d_ctx);
    a.row0 = uni(d_row0);
    a.rows = uni(d_nrow) * G;
  };
  // an item's query rows into buffer b, straight into LDS (complete once any load issued later
  // has returned: the counter runs in order); through registers if q is not 16-byte aligned
  auto load_q = [&](const Item &a, int b) __attribute__((always_inline)) {
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
      const int lr = min(a.rbg * ROWS + rb * 16 + lc, a.rows - 1);   // padding rows reuse a real row
      const uint16_t *src = q + ((int64_t)(a.row0 + lr / G) * nq + a.kvh * G + lr % G) * HD + 8 * lg;
#pragma unroll
      for (int kc = 0; kc < KC; ++kc) {
        if (q16) lds_dma16(src + kc * 32, &qs[wave][b][rb][kc][0]);
        else qs[wave][b][rb][kc][lane] = ld16(src + kc * 32);
      }
    }
  };

  // A window is a run of at most 64 pages of one item; its block ids live in one register,
  // lane l holding page base + l, and are picked with readlane.
  struct Window {
    int item, req, kvh, t, end, t1, base;   // next token to load, end of the window, of the item
    int bids;                               // per lane
  };
  auto window_at = [&](int item, int req, int kvh, int t, int t1) __attribute__((always_inline)) {
    Window w;
    w.item = item;
    w.req = req;
    w.kvh = kvh;
    w.t = t;
    w.t1 = t1;
    w.end = min(t1, t + kAttnWindowPages * kPage);
    w.base = t >> 4;
    w.bids = d.page_table[(int64_t)req * d.pt_stride + min(w.base + lane, ((w.end + 15) >> 4) - 1)];
    return w;
  };

  // Per-lane operand offsets inside a page.  Row r = lane % 16 of the S product for page
  // half h (0/1) is token 16 * (r / 8) + 8 * ((r / 4) % 2) + 4 * h + r % 4 of the pair;
  // lane group g then holds probabilities of tokens 8g .. 8g + 7, which sit in page g / 2.
  const int k_off = lg * 64 + (lc & 7) * 8;           // + (kc * 2 + h) * 256
  const int v_off = (lg & 1) * 128 + lc * 8;          // + mb * 256
  const bool k_hi = lc >= 8, v_hi = lg >= 2;           // which page of the pair
  // this lane's K and V operands of the page pair at token w.t of window w.  Block ids are
  // clamped into the pool: tokens past the range's end get zero probability, and an invalid id
  // is reported.
  const uint16_t *kptr, *vptr;
  auto point = [&](const Window &w) __attribute__((always_inline)) {
    const int pg = (w.t >> 4) - w.base;
    int p0 = __builtin_amdgcn_readlane(w.bids, pg);
    int p1 = w.t + 16 < w.t1 ? __builtin_amdgcn_readlane(w.bids, pg + 1) : p0;
    if ((p0 < 0 || p0 >= d.n_blocks || p1 < 0 || p1 >= d.n_blocks) && lane == 0) flag_error(d.err, kErrBlock);
    p0 = min(max(p0, 0), d.n_blocks - 1);
    p1 = min(max(p1, 0), d.n_blocks - 1);
    const int64_t kv0 = ((int64_t)p0 * nkv + w.kvh) * page_elems;
    const int64_t kv1 = ((int64_t)p1 * nkv + w.kvh) * page_elems;
    kptr = kp + (k_hi ? kv1 : kv0) + k_off;
    vptr = vp + (v_hi ? kv1 : kv0) + v_off;
  };
  // decoding reads every K and V byte once per step: non-temporal, so the stream does not
  // evict the attention partials that the combine kernel reads next (measured: the combine
  // runs about a third faster at long contexts, the attention itself about 5 % faster)
  bf16x8_t kf[2][KC], vf[MB];
  auto load_k = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int kc = 0; kc < KC; ++kc) {
      kf[0][kc] = as_bf16x8(ld16_stream(kptr + (kc * 2) * 256));
      kf[1][kc] = as_bf16x8(ld16_stream(kptr + (kc * 2 + 1) * 256));
    }
  };
  auto load_v = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) vf[mb] = as_bf16x8(ld16_stream(vptr + mb * 256));
  };

  // the item being computed
  Item cur;
  int tp, qb = 0;   // the pair's first token; the buffer of its query rows
  int jrow[RB];
  float m_run[RB], l_run[RB];
  floatx4 o[RB][MB];
  auto begin_item = [&](const Item &a) __attribute__((always_inline)) {
    cur = a;
    tp = a.t0;
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
      jrow[rb] = min(a.rbg * ROWS + rb * 16 + lc, a.rows - 1) / G;
      m_run[rb] = -INFINITY;
      l_run[rb] = 0.f;
#pragma unroll
      for (int mb = 0; mb < MB; ++mb) o[rb][mb] = floatx4{0.f, 0.f, 0.f, 0.f};
    }
  };
  // An item that covers its group's whole context writes the group's output itself, as the
  // combine would from one partial; otherwise partials: O [item][row slot][HD]
  // (unnormalised), (m, l) [item][row slot], rows of the group only.  The stores are
  // non-temporal: they leave the caches to the loads (256 requests: 635 -> 610 us).
  auto end_item = [&](int item) __attribute__((always_inline)) {
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
      const int lr = cur.rbg * ROWS + rb * 16 + lc;
      if (lr >= cur.rows) continue;
      if (cur.whole) {
        const int64_t row = cur.row0 + jrow[rb];
        const int col = (cur.kvh * G + lr - jrow[rb] * G) * HD + 4 * lg;
        const float inv = 1.0f / l_run[rb];
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) {
          const int64_t at = packed ? packed_off(row, col + mb * 16, out_K) : row * out_K + col + mb * 16;
          uint2 v;
          v.x = pack2bf(o[rb][mb][0] * inv, o[rb][mb][1] * inv);
          v.y = pack2bf(o[rb][mb][2] * inv, o[rb][mb][3] * inv);
          *reinterpret_cast<uint2 *>(out + at) = v;
        }
        continue;
      }
      const int64_t row = (int64_t)item * ROWS + rb * 16 + lc;
#pragma unroll
      for (int mb = 0; mb < MB; ++mb)
        __builtin_nontemporal_store(o[rb][mb], reinterpret_cast<floatx4 *>(part_o + row * HD + mb * 16 + 4 * lg));
      if (lg == 0)   // m in the scaled natural-log domain: weights are exp(m - m_max)
        *reinterpret_cast<float2 *>(part_ml + row * 2) =
            make_float2(m_run[rb] == -INFINITY ? -INFINITY : m_run[rb] * scale, l_run[rb]);
    }
  };

  // Online softmax in the raw score domain: p = 2^((s - m) * c) with c = scale * log2(e),
  // one FMA and one v_exp per score.  The running maximum m of a row is raised only when
  // a score exceeds it by more than kTau / c (p then stays below 2^kTau), so the O
  // accumulators are rescaled only on the rare pairs that raise some row's maximum; the
  // result is unchanged because numerator and denominator share the same reference.
  const float c_log2 = scale * 1.4426950408889634f;
  constexpr float kTau = 8.0f;
  const float tau_raw = kTau / c_log2;

  // One turn per page pair, in three phases over all row blocks: S = K Q^T, softmax, O += V^T
  // P^T.  Each operand has one register set, reloaded for the next pair as soon as its phase is
  // over: K is in flight during the softmax and the second product, V during the first
  // product and the softmax.  (Two sets of both would leave no room for a second wave per SIMD.)
  Item next;
  fetch(it);
  fetched(next);
  Window w = window_at(it, next.req, next.kvh, next.t0, next.t1), nx = w;
  bool nx_ready = false;   // nx is the window after w
  complete(next);
  begin_item(next);
  load_q(cur, 0);
  int ahead = 0;           // the next item: 0 asked for, 1 its descriptor is here, 2 complete, q asked for
  point(w);
  load_k();
  load_v();
  fetch(min(it + 1, it_end - 1));
  while (true) {
    // K of this pair and everything older (the item's query rows) has landed
    __builtin_amdgcn_s_waitcnt((MB & 15) | (7 << 4) | (15 << 8));
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    floatx4 s[RB][2];

#pragma unroll
    for (int kc = 0; kc < KC; ++kc) {   // independent products next to each other
      bf16x8_t qf[RB];
#pragma unroll
      for (int rb = 0; rb < RB; ++rb) qf[rb] = as_bf16x8(qs[wave][qb][rb][kc][lane]);
#pragma unroll
      for (int rb = 0; rb < RB; ++rb)
#pragma unroll
        for (int h = 0; h < 2; ++h)
          s[rb][h] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[h][kc], qf[rb], kc ? s[rb][h] : floatx4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
    // Everything the next item needs is asked for during this one, before the loads of a later
    // pair: its descriptor when this one began, then its block ids and the request's figures,
    // then its query rows.  (Waiting for them at the switch: 633 instead of 610 us at 256
    // requests.)
    const bool ends = w.t + 32 >= w.end;              // the next pair opens another window
    if (it + 1 < it_end) {
      if (ahead == 1 && (tp > cur.t0 + 32 || tp + 32 >= cur.t1)) {
        complete(next);
        load_q(next, qb ^ 1);
        ahead = 2;
      }
      if (ahead == 0 && (tp > cur.t0 || ends)) {
        fetched(next);
        ahead = 1;
      }
    }
    if (!nx_ready) {
      if (w.end < w.t1) {
        nx = window_at(w.item, w.req, w.kvh, w.end, w.t1);
        nx_ready = true;
      } else if (ahead && w.item == it) {
        nx = window_at(it + 1, next.req, next.kvh, next.t0, next.t1);
        nx_ready = true;
      }
    }
    if (ends && nx_ready) {
      asm volatile("" ::: "memory");                  // a branch: a select would wait for every load
      w = nx;
      nx_ready = false;
    } else {
      w.t = min(w.t + 32, (w.end - 1) & ~31);         // past the wave's last pair: that pair once more
    }
    point(w);
    load_k();
    __builtin_amdgcn_sched_barrier(0);

    // scalar: no token of this pair lies past the range's end or any row's causal limit
    const bool unmasked = tp + 32 <= min(cur.t1, cur.ctx + 1);
    uint4 pb[RB];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
      // s[rb][h][e]: token tp + 8 * lg + 4 * h + e, query row rb * 16 + lc of the group
      if (!unmasked) {
        const int lim = min(cur.t1, cur.ctx + jrow[rb] + 1);   // causal + range end
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (tp + 8 * lg + 4 * h + e >= lim) s[rb][h][e] = -INFINITY;
      }
      float mx = fmaxf(fmaxf(fmaxf(s[rb][0][0], s[rb][0][1]), fmaxf(s[rb][0][2], s[rb][0][3])),
                       fmaxf(fmaxf(s[rb][1][0], s[rb][1][1]), fmaxf(s[rb][1][2], s[rb][1][3])));
      mx = xor32_max(xor16_max(mx));
      const bool grow = mx > m_run[rb] + tau_raw;   // false while the row has seen no token
      if (__builtin_amdgcn_ballot_w64(grow)) {      // wave-uniform: some row raises its max
        const float alpha = grow ? __builtin_amdgcn_exp2f((m_run[rb] - mx) * c_log2) : 1.0f;
        m_run[rb] = grow ? mx : m_run[rb];
        l_run[rb] *= alpha;
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) o[rb][mb] *= alpha;
      }
      const float mc = m_run[rb] == -INFINITY ? 0.f : m_run[rb] * c_log2;
      // probabilities rounded to bf16 once; the row sum adds exactly the rounded values
      uint32_t pw[4];
      float rs = 0.f;
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int e = 0; e < 4; e += 2) {
          const float p0 = __builtin_amdgcn_exp2f(__builtin_fmaf(s[rb][h][e], c_log2, -mc));
          const float p1 = __builtin_amdgcn_exp2f(__builtin_fmaf(s[rb][h][e + 1], c_log2, -mc));
          const uint32_t pk = pack2bf_rne(p0, p1);
          pw[h * 2 + e / 2] = pk;
          rs += __uint_as_float(pk << 16) + __uint_as_float(pk & 0xFFFF0000u);
        }
      rs = xor32_sum(xor16_sum(rs));
      l_run[rb] += rs;
      pb[rb] = make_uint4(pw[0], pw[1], pw[2], pw[3]);
    }

#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
#pragma unroll
      for (int mb = 0; mb < MB; ++mb)
        o[rb][mb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf[mb], as_bf16x8(pb[rb]), o[rb][mb], 0, 0, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
    load_v();
    __builtin_amdgcn_sched_barrier(0);
    tp += 32;
    if (tp >= cur.t1) {
      end_item(it);
      if (++it == it_end) break;
      if (ahead < 2) {                                // an item of one pair
        complete(next);
        load_q(next, qb ^ 1);
        __builtin_amdgcn_s_waitcnt((0 & 15) | (7 << 4) | (15 << 8));
        asm volatile("" ::: "memory");
      }
      begin_item(next);
      qb ^= 1;
      ahead = 0;
      fetch(min(it + 1, it_end - 1));
    }
  }
}

// Fixed-order combine of each group's partials: one workgroup per (request, kv head, row
// group), several where there are few groups (a lone CU takes 0.38 us per partial of 32 rows, 47
// of them 21.8 us; in 8 workgroups 11.7), one thread per (row, 8 head dims).  Pass 1 takes the maximum of the partials'
// running maxima, pass 2 adds the rescaled sums in order.  A group of at most MAXC partials
// loads everything in one round; a longer one loads its maxima 2 MAXC at a time and keeps
// two rounds of MAXC / 2 partials in flight in pass 2 (B = 4, 22 per group: 14.6 -> 10.2 us
// per launch).  Writes the bf16 attention output of each (row, q head) into the
// O-projection's input layout.
constexpr int kCombineThreads = 512, kCombineBlocks = 512;
template <int HD, int MAXC, bool LONG>
__global__ __launch_bounds__(kCombineThreads) void attn_combine_kernel(StepDesc d, const AttnGroup *__restrict__ groups,
                                                           int ROWS, const float *__restrict__ part_o,
                                                           const float *__restrict__ part_ml,
                                                           uint16_t *__restrict__ out, bool packed, int out_K,
                                                           int nq, int nkv) {
  constexpr int CH = HD / 8;
  const AttnGroup g = groups[blockIdx.x];
  const int G = nq / nkv;
  const int rows = d.nrow[g.req] * G;
  const int n = g.n_items & ~kAttnHighGroup;
  const int kvh = attn_kvh(g.kvh_rbg), lr0 = attn_rbg(g.kvh_rbg, g.n_items != n ? kAttnHighItem : 0) * ROWS;
  const int nr = min(ROWS, rows - lr0);
  for (int u = blockIdx.y * blockDim.x + threadIdx.x; u < nr * CH; u += gridDim.y * blockDim.x) {
    const int rr = u / CH, c0 = (u % CH) * 8;   // neighbouring threads: dims of one row
    // partial c of this row; past the last: the last (in range, not used)
    auto slot = [&](int c) { return ((int64_t)g.first_item + min(c, n - 1)) * ROWS + rr; };
    auto load8 = [&](int64_t s, float (&v)[8]) {
      const float4 a = *reinterpret_cast<const float4 *>(part_o + s * HD + c0);
      const float4 b = *reinterpret_cast<const float4 *>(part_o + s * HD + c0 + 4);
      v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w;
      v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
    };
    float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    float den = 0.f;
    float m = -INFINITY;
    if (!LONG || n <= MAXC) {
      // one round of loads: every partial's (m, l) and O values at once, the maximum taken from
      // registers; the same sums in the same order as the two-pass form below
      float2 ml[MAXC];
      float pv[MAXC][8];
#pragma unroll
      for (int c = 0; c < MAXC; ++c) {
        ml[c] = make_float2(-INFINITY, 0.f);
#pragma unroll
        for (int e = 0; e < 8; ++e) pv[c][e] = 0.f;
        if (c < n) {   // uniform: partials past the group's last are not loaded at all
          ml[c] = *reinterpret_cast<const float2 *>(part_ml + slot(c) * 2);
          load8(slot(c), pv[c]);
        }
      }
#pragma unroll
      for (int c = 0; c < MAXC; ++c)
        if (c < n) m = fmaxf(m, ml[c].x);
#pragma unroll
      for (int c = 0; c < MAXC; ++c) {
        if (c >= n || ml[c].x == -INFINITY) continue;
        const float w = expf(ml[c].x - m);
        den += ml[c].y * w;
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[e] += pv[c][e] * w;
      }
    } else {
      // a longer group (the long instance, launched when some group has more than MAXC)
      // pass 1: the group's maximum, 2 MAXC partials' m per round, all loaded before any is used
      constexpr int MC1 = 2 * MAXC;
      for (int cb = 0; cb < n; cb += MC1) {
        float mc[MC1];
#pragma unroll
        for (int c = 0; c < MC1; ++c) mc[c] = part_ml[slot(cb + c) * 2];
#pragma unroll
        for (int c = 0; c < MC1; ++c) m = cb + c < n ? fmaxf(m, mc[c]) : m;
      }
      // pass 2: the rescaled sums in order, in rounds of R = MAXC / 2 with the next round's loads
      // issued before the current round is used.  The loads are unconditional (clamped to the
      // group's last) and what lies past it is dropped by selects, so no branch separates a
      // load from its use and the waits stay exact.
      constexpr int R = MAXC / 2;
      float2 ml0[R], ml1[R];
      float pv0[R][8], pv1[R][8];
      auto load = [&](float2 (&ml)[R], float (&pv)[R][8], int cb) {
#pragma unroll
        for (int c = 0; c < R; ++c) {
          ml[c] = *reinterpret_cast<const float2 *>(part_ml + slot(cb + c) * 2);
          load8(slot(cb + c), pv[c]);
        }
      };
      auto use = [&](const float2 (&ml)[R], const float (&pv)[R][8], int cb) {
#pragma unroll
        for (int c = 0; c < R; ++c) {
          const bool ok = cb + c < n && ml[c].x != -INFINITY;
          const float w = expf(ml[c].x - m);
          den = ok ? den + ml[c].y * w : den;
#pragma unroll
          for (int e = 0; e < 8; ++e) acc[e] = ok ? acc[e] + pv[c][e] * w : acc[e];
        }
      };
      load(ml0, pv0, 0);
      for (int cb = 0; cb < n; cb += 2 * R) {
        load(ml1, pv1, cb + R);
        use(ml0, pv0, cb);
        load(ml0, pv0, cb + 2 * R);
        use(ml1, pv1, cb + R);
      }
    }
    const int lr = lr0 + rr;
    const int64_t row = d.off[g.req] + lr / G;
    const int head = kvh * G + lr % G;
    const int64_t col = (int64_t)head * HD + c0;
    uint4 w4;
    const float inv = 1.0f / den;
    w4.x = pack2bf(acc[0] * inv, acc[1] * inv);
    w4.y = pack2bf(acc[2] * inv, acc[3] * inv);
    w4.z = pack2bf(acc[4] * inv, acc[5] * inv);
    w4.w = pack2bf(acc[6] * inv, acc[7] * inv);
    const int64_t o = packed ? packed_off(row, col, out_K) : row * out_K + col;
    *reinterpret_cast<uint4 *>(out + o) = w4;
  }
}

void attention_bf16_main(const StepDesc &d, const AttnItem *items, const int32_t *first, int n_waves, int item_rows,
                         const uint16_t *q, const uint16_t *k_pool, const uint16_t *v_pool, float *part_o,
                         float *part_ml, uint16_t *out, bool out_packed, int out_K, int nq, int nkv, int hd,
                         hipStream_t s) {
  if (n_waves == 0) return;
  const float scale = 1.0f / sqrtf((float)hd);
  const bool q16 = ((uintptr_t)q & 15) == 0;
  const int blocks = ((n_waves + 3) / 4 + 7) / 8 * 8;   // whole rounds of the XCDs
  auto go = [&](auto kernel) {
    launch(kernel, blocks, 256, 0, s, d, items, first, n_waves, q, k_pool, v_pool, part_o, part_ml, out,
           out_packed, out_K, q16, nq, nkv, scale);
  };
  if (hd == 128) {
    if (item_rows == 32) go(attn_bf16_kernel<128, 2>);
    else if (item_rows == 48) go(attn_bf16_kernel<128, 3>);
    else go(attn_bf16_kernel<128, 4>);
  } else {
    if (item_rows == 32) go(attn_bf16_kernel<64, 2>);
    else if (item_rows == 48) go(attn_bf16_kernel<64, 3>);
    else go(attn_bf16_kernel<64, 4>);
  }
}

void attention_bf16_combine(const StepDesc &d, const AttnGroup *groups, int n_groups, int item_rows,
                            int max_group_chunks, const float *part_o, const float *part_ml, uint16_t *out, bool out_packed,
                            int out_K, int nq, int nkv, int hd, hipStream_t s) {
  if (n_groups == 0) return;
  constexpr int kMaxC = kAttnCombineChunks;
  const bool longer = max_group_chunks > kMaxC;
  const int units = item_rows * hd / 8;
  int threads = kCombineThreads;
  while (threads > 64 && n_groups * ((units + threads - 1) / threads) < kCombineBlocks) threads /= 2;
  const dim3 grid(n_groups, (units + threads - 1) / threads);
  auto go = [&](auto kernel) {
    launch(kernel, grid, threads, 0, s, d, groups, item_rows, part_o, part_ml, out, out_packed, out_K, nq, nkv);
  };
  if (hd == 128) go(longer ? attn_combine_kernel<128, kMaxC, true> : attn_combine_kernel<128, kMaxC, false>);
  else go(longer ? attn_combine_kernel<64, kMaxC, true> : attn_combine_kernel<64, kMaxC, false>);
}

// ---------------------------------------------------------------------------------------
// fp32 path (small models): one workgroup per (row, q head), plain VALU
// ---------------------------------------------------------------------------------------
// Bound by latency at the sizes it serves (a few rows of contexts of a hundred tokens): every
// row has its own workgroup, a thread scores one token with 16-byte loads (8 consecutive
// dims of a K page element are contiguous), and the weighted sum takes 8 consecutive tokens
// per 32 bytes of a V page, the octets spread over the threads.  (One workgroup per request and
// head, its rows in turn and one thread per output dim: 144 us per layer at 4 requests of up
// to 128 tokens.)
__device__ __forceinline__ float block_reduce_256(float v, float *sh, bool is_max) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    const float w = __shfl_xor(v, o);
    v = is_max ? fmaxf(v, w) : v + w;
  }
  __syncthreads();
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
  __syncthreads();
  return is_max ? fmaxf(fmaxf(sh[0], sh[1]), fmaxf(sh[2], sh[3])) : sh[0] + sh[1] + sh[2] + sh[3];
}

// 8 consecutive floats; V16: 16-byte aligned
template <bool V16>
__device__ __forceinline__ void load8(const float *p, float (&v)[8]) {
  if constexpr (V16) {
    const float4 a = *reinterpret_cast<const float4 *>(p), b = *reinterpret_cast<const float4 *>(p + 4);
    v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w;
    v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
  } else {
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = p[e];
  }
}

template <bool V16>
__global__ __launch_bounds__(256) void attn_f32_kernel(StepDesc d, const float *__restrict__ q,
                                                       const float *__restrict__ kp,
                                                       const float *__restrict__ vp,
                                                       float *__restrict__ out, int nq, int nkv, int hd,
                                                       float scale) {
  extern __shared__ __attribute__((aligned(16))) float sc[];   // scores, then probabilities, of the row's tokens
  __shared__ float sh[4];
  __shared__ __attribute__((aligned(16))) float qs[256];       // the row's q, later the partial sums
  const int r = blockIdx.x, hq = blockIdx.y, tid = threadIdx.x;
  const int i = d.row_req[r], kvh = hq / (nq / nkv);
  const int T = d.row_pos[r] + 1;                              // causal: keys 0 .. position
  const int32_t *pt = d.page_table + (int64_t)i * d.pt_stride;
  const int page_elems = kPage * hd;
  if (tid < hd) qs[tid] = q[((int64_t)r * nq + hq) * hd + tid];
  __syncthreads();
  float mx = -INFINITY;
  for (int t = tid; t < T; t += 256) {
    const int blk = pt[t / kPage];
    float dot = 0.f;
    if (blk >= 0 && blk < d.n_blocks) {
      const float *pg = kp + ((int64_t)blk * nkv + kvh) * page_elems;
      for (int e = 0; e < hd; e += 8) {
        float k[8];
        load8<V16>(pg + k_page_off(t % kPage, e), k);
#pragma unroll
        for (int x = 0; x < 8; ++x) dot += qs[e + x] * k[x];
      }
    } else {
      flag_error(d.err, kErrBlock);
    }
    sc[t] = dot * scale;
    mx = fmaxf(mx, sc[t]);
  }
  mx = block_reduce_256(mx, sh, true);
  float sum = 0.f;
  for (int t = tid; t < T; t += 256) {
    const float p = expf(sc[t] - mx);
    sc[t] = p;
    sum += p;
  }
  sum = block_reduce_256(sum, sh, false);   // its barriers also publish the probabilities
  const int groups = max(1, 256 / hd), g = tid / hd, e = tid % hd;   // hd <= 256
  float acc = 0.f;
  if (g < groups) {
    for (int t0 = 8 * g; t0 < T; t0 += 8 * groups) {
      const int blk = pt[t0 / kPage];
      if (blk < 0 || blk >= d.n_blocks) continue;
      float v[8];
      load8<V16>(vp + ((int64_t)blk * nkv + kvh) * page_elems + v_page_off(t0 % kPage, e), v);
#pragma unroll
      for (int x = 0; x < 8; ++x)
        if (t0 + x < T) acc += sc[t0 + x] * v[x];   // slots past the row's position may hold anything
    }
  }
  __syncthreads();
  qs[tid] = acc;
  __syncthreads();
  if (tid < hd) {
    for (int x = 1; x < groups; ++x) acc += qs[x * hd + tid];
    out[((int64_t)r * nq + hq) * hd + tid] = acc / sum;
  }
}

void attention_f32(const StepDesc &d, int M, const float *q, const float *k_pool,
                   const float *v_pool, float *out, int nq, int nkv, int hd, int max_tokens,
                   hipStream_t s) {
  const float scale = 1.0f / sqrtf((float)hd);
  const bool v16 = (((uintptr_t)k_pool | (uintptr_t)v_pool) & 15) == 0;
  launch(v16 ? attn_f32_kernel<true> : attn_f32_kernel<false>, dim3(M, nq), 256, max_tokens * sizeof(float), s, d, q,
         k_pool, v_pool, out, nq, nkv, hd, scale);
}

}  // namespace wisp
