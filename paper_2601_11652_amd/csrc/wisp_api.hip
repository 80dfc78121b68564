// C ABI of the verification step (declared in include/wisp.h): validation, planning of
// the launch (row layout, GEMM K-splits, split-KV attention work list), workspace carving
// and the stream-ordered kernel sequence of one step.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdarg>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <mutex>
#include <string>
#include <vector>

#include "../../include/wisp.h"
#include "common.h"
#include "host_guard.h"
#include "kernels.h"

using namespace wisp;

namespace {

// the calling thread's last error message (a fixed buffer: reporting never allocates)
thread_local char g_last_error[512] = "";

wisp_status fail(wisp_status st, const char *fmt, ...) __attribute__((format(printf, 2, 3)));
wisp_status fail(wisp_status st, const char *fmt, ...) {
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(g_last_error, sizeof(g_last_error), fmt, ap);
  va_end(ap);
  return st;
}

inline size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

// ------------------------------------------------------------------------------------------
// launch plan
// ------------------------------------------------------------------------------------------
struct Plan {
  int B = 0, M = 0, Mp = 0, S = 0;   // requests, rows, rows padded to 32, total drafts
  int Mv = 0;                        // verification rows (root and drafts): logits rows
  bool prefill = false;              // some request forwards prompt rows before its root
  int d = 0, nq = 0, nkv = 0, hd = 0, F = 0, V = 0, qdim = 0, kvdim = 0, qkvN = 0, G = 0;
  bool bf16 = false;
  int max_tokens = 0;
  GemmCfg g_qkv{}, g_o{}, g_gu{}, g_down{}, g_lm{};
  std::vector<AttnItem> items;
  std::vector<AttnGroup> groups;
  std::vector<int32_t> first;        // wave w runs items first[w] .. first[w + 1] - 1 (empty: item w)
  int attn_waves() const { return (int)(first.empty() ? items.size() : first.size() - 1); }
  int item_rows = 0;                 // query rows of an item: 32, 48 or 64
  std::vector<int32_t> host;         // descriptor block uploaded to the device
  // int32 offsets inside the descriptor block
  size_t i_off = 0, i_doff = 0, i_gamma = 0, i_ctx = 0, i_req = 0, i_row_req = 0, i_row_pos = 0,
         i_items = 0, i_groups = 0, i_first = 0, i_voff = 0, i_nrow = 0, i_vrow = 0;
  // byte offsets inside the workspace
  size_t w_err = 0, w_desc = 0, w_rope = 0, w_h = 0, w_xn = 0, w_ao = 0, w_af = 0, w_q = 0,
         w_part = 0, w_attn_o = 0, w_attn_ml = 0, w_sm = 0, w_si = 0, w_ss = 0, w_rk = 0, w_ri = 0,
         w_rR = 0, w_vtok = 0, total = 0;
  int max_group_chunks = 0;          // most chunks any attention group combines
  int race_chunk = 0;                // vocabulary entries per workgroup of the acceptance's race
};


wisp_status check_model(const wisp_model *m, bool need_weights) {
  if (!m) return fail(WISP_E_INVALID, "model is NULL");
  if (m->n_layers <= 0 || m->d_model <= 0 || m->n_q_heads <= 0 || m->n_kv_heads <= 0 ||
      m->head_dim <= 0 || m->d_ff <= 0 || m->vocab <= 0)
    return fail(WISP_E_INVALID, "model dimensions must be positive");
  if (m->dtype != WISP_F32 && m->dtype != WISP_BF16) return fail(WISP_E_UNSUPPORTED, "dtype %d", m->dtype);
  if (m->n_q_heads % m->n_kv_heads) return fail(WISP_E_UNSUPPORTED, "n_q_heads %% n_kv_heads != 0");
  if (m->head_dim % 32 || m->head_dim > 256)
    return fail(WISP_E_UNSUPPORTED, "head_dim must be a multiple of 32, at most 256");
  if (m->d_model % 32 || m->d_ff % 32) return fail(WISP_E_UNSUPPORTED, "d_model, d_ff must be multiples of 32");
  // the residual + norm kernels hold a row in one workgroup, 8 columns per thread
  if (m->d_model > 8192) return fail(WISP_E_UNSUPPORTED, "d_model > 8192");
  if (m->dtype == WISP_BF16) {
    if (m->head_dim != 64 && m->head_dim != 128) return fail(WISP_E_UNSUPPORTED, "bf16 head_dim must be 64 or 128");
    if (m->vocab % 32) return fail(WISP_E_UNSUPPORTED, "bf16 vocab must be a multiple of 32");
    if (m->n_q_heads / m->n_kv_heads > 64) return fail(WISP_E_UNSUPPORTED, "GQA group > 64");
  }
  if (!(m->rms_eps >= 0.f) || !(m->rope_base > 0.f)) return fail(WISP_E_INVALID, "rms_eps / rope_base");
  if (need_weights) {
    if (!m->embed || !m->final_norm || !m->lm_head || !m->attn_norm || !m->w_qkv || !m->w_o ||
        !m->mlp_norm || !m->w_gate_up || !m->w_down)
      return fail(WISP_E_INVALID, "NULL weight pointer");
    for (int l = 0; l < m->n_layers; ++l)
      if (!m->attn_norm[l] || !m->w_qkv[l] || !m->w_o[l] || !m->mlp_norm[l] || !m->w_gate_up[l] ||
          !m->w_down[l])
        return fail(WISP_E_INVALID, "NULL weight pointer in layer %d", l);
  }
  return WISP_OK;
}

// forward: the call runs the model, so prompt rows count towards the batch's rows
wisp_status check_desc(const wisp_batch_desc *d, bool need_pages, bool forward) {
  if (!d) return fail(WISP_E_INVALID, "batch descriptor is NULL");
  if (d->B < 0) return fail(WISP_E_INVALID, "B < 0");
  if (d->B == 0) return WISP_OK;
  if (!d->ctx_len || !d->gamma) return fail(WISP_E_INVALID, "ctx_len / gamma is NULL");
  if (!(d->temperature >= 0.f) || std::isinf(d->temperature)) return fail(WISP_E_INVALID, "temperature must be finite and >= 0");
  int64_t rows = 0;
  for (int i = 0; i < d->B; ++i) {
    if (d->gamma[i] < 0 || d->gamma[i] > WISP_GAMMA_MAX)
      return fail(WISP_E_INVALID, "gamma[%d] = %d outside 0..%d", i, d->gamma[i], WISP_GAMMA_MAX);
    if (d->ctx_len[i] < 0) return fail(WISP_E_INVALID, "ctx_len[%d] < 0", i);
    const int pre = d->prefill_len ? d->prefill_len[i] : 0;
    if (pre < 0 || pre > WISP_PREFILL_MAX)
      return fail(WISP_E_INVALID, "prefill_len[%d] = %d outside 0..%d", i, pre, WISP_PREFILL_MAX);
    const int64_t need = (int64_t)d->ctx_len[i] + pre + d->gamma[i] + 1;
    if (need > INT32_MAX / 2) return fail(WISP_E_INVALID, "request %d: ctx_len too large", i);
    if (need_pages && (int64_t)d->pt_stride * WISP_PAGE < need)
      return fail(WISP_E_CAPACITY, "request %d needs %lld tokens but the page table holds %d", i,
                  (long long)need, d->pt_stride * WISP_PAGE);
    // the model's rows are bounded by WISP_ROWS_MAX; the acceptance alone only by int range
    rows += (forward ? pre : 0) + d->gamma[i] + 1;
    const int64_t max_rows = forward ? WISP_ROWS_MAX : kAcceptRowsMax;
    if (rows > max_rows)
      return fail(WISP_E_UNSUPPORTED, "the batch has more than %lld rows (prompt, root and draft rows)",
                  (long long)max_rows);
  }
  if (need_pages && !d->kv_page_table) return fail(WISP_E_INVALID, "kv_page_table is NULL");
  return WISP_OK;
}

void carve(size_t &w, size_t &field, size_t bytes) {
  field = w;
  w = align256(w + bytes);
}

// the logits of a step's verification rows
size_t logits_bytes(int64_t rows, int V) { return align256((size_t)rows * (size_t)V * sizeof(float)); }

// the race winners of every (request, chunk): keys, then token ids
size_t race_bytes(const Plan &p) {
  const size_t RC = (std::max(p.V, 1) + p.race_chunk - 1) / p.race_chunk;
  return 2 * align256((size_t)p.B * RC * 2 * 4);
}
void place_race(Plan &p, size_t at) {
  p.w_rk = at;
  p.w_ri = at + race_bytes(p) / 2;
}

// partial results of one attention item: O and (m, l) of its rows
size_t attn_item_bytes(const Plan &p) { return (size_t)p.item_rows * (p.hd + 2) * 4; }
// the space of all of them (none where every group is one item)
size_t attn_part_bytes(const Plan &p) {
  return p.max_group_chunks > 1 ? align256(p.items.size() * (size_t)p.hd * p.item_rows * 4) + align256(p.items.size() * (size_t)p.item_rows * 2 * 4) : 0;
}

// compute units of the current device (the attention work list is sized to them)
int device_cus() {
  int dev = 0, n = 0;
  if (hipGetDevice(&dev) != hipSuccess ||
      hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0)
    n = 256;
  return n;
}

// Attention work list.  A row group (item_rows of a request's rows x G query rows of one kv
// head) attends to a run of page pairs.  Either every item (a part of a group's pairs) has a
// wave of its own, or the waves share all groups' pairs in order (request, kv head, row group);
// a group that one wave covers alone needs no combine.  The partial results take at most `room`
// bytes.  The times below are of one layer's attention and combine.
wisp_status plan_attention(Plan &p, const wisp_batch_desc *d, const std::vector<int> &nrow, size_t room) {
  p.items.clear();
  p.groups.clear();
  p.first.clear();
  p.max_group_chunks = 0;
  const int64_t slots = 4 * (int64_t)device_cus();   // one wave per SIMD
  const bool hd64 = p.hd == 64;
  // a row group's keys end at its last row's causal limit (prompt rows see fewer)
  auto group_tokens = [&](int i, int g, int R) {
    const int last = std::min(nrow[i] * p.G, (g + 1) * R) - 1;
    return d->ctx_len[i] + last / p.G + 1;
  };
  auto group_pairs = [&](int i, int g, int R) { return (group_tokens(i, g, R) + 31) / 32; };
  auto row_groups = [&](int i, int R) { return (nrow[i] * p.G + R - 1) / R; };

  // The candidates: page pairs of every row group (of one kv head), their time at the rates
  // measured per pair and launch (ns).  A pair that comes from memory takes about the same
  // with 32, 48 and 64 rows at head_dim 128, so as few groups per request as fit (128 requests
  // of up to 36 rows: 246 us with 32 rows, 221 with 48); 64 rows leave head_dim 64 too few
  // waves (256 requests of 1-8k, one group each: 596 us with 32 rows, 625 with 48, 816 with
  // 64).  Past 256 rows (prompts: neighbouring groups share the pairs through L2) the products
  // bound it: 32 rows.
  constexpr int kRows[3] = {32, 48, 64};
  constexpr double kStream[2][3] = {{2.8, 2.85, 2.9}, {1.4, 1.45, 1.9}}, kCompute[2][3] = {{1.4, 2.4, 3.3}, {0.7, 1.4, 2.6}};
  struct Cand {
    std::vector<int> pairs;
    int64_t total = 0, most = 0;
    double us = 0;
  } cand[3];
  // the largest batch accepted: 2^22 items of at most 48 query rows and 32 page pairs, a round
  // of wave slots kept back (indices are int: what is built below is at most twice as long)
  int64_t fewest = 0, prompt = 0, unique = 0;   // unique: pairs of the requests' contexts, each once per kv head
  for (int r = 0; r < 3; ++r) {
    Cand &c = cand[r];
    for (int i = 0; i < p.B; ++i) {
      const bool long_prompt = nrow[i] > WISP_GAMMA_MAX + 1 && nrow[i] * p.G > 256;
      int64_t n = 0;
      for (int g = 0, m = row_groups(i, kRows[r]); g < m; ++g) {
        const int pr = group_pairs(i, g, kRows[r]);
        c.pairs.push_back(pr);
        n += pr;
        c.most = std::max<int64_t>(c.most, pr);
        if (r == 1) fewest += (int64_t)p.nkv * ((pr + 31) / 32);
      }
      c.total += p.nkv * n;
      c.us += n * (long_prompt ? kCompute : kStream)[hd64][r];
      if (r == 0) unique += p.nkv * (int64_t)c.pairs.back();
      if (r == 0 && long_prompt) prompt += p.nkv * n;
    }
  }
  if (fewest > kAttnMaxItems - slots)
    return fail(WISP_E_UNSUPPORTED, "the batch's contexts need %lld attention work items (at most %d)",
                (long long)fewest, kAttnMaxItems - (int)slots);
  const Cand *c = nullptr;
  auto count_items = [&](int64_t L) {
    int64_t n = 0;
    for (int pr : c->pairs) n += (pr + L - 1) / L;
    return n * p.nkv;
  };
  // the shortest items of at least L0 and at most L1 pairs that `waves` waves cover, or 0
  auto shortest = [&](int64_t L0, int64_t L1, int64_t waves) -> int64_t {
    if (c->total > L1 * waves || count_items(L1) > waves) return 0;
    int64_t L = std::max<int64_t>(L0, (c->total + waves - 1) / waves);
    while (L < L1 && count_items(L) > waves) ++L;
    return L;
  };

  // A way to give every item a wave of its own: its items' pairs and its estimated time (us),
  // the longer of a wave's chain of pairs (starting takes as long as 6, or beside a second wave
  // 10, 7 at head_dim 64) and of the K and V from memory (pairs that another row group reads too
  // count 0.3 or, with two waves per SIMD, 0.6), and the combine, 4 us up to 8 items of a group,
  // beyond it 4.9 + 0.18 per item and the partials at 6 TB/s (8 of 0.5-2k, 4 heads per kv head:
  // 23 us in 952 items of 3 pairs, 21 in 376 of 8).  (1 request of 30k, 32 rows: 66 us with
  // items of 12 pairs, 48 with 20, 52 with 32.  4 of 0.5-4k, 8 query heads per kv head: 27 us with 32 rows, 38 with
  // 48, 46 with 64.  32 of 0.5-2k, 4 heads: 37 us in 944 items of 12 pairs, 46 in 1900 of 6, two
  // waves per SIMD; at head_dim 64, 16 heads on 16, 35 in 1000 of 24, 32 in 1888 of 10.  12 of
  // 2-6k, 16 heads on 16: 91 in 1000 of 24, 72 in 1900 of 13.  22 of 3-4.5k and 28-40 rows: 90
  // in 1984 of 32 rows and 16 pairs, 70 in 1000 of 48 rows and 22.)
  constexpr double kChain[2][3] = {{1.2, 1.6, 2.0}, {1.0, 1.3, 1.6}};
  constexpr double kTwo[2] = {2.0, 1.5}, kMem[2][2] = {{3.3, 2.75}, {1.65, 1.4}};   // chain's factor; ns
  struct Items {
    int r = 0;
    int64_t L = 0;   // 0: none
    double us = 1e30;
  };
  auto partials = [&](int64_t n, int rows) { return (double)n * rows * (p.hd + 2) * 4 / 6e6; };
  // the shortest items of at most L1 pairs that one wave (two) per SIMD cover, or, with one,
  // longer ones that take less (fewer than two per SIMD would leave loads unissued)
  auto try_items = [&](Items &best, int r, bool two, int64_t L1) {
    c = &cand[r];
    const double pairs = unique + (two ? 0.6 : 0.3) * (c->total - unique);
    const double mem = pairs * kMem[hd64][two] * 1e-3;
    for (int64_t l = shortest(2, L1, two ? 2 * slots : slots); l && l <= kAttnWindowPages / 2; ++l) {
      const int64_t n = (c->most + l - 1) / l;
      const double chain = two ? (l + (hd64 ? 7 : 10)) * kChain[hd64][r] * kTwo[hd64] : (l + 6) * kChain[hd64][r];
      const double t = std::max(chain, mem) +
                       (n <= kAttnCombineChunks ? 4.0 : 4.9 + 0.18 * n + partials(count_items(l), kRows[r]));
      if (t < best.us) best = Items{r, l, t};
      if (two) break;
    }
  };

  constexpr int64_t kShort = 16;
  const bool prompts = 2 * prompt >= cand[0].total;   // most pairs belong to prompts
  int best = 0;
  int64_t L = 0;          // pairs of an item; 0: shares
  int64_t waves = 0;      // of shares
  c = &cand[0];
  if (prompts) {
    // Up to 16 pairs per wave (two waves per SIMD) the shortest items, one wave each.  Beyond
    // that items of half a wave's part, dispatched as others end: the items that run at one
    // time then attend to the same keys, which come from L2, while in shares the waves drift
    // apart; longer ones save combines, shorter ones even out the end (prompts of 2 x 4000 rows:
    // 957 us in shares, 829 / 688 / 628 in items of 16 / 32 / 64 pairs; 2048 rows: 150 us in
    // shares, 115 in items of 24, 95 of 128).
    L = shortest(2, kShort, slots);
    if (!L) {
      L = std::max<int64_t>(2, (c->total + 2 * slots - 1) / (2 * slots));
      if (L > kShort) L = std::min<int64_t>(256, std::max<int64_t>(24, L / 2));
      else
        while (L < kShort && count_items(L) > 2 * slots) ++L;
    }
  } else {
    // Items of up to 32 pairs where one wave per SIMD covers them, or of up to 16 (24 with 48 rows)
    // where two do and have room; equal shares of all pairs per wave where that is estimated to
    // take less (its pairs at the rate of kStream and 20 us, 12 at head_dim 64, and half of the
    // partials where a group has more than 8: the other half is in the rate), and beyond.  (40 of
    // 0.2-16k: 95 us in 1016 items, 114 in shares; 4 of 10-30k, 8 heads: 84 and 76.)
    // (256 of 1-8k, 110 pairs per wave: 610 us in shares, 692 in items; 48 rows, 64 of 0.5-4k:
    // 90, against 118 in 1040 items; 22 of 3-4.5k 66, against 63 in 912 items of 24 pairs.)
    // Where the row groups alone outnumber the waves, items of up to 16 pairs, dispatched as
    // others end.
    for (int r = 1; r < 3; ++r)
      if (cand[r].us < cand[best].us) best = r;
    const bool two = kRows[best] == 32 || (hd64 && kRows[best] == 48);   // waves per SIMD of shares
    waves = two ? 2 * slots : slots;
    Items a;
    if (cand[best].total > kShort * waves) {
      a.us = p.nkv * cand[best].us * 1e-3 + (hd64 ? 12.0 : 20.0);
      if (cand[best].most * waves > kAttnCombineChunks * cand[best].total)
        a.us += 0.5 * partials(waves + p.nkv * (int64_t)cand[best].pairs.size(), kRows[best]);
    }
    for (int r = 0; r < 3; ++r) try_items(a, r, false, 2 * kShort);
    try_items(a, 0, true, kShort);
    if (hd64) try_items(a, 1, true, 24);
    if (a.L) best = a.r;
    c = &cand[best];
    L = a.L;
    if (!L && c->total <= kShort * waves) L = kShort;
    // At head_dim 64, where row groups share their pairs, items of 24 pairs (more where that
    // would make more than 16 per SIMD) in turn rather than shares, which run the groups that
    // share one after another (256 of 1-8k, 8 query heads per kv head: 419 us in shares, 399 in
    // items; 64 of 1-3k, 128-136 rows: 153 and 131)
    if (!L && hd64 && 5 * c->total > 6 * unique)
      L = std::min<int64_t>(256, std::max<int64_t>(24, c->total / (16 * slots)));
  }
  const int R = p.item_rows = kRows[best];
  const int64_t total = c->total;
  // longer items where the partials would pass the room, at the longest one item per group
  // and no partials
  const int64_t cap = (int64_t)(std::min<size_t>(room, INT64_MAX) / attn_item_bytes(p));
  if ((L ? count_items(L) : waves + p.nkv * (int64_t)c->pairs.size()) > cap) {
    if (!L) L = std::max<int64_t>(2, (total + waves - 1) / waves);
    while (L < c->most && count_items(L) > cap) L = std::min(c->most, L + std::max<int64_t>(1, L / 8));
  }
  const bool single = L > 0;
  if (!single) waves = std::min(waves, total);
  // shares: wave w starts at pair w * total / waves, moved to a group's edge if one is within
  // 1/16 of a share (a sliver of a group costs an item and a partial, 1/16 more a little time)
  const int64_t snap = single ? 0 : total / waves / 16;
  int64_t at = 0, w = 0;       // pairs before this group; wave of the last item
  auto start = [&](int64_t k) { return k * total / waves; };
  p.items.reserve(single ? count_items(L) : waves + (int64_t)p.nkv * (int64_t)c->pairs.size());
  if (!single) {
    p.first.reserve(waves + 1);
    p.first.push_back(0);
  }
  for (int i = 0; i < p.B; ++i) {
    const int nrbg = row_groups(i, R);
    for (int h = 0; h < p.nkv; ++h)
      for (int g = 0; g < nrbg; ++g) {
        const int T = group_tokens(i, g, R), pairs = (T + 31) / 32;
        AttnGroup gr{};
        gr.req = i;
        gr.kvh_rbg = attn_pack(h, g);
        gr.first_item = (int32_t)p.items.size();
        auto item = [&](int64_t a, int64_t b) {
          AttnItem it{};
          it.req = i;
          it.kvh_rbg = gr.kvh_rbg;
          it.t0 = 32 * (int)a | (a == 0 && b == pairs ? kAttnWhole : 0) | (g >> 16 ? kAttnHighItem : 0);
          it.t1 = std::min(T, 32 * (int)b);
          p.items.push_back(it);
        };
        if (single) {
          const int64_t n = (pairs + L - 1) / L;
          for (int64_t k = 0; k < n; ++k) item(k * pairs / n, (k + 1) * pairs / n);
        } else {
          int64_t a = 0;
          while (w + 1 < waves && start(w + 1) < at + pairs + snap) {   // waves that start in this group
            const int64_t b = start(w + 1) - at;
            if (b >= pairs - snap) break;              // at its end: the next group's first
            if (b > a && b > snap) {
              item(a, b);
              a = b;
            }
            p.first.push_back((int32_t)p.items.size());
            ++w;
          }
          item(a, pairs);
          at += pairs;
        }
        gr.n_items = (int32_t)p.items.size() - gr.first_item;
        p.max_group_chunks = std::max(p.max_group_chunks, (int)gr.n_items);
        if (gr.n_items > 1) {
          if (g >> 16) gr.n_items |= kAttnHighGroup;
          p.groups.push_back(gr);
        }
      }
  }
  if (!single) p.first.push_back((int32_t)p.items.size());
  return WISP_OK;
}

void lay_out(Plan &p, const wisp_batch_desc *d, bool forward, const std::vector<int> &off, const std::vector<int> &doff,
             const std::vector<int> &voff, const std::vector<int> &nrow);

// forward=true: the full step; false: acceptance only (rows/drafts of the batch, vocab V).
// limit: the most bytes the workspace should take, kept by fewer attention partials if that helps.
wisp_status make_plan(Plan &p, const wisp_model *m, const wisp_batch_desc *d, bool forward, int vocab = 0,
                      size_t limit = SIZE_MAX) {
  p.B = d->B;
  p.V = forward ? m->vocab : vocab;
  // rows of request i: prefill_len prompt rows (forward only), root, gamma drafts; the
  // verification rows (root .. y_gamma) are the last gamma + 1 and alone produce logits
  std::vector<int> off(p.B + 1, 0), doff(p.B + 1, 0), voff(p.B + 1, 0), nrow(p.B, 0);
  for (int i = 0; i < p.B; ++i) {
    const int pre = (forward && d->prefill_len) ? d->prefill_len[i] : 0;
    nrow[i] = pre + d->gamma[i] + 1;
    off[i + 1] = off[i] + nrow[i];
    voff[i + 1] = voff[i] + d->gamma[i] + 1;
    doff[i + 1] = doff[i] + d->gamma[i];
    if (pre > 0) p.prefill = true;
  }
  p.M = off[p.B];
  p.Mv = voff[p.B];
  p.S = doff[p.B];
  p.Mp = (p.M + 31) / 32 * 32;
  if (forward) {
    p.d = m->d_model;
    p.nq = m->n_q_heads;
    p.nkv = m->n_kv_heads;
    p.hd = m->head_dim;
    p.F = m->d_ff;
    p.V = m->vocab;
    p.G = p.nq / p.nkv;
    p.qdim = p.nq * p.hd;
    p.kvdim = p.nkv * p.hd;
    p.qkvN = p.qdim + 2 * p.kvdim;
    p.bf16 = m->dtype == WISP_BF16;
    for (int i = 0; i < p.B; ++i) p.max_tokens = std::max(p.max_tokens, d->ctx_len[i] + nrow[i]);
    if (p.bf16) {
      p.g_qkv = gemm_bf16_plan(p.M, p.qkvN, p.d);
      p.g_o = gemm_bf16_plan(p.M, p.d, p.qdim);
      p.g_gu = gemm_bf16_plan(p.M, 2 * p.F, p.d);
      p.g_down = gemm_bf16_plan(p.M, p.d, p.F);
      p.g_lm = gemm_bf16_plan(p.Mv, p.V, p.d);
      p.g_lm.splits = 1;
      p.g_lm.kf_per_split = p.d / 16;
      wisp_status st = plan_attention(p, d, nrow, SIZE_MAX);
      if (st != WISP_OK) return st;
    }
  }
  lay_out(p, d, forward, off, doff, voff, nrow);
  for (int k = 0; k < 4 && forward && p.total > limit; ++k) {
    const size_t rest = p.total - attn_part_bytes(p);
    if (attn_part_bytes(p) == 0 || rest > limit) break;
    const wisp_status st = plan_attention(p, d, nrow, k < 3 ? limit - rest : 0);
    if (st != WISP_OK) return st;
    lay_out(p, d, forward, off, doff, voff, nrow);
  }
  return WISP_OK;
}

// the descriptor block and the workspace of a plan
void lay_out(Plan &p, const wisp_batch_desc *d, bool forward, const std::vector<int> &off, const std::vector<int> &doff,
             const std::vector<int> &voff, const std::vector<int> &nrow) {
  // descriptor block
  size_t n = 0;
  auto take = [&](size_t &f, size_t cnt) {
    f = n;
    n += (cnt + 63) / 64 * 64;
  };
  take(p.i_off, p.B + 1);
  take(p.i_doff, p.B + 1);
  take(p.i_gamma, p.B);
  take(p.i_ctx, p.B);
  take(p.i_req, p.B);
  take(p.i_row_req, p.M);
  take(p.i_row_pos, p.M);
  take(p.i_items, p.items.size() * (sizeof(AttnItem) / 4));
  take(p.i_groups, p.groups.size() * (sizeof(AttnGroup) / 4));
  take(p.i_first, p.first.size());
  take(p.i_voff, p.B + 1);
  take(p.i_nrow, p.B);
  take(p.i_vrow, p.Mv);
  p.host.assign(n, 0);
  for (int i = 0; i <= p.B; ++i) {
    p.host[p.i_off + i] = off[i];
    p.host[p.i_doff + i] = doff[i];
    p.host[p.i_voff + i] = voff[i];
  }
  for (int i = 0; i < p.B; ++i) {
    p.host[p.i_gamma + i] = d->gamma[i];
    p.host[p.i_ctx + i] = d->ctx_len[i];
    p.host[p.i_req + i] = d->req_id ? (int32_t)d->req_id[i] : i;
    p.host[p.i_nrow + i] = nrow[i];
    for (int j = 0; j < nrow[i]; ++j) {
      p.host[p.i_row_req + off[i] + j] = i;
      p.host[p.i_row_pos + off[i] + j] = d->ctx_len[i] + j;
    }
    for (int j = 0; j <= d->gamma[i]; ++j) p.host[p.i_vrow + voff[i] + j] = off[i + 1] - (d->gamma[i] + 1) + j;
  }
  if (!p.items.empty()) std::memcpy(&p.host[p.i_items], p.items.data(), p.items.size() * sizeof(AttnItem));
  std::copy(p.first.begin(), p.first.end(), p.host.begin() + p.i_first);
  if (!p.groups.empty()) std::memcpy(&p.host[p.i_groups], p.groups.data(), p.groups.size() * sizeof(AttnGroup));

  // workspace
  size_t w = 0;
  carve(w, p.w_err, 256);
  carve(w, p.w_desc, p.host.size() * sizeof(int32_t));
  const int CH = sampler_chunks(std::max(p.V, 1));
  carve(w, p.w_sm, (size_t)p.Mv * CH * 4);
  carve(w, p.w_si, (size_t)p.Mv * CH * 4);
  carve(w, p.w_ss, (size_t)p.Mv * CH * 8);
  carve(w, p.w_vtok, (size_t)(p.prefill ? p.Mv : 0) * 4);
  carve(w, p.w_rR, (size_t)p.B * 4);
  if (forward) {
    const size_t es = p.bf16 ? 2 : 4;
    carve(w, p.w_rope, (size_t)p.M * p.hd * 4);
    carve(w, p.w_h, (size_t)p.M * p.d * 4);
    carve(w, p.w_xn, (size_t)p.Mp * p.d * es);
    carve(w, p.w_ao, (size_t)p.Mp * p.qdim * es);
    carve(w, p.w_af, (size_t)p.Mp * p.F * es);
    carve(w, p.w_q, (size_t)p.M * p.qdim * es);
    size_t part = 0;
    if (p.bf16) {
      part = std::max({(size_t)p.g_qkv.splits * p.qkvN, (size_t)p.g_o.splits * p.d,
                       (size_t)p.g_gu.splits * 2 * p.F, (size_t)p.g_down.splits * p.d});
    } else {
      part = std::max({(size_t)p.qkvN, (size_t)p.d, (size_t)2 * p.F});
    }
    part *= (size_t)p.M * 4;
    p.race_chunk = sampler_race_chunk(p.B, p.V, part);
    carve(w, p.w_part, std::max(part, race_bytes(p)));
    place_race(p, p.w_part);   // the partial sums are free when the acceptance starts
    if (p.max_group_chunks > 1) {
      carve(w, p.w_attn_o, p.items.size() * (size_t)p.hd * p.item_rows * 4);
      carve(w, p.w_attn_ml, p.items.size() * (size_t)p.item_rows * 2 * 4);
    }
  } else {
    p.race_chunk = sampler_race_chunk(p.B, std::max(p.V, 1), SIZE_MAX);
    size_t at = 0;
    carve(w, at, race_bytes(p));
    place_race(p, at);
  }
  p.total = w;
}

// ------------------------------------------------------------------------------------------
// optional per-kernel-class timing: while a class scope is open, every launch in it gets a
// pair of HIP events stamped with that dispatch's own begin and end (launch_timing_events);
// a class's time is the sum of its dispatches' durations, its launch count the number of
// scopes, and its bytes / flops are those of the scope
// ------------------------------------------------------------------------------------------
struct ProfRec {
  int kind;
  int scopes;                 // 1 on a scope's first dispatch, else 0
  double bytes, flops;        // the scope's figures, on its first dispatch
  hipEvent_t a, b;
};
struct ProfState {
  bool on = false;
  int open_kind = -1;         // class of the open scope (-1: none)
  bool open_first = false;    // no dispatch of the open scope recorded yet
  double open_bytes = 0, open_flops = 0;
  std::vector<ProfRec> pending;
  std::vector<hipEvent_t> free_events;
  double ms[WISP_PROF_KINDS] = {}, bytes[WISP_PROF_KINDS] = {}, flops[WISP_PROF_KINDS] = {};
  int64_t launches[WISP_PROF_KINDS] = {};
};
ProfState g_prof;

hipEvent_t prof_event() {
  if (!g_prof.free_events.empty()) {
    hipEvent_t e = g_prof.free_events.back();
    g_prof.free_events.pop_back();
    return e;
  }
  hipEvent_t e = nullptr;
  (void)hipEventCreate(&e);
  return e;
}

struct ProfScope {   // opens a timing scope of class `kind` over the launches it encloses
  ProfScope(int kind, double bytes, double flops, hipStream_t) {
    if (g_prof.on) {
      g_prof.open_kind = kind;
      g_prof.open_first = true;
      g_prof.open_bytes = bytes;
      g_prof.open_flops = flops;
    }
  }
  ~ProfScope() { g_prof.open_kind = -1; }
};

void prof_collect() {
  for (auto &r : g_prof.pending) {
    (void)hipEventSynchronize(r.b);
    float ms = 0.f;
    (void)hipEventElapsedTime(&ms, r.a, r.b);
    g_prof.ms[r.kind] += ms;
    g_prof.bytes[r.kind] += r.bytes;
    g_prof.flops[r.kind] += r.flops;
    g_prof.launches[r.kind] += r.scopes;
    g_prof.free_events.push_back(r.a);
    g_prof.free_events.push_back(r.b);
  }
  g_prof.pending.clear();
}

}  // namespace

bool wisp::launch_timing_events(hipEvent_t *start, hipEvent_t *stop) {
  if (!g_prof.on || g_prof.open_kind < 0) return false;
  ProfRec r{g_prof.open_kind, 0, 0.0, 0.0, prof_event(), prof_event()};
  if (g_prof.open_first) {
    r.scopes = 1;
    r.bytes = g_prof.open_bytes;
    r.flops = g_prof.open_flops;
    g_prof.open_first = false;
  }
  g_prof.pending.push_back(r);
  *start = r.a;
  *stop = r.b;
  return true;
}

namespace {

// pinned staging for the descriptor upload, reused once the previous copy has finished
struct Staging {
  void *buf = nullptr;
  size_t cap = 0;
  hipEvent_t ev = nullptr;
  bool pending = false;
};
thread_local Staging g_stage;

wisp_status upload(const Plan &p, char *ws, hipStream_t s) {
  const size_t bytes = p.host.size() * sizeof(int32_t);
  if (bytes == 0) return WISP_OK;
  if (g_stage.pending) {
    if (hipEventSynchronize(g_stage.ev) != hipSuccess) return fail(WISP_E_HIP, "staging event sync failed");
    g_stage.pending = false;
  }
  if (g_stage.cap < bytes) {
    if (g_stage.buf) (void)hipHostFree(g_stage.buf);
    g_stage.buf = nullptr;
    g_stage.cap = 0;
    size_t cap = std::max<size_t>(bytes, 1 << 16);
    if (hipHostMalloc(&g_stage.buf, cap, hipHostMallocDefault) != hipSuccess)
      return fail(WISP_E_HIP, "pinned staging allocation failed");
    g_stage.cap = cap;
  }
  if (!g_stage.ev && hipEventCreateWithFlags(&g_stage.ev, hipEventDisableTiming) != hipSuccess)
    return fail(WISP_E_HIP, "event creation failed");
  std::memcpy(g_stage.buf, p.host.data(), bytes);
  if (hipMemcpyAsync(ws + p.w_desc, g_stage.buf, bytes, hipMemcpyHostToDevice, s) != hipSuccess)
    return fail(WISP_E_HIP, "descriptor upload failed");
  if (hipEventRecord(g_stage.ev, s) != hipSuccess) return fail(WISP_E_HIP, "event record failed");
  g_stage.pending = true;
  return WISP_OK;
}

SamplerScratch sampler_scratch(const Plan &p, char *ws) {
  SamplerScratch sc;
  sc.part_m = reinterpret_cast<float *>(ws + p.w_sm);
  sc.part_i = reinterpret_cast<int32_t *>(ws + p.w_si);
  sc.part_s = reinterpret_cast<double *>(ws + p.w_ss);
  sc.race_k = reinterpret_cast<float *>(ws + p.w_rk);
  sc.race_i = reinterpret_cast<int32_t *>(ws + p.w_ri);
  sc.req_R = reinterpret_cast<int32_t *>(ws + p.w_rR);
  return sc;
}

StepDesc step_desc(const Plan &p, char *ws, const wisp_batch_desc *d, int n_blocks, int *err = nullptr) {
  const int32_t *base = reinterpret_cast<const int32_t *>(ws + p.w_desc);
  StepDesc sd;
  sd.off = base + p.i_off;
  sd.doff = base + p.i_doff;
  sd.gamma = base + p.i_gamma;
  sd.ctx = base + p.i_ctx;
  sd.req_id = reinterpret_cast<const uint32_t *>(base + p.i_req);
  sd.row_req = base + p.i_row_req;
  sd.row_pos = base + p.i_row_pos;
  sd.nrow = base + p.i_nrow;
  sd.page_table = d->kv_page_table;
  sd.pt_stride = d->pt_stride;
  sd.n_blocks = n_blocks;
  sd.err = err ? err : reinterpret_cast<int *>(ws + p.w_err);
  return sd;
}

int gemm_class(const Plan &p, const GemmCfg &c) {
  if (!p.bf16) return WISP_PROF_GEMM_TILED;
  if (c.kind == 4) return WISP_PROF_GEMM_TILE;
  return c.kind == 2 ? WISP_PROF_GEMM_RING2 : WISP_PROF_GEMM_RING1;
}

wisp_status hip_check(const char *what) {
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return fail(WISP_E_HIP, "%s: %s", what, hipGetErrorString(e));
  return WISP_OK;
}

template <typename T>
wisp_status run_forward(const Plan &p, const wisp_model *m, const wisp_kv *kv, const StepDesc &sd,
                        char *ws, const int32_t *tokens, float *logits, hipStream_t s) {
  const bool packed = p.bf16;
  float *cs = reinterpret_cast<float *>(ws + p.w_rope);
  float *h = reinterpret_cast<float *>(ws + p.w_h);
  T *xn = reinterpret_cast<T *>(ws + p.w_xn);
  T *ao = reinterpret_cast<T *>(ws + p.w_ao);
  T *af = reinterpret_cast<T *>(ws + p.w_af);
  T *qb = reinterpret_cast<T *>(ws + p.w_q);
  float *part = reinterpret_cast<float *>(ws + p.w_part);
  const int64_t layer_elems = (int64_t)kv->n_blocks * p.nkv * WISP_PAGE * p.hd;
  const AttnItem *items = reinterpret_cast<const AttnItem *>(ws + p.w_desc + p.i_items * 4);
  const AttnGroup *groups = reinterpret_cast<const AttnGroup *>(ws + p.w_desc + p.i_groups * 4);
  const int32_t *first = p.first.empty() ? nullptr : reinterpret_cast<const int32_t *>(ws + p.w_desc) + p.i_first;
  const int32_t *vrow = reinterpret_cast<const int32_t *>(ws + p.w_desc) + p.i_vrow;

  const double es = p.bf16 ? 2.0 : 4.0;
  // algorithmic bytes of a projection: its weights, read once per step (activations and
  // results are a few percent at the step's row counts and not counted)
  auto gemm_bytes = [&](int N, int K) { return es * (double)N * K; };
  auto gemm_flops = [&](int N, int K) { return 2.0 * p.M * N * K; };
  const double kv_tok = 2.0 * p.nkv * p.hd * es;   // K and V bytes per token per layer
  double attn_bytes = 0.0, attn_flops = 0.0;
  for (const AttnItem &it : p.items) {
    const int G = p.G;
    const int rows = (int)p.host[p.i_nrow + it.req];
    const int rbg = attn_rbg(it.kvh_rbg, it.t0), tokens = it.t1 - (it.t0 & ~kAttnFlags);
    const int nr = std::min(p.item_rows, rows * G - rbg * p.item_rows);
    if (rbg == 0) attn_bytes += (double)tokens * kv_tok / p.nkv;
    attn_flops += 4.0 * p.hd * nr * tokens;
  }
  {
    ProfScope ps(WISP_PROF_ROWS, 0, 0, s);
    rope_table(sd, cs, p.M, p.hd, m->rope_base, s);
    embed_norm<T>(sd, (const T *)m->embed, (const T *)m->attn_norm[0], tokens, h, xn, packed, p.M, p.d,
                  p.V, m->rms_eps, s);
  }
  for (int l = 0; l < m->n_layers; ++l) {
    T *kl = (T *)kv->k_pool + l * layer_elems;
    T *vl = (T *)kv->v_pool + l * layer_elems;
    // one dense projection: C = act . W^T (fp32 partials over cfg.splits K ranges)
    auto gemm = [&](const T *act, const void *w, float *out, int N, int K, const GemmCfg &cfg) {
      ProfScope ps(gemm_class(p, cfg), gemm_bytes(N, K), gemm_flops(N, K), s);
      if (p.bf16)
        gemm_bf16((const uint16_t *)act, (const uint16_t *)w, out, p.M, N, K, N, cfg, s);
      else
        gemm_f32((const float *)act, (const float *)w, out, p.M, N, K, N, s);
      return p.bf16 ? cfg.splits : 1;
    };
    const int sq = gemm(xn, m->w_qkv[l], part, p.qkvN, p.d, p.g_qkv);
    {
      ProfScope ps(WISP_PROF_ROWS, 0, 0, s);
      qkv_rope_append<T>(sd, part, sq, cs, qb, kl, vl, p.M, p.nq, p.nkv, p.hd, s);
    }
    if (p.bf16) {
      float *po = reinterpret_cast<float *>(ws + p.w_attn_o);
      float *pml = reinterpret_cast<float *>(ws + p.w_attn_ml);
      {
        ProfScope ps(WISP_PROF_ATTN, attn_bytes, attn_flops, s);
        attention_bf16_main(sd, items, first, p.attn_waves(), p.item_rows, (const uint16_t *)qb,
                            (const uint16_t *)kl, (const uint16_t *)vl, po, pml, (uint16_t *)ao, true, p.qdim,
                            p.nq, p.nkv, p.hd, s);
      }
      ProfScope ps(WISP_PROF_ATTN_COMBINE, 0, 0, s);
      attention_bf16_combine(sd, groups, (int)p.groups.size(), p.item_rows, p.max_group_chunks, po, pml,
                             (uint16_t *)ao, true, p.qdim, p.nq, p.nkv, p.hd, s);
    } else {
      ProfScope ps(WISP_PROF_ATTN, attn_bytes, attn_flops, s);
      attention_f32(sd, p.M, (const float *)qb, (const float *)kl, (const float *)vl, (float *)ao, p.nq,
                    p.nkv, p.hd, p.max_tokens, s);
    }
    const int so = gemm(ao, m->w_o[l], part, p.d, p.qdim, p.g_o);
    {
      ProfScope ps(WISP_PROF_ROWS, 0, 0, s);
      resid_norm<T>(part, so, h, (const T *)m->mlp_norm[l], xn, packed, p.M, p.d, m->rms_eps, s);
    }
    if (p.bf16 && p.g_gu.kind == 4 && p.g_gu.splits == 1) {
      // one K range on the tile kernel: SwiGLU in the GEMM's epilogue, which writes the down
      // projection's bf16 input directly (no fp32 gate/up round trip, no SwiGLU launch)
      ProfScope ps(gemm_class(p, p.g_gu), gemm_bytes(2 * p.F, p.d), gemm_flops(2 * p.F, p.d), s);
      gemm_bf16((const uint16_t *)xn, (const uint16_t *)m->w_gate_up[l], part, p.M, 2 * p.F, p.d, 2 * p.F, p.g_gu,
                s, SwigluOut{(uint16_t *)af, p.F});
    } else {
      const int sg = gemm(xn, m->w_gate_up[l], part, 2 * p.F, p.d, p.g_gu);
      ProfScope ps(WISP_PROF_ROWS, 0, 0, s);
      swiglu<T>(part, sg, af, packed, p.M, p.F, p.bf16, s);   // bf16 gate/up: interleaved columns
    }
    const int sdn = gemm(af, m->w_down[l], part, p.d, p.F, p.g_down);
    const bool last = l + 1 == m->n_layers;
    const T *gain = last ? (const T *)m->final_norm : (const T *)m->attn_norm[l + 1];
    {
      ProfScope ps(WISP_PROF_ROWS, 0, 0, s);
      if (last && p.prefill)   // only the verification rows reach the LM head: compact them
        resid_norm<T>(part, sdn, h, gain, xn, packed, p.M, p.d, m->rms_eps, s, vrow, p.Mv);
      else
        resid_norm<T>(part, sdn, h, gain, xn, packed, p.M, p.d, m->rms_eps, s);
    }
  }
  {
    const double lm_bytes = es * (double)p.V * p.d;
    ProfScope ps(gemm_class(p, p.g_lm), lm_bytes, 2.0 * p.Mv * p.V * p.d, s);
    if (p.bf16)
      gemm_bf16((const uint16_t *)xn, (const uint16_t *)m->lm_head, logits, p.Mv, p.V, p.d, p.V, p.g_lm, s);
    else
      gemm_f32((const float *)xn, (const float *)m->lm_head, logits, p.Mv, p.V, p.d, p.V, s);
  }
  return hip_check("forward launch");
}

}  // namespace

namespace {

// validation shared by the two verification entry points
wisp_status check_verify(const wisp_model *model, const wisp_kv *kv, const wisp_batch_desc *desc,
                         const int32_t *tokens, const int32_t *accept_len, const int32_t *out_tokens) {
  wisp_status st;
  if ((st = check_model(model, true)) != WISP_OK) return st;
  if ((st = check_desc(desc, true, true)) != WISP_OK) return st;
  if (desc->B == 0) return WISP_OK;
  if (!kv || !kv->k_pool || !kv->v_pool) return fail(WISP_E_INVALID, "KV pools are NULL");
  if (kv->page_size != WISP_PAGE) return fail(WISP_E_UNSUPPORTED, "page_size must be %d", WISP_PAGE);
  if (kv->n_blocks <= 0) return fail(WISP_E_INVALID, "n_blocks must be positive");
  if (!tokens || !accept_len || !out_tokens) return fail(WISP_E_INVALID, "NULL tokens / outputs");
  return WISP_OK;
}

wisp_status plan_verify(Plan &p, const wisp_model *model, const wisp_batch_desc *desc, const float *draft_probs,
                        size_t limit = SIZE_MAX) {
  wisp_status st;
  if ((st = make_plan(p, model, desc, true, 0, limit)) != WISP_OK) return st;
  if (p.S > 0 && !draft_probs) return fail(WISP_E_INVALID, "draft_probs is NULL");
  if (!p.bf16 && p.max_tokens > 32768) return fail(WISP_E_UNSUPPORTED, "fp32 path supports <= 32768 tokens per request");
  return WISP_OK;
}

// the step's kernel sequence on a planned, uploaded workspace `ws`; `err` (or NULL: the
// workspace's own record) receives the device-side input faults
wisp_status run_verify(const Plan &p, const wisp_model *model, const wisp_kv *kv, const wisp_batch_desc *desc,
                       const int32_t *tokens, const float *draft_probs, uint64_t rng_seed, int32_t *accept_len,
                       int32_t *out_tokens, float *target_logits, char *ws, int *err, hipStream_t s) {
  wisp_status st;
  StepDesc sd = step_desc(p, ws, desc, kv->n_blocks, err);
  if (p.bf16)
    st = run_forward<uint16_t>(p, model, kv, sd, ws, tokens, target_logits, s);
  else
    st = run_forward<float>(p, model, kv, sd, ws, tokens, target_logits, s);
  if (st != WISP_OK) return st;
  // the acceptance sees the verification rows only: row offsets over them, and (with
  // prompt rows present) their tokens gathered into a compact array
  StepDesc sv = sd;
  sv.off = reinterpret_cast<const int32_t *>(ws + p.w_desc) + p.i_voff;
  const int32_t *vtok = tokens;
  if (p.prefill) {
    int32_t *g = reinterpret_cast<int32_t *>(ws + p.w_vtok);
    gather_ints(tokens, reinterpret_cast<const int32_t *>(ws + p.w_desc) + p.i_vrow, p.Mv, g, s);
    vtok = g;
  }
  // algorithmic bytes: one fp32 pass over the logits plus one logits row and one q row per request
  ProfScope ps(WISP_PROF_SAMPLER, (double)p.Mv * p.V * 4.0 + 2.0 * p.B * p.V * 4.0, 0, s);
  sampler(sv, p.B, p.Mv, p.V, target_logits, vtok, draft_probs, desc->temperature, rng_seed, p.race_chunk,
          sampler_scratch(p, ws), accept_len, out_tokens, s);
  return hip_check("sampler launch");
}

}  // namespace

// ------------------------------------------------------------------------------------------
// Scratch of the allocation-free entry point: one static array, of which every GPU the
// library runs on holds its own copy (at its own address, looked up once per device).
// Host code never uses the array's name as an address, only the looked-up pointer.
// ------------------------------------------------------------------------------------------
static __device__ __align__(256) unsigned char scratch[WISP_NOALLOC_SCRATCH_BYTES];

namespace {

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void *g_scratch_ptr[kMaxDevices] = {};

wisp_status noalloc_scratch(char **out) {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess) return fail(WISP_E_HIP, "hipGetDevice failed");
  if (dev < 0 || dev >= kMaxDevices) return fail(WISP_E_UNSUPPORTED, "device %d", dev);
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void *ptr = nullptr;
    const hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (e != hipSuccess || !ptr)
      return fail(WISP_E_HIP, "scratch address on device %d: %s", dev, hipGetErrorString(e));
    g_scratch_ptr[dev] = ptr;
  }
  *out = static_cast<char *>(g_scratch_ptr[dev]);
  return WISP_OK;
}

// The descriptor block reaches the device as kernel arguments, a few KB per launch: no
// pinned staging buffer and no host copy that must outlive the call.
constexpr int kDescChunkInts = 960;
struct DescChunk {
  int32_t n;
  int32_t v[kDescChunkInts];
};

__global__ void put_desc_kernel(DescChunk c, int32_t *__restrict__ dst) {
  for (int i = threadIdx.x; i < c.n; i += blockDim.x) dst[i] = c.v[i];
}

wisp_status upload_by_arguments(const Plan &p, char *ws, hipStream_t s) {
  int32_t *dst = reinterpret_cast<int32_t *>(ws + p.w_desc);
  const size_t n = p.host.size();
  DescChunk c;
  for (size_t o = 0; o < n; o += kDescChunkInts) {
    c.n = (int32_t)std::min<size_t>(kDescChunkInts, n - o);
    std::memcpy(c.v, p.host.data() + o, (size_t)c.n * sizeof(int32_t));
    launch(put_desc_kernel, 1, 256, 0, s, c, dst + o);
  }
  return hip_check("descriptor upload");
}

}  // namespace

namespace wisp {
// lets the host-only sources (the scheduler, the KV manager) report through wisp_last_error
wisp_status report_error(wisp_status st, const char *msg) { return fail(st, "%s", msg); }
wisp_status report_exception(const char *who, bool out_of_memory) {
  return out_of_memory ? fail(WISP_E_HOST_MEMORY, "%s: host memory exhausted", who)
                       : fail(WISP_E_INVALID, "%s: unexpected host-side exception", who);
}
}  // namespace wisp

// ------------------------------------------------------------------------------------------
// exported entry points
// ------------------------------------------------------------------------------------------
extern "C" {

const char *wisp_last_error(void) { return g_last_error; }

size_t wisp_workspace_size(const wisp_model *model, const wisp_batch_desc *desc) {
  return guarded_size([&]() -> size_t {
    if (check_model(model, false) != WISP_OK || check_desc(desc, false, true) != WISP_OK) return 0;
    Plan p;
    if (make_plan(p, model, desc, true) != WISP_OK) return 0;
    return p.total;
  });
}

size_t wisp_logits_workspace_size(const wisp_model *model, const wisp_batch_desc *desc) {
  return guarded_size([&]() -> size_t {
    if (check_model(model, false) != WISP_OK || check_desc(desc, false, true) != WISP_OK) return 0;
    Plan p;
    if (make_plan(p, model, desc, true) != WISP_OK) return 0;
    return logits_bytes(p.Mv, p.V);
  });
}

size_t wisp_accept_workspace_size(const wisp_batch_desc *desc, int32_t vocab) {
  return guarded_size([&]() -> size_t {
    if (check_desc(desc, false, false) != WISP_OK || vocab <= 0) return 0;
    Plan p;
    if (make_plan(p, nullptr, desc, false, vocab) != WISP_OK) return 0;
    return p.total;
  });
}

wisp_status wisp_pack_gate_up(void *dst, const void *w_gate, const void *w_up, int32_t d_ff, int32_t d_model,
                              int32_t dtype, void *stream) {
  return guarded("wisp_pack_gate_up", [&]() -> wisp_status {
    if (!dst || !w_gate || !w_up) return fail(WISP_E_INVALID, "NULL pointer");
    if (d_ff <= 0 || d_model <= 0) return fail(WISP_E_INVALID, "d_ff, d_model must be positive");
    hipStream_t s = (hipStream_t)stream;
    if (dtype == WISP_BF16) {
      if (d_ff % 32 || d_model % 16)
        return fail(WISP_E_UNSUPPORTED, "bf16 packing needs d_ff %% 32 == 0 and d_model %% 16 == 0");
      pack_gate_up_bf16((uint16_t *)dst, (const uint16_t *)w_gate, (const uint16_t *)w_up, d_ff, d_model, s);
    } else if (dtype == WISP_F32) {
      const size_t half = (size_t)d_ff * d_model * 4;
      if (hipMemcpyAsync(dst, w_gate, half, hipMemcpyDeviceToDevice, s) != hipSuccess ||
          hipMemcpyAsync((char *)dst + half, w_up, half, hipMemcpyDeviceToDevice, s) != hipSuccess)
        return fail(WISP_E_HIP, "copy failed");
    } else {
      return fail(WISP_E_UNSUPPORTED, "dtype %d", dtype);
    }
    return hip_check("pack");
  });
}

wisp_status wisp_pack_linear(void *dst, const void *src, int32_t rows, int32_t cols, int32_t dtype,
                             void *stream) {
  return guarded("wisp_pack_linear", [&]() -> wisp_status {
    if (!dst || !src) return fail(WISP_E_INVALID, "NULL pointer");
    if (rows <= 0 || cols <= 0) return fail(WISP_E_INVALID, "rows, cols must be positive");
    hipStream_t s = (hipStream_t)stream;
    if (dtype == WISP_BF16) {
      if (rows % 32 || cols % 16) return fail(WISP_E_UNSUPPORTED, "bf16 packing needs rows %% 32 == 0 and cols %% 16 == 0");
      pack_linear_bf16((uint16_t *)dst, (const uint16_t *)src, rows, cols, s);
    } else if (dtype == WISP_F32) {
      if (hipMemcpyAsync(dst, src, (size_t)rows * cols * 4, hipMemcpyDeviceToDevice, s) != hipSuccess)
        return fail(WISP_E_HIP, "copy failed");
    } else {
      return fail(WISP_E_UNSUPPORTED, "dtype %d", dtype);
    }
    return hip_check("pack");
  });
}

wisp_status wisp_verify(const wisp_model *model, const wisp_kv *kv, const wisp_batch_desc *desc,
                        const int32_t *tokens, const float *draft_probs, uint64_t rng_seed,
                        int32_t *accept_len, int32_t *out_tokens, float *target_logits,
                        void *workspace, size_t workspace_bytes, void *stream) {
  return guarded("wisp_verify", [&]() -> wisp_status {
    wisp_status st;
    if ((st = check_verify(model, kv, desc, tokens, accept_len, out_tokens)) != WISP_OK) return st;
    if (desc->B == 0) return WISP_OK;
    if (!workspace) return fail(WISP_E_INVALID, "NULL workspace");
    Plan p;
    if ((st = plan_verify(p, model, desc, draft_probs)) != WISP_OK) return st;
    // without a caller buffer the logits live in the workspace, after everything else
    const size_t need = p.total + (target_logits ? 0 : logits_bytes(p.Mv, p.V));
    if (workspace_bytes < need)
      return fail(WISP_E_WORKSPACE, "workspace %zu bytes < %zu needed", workspace_bytes, need);
    hipStream_t s = (hipStream_t)stream;
    char *ws = (char *)workspace;
    if (!target_logits) target_logits = reinterpret_cast<float *>(ws + p.total);
    if ((st = upload(p, ws, s)) != WISP_OK) return st;
    return run_verify(p, model, kv, desc, tokens, draft_probs, rng_seed, accept_len, out_tokens, target_logits,
                      ws, nullptr, s);
  });
}

wisp_status wisp_verify_noalloc(const wisp_model *model, const wisp_kv *kv, const wisp_batch_desc *desc,
                                const int32_t *tokens, const float *draft_probs, uint64_t rng_seed,
                                int32_t *accept_len, int32_t *out_tokens, float *target_logits, int32_t *fault,
                                void *stream) {
  return guarded("wisp_verify_noalloc", [&]() -> wisp_status {
    wisp_status st;
    if ((st = check_verify(model, kv, desc, tokens, accept_len, out_tokens)) != WISP_OK) return st;
    if (desc->B == 0) return WISP_OK;
    Plan p;
    // attention partials beyond the scratch would refuse the batch: fewer of them then
    int64_t rows = 0;
    for (int i = 0; i < desc->B; ++i) rows += desc->gamma[i] + 1;
    const size_t scratch_bytes = WISP_NOALLOC_SCRATCH_BYTES, logits = target_logits ? 0 : logits_bytes(rows, model->vocab);
    if ((st = plan_verify(p, model, desc, draft_probs, logits < scratch_bytes ? scratch_bytes - logits : 0)) != WISP_OK) return st;
    const size_t need = p.total + logits;
    if (need > (size_t)WISP_NOALLOC_SCRATCH_BYTES)
      return fail(WISP_E_WORKSPACE, "the batch needs %zu bytes of scratch, more than the %zu of the static "
                  "per-device scratch (use wisp_verify with a workspace)", need, (size_t)WISP_NOALLOC_SCRATCH_BYTES);
    char *ws = nullptr;
    if ((st = noalloc_scratch(&ws)) != WISP_OK) return st;
    hipStream_t s = (hipStream_t)stream;
    if (!target_logits) target_logits = reinterpret_cast<float *>(ws + p.total);
    if ((st = upload_by_arguments(p, ws, s)) != WISP_OK) return st;
    return run_verify(p, model, kv, desc, tokens, draft_probs, rng_seed, accept_len, out_tokens, target_logits,
                      ws, fault, s);
  });
}

wisp_status wisp_accept(const wisp_batch_desc *desc, int32_t vocab, const float *logits,
                        const int32_t *tokens, const float *draft_probs, uint64_t rng_seed,
                        int32_t *accept_len, int32_t *out_tokens, void *workspace,
                        size_t workspace_bytes, void *stream) {
  return guarded("wisp_accept", [&]() -> wisp_status {
    wisp_status st;
    if ((st = check_desc(desc, false, false)) != WISP_OK) return st;
    if (desc->B == 0) return WISP_OK;
    if (vocab <= 0) return fail(WISP_E_INVALID, "vocab must be positive");
    if (!logits || !tokens || !accept_len || !out_tokens || !workspace)
      return fail(WISP_E_INVALID, "NULL logits / tokens / outputs / workspace");
    Plan p;
    if ((st = make_plan(p, nullptr, desc, false, vocab)) != WISP_OK) return st;
    if (p.S > 0 && !draft_probs) return fail(WISP_E_INVALID, "draft_probs is NULL");
    if (workspace_bytes < p.total)
      return fail(WISP_E_WORKSPACE, "workspace %zu bytes < %zu needed", workspace_bytes, p.total);
    hipStream_t s = (hipStream_t)stream;
    char *ws = (char *)workspace;
    if ((st = upload(p, ws, s)) != WISP_OK) return st;
    StepDesc sd = step_desc(p, ws, desc, 0);
    sampler(sd, p.B, p.M, vocab, logits, tokens, draft_probs, desc->temperature, rng_seed, p.race_chunk,
            sampler_scratch(p, ws), accept_len, out_tokens, s);
    return hip_check("sampler launch");
  });
}

wisp_status wisp_attention(const wisp_model *model, const wisp_kv *kv, const wisp_batch_desc *desc,
                           const void *q, void *out, void *workspace, size_t workspace_bytes,
                           void *stream) {
  return guarded("wisp_attention", [&]() -> wisp_status {
    wisp_status st;
    if ((st = check_model(model, false)) != WISP_OK) return st;
    if ((st = check_desc(desc, true, true)) != WISP_OK) return st;
    if (desc->B == 0) return WISP_OK;
    if (!kv || !kv->k_pool || !kv->v_pool || kv->n_blocks <= 0) return fail(WISP_E_INVALID, "KV pools");
    if (kv->page_size != WISP_PAGE) return fail(WISP_E_UNSUPPORTED, "page_size must be %d", WISP_PAGE);
    if (!q || !out || !workspace) return fail(WISP_E_INVALID, "NULL q / out / workspace");
    Plan p;
    if ((st = make_plan(p, model, desc, true)) != WISP_OK) return st;
    if (!p.bf16 && p.max_tokens > 32768) return fail(WISP_E_UNSUPPORTED, "fp32 path supports <= 32768 tokens per request");
    if (workspace_bytes < p.total)
      return fail(WISP_E_WORKSPACE, "workspace %zu bytes < %zu needed", workspace_bytes, p.total);
    hipStream_t s = (hipStream_t)stream;
    char *ws = (char *)workspace;
    if ((st = upload(p, ws, s)) != WISP_OK) return st;
    StepDesc sd = step_desc(p, ws, desc, kv->n_blocks);
    if (p.bf16) {
      const AttnItem *items = reinterpret_cast<const AttnItem *>(ws + p.w_desc + p.i_items * 4);
      const AttnGroup *groups = reinterpret_cast<const AttnGroup *>(ws + p.w_desc + p.i_groups * 4);
      const int32_t *first = p.first.empty() ? nullptr : reinterpret_cast<const int32_t *>(ws + p.w_desc) + p.i_first;
      float *po = reinterpret_cast<float *>(ws + p.w_attn_o);
      float *pml = reinterpret_cast<float *>(ws + p.w_attn_ml);
      attention_bf16_main(sd, items, first, p.attn_waves(), p.item_rows, (const uint16_t *)q,
                          (const uint16_t *)kv->k_pool, (const uint16_t *)kv->v_pool, po, pml, (uint16_t *)out,
                          false, p.qdim, p.nq, p.nkv, p.hd, s);
      attention_bf16_combine(sd, groups, (int)p.groups.size(), p.item_rows, p.max_group_chunks, po, pml,
                             (uint16_t *)out, false, p.qdim, p.nq, p.nkv, p.hd, s);
    } else {
      attention_f32(sd, p.M, (const float *)q, (const float *)kv->k_pool, (const float *)kv->v_pool,
                    (float *)out, p.nq, p.nkv, p.hd, p.max_tokens, s);
    }
    return hip_check("attention launch");
  });
}

wisp_status wisp_uniform(uint64_t rng_seed, uint32_t req_id, uint32_t tag, uint32_t row, uint32_t n,
                         float *out, void *stream) {
  return guarded("wisp_uniform", [&]() -> wisp_status {
    if (!out && n) return fail(WISP_E_INVALID, "out is NULL");
    uniform_draws(rng_seed, req_id, tag, row, n, out, (hipStream_t)stream);
    return hip_check("uniform launch");
  });
}

wisp_status wisp_profile_enable(int on) {
  return guarded("wisp_profile_enable", [&]() -> wisp_status {
    if (!on) prof_collect();
    g_prof.on = on != 0;
    return WISP_OK;
  });
}

wisp_status wisp_profile_read(int kind, double *ms, int64_t *launches, double *bytes, double *flops) {
  return guarded("wisp_profile_read", [&]() -> wisp_status {
    if (kind < 0 || kind >= WISP_PROF_KINDS) return fail(WISP_E_INVALID, "profile kind %d", kind);
    prof_collect();
    if (ms) *ms = g_prof.ms[kind];
    if (launches) *launches = g_prof.launches[kind];
    if (bytes) *bytes = g_prof.bytes[kind];
    if (flops) *flops = g_prof.flops[kind];
    return WISP_OK;
  });
}

wisp_status wisp_profile_reset(void) {
  return guarded("wisp_profile_reset", [&]() -> wisp_status {
    prof_collect();
    for (int k = 0; k < WISP_PROF_KINDS; ++k) {
      g_prof.ms[k] = g_prof.bytes[k] = g_prof.flops[k] = 0.0;
      g_prof.launches[k] = 0;
    }
    return WISP_OK;
  });
}

wisp_status wisp_gemm_plan(int32_t M, int32_t N, int32_t K, int32_t out[4]) {
  return guarded("wisp_gemm_plan", [&]() -> wisp_status {
    if (!out) return fail(WISP_E_INVALID, "out is NULL");
    if (M < 1 || N < 1 || K < 1 || N % 32 || K % 16)
      return fail(WISP_E_INVALID, "M, N, K must be positive, N a multiple of 32, K of 16");
    const GemmCfg c = gemm_bf16_plan(M, N, K);
    out[0] = c.kind;
    out[1] = c.rb;
    out[2] = c.mt;
    out[3] = c.splits;
    return WISP_OK;
  });
}

wisp_status wisp_attention_plan(const wisp_model *model, const wisp_batch_desc *desc, int32_t out[6],
                                int32_t *items, int32_t max_items) {
  return guarded("wisp_attention_plan", [&]() -> wisp_status {
    wisp_status st;
    if (!out || max_items < 0 || (max_items > 0 && !items)) return fail(WISP_E_INVALID, "NULL out / items");
    if ((st = check_model(model, false)) != WISP_OK) return st;
    if ((st = check_desc(desc, false, true)) != WISP_OK) return st;
    if (model->dtype != WISP_BF16) return fail(WISP_E_UNSUPPORTED, "the fp32 attention has no plan");
    Plan p;
    if (desc->B > 0 && (st = make_plan(p, model, desc, true)) != WISP_OK) return st;
    out[0] = p.item_rows;
    out[1] = (int32_t)p.items.size();
    out[2] = p.attn_waves();
    out[3] = p.first.empty() ? 0 : 1;
    out[4] = (int32_t)p.groups.size();
    out[5] = p.max_group_chunks;
    const int n = std::min(max_items, out[1]);
    for (int k = 0, w = 0; k < n; ++k) {
      const AttnItem &it = p.items[k];
      if (p.first.empty()) w = k;
      else while (p.first[w + 1] <= k) ++w;
      const int32_t v[8] = {it.req, attn_kvh(it.kvh_rbg), attn_rbg(it.kvh_rbg, it.t0), it.t0 & ~kAttnFlags,
                            it.t1, it.t0 & kAttnWhole, w, 0};
      std::copy(v, v + 8, items + 8 * (size_t)k);
    }
    return WISP_OK;
  });
}

wisp_status wisp_check(void *workspace, void *stream) {
  return guarded("wisp_check", [&]() -> wisp_status {
    if (!workspace) return fail(WISP_E_INVALID, "workspace is NULL");
    hipStream_t s = (hipStream_t)stream;
    if (hipStreamSynchronize(s) != hipSuccess) return fail(WISP_E_HIP, "stream synchronize failed");
    int err = 0;
    if (hipMemcpy(&err, workspace, sizeof(int), hipMemcpyDeviceToHost) != hipSuccess)
      return fail(WISP_E_HIP, "error word read failed");
    if (err) {
      int zero = 0;
      (void)hipMemcpy(workspace, &zero, sizeof(int), hipMemcpyHostToDevice);
      return fail(WISP_E_DEVICE_INPUT, "device-side input check failed:%s%s",
                  (err & kErrToken) ? " token id out of range" : "",
                  (err & kErrBlock) ? " block id out of range" : "");
    }
    return WISP_OK;
  });
}

}  // extern "C"
