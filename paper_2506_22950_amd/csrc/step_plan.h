// Work split of a step launch through every layer (infs_decode_step_layers):
// how many work-groups of a KV head take prefix chunks, and where each live
// slot's response is cut into pieces for the response work-groups.
//
// A producer work-group loads one round of K/V into registers while the
// previous layer finishes, so that round is ready when the layer's queries
// arrive; whatever else it reads for the layer is loaded only after the
// queries (its registers hold the previous round until then) and lengthens
// the layer.  The per-layer launch's response chunks (a round each) fit this
// while every response work-group takes at most one.  When there are more
// chunks than response work-groups, the plan cuts each live response into
// `pieces` page ranges of near-equal length instead (piece c of a response
// of P pages holds pages [c*P/n, (c+1)*P/n)), at most one per response
// work-group, and picks the number of prefix work-groups with the cuts, so
// that the most tokens one producer reads is as small as it can be.  The
// split only decides which partial softmax holds which tokens; the merge
// combines whatever partials there are.
//
// Plain C++ with constexpr helpers (usable from host and device code) so that
// host tests can check the planner on its own.
#pragma once
#include <stdint.h>

#include "plan.h"

namespace infs {

// A wavefront holds the page numbers of its range one per lane, so a piece
// spans at most kWaves * 64 pages.
constexpr int kPiecePagesMax = kWaves * 64;
// Smallest piece the plan cuts on purpose: one page per wavefront.
constexpr int kPiecePagesMin = kWaves;

// First page of piece c of a response of `pages` pages cut into n pieces.
constexpr int piece_first_page(int c, int pages, int n) { return c * pages / n; }
// Pages per wavefront in a piece of `piece_pages` pages (wavefront w takes the
// w-th run of that many, the last runs may be short or empty).
constexpr int piece_wave_pages(int piece_pages) { return (piece_pages + kWaves - 1) / kWaves; }

struct StepRoles {
  int n_pre, n_suf, n_merge;  // work-groups per KV head taking prefix chunks, response pieces, merges
  int n_suffix_items;         // response items of the step (sum of pieces[])
  bool cut;                   // near-equal pieces chosen by the plan (else the per-layer launch's chunks)
};

namespace step_plan_detail {
inline int cdiv(int a, int b) { return (a + b - 1) / b; }
inline int pieces_at(int pages, int scmax, int t, int page_max) {
  const int lo = cdiv(pages, page_max), hi = pages < scmax ? pages : scmax;
  int n = cdiv(pages, t);
  if (n < lo) n = lo;
  if (n > hi) n = hi;
  return n;
}
}  // namespace step_plan_detail

// Cut the live responses (len[s] > 0 tokens, s < S) into at most w pieces in
// total, each slot into at most scmax and at least ceil(pages / page_max),
// with the largest piece as small as it can be (pieces of at least
// kPiecePagesMin pages where a response has them).  Writes pieces[s] (0 for an
// idle slot) and returns the largest piece in pages, or -1 when the slots
// cannot fit in w pieces or a slot's scmax pieces cannot hold it at page_max
// pages each (chunks of more tokens than that: split_tokens above 1024 with one
// piece per wavefront).
inline int cut_responses(const int32_t* len, int S, int w, int scmax, int32_t* pieces, int page_max = kPiecePagesMax) {
  using namespace step_plan_detail;
  auto total = [&](int t) {
    int n = 0;
    for (int s = 0; s < S; ++s)
      if (len[s] > 0) n += pieces_at(cdiv(len[s], kPageTokens), scmax, t, page_max);
    return n;
  };
  for (int s = 0; s < S; ++s)
    if (len[s] > 0 && cdiv(cdiv(len[s], kPageTokens), page_max) > scmax) return -1;
  if (total(page_max) > w) return -1;
  int lo = kPiecePagesMin, hi = page_max;  // smallest t with total(t) <= w
  while (lo < hi) {
    const int mid = (lo + hi) / 2;
    if (total(mid) <= w)
      hi = mid;
    else
      lo = mid + 1;
  }
  int largest = 0;
  for (int s = 0; s < S; ++s) {
    pieces[s] = 0;
    if (len[s] <= 0) continue;
    const int pages = cdiv(len[s], kPageTokens);
    pieces[s] = pieces_at(pages, scmax, lo, page_max);
    const int big = cdiv(pages, pieces[s]);
    if (big > largest) largest = big;
  }
  return largest;
}

// The split with the per-layer launch's chunks: one merge wavefront per slot,
// the producers divided between prefix and response chunks in proportion to
// their counts (at least one each when there are any), pieces[s] = the slot's
// chunks of `split` tokens.
inline StepRoles plan_step_roles_chunks(int nj, int S, int n_prefix_items, const int32_t* len, int split,
                                        int32_t* pieces) {
  using namespace step_plan_detail;
  StepRoles r{};
  r.n_merge = cdiv(S, kWaves) < nj - 1 ? cdiv(S, kWaves) : nj - 1;
  const int prod = nj - r.n_merge;
  for (int s = 0; s < S; ++s) {
    pieces[s] = len[s] > 0 ? cdiv(len[s], split) : 0;
    r.n_suffix_items += pieces[s];
  }
  const int npi = n_prefix_items, nsi = r.n_suffix_items;
  int pre = 0;
  if (npi > 0) {
    pre = (int)((int64_t)prod * npi / (npi + nsi > 1 ? npi + nsi : 1));
    pre = pre < 1 ? 1 : pre > npi ? npi : pre;
    if (nsi > 0 && pre > prod - 1) pre = prod - 1;
  }
  r.n_pre = pre > 0 ? pre : 0;
  r.n_suf = prod - r.n_pre;
  return r;
}

// Whether a step launch takes the prefix in chunks of kStepPrefixSplit tokens
// rather than the per-layer launch's (n_prefix_items of them): when the
// per-layer chunks would leave some producer two items.  Longer chunks free
// work-groups for the responses, but each prefix work-group then walks twice
// the blocks after its layer's queries arrive, which lengthens a layer that
// had room to spare.
inline bool longer_prefix_chunks(int nj, int S, int n_prefix_items, const int32_t* len, int split) {
  int32_t pieces[kMaxSlots];
  const StepRoles r = plan_step_roles_chunks(nj, S, n_prefix_items, len, split, pieces);
  return r.n_suffix_items > r.n_suf || r.n_pre < n_prefix_items;
}

// Roles of the nj work-groups per KV head and the response pieces of a step.
// n_prefix_items prefix chunks of prefix_split tokens; live slot s has len[s]
// tokens; the per-layer launch cuts responses into chunks of `split` tokens,
// at most scmax per slot.  Writes pieces[s].
//
// While the per-layer chunks leave every response work-group at most one
// chunk, they are kept: all of a producer's tokens are then in registers when
// its layer starts, and cutting finer only spreads the same bytes over more
// work-groups and partials (which measured slower).  Otherwise the number of
// prefix work-groups is chosen among the fewest that take k chunks each
// (k = 1, 2, ...) to minimise the largest per-producer token count, prefix
// tokens counted twice (every slot's merge waits for all prefix chunks, so a
// prefix work-group's second chunk delays the whole layer), and the responses
// are cut into pieces, at most one per remaining work-group; when the live
// slots outnumber those work-groups the chunks stay, dealt round robin.
inline StepRoles plan_step_roles(int nj, int S, int n_prefix_items, int prefix_split, const int32_t* len, int split,
                                 int scmax, int32_t* pieces) {
  using namespace step_plan_detail;
  StepRoles r = plan_step_roles_chunks(nj, S, n_prefix_items, len, split, pieces);
  if (r.n_suffix_items <= r.n_suf) return r;
  const int prod = nj - r.n_merge, chunks = r.n_suffix_items;
  int best = -1, best_pre = r.n_pre;
  const int kmax = n_prefix_items > 0 ? n_prefix_items : 1;
  for (int k = 1; k <= kmax; ++k) {
    const int n_pre = n_prefix_items > 0 ? cdiv(n_prefix_items, k) : 0;
    if (k > 1 && n_pre == cdiv(n_prefix_items, k - 1)) continue;
    const int w = prod - n_pre;
    if (w < 1) continue;
    const int pre_tokens = n_pre > 0 ? 2 * cdiv(n_prefix_items, n_pre) * prefix_split : 0;
    const int big = cut_responses(len, S, w, scmax, pieces);
    const int resp_tokens = big > 0 ? big * kPageTokens : cdiv(chunks, w) * split;
    const int cost = pre_tokens > resp_tokens ? pre_tokens : resp_tokens;
    if (best < 0 || cost < best) {
      best = cost;
      best_pre = n_pre;
    }
  }
  if (best < 0) {  // no split beats the chunks (a single producer)
    plan_step_roles_chunks(nj, S, n_prefix_items, len, split, pieces);
    return r;
  }
  r.n_pre = best_pre;
  r.n_suf = prod - best_pre;
  const int big = cut_responses(len, S, r.n_suf, scmax, pieces);
  r.cut = big > 0;
  if (!r.cut)
    for (int s = 0; s < S; ++s) pieces[s] = len[s] > 0 ? cdiv(len[s], split) : 0;
  r.n_suffix_items = 0;
  for (int s = 0; s < S; ++s) r.n_suffix_items += pieces[s];
  return r;
}

// Most tokens, in whole pages, the plan deals to one response work-group of a KV head (0 < n_suf <
// 2 * kMaxSlots of them; work-group i takes items i, i + n_suf, ... of the slots'
// pieces in order).
inline int most_response_tokens(const StepRoles& r, int S, const int32_t* len, int split, const int32_t* pieces) {
  int32_t tokens[2 * kMaxSlots] = {};
  int it = 0, most = 0;
  for (int s = 0; s < S; ++s) {
    const int pages = step_plan_detail::cdiv(len[s], kPageTokens);
    for (int c = 0; c < pieces[s]; ++c, ++it) {
      int32_t& t = tokens[it % r.n_suf];
      const int first = r.cut ? piece_first_page(c, pages, pieces[s]) : c * (split / kPageTokens);
      const int next = r.cut ? piece_first_page(c + 1, pages, pieces[s]) : first + split / kPageTokens;
      t += ((next < pages ? next : pages) - first) * kPageTokens;
      if (t > most) most = t;
    }
  }
  return most;
}

// Whether the prefix work-groups of a step launch load a layer's first chunk behind
// the arrival of the layer before (StepArgs::prefix_early) rather than when the layer
// may start; early_prefix_varies names the shapes where it may be either.  The 32-row
// tile asks for the most: its two row groups each load the whole 128-token
// chunk at once (the 16-row tile loads it once, wider tiles two blocks at a time).
// With long responses, whose partials and merges fill a layer's end, that costs more
// than it hides.  Loads at the layer's start and behind the arrival, us a step: 28
// layers, prompt 2048, 16 slots of 2 rows, mean response 140 tokens 270.8 and 264.6,
// 550 324.9 and 322.1, 750 360.4 and 362.1, 1900 330.8 and 334.4, 3400 319.3 and 330.7;
// 16 KV heads (12 layers) 140 159.7 and 152.2, 750 284.1 and 284.6, 2400 292.8 and 299.9;
// prompt 3000 140 149.9 and 144.9, 2400 170.3 and 173.1.  Elsewhere long responses gain
// too or stay: 64 rows (4 heads per KV head) 2400 194.1 and 185.3, (32 slots) 2700 192.1
// and 192.2, 3400 159.6 and 151.6; 16 rows (1 head) 3400 145.4 and 146.8, (two prompts)
// 2400 153.7 and 154.0; E4M3 3400 307.4 and 294.0; head size 64, 32 rows, 3400 124.2 and
// 121.9; plain rows up to 600 tokens 123.7 and 121.7, 1800 134.8 and 136.4.
constexpr bool early_prefix_varies(bool mfma, bool kv8, int head_dim, int prefix_rows) {
  return mfma && !kv8 && head_dim == 128 && prefix_rows == 32;
}
constexpr int kEarlyPrefixTokens = 768;
inline bool early_prefix_pays(bool varies, const int32_t* len, int S) {
  int64_t tokens = 0, live = 0;
  for (int s = 0; s < S; ++s) {
    tokens += len[s];
    live += len[s] > 0;
  }
  return !varies || tokens < live * kEarlyPrefixTokens;
}

// The split of a step with one response piece per wavefront (bf16 and E4M3
// pages): the four wavefronts of a response work-group take a piece each, of
// whichever slots, and hand in a partial each, without a barrier or a combine
// between them.  With many slots the work-group pieces of plan_step_roles are
// dealt several to a work-group, each loaded, combined and counted in turn;
// here every wavefront has one.  The price is more partials, which the merges
// pay.  It is taken where all of these hold (us a step of 12 layers, without and
// with it, 32/8 heads of 128 on four prompts of 256 to 4096 tokens or 16/8 heads
// on one of 1024, unless said otherwise; ms are whole group decodes):
// * Four times its largest piece, what a work-group then reads, is no more than
//   plan_step_roles deals to a work-group.  Four prompts, 64 slots up to 256
//   tokens 404 and 288, up to 700 tokens 499 and 404, up to 2048 tokens 934 and
//   777, 24 of the 64 live 411 and 332; one prompt, 64 slots up to 1000 tokens
//   437 and 362; head size 64, up to 2000 tokens 583 and 381; 8 heads per KV
//   head, up to 1000 tokens 542 and 458.  Past the line: 16 live of 64 up to 700
//   tokens 255 and 265, one prompt, 24 live up to 2000 tokens 258 and 276, 8 heads
//   per KV head, 32 live up to 1000 tokens 376 and 397.
// * kWaveMinItems4 / 4 per-layer chunks to a response work-group and more: one
//   prompt, 64 slots up to 300 tokens (1.6) 298 and 308, 48 live (1.2) 274 and
//   301; at the line 48 live up to 700 tokens 295 and 305, but four prompts,
//   64 slots up to 256 tokens (1.9) the 404 and 288 above.  kWaveMinCut4 / 4 where
//   plan_step_roles cuts, so every work-group has one piece: the steps of a decode
//   on 40 slots (prompt 2048, 1.8 to 2.1) 627 ms and 701.
// * kWaveMinLive live slots: fewer are cut into up to 32 partials each.  64 slots on
//   four prompts, 36 layers, the steps with 4 to 11 live 3496 ms and 4013, with 20 to
//   31 live 2180 and 2068; head size 64 (12 layers) 642 and 649, with 20 to 39 520 and 440.
// * More than kWaveMinSlots slots, and more than half as many as work-groups per
//   KV head.  The merge work-groups it frees are few with fewer: 32 slots up to
//   2048 tokens (28 layers) 860 and 923, 16 slots 472 and 621.  With 4 KV heads
//   (128 work-groups) plan_step_roles has a work-group for every slot: 64 slots up
//   to 4000 tokens on two prompts 680 and 812, on one 663 and 594, up to 6000
//   tokens 996 and 947, 48 live 716 and 752; 2 KV heads up to 9000 tokens (6
//   layers) 334 and 371.
// * For E4M3 pages under a 128-row prefix tile (`wide_e4m3`) not in place of whole
//   chunks dealt round robin: one prompt of 2048, 64 slots up to 500 tokens 314 and
//   323, up to 1000 tokens 371 and 530, up to 2000 tokens 560 and 605; in place of cut
//   pieces, the steps of a decode on 64 slots with 12 to 31 live 662 ms and 560.  Under
//   64 rows and fewer in place of both: four prompts, up to 256 tokens 346 and 264, up
//   to 2048 tokens 617 and 596, 16 rows up to 1500 tokens 473 and 295.
// Whole group decodes without it, and with it by this rule: 64 slots on four prompts
// (36 layers) 13936 ms and 12705, its E4M3 cache (12 layers) 3770 and 3635, d = 64 2940
// and 2235; one prompt, 64 slots 2125 and 1973; two prompts of 32 slots 2015 and 1758;
// three of 16 2257 and 1924; eight of 8 2993 and 2445; 16 KV heads (8 layers) 5911 and
// 5241.
//
// A merge work-group only waits while the others load, so the merges run on
// fewer than one wavefront each: two to a wavefront, and four where more than two
// prompts walk the layers on their own, unless the responses are deep
// (kWaveDeepItems chunks and more).  Their number follows the slots, not the live
// ones: 16 of 64 live up to 256 tokens 231 and 296 with fewer.  One, two, four
// merges to a wavefront: one prompt, 64 slots up to 1000 tokens (28 layers) 1114,
// 837, 913; two prompts up to 500 tokens 233, 222, 243 (E4M3 202, 204, 252), up to
// 1500 tokens 543, 504, 485; three up to 1000 tokens 376, 348, 345; 4 prompts (36
// layers) up to 512 tokens 1142, 1203, 961, up to 2048 tokens 2534, 2243, 2450.
// The prefix is weighed kWavePrefixCost halves, as its chunks are walked after
// the layer's queries arrive.
// False where it does not apply, or where pieces would not fit a wavefront.
constexpr int kWaveMinSlots = 32, kWaveMinLive = 12, kWaveMinItems4 = 7, kWaveMinCut4 = 9;
constexpr int kWaveDeepItems = 5, kWavePrefixCost = 3;
constexpr int kWavePagesMax = 64;  // a wavefront holds the page numbers of its piece one per lane
inline bool plan_step_waves(int nj, int S, int prompts, int n_prefix_items, int prefix_split, const int32_t* len, int split, int scmax,
                            int32_t* pieces, StepRoles* out, bool wide_e4m3 = false) {
  using namespace step_plan_detail;
  StepRoles r = plan_step_roles_chunks(nj, S, n_prefix_items, len, split, pieces);
  if (S <= kWaveMinSlots || 2 * S <= nj || 4 * r.n_suffix_items < kWaveMinItems4 * r.n_suf) return false;
  int live = 0;
  for (int s = 0; s < S; ++s) live += len[s] > 0;
  if (live < kWaveMinLive) return false;
  const StepRoles groups = plan_step_roles(nj, S, n_prefix_items, prefix_split, len, split, scmax, pieces);
  if (groups.cut ? 4 * r.n_suffix_items < kWaveMinCut4 * r.n_suf : wide_e4m3) return false;
  const int dealt = groups.n_suf > 0 ? most_response_tokens(groups, S, len, split, pieces) : 0;
  const int merges = prompts > 2 && r.n_suffix_items < kWaveDeepItems * r.n_suf ? 4 : 2;  // to a wavefront
  r.n_merge = cdiv(S, merges * kWaves) < nj - 1 ? cdiv(S, merges * kWaves) : nj - 1;
  const int prod = nj - r.n_merge;
  int best = -1, best_pre = 0;
  const int kmax = n_prefix_items > 0 ? n_prefix_items : 1;
  for (int k = 1; k <= kmax; ++k) {
    const int n_pre = n_prefix_items > 0 ? cdiv(n_prefix_items, k) : 0;
    if (k > 1 && n_pre == cdiv(n_prefix_items, k - 1)) continue;
    const int w = prod - n_pre;
    if (w < 1) continue;
    const int big = cut_responses(len, S, w * kWaves, scmax, pieces, kWavePagesMax);
    if (big <= 0) continue;
    const int pre_tokens = kWavePrefixCost * k * prefix_split / 2, resp_tokens = big * kPageTokens * kWaves;
    const int cost = pre_tokens > resp_tokens ? pre_tokens : resp_tokens;
    if (best < 0 || cost < best) {
      best = cost;
      best_pre = n_pre;
    }
  }
  if (best < 0) return false;
  r.n_pre = best_pre;
  r.n_suf = prod - best_pre;
  if (cut_responses(len, S, r.n_suf * kWaves, scmax, pieces, kWavePagesMax) * kPageTokens * kWaves > dealt) return false;
  r.cut = true;
  r.n_suffix_items = 0;
  for (int s = 0; s < S; ++s) r.n_suffix_items += pieces[s];
  *out = r;
  return true;
}

// Whether a per-layer launch of bf16 Q/K/V whose responses are all at most
// kShortResponse tokens (a load round of a wavefront) and at most its share of a
// chunk gives each response and each merge a wavefront, four to a work-group.
// Every work-group takes its place on the GPU for the length of the exchange,
// however little it reads: 64 probe samples of up to 16 tokens are 512 response and
// 512 merge work-groups, in three turns with the prefix chunks.  `busy` counts the
// prefix, response and merge work-groups; the ones that clear idle slots leave at
// once.  `partials` is the most a slot merges: a merge work-group loads them with
// four wavefronts, a merge wavefront alone, so it pays
// * past one turn where a merge is one round of loads.  12 per-layer launches of
//   responses up to 40 tokens, us without and with it, 16/8 heads of 128: prompt
//   2048, 1152 work-groups 229 and 186, 640 186 and 177, 512 177 and 178; prompt 256,
//   528 161 and 152, 400 144 and 151; E4M3, 1088 199 and 193, 448 172 and 181; 4 KV
//   heads 544 170 and 159; 8/8 heads 1088 198 and 157, but 960 153 and 156.  The length
//   matters little: prompt 2048, 1152 work-groups, up to 64 tokens 232 and 190, up to
//   17 tokens 222 and 185.
// * past two turns with two or three rounds.  32/8 heads of 128, prompts up to 1500,
//   1248 work-groups 248 and 205, 992 236 and 198, 736 168 and 190; up to 2000, 1280
//   260 and 228, 768 184 and 213; head size 64, 64/8 heads, 1192 216 and 174, 808 152
//   and 155; 4 KV heads, prompt 4000, 640 195 and 203.
// * not with more: 32/8 heads, prompts up to 4096, 1488 work-groups 332 and 373.
// Longer responses would be cut otherwise than in a step launch of split mode 0.
constexpr int kShortResponse = 64;
inline bool short_responses_pay(int busy, int resident, int partials, int outputs) {
  const int rounds = step_plan_detail::cdiv(partials, merge_wave_partials(outputs));
  return rounds <= 1 ? busy > resident : rounds <= 3 && busy > 2 * resident;
}

}  // namespace infs
