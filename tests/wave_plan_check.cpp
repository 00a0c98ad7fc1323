// Host check of the wavefront split of a step launch (plan_step_waves in
// csrc/step_plan.h) and of the line for short responses in per-layer launches, built with g++ by tests/test_wave_plan.py: over random slot
// lengths and launch shapes, the roles add up, there is a wavefront for every
// item, every live response's pieces are whole page ranges that tile it,
// pieces stay within the limits per slot and per wavefront, and no work-group
// reads more than the split by work-groups would deal to one.  Chunk lengths are
// drawn over the whole accepted range, the pieces a slot has room for as
// infs_create sizes them: the chunks of the longest response, padded to whole
// 128-byte lines of records.
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <random>
#include <vector>

#include "step_plan.h"

using namespace infs;

static int fails = 0;
#define CHECK(cond)                                                             \
  do {                                                                          \
    if (!(cond) && ++fails < 20) std::printf("case %d FAIL %s\n", cs, #cond);   \
  } while (0)

int main() {
  std::mt19937 rng(7);
  auto uni = [&](int a, int b) { return std::uniform_int_distribution<int>(a, b)(rng); };
  int applied = 0;
  for (int cs = 0; cs < 20000; ++cs) {
    const int nj = (int[]){2, 3, 8, 32, 63, 64, 128}[uni(0, 6)], S = uni(1, kMaxSlots);
    const int split = uni(0, 1) ? (int[]){128, 256, 512}[uni(0, 2)] : 128 * uni(1, kMaxSplit / 128);
    const int cap = uni(0, 2) ? uni(1, 4096) : uni(1, 20000), idle = uni(0, 3) ? 0 : uni(0, 90);
    const int line = std::max(1, kRecordsPerLine / (1 << uni(0, 3)));  // records of 1, 2, 4, 8 heads per KV head
    const int scmax = ((cap + split - 1) / split + line - 1) / line * line, npi = uni(0, 64);
    std::vector<int32_t> len(S, 0), pieces(S, -1);
    for (int s = 0; s < S; ++s)
      if (uni(0, 99) >= idle) len[s] = uni(1, cap);
    StepRoles r{};
    if (!plan_step_waves(nj, S, uni(1, 4), npi, 256, len.data(), split, scmax, pieces.data(), &r)) continue;
    ++applied;
    CHECK(S > kWaveMinSlots && 2 * S > nj && r.cut);
    CHECK(r.n_merge >= 1 && r.n_suf >= 1 && r.n_pre >= (npi > 0) && r.n_pre <= npi);
    CHECK(r.n_pre + r.n_suf + r.n_merge == nj);
    int items = 0, largest = 0;
    for (int s = 0; s < S; ++s) {
      if (len[s] == 0) {
        CHECK(pieces[s] == 0);
        continue;
      }
      const int pages = (len[s] + kPageTokens - 1) / kPageTokens, n = pieces[s];
      CHECK(n >= 1 && n <= pages && n <= scmax);
      if (n < 1) continue;
      items += n;
      CHECK(piece_first_page(0, pages, n) == 0 && piece_first_page(n, pages, n) == pages);
      for (int c = 0; c < n; ++c) {
        const int p = piece_first_page(c + 1, pages, n) - piece_first_page(c, pages, n);
        CHECK(p >= 1 && p <= kWavePagesMax);
        largest = std::max(largest, p);
      }
    }
    CHECK(items == r.n_suffix_items && items <= r.n_suf * kWaves);
    std::vector<int32_t> gp(S, 0);
    const StepRoles g = plan_step_roles(nj, S, npi, 256, len.data(), split, scmax, gp.data());
    std::vector<int> dealt(g.n_suf, 0);
    for (int s = 0, it = 0; s < S; ++s)
      for (int c = 0; c < gp[s]; ++c, ++it) {
        const int pages = (len[s] + kPageTokens - 1) / kPageTokens;
        const int pg = piece_first_page(c + 1, pages, gp[s]) - piece_first_page(c, pages, gp[s]);
        dealt[it % g.n_suf] += kPageTokens * (g.cut ? pg : std::min(split / kPageTokens, pages - c * split / kPageTokens));
      }
    CHECK(kWaves * largest * kPageTokens <= *std::max_element(dealt.begin(), dealt.end()));
  }
  // short responses a wavefront each (512 resident work-groups), measured shapes on both sides of the
  // line: busy work-groups, partials of a merge, outputs of a merge, and whether it was faster
  const struct { int busy, partials, outputs; bool pays; } shorts[] = {
      {1152, 17, 256, true}, {640, 17, 256, true}, {512, 17, 256, false}, {384, 17, 256, false}, {400, 3, 256, false},
      {448, 9, 256, false}, {640, 33, 256, false}, {1248, 13, 512, true}, {736, 13, 512, false}, {576, 9, 512, false},
      {616, 13, 512, false}, {768, 17, 512, false}, {1488, 33, 512, false}, {976, 33, 512, false}, {640, 9, 1024, false},
      {560, 4, 1024, true}, {2560, 9, 1024, true}, {2208, 5, 512, true}};
  for (int cs = 0; cs < (int)(sizeof shorts / sizeof *shorts); ++cs)
    CHECK(short_responses_pay(shorts[cs].busy, 512, shorts[cs].partials, shorts[cs].outputs) == shorts[cs].pays);
  // the prefix loads ahead of a layer: all but long responses on the bf16 32-row tile
  {
    const int cs = -1;
    const int32_t shorter[3] = {767, 0, 768}, longer[3] = {768, 0, 768};
    CHECK(early_prefix_pays(true, shorter, 3) && !early_prefix_pays(true, longer, 3) && early_prefix_pays(false, longer, 3));
    CHECK(early_prefix_varies(true, false, 128, 32) && !early_prefix_varies(true, true, 128, 32));
    CHECK(!early_prefix_varies(true, false, 64, 32) && !early_prefix_varies(true, false, 128, 64));
  }
  std::printf("applied %d failures %d\n", applied, fails);
  return fails || applied < 1000;
}
