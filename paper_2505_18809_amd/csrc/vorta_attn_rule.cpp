// The rule that chooses the form of a bf16 attention launch.  Nothing in this file touches the GPU.
#include <algorithm>

#include "vorta_internal.h"

namespace vorta {

// ------------------------------------------------------------------------------------------
// Which kernel, and how a launch is cut.  The pipelined kernel does most work per cycle but in
// 256-row items, a workgroup per CU, the window tiles in launches of their own; the split kernel takes a
// quarter of the rows per item, all of a layer in one launch, at 70 to 85 % of the rate.  Which is
// faster depends on how the items fill the chip, so that is estimated: the time of a launch is that of
// handing its items, in launch order, to whichever CU is free first.  Item costs in microseconds, fitted
// to 140 measured layers (256 to 75,600 tokens, 1 to 40 heads, one route or all): the form chosen from
// them is on average 0.6 %, at most 8 %, slower than the fastest one measured.
//   pipelined, per 64-key block of a 256-row item 1.45, of a half-row item 0.85; window form 1.7 and 0.95
//   4-wavefront window form, two workgroups per CU, per 64-key block 1.55
//   split kernel with two key shares 0.52 (two workgroups share a CU: counted as one at twice the rate)
// Measured, us (pipelined with the last 128 items in halves / split with four / two key shares):
//   3,072 tokens: 2 dense heads 44 / 29 / 34; 8 window heads 35 / 46 / 36; 8 heads on all routes 88 / 53 / 50
//   9,216 tokens: 4 dense heads 252 / 229 / 233; 16 window heads 234 / 257 / 204; 40 heads 762 / 890 / 788
//   32,760 tokens: 1 dense head 497 / 569 / 567; 4 window heads 219 / 264 / 206; 16 of them 701 / 993 / 812
// ------------------------------------------------------------------------------------------
namespace {
struct Batch {
  int items;
  double cost;       // of each
};
struct Segment {
  int items, blocks;  // 256-row (or 64-row) items, 64-key blocks of each
  bool win;
};

// Time at which `units` processors have finished the batches, each item going to the first one free.
// Processors are kept in groups of equal time; a group list that runs full forgets its finest step.
double makespan(const Batch* batch, int n, int units) {
  constexpr int MAX = 48;
  double t[MAX];
  int c[MAX], ng = 1;
  t[0] = 0.0;
  c[0] = units;
  for (int b = 0; b < n; ++b) {
    int left = batch[b].items;
    while (left > 0) {
      const double done = t[0] + batch[b].cost;
      const int take = std::min(left, c[0]);
      left -= take;
      c[0] -= take;
      if (c[0] == 0) {
        --ng;
        for (int i = 0; i < ng; ++i) { t[i] = t[i + 1]; c[i] = c[i + 1]; }
      }
      int at = 0;
      while (at < ng && t[at] < done - 1e-6) ++at;
      if ((at < ng && t[at] < done + 1e-6) || ng == MAX) {
        c[std::min(at, ng - 1)] += take;
      } else {
        for (int i = ng; i > at; --i) { t[i] = t[i - 1]; c[i] = c[i - 1]; }
        t[at] = done;
        c[at] = take;
        ++ng;
      }
    }
  }
  return t[ng - 1];
}

constexpr double LAUNCH_US = 6.0;

// Pipelined launch of the segments with its last `split` items issued as half-row items.
double pipe_time(const Segment* seg, int n, int split, int units) {
  int total = 0;
  for (int i = 0; i < n; ++i) total += seg[i].items;
  if (total == 0) return 0.0;
  int whole = total - std::min(split, total), nb = 0;
  Batch b[8];
  for (int pass = 0; pass < 2; ++pass) {
    int keep = whole;
    for (int i = 0; i < n; ++i) {
      const double fixed = seg[i].win ? 6.0 : 3.0, full = seg[i].win ? 1.7 : 1.45, half = seg[i].win ? 0.95 : 0.85;
      const int w = std::min(keep, seg[i].items);
      keep -= w;
      const int items = pass == 0 ? w : 2 * (seg[i].items - w);
      if (items > 0) b[nb++] = {items, fixed + (pass == 0 ? full : half) * seg[i].blocks};
    }
  }
  return LAUNCH_US + makespan(b, nb, units);
}

// How many of the last items to issue as half-row items.  The last items of a launch leave most CUs idle
// while a few finish them; two half-row items cost 1.2 times the whole one, so halves pay for a
// remainder of up to half the CUs and not for one that nearly fills them (two dense heads of 32,760 tokens
// are 256 items: 958 us with the last 128 in halves, 851 us whole).
// At most `most`.
int best_split(const Segment* seg, int n, int most, int units, double* time) {
  int total = 0;
  for (int i = 0; i < n; ++i) total += seg[i].items;
  const int candidates[4] = {units / 2, units / 4, total % units, 0};
  int best = 0;
  *time = 1e30;
  for (int s : candidates) {
    s = std::min(s, most);
    const double us = pipe_time(seg, n, s, units);
    if (us < *time) {
      *time = us;
      best = s;
    }
  }
  return best;
}

double split_time(const Segment* seg, int n, int units) {
  Batch b[4];
  int nb = 0;
  for (int i = 0; i < n; ++i)
    if (seg[i].items > 0) b[nb++] = {seg[i].items, seg[i].win ? 4.7 + 0.54 * seg[i].blocks : 2.5 + 0.52 * seg[i].blocks};
  return nb ? LAUNCH_US + makespan(b, nb, units) : 0.0;
}
}  // namespace

// mix: the launch is the full-attention branch of Eq. 5.  win_text = false: the text rows of the window heads are
// left out.  units: CUs of the device.
AttnForm choose_attention_form(const vorta_plan* p, const RouteLists& rl, bool mix, bool win_text, int units) {
  const int n_win = rl.count[1];
  const int rows_c = (int)(p->Lc + p->d.n_text), n_text = win_text ? p->d.n_text : 0;
  const int blocks_n = (int)((p->N + 63) / 64), blocks_c = (rows_c + 63) / 64;
  auto items_of = [](int64_t rows, int bm) { return (int)((rows + bm - 1) / bm); };
  auto list_items = [&](int l) { return n_win * (int)(p->win_list[l].size() / 4); };

  // Everything in 64-row items: one launch of the split kernel if that is estimated to be the faster form.
  // With no more items than CUs four key shares shorten each of them (3,072 keys: 29 us against
  // 34 with two shares; 256 keys, where the longer merge shows: 9.6 against 8.8).
  const Segment fine[4] = {{n_win * items_of(n_text, ATTN_ROWS_SPLIT), blocks_n, false}, {rl.count[0] * items_of(p->N, ATTN_ROWS_SPLIT), blocks_n, false},
                           {rl.count[2] * items_of(rows_c, ATTN_ROWS_SPLIT), blocks_c, false}, {list_items(2), p->win_blocks[2], true}};
  int fine_items = 0, longest = 0;
  for (const Segment& s : fine) {
    fine_items += s.items;
    if (s.items) longest = std::max(longest, s.blocks);
  }
  AttnForm f = {};
  f.empty = fine_items == 0;
  if (f.empty) return f;
  const Segment coarse[4] = {{n_win * items_of(n_text, ATTN_ROWS_LONG), blocks_n, false}, {rl.count[0] * items_of(p->N, ATTN_ROWS_LONG), blocks_n, false},
                             {rl.count[2] * items_of(rows_c, ATTN_ROWS_LONG), blocks_c, false}, {list_items(0), p->win_blocks[0], true}};
  f.n_long = coarse[0].items + coarse[1].items + coarse[2].items;
  f.n_big = coarse[3].items;
  f.shares = fine_items <= units && longest >= 16 ? 4 : 2;
  f.split_all = fine_items <= units;
  f.together = f.n_long && f.n_big && !mix;
  if (!f.split_all || p->force_form) {
    double t_long, t_big, t_both;
    f.half_long = best_split(coarse, 3, f.n_long, units, &t_long);
    f.half_big = best_split(coarse + 3, 1, f.n_big, units, &t_big);
    const Batch small = {list_items(1), 5.0 + 1.55 * p->win_blocks[1]};
    const double t_small = small.items ? LAUNCH_US + makespan(&small, 1, 2 * units) : 0.0;
    double t_pipe = t_long + t_big + t_small;
    if (f.together) {
      f.half_big = best_split(coarse, 4, f.n_big, units, &t_both);
      t_pipe = t_both + t_small;
    }
    // far above the sizes where the split kernel can win there is nothing to estimate
    int64_t work = 0;
    for (const Segment& s : fine) work += (int64_t)s.items * s.blocks;
    if (!f.split_all && work < (int64_t)4000 * units) {
      const double t_split_win = split_time(&fine[3], 1, units);
      f.split_win = n_win && t_long + t_split_win < t_pipe;
      f.split_all = split_time(fine, 4, units) < std::min(t_pipe, n_win ? t_long + t_split_win : t_pipe);
    }
  }
  if (p->force_form) {           // tests: one form for every size
    f.split_all = p->force_form == 2 || p->force_form == 4;
    if (f.split_all) f.shares = p->force_form;
    f.split_win = p->force_form == 5 && n_win;
    if (p->force_halves >= 0) {
      f.half_long = std::min(p->force_halves, f.n_long);
      f.half_big = std::min(p->force_halves, f.n_big);
    }
  }
  f.together = f.together && !f.split_all && !f.split_win;
  return f;
}

}  // namespace vorta

using namespace vorta;

extern "C" {

// For the tests, not part of the ABI: every form of the bf16 attention launch at any size.  form: 0 = by the rule;
// 2, 4 = split kernel with so many key shares; 3 = pipelined kernels; 5 = pipelined, window rows on the split
// kernel.  halves: items issued as half-row items, -1 = by the rule.  A property of the plan; not to be changed
// while a call on it runs.
int vorta_test_force_form(vorta_plan* p, int32_t form, int32_t halves) {
  if (!p || !(form == 0 || (form >= 2 && form <= 5)) || halves < -1) return fail(VORTA_EINVAL, "form %d, halves %d", form, halves);
  p->force_form = form;
  p->force_halves = halves;
  return VORTA_OK;
}

// What a layer call (mix = 0) or the full-attention launch of the mixture (1) chooses with `units` CUs:
// {split_all, shares, split_win, together, n_long, half_long, n_big, half_big}.
int vorta_test_form(const vorta_plan* p, const uint8_t* routes_host, int32_t mix, int32_t units, int32_t out[8]) {
  RouteLists rl;
  if (int rc = split_routes(p, routes_host, &rl)) return rc;
  const AttnForm f = choose_attention_form(p, rl, mix != 0, true, units);
  const int32_t v[8] = {f.split_all, f.shares, f.split_win, f.together, f.n_long, f.half_long, f.n_big, f.half_big};
  std::copy(v, v + 8, out);
  return VORTA_OK;
}

}  // extern "C"
