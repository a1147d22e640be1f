// The rule that chooses the form of a bf16 attention launch.  Nothing in this file touches the GPU.
#include <algorithm>

#include "vorta_internal.h"

namespace vorta {

// ------------------------------------------------------------------------------------------
// Which kernel, and how a launch is cut.  The pipelined kernel does most work per cycle but in 256-row items, a
// workgroup per CU, and the window rows that fill no such item -- or all of them -- in 128-row items in a launch
// of their own; the split kernel takes 64 rows per item, all of a layer in one launch, at 70 to 85 % of the rate.  Which is
// faster depends on how the items fill the chip, so that is estimated: the time of a launch is that of
// handing each XCD's items, in launch order, to whichever of its CUs is free first.
//
// Item costs are microseconds, fixed + per 64-key block, fitted to 2,098 measured layers (256 to 80,000 tokens, 1 to 40
// heads, every route alone and mixed, with and without text, every form timed on each) with the kernels of that time: before
// window keys were computed, query rows of the split kernel came by direct loads and arguments in one batch, and key shares were merged
// in two barriers.  With the kernels as they are the form chosen for 1,260 others is 1.1 % slower than the fastest on average, 32 of
// them by more than 10 %, one by 37 % (profiles/attention_forms.txt); most of those are window heads alone whose items fill the chip once or twice.  Costs
// fitted to earlier versions of the kernels were 2.6 % off on average, 71 of 798 by more than 10 % and up to 55 %, and
// without items of 128 rows a layer of 768 tokens, 24 window heads and 32-token tiles took 20.2 us instead of 17.1.
// ------------------------------------------------------------------------------------------
namespace {
struct Cost {
  double fixed, block;
  double of(double blocks) const { return fixed + block * blocks; }
};
constexpr Cost LONG = {4.0, 0.98}, LONG_HALF = {4.0, 0.737};   // pipelined: dense, core-set and text items of 256 rows; of half
constexpr Cost WIN = {7.4, 1.45}, WIN_HALF = {7.4, 0.867};     // pipelined: window items of 256 rows; of half
// 4-wavefront window items and split kernel with two key shares: two workgroups share a CU, counted as one at twice
// the rate; an item that has its CU to itself takes .._ALONE per block.  A 4-wavefront item takes WIN_128_WAVE per
// block more for each wavefront that has rows.
constexpr Cost WIN_128 = {3.3, 0.543}, SPLIT2 = {1.6, 0.4125}, SPLIT2_WIN = {3.5, 0.53};
constexpr double WIN_128_WAVE = 0.075, WIN_128_ALONE = 1.19, SPLIT2_ALONE = 0.705;
constexpr Cost SPLIT4 = {4.2, 0.573}, SPLIT4_WIN = {7.5, 0.505};  // split kernel with four: one workgroup per CU
constexpr double LAUNCH_US = 2.5;
// Half-row items read every key row twice: window items, and long items of a launch that the CUs hold at once, are
// halved only where that saves something (144 dense items of 144 blocks: 174 us whole, 189 us with 64 in halves).  Of
// more long items than CUs the last are halved unless that costs something: the order in which CUs become free is not
// quite the one assumed here, and halves even it out (306 long items: 918 us whole, 828 us with 64 in halves).
constexpr double HALVES_SAVE = 1.02, HALVES_EVEN = 0.96;
constexpr int XCDS = 8;                     // workgroups are dealt to them in turn, and each has its own CUs

struct Batch {
  int items;
  double cost;       // of each
};
struct Segment {
  int items, blocks;  // items, 64-key blocks of each
};
struct Window {       // the items of a list, head after head
  int heads = 0, list = 0;                // list: items of a head
  const int64_t* sums = nullptr;          // blocks of the items before each one of the list
  int most = 0;                           // blocks of the longest
  double waves = 0.0;                     // wavefronts with rows of an item, on average
  int items() const { return heads * list; }
  double before(int i) const { return (double)(i / list) * (double)sums[list] + (double)sums[i % list]; }
  // blocks of the items [first, last), on average
  double blocks(int first, int last) const { return last > first ? (before(last) - before(first)) / (last - first) : 0.0; }
  double blocks() const { return (double)sums[list] / list; }
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
      if (left >= units && t[ng - 1] - t[0] <= batch[b].cost) {      // whole rounds: every processor takes one item of each
        const int rounds = left / units;
        for (int i = 0; i < ng; ++i) t[i] += rounds * batch[b].cost;
        left -= rounds * units;
        continue;
      }
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

// Time of a launch from the batches of each of its XCDs: the latest of them.  XCDs with the same batches as the one
// before are not computed again.
class Launch {
 public:
  explicit Launch(int units) : units_(std::max(1, units / XCDS)) {}
  void batch(int items, double cost) {
    if (items > 0) b_[n_++] = {items, cost};
  }
  // items from index `at` of the launch on, dealt round robin: how many XCD x gets
  static int share(int at, int items, int x) { return (at + items - x + XCDS - 1) / XCDS - (at - x + XCDS - 1) / XCDS; }
  void close() {
    if (n_ != last_n_ || !std::equal(b_, b_ + n_, last_, [](const Batch& a, const Batch& b) { return a.items == b.items && a.cost == b.cost; })) {
      if (n_) worst_ = std::max(worst_, makespan(b_, n_, units_));
      last_n_ = n_;
      std::copy(b_, b_ + n_, last_);
    }
    n_ = 0;
  }
  double worst() const { return worst_; }

 private:
  int units_, n_ = 0, last_n_ = -1;
  double worst_ = 0.0;
  Batch b_[8], last_[8];
};

// Items [first, last) of XCD x where n items are dealt in contiguous ranges.
struct Range {
  int first, last;
};
Range xcd_range(int n, int x) {
  const int each = n / XCDS, more = n % XCDS, first = each * x + std::min(x, more);
  return {first, first + each + (x < more)};
}

// Pipelined launch of three segments of long items (the last half_long of them as half-row items), dealt round
// robin, and one of window items (the last half_win), dealt in contiguous ranges, so that the halves are all on the
// last XCDs; 0 without items.
double pipe_time(const Segment* longs, const Window& win, int half_long, int half_win, int units) {
  const int n_long = longs[0].items + longs[1].items + longs[2].items, n_win = win.items();
  if (n_long + n_win == 0) return 0.0;
  Launch launch(units);
  for (int x = 0; x < XCDS; ++x) {
    int at = 0;
    for (int pass = 0; pass < 2; ++pass) {
      int keep = n_long - half_long;
      for (int i = 0; i < 3; ++i) {
        const int w = std::min(keep, longs[i].items), items = pass == 0 ? w : 2 * (longs[i].items - w);
        keep -= w;
        launch.batch(Launch::share(at, items, x), (pass == 0 ? LONG : LONG_HALF).of(longs[i].blocks));
        at += items;
      }
    }
    if (n_win) {
      const int whole = n_win - half_win;
      const Range r = xcd_range(n_win + half_win, (x + XCDS - at % XCDS) % XCDS);
      const int end = std::min(r.last, whole), begin = std::max(r.first, whole);      // whole items to end, halves from begin
      auto item = [&](int half) { return whole + (half - whole) / 2; };
      if (end > r.first) launch.batch(end - r.first, WIN.of(win.blocks(r.first, end)));
      if (r.last > begin) launch.batch(r.last - begin, WIN_HALF.of(win.blocks(item(begin), std::max(item(begin) + 1, item(r.last)))));
    }
    launch.close();
  }
  const double alone = n_win ? (half_win < n_win ? WIN : WIN_HALF).of(win.most) : 0.0;
  return LAUNCH_US + std::max(alone, launch.worst());
}

double win_128_time(const Window& win, int units) {
  if (win.items() == 0) return 0.0;
  Launch launch(units);
  for (int x = 0; x < XCDS; ++x) {
    const Range r = xcd_range(win.items(), x);
    const double blocks = win.blocks(r.first, r.last);
    launch.batch(r.last - r.first, WIN_128.of(blocks) + WIN_128_WAVE * win.waves * blocks);
    launch.close();
  }
  return LAUNCH_US + std::max(WIN_128.fixed + WIN_128_ALONE * win.most, launch.worst());
}

// Split launch of the three segments of long items (or none: null) and the window items, dealt round robin.
double split_time(const Segment* longs, const Window& win, int shares, int units) {
  Launch launch(units);
  int items = win.items();
  double alone = 0.0;                      // the longest item by itself
  for (int i = 0; longs && i < 3; ++i) {
    items += longs[i].items;
    if (longs[i].items) alone = std::max(alone, shares == 2 ? SPLIT2.fixed + SPLIT2_ALONE * longs[i].blocks : SPLIT4.of(longs[i].blocks));
  }
  if (win.items()) alone = std::max(alone, shares == 2 ? SPLIT2_WIN.fixed + SPLIT2_ALONE * win.most : SPLIT4_WIN.of(win.most));
  if (items == 0) return 0.0;
  if (items <= units) return LAUNCH_US + alone;      // every item has a CU to itself
  for (int x = 0; x < XCDS; ++x) {
    int at = 0;
    auto add = [&](int items_here, double cost) {
      launch.batch(Launch::share(at, items_here, x), cost);
      at += items_here;
    };
    for (int i = 0; longs && i < 3; ++i) add(longs[i].items, (shares == 2 ? SPLIT2 : SPLIT4).of(longs[i].blocks));
    if (win.items()) add(win.items(), (shares == 2 ? SPLIT2_WIN : SPLIT4_WIN).of(win.blocks()));
    launch.close();
  }
  return LAUNCH_US + std::max(alone, launch.worst());
}

// The number of items to issue as half-row items, and its estimate: the last items of a launch leave most CUs
// idle while a few finish them, and two half-row items take 1.3 times one whole item.
template <class Time>
int best_halves(int items, int units, double margin, Time time_of, double* best_us) {
  int best = 0;
  double best_cost = *best_us = time_of(0);
  for (int h : {units / 4, units / 2, items}) {
    h = std::min(h, items);
    const double us = time_of(h);
    if (us * margin < best_cost) {
      best_cost = us * margin;
      *best_us = us;
      best = h;
    }
  }
  return best;
}
}  // namespace

// Items of the long segments of a launch in its order: text rows of the window heads, dense heads, core-set heads.  Returns their number.
static int long_segments(const vorta_plan* p, const RouteLists& rl, bool win_text, int bm, Segment (&s)[3]) {
  const int rows_c = (int)(p->Lc + p->d.n_text), blocks_n = (int)((p->N + 63) / 64);
  auto items_of = [bm](int64_t rows) { return (int)((rows + bm - 1) / bm); };
  s[0] = {win_text ? rl.count[1] * items_of(p->d.n_text) : 0, blocks_n};
  s[1] = {rl.count[0] * items_of(p->N), blocks_n};
  s[2] = {rl.count[2] * items_of(rows_c), (rows_c + 63) / 64};
  return s[0].items + s[1].items + s[2].items;
}

// A split launch of two key shares whose CUs take one or two workgroups each: which of the first `units` items the first
// workgroup takes (the others follow in turn), see launch_split.  The time of a CU is that of the longer of its two items and a
// sixth of the shorter one's, by the costs above (an item alone 0.705 us per block, two together 0.4125 each), and the launch ends
// with the last CU.  Segments are not in the order of their lengths, nor are the window items under the identity rule, so
// neither order is the better one everywhere.  Measured on 39 layers, turned against not turned: 0.92 to 1.12 times as fast;
// where this estimate turns (20 layers) 0.99 to 1.12, where it does not 0.92 to 1.01.  Worst of those that turning slows: two
// window heads whose later items have the longer key lists 25.3 -> 27.6 us, 13 core-set heads in front of 3 window heads
// of longer items 33.8 -> 35.8.
int split_round_shift(const vorta_plan* p, const RouteLists& rl, bool longs, bool win_text, int units) {
  constexpr int MOST = 512;                  // CUs
  int blocks[2 * MOST];
  if (units > MOST) return 0;
  Segment s[3] = {};
  const int n_long = longs ? long_segments(p, rl, win_text, ATTN_ROWS_SPLIT, s) : 0;
  const int list = (int)(p->win_list[2].size() / WIN_ITEM_INTS);
  const int64_t n = n_long + (int64_t)rl.count[1] * list;
  if (n <= units || n >= 2 * units) return 0;
  int* to = blocks;
  for (const Segment& seg : s) to = std::fill_n(to, seg.items, seg.blocks);
  if (rl.count[1] && list) {
    const int64_t* sums = p->win_sums[2].data();
    for (int i = 0; i < list; ++i) to[i] = (int)(sums[i + 1] - sums[i]);
    for (int h = 1; h < rl.count[1]; ++h) std::copy_n(to, list, to + h * list);
  }
  const int second = (int)n - units, shift = units - second;      // CUs with two items, with one
  int longest = 0, turned = 0, as_is = 0;    // six times the blocks
  for (int j = 0; j < second; ++j) {
    const int a = blocks[j], b = blocks[shift + j], c = blocks[units + j];
    as_is = std::max(as_is, 6 * std::max(a, c) + std::min(a, c));
    turned = std::max(turned, 6 * std::max(b, c) + std::min(b, c));
  }
  for (int j = second; j < units; ++j) longest = std::max(longest, blocks[j]);
  as_is = std::max(as_is, 6 * longest);
  longest = 0;
  for (int j = 0; j < shift; ++j) longest = std::max(longest, blocks[j]);
  return std::max(turned, 6 * longest) < as_is ? shift : 0;      // the first items come to the CUs that have one
}

// mix: the launch is the full-attention branch of Eq. 5.  win_text = false: the text rows of the window heads are
// left out.  units: CUs of the device.
AttnForm choose_attention_form(const vorta_plan* p, const RouteLists& rl, bool mix, bool win_text, int units) {
  const int n_win = rl.count[1];
  auto longs_of = [&](int bm, Segment (&s)[3]) { return long_segments(p, rl, win_text, bm, s); };
  auto list = [&](int l) {
    Window w;
    w.heads = n_win;
    w.list = (int)(p->win_list[l].size() / WIN_ITEM_INTS);
    w.sums = p->win_sums[l].data();
    w.most = p->win_most_blocks[l];
    w.waves = p->win_waves[l];
    return w;
  };
  Segment fine[3], coarse[3];
  const Segment no_longs[3] = {};
  const Window none, big = list(0), rest = list(1), fine_win = list(2), win_128 = list(3);
  const int fine_items = longs_of(ATTN_ROWS_SPLIT, fine) + fine_win.items();
  AttnForm f = {};
  f.empty = fine_items == 0;
  if (f.empty) return f;
  f.n_long = longs_of(ATTN_ROWS_LONG, coarse);
  f.n_big = big.items();
  f.together = f.n_long && f.n_big && !mix;
  f.split_all = fine_items <= units;       // 256-row items would leave three of four CUs idle
  const double t_split2 = split_time(fine, fine_win, 2, units), t_split4 = split_time(fine, fine_win, 4, units);
  f.shares = t_split4 < t_split2 ? 4 : 2;
  if (!f.split_all || p->force_form) {
    double t_long, t_pipe;
    f.half_long = best_halves(f.n_long, units, f.n_long > units ? HALVES_EVEN : HALVES_SAVE, [&](int h) { return pipe_time(coarse, none, h, 0, units); }, &t_long);
    f.half_big = best_halves(f.n_big, units, HALVES_SAVE, [&](int h) { return pipe_time(f.together ? coarse : no_longs, big, 0, h, units); }, &t_pipe);
    if (!f.together) t_pipe += t_long;
    t_pipe += win_128_time(rest, units);
    // Far above the sizes where another form can win by much there is nothing to choose, and the chip's power limit
    // changes the costs: core-set and window items of 12 heads of 32,760 tokens, 3,900 blocks per CU, are estimated
    // faster with the window rows in 128-row items and measured 0 to 1.8 % slower (the whole mixture).
    double work = fine_win.items() ? fine_win.items() * fine_win.blocks() : 0.0;
    for (const Segment& s : fine) work += (double)s.items * s.blocks;
    if (!f.split_all && work < 3000.0 * units) {
      double best = t_pipe;
      auto take = [&](bool& form, double us) {
        if (us >= best) return;
        best = us;
        f.split_win = f.win_128 = f.split_all = false;
        form = true;
      };
      if (n_win) {
        take(f.split_win, t_long + split_time(nullptr, fine_win, 2, units));
        take(f.win_128, t_long + win_128_time(win_128, units));
      }
      take(f.split_all, std::min(t_split2, t_split4));
    }
  }
  if (p->force_form) {           // tests: one form for every size
    f.split_all = p->force_form == 2 || p->force_form == 4;
    if (f.split_all) f.shares = p->force_form;
    f.split_win = p->force_form == 5 && n_win;
    f.win_128 = p->force_form == 6 && n_win;
    if (p->force_halves >= 0) {
      f.half_long = std::min(p->force_halves, f.n_long);
      f.half_big = std::min(p->force_halves, f.n_big);
    }
  }
  f.together = f.together && !f.split_all && !f.split_win && !f.win_128;
  return f;
}

}  // namespace vorta

using namespace vorta;

extern "C" {

// For the tests, not part of the ABI: every form of the bf16 attention launch at any size.  form: 0 = by the rule;
// 2, 4 = split kernel with so many key shares; 3 = pipelined kernels; 5 = pipelined, window rows on the split
// kernel; 6 = pipelined, all window rows in 128-row items.  halves: items issued as half-row items, -1 = by the rule.  A property of the plan; not to be changed
// while a call on it runs.
int vorta_test_force_form(vorta_plan* p, int32_t form, int32_t halves) {
  if (!p || !(form == 0 || (form >= 2 && form <= 6)) || halves < -1) return fail(VORTA_EINVAL, "form %d, halves %d", form, halves);
  p->force_form = form;
  p->force_halves = halves;
  return VORTA_OK;
}

// What a layer call (mix = 0) or the full-attention launch of the mixture (1) chooses with `units` CUs:
// {split_all, shares, split_win, together, n_long, half_long, n_big, half_big, win_128}.
int vorta_test_form(const vorta_plan* p, const uint8_t* routes_host, int32_t mix, int32_t units, int32_t out[9]) {
  RouteLists rl;
  if (int rc = split_routes(p, routes_host, &rl)) return rc;
  const AttnForm f = choose_attention_form(p, rl, mix != 0, true, units);
  const int32_t v[9] = {f.split_all, f.shares, f.split_win, f.together, f.n_long, f.half_long, f.n_big, f.half_big, f.win_128};
  std::copy(v, v + 9, out);
  return VORTA_OK;
}

// The first item of a split launch of two key shares (see split_round_shift): of a layer call, or with window_only of the window rows alone.
int vorta_test_round_shift(const vorta_plan* p, const uint8_t* routes_host, int32_t window_only, int32_t units, int32_t* out) {
  RouteLists rl;
  if (int rc = split_routes(p, routes_host, &rl)) return rc;
  *out = split_round_shift(p, rl, !window_only, true, units);
  return VORTA_OK;
}

// The window items of list 0 .. 3 (see vorta_plan::win_list): their number, and unless out is null for each the first place, the
// number of rows and the numbers of its keys, 16 in all.
int vorta_test_window_list(const vorta_plan* p, int32_t list, int32_t* out, int32_t* n_items) {
  if (!p || list < 0 || list > 3 || !n_items) return fail(VORTA_EINVAL, "list %d", list);
  const std::vector<int32_t>& items = p->win_list[list];
  *n_items = (int32_t)(items.size() / WIN_ITEM_INTS);
  for (size_t i = 0; out && i < items.size(); i += WIN_ITEM_INTS, out += 16) {
    std::fill_n(std::copy_n(&items[i], 2, out), 14, 0);
    std::copy_n(&p->win_keys[(size_t)items[i + 2] * WIN_KEY_INTS], WIN_KEY_INTS, out + 2);
  }
  return VORTA_OK;
}

// Bytes of the window items and their keys.
int vorta_test_window_bytes(const vorta_plan* p, int64_t* out) {
  size_t n = p->win_keys.size();
  for (const auto& list : p->win_list) n += list.size();
  *out = (int64_t)(n * sizeof(int32_t));
  return VORTA_OK;
}

}  // extern "C"
