// Host-side planner: descriptor validation and the tile schedule.  Pure C++, no HIP calls.
//
// The mask of a query row depends only on its document position p (it sees keys 0..p of its own
// document; Appendix B's shard geometry), not on which CA-task carried it.  So the planner forgets task
// boundaries: per document it lists every query row present in the batch sorted by position and cuts
// that list into tiles.  Rows of different tasks of one document share tiles, which is the paper's
// composability observation (Section 3.2: throughput depends on the aggregate tokens of a fused call,
// not on their document of origin) carried below its 128-token shard granularity.
#include <algorithm>
#include <array>
#include <cmath>
#include <cstring>
#include <functional>
#include <memory>
#include <numeric>
#include <sstream>

#include "ca_internal.h"

namespace ca {

static thread_local std::string g_err;
void set_error(const std::string &msg) { g_err = msg; }
const char *last_error() { return g_err.c_str(); }

namespace {
struct Fail {
  int code;
  std::string msg;
};
#define CA_REQUIRE(cond, code, text)        \
  do {                                      \
    if (!(cond)) {                          \
      std::ostringstream os_;               \
      os_ << text;                          \
      throw Fail{code, os_.str()};          \
    }                                       \
  } while (0)

void validate(const ca_batch_desc *d) {
  CA_REQUIRE(d != nullptr, CA_ERR_INVALID_ARG, "descriptor is null");
  CA_REQUIRE(d->n_docs >= 0 && d->n_tasks >= 0, CA_ERR_INVALID_ARG, "negative n_docs or n_tasks");
  CA_REQUIRE(d->n_q_heads >= 1 && d->n_kv_heads >= 1, CA_ERR_INVALID_ARG, "head counts must be >= 1");
  CA_REQUIRE(d->n_q_heads % d->n_kv_heads == 0, CA_ERR_UNSUPPORTED,
             "n_q_heads " << d->n_q_heads << " is not a multiple of n_kv_heads " << d->n_kv_heads);
  CA_REQUIRE(d->head_dim == 64 || d->head_dim == 128, CA_ERR_UNSUPPORTED,
             "head_dim " << d->head_dim << " not supported (64 or 128)");
  CA_REQUIRE(d->total_q >= 0 && d->total_kv >= 0, CA_ERR_INVALID_ARG, "negative total_q or total_kv");
  const int64_t lim = (int64_t(1) << 31) - 4 * SLOT_ALIGN;
  CA_REQUIRE(d->total_q < lim && d->total_kv < lim, CA_ERR_UNSUPPORTED, "total_q / total_kv beyond 2^31 rows");
  CA_REQUIRE(d->total_kv * d->n_kv_heads * d->head_dim < (int64_t(1) << 40), CA_ERR_UNSUPPORTED, "KV buffer too large");
  if (d->n_docs > 0)
    CA_REQUIRE(d->doc_kv_start && d->doc_kv_len, CA_ERR_INVALID_ARG, "document arrays are null");
  if (d->n_tasks > 0) {
    CA_REQUIRE(d->task_doc && d->task_q_start && d->task_q_len && d->task_q_pos && d->task_kv_len,
               CA_ERR_INVALID_ARG, "task arrays are null");
    CA_REQUIRE(d->n_docs > 0, CA_ERR_INVALID_ARG, "tasks given but no documents");
  }
  // documents: in bounds, pairwise disjoint KV ranges
  std::vector<int32_t> order(d->n_docs);
  std::iota(order.begin(), order.end(), 0);
  for (int i = 0; i < d->n_docs; ++i) {
    CA_REQUIRE(d->doc_kv_len[i] >= 1, CA_ERR_INVALID_ARG, "document " << i << " has kv_len " << d->doc_kv_len[i]);
    CA_REQUIRE(d->doc_kv_start[i] >= 0 && d->doc_kv_start[i] <= d->total_kv - d->doc_kv_len[i], CA_ERR_INVALID_ARG,
               "document " << i << " KV range [" << d->doc_kv_start[i] << ", +" << d->doc_kv_len[i]
                           << ") outside the packed KV buffer of " << d->total_kv << " rows");
  }
  std::sort(order.begin(), order.end(), [&](int a, int b) { return d->doc_kv_start[a] < d->doc_kv_start[b]; });
  for (int i = 1; i < d->n_docs; ++i) {
    int a = order[i - 1], b = order[i];
    CA_REQUIRE(d->doc_kv_start[a] + d->doc_kv_len[a] <= d->doc_kv_start[b], CA_ERR_INVALID_ARG,
               "KV ranges of documents " << a << " and " << b << " overlap");
  }
  // tasks: in bounds, causal geometry, pairwise disjoint Q ranges
  std::vector<int32_t> torder(d->n_tasks);
  std::iota(torder.begin(), torder.end(), 0);
  for (int t = 0; t < d->n_tasks; ++t) {
    CA_REQUIRE(d->task_doc[t] >= 0 && d->task_doc[t] < d->n_docs, CA_ERR_INVALID_ARG,
               "task " << t << " names document " << d->task_doc[t]);
    CA_REQUIRE(d->task_q_len[t] >= 1, CA_ERR_INVALID_ARG, "task " << t << " has q_len " << d->task_q_len[t]);
    CA_REQUIRE(d->task_q_start[t] >= 0 && d->task_q_start[t] <= d->total_q - d->task_q_len[t], CA_ERR_INVALID_ARG,
               "task " << t << " query range outside packed Q of " << d->total_q << " rows");
    CA_REQUIRE(d->task_q_pos[t] >= 0, CA_ERR_INVALID_ARG, "task " << t << " has negative q_pos");
    CA_REQUIRE(d->task_kv_len[t] >= 1, CA_ERR_INVALID_ARG,
               "task " << t << " has kv_len " << d->task_kv_len[t] << " (every row must see at least one key)");
    CA_REQUIRE(d->task_kv_len[t] <= d->doc_kv_len[d->task_doc[t]], CA_ERR_INVALID_ARG,
               "task " << t << ": kv_len " << d->task_kv_len[t] << " exceeds its document's resident KV "
                       << d->doc_kv_len[d->task_doc[t]]);
  }
  std::sort(torder.begin(), torder.end(), [&](int a, int b) { return d->task_q_start[a] < d->task_q_start[b]; });
  for (int i = 1; i < d->n_tasks; ++i) {
    int a = torder[i - 1], b = torder[i];
    CA_REQUIRE(d->task_q_start[a] + d->task_q_len[a] <= d->task_q_start[b], CA_ERR_INVALID_ARG,
               "query ranges of tasks " << a << " and " << b << " overlap");
  }
}

inline int64_t round_up(int64_t x, int64_t m) { return (x + m - 1) / m * m; }

// ---- cutting long units into pieces where a batch leaves the chip idle
// A kernel's unit costs `fixed` plus `per_step` for each of its steps (tiles, or query blocks x heads), and the hardware
// hands the units, sorted longest first, to whichever CU is free: the launch time is a list-scheduling makespan, which is
// simulated here (32 CUs stand for 256 where every unit comes once for each of 8 heads).  Cutting every unit longer than T
// steps into equal pieces evens the load out and costs a `fixed` per piece, the partial results (written by the pieces,
// read once more to be added up) and another launch.  The T with the shortest total is taken, if it gains a tenth: at
// 4K tokens of 1K-token documents (32/8 heads) the simulation gives 340 us for the dK/dV kernel's 256 whole units (measured
// 353) and 201 us for 472 units and pieces of at most 66 steps and their sums (measured 164 and 10): good enough to rank cuts by, not
// to predict what one gains.
// The figures are microseconds measured on MI355X.  Two or three workgroups share a CU and its throughput: a step takes a forward
// or dK/dV workgroup about as long alone on a CU as the CU takes per step of several, so a CU counts as one server at that pace
// (head_dim 128, per step alone / of two: forward 1.8 / 1.8, dK/dV 1.75 / 1.6; at 64 of three: 1.0 and 0.85).  (The dK/dV kernel at
// 64 counts as two servers per CU, each at half that pace: 1.75 per step.)  The fixed part is what a unit spends around its steps
// (descriptor, row indices, fragments, first tiles, drain, results) and another workgroup does not hide; partial results move at
// about 4 TB/s.
// Batches with more dK/dV work than this per CU run two launches.  Backward in two launches against one, documents of 1K to 4K on
// average (dK/dV work per CU), head_dim 128: 215 -> 165 us (4K tokens, 32/8 heads; 0.08 ms), 637 -> 503 (8K; 0.27), 1345 -> 1204 (16K;
// 0.65), 2281 -> 2235 (32K; 1.15), 4322 -> 4250 (64K, 16/16; 2.4).  Lone shards, whose half units read K and V twice as often, lose:
// 710 -> 719 us (1000 rows with a 32K context, 16/4; 0.45), 5.33 -> 5.40 ms (64-row shards with contexts; 2.8), 7.72 -> 8.0 ms (1000
// rows with 130K; 3.2).  The line lies where the one's gain is down to the other's loss.  Head_dim 64: 83 -> 60 us (4K, 16/16; 0.03
// ms), 412 -> 399 (16K; 0.21), 1350 -> 1335 (32K, 32/8; 0.62), 1236 -> 1205 (64K, 8/2; 0.58), 2504 -> 2605 (64K, 16/16; 1.3).
constexpr double JOINT_MAX_US = 1500, JOINT_MAX_US_64 = 1000;
// The choice between one backward launch and two simulates lists of thousands of units, at 20 to 40 ns each more than the rest
// of planning takes: ca_plan_host for 37K tokens in lone 860-row shards (8/1 heads) 65 us without it, 192 with all units
// simulated, 106 so; of 1600 batches none gets another launch, two of 600 another order in it (backward 0.7 % slower, 0.3 %
// faster).  (Cut lengths are searched with all units: simulated so, one of 1600 batches got a cut that cost 2 %.)
constexpr int64_t JOINT_UNITS = 512;
constexpr double BEYOND_STATIC_US = 25;  // what a pass has to gain for partial results beyond the static workspace, if not a tenth
constexpr double BYTES_PER_US = 4e6;  // partial results, written and read
struct CutCost {
  int slots;  // workgroups that run at a time
  double per_step, fixed, launch;
  int min_steps;
};

// The least of a heap (the least on top) becomes t, which is no less, and sinks.
inline void replace_top(std::vector<double> &heap, double t) {
  const size_t n = heap.size();
  size_t at = 0;
  for (size_t c = 1; c < n; c = 2 * at + 1) {
    if (c + 1 < n && heap[c + 1] < heap[c]) ++c;
    if (heap[c] >= t) break;
    heap[at] = heap[c];
    at = c;
  }
  heap[at] = t;
}

// When the last of `units` ((microseconds, how many), handed out in this order) ends on n_cu CUs, or a time of at least
// at_most.  A list of more than max_units is simulated with 2, 4, .. neighbours of it as one unit (of their mean length) on as
// many times fewer CUs: neighbours are of nearly equal length.
double makespan(const std::vector<std::pair<double, int64_t>> &units, int64_t n_cu, double at_most, int64_t max_units = INT64_MAX) {
  int64_t total = 0, q = 1;
  double end = 0;
  for (const auto &[us, n] : units) total += n, end = std::max(end, us);
  while (total / q > max_units && n_cu % (2 * q) == 0 && n_cu > 16 * q) q *= 2;
  std::vector<double> busy;  // once every CU has a unit: a heap, the least loaded CU on top
  const size_t n_busy = size_t(n_cu / q);
  busy.reserve(n_busy);
  int64_t held = 0;  // units that do not make up a group yet, and the sum of their lengths
  double held_us = 0;
  for (const auto &[unit_us, count] : units) {
    const int64_t n = (held + count) / q;  // groups that are complete now; the first takes in the units held
    double us = held > 0 ? (held_us + double(q - held) * unit_us) / double(q) : unit_us;
    int64_t i = 0;
    for (; i < n && busy.size() < n_busy; ++i, us = unit_us) {  // the first units find idle CUs
      busy.push_back(us);
      if (busy.size() == n_busy) std::make_heap(busy.begin(), busy.end(), std::greater<double>());
    }
    if (end >= at_most) return end;
    for (; i < n; ++i, us = unit_us) {
      const double t = busy[0] + us;
      if (t > end) {
        end = t;
        if (end >= at_most) return end;
      }
      replace_top(busy, t);
    }
    held = held + count - n * q;
    held_us = n > 0 ? double(held) * unit_us : held_us + double(count) * unit_us;
  }
  if (held > 0) end = std::max(end, (busy.size() < n_busy ? 0.0 : busy[0]) + held_us / double(held));
  return end;
}

// Forward workgroups: whole units, or their halves of 128 rows.  Halves are a finer schedule, and two of them run a unit that is
// alone on its CU in 60 % of the time; where both fill the chip a tile costs two halves 7 % more (K and V fragments feed half
// the MFMAs).  Measured, units against halves, head_dim 128: 45 -> 24 us (32 units of 16 tiles), 196 -> 182 (384 of 64), 135 -> 110
// (4K tokens of documents of about 1K: 512 units of 1 to 50 tiles), 229 -> 250 (512 of 64), 480 -> 534 (512 of 128).
// Workgroups of equal length of which a CU gets two share it evenly only if they take turns at having priority (see the kernel).
// Without and with that: 1705 -> 1630 us (512 pieces of 508 tiles), 1900 -> 1858 (halves of 256 pieces of 1016), 74.1 -> 72.2 (halves of
// 256 pieces of 32).  In a list of unequal ones the longest are the oldest, and better off served first; with more than two per CU
// there is no tail to even out (halves of 384 pieces of 22 tiles: 79 -> 89 us).  A turn is two to three tiles: workgroups of less than a
// few turns only pay for the clock.
constexpr double MIN_TURN_TILES = 12;
struct FwdUnits {
  double tiles, tiles_half;  // of a unit, and of its first half
  int64_t n;
};
struct FwdRun {
  FwdForm form;
  double us;
};
// The better form of a list, longest first, and its time.  Microseconds, start + per tile, fitted to the figures above.
FwdRun fwd_run(const std::vector<FwdUnits> &list, int d) {
  if (list.empty()) return {{}, 0.0};
  int64_t units = 0;
  for (const FwdUnits &u : list) units += u.n;
  const bool d128 = d == 128, lone = units <= N_CU, equal = list.back().tiles >= 0.9 * list.front().tiles;
  auto turns = [&](int64_t workgroups) { return d128 && equal && workgroups > N_CU && workgroups <= 2 * N_CU && list.back().tiles >= MIN_TURN_TILES; };
  const bool whole_turns = turns(units), half_turns = turns(2 * units);
  const double fixed = d128 ? 8.0 : 5.0, per = whole_turns ? 1.5 : d128 ? (lone ? 2.05 : 1.78) : lone ? 1.15 : 1.0;
  const double fixed_half = d128 ? 4.0 : 2.5, per_half = half_turns ? 0.87 : d128 ? 0.96 : 0.53;
  std::vector<std::pair<double, int64_t>> whole, half;
  for (const FwdUnits &u : list) whole.push_back({fixed + per * u.tiles, u.n});
  const FwdRun run{{false, whole_turns}, makespan(whole, N_CU, 1e30, JOINT_UNITS)};
  if (units > 4 * N_CU) return run;
  for (const FwdUnits &u : list) {
    half.push_back({fixed_half + per_half * u.tiles, u.n});
    half.push_back({fixed_half + per_half * u.tiles_half, u.n});
  }
  const double us = makespan(half, N_CU, run.us, JOINT_UNITS);
  return us < run.us ? FwdRun{{true, half_turns}, us} : run;
}

// The longest piece in steps (0: cut nothing) and the launch time that gives, under each of two limits of the partial results.
struct Cut {
  int64_t piece = 0;
  double us = 0;
};
// units: (steps, how many of that size), longest first.
std::array<Cut, 2> best_piece(const std::vector<std::pair<int64_t, int64_t>> &units, const CutCost &c, size_t bytes_per_part,
                              const std::array<size_t, 2> &max_bytes) {
  double total = 0, steps_per_cu = 0;
  int64_t longest = 0, same = c.slots;  // `same`: every size comes a multiple of this many times
  for (const auto &[steps, count] : units) {
    total += double(count) * (c.fixed + c.per_step * double(steps));
    steps_per_cu += double(count) * double(steps) / c.slots;
    longest = std::max(longest, steps);
    same = std::gcd(same, count);
  }
  std::array<Cut, 2> cut;
  // no list of pieces can beat the mean load: most batches end here
  if (c.fixed + c.per_step * double(longest) < 1.2 * total / c.slots) return cut;
  std::vector<std::pair<double, int64_t>> sizes;  // (microseconds, how many / same)
  struct Search {
    double best = 0;
    int worse = 0;
    bool done = false;
  } search[2];
  // whole units first, then pieces from a little over the mean load downwards
  for (double T = double(longest); T >= c.min_steps; T = std::min(T / 1.2, std::max(1.3 * steps_per_cu, 4.0 * c.min_steps))) {
    const int64_t t = int64_t(T);
    int64_t parts = 0;
    size_t n_cut = 0;  // the leading units are the long ones
    double sum = 0, piece = 0;
    sizes.clear();
    for (const auto &[steps, count] : units) {
      const int64_t k = std::max<int64_t>(1, (steps + t - 1) / t);  // (units without steps, which write zeros, stay whole)
      const double us = c.fixed + c.per_step * double(steps) / double(k);
      sizes.push_back({us, count / same * k});
      sum += us * double(count * k);
      if (k > 1) parts += count * k, ++n_cut;
      piece = std::max(piece, us);
    }
    const size_t bytes = size_t(parts) * bytes_per_part;
    const double extra = parts ? c.launch + double(bytes) / BYTES_PER_US : 0.0;
    for (int i = 0; i < 2; ++i)  // more and smaller pieces only cost more
      if (parts && (bytes > max_bytes[size_t(i)] || sum / c.slots + extra >= search[i].best)) search[i].done = true;
    if (search[0].done && search[1].done) break;
    auto longer = [](const auto &x, const auto &y) { return x.first > y.first; };
    std::sort(sizes.begin(), sizes.begin() + n_cut, longer);
    std::inplace_merge(sizes.begin(), sizes.begin() + n_cut, sizes.end(), longer);
    double at_most = 0;
    for (const Search &x : search)
      if (!x.done) at_most = std::max(at_most, x.best - extra);
    if (!parts) at_most = 1e30;
    const double us = piece >= at_most ? piece + extra : makespan(sizes, c.slots / same, at_most) + extra;
    for (int i = 0; i < 2; ++i) {
      Search &x = search[i];
      if (x.done) continue;
      if (!parts) x.best = 0.9 * us, cut[size_t(i)].us = us;
      else if (us < x.best) x.best = us, cut[size_t(i)] = {t, us}, x.worse = 0;
      else if (++x.worse == 3) x.done = true;
    }
  }
  return cut;
}

// ---- the backward in one pass (ca_bwd_fused.hip)
// The KV tiles of one (document, KV head) are a chain: tile j + 1 adds to a 32-row tile of dQ after tile j, in the L2 of the XCD that
// runs the chain, so a chain belongs to one of 8 queues, one per XCD, whose workgroups take its units in order.  Chains go, longest
// first, to the queue with the least work.  In a queue they follow each other by length in groups that can keep the XCD's workgroups
// busy twice over (a chain of tiles under few query rows cannot: each tile only starts when the one before it is a step or two
// ahead), and inside a group the longest unit comes first.  All units of a queue by their length, whatever their documents, end a
// little more evenly and are slower, as fewer of the sums of dQ are still in L2: 8.46 against 8.18 ms (64K tokens of documents
// of about 2K, 32/8 heads), 31.5 against 30.9 ms (64K tokens of long documents, 64/8), 4.99 against 4.47 ms (lone 64-row shards, 8/2).
//
// At head_dim 64, with three workgroups per CU, groups are half as long again.  Of 63 drawn batches there shards ran 1.5 % slower so than in
// groups as at 128, but documents 0.8 % faster (geometric means), and short lists, whose last group leaves workgroups idle,
// up to 19 % (532 -> 447 us); groups half as long again as that lose another 1.2 %.  128 would lose (64K tokens of documents
// of about 2K 7.25 -> 7.45 ms).
//
// When does the one pass pay?  It does five contractions instead of seven, but in workgroups of twice the keys (head_dim 128), one to a
// CU, bound to queues.  A unit costs `fixed`, `per_step` for each 32 rows x head and `per_masked` where they hold the diagonal, and
// starts at least `lag` after the one before it in its chain; the longest queue is simulated and compared with the simulation of the
// other kernels.  Theirs knows only steps, so it is given the time by which moving K and V (read twice), dK and dV prolongs them: 0.4
// of those bytes at the rate of partial results, from batches of short shards under long contexts (with it 12 measured at 1.03
// to 1.2 of the simulation, without it at 1.15 to 1.7).  Microseconds, fitted to drawn batches.  Of 1018 measured in both ways the rule
// takes 266: the lists were 1.13 (head_dim 128) and 1.20 times (64) slower on average (backward, geometric mean), and faster by
// more than 2 % on 3 (3.5 % on one).  Of the others 103 would have gained more than 2 %, mostly at 64 and below a millisecond.
struct FusedCost {
  int slots;  // workgroups per XCD
  double per_step, per_masked, fixed, lag;
  double groups;             // times over that a group of chains keeps the workgroups busy
  double gain, more, least;  // the lists have to take `more` microseconds more than `gain` times the one pass; the least work worth a look
};
constexpr FusedCost FUSED_128 = {N_CU / N_XCD, 2.42, 3.45, 12.0, 4.0, 2.0, 1.03, 120, 150},
                    FUSED_64 = {3 * N_CU / N_XCD, 2.05, 5.5, 11.0, 4.0, 3.0, 1.095, 0, 150};

class OnePass {
 public:
  // tiles: KV tiles, document by document, each document's from its first key on
  OnePass(const ca_plan_t &plan, std::vector<BwdUnit> kv_tiles) : cost_(plan.d == 128 ? FUSED_128 : FUSED_64), tiles_(std::move(kv_tiles)), hkv_(plan.hkv) {
    key_.reserve(tiles_.size());
    for (size_t t = 0; t < tiles_.size(); ++t) {
      const int64_t n = steps(tiles_[t]);
      key_.push_back(uint64_t(UINT32_MAX - n) << 32 | uint32_t(tiles_[t].key_pos0));
      if (tiles_[t].key_pos0 == 0) docs_.push_back({t, 0, 0});
      ++docs_.back().n, docs_.back().steps += n;
    }
    std::stable_sort(docs_.begin(), docs_.end(), [](const Doc &a, const Doc &b) { return a.steps > b.steps; });
    std::array<int64_t, N_XCD> load{};
    for (size_t d = 0; d < docs_.size(); ++d)
      for (int h = 0; h < hkv_; ++h) {
        const size_t q = size_t(std::min_element(load.begin(), load.end()) - load.begin());
        load[q] += docs_[d].steps + int64_t(docs_[d].n);
        chains_[q].push_back({d, h});
      }
    longest_ = size_t(std::max_element(load.begin(), load.end()) - load.begin());
  }
  // when the longest queue ends, or at_most where that would be later
  double time(double at_most) const {
    double all = 0;  // no order ends before the mean load
    for (const Chain &c : chains_[longest_])
      for (size_t t = docs_[c.doc].first, end = t + docs_[c.doc].n; t < end; ++t) all += us(tiles_[t]);
    if (all / cost_.slots >= at_most) return at_most;
    double end = 0;
    std::vector<double> begun(chains_[longest_].size(), -cost_.lag);  // the last unit of each chain
    std::vector<double> slots(size_t(cost_.slots), 0.0);
    each_unit(longest_, [&](const Entry &e) {
      const double at = std::max(slots[0], begun[e.chain] + cost_.lag), t = at + us(tiles_[e.tile]);
      replace_top(slots, t);
      begun[e.chain] = at, end = std::max(end, t);
    });
    return std::min(end, at_most);
  }
  void lay_out(ca_plan_t *p) const {
    p->fused_units.reserve(tiles_.size() * size_t(hkv_));
    for (size_t q = 0; q < N_XCD; ++q) {
      each_unit(q, [&](const Entry &e) {
        BwdUnit u = tiles_[e.tile];
        u.kv_head = chains_[q][e.chain].head, u.count = 1;
        p->fused_units.push_back(u);
      });
      p->fused_queue[q + 1] = int32_t(p->fused_units.size());
    }
    const size_t tiles32 = p->slot_row.size() / FUSED_BQ * size_t(p->hq);  // 32-row tiles of dQ
    auto up = [](size_t x) { return (x + 255) / 256 * 256; };
    p->ws_off_dq_sums = p->ws_bwd;
    p->ws_off_flags = p->ws_off_dq_sums + up(tiles32 * FUSED_BQ * size_t(p->d) * 4);
    p->ws_off_ctrl = p->ws_off_flags + up(tiles32 * size_t(fused_waves(p->d)) * 4);
    p->ws_bwd_fused = p->ws_off_ctrl + N_XCD * FUSED_CTRL_BYTES;
    p->fused = true;
  }

 private:
  struct Doc {
    size_t first, n;  // its tiles
    int64_t steps;
  };
  struct Chain {
    size_t doc;
    int32_t head;
  };
  struct Entry {
    uint64_t key;
    uint32_t tile, chain;
  };
  static int64_t steps(const BwdUnit &u) { return int64_t(u.slot_end - u.slot_begin) / FUSED_BQ * u.heads; }
  double us(const BwdUnit &u) const {
    const double masked = double((u.slot_full - u.slot_begin) / FUSED_BQ * u.heads);
    return cost_.fixed + cost_.per_step * double(steps(u)) + (cost_.per_masked - cost_.per_step) * masked;
  }
  // Inside a group by key_: the longer unit first, of equal ones the one of the earlier keys, then the earlier chain's.  A chain's tiles
  // are in that order already, so its chains are merged.  (Sorting made up most of what laying out tens of thousands of units takes.)
  template <class F>
  void each_unit(size_t q, F f) const {
    std::vector<Entry> group, merged;
    std::vector<size_t> runs{0}, fewer;  // where a sorted run begins, and the end
    double busy = 0;                     // workgroups that the group's chains can keep busy
    for (size_t c = 0; c < chains_[q].size(); ++c) {
      const Doc &d = docs_[chains_[q][c].doc];
      for (size_t t = d.first; t < d.first + d.n; ++t) group.push_back({key_[t], uint32_t(t), uint32_t(c)});
      runs.push_back(group.size());
      busy += std::min(double(d.n), 1.0 + cost_.per_step * double(steps(tiles_[d.first])) / cost_.lag);
      if (busy < cost_.groups * cost_.slots && c + 1 < chains_[q].size()) continue;
      while (runs.size() > 2) {
        merged.resize(group.size());
        fewer.assign(1, 0);
        for (size_t r = 0; r + 1 < runs.size(); r += 2) {
          const auto at = [&](size_t i) { return group.begin() + std::ptrdiff_t(runs[std::min(i, runs.size() - 1)]); };
          std::merge(at(r), at(r + 1), at(r + 1), at(r + 2), merged.begin() + std::ptrdiff_t(runs[r]), [](const Entry &a, const Entry &b) { return a.key < b.key; });
          fewer.push_back(runs[std::min(r + 2, runs.size() - 1)]);
        }
        group.swap(merged), runs.swap(fewer);
      }
      for (const Entry &e : group) f(e);
      group.clear(), runs.assign(1, 0), busy = 0;
    }
  }

  const FusedCost &cost_;
  std::vector<BwdUnit> tiles_;
  std::vector<uint64_t> key_;
  const int hkv_;
  std::vector<Doc> docs_;
  std::array<std::vector<Chain>, N_XCD> chains_;
  size_t longest_ = 0;
};

// beyond_static: cut units may take the backward workspace beyond the library's static one where whole units would not.
// Returns whether the search for cuts saw a tenth less time there.
bool schedule(ca_plan_t *p, bool beyond_static) {
  const int hq = p->hq, hkv = p->hkv, g = hq / hkv;
  // tasks of each document, by position
  std::vector<std::vector<int32_t>> by_doc(p->n_docs);
  for (int t = 0; t < p->n_tasks; ++t) by_doc[p->task_doc[t]].push_back(t);
  // heads packed into the units of partial tiles: the largest of 8, 4, 2, 1 that divides the group size; a document's
  // slots are padded to whole packed units (and to whole backward q blocks)
  const int hp = g % 8 == 0 ? 8 : g % 4 == 0 ? 4 : g % 2 == 0 ? 2 : 1;
  const int sub = FWD_BM / hp;  // slots of a packed unit
  const int align = std::max(sub, BWD_BQ);
  p->heads_packed = hp;
  p->slot_align = align;
  int64_t padded = 0;
  for (auto &v : by_doc) {
    int64_t n = 0;
    for (int t : v) n += p->task_q_len[t];
    padded += round_up(n, align);
  }
  CA_REQUIRE(padded < (int64_t(1) << 31) - SLOT_ALIGN, CA_ERR_UNSUPPORTED, "too many padded query rows");
  p->slot_row.assign(padded, -1);
  p->slot_pos.assign(padded, 0);
  p->block_rpk.assign(padded / BWD_BQ, 0);

  struct TileRef {
    int32_t cost;
    FwdUnit u;
    int32_t part = -1, pieces = 1, piece = 0;  // in the piece list: first part of the unit's first head, pieces, which
  };
  std::vector<TileRef> ftiles;
  std::vector<BwdUnit> btiles;
  // A tile of `keys` keys of a document.  Blocks from its slot_full on lie entirely below the diagonal: they see all keys of the
  // tile, and `beyond` more.
  struct DocTiles {
    int64_t s0, s1;
    int32_t kv_row0, len, cover, heads;
  };
  std::vector<DocTiles> doc_tiles;
  auto kv_tile = [&](const DocTiles &x, int32_t k0, int32_t keys, int32_t beyond) {
    BwdUnit u{int32_t(x.s1), int32_t(x.s1), int32_t(x.s1), x.kv_row0 + k0, std::min<int32_t>(keys, x.len - k0), k0, 0};
    u.heads = x.heads;
    if (k0 < x.cover) {
      // first slot whose position can see key k0
      const int32_t *b = p->slot_pos.data() + x.s0, *e = p->slot_pos.data() + x.s1;
      int64_t first = *b >= k0 ? 0 : std::lower_bound(b, e, k0) - b;  // (a shard behind all of them: no search)
      first = first / BWD_BQ * BWD_BQ;
      int64_t end = x.s1;
      while (end - BWD_BQ >= x.s0 + first && p->slot_row[end - BWD_BQ] < 0) end -= BWD_BQ;  // drop pure-padding blocks
      u.slot_begin = int32_t(x.s0 + first);
      u.slot_end = int32_t(end);
      const int32_t last = k0 + keys - 1 + beyond;
      int64_t full = *b >= last ? 0 : std::lower_bound(b, e, last) - b;
      full = (full + BWD_BQ - 1) / BWD_BQ * BWD_BQ;
      u.slot_full = int32_t(std::min<int64_t>(std::max<int64_t>(x.s0 + full, u.slot_begin), end));
    }
    return u;
  };
  int64_t s = 0, covered_kv = 0, covered_q = 0;
  for (int t = 0; t < p->n_tasks; ++t) covered_q += p->task_q_len[t];
  for (int dd = 0; dd < p->n_docs; ++dd) {
    auto &v = by_doc[dd];
    if (v.empty()) continue;
    std::stable_sort(v.begin(), v.end(), [&](int a, int b) { return p->task_q_pos[a] < p->task_q_pos[b]; });
    // overlapping position ranges of two tasks would interleave; a merge by position keeps slots sorted
    struct Row {
      int32_t pos, row;
    };
    const int64_t s0 = s;
    // a slot's "position" is the last key its row sees: min(document position, kv_len - 1); a task with a prefix
    // shorter than its rows' positions (a shard attending a window of its context) is thereby clipped to the window
    for (int t : v)
      for (int64_t i = 0; i < p->task_q_len[t]; ++i, ++s) {
        p->slot_row[s] = int32_t(p->task_q_start[t] + i);
        p->slot_pos[s] = int32_t(std::min(p->task_q_pos[t] + i, p->task_kv_len[t] - 1));
      }
    const bool sorted = std::is_sorted(p->slot_pos.begin() + s0, p->slot_pos.begin() + s);
    if (!sorted) {  // rare: tasks of one document covering the same positions twice, or clipped below earlier tasks
      std::vector<Row> rows(s - s0);
      for (int64_t i = s0; i < s; ++i) rows[i - s0] = {p->slot_pos[i], p->slot_row[i]};
      std::stable_sort(rows.begin(), rows.end(), [](const Row &a, const Row &b) { return a.pos < b.pos; });
      for (int64_t i = s0; i < s; ++i) p->slot_pos[i] = rows[i - s0].pos, p->slot_row[i] = rows[i - s0].row;
    }
    const int32_t last_pos = p->slot_pos[s - 1];
    // A document that brings at most 32 rows: the dK/dV kernel's 64-row tiles of its one query block take the rows of
    // 4 heads (16 rows each) or 2 heads (32 rows each) of the KV group instead of one head's rows and padding.
    const int64_t n_rows = s - s0;
    const int rpk = n_rows <= 16 && g % 4 == 0 ? 16 : n_rows <= 32 && g % 2 == 0 ? 32 : 0;
    const int32_t tiles_per_block = rpk ? g / (BWD_BQ / rpk) : g;
    if (rpk) p->block_rpk[s0 / BWD_BQ] = rpk;
    const int64_t s1 = round_up(s - s0, align) + s0;
    for (; s < s1; ++s) p->slot_pos[s] = last_pos;  // padding slots: row -1, position of the last real row
    const int32_t kv_row0 = int32_t(p->doc_kv_start[dd]);
    // forward units: full tiles of 256 slots, then head-packed units over the rest
    int64_t a = s0;
    for (; a + FWD_BM <= s1; a += FWD_BM) {
      if (p->slot_row[a] < 0) break;  // pure padding
      int32_t n_keys = p->slot_pos[a + FWD_BM - 1] + 1;
      ftiles.push_back({(n_keys + FWD_BN - 1) / FWD_BN, {int32_t(a), kv_row0, n_keys, 0, 1, 0, -1, int32_t(std::min<int64_t>(FWD_BM, s0 + n_rows - a))}});
    }
    for (; a < s1; a += sub) {
      if (p->slot_row[a] < 0) break;  // pure padding
      int32_t n_keys = p->slot_pos[a + sub - 1] + 1;
      ftiles.push_back({(n_keys + FWD_BN - 1) / FWD_BN, {int32_t(a), kv_row0, n_keys, 0, int32_t(hp), 0, -1, int32_t(std::min<int64_t>(sub, s0 + n_rows - a))}});
    }
    // backward KV tiles: every resident key of the document.  Keys beyond the last query position get a
    // unit without query blocks, which writes their zero gradient.
    const int32_t cover = last_pos + 1;
    const int32_t doc_len = int32_t(p->doc_kv_len[dd]);
    const DocTiles doc{s0, s1, kv_row0, doc_len, cover, tiles_per_block};
    for (int32_t k0 = 0; k0 < doc_len; k0 += BWD_BN) btiles.push_back(kv_tile(doc, k0, BWD_BN, 0));
    doc_tiles.push_back(doc);
    covered_kv += doc_len;
  }
  // longest first (the hardware dispatcher hands out workgroups in index order, so this is LPT
  // list scheduling); unit index modulo n_kv_heads equals the KV head, so that with workgroups dealt
  // round-robin to the 8 XCDs each L2 sees the K/V of as few KV heads as possible.
  std::stable_sort(ftiles.begin(), ftiles.end(), [](const TileRef &a, const TileRef &b) { return a.cost > b.cost; });
  p->fwd_units.reserve(ftiles.size() * hq);
  p->fwd_steps = 0;
  for (auto &t : ftiles)
    for (int i = 0; i < hq / t.u.hp; ++i) {  // KV heads fastest; inside a KV head, its groups of hp query heads
      FwdUnit u = t.u;
      u.head = (i % hkv) * g + (i / hkv) * u.hp;
      p->fwd_units.push_back(u);
      p->fwd_steps += t.cost;
    }
  std::stable_sort(btiles.begin(), btiles.end(), [](const BwdUnit &a, const BwdUnit &b) {
    return int64_t(a.slot_end - a.slot_begin) * a.heads > int64_t(b.slot_end - b.slot_begin) * b.heads;
  });
  p->pos_kv = p->slot_pos;
  for (size_t blk = 0; blk < p->block_rpk.size(); ++blk)
    if (const int rpk = p->block_rpk[blk])
      for (int i = 0; i < BWD_BQ; ++i) p->pos_kv[blk * BWD_BQ + i] = p->slot_pos[blk * BWD_BQ + i % rpk];
  auto base_workspace = [&]() {
    // workspace of backward, all in slot order: per (head, slot) fp32 -Delta and log2(e)*LSE, then bf16 copies of Q
    // and dO as [block of 64 slots][head][64][head_dim] (the dK/dV kernel re-reads their 64-slot tiles once per 128-key
    // tile: in this layout a tile is one contiguous run and needs no row indices)
    const size_t per = (size_t(padded) * hq * sizeof(float) + 255) / 256 * 256;
    const size_t copy = (size_t(padded) * hq * p->d * 2 + 255) / 256 * 256;
    p->ws_off_l2 = per;
    p->ws_off_qs = 2 * per;
    p->ws_off_dos = 2 * per + copy;
    p->ws_off_stats_kv = 2 * per + 2 * copy;
    return 4 * per + 2 * copy;
  };
  // Partial results are bounded: at most this much more than whole units need, and, unless beyond_static, no more than what the
  // library's static workspace has left over (at 8 query heads of 128 it holds 15.8K rows, so from 8K rows on too little to cut
  // with: forward + backward of 9K rows, 8/1 heads, 1.75 ms with what is left and 0.85 ms with 256 MiB).
  constexpr size_t MAX_CUT_BYTES = size_t(256) << 20;
  size_t cut_budget = 0;
  std::array<size_t, 2> limits{};
  bool more = false;
  bool us_wanted = false;
  bool one_pass = false;  // worth a look
  double us_kv = 0;       // (see where it is set)
  double us_apart = 0, us_lists = 0;  // simulated time of the backward in two launches, and as the lists run it
  const CutCost cost_dkv = p->d == 128 ? CutCost{N_CU, 1.65, 10.0, 5.0, 4} : CutCost{2 * N_CU, 1.75, 12.0, 5.0, 4};
  const double dq_per_tile = p->d == 128 ? 2.4 : 1.4, dq_fixed = 8.0;  // of the dQ kernel
  const CutCost cost_fwd = {N_CU, p->d == 128 ? 1.9 : 1.1, 8.0, 5.0, 4};
  std::vector<int64_t> wg_steps;  // of the dK/dV kernel's workgroups of one KV head, as they are launched
  p->bwd_steps = 0;
  for (auto &t : btiles) p->bwd_steps += int64_t(t.slot_end - t.slot_begin) / BWD_BQ * t.heads * hkv;
  {
    // Chains of the dK/dV kernel: consecutive KV tiles of the sorted list (equal or similar cost; the tiles of one
    // document under the same query rows are neighbours in it) whose units are short - at most CHAIN_UNIT_STEPS
    // steps each - go to one workgroup per KV head.  A chain
    // takes at most CHAIN_STEPS_MAX steps and CHAIN_UNITS_MAX units, and at most 1/(2 N_CU) of the short units' steps
    // still to be handed out: chains shrink towards the end of the list, so that the last workgroups of the launch
    // are small ones and the CUs finish together.
    constexpr int64_t CHAIN_UNIT_STEPS = 16, CHAIN_STEPS_MAX = 256, CHAIN_UNITS_MAX = 32;
    auto cost = [&](const BwdUnit &u) { return int64_t(u.slot_end - u.slot_begin) / BWD_BQ * u.heads; };
    int64_t remaining = 0;  // steps of short units, all KV heads
    for (auto &t : btiles)
      if (cost(t) <= CHAIN_UNIT_STEPS) remaining += cost(t) * hkv;
    struct Chain {
      size_t a, b;  // tiles [a, b) of the sorted list
      int64_t steps;
    };
    std::vector<Chain> chains;
    for (size_t a = 0; a < btiles.size();) {
      size_t b = a + 1;
      int64_t sum = cost(btiles[a]);
      if (sum <= CHAIN_UNIT_STEPS) {
        const int64_t target = std::min<int64_t>(CHAIN_STEPS_MAX, remaining / (2 * N_CU));
        while (b < btiles.size() && sum + cost(btiles[b]) <= target && int64_t(b - a) < CHAIN_UNITS_MAX)
          sum += cost(btiles[b++]);
        remaining -= sum * hkv;
      }
      chains.push_back({a, b, sum});
      a = b;
    }
    // workgroups are handed out in index order: longest first, a chain counting with all its steps
    auto lay_out = [&](std::vector<Chain> &list, const std::vector<BwdUnit> &tiles, std::vector<BwdUnit> &units,
                       const std::vector<int32_t> &pieces, int32_t &workgroups) {
      // (pieces: 0, or how many pieces the unit is cut into; those have their first head's part in `follow`)
      std::stable_sort(list.begin(), list.end(), [](const Chain &x, const Chain &y) { return x.steps > y.steps; });
      workgroups = int32_t(list.size() * hkv);
      units.reserve(tiles.size() * hkv);
      units.resize(size_t(workgroups));
      wg_steps.clear();
      for (auto &c : list) wg_steps.push_back(c.steps);
      for (size_t ci = 0; ci < list.size(); ++ci) {
        const size_t a = list[ci].a, b = list[ci].b;
        for (int h = 0; h < hkv; ++h) {
          BwdUnit u = tiles[a];
          u.kv_head = h;
          u.count = int32_t(b - a);
          if (!pieces.empty() && pieces[a] > 0) u.follow -= h * pieces[a];  // the pieces' parts of a head are neighbours
          else u.follow = b - a > 1 ? int32_t(units.size()) : 0;
          units[ci * hkv + h] = u;
          for (size_t t = a + 1; t < b; ++t) {
            BwdUnit f = tiles[t];
            f.kv_head = h;
            units.push_back(f);
          }
        }
      }
    };
    lay_out(chains, btiles, p->bwd_units, {}, p->bwd_workgroups);
    p->ws_bwd = base_workspace();
    // the list in which long units that run alone are cut along their query blocks
    cut_budget = p->ws_bwd <= CA_STATIC_WS_BYTES && !beyond_static ? CA_STATIC_WS_BYTES - p->ws_bwd : MAX_CUT_BYTES;
    limits = {cut_budget, MAX_CUT_BYTES};
    std::vector<std::pair<int64_t, int64_t>> sizes;
    for (auto &c : chains) {
      if (!sizes.empty() && sizes.back().first == c.steps) sizes.back().second += hkv;
      else sizes.push_back({c.steps, hkv});
    }
    const auto [cut, free_cut] = best_piece(sizes, cost_dkv, part_bytes(p->d), limits);
    more = more || free_cut.us < 0.9 * cut.us;
    const int64_t T = cut.piece;
    if (T > 0) {
      std::vector<BwdUnit> tiles;
      std::vector<int32_t> pieces;
      std::vector<Chain> list;
      for (auto &c : chains) {
        const BwdUnit &u = btiles[c.a];
        const int64_t blocks = (u.slot_end - u.slot_begin) / BWD_BQ;
        const int64_t k = c.b - c.a == 1 && c.steps > T ? std::min(blocks, (c.steps + T - 1) / T) : 1;
        if (k <= 1) {
          list.push_back({tiles.size(), tiles.size() + (c.b - c.a), c.steps});
          tiles.insert(tiles.end(), btiles.begin() + c.a, btiles.begin() + c.b);
          pieces.resize(tiles.size(), 0);
          continue;
        }
        for (int64_t i = 0; i < k; ++i) {
          BwdUnit v = u;
          v.slot_begin = int32_t(u.slot_begin + blocks * i / k * BWD_BQ);
          v.slot_end = int32_t(u.slot_begin + blocks * (i + 1) / k * BWD_BQ);
          v.slot_full = std::min(std::max(u.slot_full, v.slot_begin), v.slot_end);
          v.follow = -1 - (p->n_bwd_parts + int32_t(i));
          list.push_back({tiles.size(), tiles.size() + 1, cost(v)});
          tiles.push_back(v);
          pieces.push_back(int32_t(k));
        }
        for (int h = 0; h < hkv; ++h, p->n_bwd_parts += int32_t(k))
          p->bwd_combine.push_back({p->n_bwd_parts, int32_t(k), u.kv_row, u.n_valid, h, 0});
      }
      if (!p->bwd_combine.empty()) lay_out(list, tiles, p->bwd_pieces, pieces, p->bwd_piece_workgroups);
    }
  }
  {
    // the list in which long forward / dQ units are cut along their keys (one list for both kernels: per step 1.5 to
    // 2.05 and 2.4 us at head_dim 128, for which 1.9 stands)
    std::vector<std::pair<int64_t, int64_t>> sizes;
    for (auto &t : ftiles) {
      if (!sizes.empty() && sizes.back().first == t.cost) sizes.back().second += hq / t.u.hp;
      else sizes.push_back({t.cost, hq / t.u.hp});
    }
    const auto [cut, free_cut] = best_piece(sizes, cost_fwd, part_bytes(p->d) + FWD_STAT_BYTES, limits);
    more = more || free_cut.us < 0.9 * cut.us;
    p->us_fwd = cut.us;
    int64_t T = cut.piece;
    // That search takes a CU for one server.  Long pieces are worth a look at both forms of a workgroup, in both kernels.  By the
    // search 128 units of 2032 tiles are 256 pieces, and 176 of 938 stay whole; 512 pieces, of which two whole ones share a CU, and
    // 704 take 1.64 ms instead of 1.85 and 1.15 instead of 1.41 in the forward, and no longer in the backward.  (Not where units hold
    // a few rows: four rows of each of five documents, 16/16 heads, gained 200 us of 1130 and lost 150 of 3900 in the backward, whose
    // halves of padding read all keys.)
    constexpr int64_t LONG_PIECE = 128;
    const int64_t longest = ftiles.empty() ? 0 : ftiles[0].cost, units = int64_t(p->fwd_units.size());
    const bool filled = std::all_of(ftiles.begin(), ftiles.end(), [&](const TileRef &t) { return t.u.rows > 4 / t.u.hp * 32; });
    if (filled && longest >= 2 * LONG_PIECE && 2 * units <= 4 * N_CU) {
      struct Run {
        double fwd, both;
        size_t bytes;
      };
      auto run_of = [&](int64_t t) {
        std::vector<FwdUnits> list;
        std::vector<std::pair<double, int64_t>> dq;
        int64_t parts = 0;
        for (const auto &[tiles, n] : sizes) {
          const int64_t k = t > 0 ? std::max<int64_t>(1, (tiles + t - 1) / t) : 1;
          const double of_piece = double(tiles) / double(k);
          list.push_back({of_piece, of_piece, n * k});
          if (k > 1) parts += n * k;
        }
        std::stable_sort(list.begin(), list.end(), [](const FwdUnits &a, const FwdUnits &b) { return a.tiles > b.tiles; });
        for (const FwdUnits &x : list) dq.push_back({dq_fixed + dq_per_tile * x.tiles, x.n});
        Run r{fwd_run(list, p->d).us, 0.0, size_t(parts) * (part_bytes(p->d) + FWD_STAT_BYTES)};
        if (parts > 0) r.fwd += cost_fwd.launch + double(r.bytes) / BYTES_PER_US;
        r.both = r.fwd + makespan(dq, N_CU, 1e30, JOINT_UNITS);
        if (parts > 0) r.both += cost_fwd.launch + double(r.bytes) / BYTES_PER_US;
        return r;
      };
      Run best = run_of(T), beyond = best;
      for (int64_t k = 2; k * units <= 4 * N_CU && longest >= k * LONG_PIECE; ++k) {
        const int64_t t = (longest + k - 1) / k;
        const Run r = run_of(t);
        if (r.bytes <= limits[0] && r.both + BEYOND_STATIC_US < best.both) best = r, T = t;
        if (r.bytes <= limits[1] && r.both < beyond.both) beyond = r;
      }
      p->pieces_lost = best.both - beyond.both > BEYOND_STATIC_US;
      more = more || p->pieces_lost;
      p->us_fwd = best.fwd;
    }
    if (T > 0) {
      std::vector<TileRef> pieces;
      for (auto &t : ftiles) {
        const int64_t k = t.cost > T ? (t.cost + T - 1) / T : 1;
        if (k <= 1) {
          pieces.push_back(t);
          continue;
        }
        for (int64_t i = 0; i < k; ++i) {
          TileRef v = t;
          const int32_t a = int32_t(t.cost * i / k), b = int32_t(t.cost * (i + 1) / k);  // tiles [a, b)
          v.cost = b - a;
          v.u.key0 = a * FWD_BN;
          v.u.kv_row0 = t.u.kv_row0 + v.u.key0;
          v.u.n_keys = std::min(t.u.n_keys, b * FWD_BN) - v.u.key0;
          v.part = p->n_fwd_parts, v.pieces = int32_t(k), v.piece = int32_t(i);
          pieces.push_back(v);
        }
        for (int i = 0; i < hq / t.u.hp; ++i, p->n_fwd_parts += int32_t(k))
          p->fwd_combine.push_back({p->n_fwd_parts, int32_t(k), t.u.slot0, (i % hkv) * g + (i / hkv) * t.u.hp, t.u.hp, 0});
      }
      // (pieces of one length by the window they attend: the pieces that read the same keys run side by side)
      std::stable_sort(pieces.begin(), pieces.end(), [](const TileRef &a, const TileRef &b) {
        return a.cost != b.cost ? a.cost > b.cost : a.u.kv_row0 < b.u.kv_row0;
      });
      for (auto &t : pieces)
        for (int i = 0; i < hq / t.u.hp; ++i) {
          FwdUnit u = t.u;
          u.head = (i % hkv) * g + (i / hkv) * u.hp;
          u.part = t.part < 0 ? -1 : t.part + i * t.pieces + t.piece;
          p->fwd_pieces.push_back(u);
        }
    }
  }
  {
    auto form = [&](const std::vector<FwdUnit> &units) {
      std::vector<FwdUnits> list;
      if (units.size() > size_t(4 * N_CU)) return FwdForm{};
      for (size_t i = 0, n; i < units.size(); i += n) {
        const FwdUnit &u = units[i];
        n = size_t(hq / u.hp);
        const int32_t tiles = (u.n_keys + FWD_BN - 1) / FWD_BN;
        // the tiles the first half's rows see (its last slot has its highest position)
        const int32_t last = p->slot_pos[size_t(u.slot0 + (3 / u.hp) * 32 + 31)] - u.key0;
        list.push_back({double(tiles), double(std::max(1, std::min(tiles, last / FWD_BN + 1))), int64_t(n)});
      }
      return fwd_run(list, p->d).form;
    };
    p->fwd_form = form(p->fwd_units);
    p->fwd_piece_form = form(p->fwd_pieces);
  }
  {
    // One launch or two for the backward.  The dQ kernel proper runs 256 rows per workgroup; in the joint launch a workgroup is
    // half of that, two to a CU at the same pace per row (2.4 us per tile of 256 rows at head_dim 128, 1.4 at 64), which fills
    // the CUs that too few dK/dV units leave idle, and saves a launch.
    const int slots = cost_dkv.slots;
    double mean = 0;
    for (int64_t s : wg_steps) mean += (cost_dkv.fixed + cost_dkv.per_step * double(s)) * hkv / slots;
    {
      // the one pass is worth a look where there is enough work, not too much of it around the steps of its units, and its 32-bit
      // offsets reach; `level`: both kinds of list, were they spread evenly
      const FusedCost &cost = p->d == 128 ? FUSED_128 : FUSED_64;
      const int32_t keys = 32 * fused_waves(p->d);
      double n_tiles = 0, level = mean;
      for (const DocTiles &x : doc_tiles) n_tiles += double((x.len + keys - 1) / keys);
      for (const TileRef &t : ftiles) level += (dq_fixed + dq_per_tile * t.cost) * (hq / t.u.hp) / N_CU;
      const double in_steps = cost.per_step * 2.0 * double(p->bwd_steps) * BWD_BN / keys / (cost.slots * N_XCD);
      us_kv = 0.4 * 6.0 * double(p->total_kv) * hkv * p->d * 2 / BYTES_PER_US;
      if (in_steps >= cost.least && cost.gain * (in_steps + cost.fixed * n_tiles * hkv / (cost.slots * N_XCD)) < 1.2 * (level + us_kv) &&
          size_t(padded) * size_t(hq) * size_t(p->d) * 4 <= UINT32_MAX)
        one_pass = true;
    }
    const bool may_join = mean < (p->d == 128 ? JOINT_MAX_US : JOINT_MAX_US_64);
    const bool wanted = may_join || p->pieces_lost || beyond_static;
    us_wanted = wanted;
    if (!wg_steps.empty() && !p->fwd_units.empty() && (wanted || one_pass)) {
      // groups of equal workgroups that follow each other in their list: (microseconds, how many, first entry of joint_order,
      // step from entry to entry)
      struct Group {
        double us;
        int32_t n, entry, step;
      };
      std::vector<Group> groups;
      const std::vector<FwdUnit> &units = p->fwd_pieces.empty() ? p->fwd_units : p->fwd_pieces;
      const int32_t n_dq = int32_t(units.size());
      const int64_t same = std::gcd<int64_t>(N_CU, std::gcd(hkv, hq / hp));
      std::vector<std::pair<double, int64_t>> dkv, dq;
      double sum = 0, longest = 0;
      for (size_t i = 0; i < wg_steps.size(); ++i) {
        const double us = cost_dkv.fixed + cost_dkv.per_step * double(wg_steps[i]);
        dkv.push_back({us, hkv / same});
        if (may_join) groups.push_back({us, hkv, int32_t(i) * hkv, 1});
        sum += us * hkv;
        longest = std::max(longest, us);
      }
      const double per_half = p->d == 128 ? 1.2 : 1.4, fixed_half = p->d == 128 ? 4.0 : 7.0;
      for (int32_t half = 1; half >= (may_join ? 0 : 1); --half)
        for (int32_t i = 0, n; i < n_dq; i += n) {
          const FwdUnit &u = units[size_t(i)];
          const int32_t tiles = (u.n_keys + FWD_BN - 1) / FWD_BN;
          n = hq / u.hp;
          if (half == 1) dq.push_back({dq_fixed + dq_per_tile * tiles, n / same});
          if (!may_join) continue;
          // the tiles the half's rows see (its last slot has its highest position)
          const int32_t last = p->slot_pos[size_t(u.slot0 + ((4 * half + 3) / u.hp) * 32 + 31)] - u.key0;
          const double us = fixed_half + per_half * std::max(1, std::min(tiles, last / FWD_BN + 1));
          groups.push_back({us, n, -1 - (half * n_dq + i), -1});
          sum += us * n;
          longest = std::max(longest, us);
        }
      const double parts_us = p->n_fwd_parts + p->n_bwd_parts > 0
                                  ? cost_dkv.launch + double(size_t(p->n_fwd_parts + p->n_bwd_parts) * part_bytes(p->d)) / BYTES_PER_US
                                  : 0.0;
      const double apart = makespan(dkv, slots / same, 1e30, JOINT_UNITS) + makespan(dq, N_CU / same, 1e30, JOINT_UNITS) + cost_dkv.launch;
      us_lists = us_apart = apart + parts_us;
      if (may_join && sum / slots < apart) {
        std::vector<std::pair<double, int64_t>> all;
        auto span_of = [&](double at_most) {
          all.clear();
          for (const Group &x : groups) all.push_back({x.us, x.n / same});
          return makespan(all, slots / same, at_most, JOINT_UNITS);
        };
        // dK/dV units, then dQ halves, or, where that is shorter by more than the look-up it takes, all by their length
        const double listed = span_of(apart + 2.0);
        const double goal = std::min(listed - 2.0, apart);  // what the order by length has to beat; no order beats the mean load
        double sorted = goal;
        if (sum / slots < goal && longest < goal) {
          std::stable_sort(groups.begin(), groups.end(), [](const Group &x, const Group &y) { return x.us > y.us; });
          sorted = span_of(goal);
        }
        const bool order = sorted < goal;
        p->joint = order || listed < apart;
        if (p->joint) us_lists = (order ? sorted : listed) + parts_us;
        if (p->joint && order)
          for (const Group &x : groups)
            for (int32_t i = 0; i < x.n; ++i) p->joint_order.push_back(x.entry + i * x.step);
      }
    }
  }
  // workspace with which the piece lists are used
  if (p->n_fwd_parts > 0) p->ws_fwd_split = size_t(p->n_fwd_parts) * (part_bytes(p->d) + FWD_STAT_BYTES);
  p->ws_bwd_split = p->ws_bwd;
  if (p->n_fwd_parts + p->n_bwd_parts > 0) {
    // [dK/dV parts][dQ parts], or, where that is beyond the budget, one region that the dQ parts use after the dK/dV parts have been added up (one launch more)
    p->ws_off_parts_kv = p->ws_off_parts_dq = p->ws_bwd;
    const size_t kv = size_t(p->n_bwd_parts) * part_bytes(p->d), dq = size_t(p->n_fwd_parts) * part_bytes(p->d);
    p->shared_parts = kv > 0 && dq > 0 && kv + dq > cut_budget;
    if (p->shared_parts) {
      p->joint_lost = p->joint;
      p->joint = false, p->joint_order.clear(), us_lists = us_apart;
    }
    if (!p->shared_parts) p->ws_off_parts_dq += kv;
    p->ws_bwd_split = std::max(p->ws_off_parts_kv + kv, p->ws_off_parts_dq + dq);
  }
  if (us_wanted) p->us_bwd = us_lists;
  // the one pass, where it is faster than the lists above
  if (one_pass) {
    const FusedCost &cost = p->d == 128 ? FUSED_128 : FUSED_64;
    const int32_t keys = 32 * fused_waves(p->d);
    size_t n_tiles = 0;
    for (const DocTiles &x : doc_tiles) n_tiles += size_t((x.len + keys - 1) / keys);
    std::vector<BwdUnit> tiles;
    tiles.reserve(n_tiles);
    for (const DocTiles &x : doc_tiles)
      for (int32_t k0 = 0; k0 < x.len; k0 += keys) tiles.push_back(kv_tile(x, k0, keys, 1));  // (1: another tile adds to their dQ)
    const OnePass pass(*p, std::move(tiles));
    const double at_most = (us_lists + us_kv - cost.more) / cost.gain;
    if (pass.time(at_most) < at_most) pass.lay_out(p);
  }
  p->q_covered = covered_q == p->total_q;
  p->kv_covered = covered_kv == p->total_kv;
  return more;
}

std::unique_ptr<ca_plan_t> described(const ca_batch_desc *desc) {
  auto p = std::make_unique<ca_plan_t>();
  p->n_docs = desc->n_docs, p->n_tasks = desc->n_tasks;
  p->hq = desc->n_q_heads, p->hkv = desc->n_kv_heads, p->d = desc->head_dim;
  p->total_q = desc->total_q, p->total_kv = desc->total_kv;
  p->scale = desc->softmax_scale > 0.f ? desc->softmax_scale : 1.0f / std::sqrt(float(desc->head_dim));
  if (desc->n_docs > 0) {
    p->doc_kv_start.assign(desc->doc_kv_start, desc->doc_kv_start + desc->n_docs);
    p->doc_kv_len.assign(desc->doc_kv_len, desc->doc_kv_len + desc->n_docs);
  }
  if (desc->n_tasks > 0) {
    p->task_doc.assign(desc->task_doc, desc->task_doc + desc->n_tasks);
    p->task_q_start.assign(desc->task_q_start, desc->task_q_start + desc->n_tasks);
    p->task_q_len.assign(desc->task_q_len, desc->task_q_len + desc->n_tasks);
    p->task_q_pos.assign(desc->task_q_pos, desc->task_q_pos + desc->n_tasks);
    p->task_kv_len.assign(desc->task_kv_len, desc->task_kv_len + desc->n_tasks);
  }
  return p;
}
}  // namespace

int build_plan(const ca_batch_desc *desc, ca_plan_t **out) {
  if (!out) {
    set_error("output plan pointer is null");
    return CA_ERR_INVALID_ARG;
  }
  *out = nullptr;
  try {
    validate(desc);
    auto p = described(desc);
    // Where cutting units beyond the static workspace looks better by a tenth, or would save a backward launch worth it (the dQ parts
    // take the place of the dK/dV parts inside, which needs two), or leaves room for two long forward pieces per CU, both plans are
    // made, and kept if the whole pass is better: the larger for callers that bring the workspace, the smaller inside it for all others.  (Forward + backward, 8/2 heads,
    // without and with the launch saved: 2048 rows with an 8K context 318 -> 266 us, 3072 rows 404 -> 356 us; simulated to gain 34 and
    // 38 us.  Below 25 us the larger workspace is not taken for it.)
    const bool more = schedule(p.get(), false);
    if (more || p->joint_lost) {
      auto large = described(desc);
      schedule(large.get(), true);
      const double inside = p->us_fwd + p->us_bwd, beyond = large->us_fwd + large->us_bwd;
      if (p->us_bwd > 0 && large->us_bwd > 0 && ((more && beyond < 0.9 * inside) || ((p->joint_lost || p->pieces_lost) && inside - beyond > BEYOND_STATIC_US))) {
        // (the one pass needs no pieces: what it needs fits behind either plan's whole units, and the larger one offers it)
        p->fused = false, p->fused_units = {}, p->ws_bwd_fused = 0;
        large->within_static = std::move(p);
        p = std::move(large);
      }
    }
    *out = p.release();
  } catch (const Fail &f) {
    set_error(f.msg);
    return f.code;
  } catch (const std::bad_alloc &) {
    set_error("out of host memory while planning");
    return CA_ERR_INVALID_ARG;
  }
  return CA_OK;
}

}  // namespace ca

// the first n_fields ints of every entry of a schedule list
template <class T>
static int64_t leading_fields(const std::vector<T> &list, int32_t *out, size_t n_fields) {
  if (out)
    for (size_t i = 0; i < list.size(); ++i) std::memcpy(out + i * n_fields, &list[i], n_fields * sizeof(int32_t));
  return int64_t(list.size());
}

extern "C" {

int ca_plan_host(const ca_batch_desc *desc, ca_plan_t **out) { return ca::build_plan(desc, out); }

const char *ca_last_error(void) { return ca::last_error(); }

const char *ca_error_string(int code) {
  switch (code) {
    case CA_OK: return "ok";
    case CA_ERR_INVALID_ARG: return "invalid argument";
    case CA_ERR_UNSUPPORTED: return "unsupported configuration";
    case CA_ERR_WORKSPACE: return "workspace missing, too small or misaligned";
    case CA_ERR_HIP: return "HIP runtime error";
    case CA_ERR_STATE: return "plan not uploaded to this device";
    default: return "unknown error code";
  }
}

int ca_plan_workspace_bytes(const ca_plan_t *p, size_t *fwd, size_t *bwd) {
  if (!p) {
    ca::set_error("plan is null");
    return CA_ERR_INVALID_ARG;
  }
  if (fwd) *fwd = p->ws_fwd;
  if (bwd) *bwd = p->ws_bwd;
  return CA_OK;
}

int ca_plan_info(const ca_plan_t *p, int64_t *out, int n) {
  if (!p) return 0;
  int64_t full_tiles = 0;
  for (auto &u : p->fwd_units) full_tiles += u.hp == 1 && u.head == 0;
  const int64_t v[19] = {ca::FWD_BM, full_tiles, int64_t(p->fwd_units.size()),
                         ca::BWD_BN, int64_t(p->bwd_units.size()), ca::FWD_BN, int64_t(p->slot_row.size()),
                         p->fwd_steps, p->bwd_steps, ca::BWD_BQ, p->slot_align, p->heads_packed, p->bwd_workgroups,
                         p->joint, p->fwd_form.halves, p->fwd_piece_form.halves, p->fwd_form.turns, p->fwd_piece_form.turns, p->fused};
  for (int i = 0; i < n && i < 19 && out; ++i) out[i] = v[i];
  return 19;
}

int64_t ca_plan_rows(const ca_plan_t *p, int32_t *rows, int32_t *pos) {
  if (!p) return 0;
  if (rows) std::memcpy(rows, p->slot_row.data(), p->slot_row.size() * sizeof(int32_t));
  if (pos) std::memcpy(pos, p->slot_pos.data(), p->slot_pos.size() * sizeof(int32_t));
  return int64_t(p->slot_row.size());
}

int64_t ca_plan_fwd_units(const ca_plan_t *p, int32_t *units) {
  if (!p) return 0;
  return leading_fields(p->fwd_units, units, ca::FWD_UNIT_INTS);
}

int64_t ca_plan_bwd_units(const ca_plan_t *p, int32_t *units) {
  if (!p) return 0;
  return leading_fields(p->bwd_units, units, sizeof(ca::BwdUnit) / 4);
}

int64_t ca_plan_fwd_pieces(const ca_plan_t *p, int32_t *units) {
  return p ? leading_fields(p->fwd_pieces, units, sizeof(ca::FwdUnit) / 4) : 0;
}

int64_t ca_plan_bwd_pieces(const ca_plan_t *p, int32_t *units, int32_t *n_workgroups) {
  if (!p) return 0;
  if (n_workgroups) *n_workgroups = p->bwd_piece_workgroups;
  return leading_fields(p->bwd_pieces, units, sizeof(ca::BwdUnit) / 4);
}

int64_t ca_plan_one_pass_units(const ca_plan_t *p, int32_t *units, int32_t *queue) {
  if (!p) return 0;
  if (queue) std::copy(std::begin(p->fused_queue), std::end(p->fused_queue), queue);
  return leading_fields(p->fused_units, units, sizeof(ca::BwdUnit) / 4);
}

int64_t ca_plan_combine_units(const ca_plan_t *p, int32_t backward, int32_t *units) {
  return p ? leading_fields(backward ? p->bwd_combine : p->fwd_combine, units, sizeof(ca::CombineUnit) / 4) : 0;
}

int ca_plan_workspace_bytes_split(const ca_plan_t *p, size_t *fwd, size_t *bwd) {
  if (!p) {
    ca::set_error("plan is null");
    return CA_ERR_INVALID_ARG;
  }
  if (fwd) *fwd = std::max(p->ws_fwd, p->ws_fwd_split);
  if (bwd) *bwd = p->ws_bwd_split;
  return CA_OK;
}

int ca_plan_workspace_bytes_one_pass(const ca_plan_t *p, size_t *bwd) {
  if (!p) {
    ca::set_error("plan is null");
    return CA_ERR_INVALID_ARG;
  }
  if (bwd) *bwd = p->ws_bwd_fused;
  return CA_OK;
}

}  // extern "C"
