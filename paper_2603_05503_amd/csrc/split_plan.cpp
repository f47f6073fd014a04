// Plan of a forward whose rows of kept blocks are cut along the keys (calibatt_plan_split): which part of which row
// every workgroup takes.  Integer and cost arithmetic on the host, no device calls.
#include "split_plan.h"

#include <algorithm>
#include <new>
#include <vector>

#include "calibatt.h"

namespace {

struct Part {
  int32_t item, id, first, count, part, n_parts, slot, row, b;
};

// Costs in stages of 64 keys, fitted to every second of 2 487 calls for which the longest part was swept (1 to 40 heads of 900
// to 40 000 tokens, densities 0.12 to 1, banded and uniform masks, every block size and head dimension): what a part costs
// beside its stages (its start, its sums to memory); what adding up costs the longest row, once and for each of its parts;
// and how the longest part, the part that is the first to share a CU, and the rounds weigh against an even share of the
// whole.  Over all of them the lengths chosen take 1.6 % more time than the best ones of the sweep, and 12 calls over 2 % more
// than whole rows; without adding up and shared CUs 2.5 %, and 33: 24 heads of 992 tokens 12.6 us whole, 14.9 with 10 rows
// cut; one head of 8 190 tokens 34.9 us in 288 parts, 30.5 in 256.  Without the rounds 2 heads of 16 320 tokens, 256 rows of 48
// blocks, were cut into a few more parts than there are slots: whole 130 us, in 520 parts 147, in 768 128.
constexpr double PART_COST = 10.0, CHAIN_WEIGHT = 0.75, SHARED_WEIGHT = 0.2, ROUNDS_WEIGHT = 0.8;
constexpr double MERGE_COST = 1.5, MERGE_COST_PER_PART = 0.9;
constexpr int CUS = 256;
// Workgroups that the device holds at a time: two per CU of 128 queries, four of 64.
constexpr int slots_of(int block_q) { return CUS * (block_q >= 128 ? 2 : 4); }
// Above so many stages per slot every call takes whole rows: their workgroups pop from queues that keep an XCD at one head,
// which outweighs an even end where there are many rows for every slot.  The line is a coarse one.  It goes by the work, not
// by what the last round leaves idle, and above it calls of 1 to 1.5 rows a slot would gain from cutting.  us, whole rows /
// by the plan if this line were not there, with stages a slot: 40 heads of 10 000 tokens (6.2 rows a slot) 449 / 440 at 206,
// 565 / 563 at 273, 956 / 989 at 494; 8 heads of 33 000 (4.0) 1 216 / 1 267 at 628; 12 heads of 16 380 (3.0) 520 / 499 at 257,
// 573 / 557 at 287; 2 heads of 33 000 (1.01) 648 / 592 at 262, 789 / 661 at 313, 1 216 / 955 at 468; one of 75 600 (1.15)
// 814 / 696 at 341; 64-query blocks, 2 heads of 33 000 (1.01) 506 / 375 at 261, 682 / 498 at 364.
constexpr int64_t MAX_STAGES_PER_SLOT = 270;

int32_t parts_of(int32_t len, int32_t longest) {
  return std::max(1, std::min<int32_t>(CALIBATT_MAX_PARTS, len / longest + (len % longest != 0)));
}

// The longest part, in key blocks, whose estimated time is least: an even share of all work, the longest row's way, and
// the rounds, whichever is largest, smoothly.  Sorted by length, the part behind one for every CU shares the CU of a longer
// one, and of k * slots + 1 parts some slot takes k + 1, none of them shorter than the last of these.  Rows stay whole
// where cutting them promises less than 3 %.
int32_t choose_longest(const std::vector<int32_t> &rows_of_length, int B, double stages, int slots) {
  const int32_t max_row = (int32_t)rows_of_length.size() - 1;
  std::vector<std::pair<int32_t, int64_t>> lengths;  // (length, rows of it over the batch)
  for (int32_t len = 0; len <= max_row; ++len)
    if (rows_of_length[(size_t)len]) lengths.push_back({len, (int64_t)B * rows_of_length[(size_t)len]});
  std::vector<int64_t> parts((size_t)max_row + 1);  // by length
  auto cube = [](double x) { return x * x * x; };
  int32_t best = max_row;
  double best_cost = 0.0;
  for (int32_t longest = max_row;; longest = longest * 7 / 8) {
    std::fill(parts.begin(), parts.end(), 0);
    int32_t chain = 0;
    for (const auto &l : lengths) {
      const int32_t k = parts_of(l.first, longest), less = l.first / k, more = l.first % k;
      parts[(size_t)less] += (k - more) * l.second;
      if (more) parts[(size_t)less + 1] += more * l.second;
      chain = std::max(chain, less + (more != 0));
    }
    double total = 0.0, rounds = 0.0, way = CHAIN_WEIGHT * chain * stages;
    if (longest < max_row) way += MERGE_COST + MERGE_COST_PER_PART * parts_of(max_row, longest);
    int64_t n = 0;
    for (int32_t len = chain; len >= 0; --len)
      if (parts[(size_t)len]) {
        const double cost = len * stages + PART_COST;
        total += cost * (double)parts[(size_t)len];
        if (n <= CUS && n + parts[(size_t)len] > CUS) way += SHARED_WEIGHT * cost;
        n += parts[(size_t)len];
        if (n > slots) rounds = std::max(rounds, (double)((n - 1) / slots + 1) * cost);
      }
    const double cost = cube(total / slots) + cube(way) + cube(ROUNDS_WEIGHT * rounds);
    if (longest == max_row) best_cost = cube(0.97) * cost;
    else if (cost < best_cost) best = longest, best_cost = cost;
    if (longest <= 1) return best;
  }
}

// Sorts by key(x), in [0, n_keys), and keeps equals in order.  (Comparing instead takes 50 ns an entry and sort, most of a
// plan: 704 rows of 64 blocks 45 us.)
template <typename KeyOf>
void sort_by(std::vector<int32_t> &a, int32_t n_keys, KeyOf key) {
  std::vector<int32_t> at((size_t)n_keys + 1, 0), sorted(a.size());
  for (int32_t x : a) ++at[(size_t)key(x) + 1];
  for (int32_t k = 0; k < n_keys; ++k) at[(size_t)k + 1] += at[(size_t)k];
  for (int32_t x : a) sorted[(size_t)at[(size_t)key(x)]++] = x;
  a.swap(sorted);
}

}  // namespace

extern "C" int calibatt_plan_split(const calibatt_pattern *pattern, int B, int max_blocks, int32_t *parts,
                                   int64_t cap_parts, calibatt_split *split) {
  if (!pattern || !split || !pattern->row_ptr || !pattern->work || !pattern->fan_ptr) return CALIBATT_ERR_NULL;
  if (B <= 0 || max_blocks < 0 || cap_parts < 0 || pattern->n_work < 0 || pattern->block_k <= 0 || pattern->nbq <= 0) return CALIBATT_ERR_SHAPE;
  *split = calibatt_split{};
  split->B = B;
  const int n = pattern->n_work;
  const double stages = pattern->block_k / 64.0;
  const int slots = slots_of(pattern->block_q);
  if (n == 0 || (int64_t)n * B > 1 << 20 || (max_blocks == 0 && (double)pattern->nnz * B * stages > (double)MAX_STAGES_PER_SLOT * slots))
    return CALIBATT_OK;
  const int32_t *const row_ptr = pattern->row_ptr;
  auto length = [&](int32_t id) { return row_ptr[id + 1] - row_ptr[id]; };
  try {
    // rows in the order of heads and query blocks
    std::vector<int32_t> rows((size_t)n);  // items
    int32_t max_row = 1, max_id = 0;
    for (int i = 0; i < n; ++i) {
      rows[(size_t)i] = i;
      max_id = std::max(max_id, pattern->work[i]);
      max_row = std::max(max_row, length(pattern->work[i]));
    }
    sort_by(rows, max_id + 1, [&](int32_t i) { return pattern->work[i]; });
    int32_t longest = max_blocks;
    if (longest == 0) {
      std::vector<int32_t> rows_of_length((size_t)max_row + 1, 0);
      for (int32_t i : rows) ++rows_of_length[(size_t)length(pattern->work[i])];
      longest = choose_longest(rows_of_length, B, stages, slots);
    }
    // cut into parts of nearly equal length
    std::vector<Part> all;
    all.reserve((size_t)n * B);
    int32_t n_slots = 0, n_rows = 0;
    double total = 0.0;
    auto cost = [&](const Part &p) { return p.count * stages + PART_COST; };
    for (int b = 0; b < B; ++b)
      for (int32_t i : rows) {
        const int32_t id = pattern->work[i], len = length(id), k = parts_of(len, longest);
        for (int32_t j = 0; j < k; ++j) {
          const int32_t lo = (int32_t)((int64_t)len * j / k), hi = (int32_t)((int64_t)len * (j + 1) / k);
          all.push_back({i, id, lo, hi - lo, j, k, k > 1 ? n_slots : 0, k > 1 ? n_rows : 0, b});
          total += cost(all.back());
        }
        if (k > 1) n_slots += k, ++n_rows;
      }
    // eight ranges of equal cost, one per XCD, of the parts ordered by batch, head and the keys in their middle, so that
    // an XCD's workgroups share keys in its L2; in each the longest parts first
    std::vector<int32_t> order(all.size());
    for (size_t i = 0; i < all.size(); ++i) order[i] = (int32_t)i;
    if (pattern->col_idx) {
      const int32_t nbq = pattern->nbq, heads = max_id / nbq + 1, last = std::max(pattern->nbk, 1) - 1;
      sort_by(order, last + 1, [&](int32_t i) {
        const Part &p = all[(size_t)i];
        const int32_t middle = p.count ? pattern->col_idx[row_ptr[p.id] + p.first + p.count / 2] : 0;
        return std::min(std::max(middle, 0), last);
      });
      sort_by(order, B * heads, [&](int32_t i) { return all[(size_t)i].b * heads + all[(size_t)i].id / nbq; });
    }
    // An XCD has an eighth of the slots, and no XCD gets more parts than its slots take in the rounds that all parts need:
    // 1 020 rows of 58 blocks (10 846 tokens, 12 heads) 507 us where one XCD had a third round for a few of them, and 709
    // for 1 024 rows of 116 with 64-query blocks, against 459 and 564 for whole rows from the queues.
    // Of parts that fit at a time no XCD gets more than its CUs take by ones, by twos and so on: of 255 rows (15 heads of
    // 2 115 tokens) an XCD got 33 for its 32 CUs, uncut 49.6 us against 41.1 and 42.0 whole; one head of 30 679, 240 rows,
    // 543 against 474 and 492.
    const int32_t n_all = (int32_t)order.size(), step = n_all <= slots ? CUS : slots,
                  most_of_xcd = step / CALIBATT_GROUPS * ((n_all - 1) / step + 1);
    std::vector<int32_t> list[CALIBATT_GROUPS];
    double before = 0.0;
    int xcd = 0;
    for (int32_t at = 0; at < n_all; ++at) {
      const int32_t i = order[(size_t)at];
      const Part &p = all[(size_t)i];
      const int by_cost = (int)((before + 0.5 * cost(p)) * CALIBATT_GROUPS / total);
      const int room_for_rest = CALIBATT_GROUPS - (n_all - at + most_of_xcd - 1) / most_of_xcd;
      xcd = std::max(xcd, std::min(std::min(by_cost, CALIBATT_GROUPS - 1), room_for_rest));
      if ((int32_t)list[xcd].size() == most_of_xcd) ++xcd;
      list[xcd].push_back(i);
      before += cost(p);
    }
    size_t most = 0;
    for (auto &l : list) {
      sort_by(l, max_row + 1, [&](int32_t i) { return max_row - all[(size_t)i].count; });
      most = std::max(most, l.size());
    }
    const int64_t n_parts = (int64_t)most * CALIBATT_GROUPS;
    if (n_parts > 0x7fffffffLL / CALIBATT_PART_WORDS) return CALIBATT_ERR_SHAPE;
    split->n_parts = (int32_t)n_parts;
    split->n_rows = n_rows;
    split->n_slots = n_slots;
    if (!parts) return CALIBATT_OK;
    if (cap_parts < n_parts) return CALIBATT_ERR_BUFFER_TOO_SMALL;
    // one part of every XCD's list in turn, as workgroups are dealt to the XCDs; a list that has ended gives -1
    const int32_t *const iv_ptr = pattern->iv_ptr;
    for (size_t i = 0; i < most; ++i)
      for (int x = 0; x < CALIBATT_GROUPS; ++x) {
        int32_t *const rec = parts + (i * CALIBATT_GROUPS + (size_t)x) * CALIBATT_PART_WORDS;
        if (i >= list[x].size()) {
          std::fill(rec, rec + CALIBATT_PART_WORDS, -1);
          continue;
        }
        const Part &p = all[(size_t)list[x][i]];
        const int32_t fan = pattern->fan_ptr[p.item];
        const int32_t words[CALIBATT_PART_WORDS] = {
            p.id, p.first, p.count, row_ptr[p.id] + p.first,
            iv_ptr ? iv_ptr[p.id] : 0, iv_ptr ? iv_ptr[p.id + 1] - 1 : 0, fan, pattern->fan_ptr[p.item + 1] - fan,
            p.part | p.n_parts << 16, p.b, p.slot, p.row};
        std::copy(words, words + CALIBATT_PART_WORDS, rec);
      }
  } catch (const std::bad_alloc &) {
    return CALIBATT_ERR_NOMEM;
  }
  return CALIBATT_OK;
}

extern "C" int64_t calibatt_split_workspace_bytes(const calibatt_split *split, int block_q, int D) {
  return split ? (int64_t)split->n_slots * calibatt_part_bytes(block_q, D) : 0;
}
