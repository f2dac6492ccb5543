// Host build of the integer arithmetic that the decode kernel's workgroups share (see test_decode_schedule.py and test_decode_handoff.py).
#include <algorithm>
#include <map>
#include <set>
#include <vector>

#include "kvlinc_handoff.h"
#include "kvlinc_schedule.h"

using namespace kvlinc;

namespace {

// Every order in which the workgroups of a (sequence, kv head) can reach its counter.  A workgroup is run again from its start for each of
// its accesses: the results of the earlier ones are given back to it, the next access is the one that is taken now.
struct Pending { bool is_add; int n; };
struct Replay {
  const std::vector<int>& seen;
  size_t at = 0;
  int adds = 0, looks = 0;
  int take(bool is_add, int n) {
    (is_add ? adds : looks)++;
    if (at < seen.size()) return seen[at++];
    throw Pending{is_add, n};
  }
  int add(int n) { return take(true, n); }
  int look() { return take(false, 0); }
  void pause() {}
};

struct Launch {
  int n_splits, n_parts;
  bool awaited;
  int looks;
};

struct Workgroup {
  bool stream;
  std::vector<int> seen;
  bool operator<(const Workgroup& o) const { return stream != o.stream ? stream < o.stream : seen < o.seen; }
};

// What the kernel does at the counter.  Returns whether the workgroup merges.
bool run(const Launch& l, bool stream, Replay& counter) {
  if (!stream) return correction_merges(counter.add(kCorrArrival), l.n_splits, l.n_parts, l.awaited);
  bool keep = false;
  if (l.n_splits == 1) {
    if (l.n_parts == 0 || parts_arrived(counter.look()) == l.n_parts) return true;
    keep = l.awaited;
    if (keep && await_parts(counter, l.n_parts, l.looks)) return true;
  }
  return stream_arrives(counter, l.n_splits, l.n_parts, l.awaited, keep, l.looks);
}

struct Search {
  Launch l;
  std::set<std::pair<int, std::vector<Workgroup>>> known;
  int orders_end = 0, most_looks = 0, correction_merged = 0;
  bool ok = true;

  void visit(int count, std::vector<Workgroup> all) {
    std::sort(all.begin(), all.end());
    if (!ok || !known.insert({count, all}).second) return;
    std::vector<std::pair<size_t, Pending>> next;
    int merges = 0;
    for (size_t i = 0; i < all.size(); ++i) {
      Replay c{all[i].seen};
      try {
        if (run(l, all[i].stream, c)) {
          ++merges;
          correction_merged |= !all[i].stream;
        }
      } catch (Pending p) {
        next.push_back({i, p});
      }
      most_looks = std::max(most_looks, c.looks);
    }
    if (merges > 0) {  // by one workgroup, after everybody's last access: it clears the counter
      const bool all_parts = parts_arrived(count) == l.n_parts;
      ok = merges == 1 && next.empty() && all_parts;
      ++orders_end;
      return;
    }
    if (next.empty()) ok = false;  // nobody merges
    for (const auto& [i, p] : next) {
      std::vector<Workgroup> after = all;
      after[i].seen.push_back(count);
      visit(p.is_add ? count + p.n : count, after);
    }
  }
};

}  // namespace

extern "C" {

int rounds_left_out(int count, int n_splits, int bits) { return window_rounds(count, n_splits, bits); }

int group_of_round(int n_splits, int split, int wave, int skip, int round) { return GroupOrder(n_splits, split, wave, skip).group(round); }

// Whether every order ends in exactly one merge; the most looks of a workgroup, and whether a correction workgroup merges in any order.
int every_order_merges_once(int n_splits, int n_parts, int awaited, int looks, int* most_looks, int* correction_merged) {
  Search s{{n_splits, n_parts, awaited != 0, looks}};
  std::vector<Workgroup> all;
  for (int i = 0; i < n_splits; ++i) all.push_back({true, {}});
  for (int i = 0; i < n_parts; ++i) all.push_back({false, {}});
  s.visit(0, all);
  *most_looks = s.most_looks;
  *correction_merged = s.correction_merged;
  return s.ok && s.orders_end > 0;
}

}  // extern "C"
