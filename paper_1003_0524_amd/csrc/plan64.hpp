// Work items of the FP64 Cholesky/HERK kernel (herk64.hpp) and the choice among their splits: host code only. An item is
// a pair, a run of n'' passes and a run of row parts (part 0 the block-sparse rows, part 1 + j the dense rows
// [64 j, 64 j + 64)); costs are in matrix instructions of one wavefront (64 cycles each).
#pragma once
#include <algorithm>
#include <cstddef>
#include <vector>

namespace exc {

// What the costs need of an instance: band tiles, n'' values a pass, wavefronts, Gram tiles and column tiles of a wavefront.
struct Shape64 { int nbt, ng, nw, npw, ctw; };

// The system, as far as the costs go. n_chunk: chunks of block-sparse rows that the kernel forms itself (0: it reads them).
struct System64 { int n_occ, n_s, n_chunk, n_cu; size_t slot_bytes; };

struct Split64 {
  int inst = -1;                    // index of the instance
  int passes = 1;                   // n'' passes per item (0: all)
  int groups = 1;                   // runs of row parts per pair (0: one item per part)
};

inline double part_cost64(const System64& c, const Shape64& k, int nd, int part) {
  const bool regg = k.nbt <= 3;
  const int npt = k.nbt * (k.nbt + 1) / 2;
  const int gram = regg ? 4 * k.ng * npt : 16 * k.npw * k.ng + 12;      // of 64 rows
  // block-sparse rows: four chunks at a time formed by five steps, or 16 rows at a time read from the workspace
  if (part == 0)
    return c.n_chunk ? (double)((c.n_chunk + 3) / 4) * (10 * k.ctw + gram)
                     : (double)((c.n_s + 15) / 16) * std::max(10, gram / 4);
  const int np = (nd - 64 * (part - 1) + 15) / 16;
  // (a panel shorter than its barrier and loads costs those)
  return (double)np * std::max(12, 8 * k.ctw + 2) + gram + 10;
}

// The runs of row parts of a pair of nd dense rows, through push(part0, part1, cost of one pass).
template <class F>
void runs64(const System64& c, const Shape64& k, int groups, int nd, F&& push) {
  const int nparts = 1 + (nd + 63) / 64, first = c.n_s > 0 ? 0 : 1;
  double left = 0.0;
  for (int i = first; i < nparts; ++i) left += part_cost64(c, k, nd, i);
  int at = first;
  for (int r = groups ? groups : nparts; at < nparts; --r) {
    // the next run: parts until its share of what is left is reached
    const double want = r > 1 ? left / r : 1e300;
    double cs = part_cost64(c, k, nd, at);
    int e = at + 1;
    for (; e < nparts && groups; ++e) {
      const double x = part_cost64(c, k, nd, e);
      if (cs + 0.5 * x > want) break;
      cs += x;
    }
    push(at, e, cs);
    left -= cs;
    at = e;
  }
}

// The split with the smallest estimated time for pairs of nd dense rows in one launch: the longest-first schedule of its
// items (each with a fixed overhead) on the CUs, whose matrix cores two workgroups share, plus half of the longest item
// where there are more items than workgroup slots (costs are estimates, and a long item that starts late is waited for:
// one k of the ZnO-like workload takes 7.6 ms with one item per part of a pair, 6.9 ms with the items of a few
// passes that this picks), plus the traffic of the partial slots. `launches` are the dense rows of the pairs of each launch
// of the plan; the time is that of launch `at`, but every launch keeps to max_slots items (0: 2 GiB of partials), unless it
// has more pairs than that (no split would do), and all launches together to total_slots (0: no limit). The coarsest
// split (one item per pair) always qualifies.
//
// Pairs of the same nd have the same items, and a split whose schedule cannot be shorter than the best so far (work over
// CUs, longest item) needs none: 288 pairs of 144 different nd 11.5 -> 3.1 ms, 4096 small pairs 17 -> 0.3 ms against
// every item listed, sorted and scheduled for every split.
inline Split64 pick_split64(const System64& c, const std::vector<Shape64>& shapes, int nbt,
                            const std::vector<std::vector<int>>& launches, int at, size_t max_slots,
                            size_t total_slots) {
  struct Group { double cost; size_t n; };               // n items of a cost
  static const int kGroups[6] = {1, 2, 3, 4, 6, 0}, kPasses[4] = {0, 4, 2, 1};
  Split64 best;
  double best_t = 1e300;
  const size_t n_cu = (size_t)c.n_cu;
  if (!max_slots) max_slots = ((size_t)2 << 30) / c.slot_bytes;
  std::vector<int> nd(launches[at]);
  std::sort(nd.begin(), nd.end());
  std::vector<int> sizes;                                // every nd
  for (const auto& l : launches) sizes.insert(sizes.end(), l.begin(), l.end());
  std::sort(sizes.begin(), sizes.end());
  sizes.erase(std::unique(sizes.begin(), sizes.end()), sizes.end());
  std::vector<size_t> parts(sizes.back() + 1);           // runs of a pair of nd dense rows under one grouping
  std::vector<Group> runs[6], items;
  size_t most[6], all[6];                                // items in one run of passes: most of a launch, of the plan
  std::vector<double> h;
  for (int i = 0; i < (int)shapes.size(); ++i) {
    const Shape64& k = shapes[i];
    if (k.nbt != nbt) continue;
    for (int g = 0; g < 6; ++g) {
      for (int x : sizes) {
        parts[x] = 0;
        runs64(c, k, kGroups[g], x, [&](int, int, double) { ++parts[x]; });
      }
      most[g] = all[g] = 0;
      for (const auto& l : launches) {
        size_t n = 0;
        for (int x : l) n += parts[x];
        all[g] += n;
        if (l.size() <= max_slots || &l == &launches[at]) most[g] = std::max(most[g], n);
      }
      runs[g].clear();
      for (size_t a = 0, b; a < nd.size(); a = b) {
        b = std::upper_bound(nd.begin() + a, nd.end(), nd[a]) - nd.begin();
        runs64(c, k, kGroups[g], nd[a], [&](int, int, double x) { runs[g].push_back({x, b - a}); });
      }
    }
    const int npass = (c.n_occ + k.ng - 1) / k.ng;
    for (int passes : kPasses) {
      if (passes >= npass) continue;
      const int per = passes ? passes : npass, rest = npass % per;
      for (int g = 0; g < 6; ++g) {
        items.clear();
        for (const Group& r : runs[g]) {
          items.push_back({r.cost * per + 60.0, r.n * (npass / per)});
          if (rest) items.push_back({r.cost * rest + 60.0, r.n});
        }
        size_t n = 0;
        double sum = 0.0, mx = 0.0;
        for (const Group& x : items) {
          n += x.n;
          sum += x.cost * x.n;
          mx = std::max(mx, x.cost);
        }
        const size_t np = (npass + per - 1) / per;
        const bool over = most[g] * np > max_slots || (total_slots && all[g] * np > total_slots);
        if (over && !(passes == 0 && kGroups[g] == 1)) continue;
        const bool many = n > 64 * n_cu;
        const double extra = (many || n > n_cu * (k.nw == 4 ? 2 : 1) ? 0.5 * mx : 0.0) +
                             (double)n * c.slot_bytes * 2 / 5e12 * 2.4e9 / 64;
        double t = many ? sum / n_cu : std::max(sum / n_cu, mx);
        if (t + extra >= 0.98 * best_t) continue;
        if (!many) {                                     // each CU's load in a heap, the smallest at its root
          std::sort(items.begin(), items.end(), [](const Group& x, const Group& y) { return x.cost > y.cost; });
          h.assign(n_cu, 0.0);
          t = 0.0;
          for (const Group& x : items)
            for (size_t u = 0; u < x.n; ++u) {
              const double end = h[0] + x.cost;
              t = std::max(t, end);
              size_t p = 0;
              for (size_t q = 1; q < n_cu; q = 2 * p + 1) {
                if (q + 1 < n_cu && h[q + 1] < h[q]) ++q;
                if (h[q] >= end) break;
                h[p] = h[q];
                p = q;
              }
              h[p] = end;
            }
        }
        t += extra;
        if (t < 0.98 * best_t) {
          best_t = t;
          best = Split64{i, passes, kGroups[g]};
        }
      }
    }
  }
  return best;
}

}  // namespace exc
