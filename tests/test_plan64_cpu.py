"""The planner of the FP64 Cholesky/HERK kernel (plan64.hpp, host code) against its plain form, which lists, sorts and
schedules every item of every split: the same choice at a fraction of the time. And its limit on the items of a launch, for
every launch of a plan and not only the one that the split is chosen for. Built with the host compiler.
"""
import os
import random
import re
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1003_0524_amd", "csrc")

DRIVER = r"""
#include "plan64.hpp"
#include <chrono>
#include <cstdio>
#include <functional>
#include <queue>
using namespace exc;
static Shape64 shape(int nbt, int ng) {                    // Herk64Cfg's constants
  const int nwc = nbt * ng > 12 || nbt > 8 ? 2 : 1, nw = 4 * nwc, nct = (nbt * ng + nwc - 1) / nwc * nwc;
  const int npt = nbt * (nbt + 1) / 2;
  return {nbt, ng, nw, nbt <= 3 ? npt : (npt + nw - 1) / nw, nct / nwc};
}
template <class F>
static void items(const System64& c, const Shape64& k, int passes, int groups, int nd, F&& f) {
  const int npass = (c.n_occ + k.ng - 1) / k.ng, per = passes ? passes : npass;
  for (int g = 0; g < npass; g += per)
    runs64(c, k, groups, nd, [&](int, int, double x) { f(x * std::min(per, npass - g)); });
}
static Split64 plain(const System64& c, const std::vector<Shape64>& sh, int nbt, const std::vector<int>& nd, size_t max) {
  Split64 best;
  double best_t = 1e300;
  if (!max) max = std::max(nd.size(), ((size_t)2 << 30) / c.slot_bytes);
  std::vector<double> cs;
  for (int i = 0; i < (int)sh.size(); ++i) {
    const Shape64& k = sh[i];
    if (k.nbt != nbt) continue;
    for (int passes : {0, 4, 2, 1}) {
      if (passes >= (c.n_occ + k.ng - 1) / k.ng) continue;
      for (int groups : {1, 2, 3, 4, 6, 0}) {
        cs.clear();
        for (int n : nd) items(c, k, passes, groups, n, [&](double x) { cs.push_back(x + 60.0); });
        if (cs.size() > max && !(passes == 0 && groups == 1)) continue;
        double sum = 0.0, mx = 0.0, t;
        for (double x : cs) { sum += x; mx = std::max(mx, x); }
        if (cs.size() > (size_t)64 * c.n_cu) t = sum / c.n_cu + 0.5 * mx;
        else {
          std::sort(cs.begin(), cs.end(), std::greater<double>());
          std::priority_queue<double, std::vector<double>, std::greater<double>> h;
          t = 0.0;
          for (double x : cs) {
            double at = 0.0;
            if ((int)h.size() == c.n_cu) { at = h.top(); h.pop(); }
            h.push(at + x);
            t = std::max(t, at + x);
          }
          if (cs.size() > (size_t)c.n_cu * (k.nw == 4 ? 2 : 1)) t += 0.5 * mx;
        }
        t += (double)cs.size() * c.slot_bytes * 2 / 5e12 * 2.4e9 / 64;
        if (t < 0.98 * best_t) { best_t = t; best = Split64{i, passes, groups}; }
      }
    }
  }
  return best;
}
// each line: nbt n_occ n_s n_chunk max_slots total_slots pairs nd... launches (pairs nd...)...: the split is chosen for the first ones,
// the launches after them keep to the limit too; out: the two choices and the items of each (the plain form sees the first
// launch only), microseconds of each, items of the further launches under the plain choice and under the planner's
int main() {
  std::vector<Shape64> sh;
  for (auto& x : (int[][2]){INSTANCES}) sh.push_back(shape(x[0], x[1]));
  int nbt, n_occ, n_s, n_chunk, pairs;
  size_t max, total;
  while (scanf("%d %d %d %d %zu %zu %d", &nbt, &n_occ, &n_s, &n_chunk, &max, &total, &pairs) == 7) {
    std::vector<int> nd(pairs);
    for (int& x : nd) if (scanf("%d", &x) != 1) return 1;
    std::vector<std::vector<int>> all(1, nd);
    int more;
    if (scanf("%d", &more) != 1) return 1;
    for (int l = 0; l < more; ++l) {
      int n;
      if (scanf("%d", &n) != 1) return 1;
      all.push_back(std::vector<int>(n));
      for (int& x : all.back()) if (scanf("%d", &x) != 1) return 1;
    }
    const System64 c{n_occ, n_s, n_chunk, 256, (size_t)nbt * (nbt + 1) / 2 * 2048};
    const auto a = std::chrono::steady_clock::now();
    const Split64 p = plain(c, sh, nbt, nd, max);
    const auto b = std::chrono::steady_clock::now();
    const Split64 q = pick_split64(c, sh, nbt, all, 0, max, total);
    const auto e = std::chrono::steady_clock::now();
    for (const Split64& s : {p, q}) {
      size_t n = 0;
      for (int x : nd) items(c, sh[s.inst], s.passes, s.groups, x, [&](double) { ++n; });
      printf("%d %d %d %zu ", sh[s.inst].ng, s.passes, s.groups, n);
    }
    printf("%.1f %.1f", std::chrono::duration<double, std::micro>(b - a).count(),
           std::chrono::duration<double, std::micro>(e - b).count());
    for (const Split64& s : {p, q})
      for (int l = 1; l <= more; ++l) {
        size_t n = 0;
        for (int x : all[l]) items(c, sh[s.inst], s.passes, s.groups, x, [&](double) { ++n; });
        printf(" %zu", n);
      }
    printf("\n");
  }
}
"""


@pytest.fixture(scope="module")
def planner(tmp_path_factory):
    cxx = shutil.which("g++")
    if not cxx:
        pytest.skip("no host compiler")
    d = tmp_path_factory.mktemp("plan64")
    with open(os.path.join(CSRC, "configs_herk64.hip")) as f:
        inst = re.findall(r"HCFG\((\d+), (\d+)\)", f.read())
    assert len(inst) == 28
    src = d / "plan.cpp"
    src.write_text(DRIVER.replace("INSTANCES", ", ".join("{%s, %s}" % x for x in inst)))
    subprocess.run([cxx, "-O2", "-std=c++17", "-I", CSRC, str(src), "-o", str(d / "plan")], check=True)

    def run(cases):
        def line(c):
            more = c[6] if len(c) > 6 else []
            return [*c[:5], c[7] if len(c) > 7 else 0, len(c[5]), *c[5], len(more), *(x for l in more for x in [len(l), *l])]

        text = "\n".join(" ".join(map(str, line(c))) for c in cases)
        out = subprocess.run([str(d / "plan")], input=text, capture_output=True, text=True, check=True, timeout=300)
        rows = [r.split() for r in out.stdout.splitlines()]
        assert len(rows) == len(cases)
        return [([int(x) for x in r[:4]], [int(x) for x in r[4:8]], float(r[8]), float(r[9]), [int(x) for x in r[10:]])
                for r in rows]

    return run


def _nd(rng, n, lo, hi):
    return [rng.randint(lo, hi) for _ in range(n)]


def _random_cases():
    rng = random.Random(5)
    out = []
    for _ in range(150):
        n_s = rng.choice([0, rng.randint(1, 500)])
        n_chunk = (n_s + 14) // 15 if n_s and rng.random() < 0.7 else 0
        lo = rng.randint(1, 600)
        nd = _nd(rng, rng.randint(1, rng.choice([40, 400])), lo, lo + rng.randint(0, 500))
        out.append((rng.randint(1, 16), rng.randint(1, 30), n_s, n_chunk, rng.choice([0, 0, len(nd) + rng.randint(0, 3000)]), nd))
    return out


def test_same_choice_as_the_plain_form(planner):
    for case, (p, q, *_) in zip(cases := _random_cases(), planner(cases)):
        assert p == q, (case, p, q)


def test_a_fraction_of_its_time(planner):
    """Context creation waits for it: the plain form takes 7-30 ms of these on this kind of host."""
    rng = random.Random(1)
    cases = [(3, 4, 250, 16, 0, [310] * 512), (8, 18, 455, 29, 0, _nd(rng, 288, 372, 944)),
             (1, 4, 16, 1, 0, [48] * 4096), (2, 8, 100, 7, 0, _nd(rng, 1000, 100, 300)),
             (13, 20, 1200, 75, 0, _nd(rng, 216, 802, 1400))]
    rows = planner(cases)
    assert all(r[0] == r[1] for r in rows)
    old, new = sum(r[2] for r in rows), sum(r[3] for r in rows)
    print(f"[plan64] plain {old:.0f} us, pick_split64 {new:.0f} us")
    assert new < old / 3, (old, new)


def test_every_launch_keeps_to_the_limit(planner):
    """Two k of a subset each: fewer but larger pairs in the second one, whose items follow the split chosen for the first."""
    rng = random.Random(9)
    cases = [(16, 3, 0, 0, 240, [640] * 7, [[1739] * 5]), (8, 2, 0, 0, 903, [448] * 34, [[1251] * 29]),
             (5, 2, 0, 0, 2161, [576] * 89, [[1592] * 59, [100] * 80])]
    for _ in range(60):
        n = rng.randint(2, 60)
        lo = 64 * rng.randint(1, 10)
        more = [_nd(rng, rng.randint(1, n), lo, lo + rng.randint(0, 1200)) for _ in range(rng.randint(1, 4))]
        cases.append((rng.randint(1, 16), rng.randint(1, 20), 0, 0, n + rng.randint(0, 2000), [lo] * n, more))
    over = 0
    for case, (p, q, _, _, items) in zip(cases, planner(cases)):
        n = len(case[6])
        assert q[3] <= case[4] and max(items[n:]) <= case[4], (case, q, items)
        over += max(items[:n]) > case[4]
    assert over >= 3                     # (the split of the first launch alone exceeds the limit in the others)


def test_all_launches_keep_to_the_total(planner):
    """One launch per pair: the split of the largest one, for all of them within a total of partial slots."""
    rng = random.Random(11)
    cases = []
    for _ in range(60):
        nd = sorted(_nd(rng, rng.randint(2, 80), 1, 900), reverse=True)
        cases.append((rng.randint(1, 16), rng.randint(1, 20), 0, 0, 0, nd[:1], [[x] for x in nd[1:]],
                      len(nd) + rng.randint(0, 2000)))
    over = 0
    for case, (p, q, _, _, items) in zip(cases, planner(cases)):
        n = len(case[6])
        assert q[3] + sum(items[n:]) <= case[7], (case, q)
        over += p[3] + sum(items[:n]) > case[7]
    assert over >= 10
