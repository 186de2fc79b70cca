// Host-only driver for tests/test_small_tiles.py: prints the small-tile variant
// of each product of a list ("bf16" or "fp32", then "rows cols" pairs, on the
// command line), and
// checks the lists that replace the planner's tiles: every tile that holds
// matrix data exactly once (the lower triangle for the symmetric products),
// none past the padded buffers, each XCD segment a partition. Prints what the
// choice costs, too.
#include <algorithm>
#include <chrono>
#include <cstdio>
#include <cstdlib>
#include <set>
#include <string>
#include <tuple>
#include <vector>

#include "plan.h"
using namespace lm;

int main(int argc, char** argv) {
  std::vector<TensorIn> x;
  NsPrecision prec;
  prec.all_fp32 = argc > 1 && std::string(argv[1]) == "fp32";
  for (int i = 2; i + 1 < argc; i += 2) {
    TensorIn t{};
    const uintptr_t base = 0x100000000ull + uintptr_t(i) * 0x1000000000ull;
    t.w = reinterpret_cast<float*>(base);
    t.g = reinterpret_cast<const float*>(base + 0x400000000ull);
    t.m = reinterpret_cast<float*>(base + 0x800000000ull);
    t.rows = atol(argv[i]);
    t.cols = atol(argv[i + 1]);
    x.push_back(t);
  }
  Plan p;
  std::string err;
  if (build_plan(x.data(), int32_t(x.size()), StepKind::kMuon, prec, false, ChipShape(), &p,
                 &err) != Status::kOk)
    return 1;
  int bad = 0;
  for (int pr = 0; pr < 2; ++pr)
    for (int st = 0; st < 3; ++st) {
      const GemmVariant& v = p.variant[pr][st];
      const std::vector<GemmTask>& list = p.fine[pr][st];
      if (pr == (prec.all_fp32 ? 1 : 0)) printf("%d/%d ", v.tile, v.bufs);
      if (v.tile == 0) {
        bad += !list.empty();
        continue;
      }
      const XcdSplit& sp = p.fine_split[pr][st];
      int32_t pos = 0;
      for (int k = 0; k < p.chip.xcds; ++k) {
        bad += sp.start[k] != pos || sp.count[k] > sp.max_count;
        pos += sp.count[k];
      }
      bad += pos != int32_t(list.size());
      std::set<std::tuple<int, int, int>> seen;
      for (const GemmTask& t : list) {
        const MuonMat& m = p.mats[size_t(t.mat)];
        bad += m.fp32 != pr || (st < 2 && t.tn > t.tm) || (t.tm + 1) * v.tile > m.s_pad ||
               (t.tn + 1) * v.tile > (st < 2 ? m.s_pad : m.l_pad);
        bad += !seen.insert(std::make_tuple(int(t.mat), int(t.tm), int(t.tn))).second;
      }
      size_t want = 0;
      for (const MuonMat& m : p.mats) {
        if (m.fp32 != pr) continue;
        const size_t ts = size_t((m.s + v.tile - 1) / v.tile), tl = size_t((m.l + v.tile - 1) / v.tile);
        want += st < 2 ? ts * (ts + 1) / 2 : ts * tl;
      }
      bad += want != list.size();
    }
  // least time of a plan with its small tiles over one without (a size query)
  double us[2] = {1e9, 1e9};
  for (int r = 0; r < 40; ++r) {
    const auto t0 = std::chrono::steady_clock::now();
    Plan q;
    if (build_plan(x.data(), int32_t(x.size()), StepKind::kMuon, prec, false, ChipShape(),
                   &q, &err, r & 1) != Status::kOk)
      return 1;
    const auto t1 = std::chrono::steady_clock::now();
    us[r & 1] = std::min(us[r & 1], std::chrono::duration<double, std::micro>(t1 - t0).count());
    bad += q.ws_bytes != p.ws_bytes || (!(r & 1) && !q.fine[0][0].empty());
  }
  printf("bad %d cost %.2f\n", bad, us[1] / us[0]);
  return bad != 0;
}
