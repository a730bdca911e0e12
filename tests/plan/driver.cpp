// Replays the launch plan of the interleaved attention kernels on the host: random small batches, empty prefixes and trees among
// them.  What the merges rely on: every worker from a segment's first to its last has a part of it (one that has none leaves
// no partial, and counts nobody in), and nobody else has.
#include <cstdio>
#include <random>
#include <set>
#include <vector>

#include "tva_plan.h"

using namespace smart::tva;

static int failures;

template <bool kFp8, bool kFinish>
static void replay(const std::vector<int>& lens, const std::vector<int>& sizes, int G, int Hkv, int workgroups, TreeCost tc) {
  const int batch = (int)lens.size();
  struct Segment { int64_t ub, span; };
  std::vector<Segment> segments[kClasses];
  int64_t units[kClasses] = {0, 0, 0}, segs[kClasses] = {0, 0, 0}, workers[kClasses], first_wg[kClasses + 1];
  int base = 0, total = 0;
  for (int n : sizes) total += n;
  for (int b = 0; b < batch; base += sizes[b++]) {
    const SeqInfo si = sequence_info<kFp8>(lens[b], base, base + sizes[b], total, G, 1 << 16);
    const int c = plan_class<kFp8>(si.n * G);
    const LargeSpans ls = large_spans<kFinish>(si, G, tc);
    int64_t ub = units[c];
    for (int g = 0; g < Hkv; ++g)
      for (int r = 0; r < si.rg; ++r) {
        const int64_t span = c < 2 ? segment_units<kFinish>(si, tc) : (r < si.rg - 1 ? ls.span_full : ls.span_last);
        if (kFinish || si.tiles > 0) segments[c].push_back({ub, span});
        ub += span;
      }
    units[c] += sequence_units<kFinish>(si, c, G, Hkv, tc);
    segs[c] += (int64_t)Hkv * si.rg;
    if (ub != units[c]) printf("segments do not add up\n"), ++failures;
  }
  apportion<kFp8, kFinish>(units, segs, tc, workgroups, workers, first_wg);
  bool bad = first_wg[kClasses] > (workgroups > kClasses ? workgroups : kClasses);
  for (int c = 0; c < kClasses; ++c) {
    const int64_t U = units[c], W = workers[c];
    bad = bad || (U > 0 && W < 1);
    for (const Segment& s : segments[c]) {
      int64_t w_first, w_last;
      segment_workers(s.ub, s.span, U, W, w_first, w_last);
      for (int64_t w = 0; w < W; ++w) {
        const int64_t u0 = share_begin(w, U, W), u1 = share_begin(w + 1, U, W);
        const bool part = u0 < u1 && u0 < s.ub + s.span && u1 > s.ub;
        bad = bad || part != (w >= w_first && w <= w_last);
      }
    }
  }
  if (bad && ++failures <= 10) {
    printf("fp8 %d finish %d G %d Hkv %d workgroups %d:", kFp8, kFinish, G, Hkv, workgroups);
    for (int b = 0; b < batch; ++b) printf(" (%d tokens, %d nodes)", lens[b], sizes[b]);
    printf("\n");
  }
}

static void all_forms(const std::vector<int>& lens, const std::vector<int>& sizes, int G, int Hkv, int workgroups) {
  replay<false, false>(lens, sizes, G, Hkv, workgroups, TreeCost{0, 0});
  replay<true, false>(lens, sizes, G, Hkv, workgroups, TreeCost{0, 0});
  for (TreeCost tc : {TreeCost{4, 60}, TreeCost{12, 160}}) replay<false, true>(lens, sizes, G, Hkv, workgroups, tc);
  for (TreeCost tc : {TreeCost{8, 60}, TreeCost{40, 160}}) replay<true, true>(lens, sizes, G, Hkv, workgroups, tc);
}

int main() {
  all_forms({64, 0, 0, 0}, {4, 4, 4, 4}, 4, 4, 256);
  all_forms({40, 0, 0, 0, 0, 0, 0}, {3, 1, 1, 1, 1, 1, 1}, 7, 4, 256);
  std::mt19937 g(1);
  auto pick = [&](int lo, int hi) { return std::uniform_int_distribution<int>(lo, hi)(g); };
  for (int i = 0; i < 6000; ++i) {
    std::vector<int> lens(pick(1, 20)), sizes;
    const int empty = pick(0, 10), longest = 1 << pick(4, 12), largest = 1 << pick(0, 7);
    for (int& len : lens) {
      len = pick(0, 9) < empty ? 0 : pick(1, longest);
      sizes.push_back(pick(0, 12) == 0 ? 0 : pick(1, largest));
    }
    const int workgroups[] = {1, 3, 40, 256, 304};
    all_forms(lens, sizes, pick(1, 8), 1 << pick(0, 3), workgroups[pick(0, 4)]);
  }
  puts(failures ? "failed" : "plan driver ok");
  return failures != 0;
}
