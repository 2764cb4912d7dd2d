// The workgroup order of every launch of the planner (built by
// tests/test_tile_order.py with g++; no GPU, no HIP call), over the shapes on
// its command line ("rows cols grid_rows grid_cols layers", repeated) and both
// element sizes: each unit's tiles appear exactly once (upper ones of the
// symmetric products; of the pack, every 64 x 64 tile), empty entries name no
// problem, and no XCD's share of a launch of several rounds is more than the
// mean by more than one tile and the rounding of one unit per XCD.  Prints "ok"
// at the end.
#include <cstdio>
#include <cstdlib>
#include <map>
#include <set>
#include <string>
#include <tuple>
#include <vector>

#include "plan.h"

using namespace muonbp;

int main(int argc, char** argv) {
  std::vector<MatrixShape> mats;
  for (int i = 1; i + 4 < argc; i += 5)
    for (int l = 0; l < std::atoi(argv[i + 4]); ++l)
      mats.push_back(MatrixShape{std::atoll(argv[i]), std::atoll(argv[i + 1]), std::atoi(argv[i + 2]),
                                 std::atoi(argv[i + 3])});
  for (int es : {2, 4})
    for (int lean = 0; lean < 2; ++lean) {
      Layout lay;
      bool shape_err = false;
      const std::string msg =
          build_layout(mats.data(), int32_t(mats.size()), es, 5, 1, 0, 0, 0, &lay, &shape_err, 0, false, lean != 0);
      if (!msg.empty()) return std::printf("refused: %s\n", msg.c_str()), 1;
      for (const Plan& plan : lay.plan) {
        std::map<std::tuple<int, int64_t, int64_t>, int> packed;
        for (const TileRef& t : plan.pack_tiles) ++packed[{t.prob, tile_row(t.ij), tile_col(t.ij)}];
        size_t pack_want = 0;
        for (size_t pi = 0; pi < plan.probs.size(); ++pi) {
          const Problem& p = plan.probs[pi];
          if (p.in_place) continue;
          for (int64_t i = 0; i < (p.rows + kPackTile - 1) / kPackTile; ++i)
            for (int64_t j = 0; j < (p.cols + kPackTile - 1) / kPackTile; ++j, ++pack_want)
              if (packed[{int(pi), i, j}] != 1) return std::printf("pack tile missing or twice\n"), 1;
        }
        if (plan.pack_tiles.size() != pack_want) return std::printf("pack tiles\n"), 1;
        for (const GemmPhase& ph : plan.phases) {
          const int64_t bm = kGemmTileRows[ph.variant], bn = kGemmTileCols[ph.variant];
          std::map<std::tuple<int, int64_t, int64_t>, int> seen;  // descriptor, row and column as the kernels decode them
          std::set<int> descs;
          int64_t load[kNumXCDs] = {}, total = 0, tiles = 0, longest = 0, unit = 0;
          for (size_t w = 0; w < ph.tiles.size(); ++w) {
            const TileRef& t = ph.tiles[w];
            if (t.prob < 0) {
              if (lean) return std::printf("empty entry in a lean plan\n"), 1;
              continue;
            }
            ++seen[{t.prob, tile_row(t.ij), tile_col(t.ij)}];
            descs.insert(t.prob);
            const Problem& p = plan.probs[size_t(t.prob / lay.desc_per_problem)];
            const int64_t cost = ((ph.kind == kGram ? p.L : p.S) + 31) / 32 + 14;
            load[w % kNumXCDs] += cost;
            total += cost;
            ++tiles;
            longest = std::max(longest, cost);
          }
          int64_t want = 0;
          for (int dsc : descs) {
            const Problem& p = plan.probs[size_t(dsc / lay.desc_per_problem)];
            const int64_t tm = (p.S + bm - 1) / bm, tn = ((ph.kind == kApply ? p.L : p.S) + bn - 1) / bn;
            int64_t n = 0;
            for (int64_t i = 0; i < tm; ++i)
              for (int64_t j = ph.kind == kApply ? 0 : i; j < tn; ++j, ++n)
                if (seen[{dsc, i, j}] != ph.nsplit) return std::printf("tile missing or twice\n"), 1;
            want += n;
            unit = std::max(unit, longest * n);
          }
          if (tiles != want * ph.nsplit) return std::printf("%lld tiles, %lld wanted\n", (long long)tiles, (long long)want), 1;
          if (!lean && ph.nsplit == 1 && tiles > kNumCUs)
            for (int64_t l : load)
              if (l > total / kNumXCDs + unit / kNumXCDs + longest + kNumXCDs)
                return std::printf("XCD load %lld of mean %lld\n", (long long)l, (long long)(total / kNumXCDs)), 1;
        }
      }
    }
  std::printf("ok\n");
  return 0;
}
