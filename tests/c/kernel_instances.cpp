// Asks the library (host side only) for the kernel of every record tile, window depth, table
// place and vote size that the launch plans can ask for: each must exist, the list kernel only
// with its list in the LDS.  Prints the number of distinct kernels met, which is the number
// the library holds if no instance is out of every plan's reach.
#include <cstdio>
#include <cstdlib>
#include <set>

#include "kernels.hpp"
#include "tiles.hpp"

using namespace dtree;

namespace {

std::set<const void *> met;

void need(const void *fn, const char *what, int a, int b, int c, int d) {
    if (!fn) {
        std::printf("no kernel: %s %d %d %d %d\n", what, a, b, c, d);
        std::exit(1);
    }
    met.insert(fn);
}

void trees() {
    for (int xt = 0; xt < kElemTypes; ++xt)
        for (int algo : {kAlgoData, kAlgoSpec, kAlgoPath, kAlgoList})
            for (int f = 1; f <= kMaxRowStride; ++f)
                for (int mode = 0; mode < kLoadModes; ++mode) {
                    const int es = elem_bytes(xt);
                    if (mode == kLoadExact && !exact_rows(f, es)) continue;
                    if (mode == kLoadBytes && es == 4) continue;
                    for (int depth = 1; depth <= 6; ++depth)
                        for (bool lds : {false, true}) {
                            if (mode == kLoadFlat && !flat_rows(algo, xt, f, depth)) continue;
                            const TileShape s = tile_shape(algo, xt, f, mode, depth);
                            const void *fn = kernel_for(algo, xt, s, lds, depth);
                            if ((algo == kAlgoPath && xt != kXF32) || (algo == kAlgoList && !lds)) {
                                if (fn) {
                                    std::printf("kernel that must not be: %d %d %d\n", algo, xt, f);
                                    std::exit(1);
                                }
                                continue;
                            }
                            need(fn, "tree", algo, xt, f, mode);
                        }
                }
}

void forests() {
    for (int algo : {kAlgoData, kAlgoSpec})
        for (int f = 1; f <= kMaxRowStride; ++f)
            for (int mode = 0; mode < kForestLoadModes; ++mode) {
                if (mode == kLoadExact && (!exact_rows(f, 4) || f > 32)) continue;
                if (mode == kLoadFlat &&
                    (f % 4 == 0 || (algo == kAlgoSpec && f <= 4 * kMaxForestPitchVecs)))
                    continue;
                for (int split : {0, 1})
                    for (int votes : {2, 4, 16})
                        for (bool lds : {false, true})
                            for (int kind = 0; kind < (algo == kAlgoData ? 4 : 2); ++kind) {
                                if (mode == kLoadExact && split > 0) continue;
                                const bool in_place_rows = mode == kLoadExact && !lds;
                                ForestShape s;
                                s.algo = algo;
                                s.vote_words = votes;
                                s.tables_in_lds = lds;
                                s.split = split;
                                s.exit_mode = algo == kAlgoData ? kind : int(kExitInt32);
                                s.depth = algo == kAlgoData ? 8 : kind == 0 ? 2 : 4;
                                s.tile = forest_tile_shape(algo, f, in_place_rows ? int(kLoadRows) : mode,
                                                           split == 0 && lds);
                                need(forest_kernel_for(s), "forest", algo, f, mode, split);
                            }
            }
}

}  // namespace

int main() {
    trees();
    forests();
    std::printf("ok %zu\n", met.size());
    return 0;
}
