// The work items of the tile GEMM's grid, as every workgroup of every possible grid meets them: each product is handed
// out once, and an id of the padding still names a tile that exists, because the kernel forms an item's addresses and
// descriptor ranges before it looks whether the item is a real one.
// Exit code 0 = every expectation held.
#include <stdio.h>
#include <vector>

#include "flurka_fast.h"
#include "flurka_gemm_tile.h"

using namespace flurka;

template <bool SHARE_A>
static int check(int tilesM, int tilesN, int splits, int item_lo_groups) {
    GemmParams g{};
    g.tilesM = tilesM; g.tilesN = tilesN; g.splits = splits;
    const int count = tile_item_count<SHARE_A>(g), lo = 8 * item_lo_groups;
    if (lo >= count) return 0;
    int bad = 0;
    for (int blocks : {8, 16, 64, 256, 512, count}) {
        std::vector<int> seen((size_t)2 * splits * tilesM * tilesN, 0);
        for (int block = 0; block < blocks && bad == 0; ++block) {
            bool real = true;
            for (int id = lo + block; real; id += blocks) {
                const TileItem it = tile_item<SHARE_A>(g, id, count);
                real = it.valid;
                if (it.tm < 0 || it.tm >= tilesM || it.tn < 0 || it.tn >= tilesN || it.which < 0 || it.which > 1 ||
                    it.split < 0 || it.split >= splits) {
                    printf("share %d, %d x %d tiles, %d splits, %d workgroups: id %d names tile (%d, %d) of operand %d, split %d\n",
                           (int)SHARE_A, tilesM, tilesN, splits, blocks, id, it.tm, it.tn, it.which, it.split);
                    ++bad;
                    break;
                }
                if (real) ++seen[(((size_t)it.which * splits + it.split) * tilesN + it.tn) * tilesM + it.tm];
            }
        }
        if (lo == 0)
            for (int x : seen)
                if (x != 1) { printf("an item handed out %d times\n", x); ++bad; break; }
        if (bad) return bad;
    }
    return bad;
}

int main() {
    int bad = 0;
    for (int tilesM : {1, 2, 3, 7, 19})
        for (int tilesN : {1, 2, 5, 18, 37, 130})
            for (int splits : {1, 2, 3, 5, 8, 16})
                for (int lo : {0, 1, 5}) bad += check<false>(tilesM, tilesN, splits, lo) + check<true>(tilesM, tilesN, splits, lo);
    printf(bad ? "%d expectation(s) failed\n" : "all expectations held\n", bad);
    return bad ? 1 : 0;
}
