// Prints the plans of the sequence-length GEMMs for a chip of 256 compute units.  One request a line on standard input:
//   proj B H n d k        -> tile rows, tile columns, splits, row tiles, column tiles, steps per split
//   fused B H n d k dm    -> the same for the first product, then for the second
//   grad B H n d k        -> fine (128 x 128 tiles) or not, splits, row tiles, column tiles, workgroups that start with dE, dF
#include <stdio.h>
#include <string.h>

#include "flurka_plan.h"

using namespace flurka;

namespace flurka {
int chip_cus() { return 256; }
bool kernel_facts(const void*, int, int, KernelFacts*) { return false; }
}  // namespace flurka

static void print(const SplitGemmPlan& q) {
    printf("%d %d %d %d %d %d ", q.t.tm, q.t.tn, q.splits, q.tilesM, q.tilesN, q.steps_per_split);
}

int main() {
    char what[16];
    while (scanf("%15s", what) == 1) {
        Problem p{};
        if (scanf("%d %d %d %d %d", &p.B, &p.H, &p.n, &p.d, &p.k) != 5) return 1;
        p.BH = p.B * p.H;
        p.bf16 = 1;
        if (!strcmp(what, "proj")) {
            print(proj_plan(p));
        } else if (!strcmp(what, "fused")) {
            int dm;
            if (scanf("%d", &dm) != 1) return 1;
            const FusedWPlan q = fusedw_plan(p, dm);
            print(q.s1);
            print(q.s2);
        } else {
            const GradEPlan q = grad_e_plan(p);
            printf("%d %d %d %d %d", (int)q.fine, q.splits, q.tilesM, q.tilesN, q.pair.blocks_a);
        }
        printf("\n");
    }
    return 0;
}
