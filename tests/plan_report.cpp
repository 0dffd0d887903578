// Host program around the planner for test_plan_groups.py.
//   runs         checks every cut of a run of bins into work items
//   plan [file]  reads products from stdin, prints each one's plan as a line of
//                JSON; file: remembered tuning choices
#include <stdio.h>
#include <string.h>

#include <vector>

#include "pm_plan.hpp"

using namespace pm;

// Work items of a run tile it, none of them wider than the LDS cells.
static int runs() {
    constexpr u32 KMAX = 2048;
    std::vector<u32> widest((KMAX + 1) * (KMAX + 1));
    for (u32 K = 1; K <= KMAX; K++)
        for (u32 n = 1; n <= K; n++) {
            u32 w = 0;
            for (u32 e = 0; e < n; e++) w = std::max(w, gp_run_bin(K, n, e + 1) - gp_run_bin(K, n, e));
            if (gp_run_bin(K, n, 0) != 0 || gp_run_bin(K, n, n) != K) return printf("%u bins in %u do not tile\n", K, n), 1;
            widest[K * (KMAX + 1) + n] = w;
        }
    for (u32 K = 1; K <= KMAX; K++)
        for (u32 S = 1; S <= (u32)GP_CELLS; S++)
            for (u32 asked : {0u, 1u, 2u, 3u, 5u, 8u, K / 2 + 1, K, K + 7}) {
                const u32 n = gp_run_items(K, S, asked);
                if (n < 1 || n > K || n < std::min(asked, K) || (u64)widest[K * (KMAX + 1) + n] * S > (u64)GP_CELLS)
                    return printf("K %u S %u asked %u: %u work items\n", K, S, asked, n), 1;
            }
    return 0;
}

// A product: nvars bits ring na nb tile_cfg combine tiny, then per variable
// f's and g's minima, maxima and group counts as fmin fmax gmin gmax fcnt gcnt.
static int plan() {
    int nv, bits, ring;
    while (scanf("%d %d %d", &nv, &bits, &ring) == 3) {
        long long na, nb;
        Tuning t;
        int tiny;
        if (scanf("%lld %lld %d %d %d", &na, &nb, &t.tile_cfg, &t.combine, &tiny) != 5) return 2;
        t.tiny = tiny != 0;
        std::vector<uint64_t> st(4 * nv);
        for (int v = 0; v < nv; v++) {
            unsigned long long x[6];
            for (auto &y : x)
                if (scanf("%llu", &y) != 1) return 2;
            st[v] = x[0] | x[4] << 32;
            st[nv + v] = x[1];
            st[2 * nv + v] = x[2] | x[5] << 32;
            st[3 * nv + v] = x[3];
        }
        const uint32_t flags[2] = {0, 0};
        Plan P;
        const int rc = plan_build(nv, bits, ring, {SegInput{nullptr, nullptr, nullptr, nullptr, na, nb}}, st.data(), flags, t, P);
        if (rc) {
            printf("{\"rc\": %d}\n", rc);
            continue;
        }
        const DevSeg &s = P.segs[0];
        const GrpSeg g = s.mode == SEG_GRP || s.mode == SEG_GRPD ? s.gp : GrpSeg{};
        printf("{\"rc\": 0, \"mode\": %d, \"S\": %u, \"K\": %u, \"nbins\": %u, \"T\": %u, \"csh\": %u, \"span_bins\": %u, \"heavy\": %u, "
               "\"rows\": %u, \"d\": %u, \"least\": %u, \"ibound\": %lld, \"cells\": %d, \"total\": %zu, \"report\": %zu}\n",
               s.mode, g.S, g.K, g.nbins, g.T, g.csh, g.span_bins, g.heavy, g.rows, g.d, g.K ? gp_run_items(g.K, g.S, 0) : 0u, (long long)P.gp_ibound, GP_CELLS, P.total,
               P.report);
    }
    return 0;
}

int main(int argc, char **argv) {
    if (argc == 2 && !strcmp(argv[1], "runs")) return runs();
    if (argc == 3 && tune_load(argv[2]) != 0) return 2;
    if (argc >= 2 && !strcmp(argv[1], "plan")) return plan();
    return 2;
}
