// Which kernels a plan runs: reads lines "M K Ncols bits w_bits L prime ... prime" from standard input and prints a line for each.
//   shortk
//   resident D S NT epilogue nt|cached k-steps-beyond-whole-register-sets one-turn|turns
//   gemm  and for each launch group (limb pairs first): " | waves D S epilogue pair|single odd|even alone|shared", then " launches n", " split kind",
//         " stores nt|cached", " scratch digit-plane-bytes"
// C and A are taken to start on 128-byte lines.
#include <stdio.h>
#include <vector>

#include "pcmm_host.hpp"

using namespace pcmm_host;

int main()
{
    long M, K, N;
    int bits, w_bits, L;
    while (scanf("%ld %ld %ld %d %d %d", &M, &K, &N, &bits, &w_bits, &L) == 6) {
        std::vector<uint64_t> q(L);
        for (uint64_t &x : q) {
            unsigned long v;
            if (scanf("%lu", &v) != 1) return 1;
            x = v;
        }
        Geometry g;
        if (plan_geometry(M, K, N, L, q.data(), bits, w_bits, 0, &g) != PCMM_OK) {
            printf("refused\n");
            continue;
        }
        static const char *const epis[] = {"f64", "?", "int", "g4", "g4p", "pair"};
        if (g.nkb == 2 && g.D <= 7 && g.epi != epi::EPI_INT) {
            printf("shortk\n");
        } else if (g.resident.NT) {
            const ResidentTile &t = g.resident;
            const int64_t ks = resident_ksteps(K), groups = (M + 16 * t.MT - 1) / (16 * t.MT);
            const int sets = resident_ahead(g.D, g.S, t.NT, t.MT) + 1;
            printf("resident %d %d %d %s %s %d %s\n", g.D, g.S, t.NT, epis[g.epi], resident_nt_stores(K, N, 0, g.D, g.S) ? "nt" : "cached",
                   (int)(ks % sets), (t.groups_per_part < groups ? t.groups_per_part : groups) > t.waves ? "turns" : "one-turn");
        } else {
            printf("gemm");
            const int64_t launches = (g.ksteps + g.nkb_launch - 1) / g.nkb_launch, last = g.ksteps - (launches - 1) * g.nkb_launch;
            for (int pair = 1; pair >= 0; --pair) {
                const int64_t limbs = pair ? g.pairs : L - 2 * g.pairs;
                if (!limbs) continue;
                printf(" | %d %d %d %s %s %s %s", g.WM, pair ? kPairDigits : g.D, g.S, epis[pair ? epi::EPI_F64_PAIR : g.epi], pair ? "pair" : "single",
                       last % 2 ? "odd" : "even", limbs * g.mtiles * (pair ? g.pair_ntiles : g.ntiles) <= 2 * 256 ? "alone" : "shared");
            }
            static const char *const splits[] = {"none", "stores", "both"};
            printf(" | launches %ld | split %s | stores %s | scratch %ld\n", (long)launches, splits[split_nt(L, K, N, 0)],
                   gemm_nt_stores(M, K, g.S, N, 0) ? "nt" : "cached", (long)g.ad_bytes);
        }
    }
    return 0;
}
