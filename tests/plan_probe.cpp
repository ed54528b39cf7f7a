// Forward plans (paper_2404_01817_amd/csrc/launch.h) printed as JSON, without a
// GPU: linked against libneat.so, whose planner is host code.  Standard input,
// one plan per line: "how max_lds n", then n times "P N C I O B side variant
// recurrent aligned".  how: -1 takes every job's variant as it is, 0 resolves
// FWD_AUTO as a batch recorded into a graph does, 1 as one launched in order, 2
// and 3 plan n copies of the (first) job with what the autotuner times for
// FWD_AUTO alone and on a full GPU ("tune": that variant; no launches for -1).
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "launch.h"
#include "neat.h"
#include "tune.h"

int main() {
    int how, n;
    unsigned long long lds;
    while (std::scanf("%d %llu %d", &how, &lds, &n) == 3) {
        std::vector<neat::FwdJob> jobs((size_t)n);
        for (neat::FwdJob &j : jobs) {
            int aligned;
            if (std::scanf("%d %d %d %d %d %d %d %d %d %d", &j.P, &j.N, &j.C, &j.I, &j.O, &j.B,
                           &j.side, &j.variant, &j.recurrent, &aligned) != 10)
                return 2;
            j.inputs = (const float *)(size_t)(aligned ? 4096 : 4100);
            j.gstride = 4 * (((long long)j.B * j.I + 3) / 4);
            j.sweeps = j.recurrent ? 3 : 0;
        }
        int tune = -2;
        if (how >= 2) {
            jobs[0].variant = -1;
            tune = neat::tune_auto(jobs[0], n, how == 3, lds);
            for (neat::FwdJob &j : jobs) j.variant = tune;
        }
        std::vector<neat::FwdKernelLaunch> out;
        char err[256] = "";
        int rc = NEAT_OK;
        if (how == 0 || how == 1)
            rc = neat::forward_plan_auto(jobs, how == 1, lds, out, err, sizeof(err));
        else if (tune != -1)
            rc = neat::forward_plan(jobs.data(), n, neat::FWD_AUTO, lds, out, err, sizeof(err));
        std::printf("{\"rc\": %d, \"tune\": %d, \"launches\": [", rc, tune);
        for (size_t k = 0; k < out.size(); ++k) {
            const neat::FwdKernelLaunch &L = out[k];
            std::printf("%s{\"kind\": \"%s\", \"grid_mode\": %d, \"grid\": %u, \"block\": %u, \"lds\": "
                        "%zu, \"wave_floats\": %d, \"stage_floats\": %d, \"units\": %lld, "
                        "\"items\": [",
                        k ? ", " : "", neat::kind_name(L.kind), L.grid_mode, L.grid, L.block, L.lds,
                        L.args.wave_floats, L.args.stage_floats, L.args.units);
            for (size_t i = 0; i < L.items.size(); ++i) {
                const neat::FwdItem &it = L.items[i];
                std::printf("%s{\"P\": %d, \"N\": %d, \"B\": %d, \"cls\": %d, \"tiles\": %d, \"tpw\": %d, "
                            "\"lvl_sh\": %d, \"lvl_rows\": %d, \"vec4\": %d}",
                            i ? ", " : "", it.P, it.N, it.B, it.cls, it.tiles, it.tpw, it.lvl_sh,
                            it.lvl_rows, it.vec4);
            }
            std::printf("]}");
        }
        std::printf("]}\n");
    }
    return 0;
}
