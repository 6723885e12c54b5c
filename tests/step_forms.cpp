// Decisions of the step-form rule: reads lines "fp64 cus n beads:wave_tasks:queue_only ..."
// and prints the workgroups per CU and each group's form.  Test helper only; compiled
// by the test into a temporary directory.
#include <cstdio>
#include <vector>

#include "ssp_schedule.h"

int main()
{
    int fp64, cus, n;
    while (std::scanf("%d %d %d", &fp64, &cus, &n) == 3) {
        std::vector<ssp::StepGroup> groups;
        for (int i = 0; i < n; ++i) {
            int beads, queue_only;
            long tasks;
            if (std::scanf("%d:%ld:%d", &beads, &tasks, &queue_only) != 3) return 1;
            groups.push_back({beads, tasks, queue_only != 0, false});
        }
        const int per_cu = ssp::choose_step_forms(fp64 != 0, cus, groups.data(), (int)groups.size());
        std::printf("%d", per_cu);
        for (const ssp::StepGroup& g : groups) std::printf(" %d", (int)g.low_latency);
        std::printf("\n");
    }
    return 0;
}
