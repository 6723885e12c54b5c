// Which step kernel the mapping groups of a plain launch take: the low-latency form
// (k_step_pair) or the queue (k_step_queue).  Host code.
#pragma once

#include <stdint.h>

namespace ssp {

struct StepGroup {
    int beads;              // per lane, 1 or 2
    int64_t wave_tasks;
    bool queue_only;        // packed wavefronts
    bool low_latency;       // chosen
};

// Wave tasks per CU up to which the low-latency form is the faster one for a group
// alone: in FP32 as many as are resident at once (us per 1000 steps, queue form / this:
// 2048 tasks of 32 lanes 1091 / 1028 at rest and 1243 / 1088 under shear, 2560 tasks
// 1329 / 1670; 1280 tasks of 64 x 2 2432 / 1767, 1536 tasks 2442 / 2978), in FP64 4 and 2
// (1024 tasks of 32 lanes 1494 / 1225, 1536 tasks 2123 / 2433; 512 tasks of 64 x 2 3155 /
// 2189, 768 tasks 3150 / 4193).
inline int low_latency_limit(bool fp64, int beads) { return fp64 ? (beads == 1 ? 4 : 2) : (beads == 1 ? 8 : 5); }

// Chooses for groups that run side by side on `cus` CUs.  Groups beyond their own
// limit take the queue.  The others take the low-latency form when they fit on the
// CUs together; when they don't, workgroups would wait for whole launches of others,
// and groups with two beads per lane, the last to end, take it alone beside the
// others' queues, which fill what they leave (300 steps, us, all low-latency / all
// queues / so: FP32 64:1000 + 128:700 -- wave tasks of chains of 64 and of 128 beads --
// 741 / 742 / 556, 16, 32, 64 and 128:600 804 / 884 / 704, 16:2000 + 128:100 710 / 803 / 529,
// 32:2048 + 64:2048 708 / 585 / 585; FP64 32:400 + 128:400 1065 / 1201 / 740, 32:700 + 64:700
// 847 / 706 / 706).  In FP64 a few one-bead tasks beside nearly full two-bead ones are
// better off with them, since the queue's wavefronts find no registers there
// (32:200 + 128:500 798 / 1197 / 1163).
// Returns the low-latency workgroups per CU when every group takes that form, the
// number that the launches spread evenly (300 steps of FP64 32:300 + 64:300: 590 -> 470
// us), and 1 beside queues, which then fill the rest (FP32 64:600 + 128:1000: 906 without,
// 527).
inline int choose_step_forms(bool fp64, int cus, StepGroup* groups, int n)
{
    double share[3] = {0.0, 0.0, 0.0};  // by beads per lane: parts of the CUs that the groups take
    auto part = [&](const StepGroup& g) {
        return (double)g.wave_tasks / ((double)cus * low_latency_limit(fp64, g.beads));
    };
    auto can = [&](const StepGroup& g) { return !g.queue_only && part(g) <= 1.0; };
    for (int i = 0; i < n; ++i)
        if (can(groups[i])) share[groups[i].beads] += part(groups[i]);
    const bool together = share[1] + share[2] <= 1.0 || (fp64 && share[1] <= 0.25 && share[2] <= 1.0);
    bool all = true;
    int64_t workgroups = 0;
    for (int i = 0; i < n; ++i) {
        StepGroup& g = groups[i];
        g.low_latency = can(g) && (together || (g.beads == 2 && share[2] <= 1.0));
        all = all && g.low_latency;
        workgroups += g.wave_tasks;
    }
    return all ? (int)((workgroups + cus - 1) / cus) : 1;
}

}  // namespace ssp
