// Host build of the arithmetic that kernels and launches share.
#include "../paper_2008_12260_amd/csrc/pollux_launch.h"

#include <stddef.h>
#include <vector>

extern "C" {
// Whether the launch for (jobs, tasks, counters) gives every (job, task) exactly one wavefront.
int px_host_prep_covers(int jobs, int tasks, long long counters)
{
    std::vector<int> taken((size_t)jobs * tasks, 0);
    const unsigned blocks = px::prep_blocks(jobs, tasks, counters);
    for (unsigned b = 0; b < blocks; ++b) {
        for (int w = 0; w < px::kWavesPerBlock; ++w) {
            const px::PrepSlot s = px::prep_slot(b, w, tasks);
            if (s.task < 0 || s.task >= tasks) return 0;
            if (s.job < jobs) ++taken[(size_t)s.job * tasks + s.task];
        }
    }
    for (int t : taken) {
        if (t != 1) return 0;
    }
    return 1;
}
unsigned px_host_prep_blocks(int jobs, int tasks, long long counters) { return px::prep_blocks(jobs, tasks, counters); }
int px_host_record_or_first(int found, int records) { return px::record_or_first(found, records); }
}
