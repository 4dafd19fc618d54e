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
// Candidates a wavefront takes, | 16 swept in fours, | 32 read entry by entry.
int px_host_split(int candidates, int jobs, int Gm, int Gs, int f32, int row4, int whole_rows, int inherit)
{
    const px::PairSplit p = px::split_pairs(candidates, jobs, Gm, Gs, f32 != 0, row4 != 0, whole_rows != 0, inherit != 0);
    return (p.per_wave - 1) | (p.four ? 16 : 0) | (p.entry_by_entry ? 32 : 0);
}
// The same for any row length (nodes).
int px_host_split_nodes(int candidates, int jobs, int nodes, int Gm, int Gs, int f32)
{
    const bool row1 = nodes >= 4 && nodes <= 256, whole = nodes % 4 == 0 && Gm % 64 == 0;
    return px::split_pairs(candidates, jobs, Gm, Gs, f32 != 0, row1 && nodes <= 64, whole, false, row1).per_wave;
}
// The split a call takes, and what split_pairs had for it: as px_host_split, in bits above 8 the workgroups a job's candidates are shared
// out among.  (The sampling argmax does not read the rows of four candidates with one load.)
static int packed(const px::PairSplit &p, int candidates)
{
    return (p.per_wave - 1) | (p.four ? 16 : 0) | (p.entry_by_entry ? 32 : 0) | px::pair_groups(candidates, p.per_wave) << 8;
}
static px::PairSplit call_split(int candidates, int jobs, int nodes, int Gm, int Gs, bool f32, bool inherit, bool sampled, bool balanced)
{
    const bool row1 = nodes >= 4 && nodes <= 256, row4 = row1 && nodes <= 64 && !sampled, whole = nodes % 4 == 0 && Gm % 64 == 0;
    const px::PairSplit p = px::split_pairs(candidates, jobs, Gm, Gs, f32, row4, whole, inherit, row1, sampled);
    return balanced ? px::balanced_split(p, candidates, jobs, Gm, Gs, f32, row4, inherit, row1, sampled) : p;
}
int px_host_balanced(int candidates, int jobs, int nodes, int Gm, int Gs, int f32, int inherit, int sampled)
{
    return packed(call_split(candidates, jobs, nodes, Gm, Gs, f32 != 0, inherit != 0, sampled != 0, true), candidates);
}
int px_host_unbalanced(int candidates, int jobs, int nodes, int Gm, int Gs, int f32, int inherit, int sampled)
{
    return packed(call_split(candidates, jobs, nodes, Gm, Gs, f32 != 0, inherit != 0, sampled != 0, false), candidates);
}
int px_host_table_rows(int jobs, int Gm) { return px::table_rows(jobs, Gm); }
int px_host_pair_groups(int candidates, int per_wave) { return px::pair_groups(candidates, per_wave); }
int px_host_record_or_first(int found, int records) { return px::record_or_first(found, records); }
}
