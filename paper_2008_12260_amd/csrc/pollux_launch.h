// Plain arithmetic shared by the kernels, their launches and a host test: how the job-level launch and the population pass divide
// their work, and which record a fit starts from.
#pragma once

#if defined(__HIPCC__)
#define PX_HOST_DEVICE __host__ __device__ __forceinline__
#else
#define PX_HOST_DEVICE inline
#endif

namespace px {

constexpr int kWavesPerBlock = 4;

// The (job, task) a wavefront of prepare_kernel takes; job may lie beyond the last one.  Workgroups are dealt to the eight
// XCDs round-robin: every task of job j runs on XCD j % 8.
struct PrepSlot {
    int job, task;
};

PX_HOST_DEVICE PrepSlot prep_slot(unsigned block, int wave, int tasks)
{
    const int slot = (int)(block >> 3) * kWavesPerBlock + wave;
    return PrepSlot{(slot / tasks) * 8 + (int)(block & 7), slot % tasks};
}

// Workgroups of prepare_kernel for `tasks` wavefronts a job, with `counters` words to clear: never fewer than the (job, task)
// pairs need, one wavefront each; more, up to 1024, where a few jobs come with many candidates (the clearing loop strides
// over whatever the launch has).
inline unsigned prep_blocks(int jobs, int tasks, long long counters)
{
    const long long slots = ((long long)(jobs + 7) / 8) * tasks;
    const long long needed = (slots + kWavesPerBlock - 1) / kWavesPerBlock * 8;
    const long long clear = (counters + 4095) / 4096, clearing = clear < 1024 ? clear : 1024;
    return (unsigned)(needed > clearing ? needed : clearing);
}

constexpr int kMaxCandPerWave = 16;   // candidates one wavefront of pairs_kernel walks at most (lane r keeps what candidate r needs)

// How many candidates a wavefront of pairs_kernel takes: enough wavefronts to fill the chip several times over.  And, for rows of at
// most 64 nodes whose count tables are on chip (row4), whether one load covers the rows of four candidates, which with chunks of up
// to 16 counts also sweeps the four, a row of 16 lanes each.
// A sweep of four saves three elections and lasts as long with one candidate as with four: it wants candidates in whole fours and
// narrow grids.  In fp32 on whole rows and grids the instance that sweeps one at a time has eight wavefronts a SIMD against six, and
// is quicker from nine candidates a wavefront on.  fp64 on whole rows and grids takes four always.  Calls that keep their tables,
// us, 16 nodes (whole rows) and 17: one at a time, four at a time in whole fours (in brackets: one candidate a wavefront)
//   fp32, 16 nodes,  64 x 16   64 candidates of 500 jobs 25.6, 16.6 (33.7); 1000 of 200 49.0, 48.7; 2000 of 300 92.9, 113.6
//   fp32, 16 nodes, 512 x 16   64 of 500 30.2, 42.7 (119)
//   fp32, 16 nodes,  64 x 32   1000 of 200 56.4, 59.1
//   fp64, 17 nodes,  64 x 16   64 of 500 25.7, 17.6 (38.2); 2000 of 300 157, 129
//   fp64, 17 nodes, 100 x 16   100 of 30 10.0, 11.0; 64 of 500 27.5, 22.3 (48.7); 1200 of 200 104, 86.5
//   fp64, 16 nodes, 100 x 16   2000 of 300 162, 181
//   fp64, 17 nodes, 500 x 12   64 of 500 47.0, 59.8 (144)
// With row inheritance a job's list is shorter than the candidates, of no length known here, and the split is not rounded to fours
// (128 children of 1000 jobs, 64 x 8: 60.5 us, 67.3 in fours).
// entry_by_entry: ragged rows with fewer than four candidates a wavefront, none of them a generation's child (see launch_fitness).
struct PairSplit {
    int per_wave;
    bool four, entry_by_entry;
};

inline PairSplit split_pairs(int candidates, int jobs, int Gm, int Gs, bool f32, bool row4, bool whole_rows, bool inherit)
{
    const long long pairs = (long long)candidates * jobs;
    const int share = (candidates - 1) / kWavesPerBlock + 1;                    // a workgroup's wavefronts take the candidates in turn
    int n = (int)(pairs / 25000 < kMaxCandPerWave ? pairs / 25000 : kMaxCandPerWave);
    n = n < share ? n : share;
    n = n > 1 ? n : 1;
    if (!row4) return PairSplit{n, false, false};
    if (!f32 && (whole_rows || Gs > 16)) return PairSplit{n, true, false};
    const bool narrow = Gm <= 64 && (Gs <= 16 || !whole_rows);
    bool four;
    if (inherit) four = narrow;
    else if (narrow && Gs <= 16) four = share >= 4 && !(whole_rows && n > 9);
    else four = share >= 4 && Gm <= 128 && !whole_rows && pairs >= 6000 && n <= 9;
    if (four && !inherit) n = n < 4 ? 4 : n & ~3;
    return PairSplit{n, four, !four && n < 4};
}

// Workgroups a job's candidates are shared out among.
inline int pair_groups(int candidates, int per_wave)
{
    const int group = per_wave * kWavesPerBlock;
    return (int)(((long long)candidates + group - 1) / group);
}

// The record a search over a job's records has found, or the first where it has found none (no time below infinity).
PX_HOST_DEVICE int record_or_first(int found, int records) { return found < records ? found : 0; }

}  // namespace px
