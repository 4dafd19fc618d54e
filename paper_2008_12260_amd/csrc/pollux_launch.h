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

// How many candidates a wavefront of pairs_kernel takes: enough wavefronts to fill the chip several times over.  Calls of 200 jobs, us
// with 25000, 16600 and 12400 wavefronts:
//   64 nodes, 64 x 16    125 candidates 45.6, 45.6, 34.1; 250 46.8, 38.7, 35.1; 500 47.6, 50.1 (six each), 44.9; 750 63.0, 61.6, 55.1;
//                        1000 65.4, 64.3, 65.2; 1250 85.6 (ten), 79.0 (fifteen), 76.8: swept in fours, so in whole fours
//   100 nodes, 64 x 16   125 39.3, 39.3, 33.8; 500 58.0, 54.7, 54.0; 1000 83.8, 83.1, 83.7; 1500 111.2, 109.4, 109.4
//   100 nodes, 128 x 32  125 51.1, 51.2, 46.5; 500 87.5, 84.1, 84.9; 1000 131.3, 133.2, 136.9; 1500 178.2, 181.0, 180.6
// And, for rows of at most 64 nodes whose count tables are on chip (row4), whether one load covers the rows of four candidates, which with chunks of up
// to 16 counts also sweeps the four, a row of 16 lanes each.
// A sweep of four saves three elections and lasts as long with one candidate as with four: it wants candidates in whole fours,
// enough pairs to fill the chip with so few wavefronts, and narrow grids (chunk: batch sizes x chunks of 16 counts).
// fp64 on whole rows and grids takes four always.  Calls that keep their tables, at 1.3 to 10 GPUs a job, us one at a time and
// four at a time:
//   17 nodes, 50 x 16, fp64    66 candidates of 30 jobs 9.1, 9.7; 166 of 30 11.5, 10.1; 300 of 100 30.9, 16.8
//   16 nodes, 64 x 16, fp32    66 of 30 9.2, 10.0; 166 of 30 11.2, 10.5; 300 of 100 26.5, 16.4; 1300 of 100 48.0, 43.1
// over the 16 to 64 nodes and 6 grids tried: 2000 pairs 1.04 to 1.19 times as long in fours, 5000 0.93 to 1.03, 10000 0.79 to 0.91,
// from there on 0.65 to 0.98.  Grids of 300 take 1.4 times as long at 2000 pairs and 0.9 from 12000 on, but more again where most
// rows are empty and fours cannot be filled (1000 candidates of 200 jobs on 128 GPUs, 500 x 12: 228 and 175): wide grids go one at a time.
// With row inheritance a job's list is shorter than the candidates, of no length known here: its split is not rounded to fours (128
// children of 1000 jobs, 64 x 8: 60.5 us, 67.3 in fours), and four at a time pay from 80000 pairs on (1000 children of 200 jobs on
// 61 nodes, 64 x 16: 60.1 and 65.6; 100 children of 200 jobs 1.03 times as long), in fp32 on whole rows not at all (1.02 to 1.06).
// entry_by_entry: ragged rows with fewer than four candidates a wavefront, none of them a generation's child (see launch_fitness).
struct PairSplit {
    int per_wave;
    bool four, entry_by_entry;
};

inline PairSplit split_pairs(int candidates, int jobs, int Gm, int Gs, bool f32, bool row4, bool whole_rows, bool inherit)
{
    const long long pairs = (long long)candidates * jobs;
    const int share = (candidates - 1) / kWavesPerBlock + 1;                    // a workgroup's wavefronts take the candidates in turn
    const int chunk = Gm * ((Gs + 15) / 16);
    // What a wavefront does once (job terms, table in LDS, prices) is worth the sweeps of two candidates of 64 x 16: as many as 12400
    // wavefronts leave each.  Wider grids weigh it less, and the last wavefronts last longer: up to six that way.
    const long long by_25000 = pairs / 25000, by_12400 = pairs / 12400;
    long long want = by_25000;
    if (!inherit) want = chunk <= 64 ? by_12400 : (by_25000 > 6 ? by_25000 : (by_12400 < 6 ? by_12400 : 6));
    int n = (int)(want < kMaxCandPerWave ? want : kMaxCandPerWave);
    n = n < share ? n : share;
    n = n > 1 ? n : 1;
    if (!row4) return PairSplit{n, false, false};
    if (!f32 && (whole_rows || Gs > 16)) return PairSplit{Gs > 16 || n < 4 || inherit ? n : n & ~3, true, false};
    const bool four = inherit ? chunk <= 64 && pairs >= 80000 && !whole_rows : chunk <= 128 && pairs >= 8000 && share >= 4;
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
