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

// Rows (placement class, K) of the sweep's tables one wavefront of prepare_kernel makes: eight from 128 jobs on, below that as many
// as keep its chain, rows x groups of 64 batch sizes, short while SIMDs are idle: two, four, or eight where those fill whole rounds.
// The terms of a group of batch sizes, formed once for all rows, are as much work as three.  Calls of 40 candidates, us with two, four
// and eight rows:
//    12 jobs   100 x 8 15.6, 15.7, 17.7; 257 x 8 20.4, 22.2, 28.8
//    24 jobs   64 x 8 15.2, 14.8, 15.0; 128 x 8 18.2, 17.2, 19.3; 384 x 32 fp32 29.4, 28.2, 36.9
//    48 jobs   64 x 8 16.7, 16.1, 15.4; 128 x 8 20.5, 19.6, 20.2; 448 x 8 45.0, 45.5, 48.1
//    96 jobs   64 x 8 20.8, 19.0, 18.8; 128 x 8 27.6, 24.7, 26.1
//   110 jobs   128 x 16 26.7, 26.3, 24.9 (two workgroups of eight rows a job and XCD, up to 120); 384 x 32 48.4, 49.8, 48.7
//   127 jobs   64 x 32 21.3, 20.9, 21.1; 128 x 32 27.6, 27.4, 29.1; 320 x 16 fp32 42.0, 44.5, 51.0
//   200 jobs   64 x 16 (1000 candidates) 66.7 with eight, 68.3 with sixteen; 1000 jobs, 32 x 8, 102.6, 87.6, 81.8
inline int table_rows(int jobs, int Gm)
{
    if (jobs >= 128 || (Gm <= 64 && jobs > 32) || (Gm <= 256 && jobs > 96 && jobs <= 120)) return 8;
    return jobs <= 16 || Gm > 256 ? 2 : 4;
}

constexpr int kMaxCandPerWave = 16;   // candidates one wavefront of pairs_kernel walks at most (lane r keeps what candidate r needs)

// How many candidates a wavefront of pairs_kernel takes, and how it reads and sweeps them.
struct PairSplit {
    int per_wave;
    bool four;              // (rows of at most 64 nodes) one load covers the rows of four candidates, and with chunks of up to 16
                            // counts one sweep does: a row of 16 lanes each
    bool entry_by_entry;    // ragged rows, fewer than four candidates a wavefront, none of them a generation's child
};

// row1: rows of 4 to 256 nodes.  row4: of at most 64, with count tables that fit on chip.  sampled: the sampling argmax.
// balanced_split then sets the count of calls on rows of 65 to 256 nodes (shorter ones where the count tables do not fit) and, on shorter
// ones, of those that go four at a time or are put to it there.  What is said here of the count holds for the others: short rows one at a
// time (fp32 and ragged on few pairs or wide grids), row inheritance, the sampling argmax, longer rows.  Its figures are of sweeps that
// took longer than today's.
//
// per_wave: 25000 wavefronts fill the chip several times over.  Fewer with more candidates each save what a wavefront does once (job
// terms, table in LDS, prices), until the last wavefronts to end cost more: down to 12400 wavefronts with as many candidates as that
// takes on short rows and narrow grids, up to six on others, up to four on rows of more than 256 nodes, which are read one after the
// other.  (The sampling argmax of a pair has no such start to save: 40 candidates of 1000 jobs on 250 nodes, 128 sizes, 74 us, 83 with
// three a wavefront.)  us with 25000 wavefronts and so:
//   64 nodes, 64 x 16      200 jobs: 125 candidates 45.6, 34.1; 500 47.6, 44.9; 1250 85.6, 76.8
//   64 nodes, 128 x 32     100 jobs, fp32: 250 candidates 42.9, 39.0
//   100 nodes, 64 x 16     1000 jobs: 62 candidates, fp32, 73.2, 70.4; 200 candidates 97.7, 98.0 (sixteen each: 105.0)
//   320 nodes, 32 x 16     fp32: 100 candidates of 331 jobs 54.7, 52.3; 150 of 1000 jobs 153.9, 153.9 (twelve each: 168.4)
// four: a sweep of four saves three elections and lasts as long with one candidate as with four.  fp64 on whole rows and grids, and
// with more than 16 counts (loads only), always.  Else from 8000 pairs on and on narrow grids (at 2000 pairs 1.04 to 1.19 times as
// long in fours, at 5000 0.93 to 1.03, at 10000 0.79 to 0.91; grids of 300 batch sizes 1.4 times at 2000 and, with most rows empty,
// still 1.3 at 200000), and in whole fours.  With row inheritance a job's list has no length known here: no rounding, and fours from
// 80000 pairs on (1000 children of 200 jobs on 61 nodes, 64 x 16: 60.1 and 65.6 us one at a time), in fp32 on whole rows not at all.
inline PairSplit split_pairs(int candidates, int jobs, int Gm, int Gs, bool f32, bool row4, bool whole_rows, bool inherit, bool row1 = true,
                             bool sampled = false)
{
    const long long pairs = (long long)candidates * jobs;
    const int share = (candidates - 1) / kWavesPerBlock + 1;                    // a workgroup's wavefronts take the candidates in turn
    const int chunk = Gm * ((Gs + 15) / 16);                                    // the grid's width: batch sizes x chunks of 16 counts
    long long want = pairs / 25000;
    if (!inherit && !sampled) {
        const long long most = row4 && chunk <= 64 ? kMaxCandPerWave : (row1 ? 6 : 4), more = pairs / 12400;
        const long long wider = more < most ? more : most;
        want = want > wider ? want : wider;
    }
    int n = (int)(want < kMaxCandPerWave ? want : kMaxCandPerWave);
    n = n < share ? n : share;
    n = n > 1 ? n : 1;
    if (!row4) return PairSplit{n, false, false};
    if (!f32 && (whole_rows || Gs > 16)) return PairSplit{Gs > 16 || n < 4 || inherit ? n : n & ~3, true, false};
    const bool four = inherit ? chunk <= 64 && pairs >= 80000 && !whole_rows : chunk <= 128 && pairs >= 8000 && share >= 4;
    if (four && !inherit) n = n < 4 ? 4 : (n + 2) & ~3;
    return PairSplit{n, four, !four && n < 4};
}

// Workgroups a job's candidates are shared out among.
inline int pair_groups(int candidates, int per_wave)
{
    const int group = per_wave * kWavesPerBlock;
    return (int)(((long long)candidates + group - 1) / group);
}

// The split of a call on rows of 4 to 256 nodes whose candidates are known: what all wavefronts do once (job terms, table in LDS, table
// rows, prices: some 250 vector instructions each; 2 ns of the whole chip's time a workgroup, beyond three a compute unit) against what
// each candidate adds to the last wavefront's chain (its sweeps, one after the other, by the grid's width: 0.3 us and 0.12 us per 64
// batch sizes x 16 counts on rows of 65 nodes and more; 0.2 and 0.15 where four are swept at a time; 0.28 per 64 x 16 one at a time
// on short rows).  The sum is least at about the root of pairs / 2000; this finds the least, the unequal shares of a job's last
// workgroup included, in whole fours where four are swept at a time (a sweep lasts as long with one as with four).  Sweep and mean of
// kept calls, us (candidates a wavefront), with split_pairs' count, so, and the least of 1 .. 16:
//   80 nodes    60 candidates of 100 jobs, 64 x 16      13.4 (1)   12.1 (2)   12.1
//   100 nodes   60 of 400, 64 x 16                      28.7 (1)   19.7 (5)   19.7;  128 x 32  32.8, 25.3, 25.3
//   200 nodes   120 of 300, 64 x 16                     28.5 (2)   25.2 (6)   25.2
//   90 nodes    500 of 200, 64 x 16                     43.3 (6)   43 (9)     42.5 (8)
//   200 nodes   400 of 400, 64 x 16                     64.1 (6)   61.3 (10)  61.3;  128 x 32  89.8, 87.8, 87.8
//   130 nodes   1021 of 331, 50 x 21                    115 (13)   110 (16)   110
//   64 nodes    30 of 200, 64 x 16                      15.0 (1)   10.1 (4)   10.1
//   64 nodes    60 of 400, 64 x 16                      32.4 (1)   15.4 (8)   15.4;  50 x 21  26.0, 18.0, 18.0
// Fp32 and ragged short rows go four at a time from 4000 pairs on: one at a time and four, 60 x 60 on 33 nodes, 50 x 12, 10.3, 9.9, 100 x 12
// 10.7, 10.8, fp32 64 x 16 11.0, 10.9; 40 x 40 on 22 nodes 9.1, 9.7; 44 x 137 on 57 nodes, 100 x 12, 12.6, 11.4.  Grids wider than
// 64 batch sizes x 16 counts from 6000: fp32 69 x 64 on 8 nodes, 128 x 12, 11.3, 11.9, 242 x 24 on 6, 100 x 12, 14.5, 15.4; 51 x 120 on 15,
// 100 x 8, 12.9, 12.3; 184 x 35 on 13, 128 x 12, 13.6, 12.4.
// Row inheritance, whose lists have no length known here, the sampling argmax and longer rows keep split_pairs' count, and so do short
// rows below those lines or on grids of more than 128 batch sizes x chunks of 16 counts, unless split_pairs has them in fours already.
inline PairSplit balanced_split(PairSplit s, int candidates, int jobs, int Gm, int Gs, bool f32, bool row4, bool inherit, bool row1, bool sampled)
{
    if (inherit || sampled || !row1) return s;
    const int share = (candidates - 1) / kWavesPerBlock + 1;
    if (row4 && !s.four) {
        const long long chunk = (long long)Gm * ((Gs + 15) / 16);
        if (chunk > 128 || (long long)candidates * jobs < (chunk > 64 ? 6000 : 4000) || share < 4) return s;
        s.four = true;
        s.entry_by_entry = false;
    }
    const bool swept = row4 && (f32 || Gs <= 16);
    const int step = swept ? 4 : 1;
    if (share < step) return s.four ? PairSplit{share, true, false} : s;
    const long long width = (long long)((Gm + 63) / 64) * ((Gs + 15) / 16);
    const long long chain = !row4 ? 300 + 120 * width : (swept ? 200 + 150 * width : 280 * width);        // ns a candidate
    long long least = -1;
    for (int n = step; n <= kMaxCandPerWave && n < share + step; n += step) {
        const long long crowd = (long long)jobs * pair_groups(candidates, n) - 768;                        // workgroups
        const long long cost = 2 * (crowd > 0 ? crowd : 0) + chain * n;
        if (least < 0 || cost < least) {
            least = cost;
            s.per_wave = n;
        }
    }
    return s;
}

// Queries (GPU count, placement) of one job that a wavefront takes.  Forming the terms of a job's batch sizes is as much work as three
// argmaxes and is shared by them, but they follow one another: up to some six wavefronts a SIMD one each is as quick.  us with one,
// with two, four and six: 3400 queries 64 x 16 6.3, 6.1, 6.1, 7.2; 7500 of 32 x 8 9.3, 8.4, 9.2, 9.1; 11000 of 128 x 32 16.6, 14.2, 12.9,
// 11.8; 25000 of 64 x 16 23.7, 19.6, 17.0, 16.9 (twelve: 18.9).
inline int query_rows(int jobs, int per_job)
{
    const long long want = (long long)jobs * per_job / 3000;
    const int rows = (int)(want < 1 ? 1 : (want < 6 ? want : 6));
    return rows < per_job ? rows : per_job;
}

// The record a search over a job's records has found, or the first where it has found none (no time below infinity).
PX_HOST_DEVICE int record_or_first(int found, int records) { return found < records ? found : 0; }

}  // namespace px
