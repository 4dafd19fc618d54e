// Plain arithmetic shared by the kernels, their launches and a host test: how the job-level launch divides its work, and which
// record a fit starts from.
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

// The record a search over a job's records has found, or the first where it has found none (no time below infinity).
PX_HOST_DEVICE int record_or_first(int found, int records) { return found < records ? found : 0; }

}  // namespace px
