// Queue of the large windows of the window build (build_windows.hip): how many entries a window takes and how many
// the workspace has room for.  Plain C++, so that the two can be held against each other on the host.
#pragma once
#include <stdint.h>

#if defined(__HIPCC__)
#define FTC_HD __host__ __device__
#else
#define FTC_HD
#endif

namespace ftc {

constexpr int MID_CAP = 4096;  // windows of at most this many edges are never queued for the direct kernels

// Parts a window of `cnt` edges is queued in for the direct kernels: every part builds the window's whole bitmap
// and ranks DIRECT_PART_EDGES of its edges or fewer, so that the few windows of 10^5 edges of a power-law graph do not
// keep one workgroup busy long after every other one has finished (one workgroup took 0.31 ms for the R-MAT
// benchmark graph's largest window, 256 000 edges; building the bitmap is the cheaper half of the work, 0.18 ns per
// edge against 0.40 ns for ranking and writing).
constexpr int DIRECT_SPLIT_MIN = 32768, DIRECT_PART_EDGES = 16384, DIRECT_PARTS_MAX = 16;
FTC_HD inline int direct_parts(int cnt)
{
    if (cnt <= DIRECT_SPLIT_MIN) return 1;
    const int p = static_cast<int>((static_cast<int64_t>(cnt) + DIRECT_PART_EDGES - 1) / DIRECT_PART_EDGES);
    return p < DIRECT_PARTS_MAX ? p : DIRECT_PARTS_MAX;
}

// Entries the queue has room for, the smaller of two bounds on what can be asked of it; every rule that says how many
// parts a window above MID_CAP edges is queued in has to keep both:
//   at most DIRECT_PARTS_MAX parts a window;
//   at most cnt / (MID_CAP + 1) parts of a window of cnt edges (cnt / DIRECT_PART_EDGES + 1 is no more than that above
//   DIRECT_SPLIT_MIN), which makes nnz / (MID_CAP + 1) in all.
FTC_HD inline int direct_capacity(int nnz, int n_windows)
{
    const int64_t by_parts = static_cast<int64_t>(n_windows) * DIRECT_PARTS_MAX;
    const int by_edges = nnz / (MID_CAP + 1) + 1;
    return by_edges < by_parts ? by_edges : static_cast<int>(by_parts);
}

}  // namespace ftc
