// What the edge-balanced kernels (SpMM, fused AGNN forward and backward) share: how a wave stages the entries of its
// range in LDS, adds up over the lanes of a group and joins the rows that its groups cut.
//
// These kernels issue one gather per entry and little arithmetic, so what surrounds the gather decides: at 16 rows of 64
// bytes per load instruction the earlier form spent more instructions on it (two quarter-rate 64-bit multiplications, an execution
// mask and four LDS reads per entry) than on the row itself.  Here an entry is staged as the byte offset of its row (one
// multiplication where it is loaded, not one per lane of the group), four entries are one LDS read, entries past the end are
// a row of their own (-1) instead of a mask, and no wave waits for another.
#pragma once
#include "ftc_common.hpp"

namespace ftc {
#if defined(__HIPCC__)

// The LDS accesses of one wave are carried out in order: what is needed is that the compiler keeps that order.
__device__ __forceinline__ void wave_lds_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// A wave's R entries are cut into runs of RUN, one per group of LPR lanes; the runs lie RUNP words apart: four words of padding
// keep them 16-byte aligned and the 16-byte reads of the groups on different banks.
template <int LPR, int R>
struct EdgeRange {
    static constexpr int NG = 64 / LPR;
    static constexpr int RUN = R / NG;
    static constexpr int RUNP = RUN + 4;
    static constexpr int WORDS = NG * RUNP;  // one staged array
    static_assert(RUN % 4 == 0, "runs are whole batches of four entries");
    __device__ static __forceinline__ int slot(int i) { return i + i / RUN * 4; }
};

// Where row c of a gathered matrix begins: its byte offset in 32 bits, or (BIG: matrices of 4 GiB and more) c itself.
template <bool BIG>
__device__ __forceinline__ uint32_t row_slot(int c, uint64_t ldb)
{
    return BIG ? static_cast<uint32_t>(c) : static_cast<uint32_t>(c) * static_cast<uint32_t>(ldb);
}
template <bool BIG>
__device__ __forceinline__ const char *row_addr(const void *base, uint32_t slot, uint64_t ldb, uint32_t lane_bytes)
{
    if constexpr (BIG) return static_cast<const char *>(base) + (slot * ldb + lane_bytes);
    else return static_cast<const char *>(base) + (slot + lane_bytes);
}
inline bool rows_need_64_bits(int64_t n, int64_t row_bytes) { return n * row_bytes > static_cast<int64_t>(UINT32_MAX); }

// Loads the range's column ids and rows into s_off / s_row (and vals into s_val): base, n_valid and v are the same in the whole wave.
// Rows of a full range come from its first and last row and the row starts in between, marked as bits in LDS and counted
// (reading edge_to_row for every entry is a second 4-byte stream next to the column ids); where a row is empty two starts fall on one
// bit, the count is short and edge_to_row is read, as for the last, partial range.  DENSE: entries of flagged windows gather row 0.
template <int LPR, int R, bool VALS, bool BIG>
__device__ __forceinline__ void stage_range(const int *__restrict__ row_ptr, const int *__restrict__ col_idx,
                                            const int *__restrict__ edge_to_row, const float *__restrict__ vals, int base,
                                            int n_valid, uint64_t ldb, const uint8_t *__restrict__ dense, int lane,
                                            uint32_t *s_off, int *s_row, float *s_val)
{
    using E = EdgeRange<LPR, R>;
    constexpr int J = R / 64;
    int rows[J];
    int col[J];
    float val[VALS ? J : 1];
#pragma unroll
    for (int j = 0; j < J; ++j) {
        const int i = min(j * 64 + lane, n_valid - 1);
        col[j] = __builtin_nontemporal_load(col_idx + base + i);  // streamed once: no need to keep it in L2
        if constexpr (VALS) val[j] = __builtin_nontemporal_load(vals + base + i);
    }
    bool found = false;
    if (n_valid == R) {
        const int r_first = edge_to_row[base], r_last = edge_to_row[base + R - 1];
        const int n_starts = r_last - r_first;  // rows r_first + 1 .. r_last begin inside the range
        if (n_starts <= R / 2) {
            uint32_t *mark = reinterpret_cast<uint32_t *>(s_row);  // bit p - 1: a row starts at entry p
            if (lane < R / 32) mark[lane] = 0u;
            wave_lds_sync();
            for (int t = lane; t < n_starts; t += 64) {
                const int p = row_ptr[r_first + 1 + t] - base - 1;
                atomicOr(mark + (p >> 5), 1u << (p & 31));
            }
            wave_lds_sync();
            int before = 0;
#pragma unroll
            for (int j = 0; j < J; ++j) {
                const uint32_t lo = mark[2 * j], hi = mark[2 * j + 1];
                rows[j] = r_first + static_cast<int>(__builtin_amdgcn_mbcnt_hi(hi, __builtin_amdgcn_mbcnt_lo(lo, before)));
                before += __popc(lo) + __popc(hi);
            }
            found = before == n_starts;
            wave_lds_sync();  // the marks are overwritten below
        }
    }
    if (!found) {
#pragma unroll
        for (int j = 0; j < J; ++j) {
            const int i = j * 64 + lane;
            rows[j] = __builtin_nontemporal_load(edge_to_row + base + min(i, n_valid - 1));
            if (i >= n_valid) rows[j] = -1;
        }
    }
#pragma unroll
    for (int j = 0; j < J; ++j) {
        const int p = E::slot(j * 64 + lane);
        s_off[p] = (dense && dense[max(rows[j], 0) >> 4]) ? 0u : row_slot<BIG>(col[j], ldb);
        s_row[p] = rows[j];
        if constexpr (VALS) s_val[p] = val[j];
    }
    wave_lds_sync();
}

// v from lane ^ 4 of the same eight lanes
__device__ __forceinline__ float dpp_xor4(float v)
{
    const int t = __builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x1b, 0xf, 0xf, false);  // quad_perm [3,2,1,0]
    return __int_as_float(__builtin_amdgcn_update_dpp(0, t, 0x141, 0xf, 0xf, false));         // row_half_mirror
}

// Sums of four values over the lanes of a group: lane `sub` gets that of v[sub & 3].  Fewer instructions than four full sums, and
// what follows is done once for four entries instead of four times by every lane.
template <int LPR>
__device__ __forceinline__ float group_sum4(const float (&v)[4], bool odd, bool upper)
{
    const float a = (odd ? v[1] : v[0]) + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(odd ? v[0] : v[1]), 0xb1, 0xf, 0xf, false));
    const float b = (odd ? v[3] : v[2]) + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(odd ? v[2] : v[3]), 0xb1, 0xf, 0xf, false));
    float s = (upper ? b : a) + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(upper ? a : b), 0x4e, 0xf, 0xf, false));
    if constexpr (LPR >= 8) s += dpp_xor4(s);
    if constexpr (LPR >= 16) s = dpp_add<0x128>(s);  // row_ror:8
    if constexpr (LPR >= 32) s += __shfl_xor(s, 16, 64);
    return s;
}

// v of lane K of the quad
template <int K>
__device__ __forceinline__ float quad_lane(float v)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), K * 0x55, 0xf, 0xf, false));
}

// Where the pieces of a row cut by run boundaries lie.  A group's piece at the right end of its run is open when its row goes on
// in the next run: OPEN_TAIL when the row begins in this run, OPEN_THROUGH when it fills the run and came in from the left.
// The row that a group closes (or, in the last group, leaves open) began in group first_group(), or before this wave (-1).
enum { OPEN_NONE = 0, OPEN_TAIL = 1, OPEN_THROUGH = 2 };
template <int LPR>
__device__ __forceinline__ int first_group(int open, int g)
{
    const unsigned long long begun = __builtin_amdgcn_ballot_w64(open != OPEN_THROUGH);
    const unsigned long long before = begun & ((1ull << (g * LPR)) - 1ull);  // the lanes of the groups to the left
    return before ? (63 - __builtin_clzll(before)) / LPR : -1;
}

// Called by whole waves.  Sum of one slot of the head pieces of ranges first, first + step, ... last, stride floats from range to range: the ranges of a long row,
// shared by teams of lanes.  Sixteen loads in flight (a hub of the R-MAT graph spans 126 ranges: one after the other, four at a time, they
// were what the second pass waited for: fused AGNN layer 17.9 / 14.6 us), the remainder four at a time from clamped addresses, or
// one, which is all there is where a row has no more pieces than teams (four always: 8 fp16 columns, rows of 600 entries 18.6 / 19.8 us); the order depends on the shape alone.
__device__ __forceinline__ float sum_pieces(const float *__restrict__ base, size_t stride, int first, int last, int step)
{
    constexpr int U = 16;
    float s[4] = {0.f, 0.f, 0.f, 0.f};
    int u = first;
    for (; u + (U - 1) * step <= last; u += U * step) {
        float a[U];
#pragma unroll
        for (int j = 0; j < U; ++j) a[j] = base[static_cast<size_t>(u + j * step) * stride];
#pragma unroll
        for (int j = 0; j < U; ++j) s[j & 3] += a[j];
    }
    for (; __builtin_amdgcn_ballot_w64(u + step <= last); u += 4 * step) {  // uniform: one wait for all teams
        float a[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) a[j] = base[static_cast<size_t>(min(u + j * step, last)) * stride];
#pragma unroll
        for (int j = 0; j < 4; ++j) s[j] += u + j * step <= last ? a[j] : 0.f;
    }
    if (u <= last) s[0] += base[static_cast<size_t>(u) * stride];
    return (s[0] + s[1]) + (s[2] + s[3]);
}

#endif  // __HIPCC__
}  // namespace ftc
