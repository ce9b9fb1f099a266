// Row-wise kernels of the reordering step for graphs of at most ROW_SORT_NODES nodes: the relabelled graph and a
// round of label propagation both look every entry's column up in an array of n ints and need the results of ONE
// row in ascending order -- the new columns to write them out, the labels to find the longest run of equal ones.
// Rows are independent, so nothing is sorted across rows: a row is sorted where it fits,
//   at most 16 / 32 / 64        a quarter, half or whole wave, one entry per lane (bitonic, data-parallel-primitive moves),
//   at most 256 / 1024          a wave, 4 / 16 entries per lane,
//   at most 8192                a workgroup of 1024 threads, in LDS,
//   longer                      a bitmap of the columns in LDS (relabelling; duplicates: counters, see below) or
//                               counters in LDS per 32 768 labels (label propagation); with more than 2^19 nodes those of
//                               at most 32 768 entries are sorted in LDS instead of counted (many_ranges()).
// What bounds them: the look-up.  Every entry is one 4-byte gather from an array that about fills an L2 (4 MB at
// a million nodes); the streams around it (column ids in, columns out) are read and written once, non-temporal.
// On the block model with a million nodes and 32 M entries a round of label propagation takes 0.21 ms and the
// relabelled graph 0.33 ms (R-MAT, 2^20 nodes: 0.48); sorting all entries by label and row with the global radix sort took
// 4.0 and 4.1 ms.  The sorting network is the other half: with min, max and a selection per stage, rows of 33 to 64 two at a time,
// rows of any length below side by side in halves of the wave and each row's look-ups waiting for the one's before, a round took
// 0.24 ms (500 000 nodes with nine entries each, the whole plan: 1.39 / 1.01 ms).
// Larger graphs keep the radix sort: the counters of the long rows cost one pass over the row per 32 768 nodes.  Up to
// ROW_SORT_NODES the rows are ahead on every graph that was measured but for one kind: the relabelled graph where nearly all
// entries are in rows of more than 32 768 entries with repeated columns (2^22 nodes, 65 M entries, 95 % of them in rows of
// 60 000: 18 against 9 ms; half of them: 9.7 against 9.4; label propagation on the first: 16 ms a round on either).
#include "edge_ranges.hpp"

namespace ftc {

constexpr int RS_ROWS = 32;         // consecutive rows per wave of the short-row part
constexpr int RS_SHORT = 64;        // longest row handled there; the queues hold the rows above
constexpr int RS_MID = 256, RS_LONG = 1024, RS_LDS = 8192;  // longest row of queues 0, 1, 2; queue 3 has the rest
constexpr int RS_LDS_MOST = 32768;  // longest row of queue 2 in label propagation on many nodes (many_ranges())
constexpr int RS_RANGE = 32768;     // counters per pass over a long row
constexpr int RS_WORDS = RS_RANGE + RS_RANGE / 32;  // LDS words of the workgroups that take long rows
constexpr int RS_BITS_LOG2 = 20;    // columns per bitmap pass over a long row (32 768 words)
constexpr int RS_NONE = 0x7fffffff; // sorts behind every column and label

// lengths of the rows: len[r] = rp[r + 1] - rp[r]; counts[q] rows of class q in rows[q]
struct RowQueues {
    int *counts;
    int *rows[4];
    int *dup_rows;               // relabelling: long rows with duplicate columns, counts[4] of them
    unsigned long long *best;    // label propagation: winner of every row of queue 3
    int *values;                 // what the columns of the counted rows become, at the place of the entry; NULL: not kept
};

// Passes over a row longer than queue 2's: counters for RS_RANGE of the n values each.
__host__ __device__ inline int value_ranges(int n) { return (n + RS_RANGE - 1) / RS_RANGE; }

// From this many passes on rows of up to 32 768 entries are sorted instead of counted (an entry costs about 25 ps sorted, 6 a
// pass counted, but one row of 30 000 entries alone keeps a workgroup for 60 us), and the look-ups of the counted rows are made
// once and kept.  Ten rounds of label propagation, ms, counted with a look-up in every pass / sorted or looked up once / radix
// sort of all entries ("share": of the 64 M entries, with 2^18 nodes 16 M, that are in rows of 8200 or of 60 000 entries):
//   2^18 nodes, 8 passes     0.1 of 8200 2.0 / 1.6 / 18, of 60 000 1.8 / 2.0 / 19; R-MAT, degree 64 2.9 / 3.5 / 16
//   2^19 nodes, 16 passes    R-MAT, degree 16 1.7 / 2.3 / 8.7; degree 64 6.1 / 5.6 / 31
//   2^20 nodes, 32 passes    0.95 of 8200 124 / 17 / 106, of 60 000 87 / 43 / 106; R-MAT, degree 8 2.2 / 2.6 / 10, 32 9.0 / 6.4 / 32
//   2^22 nodes, 128 passes   0.5 of 8200 273 / 15 / 102, of 60 000 190 / 78 / 105; R-MAT, degree 16 33 / 16 / 67
__host__ __device__ inline bool many_ranges(int n) { return value_ranges(n) > 16; }

__global__ __launch_bounds__(1024) void row_classes_kernel(int n, const int *__restrict__ rp, int in_lds, RowQueues q)
{
    constexpr int PER = 4;
    __shared__ int cnt_s[4], base_s[4];
    if (threadIdx.x < 4) cnt_s[threadIdx.x] = 0;
    __syncthreads();
    int cls[PER], pos[PER];
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        const int64_t r = (static_cast<int64_t>(blockIdx.x) * PER + k) * 1024 + threadIdx.x;
        const int len = r < n ? rp[r + 1] - rp[r] : 0;
        cls[k] = len <= RS_SHORT ? -1 : len <= RS_MID ? 0 : len <= RS_LONG ? 1 : len <= in_lds ? 2 : 3;
        pos[k] = cls[k] >= 0 ? atomicAdd(&cnt_s[cls[k]], 1) : 0;
    }
    __syncthreads();
    if (threadIdx.x < 4 && cnt_s[threadIdx.x] > 0) base_s[threadIdx.x] = atomicAdd(&q.counts[threadIdx.x], cnt_s[threadIdx.x]);
    __syncthreads();
#pragma unroll
    for (int k = 0; k < PER; ++k)
        if (cls[k] >= 0)
            q.rows[cls[k]][base_s[cls[k]] + pos[k]] = static_cast<int>((static_cast<int64_t>(blockIdx.x) * PER + k) * 1024 + threadIdx.x);
}

// ---- the two uses -----------------------------------------------------------------------------------
// Row r of the result: entries [start, start + len) of col_idx; value(c) is what column c becomes: map[lookup_index(c)], checked by
// settle().  Loads are unconditional and the checks made on what came back: a load inside a branch is waited for at the branch's
// end, so that the look-ups of several rows would follow one another instead of being in flight together.
__device__ __forceinline__ int lookup_index(int c, int n) { return static_cast<unsigned>(c) < static_cast<unsigned>(n) ? c : 0; }
struct Relabel {
    static constexpr bool VOTES = false;
    int n;
    const int *row_ptr, *col_idx, *perm, *map, *rp;  // map: inv; rp: row starts of the relabelled graph
    int *out, *flag;
    __device__ __forceinline__ void row(int r, int &start, int &len) const
    {
        len = rp[r + 1] - rp[r];
        start = len > 0 ? row_ptr[perm[r]] : 0;  // a row that has entries has passed the check of perm[r]
    }
    __device__ __forceinline__ int settle(int c, int v, bool active) const
    {
        if (!active || (c >= 0 && c < n && v >= 0 && v < n)) return v;
        atomicOr(flag, 1);
        return 0;
    }
    __device__ __forceinline__ int value(int c) const { return settle(c, map[lookup_index(c, n)], true); }
};
struct Votes {
    static constexpr bool VOTES = true;
    int n;
    const int *col_idx, *map, *rp;  // map: labels of the round before
    int *out;                       // labels of this round
    __device__ __forceinline__ void row(int r, int &start, int &len) const
    {
        start = rp[r];
        len = rp[r + 1] - start;
    }
    __device__ __forceinline__ int settle(int c, int v, bool) const { return c >= 0 && c < n ? v : 0; }  // out of range: a vote for label 0
    __device__ __forceinline__ int value(int c) const { return settle(c, map[lookup_index(c, n)], true); }
};

// ---- sorting in registers ------------------------------------------------------------------------------
// value of lane (lane ^ S)
template <int S>
__device__ __forceinline__ int lane_xor(int v)
{
    if constexpr (S == 1) return __builtin_amdgcn_update_dpp(0, v, 0xb1, 0xf, 0xf, true);         // quad_perm [1,0,3,2]
    else if constexpr (S == 2) return __builtin_amdgcn_update_dpp(0, v, 0x4e, 0xf, 0xf, true);    // quad_perm [2,3,0,1]
    else if constexpr (S == 4) {
        const int m = __builtin_amdgcn_update_dpp(0, v, 0x141, 0xf, 0xf, true);                   // row_half_mirror: ^ 7
        return __builtin_amdgcn_update_dpp(0, m, 0x1b, 0xf, 0xf, true);                           // quad_perm [3,2,1,0]: ^ 3
    } else if constexpr (S == 8) return __builtin_amdgcn_update_dpp(0, v, 0x128, 0xf, 0xf, true); // row_ror:8
    else if constexpr (S == 16) {  // [0]: the even rows of 16 lanes twice, [1]: the odd ones
        const auto r = __builtin_amdgcn_permlane16_swap(v, v, false, false);
        return threadIdx.x & 16 ? r[0] : r[1];
    } else {
        const auto r = __builtin_amdgcn_permlane32_swap(v, v, false, false);  // the halves of the wave
        return threadIdx.x & 32 ? r[0] : r[1];
    }
}

// The lanes that keep the smaller element in the stage (STRIDE, SIZE) of a sort of `all` elements, W lanes each, register 0.
constexpr unsigned long long lanes_of_the_smaller(int stride, int size, int all, int W)
{
    unsigned long long m = 0ull;
    for (int lane = 0; lane < 64; ++lane) {
        const int li = lane % W;
        const bool up = size >= all || (li & size) == 0;
        if (up == ((li & stride) == 0)) m |= 1ull << lane;
    }
    return m;
}
// The smaller of a and b in the lanes of `smaller`, the larger in the others.  Two instructions (min, max and a selection
// are three), and the mask stays in scalar registers: as a bound per stage in vector registers, which the compiler makes of it
// by itself, the masks of all sorts cost half of the occupancy.
__device__ __forceinline__ int pick(int a, int b, unsigned long long smaller)
{
    int r;
    asm("v_cndmask_b32_e64 %0, %4, %5, %3\n\tv_med3_i32 %0, %1, %2, %0" : "=&v"(r) : "v"(a), "v"(b), "s"(smaller), "v"(INT32_MAX), "v"(INT32_MIN));
    return r;
}

template <int STRIDE, int SIZE, int K, int W>
__device__ __forceinline__ void bitonic_stage(int (&v)[K])
{
    if constexpr (STRIDE >= 64) {  // the partner sits in the same lane
#pragma unroll
        for (int k = 0; k < K; ++k) {
            constexpr int KS = STRIDE / 64;
            if ((k & KS) == 0) {
                const bool up = ((k * 64) & SIZE) == 0;
                const int a = v[k], b = v[k | KS];
                v[k] = up ? min(a, b) : max(a, b);
                v[k | KS] = up ? max(a, b) : min(a, b);
            }
        }
    } else {
        constexpr unsigned long long smaller = lanes_of_the_smaller(STRIDE, SIZE, K * W, W);
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const int o = lane_xor<STRIDE>(v[k]);
            const bool down = SIZE < K * W && ((k * 64) & SIZE) != 0;
            v[k] = pick(v[k], o, down ? ~smaller : smaller);
        }
    }
    if constexpr (STRIDE > 1) bitonic_stage<STRIDE / 2, SIZE, K, W>(v);
}

// Element i of the row sits in register i / 64, lane i % 64 (W = 64), or in lane i of its W lanes (W = 16 or 32, K = 1).
template <int SIZE, int K, int W>
__device__ __forceinline__ void bitonic_sort(int (&v)[K])
{
    if constexpr (SIZE > 2) bitonic_sort<SIZE / 2, K, W>(v);
    bitonic_stage<SIZE / 2, SIZE, K, W>(v);
}

template <int W>
__device__ __forceinline__ uint32_t group_max(uint32_t x)
{
    int v = static_cast<int>(x);
    auto larger = [](int a, int b) { return static_cast<int>(max(static_cast<uint32_t>(a), static_cast<uint32_t>(b))); };
    v = larger(v, lane_xor<1>(v)); v = larger(v, lane_xor<2>(v)); v = larger(v, lane_xor<4>(v)); v = larger(v, lane_xor<8>(v));
    if constexpr (W >= 32) v = larger(v, lane_xor<16>(v));
    if constexpr (W == 64) v = larger(v, lane_xor<32>(v));
    return static_cast<uint32_t>(v);
}

// The value of the longest run of equal values among the first `len` sorted ones, the smallest on a tie.  Values lie below
// ROW_SORT_NODES and a row here has at most RS_LONG entries: length and value are one 32-bit word.
template <int K, int W>
__device__ __forceinline__ int longest_run(const int (&v)[K], int len, int lane)
{
    constexpr int VALUE_BITS = 22;
    constexpr uint32_t VALUES = (1u << VALUE_BITS) - 1u;
    static_assert(ROW_SORT_NODES <= 1 << VALUE_BITS && RS_LONG <= 1 << (32 - VALUE_BITS), "a run and its value fit into 32 bits");
    const int li = lane & (W - 1);
    uint32_t best = 0u;
    int next = len;  // where the first run after register k begins
#pragma unroll
    for (int k = K - 1; k >= 0; --k) {
        int prev = __builtin_amdgcn_update_dpp(0, v[k], 0x138, 0xf, 0xf, false);  // wave_shr:1
        if constexpr (K > 1) {
            if (k > 0) {
                const int last = __builtin_amdgcn_readlane(v[k > 0 ? k - 1 : 0], 63);
                if (lane == 0) prev = last;
            }
        }
        const int i = k * 64 + li;
        const bool start = i < len && (i == 0 || prev != v[k]);
        const unsigned long long all = __builtin_amdgcn_ballot_w64(start);
        int end;
        if constexpr (W == 64) {
            const unsigned long long above = li < 63 ? all & (~0ull << (li + 1)) : 0ull;
            end = above ? k * 64 + __ffsll(static_cast<long long>(above)) - 1 : next;
            if (all) next = k * 64 + __ffsll(static_cast<long long>(all)) - 1;
        } else {
            uint32_t m = lane < 32 ? static_cast<uint32_t>(all) : static_cast<uint32_t>(all >> 32);
            if constexpr (W == 16) m = m >> (lane & 16) & 0xffffu;
            const uint32_t above = m & (0xfffffffeu << li);
            end = above ? __ffs(static_cast<int>(above)) - 1 : len;
        }
        const uint32_t score = static_cast<uint32_t>(end - i - 1) << VALUE_BITS | (VALUES - (static_cast<uint32_t>(v[k]) & VALUES));
        best = start ? max(best, score) : best;
    }
    return static_cast<int>(VALUES - (group_max<W>(best) & VALUES));
}

// Sorted values of row r leave: all of them, or the winner's label.
template <class Use, int K, int W>
__device__ __forceinline__ void row_done(const Use &u, int r, int dst, int len, const int (&v)[K], int lane)
{
    const int li = lane & (W - 1);
    if constexpr (Use::VOTES) {
        const int w = longest_run<K, W>(v, len, lane);
        if (li == 0 && len > 0) u.out[r] = w;
    } else {
#pragma unroll
        for (int k = 0; k < K; ++k)
            if (k * 64 + li < len) __builtin_nontemporal_store(v[k], u.out + dst + k * 64 + li);
    }
}

// one row of a queue by one wave, K entries per lane
template <class Use, int K>
__device__ __forceinline__ void queued_row(const Use &u, int r, int lane)
{
    int start, len;
    u.row(r, start, len);
    int c[K], v[K];
#pragma unroll
    for (int k = 0; k < K; ++k) c[k] = __builtin_nontemporal_load(u.col_idx + start + min(k * 64 + lane, len - 1));  // (no queued row is empty)
#pragma unroll
    for (int k = 0; k < K; ++k) v[k] = u.map[lookup_index(c[k], u.n)];
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const bool in = k * 64 + lane < len;
        v[k] = u.settle(c[k], v[k], in);
        if (!in) v[k] = RS_NONE;
    }
    bitonic_sort<64 * K, K, 64>(v);
    row_done<Use, K, 64>(u, r, u.rp[r], len, v, lane);
}

// The rows among the wave's RS_ROWS with more than `above` and at most W entries: 64 / W of them side by side in the wave, SETS such
// sets in flight.  order: LDS of the wave.
template <class Use, int W, int SETS>
__device__ __forceinline__ void short_rows(const Use &u, int r0, int above, int start_l, int len_l, int dst_l, int lane, int *order)
{
    constexpr int PER = 64 / W;
    const int part = lane / W, li = lane % W;
    const bool mine = len_l > above && len_l <= W;
    const unsigned long long rows = __builtin_amdgcn_ballot_w64(mine);
    const int count = __popcll(rows);
    if (count == 0) return;  // uniform
    wave_lds_sync();  // the order of the class before has been read
    if (mine) order[__builtin_amdgcn_mbcnt_hi(static_cast<uint32_t>(rows >> 32), __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(rows), 0u))] = lane;
    wave_lds_sync();
    for (int s0 = 0; s0 < count; s0 += PER * SETS) {
        int t[SETS], len[SETS], c[SETS], v[SETS];
#pragma unroll
        for (int p = 0; p < SETS; ++p) {
            const int at = s0 + p * PER + part;
            t[p] = order[min(at, count - 1)];
            const int st = __shfl(start_l, t[p], 64), ln = __shfl(len_l, t[p], 64);
            c[p] = __builtin_nontemporal_load(u.col_idx + st + min(li, ln - 1));
            len[p] = at < count ? ln : 0;
        }
#pragma unroll
        for (int p = 0; p < SETS; ++p) v[p] = u.map[lookup_index(c[p], u.n)];
#pragma unroll
        for (int p = 0; p < SETS; ++p) {
            if (s0 + p * PER >= count) break;  // uniform
            const bool in = li < len[p];
            int x[1] = {u.settle(c[p], v[p], in)};
            if (!in) x[0] = RS_NONE;
            if constexpr (Use::VOTES && W > 16) {
                // a label that more than half of a row's entries hold wins without any sorting; two of the entries are tried.
                // Labels settle after a few rounds and most rows pass then
                const int c0 = __shfl(x[0], lane & ~(W - 1), 64), c1 = __shfl(x[0], (lane & ~(W - 1)) + 7, 64);
                unsigned long long e0 = __builtin_amdgcn_ballot_w64(in && x[0] == c0), e1 = __builtin_amdgcn_ballot_w64(in && x[0] == c1);
                if constexpr (W == 32) {
                    e0 = lane < 32 ? e0 & 0xffffffffull : e0 >> 32;
                    e1 = lane < 32 ? e1 & 0xffffffffull : e1 >> 32;
                }
                const bool won0 = 2 * __popcll(e0) > len[p], won1 = 2 * __popcll(e1) > len[p];
                if (__builtin_amdgcn_ballot_w64(len[p] > 0 && !won0 && !won1) == 0ull) {
                    if (li == 0 && len[p] > 0) u.out[r0 + t[p]] = won0 ? c0 : c1;
                    continue;
                }
            }
            bitonic_sort<W, 1, W>(x);
            row_done<Use, 1, W>(u, r0 + t[p], __shfl(dst_l, t[p], 64), len[p], x, lane);
        }
    }
}

// Workgroups below `queue_blocks` take the rows of 65 to 1024 entries from the queues, one wave a row; the
// others take RS_ROWS consecutive rows per wave and sort the short ones among them: rows of at most 16 entries four at
// a time, of at most 32 two at a time, then those of 33 to 64; four sets in flight.
template <class Use>
__global__ __launch_bounds__(256, 6) void row_sort_kernel(Use u, RowQueues q, int queue_blocks)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (static_cast<int>(blockIdx.x) < queue_blocks) {
        const int first = blockIdx.x * 4 + wave, step = queue_blocks * 4;
        const int n1 = q.counts[1], n0 = q.counts[0];
        if constexpr (Use::VOTES) {  // the rows above RS_LDS collect their winner in q.best (row_sort_big_kernel)
            const int n3 = q.counts[3];
            for (int i = blockIdx.x * 256 + threadIdx.x; i < n3; i += queue_blocks * 256) q.best[i] = 0ull;
        }
        for (int i = first; i < n1; i += step) queued_row<Use, RS_LONG / 64>(u, q.rows[1][i], lane);
        for (int i = first; i < n0; i += step) queued_row<Use, RS_MID / 64>(u, q.rows[0][i], lane);
        return;
    }
    const int64_t r0 = (static_cast<int64_t>(blockIdx.x - queue_blocks) * 4 + wave) * RS_ROWS;
    if (r0 >= u.n) return;
    int start_l = 0, len_l = 0, dst_l = 0;
    const int r_l = static_cast<int>(r0) + lane;
    if (lane < RS_ROWS && r_l < u.n) {
        u.row(r_l, start_l, len_l);
        dst_l = u.rp[r_l];
        if constexpr (Use::VOTES) {
            if (len_l == 0) u.out[r_l] = u.map[r_l];  // a row without entries keeps its label
        }
    }
    __shared__ int order[4][RS_ROWS];
    short_rows<Use, 16, 4>(u, static_cast<int>(r0), 0, start_l, len_l, dst_l, lane, order[wave]);
    short_rows<Use, 32, 4>(u, static_cast<int>(r0), 16, start_l, len_l, dst_l, lane, order[wave]);
    short_rows<Use, 64, 4>(u, static_cast<int>(r0), 32, start_l, len_l, dst_l, lane, order[wave]);
}

// ---- rows above 1024 entries: a workgroup of 1024 threads ------------------------------------------------
constexpr int RS_NT = 1024;

// exclusive sum over the workgroup; every thread gets its prefix, *total the sum
__device__ __forceinline__ int group_exclusive_scan(int v, int *total, int *tmp)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int incl = wave_inclusive_scan(v);
    __syncthreads();  // tmp of a previous call is consumed
    if (lane == 63) tmp[wave] = incl;
    __syncthreads();
    int before = 0, all = 0;
#pragma unroll
    for (int w = 0; w < RS_NT / 64; ++w) {
        before += w < wave ? tmp[w] : 0;
        all += tmp[w];
    }
    *total = all;
    return before + incl - v;
}

// largest value over the workgroup, valid in thread 0
__device__ __forceinline__ unsigned long long group_max_u64(unsigned long long v, unsigned long long *tmp)
{
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) {
        const unsigned long long o = __shfl_xor(v, m, 64);
        v = o > v ? o : v;
    }
    __syncthreads();
    if ((threadIdx.x & 63) == 0) tmp[threadIdx.x >> 6] = v;
    __syncthreads();
    if (threadIdx.x == 0)
        for (int w = 1; w < RS_NT / 64; ++w) v = tmp[w] > v ? tmp[w] : v;
    return v;
}

// votes and label as one number whose maximum is the winner: most votes, then the smallest label
__device__ __forceinline__ unsigned long long ballot_of(int votes, int label)
{
    return (static_cast<unsigned long long>(static_cast<uint32_t>(votes)) << 32) | (0xffffffffu - static_cast<uint32_t>(label));
}

// 1025 .. 1024 K entries by 16 waves, K per lane (element i of the padded row in wave i / (64 K), register i / 64 % K, lane
// i % 64).  Every wave sorts its share in registers, then the shares are merged: only the steps whose partner sits in
// another wave go through LDS (ten of them, in two buffers taken in turn with one barrier each, or for K = 32 in one buffer with
// two), the rest stays in registers.
// A share that has to descend is sorted as its complement.  (All steps in LDS, 66 to 91
// barriers a row: the kernel takes 0.60 ms on the R-MAT graph, this way 0.26.)
template <class Use, int K>
__device__ __forceinline__ void group_row(const Use &u, int r, int start, int len, int *s, unsigned long long *tmp)
{
    constexpr int SHARE = 64 * K, ALL = RS_NT * K;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, base = wave * SHARE;
    int v[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int i = base + k * 64 + lane;
        v[k] = i < len ? __builtin_nontemporal_load(u.col_idx + start + i) : -1;
    }
#pragma unroll
    for (int k = 0; k < K; ++k) v[k] = base + k * 64 + lane < len ? u.value(v[k]) : RS_NONE;
    const int flip0 = (base & SHARE) ? -1 : 0;
#pragma unroll
    for (int k = 0; k < K; ++k) v[k] ^= flip0;
    bitonic_sort<SHARE, K, 64>(v);
#pragma unroll
    for (int k = 0; k < K; ++k) v[k] ^= flip0;
    __syncthreads();  // the row before is done with s
    int *buf = s;
    for (int size = 2 * SHARE; size <= ALL; size *= 2) {  // uniform
        const bool up = (base & size) == 0;
        for (int stride = size / 2; stride >= SHARE; stride /= 2) {
#pragma unroll
            for (int k = 0; k < K; ++k) buf[base + k * 64 + lane] = v[k];
            __syncthreads();
            const bool low = ((base & stride) == 0) == up;
#pragma unroll
            for (int k = 0; k < K; ++k) {
                const int o = buf[(base ^ stride) + k * 64 + lane];
                v[k] = low ? min(v[k], o) : max(v[k], o);
            }
            if constexpr (2 * ALL <= RS_WORDS) buf = buf == s ? s + ALL : s;  // the next step writes where nobody reads any more
            else __syncthreads();
        }
        const int flip = up ? 0 : -1;
#pragma unroll
        for (int k = 0; k < K; ++k) v[k] ^= flip;
        bitonic_stage<SHARE / 2, SHARE, K, 64>(v);
#pragma unroll
        for (int k = 0; k < K; ++k) v[k] ^= flip;
    }
    if constexpr (Use::VOTES) {
#pragma unroll
        for (int k = 0; k < K; ++k) buf[base + k * 64 + lane] = v[k];
        __syncthreads();
        unsigned long long best = 0ull;
        for (int i = threadIdx.x; i < len; i += RS_NT) {
            const int x = buf[i];
            if (i > 0 && buf[i - 1] == x) continue;
            int lo = i + 1, hi = len;  // first element of the next run
            while (lo < hi) {
                const int mid = (lo + hi) >> 1;
                if (buf[mid] == x) lo = mid + 1; else hi = mid;
            }
            const unsigned long long cand = ballot_of(lo - i, x);
            best = cand > best ? cand : best;
        }
        best = group_max_u64(best, tmp);
        if (threadIdx.x == 0) u.out[r] = static_cast<int>(0xffffffffu - static_cast<uint32_t>(best & 0xffffffffull));
    } else {
        const int dst = u.rp[r];
#pragma unroll
        for (int k = 0; k < K; ++k)
            if (base + k * 64 + lane < len) __builtin_nontemporal_store(v[k], u.out + dst + base + k * 64 + lane);
    }
}

template <class Use>
__device__ __forceinline__ void lds_row(const Use &u, int r, int *s, unsigned long long *tmp)
{
    int start, len;
    u.row(r, start, len);  // uniform
    if (len <= 2 * RS_NT) group_row<Use, 2>(u, r, start, len, s, tmp);
    else if (len <= 4 * RS_NT) group_row<Use, 4>(u, r, start, len, s, tmp);
    else if (len <= 8 * RS_NT) group_row<Use, 8>(u, r, start, len, s, tmp);
    else if (len <= 16 * RS_NT) group_row<Use, 16>(u, r, start, len, s, tmp);
    else group_row<Use, 32>(u, r, start, len, s, tmp);
}

__device__ __forceinline__ int pad_word(int i) { return i + (i >> 5); }  // a thread's 32 consecutive words on all banks

// more than RS_LDS entries, relabelling: the columns as bits, read back in ascending order.  false (uniform): a column
// occurs twice.
__device__ __forceinline__ bool bitmap_row(const Relabel &u, int r, uint32_t *bits, int *tmp, int *dup)
{
    int start, len;
    u.row(r, start, len);
    int dst = u.rp[r];
    for (int base = 0; base < u.n; base += 1 << RS_BITS_LOG2) {
        const int span = min(u.n - base, 1 << RS_BITS_LOG2);
        __syncthreads();
        for (int i = threadIdx.x; i < pad_word(1 << (RS_BITS_LOG2 - 5)); i += RS_NT) bits[i] = 0u;
        if (threadIdx.x == 0) *dup = 0;
        __syncthreads();
        bool twice = false;
        for (int i = threadIdx.x; i < len; i += RS_NT) {
            const int c = u.value(u.col_idx[start + i]) - base;
            if (c >= 0 && c < span) {
                const uint32_t m = 1u << (c & 31);
                twice = twice || (atomicOr(&bits[pad_word(c >> 5)], m) & m) != 0u;
            }
        }
        if (twice) *dup = 1;
        __syncthreads();
        if (*dup) return false;
        int mine = 0;
        const int w0 = threadIdx.x * 32;
        for (int w = 0; w < 32; ++w) mine += __popc(bits[pad_word(w0 + w)]);
        int total;
        int pos = dst + group_exclusive_scan(mine, &total, tmp);
        if (mine > 0)
            for (int w = 0; w < 32; ++w) {
                uint32_t b = bits[pad_word(w0 + w)];
                while (b) {
                    u.out[pos++] = base + (w0 + w) * 32 + __ffs(static_cast<int>(b)) - 1;
                    b &= b - 1;
                }
            }
        dst += total;
    }
    return true;
}

// counters of the values [base, base + RS_RANGE) of a row (values: looked up before, or NULL); returns the thread's number of
// smaller values
template <class Use>
__device__ __forceinline__ int count_range(const Use &u, const int *__restrict__ values, int start, int len, int base, int *cnt)
{
    __syncthreads();
    for (int i = threadIdx.x; i < pad_word(RS_RANGE); i += RS_NT) cnt[i] = 0;
    __syncthreads();
    int less = 0;
    for (int i = threadIdx.x; i < len; i += RS_NT) {
        const int c = (values ? values[start + i] : u.value(u.col_idx[start + i])) - base;
        if (c < 0) ++less;
        else if (c < RS_RANGE) atomicAdd(&cnt[pad_word(c)], 1);
    }
    __syncthreads();
    return less;
}

// The look-ups of the rows that are counted, once instead of in every pass: one workgroup a row, eight in flight a thread.
// *count rows in `rows`.
template <class Use>
__global__ __launch_bounds__(RS_NT) void long_row_values_kernel(Use u, const int *__restrict__ rows, const int *__restrict__ count,
                                                                int *__restrict__ values)
{
    const int n_rows = *count;
    for (int h = blockIdx.x; h < n_rows; h += gridDim.x) {
        int start, len;
        u.row(rows[h], start, len);
        for (int i0 = threadIdx.x; i0 < len; i0 += RS_NT * 8) {
            int c[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) c[k] = u.col_idx[start + min(i0 + k * RS_NT, len - 1)];
#pragma unroll
            for (int k = 0; k < 8; ++k) c[k] = u.value(c[k]);
#pragma unroll
            for (int k = 0; k < 8; ++k)
                if (i0 + k * RS_NT < len) values[start + i0 + k * RS_NT] = c[k];
        }
    }
}

template <class Use>
__global__ __launch_bounds__(RS_NT) void row_sort_big_kernel(Use u, RowQueues q)
{
    __shared__ int s[RS_WORDS];
    __shared__ unsigned long long tmp64[RS_NT / 64];
    __shared__ int tmp[RS_NT / 64];
    __shared__ int dup;
    const int n3 = q.counts[3], n2 = q.counts[2];
    if constexpr (Use::VOTES) {
        const int ranges = value_ranges(u.n);
        const int64_t tasks = static_cast<int64_t>(n3) * ranges;
        for (int64_t t = blockIdx.x; t < tasks; t += gridDim.x) {  // uniform
            const int h = static_cast<int>(t / ranges), base = static_cast<int>(t % ranges) * RS_RANGE;
            int start, len;
            u.row(q.rows[3][h], start, len);
            count_range(u, q.values, start, len, base, s);
            unsigned long long best = 0ull;
            for (int i = threadIdx.x; i < RS_RANGE; i += RS_NT) {
                const int votes = s[pad_word(i)];
                const unsigned long long cand = votes > 0 ? ballot_of(votes, base + i) : 0ull;
                best = cand > best ? cand : best;
            }
            best = group_max_u64(best, tmp64);
            if (threadIdx.x == 0 && best != 0ull) atomicMax(&q.best[h], best);
        }
    } else {
        for (int h = blockIdx.x; h < n3; h += gridDim.x) {
            const int r = q.rows[3][h];
            if (bitmap_row(u, r, reinterpret_cast<uint32_t *>(s), tmp, &dup)) continue;  // uniform
            if (many_ranges(u.n) && u.rp[r + 1] - u.rp[r] <= RS_LDS_MOST) lds_row(u, r, s, tmp64);
            else if (threadIdx.x == 0) q.dup_rows[atomicAdd(&q.counts[4], 1)] = r;
        }
    }
    for (int i = blockIdx.x; i < n2; i += gridDim.x) lds_row(u, q.rows[2][i], s, tmp64);
}

// long rows in which a column occurs more than once: counters instead of bits, one workgroup per row and range
__global__ __launch_bounds__(RS_NT) void row_sort_dup_kernel(Relabel u, RowQueues q)
{
    __shared__ int s[RS_WORDS];
    __shared__ int tmp[RS_NT / 64];
    const int ranges = value_ranges(u.n);
    const int64_t tasks = static_cast<int64_t>(q.counts[4]) * ranges;
    for (int64_t t = blockIdx.x; t < tasks; t += gridDim.x) {  // uniform
        const int r = q.dup_rows[t / ranges], base = static_cast<int>(t % ranges) * RS_RANGE;
        int start, len;
        u.row(r, start, len);
        const int less = count_range(u, q.values, start, len, base, s);
        int before;
        group_exclusive_scan(less, &before, tmp);
        int mine = 0;
        const int i0 = threadIdx.x * 32;
        for (int i = 0; i < 32; ++i) mine += s[pad_word(i0 + i)];
        int total;
        int pos = u.rp[r] + before + group_exclusive_scan(mine, &total, tmp);
        if (mine > 0)
            for (int i = 0; i < 32; ++i)
                for (int k = s[pad_word(i0 + i)]; k > 0; --k) u.out[pos++] = base + i0 + i;
    }
}

__global__ __launch_bounds__(256) void take_winners_kernel(RowQueues q, int *__restrict__ out)
{
    const int n3 = q.counts[3];
    for (int h = blockIdx.x * 256 + threadIdx.x; h < n3; h += gridDim.x * 256)
        out[q.rows[3][h]] = static_cast<int>(0xffffffffu - static_cast<uint32_t>(q.best[h] & 0xffffffffull));
}

// ---- launchers --------------------------------------------------------------------------------------------
// Queue capacities for nnz entries, in rows.
static int64_t queue_cap(int nnz, int longer_than) { return nnz / (longer_than + 1) + 1; }

size_t row_sort_ws(int n, int nnz)
{
    auto ints = [](int64_t k) { return align_up(static_cast<size_t>(k) * sizeof(int), 256); };
    return 256 + ints(queue_cap(nnz, RS_SHORT)) + ints(queue_cap(nnz, RS_MID)) + ints(queue_cap(nnz, RS_LONG)) +
           2 * ints(queue_cap(nnz, RS_LDS)) + align_up(static_cast<size_t>(queue_cap(nnz, RS_LDS)) * 8, 256) + ints(n) +
           (nnz > RS_LDS_MOST && many_ranges(n) ? ints(nnz) : 0);
}

static RowQueues carve(int n, int nnz, void *ws, int **labels)
{
    char *p = static_cast<char *>(ws);
    auto ints = [&](int64_t k) {
        int *a = reinterpret_cast<int *>(p);
        p += align_up(static_cast<size_t>(k) * sizeof(int), 256);
        return a;
    };
    RowQueues q;
    q.counts = ints(64);
    q.rows[0] = ints(queue_cap(nnz, RS_SHORT));
    q.rows[1] = ints(queue_cap(nnz, RS_MID));
    q.rows[2] = ints(queue_cap(nnz, RS_LONG));
    q.rows[3] = ints(queue_cap(nnz, RS_LDS));
    q.dup_rows = ints(queue_cap(nnz, RS_LDS));
    q.best = reinterpret_cast<unsigned long long *>(p);
    p += align_up(static_cast<size_t>(queue_cap(nnz, RS_LDS)) * 8, 256);
    *labels = ints(n);
    q.values = nnz > RS_LDS_MOST && many_ranges(n) ? ints(nnz) : nullptr;
    return q;
}

// clears the queue counters; labels: every node starts with its own id (NULL: none)
__global__ __launch_bounds__(256) void row_sort_begin_kernel(int n, int *__restrict__ counts, int *__restrict__ labels)
{
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i < 64) counts[i] = 0;
    if (labels && i < n) labels[i] = i;
}

struct RowSortGrid {
    int queue_blocks, blocks, big_blocks;
};

static RowSortGrid row_sort_grid(int n, int nnz)
{
    RowSortGrid g;
    const int64_t queued = queue_cap(nnz, RS_SHORT);
    g.queue_blocks = static_cast<int>((queued + 3) / 4 < 1024 ? (queued + 3) / 4 : 1024);
    g.blocks = g.queue_blocks + static_cast<int>((static_cast<int64_t>(n) + 4 * RS_ROWS - 1) / (4 * RS_ROWS));
    const int64_t big = queue_cap(nnz, RS_LONG);
    g.big_blocks = static_cast<int>(big < 256 ? big : 256);
    return g;
}

static void classify_rows(int n, const int *rp, int in_lds, const RowQueues &q, int *labels, hipStream_t s)
{
    hipLaunchKernelGGL(row_sort_begin_kernel, dim3(labels ? (n + 255) / 256 : 1), dim3(256), 0, s, n, q.counts, labels);
    hipLaunchKernelGGL(row_classes_kernel, dim3((n + 4095) / 4096), dim3(1024), 0, s, n, rp, in_lds, q);
}

// rp: row starts of the relabelled graph, complete before this on the stream; ws: row_sort_ws(n, nnz) bytes
int32_t launch_relabel_rows(const ftc_csr &g, const int *perm, const int *inv, const int *rp, int *col_idx_out, int *flag,
                            void *ws, hipStream_t s)
{
    int *unused;
    const RowQueues q = carve(g.n, g.nnz, ws, &unused);
    const RowSortGrid grid = row_sort_grid(g.n, g.nnz);
    const Relabel u{g.n, g.row_ptr, g.col_idx, perm, inv, rp, col_idx_out, flag};
    classify_rows(g.n, rp, RS_LDS, q, nullptr, s);
    if (g.nnz > RS_LONG) hipLaunchKernelGGL(row_sort_big_kernel<Relabel>, dim3(grid.big_blocks), dim3(RS_NT), 0, s, u, q);
    hipLaunchKernelGGL(row_sort_kernel<Relabel>, dim3(grid.blocks), dim3(256), 0, s, u, q, grid.queue_blocks);
    if (g.nnz > RS_LDS) {
        if (q.values)
            hipLaunchKernelGGL(long_row_values_kernel<Relabel>, dim3(grid.big_blocks), dim3(RS_NT), 0, s, u, q.dup_rows,
                               q.counts + 4, q.values);
        hipLaunchKernelGGL(row_sort_dup_kernel, dim3(grid.big_blocks), dim3(RS_NT), 0, s, u, q);
    }
    return launch_status("relabel rows");
}

// `labels` holds the labels after the last round; ws: row_sort_ws(n, nnz) bytes
int32_t launch_label_rounds(const ftc_csr &g, int iters, int *labels, void *ws, hipStream_t s)
{
    int *other;
    const RowQueues q = carve(g.n, g.nnz, ws, &other);
    const RowSortGrid grid = row_sort_grid(g.n, g.nnz);
    // the rounds alternate between the two arrays and end in `labels`
    int *from = iters % 2 == 0 ? labels : other, *to = iters % 2 == 0 ? other : labels;
    classify_rows(g.n, g.row_ptr, many_ranges(g.n) ? RS_LDS_MOST : RS_LDS, q, from, s);
    for (int it = 0; it < iters; ++it) {
        const Votes u{g.n, g.col_idx, from, g.row_ptr, to};
        hipLaunchKernelGGL(row_sort_kernel<Votes>, dim3(grid.blocks), dim3(256), 0, s, u, q, grid.queue_blocks);
        if (q.values)
            hipLaunchKernelGGL(long_row_values_kernel<Votes>, dim3(grid.big_blocks), dim3(RS_NT), 0, s, u, q.rows[3], q.counts + 3,
                               q.values);
        if (g.nnz > RS_LONG) hipLaunchKernelGGL(row_sort_big_kernel<Votes>, dim3(grid.big_blocks), dim3(RS_NT), 0, s, u, q);
        if (g.nnz > RS_LDS)
            hipLaunchKernelGGL(take_winners_kernel, dim3(static_cast<unsigned>((queue_cap(g.nnz, RS_LDS) + 255) / 256)),
                               dim3(256), 0, s, q, to);
        int *t = from;
        from = to;
        to = t;
    }
    return launch_status("label propagation");
}

}  // namespace ftc
