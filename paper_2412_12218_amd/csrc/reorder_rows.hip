// Row-wise kernels of the reordering step for graphs of at most ROW_SORT_NODES nodes: the relabelled graph and a
// round of label propagation both look every entry's column up in an array of n ints and need the results of ONE
// row in ascending order -- the new columns to write them out, the labels to find the longest run of equal ones.
// Rows are independent, so nothing is sorted across rows: a row is sorted where it fits,
//   at most 16 / 32 / 64        a quarter, half or whole wave, one entry per lane (bitonic, data-parallel-primitive moves),
//   at most 256 / 1024          a wave, 4 / 16 entries per lane,
//   at most 4096 / 8192         a workgroup of 256 / 1024 threads, in registers and LDS (see RS_GROUP_FEW),
//   longer                      a bitmap of the columns in LDS (relabelling; duplicates: counters, see below) or
//                               counters in LDS per 32 768 labels (label propagation); with more than 2^19 nodes those of
//                               at most 32 768 entries are sorted in LDS instead of counted (many_ranges()).
// What bounds them: the look-up.  Every entry is one 4-byte gather from an array that about fills an L2 (4 MB at
// a million nodes); the streams around it (column ids in, columns out) are read and written once, non-temporal.
// On the block model with a million nodes and 32 M entries a round of label propagation takes 0.21 ms (the first, without look-ups, 0.06,
// ten together 1.74: see vote_check_kernel) and the relabelled graph 0.33 ms (R-MAT, 2^20 nodes: 0.31); sorting all entries by label and row with the global radix sort took
// 4.0 and 4.1 ms.  The sorting network is the other half: with min, max and a selection per stage, rows of 33 to 64 two at a time,
// rows of any length below side by side in halves of the wave and each row's look-ups waiting for the one's before, a round took
// 0.24 ms (500 000 nodes with nine entries each, the whole plan: 1.39 / 1.01 ms).
// Larger graphs keep the radix sort: the counters of the long rows cost one pass over the row per 32 768 nodes.  Up to
// ROW_SORT_NODES the rows are ahead on every graph that was measured but for one kind: the relabelled graph where nearly all
// entries are in rows of more than 32 768 entries with repeated columns (2^22 nodes, 65 M entries, 95 % of them in rows of
// 60 000: 18 against 9 ms; half of them: 9.7 against 9.4; label propagation on the first: 16 ms a round on either).
#include "edge_ranges.hpp"
#include "entry_index.hpp"

namespace ftc {

constexpr int RS_ROWS = 32;         // consecutive rows per wave of the short-row part
constexpr int RS_SHORT = 64;        // longest row handled there; the queues hold the rows above
constexpr int RS_MID = 256, RS_LONG = 1024, RS_GROUP = 4096, RS_LDS = 8192;  // longest row of queues 0, 1, 2, 3; queue 4 has the rest
constexpr int RS_QUEUES = 5;
constexpr int RS_LDS_MOST = 32768;  // longest row of queue 3 in label propagation on many nodes (many_ranges())
constexpr int RS_RANGE = 32768;     // counters per pass over a long row
constexpr int RS_WORDS = RS_RANGE + RS_RANGE / 32;  // LDS words of the workgroups that take long rows
constexpr int RS_BITS_LOG2 = 20;    // columns per bitmap pass over a long row (32 768 words)
constexpr int VT_COUNTERS = 256;
// Up to this many rows in queue 2, the workgroups of the kernel of the longer ones, those above 2048 entries are sorted there, by 1024 threads: beside
// the short rows a workgroup of 256 needs 60 us for one, which a small graph waits for.  us, label propagation of ten rounds, always beside the
// short ones / by this line: R-MAT, 2^15 nodes, 10^6 entries (120 rows) 605 / 406, 2^17 nodes, 1.1 M (17) 617 / 422, 3.1 M (136) 789 / 690, 2^18 nodes, 4.2 M (153)
// 890 / 808; with 512 instead 2^20 nodes, 8.8 M (388) 2002 / 2042, with 1024 or for all rows of the queue 2^17 nodes, 6 M (816) 820 / 990.
constexpr int RS_GROUP_FEW = 256;
constexpr int RS_SHORT_ENTRIES = RS_QUEUES + 1;  // of RowQueues::counts: entries of the rows in no queue
constexpr int RS_NONE = 0x7fffffff; // sorts behind every column and label

// lengths of the rows: len[r] = rp[r + 1] - rp[r]; counts[q] rows of class q in rows[q]
struct RowQueues {
    int *counts;
    int *rows[RS_QUEUES];
    int *dup_rows;               // relabelling: long rows with duplicate columns, counts[RS_QUEUES] of them; label propagation:
                                 // ranges of every row of queue 4 that have been counted
    unsigned long long *best;    // label propagation: winner of every row of queue 4
    int *values;                 // what the columns of the counted rows become, at the place of the entry; NULL: not kept
};

// Passes over a row longer than queue 3's: counters for RS_RANGE of the n values each.
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
    __shared__ int cnt_s[RS_QUEUES], base_s[RS_QUEUES], short_s;
    if (threadIdx.x < RS_QUEUES) cnt_s[threadIdx.x] = 0;
    if (threadIdx.x == 0) short_s = 0;
    __syncthreads();
    int cls[PER], pos[PER], in_short = 0;
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        const int64_t r = (static_cast<int64_t>(blockIdx.x) * PER + k) * 1024 + threadIdx.x;
        const int len = r < n ? rp[r + 1] - rp[r] : 0;
        cls[k] = len <= RS_SHORT ? -1 : len <= RS_MID ? 0 : len <= RS_LONG ? 1 : len <= RS_GROUP ? 2 : len <= in_lds ? 3 : 4;
        pos[k] = cls[k] >= 0 ? atomicAdd(&cnt_s[cls[k]], 1) : 0;
        in_short += cls[k] < 0 ? len : 0;
    }
    in_short = wave_inclusive_scan(in_short);
    if ((threadIdx.x & 63) == 63) atomicAdd(&short_s, in_short);
    __syncthreads();
    if (threadIdx.x == 0 && short_s > 0) atomicAdd(&q.counts[RS_SHORT_ENTRIES], short_s);
    if (threadIdx.x < RS_QUEUES && cnt_s[threadIdx.x] > 0) base_s[threadIdx.x] = atomicAdd(&q.counts[threadIdx.x], cnt_s[threadIdx.x]);
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
    static constexpr bool VOTES = false, FIRST = false;
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
    __device__ __forceinline__ int look(int c) const { return map[lookup_index(c, n)]; }
    __device__ __forceinline__ int value(int c) const { return settle(c, look(c), true); }
};
constexpr int VT_BITS_LOG2 = 20;
constexpr float VT_MOST = 0.6f;
// Only rows of at most RS_SHORT entries are left out (see vote_check_kernel): worth looking for where three quarters of the entries are in these
// (see VT_FROM; 10^6 nodes, 60 entries each, 0.66 3631 / 3513 us always looking, power law with 0.72 1393 / 1577).
__host__ __device__ inline bool short_rows_count(int in_short, int nnz) { return static_cast<int64_t>(in_short) * 4 >= static_cast<int64_t>(nnz) * 3; }
// FIRST: the first round, in which every node's label is its own id and nothing is looked up.
template <bool FIRST_ROUND>
struct Votes {
    static constexpr bool VOTES = true, FIRST = FIRST_ROUND;
    int n;
    const int *col_idx, *map, *rp;  // map: labels of the round before
    int *out;                       // labels of this round
    uint32_t *changed;              // bit r >> shift of every row r whose label is another than before is set; NULL: not kept
    int *changes;                   // .. and counted, spread over VT_COUNTERS
    int shift;
    int nnz;
    const uint32_t *todo;           // rows of at most RS_SHORT entries that may change, a bit each; NULL: all
    __device__ __forceinline__ void row(int r, int &start, int &len) const
    {
        start = rp[r];
        len = rp[r + 1] - start;
    }
    __device__ __forceinline__ int settle(int c, int v, bool) const { return c >= 0 && c < n ? v : 0; }  // out of range: a vote for label 0
    __device__ __forceinline__ int look(int c) const
    {
        if constexpr (FIRST) return c;
        else return map[lookup_index(c, n)];
    }
    __device__ __forceinline__ int value(int c) const { return settle(c, look(c), true); }
    __device__ __forceinline__ int before(int r) const
    {
        if constexpr (FIRST) return r;
        else return map[r];
    }
    // one row's winner, by one lane
    __device__ __forceinline__ void vote(int r, int w) const
    {
        out[r] = w;
        if (changed && before(r) != w) {
            atomicOr(&changed[(r >> shift) >> 5], 1u << ((r >> shift) & 31));
            atomicAdd(&changes[r & (VT_COUNTERS - 1)], 1);
        }
    }
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
        if (li == 0 && len > 0) u.vote(r, w);
    } else {
#pragma unroll
        for (int k = 0; k < K; ++k)
            if (k * 64 + li < len) __builtin_nontemporal_store(v[k], u.out + dst + k * 64 + li);
    }
}

// one row of a queue by one wave, K entries per lane
template <class Use, int K>
__device__ __forceinline__ void queued_row(const Use &u, int r, int start, int len, int lane)
{
    int c[K], v[K];
#pragma unroll
    for (int k = 0; k < K; ++k) c[k] = __builtin_nontemporal_load(u.col_idx + start + min(k * 64 + lane, len - 1));  // (no queued row is empty)
#pragma unroll
    for (int k = 0; k < K; ++k) v[k] = u.look(c[k]);
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
// sets in flight.  order, win: LDS of the wave; votes: win[r - r0] becomes the winner of row r.  Which rows a set holds is scalar work for
// sets of one or two, and the winners leave in one store for all rows: through LDS, cross-lane moves and a store per row a round without
// look-ups took 79 us, this way 64, one with look-ups 217 / 211 (block model with 10^6 nodes, 32 M entries).
template <class Use, int W, int SETS>
__device__ __forceinline__ void short_rows(const Use &u, int r0, int above, int start_l, int len_l, int dst_l, int lane, int *order, int *win)
{
    constexpr int PER = 64 / W;
    const int part = lane / W, li = lane % W;
    const bool mine = len_l > above && len_l <= W;
    uint32_t left = static_cast<uint32_t>(__builtin_amdgcn_ballot_w64(mine));  // rows that are not in a set yet
    const int count = __popc(left);
    if (count == 0) return;  // uniform
    if constexpr (PER > 2) {
        wave_lds_sync();  // the order of the class before has been read
        if (mine) order[__popc(left & ((1u << lane) - 1u))] = lane;
        wave_lds_sync();
    }
    int last = 0;
    auto next_row = [&](int &st, int &ln, int &dst, bool &ok) {  // beyond the last row that one's
        ok = left != 0u;
        if (ok) last = __ffs(static_cast<int>(left)) - 1;
        left &= left - 1u;
        st = __builtin_amdgcn_readlane(start_l, last);
        ln = __builtin_amdgcn_readlane(len_l, last);
        dst = Use::VOTES ? 0 : __builtin_amdgcn_readlane(dst_l, last);
        return last;
    };
    for (int s0 = 0; s0 < count; s0 += PER * SETS) {
        int t[SETS], len[SETS], c[SETS], v[SETS], dst[SETS];
#pragma unroll
        for (int p = 0; p < SETS; ++p) {
            int st, ln;
            bool ok;
            if constexpr (PER == 1) {
                t[p] = next_row(st, ln, dst[p], ok);
            } else if constexpr (PER == 2) {
                int st1, ln1, dst1;
                bool ok1;
                const int t0 = next_row(st, ln, dst[p], ok), t1 = next_row(st1, ln1, dst1, ok1);
                t[p] = part ? t1 : t0;
                st = part ? st1 : st;
                ln = part ? ln1 : ln;
                dst[p] = part ? dst1 : dst[p];
                ok = part ? ok1 : ok;
            } else {
                const int at = s0 + p * PER + part;
                ok = at < count;
                t[p] = order[min(at, count - 1)];
                st = __shfl(start_l, t[p], 64);
                ln = __shfl(len_l, t[p], 64);
                dst[p] = Use::VOTES ? 0 : __shfl(dst_l, t[p], 64);
            }
            c[p] = __builtin_nontemporal_load(u.col_idx + st + min(li, ln - 1));
            len[p] = ok ? ln : 0;
        }
#pragma unroll
        for (int p = 0; p < SETS; ++p) v[p] = u.look(c[p]);
#pragma unroll
        for (int p = 0; p < SETS; ++p) {
            if (s0 + p * PER >= count) break;  // uniform
            const bool in = li < len[p];
            int x[1] = {u.settle(c[p], v[p], in)};
            if (!in) x[0] = RS_NONE;
            if constexpr (Use::FIRST) {
                // distinct columns in ascending order have a vote each, and the first is the smallest
                const int prev = __builtin_amdgcn_update_dpp(0, x[0], 0x138, 0xf, 0xf, false);  // wave_shr:1
                if (__builtin_amdgcn_ballot_w64(in && li > 0 && x[0] <= prev) == 0ull) {
                    if (li == 0 && len[p] > 0) win[t[p]] = x[0];
                    continue;
                }
            } else if constexpr (Use::VOTES && W > 16) {
                // a label that more than half of a row's entries hold wins without any sorting; two of the entries are tried.
                // Labels settle after a few rounds and most rows pass then
                int c0 = __builtin_amdgcn_readlane(x[0], 0), c1 = __builtin_amdgcn_readlane(x[0], 7);
                if constexpr (W == 32) {
                    const int d0 = __builtin_amdgcn_readlane(x[0], 32), d1 = __builtin_amdgcn_readlane(x[0], 39);
                    c0 = part ? d0 : c0;
                    c1 = part ? d1 : c1;
                }
                unsigned long long e0 = __builtin_amdgcn_ballot_w64(in && x[0] == c0), e1 = __builtin_amdgcn_ballot_w64(in && x[0] == c1);
                if constexpr (W == 32) {
                    e0 = lane < 32 ? e0 & 0xffffffffull : e0 >> 32;
                    e1 = lane < 32 ? e1 & 0xffffffffull : e1 >> 32;
                }
                const bool won0 = 2 * __popcll(e0) > len[p], won1 = 2 * __popcll(e1) > len[p];
                if (__builtin_amdgcn_ballot_w64(len[p] > 0 && !won0 && !won1) == 0ull) {
                    if (li == 0 && len[p] > 0) win[t[p]] = won0 ? c0 : c1;
                    continue;
                }
            }
            bitonic_sort<W, 1, W>(x);
            if constexpr (Use::VOTES) {
                const int w = longest_run<1, W>(x, len[p], lane);
                if (li == 0 && len[p] > 0) win[t[p]] = w;
            } else row_done<Use, 1, W>(u, r0 + t[p], dst[p], len[p], x, lane);
        }
    }
}

// ---- rows above 1024 entries: a workgroup of 256 (up to RS_GROUP entries) or 1024 threads ---------------------
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

// largest value over a workgroup of NT threads, valid in thread 0
template <int NT>
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
        for (int w = 1; w < NT / 64; ++w) v = tmp[w] > v ? tmp[w] : v;
    return v;
}

// votes and label as one number whose maximum is the winner: most votes, then the smallest label
__device__ __forceinline__ unsigned long long ballot_of(int votes, int label)
{
    return (static_cast<unsigned long long>(static_cast<uint32_t>(votes)) << 32) | (0xffffffffu - static_cast<uint32_t>(label));
}

// At most NT K entries by NT / 64 waves, K per lane (element i of the padded row in wave i / (64 K), register i / 64 % K, lane
// i % 64).  Every wave sorts its share in registers, then the shares are merged: only the steps whose partner sits in
// another wave go through LDS (ten of them, in two buffers taken in turn with one barrier each, or for K = 32 in one buffer with
// two), the rest stays in registers.
// A share that has to descend is sorted as its complement.  (All steps in LDS, 66 to 91
// barriers a row: 0.60 ms on the R-MAT graph, this way 0.26; rows of up to 4096 entries by four waves beside the shorter rows instead of by
// sixteen, alone on a compute unit, after them: relabelled R-MAT graph 0.46 / 0.37 ms, ten rounds of label propagation 6.5 / 4.8.)
template <class Use, int K, int NT, int BUF>
__device__ __forceinline__ void group_row(const Use &u, int r, int start, int len, int *s, unsigned long long *tmp)
{
    constexpr int SHARE = 64 * K, ALL = NT * K;
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
            if constexpr (2 * ALL <= BUF) buf = buf == s ? s + ALL : s;  // the next step writes where nobody reads any more
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
        for (int i = threadIdx.x; i < len; i += NT) {
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
        best = group_max_u64<NT>(best, tmp);
        if (threadIdx.x == 0) u.vote(r, static_cast<int>(0xffffffffu - static_cast<uint32_t>(best & 0xffffffffull)));
    } else {
        const int dst = u.rp[r];
#pragma unroll
        for (int k = 0; k < K; ++k)
            if (base + k * 64 + lane < len) __builtin_nontemporal_store(v[k], u.out + dst + base + k * 64 + lane);
    }
}

// entries first, first + step, .. of a row looked up, eight in flight a thread
template <class Use>
__device__ __forceinline__ void look_up_row(const Use &u, int start, int len, int first, int step, int *__restrict__ values)
{
    for (int64_t i0 = first; i0 < len; i0 += static_cast<int64_t>(step) * 8) {
        int c[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) c[k] = u.col_idx[start + min(i0 + static_cast<int64_t>(k) * step, static_cast<int64_t>(len - 1))];
#pragma unroll
        for (int k = 0; k < 8; ++k) c[k] = u.value(c[k]);
#pragma unroll
        for (int k = 0; k < 8; ++k)
            if (i0 + static_cast<int64_t>(k) * step < len) values[start + i0 + static_cast<int64_t>(k) * step] = c[k];
    }
}

// Workgroups below `queue_blocks` take the rows of 65 to 4096 entries from the queues, those of 1025 and more one at a time, the
// others one per wave; the
// others take RS_ROWS consecutive rows per wave and sort the short ones among them: rows of at most 16 entries four at
// a time, of at most 32 two at a time, then those of 33 to 64; four sets in flight.
template <class Use>
__global__ __launch_bounds__(256, 6) void row_sort_kernel(Use u, RowQueues q, int queue_blocks)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (static_cast<int>(blockIdx.x) < queue_blocks) {
        const int n2 = q.counts[2], longest = n2 > RS_GROUP_FEW ? RS_GROUP : RS_GROUP / 2, n1 = q.counts[1], n0 = q.counts[0];
        // each class of rows begins with the workgroup (wave) after the last one of the class before, which was the longer one (ten rounds of label
        // propagation, R-MAT, 2^15 nodes 427 / 406 us, 2^16 nodes, 553 000 entries 337 / 314)
        const int first = static_cast<int>((blockIdx.x + queue_blocks - n2 % queue_blocks) % queue_blocks) * 4 + wave, step = queue_blocks * 4;
        if constexpr (Use::VOTES) {  // the rows that are counted collect their winner in q.best (row_sort_big_kernel)
            const int n4 = q.counts[4];
            for (int i = blockIdx.x * 256 + threadIdx.x; i < n4; i += queue_blocks * 256) {
                q.best[i] = 0ull;
                q.dup_rows[i] = 0;
            }
            // what they are looked up to, once for all passes, the workgroups spread over the rows
            const int parts = n4 > 0 ? max(queue_blocks / n4, 1) : 0;
            for (int h = n4 > 0 ? blockIdx.x % min(n4, queue_blocks) : 0; q.values && h < n4; h += queue_blocks) {
                const int part = blockIdx.x / min(n4, queue_blocks);
                if (part >= parts) break;
                int start, len;
                u.row(q.rows[4][h], start, len);
                look_up_row(u, start, len, part * 256 + threadIdx.x, parts * 256, q.values);
            }
        }
        __shared__ int s[RS_GROUP];
        __shared__ unsigned long long tmp64[4];
        for (int i = blockIdx.x; i < n2; i += queue_blocks) {  // uniform
            const int r = q.rows[2][i];
            int start, len;
            u.row(r, start, len);
            if (len <= RS_GROUP / 2) group_row<Use, RS_GROUP / 512, 256, RS_GROUP>(u, r, start, len, s, tmp64);
            else if (len <= longest) group_row<Use, RS_GROUP / 256, 256, RS_GROUP>(u, r, start, len, s, tmp64);
        }
        // the network of half the size costs 0.4 of the whole one, and most rows of a class need no more (all in whole ones: relabelled R-MAT
        // graph 0.30 ms of this kernel for 0.25, ten rounds of label propagation 4.8 for 4.2)
        for (int i = first; i < n1; i += step) {
            const int r = q.rows[1][i];
            int start, len;
            u.row(r, start, len);
            if (len <= RS_LONG / 2) queued_row<Use, RS_LONG / 128>(u, r, start, len, lane);
            else queued_row<Use, RS_LONG / 64>(u, r, start, len, lane);
        }
        const int first0 = (first + step - n1 % step) % step;
        for (int i = first0; i < n0; i += step) {
            const int r = q.rows[0][i];
            int start, len;
            u.row(r, start, len);
            if (len <= RS_MID / 2) queued_row<Use, RS_MID / 128>(u, r, start, len, lane);
            else queued_row<Use, RS_MID / 64>(u, r, start, len, lane);
        }
        return;
    }
    const int64_t r0 = (static_cast<int64_t>(blockIdx.x - queue_blocks) * 4 + wave) * RS_ROWS;
    if (r0 >= u.n) return;
    bool kept = false;  // votes: the rows whose label is another than before are
    if constexpr (Use::VOTES) kept = u.changed && short_rows_count(q.counts[RS_SHORT_ENTRIES], u.nnz);
    int start_l = 0, len_l = 0, dst_l = 0, old_l = 0;
    bool short_row = false;  // votes: this lane's row is decided here
    const int r_l = static_cast<int>(r0) + lane;
    if (lane < RS_ROWS && r_l < u.n) {
        u.row(r_l, start_l, len_l);
        dst_l = u.rp[r_l];
        if constexpr (Use::VOTES) {
            old_l = u.before(r_l);
            short_row = len_l <= RS_SHORT;
            if (u.todo && short_row && !(u.todo[r0 >> 5] >> lane & 1u)) len_l = 0;  // nothing in the row has changed
        }
    }
    __shared__ int order[4][RS_ROWS], win[4][RS_ROWS];
    static_assert(RS_ROWS == 32, "a word of u.todo and of u.changed, of the masks in short_rows()");
    short_rows<Use, 16, 4>(u, static_cast<int>(r0), 0, start_l, len_l, dst_l, lane, order[wave], win[wave]);
    short_rows<Use, 32, 4>(u, static_cast<int>(r0), 16, start_l, len_l, dst_l, lane, order[wave], win[wave]);
    short_rows<Use, 64, 4>(u, static_cast<int>(r0), 32, start_l, len_l, dst_l, lane, order[wave], win[wave]);
    if constexpr (Use::VOTES) {
        wave_lds_sync();
        // a row that has no entries, or none that changed, keeps its label
        const int w = len_l > 0 ? win[wave][lane & (RS_ROWS - 1)] : old_l;
        if (short_row) u.out[r_l] = w;
        if (!kept) return;
        const uint32_t m = static_cast<uint32_t>(__builtin_amdgcn_ballot_w64(short_row && w != old_l));
        const int first = static_cast<int>(r0) >> u.shift;  // the 32 >> shift bits of these rows lie in one word
        uint32_t bits = 0u;
        if (u.shift == 0) bits = m;
        else
            for (uint32_t b = m; b; b &= b - 1u) bits |= 1u << (((__ffs(static_cast<int>(b)) - 1) >> u.shift) + (first & 31));
        if (lane == 0 && m) {
            atomicOr(&u.changed[first >> 5], bits);
            atomicAdd(&u.changes[(r0 >> 5) & (VT_COUNTERS - 1)], __popc(m));
        }
    }
}

template <class Use>
__device__ __forceinline__ void lds_row(const Use &u, int r, int *s, unsigned long long *tmp)
{
    int start, len;
    u.row(r, start, len);  // uniform
    if (len <= 4 * RS_NT) group_row<Use, 4, RS_NT, RS_WORDS>(u, r, start, len, s, tmp);
    else if (len <= 8 * RS_NT) group_row<Use, 8, RS_NT, RS_WORDS>(u, r, start, len, s, tmp);
    else if (len <= 16 * RS_NT) group_row<Use, 16, RS_NT, RS_WORDS>(u, r, start, len, s, tmp);
    else group_row<Use, 32, RS_NT, RS_WORDS>(u, r, start, len, s, tmp);
}

__device__ __forceinline__ int pad_word(int i) { return i + (i >> 5); }  // a thread's 32 consecutive words on all banks

// more than RS_LDS entries, relabelling: the columns as bits, read back in ascending order.  false (uniform): a column
// occurs twice.
__device__ __forceinline__ bool bitmap_row(const Relabel &u, int r, uint32_t *bits, int *tmp, int *piece, int *dup)
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
        for (uint32_t i0 = threadIdx.x; entry_in(i0, len); i0 += RS_NT * 8) {  // eight look-ups in flight
            int c[8], v[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) c[k] = u.col_idx[start + entry_or_last(i0 + k * RS_NT, len)];
#pragma unroll
            for (int k = 0; k < 8; ++k) v[k] = u.look(c[k]);
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                const int x = u.settle(c[k], v[k], true) - base;
                if (entry_in(i0 + k * RS_NT, len) && x >= 0 && x < span) {
                    const uint32_t m = 1u << (x & 31);
                    twice = twice || (atomicOr(&bits[pad_word(x >> 5)], m) & m) != 0u;
                }
            }
        }
        if (twice) *dup = 1;
        __syncthreads();
        if (*dup) return false;
        // 64 words at a time by a wave, a word a lane: the columns of a row can all lie close together, and a wave's words are as full
        // as each other (32 words in a row by one thread: 74 us for the 211 rows of the R-MAT graph, this way 59)
        constexpr int PIECES = 1 << (RS_BITS_LOG2 - 11), WAVES = RS_NT / 64;
        const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
        for (int p = wave; p < PIECES; p += WAVES) {
            const int incl = wave_inclusive_scan(__popc(bits[pad_word(p * 64 + lane)]));
            if (lane == 63) piece[p] = incl;
        }
        __syncthreads();
        int total;
        const int before = group_exclusive_scan(threadIdx.x < PIECES ? piece[threadIdx.x] : 0, &total, tmp);
        if (threadIdx.x < PIECES) piece[threadIdx.x] = dst + before;
        __syncthreads();
        for (int p = wave; p < PIECES; p += WAVES) {
            uint32_t b = bits[pad_word(p * 64 + lane)];
            const int mine = __popc(b);
            int pos = piece[p] + wave_inclusive_scan(mine) - mine;
            while (b) {
                u.out[pos++] = base + (p * 64 + lane) * 32 + __ffs(static_cast<int>(b)) - 1;
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
    for (uint32_t i = threadIdx.x; entry_in(i, len); i += RS_NT) {
        const int c = (values ? values[start + i] : u.value(u.col_idx[start + i])) - base;
        if (c < 0) ++less;
        else if (c < RS_RANGE) atomicAdd(&cnt[pad_word(c)], 1);
    }
    __syncthreads();
    return less;
}

// The look-ups of the relabelled rows that are counted, once instead of in every pass: one workgroup a row.  *count rows in `rows`.
__global__ __launch_bounds__(RS_NT) void long_row_values_kernel(Relabel u, const int *__restrict__ rows, const int *__restrict__ count,
                                                                int *__restrict__ values)
{
    const int n_rows = *count;
    for (int h = blockIdx.x; h < n_rows; h += gridDim.x) {
        int start, len;
        u.row(rows[h], start, len);
        look_up_row(u, start, len, threadIdx.x, RS_NT, values);
    }
}

template <class Use>
__global__ __launch_bounds__(RS_NT) void row_sort_big_kernel(Use u, RowQueues q)
{
    __shared__ int s[RS_WORDS];
    __shared__ unsigned long long tmp64[RS_NT / 64];
    __shared__ int tmp[RS_NT / 64];
    __shared__ int dup;
    const int n4 = q.counts[4], n3 = q.counts[3], n2 = q.counts[2], n32 = n3 + (n2 <= RS_GROUP_FEW ? n2 : 0);
    if (n4 + n32 == 0) return;  // uniform over the grid
    if constexpr (Use::VOTES) {
        const int ranges = value_ranges(u.n);
        const int64_t tasks = static_cast<int64_t>(n4) * ranges;
        for (int64_t t = blockIdx.x; t < tasks; t += gridDim.x) {  // uniform
            const int h = static_cast<int>(t / ranges), base = static_cast<int>(t % ranges) * RS_RANGE;
            int start, len;
            u.row(q.rows[4][h], start, len);
            count_range(u, q.values, start, len, base, s);
            unsigned long long best = 0ull;
            for (int i = threadIdx.x; i < RS_RANGE; i += RS_NT) {
                const int votes = s[pad_word(i)];
                const unsigned long long cand = votes > 0 ? ballot_of(votes, base + i) : 0ull;
                best = cand > best ? cand : best;
            }
            best = group_max_u64<RS_NT>(best, tmp64);
            if (threadIdx.x == 0) {  // the last of the row's ranges takes the winner
                if (best != 0ull) atomicMax(&q.best[h], best);
                __threadfence();
                if (atomicAdd(&q.dup_rows[h], 1) == ranges - 1)
                    u.vote(q.rows[4][h], static_cast<int>(0xffffffffu - static_cast<uint32_t>(atomicMax(&q.best[h], 0ull) & 0xffffffffull)));
            }
        }
    } else {
        __shared__ int piece[1 << (RS_BITS_LOG2 - 11)];
        for (int h = blockIdx.x; h < n4; h += gridDim.x) {
            const int r = q.rows[4][h];
            if (bitmap_row(u, r, reinterpret_cast<uint32_t *>(s), tmp, piece, &dup)) continue;  // uniform
            if (many_ranges(u.n) && u.rp[r + 1] - u.rp[r] <= RS_LDS_MOST) lds_row(u, r, s, tmp64);
            else if (threadIdx.x == 0) q.dup_rows[atomicAdd(&q.counts[RS_QUEUES], 1)] = r;
        }
    }
    // the classes begin with the workgroup after the last one above: a row a workgroup where there are few (2^17 nodes, 2.6 M entries, one row
    // counted in four parts, 17 of up to 8192 entries: 38 / 26 us a round)
    const int grid = gridDim.x;
    const int end4 = static_cast<int>((Use::VOTES ? static_cast<int64_t>(n4) * value_ranges(u.n) : n4) % grid);
    for (int i = (static_cast<int>(blockIdx.x) + grid - end4) % grid; i < n32; i += grid) {
        const int r = i < n3 ? q.rows[3][i] : q.rows[2][i - n3];
        int start, len;
        u.row(r, start, len);
        if (len > RS_GROUP / 2) lds_row(u, r, s, tmp64);
    }
}

// long rows in which a column occurs more than once: counters instead of bits, one workgroup per row and range
__global__ __launch_bounds__(RS_NT) void row_sort_dup_kernel(Relabel u, RowQueues q)
{
    __shared__ int s[RS_WORDS];
    __shared__ int tmp[RS_NT / 64];
    const int ranges = value_ranges(u.n);
    const int64_t tasks = static_cast<int64_t>(q.counts[RS_QUEUES]) * ranges;
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

// ---- label propagation: rows that may change ---------------------------------------------------------------
// After some rounds few labels change, and a row none of whose columns has changed keeps its label: it is not voted on again.
// Which rows these are takes a bit per column and no look-up in memory: the bits of the nodes that changed in the round before fit
// into LDS (up to 2^20 nodes one each, above one for two or four nodes in a row).  Bound by reading the column ids.  Where most
// rows would be left (the changed share times the mean number of entries above VT_MOST) all of them are, at once.
// On the block model with a million nodes, 32 M entries, a check that leaves rows out takes 50 us, one that doesn't 5; the ninth and the
// tenth round take 37 and 25 us after it instead of 210.

__global__ __launch_bounds__(RS_NT) void vote_check_kernel(int n, int nnz, const int *__restrict__ in_short, const int *__restrict__ rp, const int *__restrict__ col_idx,
                                                           const uint32_t *__restrict__ changed, const int *__restrict__ changes,
                                                           uint32_t *__restrict__ next_changed, int *__restrict__ next_changes, int shift,
                                                           uint32_t *__restrict__ todo)
{
    constexpr int WAVES = RS_NT / 64, U = 8;
    __shared__ uint32_t bits[1 << (VT_BITS_LOG2 - 5)];
    __shared__ int starts[WAVES][65], tmp[WAVES];
    __shared__ uint32_t hit[WAVES][2];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int words = (((n - 1) >> shift) >> 5) + 1, todo_words = (n + 31) / 32;
    const int thread = blockIdx.x * RS_NT + threadIdx.x, threads = gridDim.x * RS_NT;
    const bool worth = short_rows_count(*in_short, nnz);  // this and the next are uniform over the grid
    for (int i = thread; i < words; i += threads) next_changed[i] = 0u;
    if (thread < VT_COUNTERS) next_changes[thread] = 0;
    int total;
    group_exclusive_scan(threadIdx.x < VT_COUNTERS ? changes[threadIdx.x] : 0, &total, tmp);
    if (!worth || static_cast<float>(total) * static_cast<float>(nnz) > VT_MOST * static_cast<float>(n) * static_cast<float>(n)) {
        for (int i = thread; i < todo_words; i += threads) todo[i] = ~0u;
        return;
    }
    for (int i = threadIdx.x; i < words; i += RS_NT) bits[i] = changed[i];
    __syncthreads();  // (none below)
    auto has_changed = [&](int c) {
        const unsigned b = static_cast<unsigned>(lookup_index(c, n)) >> shift;
        return c >= 0 && c < n && (bits[b >> 5] >> (b & 31u) & 1u);
    };
    for (int64_t r0 = (static_cast<int64_t>(blockIdx.x) * WAVES + wave) * 64; r0 < n; r0 += static_cast<int64_t>(gridDim.x) * WAVES * 64) {
        const int r = static_cast<int>(min(r0 + lane, static_cast<int64_t>(n)));
        const int st = rp[r], len = rp[min(r + 1, n)] - st;
        wave_lds_sync();
        starts[wave][lane] = st;
        if (lane == 63) starts[wave][64] = st + len;
        if (lane < 2) hit[wave][lane] = 0u;
        wave_lds_sync();
        if (__builtin_amdgcn_ballot_w64(len > RS_SHORT) == 0ull) {  // the entries of all 64 rows in one go
            const int end = starts[wave][64];
            for (uint32_t e0 = starts[wave][0]; entry_in(e0, end); e0 += 64 * U) {
                int c[U];
#pragma unroll
                for (int k = 0; k < U; ++k) c[k] = __builtin_nontemporal_load(col_idx + entry_or_last(e0 + k * 64 + lane, end));
#pragma unroll
                for (int k = 0; k < U; ++k) {
                    if (entry_in(e0 + k * 64 + lane, end) && has_changed(c[k])) {
                        const int e = static_cast<int>(e0) + k * 64 + lane;
                        int t = 0;  // the last of the 64 rows that begins at or before e
#pragma unroll
                        for (int h = 32; h > 0; h /= 2) t += starts[wave][t + h] <= e ? h : 0;
                        atomicOr(&hit[wave][t >> 5], 1u << (t & 31));
                    }
                }
            }
        } else {  // longer rows, which are voted on in any case, are left out: row by row, U rows in flight
            for (int t0 = 0; t0 < 64; t0 += U) {
                int c[U], ln[U];
#pragma unroll
                for (int k = 0; k < U; ++k) {
                    const int s = __shfl(st, t0 + k, 64);
                    ln[k] = __shfl(len, t0 + k, 64);
                    if (ln[k] > RS_SHORT) ln[k] = 0;
                    c[k] = col_idx[max(min(s + min(lane, ln[k] - 1), nnz - 1), 0)];
                }
#pragma unroll
                for (int k = 0; k < U; ++k)
                    if (__builtin_amdgcn_ballot_w64(lane < ln[k] && has_changed(c[k])) != 0ull && lane == 0)
                        atomicOr(&hit[wave][(t0 + k) >> 5], 1u << ((t0 + k) & 31));
            }
        }
        wave_lds_sync();
        if (lane < 2 && (r0 >> 5) + lane < todo_words) todo[(r0 >> 5) + lane] = hit[wave][lane];
    }
}

// ---- launchers --------------------------------------------------------------------------------------------
// Queue capacities for nnz entries, in rows.
static int64_t queue_cap(int nnz, int longer_than) { return nnz / (longer_than + 1) + 1; }

// Label propagation looks for the rows that may change from this many entries on: a launch more a round (5 us) against the share of
// a round (6.5 us a million entries) that the last ones save, which depends on the graph.  Ten rounds, never / always, us: uniform 10^6 nodes, 5.0 M entries 399 / 389,
// 8.9 M 570 / 486, 250 000 nodes, 8.2 M 580 / 602, 500 000 nodes, 12.4 M 807 / 838, 10^6 nodes, 12.9 M 830 / 609, 16.8 M 1086 / 757, 32.7 M 2004 / 2038, 2 10^6 nodes, 29.7 M
// 2518 / 1508; blocks 10^6 nodes, 8.8 M 566 / 649, 12.8 M 820 / 855, 500 000 nodes, 12.3 M 789 / 736, 16.2 M 1021 / 922, 10^6 nodes, 32.4 M 1975 / 1729.  Graphs with most entries
// in longer rows lose 3 to 17 % (power law, 10^6 nodes, 19 M, 0.59 of them in short rows 1418 / 1569, now 1463; R-MAT, 2^20 nodes, 32 M, 0.22 3620 / 3974,
// now 3673): short_rows_count(), which leaves them the empty launch.
constexpr int VT_FROM = 12000000;
static bool votes_are_checked(int nnz) { return nnz >= VT_FROM; }
static int changed_shift(int n)
{
    int s = 0;
    while ((n - 1) >> s >> VT_BITS_LOG2) ++s;
    return s;
}
static int changed_words(int n) { return ((n - 1) >> changed_shift(n) >> 5) + 1; }

size_t row_sort_ws(int n, int nnz)
{
    auto ints = [](int64_t k) { return align_up(static_cast<size_t>(k) * sizeof(int), 256); };
    return 256 + ints(queue_cap(nnz, RS_SHORT)) + ints(queue_cap(nnz, RS_MID)) + ints(queue_cap(nnz, RS_LONG)) +
           ints(queue_cap(nnz, RS_GROUP)) + 2 * ints(queue_cap(nnz, RS_LDS)) + align_up(static_cast<size_t>(queue_cap(nnz, RS_LDS)) * 8, 256) + ints(n) +
           (nnz > RS_LDS_MOST && many_ranges(n) ? ints(nnz) : 0) +
           (votes_are_checked(nnz) ? 2 * ints(VT_COUNTERS) + 2 * ints(changed_words(n)) + ints((n + 31) / 32) : 0);
}

// of rounds with an even and an odd number
struct VoteCheck {
    int *changes[2];
    uint32_t *changed[2], *todo;
};

static RowQueues carve(int n, int nnz, void *ws, int **labels, VoteCheck *vc)
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
    q.rows[3] = ints(queue_cap(nnz, RS_GROUP));
    q.rows[4] = ints(queue_cap(nnz, RS_LDS));
    q.dup_rows = ints(queue_cap(nnz, RS_LDS));
    q.best = reinterpret_cast<unsigned long long *>(p);
    p += align_up(static_cast<size_t>(queue_cap(nnz, RS_LDS)) * 8, 256);
    *labels = ints(n);
    q.values = nnz > RS_LDS_MOST && many_ranges(n) ? ints(nnz) : nullptr;
    if (vc) {
        const bool kept = votes_are_checked(nnz);
        for (int k = 0; k < 2; ++k) vc->changes[k] = kept ? ints(VT_COUNTERS) : nullptr;
        for (int k = 0; k < 2; ++k) vc->changed[k] = kept ? reinterpret_cast<uint32_t *>(ints(changed_words(n))) : nullptr;
        vc->todo = kept ? reinterpret_cast<uint32_t *>(ints((n + 31) / 32)) : nullptr;
    }
    return q;
}

// clears the queue counters and, where they are kept, the changes of the second round
__global__ __launch_bounds__(256) void row_sort_begin_kernel(int *__restrict__ counts, int *__restrict__ changes, uint32_t *__restrict__ changed,
                                                             int changed_words)
{
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i < 64) counts[i] = 0;
    if (!changes) return;
    if (i < VT_COUNTERS) changes[i] = 0;
    if (i < changed_words) changed[i] = 0u;
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

static void classify_rows(int n, const int *rp, int in_lds, const RowQueues &q, const VoteCheck *vc, hipStream_t s)
{
    const int words = vc && vc->todo ? changed_words(n) : 0;
    hipLaunchKernelGGL(row_sort_begin_kernel, dim3((words + 255) / 256 + 1), dim3(256), 0, s, q.counts, words ? vc->changes[1] : nullptr,
                       words ? vc->changed[1] : nullptr, words);
    hipLaunchKernelGGL(row_classes_kernel, dim3((n + 4095) / 4096), dim3(1024), 0, s, n, rp, in_lds, q);
}

// rp: row starts of the relabelled graph, complete before this on the stream; ws: row_sort_ws(n, nnz) bytes
int32_t launch_relabel_rows(const ftc_csr &g, const int *perm, const int *inv, const int *rp, int *col_idx_out, int *flag,
                            void *ws, hipStream_t s)
{
    int *unused;
    const RowQueues q = carve(g.n, g.nnz, ws, &unused, nullptr);
    const RowSortGrid grid = row_sort_grid(g.n, g.nnz);
    const Relabel u{g.n, g.row_ptr, g.col_idx, perm, inv, rp, col_idx_out, flag};
    classify_rows(g.n, rp, RS_LDS, q, nullptr, s);
    if (g.nnz > RS_LONG) hipLaunchKernelGGL(row_sort_big_kernel<Relabel>, dim3(grid.big_blocks), dim3(RS_NT), 0, s, u, q);
    hipLaunchKernelGGL(row_sort_kernel<Relabel>, dim3(grid.blocks), dim3(256), 0, s, u, q, grid.queue_blocks);
    if (g.nnz > RS_LDS) {
        if (q.values)
            hipLaunchKernelGGL(long_row_values_kernel, dim3(grid.big_blocks), dim3(RS_NT), 0, s, u, q.dup_rows,
                               q.counts + RS_QUEUES, q.values);
        hipLaunchKernelGGL(row_sort_dup_kernel, dim3(grid.big_blocks), dim3(RS_NT), 0, s, u, q);
    }
    return launch_status("relabel rows");
}

template <bool FIRST>
static void label_round(const ftc_csr &g, const Votes<FIRST> &u, const RowQueues &q, const RowSortGrid &grid, hipStream_t s)
{
    hipLaunchKernelGGL(row_sort_kernel<Votes<FIRST>>, dim3(grid.blocks), dim3(256), 0, s, u, q, grid.queue_blocks);
    if (g.nnz > RS_LONG) hipLaunchKernelGGL(row_sort_big_kernel<Votes<FIRST>>, dim3(grid.big_blocks), dim3(RS_NT), 0, s, u, q);
}

// `labels` holds the labels after the last round; ws: row_sort_ws(n, nnz) bytes
int32_t launch_label_rounds(const ftc_csr &g, int iters, int *labels, void *ws, hipStream_t s)
{
    int *other;
    VoteCheck vc;
    const RowQueues q = carve(g.n, g.nnz, ws, &other, &vc);
    const RowSortGrid grid = row_sort_grid(g.n, g.nnz);
    const int shift = changed_shift(g.n);
    // the rounds alternate between the two arrays and end in `labels`
    int *from = iters % 2 == 0 ? labels : other, *to = iters % 2 == 0 ? other : labels;
    classify_rows(g.n, g.row_ptr, many_ranges(g.n) ? RS_LDS_MOST : RS_LDS, q, &vc, s);
    for (int it = 0; it < iters; ++it) {
        // nearly all labels change in the first two rounds; the third is the first to ask which did in the one before
        const bool kept = vc.todo && it >= 1 && it + 1 < iters, check = vc.todo && it >= 2;
        if (check)
            hipLaunchKernelGGL(vote_check_kernel, dim3(256), dim3(RS_NT), 0, s, g.n, g.nnz, q.counts + RS_SHORT_ENTRIES, g.row_ptr, g.col_idx, vc.changed[(it - 1) & 1],
                               vc.changes[(it - 1) & 1], vc.changed[it & 1], vc.changes[it & 1], shift, vc.todo);
        if (it == 0)
            label_round(g, Votes<true>{g.n, g.col_idx, from, g.row_ptr, to, nullptr, nullptr, 0, g.nnz, nullptr}, q, grid, s);
        else
            label_round(g, Votes<false>{g.n, g.col_idx, from, g.row_ptr, to, kept ? vc.changed[it & 1] : nullptr, vc.changes[it & 1], shift, g.nnz,
                                        check ? vc.todo : nullptr}, q, grid, s);
        int *t = from;
        from = to;
        to = t;
    }
    return launch_status("label propagation");
}

}  // namespace ftc
