// Small graphs: aggregation and AGNN layer in one launch.
//
// Bound by latency: launch, row start, column ids, gathered rows, store, each a dependent step of about a microsecond.  The
// edge-balanced kernels take two launches (the second one for rows cut by a range boundary) and a chain of their own in each; here rows
// are not cut.  A row belongs to 16 lanes (more where one row of the matrix takes more): S groups of LPR lanes take every S-th
// entry, several gathers in flight, and their sums are added in the wave.  Rows of more than SHORT entries are put aside and
// summed by the whole workgroup, so that the hubs of a small power-law graph do not hold up the rest; a workgroup's rows lie gridDim.x apart,
// a prime number (the long rows of an R-MAT graph lie side by side).  No scratch memory, no float atomics: reproducible bit for bit.
#include "edge_ranges.hpp"

namespace ftc {

constexpr int SG_NT = 512;

template <int LPR>
struct SmallRows {
    static constexpr int LANES = LPR <= 16 ? 16 : LPR;  // of a row
    static constexpr int S = LANES / LPR;               // entries side by side
    static constexpr int ROWS = SG_NT / LANES;          // rows of a workgroup
    static constexpr int SHORT = 16 * S;                // entries of a row that its own lanes add up: two batches of gathers
    static constexpr int WAVE_S = 64 / LPR, WAVE = 32 * WAVE_S;  // entries side by side in a wave, and those left to one
    static constexpr int GROUP_S = SG_NT / LPR;
};

// Sum over the groups of LPR lanes among LANES neighbouring lanes; every lane of the wave takes part.
template <int LPR, int LANES, int N>
__device__ __forceinline__ void sum_over_groups(float (&v)[N])
{
#pragma unroll
    for (int m = LPR; m < LANES; m <<= 1) {
#pragma unroll
        for (int j = 0; j < N; ++j) v[j] += __shfl_xor(v[j], m, 64);
    }
}

// Runs add(r, e, e1, step, acc), which adds the entries e, e + step, ... below e1 of row r into acc[N], for every row of the workgroup
// and hands the row's sums to finish(r, e, e1, step, acc, first) in the lanes that added (first: of the row's first group).
// Rows of up to ALONE entries, one batch of gathers, are left to the row's first group: as fast, and the fewest roundings.
template <int LPR, int ALONE, int N, class Add, class Finish>
__device__ __forceinline__ void small_rows(int n, const int *__restrict__ row_ptr, Add add, Finish finish)
{
    using R = SmallRows<LPR>;
    __shared__ int count[2], rows[2][R::ROWS];
    __shared__ float part[SG_NT / 64][LPR * N];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, sub = tid % LPR;
    if (tid < 2) count[tid] = 0;
    __syncthreads();
    float acc[N];
    {
        const int64_t row = static_cast<int64_t>(tid / R::LANES) * gridDim.x + blockIdx.x;
        const int r = static_cast<int>(row < n ? row : 0);
        int e0 = 0, e1 = 0;
        if (row < n) { e0 = row_ptr[r]; e1 = row_ptr[r + 1]; }
        const bool own = e1 - e0 <= R::SHORT;
        if (!own && tid % R::LANES == 0) {
            const int q = e1 - e0 <= R::WAVE ? 0 : 1;
            rows[q][atomicAdd(&count[q], 1)] = r;  // (their order does not matter: rows are independent)
        }
#pragma unroll
        for (int j = 0; j < N; ++j) acc[j] = 0.f;
        const int group = tid % R::LANES / LPR;
        const bool alone = e1 - e0 <= ALONE;
        const int mine = alone && group ? e1 : e0 + group, step = alone ? 1 : R::S;
        add(r, mine, own ? e1 : e0, step, acc);
        sum_over_groups<LPR, R::LANES>(acc);
        if (row < n && own) finish(r, mine, e1, step, acc, group == 0);
    }
    __syncthreads();
    const int n_wave = count[0], n_group = count[1];
    for (int i = wave; i < n_wave; i += SG_NT / 64) {  // the waves take the middle rows in turn ...
        const int r = rows[0][i], e0 = row_ptr[r], e1 = row_ptr[r + 1];
#pragma unroll
        for (int j = 0; j < N; ++j) acc[j] = 0.f;
        add(r, e0 + lane / LPR, e1, R::WAVE_S, acc);
        sum_over_groups<LPR, 64>(acc);
        finish(r, e0 + lane / LPR, e1, R::WAVE_S, acc, lane < LPR);
    }
    for (int i = 0; i < n_group; ++i) {  // uniform: ... and all together the long ones
        const int r = rows[1][i], e0 = row_ptr[r], e1 = row_ptr[r + 1];
#pragma unroll
        for (int j = 0; j < N; ++j) acc[j] = 0.f;
        add(r, e0 + tid / LPR, e1, R::GROUP_S, acc);
        sum_over_groups<LPR, 64>(acc);
        __syncthreads();  // the sums of the row before have been read
        if (lane < LPR) {
#pragma unroll
            for (int j = 0; j < N; ++j) part[wave][sub * N + j] = acc[j];
        }
        __syncthreads();
#pragma unroll
        for (int j = 0; j < N; ++j) {
            float t = part[0][sub * N + j];
            for (int w = 1; w < SG_NT / 64; ++w) t += part[w][sub * N + j];
            acc[j] = t;
        }
        finish(r, e0 + tid / LPR, e1, R::GROUP_S, acc, tid < LPR);
    }
}

// blockIdx.y: the columns, LPR * VEC at a time, so that a long row is shared by as many workgroups as its width allows.
// D <= gridDim.y * LPR * VEC; rows of X are 16-byte aligned (or whole pieces of narrower lanes) and at least LPR * VEC elements long where D is no
// multiple of VEC.
template <class T, int VEC, int LPR>
__global__ __launch_bounds__(SG_NT) void spmm_group_kernel(int n, const int *__restrict__ row_ptr, const int *__restrict__ col_idx,
                                                           const float *__restrict__ vals, const void *__restrict__ X,
                                                           uint32_t ldb, int D, void *__restrict__ out, int ldo, int odt, Epi epi,
                                                           bool out_vec)
{
    const int sub = blockIdx.y * LPR + threadIdx.x % LPR;  // the lane's piece of a row
    const bool live = sub * VEC < D;
    const int col0 = live ? sub * VEC : 0;  // lanes beyond the row gather its first piece and store nothing
    const uint32_t lane_bytes = static_cast<uint32_t>(col0) * T::BYTES;
    auto add = [&](int, int e, int e1, int step, float (&acc)[VEC]) {
        constexpr int U = 8;
        for (; e < e1; e += U * step) {  // an entry past the end is the last one, and not added
            int c[U];
            float a[U];
            RawVec<T, VEC> x[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int at = min(e + u * step, e1 - 1);
                c[u] = col_idx[at];
                a[u] = vals ? vals[at] : 1.f;
            }
#pragma unroll
            for (int u = 0; u < U; ++u) load_raw<T, VEC>(row_addr<false>(X, row_slot<false>(c[u], ldb), ldb, lane_bytes), 0, x[u]);
#pragma unroll
            for (int u = 0; u < U; ++u) {
                float xf[VEC];
                unpack<T, VEC>(x[u], xf);
                if (e + u * step < e1) {
#pragma unroll
                    for (int j = 0; j < VEC; ++j) acc[j] = fmaf(a[u], xf[j], acc[j]);
                }
            }
        }
    };
    auto finish = [&](int r, int, int, int, float (&acc)[VEC], bool first) {
        if (!live || !first) return;
        const float f = epi.factor(r);
#pragma unroll
        for (int j = 0; j < VEC; ++j) acc[j] = epi.apply(f, acc[j]);
        if (out_vec) {
            store_vec<VEC>(out, static_cast<int64_t>(r) * ldo + col0, odt, acc);
        } else {
#pragma unroll
            for (int j = 0; j < VEC; ++j)
                if (col0 + j < D) store_elem(out, static_cast<int64_t>(r) * ldo + col0 + j, odt, acc[j]);
        }
    };
    small_rows<LPR, 8, VEC>(n, row_ptr, add, finish);
}

// AGNN layer: out_i = sum_j w_ij h_j / sum_j w_ij, w_ij = exp(beta cos(h_i, h_j) - |beta|) as in agnn_fused.hip; row_z, out32 and
// edge_p (the probabilities: the weights first, divided by the row's sum by the lanes that have it) may be NULL.
template <class T, int VEC, int LPR, bool P>
__global__ __launch_bounds__(SG_NT) void agnn_group_kernel(int n, const int *__restrict__ row_ptr, const int *__restrict__ col_idx,
                                                           const void *__restrict__ H, uint32_t ldb, int D, float beta,
                                                           void *__restrict__ out, int ldo, int odt, float *__restrict__ row_z,
                                                           float *__restrict__ out32, int ld32, float *edge_p)
{
    const int sub = threadIdx.x % LPR;
    const bool live = sub * VEC < D, odd = threadIdx.x & 1, upper = threadIdx.x & 2;
    const int col0 = live ? sub * VEC : 0;
    const uint32_t lane_bytes = static_cast<uint32_t>(col0) * T::BYTES;
    const float beta2 = beta * 1.44269504f;  // in powers of two, see agnn_fused.hip
    const float beta2_rest = fmaf(beta, 1.92596299e-8f, fmaf(beta, 1.44269504f, -beta2));
    // acc: even entries' sums and weights, then odd entries', which meet in the quotient as in agnn_fused.hip
    auto add = [&](int r, int e, int e1, int step, float (&acc)[2 * VEC + 2]) {
        constexpr int U = 4;
        if (e >= e1) return;  // the lanes of a group return together
        RawVec<T, VEC> xi;
        load_raw<T, VEC>(row_addr<false>(H, row_slot<false>(r, ldb), ldb, lane_bytes), 0, xi);
        if (!live) zero_raw(xi);
        const float ri = __frsqrt_rn(fmaxf(group_sum_dpp<LPR>(dot_raw<T, VEC>(xi, xi, 0.f)), 1e-24f));
        for (; e < e1; e += U * step) {
            int c[U];
            RawVec<T, VEC> y[U];
#pragma unroll
            for (int u = 0; u < U; ++u) c[u] = col_idx[min(e + u * step, e1 - 1)];
#pragma unroll
            for (int u = 0; u < U; ++u) load_raw<T, VEC>(row_addr<false>(H, row_slot<false>(c[u], ldb), ldb, lane_bytes), 0, y[u]);
            // the weights as in agnn_fused.hip and its backward pass, in the same order: what the row's sum is made of there
            // has to be what it was made of here
            float dots[U], squares[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const float q = dot_raw<T, VEC>(y[u], y[u], 0.f);
                squares[u] = live ? q : 0.f;
                dots[u] = dot_raw<T, VEC>(xi, y[u], 0.f);
            }
            const float rj = __frsqrt_rn(fmaxf(group_sum4<LPR>(squares, odd, upper), 1e-24f));
            const float cosine = ri * rj * group_sum4<LPR>(dots, odd, upper);
            const float wgt = __builtin_amdgcn_exp2f(fmaf(beta2_rest, cosine, fmaf(beta2, cosine, -fabsf(beta2))));
            if (P && sub < 4 && e + sub * step < e1) edge_p[e + sub * step] = wgt;
            const float w[U] = {quad_lane<0>(wgt), quad_lane<1>(wgt), quad_lane<2>(wgt), quad_lane<3>(wgt)};
#pragma unroll
            for (int u = 0; u < U; ++u) {
                float yf[VEC];
                unpack<T, VEC>(y[u], yf);
                if (e + u * step < e1) {
#pragma unroll
                    for (int j = 0; j < VEC; ++j) {
                        float &t = acc[(u & 1) * (VEC + 1) + j];
                        t = fmaf(w[u], yf[j], t);
                    }
                    acc[(u & 1) * (VEC + 1) + VEC] += w[u];
                }
            }
        }
    };
    auto finish = [&](int r, int e, int e1, int step, float (&acc)[2 * VEC + 2], bool first) {
        const float z = acc[VEC] + acc[2 * VEC + 1];
        if constexpr (P)
            if (sub < 4)
                for (e += sub * step; e < e1; e += 4 * step) edge_p[e] /= z;  // written by this lane
        if (!first) return;
        const float inv = z == 0.f ? 0.f : __builtin_amdgcn_rcpf(z);  // a row without entries: 0
        const float rest = fmaf(-z, inv, 1.f) * inv;                  // what the reciprocal is short of
        float o[VEC];
#pragma unroll
        for (int j = 0; j < VEC; ++j)
            o[j] = fmaf(acc[j], inv, fmaf(acc[VEC + 1 + j], inv, (acc[j] + acc[VEC + 1 + j]) * rest));
        if (live) {
            store_vec<VEC>(out, static_cast<int64_t>(r) * ldo + col0, odt, o);
            if (out32) store_vec<VEC>(out32, static_cast<int64_t>(r) * ld32 + col0, FTC_F32, o);
        }
        if (row_z && sub == 0) row_z[r] = z;
    };
    small_rows<LPR, 4, 2 * VEC + 2>(n, row_ptr, add, finish);
}

bool seg_shape(int dtype, int D, int *vec, int *lpr);

// Up to which graphs.  Two things speak for the edge-balanced kernels: many entries, and a long row, which is one workgroup's chain here
// (of up to 1024 gathers at a time, about 90 GB/s).  The host knows no row length, but a row without repeated columns has at most n entries,
// so the lines are drawn by nnz and by n.  us, edge-balanced kernels / here (6 us are what a call takes from Python):
//   SpMM, entries         uniform, 2048 nodes  uniform, 8192 nodes  R-MAT, 8192 nodes  uniform, 16 384  star, 4000    star, 8000    star, 16 000
//                         8 th.                33 th.               59 th.             66 th.           8 th.         16 th.        32 th.
//   fp16, 8 columns       8.4 / 5.8            8.8 / 5.8            11.4 / 7.1         8.8 / 6.0        8.0 / 6.1     8.1 / 7.0     8.8 / 8.8
//   fp16, 32 columns      11.7 / 5.8           12.0 / 5.8           14.4 / 9.3         12.1 / 8.7       9.6 / 7.9     10.5 / 11.2   11.5 / 12.7
//   bf16, 64 columns      20.9 / 5.8           20.8 / 5.9           22.8 / 11.5        21.3 / 9.0       16.5 / 12.2   17.8 / 19.8   19.5 / 21.0
//   fp32, 64 columns      19.1 / 5.9           19.7 / 5.9           21.5 / 11.3        20.1 / 7.0       16.5 / 10.4   18.0 / 16.7   20.1 / 29.5
//   fp32, 128 columns     29.9 / 5.9           30.5 / 6.9           35.4 / 13.0        33.2 / 11.7      28.9 / 11.1   31.5 / 18.1   35.5 / 45.2
//   AGNN layer with P     uniform, 2048        uniform, 4096        R-MAT, 2048        uniform, 10 000  star, 2000    star, 4000    star, 8000
//                         8 th.                16 th.               14 th.             40 th.           4 th.         8 th.         16 th.
//   fp16, 32 columns      15.4 / 6.0           15.3 / 6.2           17.2 / 10.7        15.8 / 7.8       13.7 / 10.9   14.7 / 14.2   16.1 / 21.1
//   fp32, 128 columns     39.5 / 6.1           39.6 / 6.3           43.4 / 14.7                         42.0 / 31.1   44.3 / 56.5   48.2 / 141
// At the lines what uniform graphs gain is about what a star, which is all one row, loses: without a line by n a star of 64 000 nodes took
// 18 / 90 (fp16, 32 columns), and a million nodes with 40 000 entries 19 / 101 (fp16, 8 columns): 16 lanes a row, empty ones too.
// Dense graphs leave their entries to few workgroups, of 32 rows each, so there is a line by the mean row as well.  Complete graphs of 50 / 120 / 200 / 280
// nodes, edge-balanced kernels / here: fp16, 32 columns 8.1 / 5.5, 8.1 / 7.7, 10.3 / 12.0, 10.8 / 14.4; bf16, 64 columns 8.3 / 6.8, 8.7 / 10.9,
// 9.9 / 19, 9.6 / 50; AGNN layer, bf16, 64 columns 9.3 / 9.8, 10.0 / 15.7; with P, fp32, 128 columns 18.5 / 13.9, 18.7 / 36.5.  Rows of 16 bytes have the
// edge-balanced kernel for narrow rows against them: 400 nodes 16.2 / 10.4, 50 with 800 entries each (repeated columns) 14.9 / 10.0, 3000 each 8.3 / 42.
static bool rows_fit(int n, int nnz, int most_rows, int mean) { return n <= most_rows && nnz <= static_cast<int64_t>(n) * mean; }
bool spmm_group_ok(int n, int64_t row_bytes, int piece_bytes, int nnz)
{
    const int most = piece_bytes <= 16 ? 512 << 10 : piece_bytes <= 64 ? 160 << 10 : 80 << 10;
    const int rows = piece_bytes <= 16 ? 32 << 10 : piece_bytes <= 128 ? 20 << 10 : 16 << 10;
    return nnz <= most && rows_fit(n, nnz, rows, piece_bytes <= 16 ? 1024 : 96) && !rows_need_64_bits(n, row_bytes);
}
bool agnn_group_ok(int n, int64_t row_bytes, int piece_bytes, int nnz)
{
    const int most = piece_bytes <= 64 ? 48 << 10 : piece_bytes <= 128 ? 32 << 10 : 16 << 10;
    const int rows = piece_bytes <= 64 ? 10 << 10 : piece_bytes <= 128 ? 8 << 10 : 4 << 10;
    return nnz <= most && rows_fit(n, nnz, rows, 64) && !rows_need_64_bits(n, row_bytes);
}

// Lanes of the SpMM per row and workgroup: 8, the other columns are other workgroups', and half of the row's above 8192 nodes, where a
// row may be so long that the chip has to share it: us with whole rows / halves, fp16, 32 columns: uniform, 16 384 nodes 5.9 / 8.7, star, 16 000
// nodes 17.9 / 12.7; bf16, 64 columns: 6.3 / 9.0, 34 / 21; pieces of 512 bytes whole / in pieces of 128: star, 8000 nodes 84 / 18, uniform, 8192 nodes 5.9 / 6.9.
static int group_lanes(int n, int lpr) { return lpr > 8 ? 8 : n > 8 << 10 && lpr > 2 ? lpr / 2 : lpr; }

// Workgroups: a prime number of them, so that rows any distance apart fall to different ones.  (The long rows of an R-MAT graph are those
// whose numbers have few one-bits, those of a batch of like graphs lie a period apart.)
static unsigned group_grid(int n, int lpr)
{
    unsigned p = static_cast<unsigned>(ceil_div(n, SG_NT / (lpr <= 16 ? 16 : lpr))) | 1u;
    auto prime = [](unsigned x) {
        for (unsigned d = 3; d * d <= x; d += 2)
            if (x % d == 0) return false;
        return true;
    };
    while (!prime(p)) p += 2;
    return p;
}

int32_t launch_spmm_group(const ftc_csr &g, const float *vals, const void *X, int ldx, int xdt, int D, void *out, int ldo, int odt,
                          Epi epi, hipStream_t s)
{
    const int vm = xdt == FTC_F32 ? 4 : 8;
    int vec = vm, lpr = (D + vm - 1) / vm;  // one or two lanes: rows of at most 32 bytes, as in spmm_lane.hip
    if (!spmm_lane_shape(xdt, D, ldx)) seg_shape(xdt, D, &vec, &lpr);
    lpr = group_lanes(g.n, lpr);
    const uint32_t ldb = static_cast<uint32_t>(ldx) * elem_size(xdt);
    const bool out_vec = D % vec == 0 && aligned16(out) && (static_cast<int64_t>(ldo) * elem_size(odt)) % 16 == 0;
    const dim3 grid(group_grid(g.n, lpr), ceil_div(D, vec * lpr));
#define FTC_SG(T, V, L)                                                                                                  \
    hipLaunchKernelGGL((spmm_group_kernel<T, V, L>), grid, dim3(SG_NT), 0, s, g.n, g.row_ptr, g.col_idx, vals, X, ldb, D, \
                       out, ldo, odt, epi, out_vec)
#define FTC_SGT(T)                                     \
    do {                                               \
        constexpr int VM = T::VEC;                     \
        if (lpr == 1) FTC_SG(T, VM, 1);                \
        else if (lpr == 2) FTC_SG(T, VM, 2);           \
        else if (lpr == 4) FTC_SG(T, VM, 4);           \
        else FTC_SG(T, VM, 8);                         \
    } while (0)
    if (xdt == FTC_F32) FTC_SGT(F32);
    else if (xdt == FTC_F16) FTC_SGT(F16);
    else FTC_SGT(BF16);
#undef FTC_SGT
#undef FTC_SG
    return launch_status("spmm_group");
}

int32_t launch_agnn_group(const ftc_csr &g, const void *H, int ld, int dt, int D, float beta, void *out, int ldo, int odt,
                          float *row_z, float *out32, int ld32, float *edge_p, hipStream_t s)
{
    int vec, lpr;
    seg_shape(dt, D, &vec, &lpr);
    const uint32_t ldb = static_cast<uint32_t>(ld) * elem_size(dt);
    const dim3 grid(group_grid(g.n, lpr));
#define FTC_SG1(T, V, L, P)                                                                                               \
    hipLaunchKernelGGL((agnn_group_kernel<T, V, L, P>), grid, dim3(SG_NT), 0, s, g.n, g.row_ptr, g.col_idx, H, ldb, D, beta, \
                       out, ldo, odt, row_z, out32, ld32, edge_p)
#define FTC_SG(T, V, L)                      \
    do {                                     \
        if (edge_p) FTC_SG1(T, V, L, true);  \
        else FTC_SG1(T, V, L, false);        \
    } while (0)
#define FTC_SGT(T)                                     \
    do {                                               \
        constexpr int VM = T::VEC;                     \
        if (vec == VM) {                               \
            if (lpr == 4) FTC_SG(T, VM, 4);            \
            else if (lpr == 8) FTC_SG(T, VM, 8);       \
            else if (lpr == 16) FTC_SG(T, VM, 16);     \
            else FTC_SG(T, VM, 32);                    \
        } else if (vec == VM / 2) {                    \
            FTC_SG(T, VM / 2, 4);                      \
        } else {                                       \
            FTC_SG(T, VM / 4, 4);                      \
        }                                              \
    } while (0)
    if (dt == FTC_F32) FTC_SGT(F32);
    else if (dt == FTC_F16) FTC_SGT(F16);
    else FTC_SGT(BF16);
#undef FTC_SGT
#undef FTC_SG
#undef FTC_SG1
    return launch_status("agnn_group");
}

}  // namespace ftc
