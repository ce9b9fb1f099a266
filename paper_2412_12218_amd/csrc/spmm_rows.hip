// Row-oriented SpMM on the plain CSR (no window index needed): a group of LPR lanes owns one
// output row and walks its stored entries, every lane holding one 16-byte slice of the
// feature row.  This is the definition C = A x B of Section I.A.2 evaluated row by row; it is
// the path taken when the caller has no window index, and the reference the balanced
// segmented kernels are compared with.
#include "ftc_common.hpp"

namespace ftc {

template <class T, int LPR>
__global__ __launch_bounds__(256) void spmm_rows_kernel(int n, const int *__restrict__ row_ptr,
                                                        const int *__restrict__ col_idx,
                                                        const float *__restrict__ vals,
                                                        const void *__restrict__ X, int ldx, int D,
                                                        void *__restrict__ out, int ldo, int odt, Epi epi)
{
    constexpr int V = T::VEC;
    constexpr int GROUPS = 256 / LPR;
    const int sub = threadIdx.x % LPR;
    const int grp = threadIdx.x / LPR;
    const int64_t row = static_cast<int64_t>(blockIdx.x) * GROUPS + grp;
    if (row >= n) return;
    const bool live = sub * V < D;  // D may be smaller than LPR * V (D = 24, 40, ...)
    const int e0 = row_ptr[row], e1 = row_ptr[row + 1];
    float acc[V];
#pragma unroll
    for (int k = 0; k < V; ++k) acc[k] = 0.f;
    if (live) {
        int e = e0;
        for (; e + 4 <= e1; e += 4) {
            int c[4];
            float a[4];
            float x[4][V];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                c[u] = col_idx[e + u];
                a[u] = vals ? vals[e + u] : 1.f;
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) load_vec<T>(X, static_cast<int64_t>(c[u]) * ldx + sub * V, x[u]);
#pragma unroll
            for (int u = 0; u < 4; ++u)
#pragma unroll
                for (int k = 0; k < V; ++k) acc[k] = fmaf(a[u], x[u][k], acc[k]);
        }
        for (; e < e1; ++e) {
            float x[V];
            const float a = vals ? vals[e] : 1.f;
            load_vec<T>(X, static_cast<int64_t>(col_idx[e]) * ldx + sub * V, x);
#pragma unroll
            for (int k = 0; k < V; ++k) acc[k] = fmaf(a, x[k], acc[k]);
        }
        const float f = epi.factor(row);
#pragma unroll
        for (int k = 0; k < V; ++k) acc[k] = epi.apply(f, acc[k]);
        store_vec<V>(out, row * ldo + sub * V, odt, acc);
    }
}

// Any D, any alignment: one thread per output element.
__global__ __launch_bounds__(256) void spmm_generic_kernel(int n, const int *__restrict__ row_ptr,
                                                           const int *__restrict__ col_idx,
                                                           const float *__restrict__ vals, const void *X,
                                                           int ldx, int xdt, int D, void *out, int ldo,
                                                           int odt, Epi epi)
{
    const int64_t t = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
    if (t >= static_cast<int64_t>(n) * D) return;
    const int64_t row = t / D;
    const int k = static_cast<int>(t - row * D);
    float acc = 0.f;
    for (int e = row_ptr[row]; e < row_ptr[row + 1]; ++e)
        acc = fmaf(vals ? vals[e] : 1.f, load_elem(X, static_cast<int64_t>(col_idx[e]) * ldx + k, xdt), acc);
    acc = epi.apply(epi.factor(row), acc);
    store_elem(out, row * ldo + k, odt, acc);
}

// Any width up to RW_NT / 4, any alignment, small graphs: one launch that no long row holds up.  A workgroup owns
// whole rows, every gridDim.x-th one (the long rows of an R-MAT graph lie side by side); a row of at most RW_THREAD entries is
// summed by a thread per column, one of at most RW_SLOT entries per entry that fits into a wave side by side by a wave, a
// longer one by the workgroup, the partial sums added in order through LDS.
// Bound by latency: launch, row start, column id, row of X.  The edge-balanced kernels are two launches, each a chain of
// its own, 12 to 40 us on the smallest graphs; a thread per column alone takes as long as the longest row.  Thread per
// column / edge-balanced / this, us:
//   fp32, 7 columns    uniform, 2000 nodes, 18 thousand entries 5 / 13 / 8; R-MAT, 4096 nodes, 65 thousand 143 / 19 / 13; power law,
//                      16 000 nodes, 246 thousand 81 / 16 / 14; R-MAT, 65 536 nodes, 309 thousand 388 / 20 / 22
//   fp16, 47 columns   uniform, 4000 nodes, 20 thousand 5 / 16 / 4; R-MAT, 4096 nodes, 65 thousand 161 / 20 / 16, 260 thousand 394 / 21 / 30
//   fp16, 131 columns  uniform, 4000 nodes, 20 thousand 6 / 30 / 6; R-MAT, 4096 nodes, 65 thousand 157 / 41 / 23, 260 thousand 464 / 48 / 72
// (One row that holds all entries is the exception: 48 thousand of them, 7 columns 2240 / 14 / 18, 131 columns 5600 / 60 / 268.)
constexpr int RW_NT = 1024, RW_THREAD = 32, RW_SLOT = 96;

template <class T>
__device__ __forceinline__ float rw_elem(const void *X, int64_t idx)
{
    if constexpr (T::BYTES == 4) return static_cast<const float *>(X)[idx];
    const uint32_t b = static_cast<const uint16_t *>(X)[idx];
    return std::is_same<T, F16>::value ? f16_bits_to_f32(b) : bf16_bits_to_f32(b);
}

// entries e, e + step, ... below e1 of a row, column k of X
template <class T, int U>
__device__ __forceinline__ float rw_sum(const int *__restrict__ col_idx, const float *__restrict__ vals,
                                        const void *__restrict__ X, int64_t ldx, int k, int e, int e1, int step)
{
    float acc = 0.f;
    for (; e < e1; e += U * step) {  // an index past the end is clamped, its value 0
        int c[U];
        float a[U], x[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int at = min(e + u * step, e1 - 1);
            c[u] = col_idx[at];
            a[u] = vals ? vals[at] : 1.f;
        }
#pragma unroll
        for (int u = 0; u < U; ++u) x[u] = rw_elem<T>(X, c[u] * ldx + k);
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (e + u * step < e1) acc = fmaf(a[u], x[u], acc);
    }
    return acc;
}

template <class T>
__global__ __launch_bounds__(RW_NT) void spmm_small_kernel(int n, const int *__restrict__ row_ptr,
                                                           const int *__restrict__ col_idx, const float *__restrict__ vals,
                                                           const void *__restrict__ X, int ldx, int D, void *__restrict__ out,
                                                           int ldo, int odt, Epi epi)
{
    __shared__ int count[2], rows[2][RW_NT];
    __shared__ float part[RW_NT];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    if (tid < 2) count[tid] = 0;
    __syncthreads();
    const int per = RW_NT / D, slots = 64 / D;  // rows of the workgroup, entries of a row side by side in a wave
    const int64_t row = static_cast<int64_t>(tid / D) * gridDim.x + blockIdx.x;
    const int k = tid % D;
    auto store = [&](int64_t r, int c, float v) { store_elem(out, r * ldo + c, odt, epi.apply(epi.factor(r), v)); };
    if (tid < per * D && row < n) {
        const int e0 = row_ptr[row], e1 = row_ptr[row + 1];
        if (e1 - e0 <= RW_THREAD) {
            store(row, k, rw_sum<T, 4>(col_idx, vals, X, ldx, k, e0, e1, 1));
        } else if (k == 0) {
            const int q = e1 - e0 <= RW_SLOT * slots ? 0 : 1;
            rows[q][atomicAdd(&count[q], 1)] = static_cast<int>(row);  // (their order does not matter: rows are independent)
        }
    }
    __syncthreads();
    const int n_wave = count[0], n_group = count[1];
    for (int i = wave; i < n_wave; i += RW_NT / 64) {
        const int r = rows[0][i], e0 = row_ptr[r], e1 = row_ptr[r + 1];
        const int s = lane / D, c = lane % D;
        part[tid] = s < slots ? rw_sum<T, 8>(col_idx, vals, X, ldx, c, e0 + s, e1, slots) : 0.f;
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        if (s == 0) {
            float v = 0.f;
            for (int j = 0; j < slots; ++j) v += part[wave * 64 + j * D + c];
            store(r, c, v);
        }
        __builtin_amdgcn_wave_barrier();  // the patch is rewritten by the next row
    }
    for (int i = 0; i < n_group; ++i) {  // uniform
        const int r = rows[1][i], e0 = row_ptr[r], e1 = row_ptr[r + 1];
        __syncthreads();  // the patch is free
        if (tid < per * D) part[tid] = rw_sum<T, 8>(col_idx, vals, X, ldx, k, e0 + tid / D, e1, per);
        __syncthreads();
        if (tid < D) {
            float v = 0.f;
            for (int j = 0; j < per; ++j) v += part[j * D + tid];
            store(r, tid, v);
        }
    }
}

// The lines lie where the edge-balanced kernels draw level on R-MAT graphs (figures above).
bool spmm_small_ok(int D, int nnz) { return D <= RW_NT / 4 && nnz <= (D <= 16 ? 320 << 10 : 80 << 10); }

int32_t launch_spmm_small(const ftc_csr &g, const float *vals, const void *X, int ldx, int xdt, int D, void *out, int ldo,
                          int odt, Epi epi, hipStream_t s)
{
    const int per = RW_NT / D;
    const dim3 grid(static_cast<unsigned>((static_cast<int64_t>(g.n) + per - 1) / per));
#define FTC_SM(T) hipLaunchKernelGGL(spmm_small_kernel<T>, grid, dim3(RW_NT), 0, s, g.n, g.row_ptr, g.col_idx, vals, X, ldx, D, \
                                     out, ldo, odt, epi)
    if (xdt == FTC_F32) FTC_SM(F32);
    else if (xdt == FTC_F16) FTC_SM(F16);
    else FTC_SM(BF16);
#undef FTC_SM
    return launch_status("spmm_small");
}

template <class T>
static void launch_rows_t(int lpr, const ftc_csr &g, const float *vals, const void *X, int ldx, int D,
                          void *out, int ldo, int odt, Epi epi, hipStream_t s)
{
#define FTC_CASE(L)                                                                                  \
    case L: {                                                                                        \
        const int groups = 256 / L;                                                                  \
        const unsigned grid = static_cast<unsigned>((static_cast<int64_t>(g.n) + groups - 1) / groups); \
        hipLaunchKernelGGL((spmm_rows_kernel<T, L>), dim3(grid), dim3(256), 0, s, g.n, g.row_ptr,    \
                           g.col_idx, vals, X, ldx, D, out, ldo, odt, epi);                        \
    } break;
    switch (lpr) {
        FTC_CASE(1)
        FTC_CASE(2)
        FTC_CASE(4)
        FTC_CASE(8)
        FTC_CASE(16)
        FTC_CASE(32)
    }
#undef FTC_CASE
}

// Vector path usable? (alignment and shape); mirrors the rule stated in ftc.h.
static bool vec_ok(const void *p, int ld, int dt, int D)
{
    const int v = dt == FTC_F32 ? 4 : 8;
    return aligned16(p) && (static_cast<int64_t>(ld) * elem_size(dt)) % 16 == 0 && D % v == 0 && D / v <= 32;
}

int32_t launch_spmm_rows(const ftc_csr &g, const float *vals, const void *X, int ldx, int xdt, int D,
                         void *out, int ldo, int odt, Epi epi, hipStream_t s)
{
    if (g.n == 0) return FTC_OK;
    const int v = xdt == FTC_F32 ? 4 : 8;
    // output rows are written in slices of v elements: 16 B (fp32, v=4), 32 B (fp32, v=8),
    // 8 or 16 B (16-bit); requiring 16-byte aligned rows covers all of them
    if (vec_ok(X, ldx, xdt, D) && aligned16(out) && (static_cast<int64_t>(ldo) * elem_size(odt)) % 16 == 0) {
        int lpr = 1;
        while (lpr * v < D) lpr *= 2;
        if (xdt == FTC_F32) launch_rows_t<F32>(lpr, g, vals, X, ldx, D, out, ldo, odt, epi, s);
        else if (xdt == FTC_F16) launch_rows_t<F16>(lpr, g, vals, X, ldx, D, out, ldo, odt, epi, s);
        else launch_rows_t<BF16>(lpr, g, vals, X, ldx, D, out, ldo, odt, epi, s);
    } else {
        const int64_t total = static_cast<int64_t>(g.n) * D;
        const unsigned grid = static_cast<unsigned>((total + 255) / 256);
        hipLaunchKernelGGL(spmm_generic_kernel, dim3(grid), dim3(256), 0, s, g.n, g.row_ptr, g.col_idx, vals,
                           X, ldx, xdt, D, out, ldo, odt, epi);
    }
    return launch_status("spmm_rows");
}

}  // namespace ftc
