// Kernels of the backward pass of the two layers that have no forward counterpart.  The sparse
// products of the backward pass (A^T dP, P^T dY, the edge scores <dY_i, h_j>, ...) reuse the forward
// SpMM / SDDMM kernels; what is here is the glue around them:
//   transposed index of a symmetric pattern, derivative of the row-wise softmax, the ReLU mask,
//   the weight gradient X^T G, the input gradient G W^T, edge-wise combinations and the derivative
//   of the row normalisation of the AGNN cosine.
// The paper speaks of training (Sections II and V) but gives no gradient formulas; these are the
// derivatives of the forward definitions.  Gradients are fp32.
#include "ftc_common.hpp"

namespace ftc {

// ---- T[e] = position of (j, i) for e = (i, j) -----------------------------------------------------
__global__ __launch_bounds__(256) void transpose_index_kernel(int n, int nnz, const int *__restrict__ row_ptr,
                                                              const int *__restrict__ col_idx,
                                                              const int *__restrict__ edge_to_row,
                                                              int *__restrict__ T, int *flag)
{
    const int64_t e = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
    if (e >= nnz) return;
    int i;
    if (edge_to_row) {
        i = edge_to_row[e];
    } else {  // last row with row_ptr[i] <= e
        int a = 0, b = n;
        while (b - a > 1) {
            const int mid = (a + b) >> 1;
            if (row_ptr[mid] <= e) a = mid; else b = mid;
        }
        i = a;
    }
    const int j = col_idx[e];
    int lo = row_ptr[j], hi = row_ptr[j + 1];  // first position in row j with column >= i
    const int end = hi;
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (col_idx[mid] < i) lo = mid + 1; else hi = mid;
    }
    const bool found = lo < end && col_idx[lo] == i;
    T[e] = found ? lo : -1;
    if (!found) atomicOr(flag, 1);
}

__global__ void set_int_kernel(int *p, int v) { *p = v; }

int32_t launch_transpose_index(const ftc_csr &g, const int *edge_to_row, int *T, int *flag, hipStream_t s)
{
    hipLaunchKernelGGL(set_int_kernel, dim3(1), dim3(1), 0, s, flag, 0);
    if (g.nnz > 0)
        hipLaunchKernelGGL(transpose_index_kernel, dim3(ceil_div(g.nnz, 256)), dim3(256), 0, s, g.n, g.nnz, g.row_ptr,
                           g.col_idx, edge_to_row, T, flag);
    return launch_status("transpose_index");
}

// ---- ds = p * (dp - sum over the row of p * dp) ----------------------------------------------------
// Row classes as in the row-wise softmax: a lane, a wave or the workgroup per row, by length; the
// order of every row's sum depends on its length alone.
__device__ __forceinline__ float bw_wave_sum(float v)
{
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) v += __shfl_xor(v, m, 64);
    return v;
}

__global__ __launch_bounds__(256) void softmax_backward_kernel(int n, const int *__restrict__ row_ptr, const float *p,
                                                               const float *dp, float *ds)
{
    __shared__ int mid_rows[256];
    __shared__ int big_rows[256];
    __shared__ int n_mid, n_big;
    __shared__ float red[4];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    if (tid == 0) { n_mid = 0; n_big = 0; }
    __syncthreads();
    const int64_t row = static_cast<int64_t>(blockIdx.x) * 256 + tid;
    int e0 = 0, e1 = 0;
    if (row < n) { e0 = row_ptr[row]; e1 = row_ptr[row + 1]; }
    const int len = e1 - e0;
    if (len > 0 && len <= 16) {
        float t = 0.f;
        for (int e = e0; e < e1; ++e) t += p[e] * dp[e];
        for (int e = e0; e < e1; ++e) ds[e] = p[e] * (dp[e] - t);
    } else if (len > 16 && len <= 2048) {
        mid_rows[atomicAdd(&n_mid, 1)] = static_cast<int>(row);
    } else if (len > 2048) {
        big_rows[atomicAdd(&n_big, 1)] = static_cast<int>(row);
    }
    __syncthreads();
    const int nm = n_mid, nb = n_big;
    for (int i = wave; i < nm; i += 4) {
        const int r = mid_rows[i];
        const int a = row_ptr[r], b = row_ptr[r + 1];
        float t = 0.f;
        for (int e = a + lane; e < b; e += 64) t += p[e] * dp[e];
        t = bw_wave_sum(t);
        for (int e = a + lane; e < b; e += 64) ds[e] = p[e] * (dp[e] - t);
    }
    for (int i = 0; i < nb; ++i) {  // nb is uniform over the workgroup
        const int r = big_rows[i];
        const int a = row_ptr[r], b = row_ptr[r + 1];
        float t = 0.f;
        for (int e = a + tid; e < b; e += 256) t += p[e] * dp[e];
        t = bw_wave_sum(t);
        __syncthreads();
        if (lane == 0) red[wave] = t;
        __syncthreads();
        t = (red[0] + red[1]) + (red[2] + red[3]);
        for (int e = a + tid; e < b; e += 256) ds[e] = p[e] * (dp[e] - t);
    }
}

int32_t launch_softmax_backward(const ftc_csr &g, const float *p, const float *dp, float *ds, hipStream_t s)
{
    if (g.n == 0 || g.nnz == 0) return FTC_OK;
    hipLaunchKernelGGL(softmax_backward_kernel, dim3((g.n + 255) / 256), dim3(256), 0, s, g.n, g.row_ptr, p, dp, ds);
    return launch_status("edge_softmax_backward");
}

// ---- out = dY * [Y > 0] * scale[row] (fp32) --------------------------------------------------------
__global__ __launch_bounds__(256) void mask_scale_kernel(int n, int d, const float *__restrict__ dY, int lddy,
                                                         const void *__restrict__ Y, int ldy, int ydt,
                                                         const float *__restrict__ scale, float *__restrict__ out,
                                                         int ldo)
{
    const int64_t t = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
    if (t >= static_cast<int64_t>(n) * d) return;
    const int64_t row = t / d;
    const int k = static_cast<int>(t % d);
    float v = dY[row * lddy + k];
    if (Y && !(load_elem(Y, row * ldy + k, ydt) > 0.f)) v = 0.f;
    if (scale) v *= scale[row];
    out[row * ldo + k] = v;
}

int32_t launch_mask_scale(int n, int d, const float *dY, int lddy, const void *Y, int ldy, int ydt,
                          const float *scale, float *out, int ldo, hipStream_t s)
{
    const int64_t total = static_cast<int64_t>(n) * d;
    if (total == 0) return FTC_OK;
    hipLaunchKernelGGL(mask_scale_kernel, dim3(static_cast<unsigned>((total + 255) / 256)), dim3(256), 0, s, n, d, dY,
                       lddy, Y, ldy, ydt, scale, out, ldo);
    return launch_status("mask_scale");
}

// ---- dW = X^T G -----------------------------------------------------------------------------------
// (many rows and columns: weight_grad_tile.hip)
// A contraction over the rows, on the matrix cores in fp32 (v_mfma_f32_16x16x4_f32; 16-bit elements of X are widened), so
// products and sums are those of fp32 arithmetic.  A wave takes four rows per step:
//   A operand  lane l holds VA consecutive columns of row l/16 from column a0 + VA (l%16) on (one load; 64 columns a step for
//              VA = 4); the j-th of them goes into the j-th of VA tiles, whose rows are the columns a0 + VA m + j;
//   B operand  the same of G: VB consecutive columns per lane, NT tiles in all.
// A workgroup owns 16 VA columns of X, 16 NT columns of G and one of `splits` shares of the rows; its four waves take every
// fourth step and are added in a fixed order through LDS, the shares' results by a second kernel: reproducible, no
// floating-point atomics.  Columns beyond the end: the last lanes' pieces are moved back to end with the row, and an
// element is written by the lane whose own piece it lies in.
// ReLU: with Y (the layer's output, limit = the largest finite or infinite bits of its 16-bit type, 0: fp32) an element
// of G counts only where Y is positive; no masked copy of G has to exist.
// Bound by reading X and G (2^20 x 128 fp16, 32 columns of G: 0.40 GB) up to about 64 columns of G, by the fp32 matrix
// rate beyond.  Measured, against rows staged in LDS and 4 x 4 register tiles on the vector units (us, with the sum over
// the shares): fp32 100 000 x 300 -> 128: 324 / 126 (weight_grad_tile.hip: 78); fp16 2^20 x 128 -> 32:
// 250 / 128 (with the mask, before as a pass of its own: 340 / 145).
typedef float wg_f32x4 __attribute__((ext_vector_type(4)));

template <class T, int N>  // N consecutive elements at element alignment
__device__ __forceinline__ void wg_load(const void *base, int64_t idx, float (&f)[N])
{
    if constexpr (N == 1) {
        if constexpr (T::BYTES == 4) f[0] = static_cast<const float *>(base)[idx];
        else f[0] = std::is_same<T, F16>::value ? f16_bits_to_f32(static_cast<const uint16_t *>(base)[idx])
                                                : bf16_bits_to_f32(static_cast<const uint16_t *>(base)[idx]);
    } else if constexpr (T::BYTES == 4) {
        typedef float fv __attribute__((ext_vector_type(N), aligned(4)));
        const fv v = *reinterpret_cast<const fv *>(static_cast<const float *>(base) + idx);
#pragma unroll
        for (int j = 0; j < N; ++j) f[j] = v[j];
    } else {
        typedef uint16_t hv __attribute__((ext_vector_type(N), aligned(2)));
        const hv v = *reinterpret_cast<const hv *>(static_cast<const uint16_t *>(base) + idx);
#pragma unroll
        for (int j = 0; j < N; ++j) f[j] = std::is_same<T, F16>::value ? f16_bits_to_f32(v[j]) : bf16_bits_to_f32(v[j]);
    }
}

// MASK: 0 none, 1 by an fp32 Y, 2 by a 16-bit Y.  ldp: columns of a whole result, of which these d_out are some
template <class T, int VA, int NT, int MASK>
__global__ __launch_bounds__(256) void weight_grad_kernel(int n, const void *__restrict__ X, int ldx, int d_in,
                                                          const float *__restrict__ G, int ldg, int d_out,
                                                          const void *__restrict__ Y, int ldy, unsigned limit,
                                                          float *__restrict__ partial, int ldp, int splits)
{
    constexpr int VB = NT < 4 ? NT : 4, NB = NT / VB, U = NT * VA > 16 ? 2 : VA == 1 ? 8 : 4;
    constexpr int TILES = VA * NT;
    __shared__ float red[2][TILES * 256];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int m = lane & 15, kb = lane >> 4;
    const int a0 = blockIdx.y * (16 * VA), b0 = blockIdx.z * (16 * NT);
    const int ca = min(a0 + VA * m, d_in - VA);  // first column of this lane's piece of X
    int cb[NB];                                  // ... and of its pieces of G
#pragma unroll
    for (int q = 0; q < NB; ++q) cb[q] = min(b0 + q * 16 * VB + VB * m, d_out - VB);
    const int64_t per = ((static_cast<int64_t>(n) + splits - 1) / splits + 15) / 16 * 16;
    const int64_t r_begin = per * blockIdx.x, r_end = min(static_cast<int64_t>(n), r_begin + per);
    // two sums per element (of every other step) where they cost nothing: half the chain of roundings (with 32 columns of G
    // the registers of the second sum cost a quarter of the time, with 64 half; more shares of the rows shorten it there)
    constexpr int PAR = NT == 1 ? 2 : 1;
    wg_f32x4 part[PAR][VA][NT];
#pragma unroll
    for (int p = 0; p < PAR; ++p)
#pragma unroll
        for (int i = 0; i < VA; ++i)
#pragma unroll
            for (int j = 0; j < NT; ++j) part[p][i][j] = wg_f32x4{0.f, 0.f, 0.f, 0.f};

    auto load = [&](int64_t row, bool ok, float (&xa)[VA], float (&gb)[NT]) {
        wg_load<T, VA>(X, row * ldx + ca, xa);
#pragma unroll
        for (int q = 0; q < NB; ++q) {
            float g[VB];
            wg_load<F32, VB>(G, row * ldg + cb[q], g);
            if constexpr (MASK == 1) {
                float y[VB];
                wg_load<F32, VB>(Y, row * ldy + cb[q], y);
#pragma unroll
                for (int j = 0; j < VB; ++j) g[j] = y[j] > 0.f ? g[j] : 0.f;
            } else if constexpr (MASK == 2) {
                typedef uint16_t yv __attribute__((ext_vector_type(VB), aligned(2)));
                const yv y = *reinterpret_cast<const yv *>(static_cast<const uint16_t *>(Y) + row * ldy + cb[q]);
#pragma unroll
                for (int j = 0; j < VB; ++j) {
                    const unsigned bits = y[j];
                    g[j] = (bits != 0u && bits <= limit) ? g[j] : 0.f;  // positive, not NaN
                }
            }
#pragma unroll
            for (int j = 0; j < VB; ++j) gb[q * VB + j] = ok ? g[j] : 0.f;
        }
        if (!ok) {
#pragma unroll
            for (int j = 0; j < VA; ++j) xa[j] = 0.f;
        }
    };
    auto multiply = [&](const float (&xa)[VA], const float (&gb)[NT], wg_f32x4 (&to)[VA][NT]) {
#pragma unroll
        for (int i = 0; i < VA; ++i)
#pragma unroll
            for (int j = 0; j < NT; ++j) to[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(xa[i], gb[j], to[i][j], 0, 0, 0);
    };
    int64_t r = r_begin + wave * 4;  // steps of four rows, every fourth one this wave's
    for (; r + (U - 1) * 16 + 4 <= r_end; r += U * 16) {
        float xa[U][VA], gb[U][NT];
#pragma unroll
        for (int s = 0; s < U; ++s) load(r + s * 16 + kb, true, xa[s], gb[s]);
#pragma unroll
        for (int s = 0; s < U; ++s) multiply(xa[s], gb[s], part[s % PAR]);
    }
    for (; r < r_end; r += 16) {
        float xa[VA], gb[NT];
        const int64_t row = r + kb;
        load(min(row, r_end - 1), row < r_end, xa, gb);
        multiply(xa, gb, part[0]);
    }
    wg_f32x4 acc[VA][NT];
#pragma unroll
    for (int i = 0; i < VA; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j) acc[i][j] = PAR == 2 ? part[0][i][j] + part[PAR - 1][i][j] : part[0][i][j];
    // (wave 0 + wave 2) + (wave 1 + wave 3)
    auto park = [&](float *dst) {
#pragma unroll
        for (int i = 0; i < VA; ++i)
#pragma unroll
            for (int j = 0; j < NT; ++j)
#pragma unroll
                for (int e = 0; e < 4; ++e) dst[((i * NT + j) * 4 + e) * 64 + lane] = acc[i][j][e];
    };
    auto take = [&](const float *src) {
#pragma unroll
        for (int i = 0; i < VA; ++i)
#pragma unroll
            for (int j = 0; j < NT; ++j)
#pragma unroll
                for (int e = 0; e < 4; ++e) acc[i][j][e] += src[((i * NT + j) * 4 + e) * 64 + lane];
    };
    if (wave >= 2) park(red[wave - 2]);
    __syncthreads();
    if (wave < 2) take(red[wave]);
    __syncthreads();
    if (wave == 1) park(red[0]);
    __syncthreads();
    if (wave != 0) return;
    take(red[0]);
    float *out = partial + static_cast<size_t>(blockIdx.x) * d_in * ldp;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int own_a = a0 + VA * (kb * 4 + e), first_a = min(own_a, d_in - VA);
#pragma unroll
        for (int i = 0; i < VA; ++i) {
            const int a = first_a + i;
            if (a < own_a) continue;
#pragma unroll
            for (int j = 0; j < NT; ++j) {
                const int own_b = b0 + (j / VB) * 16 * VB + VB * m, b = cb[j / VB] + j % VB;
                if (b >= own_b) out[static_cast<size_t>(a) * ldp + b] = acc[i][j][e];
            }
        }
    }
}

// sum over the shares: 64 results per workgroup, four threads a result with every fourth share each, eight loads in flight
// (lost, where the rows are taken in rounds: what the additions to `out` have rounded away so far, one float a result, added
// back with the next one; first: the first round)
__global__ __launch_bounds__(256) void sum_partials_kernel(int count, int n_partials, const float *__restrict__ partial,
                                                           float *__restrict__ out, float *__restrict__ lost, bool first)
{
    __shared__ float red[4][64];
    const int lane = threadIdx.x & 63, part = threadIdx.x >> 6;
    const int t = blockIdx.x * 64 + lane;
    float s[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    if (t < count) {
        int b = part;
        for (; b + 28 < n_partials; b += 32) {
#pragma unroll
            for (int k = 0; k < 8; ++k) s[k] += partial[static_cast<size_t>(b + 4 * k) * count + t];
        }
        for (; b < n_partials; b += 4) s[0] += partial[static_cast<size_t>(b) * count + t];
    }
    red[part][lane] = ((s[0] + s[1]) + (s[2] + s[3])) + ((s[4] + s[5]) + (s[6] + s[7]));
    __syncthreads();
    if (part == 0 && t < count) {
        const float sum = (red[0][lane] + red[1][lane]) + (red[2][lane] + red[3][lane]);
        if (lost && !first) {
            const float was = out[t], with = sum - lost[t], now = was + with;
            const float e = (now - was) - with;
            lost[t] = e == e ? e : 0.f;  // an infinite sum stays infinite
            out[t] = now;
        } else {
            out[t] = sum;
            if (lost) lost[t] = 0.f;
        }
    }
}

// The workspace and the widest d_out are part of the interface (ftc_weight_grad_workspace_bytes, FTC_EUNSUPPORTED): room for
// min(n / 128, 1024) partial results of weight_grad_group() columns of X, whatever the kernels make of it.
constexpr int WG_MAX_BLOCKS = 1024, WG_MAX_PIECES = 1024, WG_MAX_COLUMNS = 512;
static int weight_grad_blocks(int n)
{
    const int by_rows = (n + 127) / 128;
    return by_rows < 1 ? 1 : (by_rows > WG_MAX_BLOCKS ? WG_MAX_BLOCKS : by_rows);
}

static bool weight_grad_shape_ok(int d_in, int d_out)  // at least eight columns of X fit next to up to 504 of G
{
    return d_in >= 1 && d_out >= 1 && ((d_in + 3) / 4) * ((d_out + 3) / 4) <= WG_MAX_PIECES &&
           (d_in + 3) / 4 * 4 + (d_out + 3) / 4 * 4 <= WG_MAX_COLUMNS;
}

// Input columns that weight_grad_ws() counts next to d_out output columns; 0: d_out is too wide.
int weight_grad_group(int d_in, int d_out)
{
    if (weight_grad_shape_ok(d_in, d_out)) return d_in;
    for (int gk = 256; gk >= 8; gk -= 8)
        if (gk < d_in && weight_grad_shape_ok(gk, d_out)) return gk;
    return 0;
}

size_t weight_grad_ws(int n, int d_in, int d_out)
{
    const int gk = weight_grad_group(d_in, d_out);
    return align_up(static_cast<size_t>(weight_grad_blocks(n)) * (gk > 0 ? gk : d_in) * d_out * sizeof(float), 256);
}

template <class T, int VA>
static void weight_grad_t(int nt, int mask, dim3 grid, hipStream_t s, int n, const void *X, int ldx, int d_in, const float *G,
                          int ldg, int d_out, const void *Y, int ldy, unsigned limit, float *partial, int ldp, int splits)
{
#define FTC_WG(N, M)                                                                                                   \
    hipLaunchKernelGGL((weight_grad_kernel<T, VA, N, M>), grid, dim3(256), 0, s, n, X, ldx, d_in, G, ldg, d_out, Y, ldy, \
                       limit, partial, ldp, splits)
#define FTC_WGN(N)                      \
    if (nt == N) {                      \
        if (mask == 0) FTC_WG(N, 0);    \
        else if (mask == 1) FTC_WG(N, 1); \
        else FTC_WG(N, 2);              \
    }
    FTC_WGN(1) FTC_WGN(2) FTC_WGN(4)
    if constexpr (VA < 4) { FTC_WGN(8) }  // (never the tile of least cost with VA = 4)
#undef FTC_WGN
#undef FTC_WG
}

// Tile of the weight gradient: 16 va columns of X and 16 nt columns of G per workgroup.  Time goes with the padded area of
// the result, and the more of it a workgroup holds the less often X and G are read; COST is the measured time per padded
// element and row (10^-4 ps, 2^20 rows, median over 117 widths).  X of up to 16 columns: va = 1.  The vector units' 4 x 4 register
// tiles / va = 4 with nt by the width of G alone / this (10^6 rows, us): fp16 65 x 136 536 / 1100 / 543, 17 x 136 286 / 511 / 186,
// 128 x 136 804 / 1156 / 540; fp32 100 000 x 300 -> 128 328 / 140 / 126.  At 10^6 rows a few results that pad by half stay
// behind the register tiles: fp32 100 x 136 585 / - / 759, 200 x 72 631 / - / 826, 200 x 65 670 / 1099 / 877.
struct WgTile { int va, nt; int64_t cost; };
static int64_t weight_grad_cost(int i, int j, int d_in, int d_out)
{
    constexpr int COST[3][4] = {{1440, 760, 505, 387}, {790, 430, 320, 300}, {450, 310, 298, 0}};  // [log2 va][log2 nt]
    const int a = 16 << i, b = 16 << j;
    return static_cast<int64_t>((d_in + a - 1) / a * a) * ((d_out + b - 1) / b * b) * COST[i][j];
}
static WgTile weight_grad_tile(int d_in, int d_out)
{
    WgTile best = {1, 1, INT64_MAX};
    for (int i = d_in <= 16 ? 0 : 2; i >= (d_in <= 16 ? 0 : 1); --i)
        for (int j = 3; j >= 0; --j) {
            if ((i == 2 && j == 3) || (j > 0 && d_out <= 8 << j)) continue;  // (a piece of G is no wider than G)
            const int64_t cost = weight_grad_cost(i, j, d_in, d_out);
            if (cost < best.cost) best = {1 << i, 1 << j, cost};
        }
    return best;
}

// Columns of G that come first: all of them, or whole tiles of 128 where up to eight more are cheaper on a narrow tile in a
// launch of their own.  X is read once more for those, so the line lies where the table says a sixth of the time and 20 us
// less, next to more than 64 columns of X in fp32 (24 such products of 200 000 to 10^6 rows: 0.82 of the time on average, at
// most 1.03; fp32 10^6 x 200 -> 136 1433 / 1192 us, 200 000 x 200 -> 129 327 / 199).  With a tenth instead of a sixth 100 -> 129 and
// 65 -> 264 lose 10 to 17 % at 500 000 rows; 16-bit X, where the first launch is bound by its reads sooner, up to 16 %.
// *cost: of the launches, 10^-4 ps a row.
static int weight_grad_first_columns(int n, int xdt, int d_in, int d_out, int64_t *cost)
{
    const int first = d_out / 128 * 128, rest = d_out - first;
    const int64_t whole = *cost = weight_grad_tile(d_in, d_out).cost;
    if (xdt != FTC_F32 || first == 0 || rest == 0 || rest > 8 || d_in <= 64) return d_out;
    const int64_t split = weight_grad_tile(d_in, first).cost + weight_grad_tile(d_in, rest).cost, saved = whole - split;
    if (saved * 6 < whole || saved < 200000000000 / (n < 1 ? 1 : n)) return d_out;
    *cost = split;
    return first;
}

// dW = X^T (G masked by Y; Y == NULL: no mask).  The shares of the rows: enough workgroups for the chip, at least 64 rows
// each, and as many as the workspace of weight_grad_ws() bytes holds results of; where that would be fewer than four, X may
// be taken in groups of columns instead (rows [k0, k0 + group) of dW are one contiguous block; the passes share the workspace).
// A wave adds up a quarter of a share's rows in one chain, so the shares are also bounded from above: with at most
// 384 + n / 384 rows each the error stays below that of the kernel this one replaced (which had n / 1024 rows, but added
// twice as many shares in a chain; normal inputs, 2-norm against 64 bits, former kernel / chip-filling shares / weight_grad_kernel with
// this bound; the kernel of weight_grad_tile.hip, which most of these sizes take, is below it):
//   400 000 x 1433 -> 128 4.1e-7 / 8.6e-7 / 3.1e-7 (us 3970 / 2110 / 2030), 400 000 x 1433 -> 256 4.1e-7 / 1.2e-6 / 3.3e-7 (7430 /
//   4330 / 3760), 2^20 x 1433 -> 128 6.1e-7 / 1.4e-6 / 4.9e-7 (8780 / 5710 / 4890), 2^20 x 1024 -> 504 6.1e-7 / 3.2e-6 / 5.0e-7
//   (113 000 / 15 300 / 14 100), 20 000 x 1433 -> 64 2.3e-7 / 2.5e-7 / 1.9e-7 (598 / 69 / 94).
// Where the workspace does not hold so many results the rows are taken in rounds, each added to dW with the error of the
// additions carried along.
int32_t launch_weight_grad(int n, const void *X, int ldx, int xdt, int d_in, const float *G, int ldg, int d_out,
                           const void *Y, int ldy, int ydt, float *dW, void *ws, hipStream_t s)
{
    const int64_t room = static_cast<int64_t>(weight_grad_blocks(n)) * weight_grad_group(d_in, d_out);  // columns x shares
    int64_t cost;
    int first = weight_grad_first_columns(n, xdt, d_in, d_out, &cost);
    const WgPieces pieces = weight_grad_pieces(n, d_in, d_out, cost);
    if (pieces.na) first = d_out;
    const int64_t least = n / (384 + n / 384);
    int64_t want = 0;
    for (int b = 0; b < d_out; b = b == 0 ? first : d_out) {
        const int db = b == 0 ? first : d_out - first;
        const WgTile tile = pieces.na ? WgTile{pieces.na, pieces.nb, 0} : weight_grad_tile(d_in, db);
        const int64_t tiles = static_cast<int64_t>((d_in + 16 * tile.va - 1) / (16 * tile.va)) *
                              ((db + 16 * tile.nt - 1) / (16 * tile.nt));
        // with 33 to 64 columns of G more, for shorter sums; what a CU holds of the other kernel's workgroups
        const int64_t fill = (pieces.na ? (pieces.nb == 8 ? 512 : 1024) : tile.nt == 4 ? 2048 : 1024) / tiles;
        if (fill > want) want = fill;
    }
    if (want < least) want = least;
    if (want > (n + 63) / 64) want = (n + 63) / 64;
    if (want < 1) want = 1;
    int64_t splits = room / d_in < want ? room / d_in : want;
    int group = d_in;
    if (splits < 4 && splits < want) {  // (never narrower groups than weight_grad_group() columns)
        splits = want < 4 ? want : 4;
        if (splits > weight_grad_blocks(n)) splits = weight_grad_blocks(n);
        group = static_cast<int>(room / splits < d_in ? room / splits : d_in);
    }
    int64_t rounds = 1;
    if (splits < least && splits > 1) {  // the last share's place holds what the rounds' additions lose
        --splits;
        rounds = (least + splits - 1) / splits;
    }
    const int64_t per_round = rounds == 1 ? n : ((n + rounds - 1) / rounds + 15) / 16 * 16;
    float *partial = static_cast<float *>(ws);
    const int mask = !Y ? 0 : ydt == FTC_F32 ? 1 : 2;
    const unsigned limit = ydt == FTC_F16 ? 0x7c00u : 0x7f80u;
    for (int k0 = 0; k0 < d_in; k0 += group) {
        const int dk = d_in - k0 < group ? d_in - k0 : group;
        float *lost = rounds > 1 ? partial + static_cast<size_t>(splits) * dk * d_out : nullptr;
        int64_t r0 = 0;
        do {  // once with n == 0: dW is cleared
            const int rows = static_cast<int>(n - r0 < per_round ? n - r0 : per_round);
            const void *Xr = static_cast<const char *>(X) + (r0 * ldx + k0) * elem_size(xdt);
            for (int b = 0; b < d_out; b = b == 0 ? first : d_out) {
                const int db = b == 0 ? first : d_out - first;
                const float *Gr = G + r0 * ldg + b;
                const void *Yr = Y ? static_cast<const char *>(Y) + (r0 * ldy + b) * elem_size(ydt) : nullptr;
                if (pieces.na && dk > 1) {  // (it loads two columns at a time)
                    launch_weight_grad_tile(pieces, rows, Xr, ldx, xdt, dk, Gr, ldg, db, Yr, ldy, mask, limit, partial,
                                            static_cast<int>(splits), s);
                    continue;
                }
                const WgTile tile = weight_grad_tile(d_in, db);
                const int nt = tile.nt, va = dk <= 16 ? 1 : tile.va;
                const dim3 grid(static_cast<unsigned>(splits), (dk + 16 * va - 1) / (16 * va), (db + 16 * nt - 1) / (16 * nt));
#define FTC_WGT(T)                                                                                                        \
    do {                                                                                                                  \
        if (va == 1) weight_grad_t<T, 1>(nt, mask, grid, s, rows, Xr, ldx, dk, Gr, ldg, db, Yr, ldy, limit, partial + b,  \
                                         d_out, static_cast<int>(splits));                                                \
        else if (va == 2) weight_grad_t<T, 2>(nt, mask, grid, s, rows, Xr, ldx, dk, Gr, ldg, db, Yr, ldy, limit,          \
                                              partial + b, d_out, static_cast<int>(splits));                              \
        else weight_grad_t<T, 4>(nt, mask, grid, s, rows, Xr, ldx, dk, Gr, ldg, db, Yr, ldy, limit, partial + b, d_out,   \
                                 static_cast<int>(splits));                                                               \
    } while (0)
                if (xdt == FTC_F32) FTC_WGT(F32);
                else if (xdt == FTC_F16) FTC_WGT(F16);
                else FTC_WGT(BF16);
#undef FTC_WGT
            }
            hipLaunchKernelGGL(sum_partials_kernel, dim3((dk * d_out + 63) / 64), dim3(256), 0, s, dk * d_out,
                               static_cast<int>(splits), partial, dW + static_cast<size_t>(k0) * d_out, lost, r0 == 0);
            r0 += per_round;
        } while (r0 < n);
    }
    return launch_status("weight_grad");
}

// ---- dX = G W^T, large and from few columns -----------------------------------------------------------
// A thread owns one input feature a and keeps row a of W in registers; the rows of G are staged in LDS and read as broadcasts.  Bound by
// writing dX, in rows of which a workgroup stores 256 columns at once: beyond the memory-side cache (256 MB) that is ahead of the tiles of 64 columns of
// gemm_tile.hip, which leave lines of memory in parts, most of all where rows are no whole lines (launch_input_grad() there has the line).
constexpr int IG_ROWS = 64;

template <int DOUT>  // d_out padded to a multiple of 4
__global__ __launch_bounds__(256) void input_grad_kernel(int n, const float *__restrict__ G, int ldg, int d_out,
                                                         const void *__restrict__ W, int wdt, int d_in,
                                                         void *__restrict__ dX, int lddx, int dx_dt)
{
    __shared__ __attribute__((aligned(16))) float Gs[IG_ROWS * DOUT];
    const int tid = threadIdx.x;
    const int64_t r0 = static_cast<int64_t>(blockIdx.x) * IG_ROWS;
    for (int t = tid; t < IG_ROWS * DOUT; t += 256) {
        const int r = t / DOUT, b = t % DOUT;
        Gs[t] = (r0 + r < n && b < d_out) ? G[(r0 + r) * ldg + b] : 0.f;
    }
    __syncthreads();
    for (int a = tid; a < d_in; a += 256) {
        float w[DOUT];
#pragma unroll
        for (int b = 0; b < DOUT; ++b) w[b] = b < d_out ? load_elem(W, static_cast<int64_t>(a) * d_out + b, wdt) : 0.f;
        for (int r = 0; r < IG_ROWS && r0 + r < n; ++r) {
            float acc = 0.f;
#pragma unroll
            for (int b = 0; b < DOUT; b += 4) {
                const float4 z = *reinterpret_cast<const float4 *>(&Gs[r * DOUT + b]);
                acc = fmaf(z.x, w[b], acc);
                acc = fmaf(z.y, w[b + 1], acc);
                acc = fmaf(z.z, w[b + 2], acc);
                acc = fmaf(z.w, w[b + 3], acc);
            }
            store_elem(dX, (r0 + r) * lddx + a, dx_dt, acc);
        }
    }
}

int32_t launch_input_grad_rows(int n, const float *G, int ldg, int d_out, const void *W, int wdt, int d_in, void *dX, int lddx, int dx_dt,
                               hipStream_t s)
{
    const unsigned grid = static_cast<unsigned>((static_cast<int64_t>(n) + IG_ROWS - 1) / IG_ROWS);
    if (d_out <= 8) hipLaunchKernelGGL(input_grad_kernel<8>, dim3(grid), dim3(256), 0, s, n, G, ldg, d_out, W, wdt, d_in, dX, lddx, dx_dt);
    else hipLaunchKernelGGL(input_grad_kernel<16>, dim3(grid), dim3(256), 0, s, n, G, ldg, d_out, W, wdt, d_in, dX, lddx, dx_dt);
    return launch_status("input_grad rows");
}

// ---- out[e] = alpha * (wa * a[e] + wb * a[T[e]]) * cs[col[e]] -------------------------------------
__global__ __launch_bounds__(256) void edge_combine_kernel(int nnz, const float *__restrict__ a,
                                                           const int *__restrict__ T, float wa, float wb, float alpha,
                                                           const float *__restrict__ cs,
                                                           const int *__restrict__ col_idx, float *__restrict__ out)
{
    const int64_t e = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
    if (e >= nnz) return;
    const int t = T[e];  // -1 where the pattern has no partner: that term is dropped, nothing is read
    float v = alpha * (wa * a[e] + ((t >= 0 && t < nnz) ? wb * a[t] : 0.f));
    if (cs) v *= cs[col_idx[e]];
    out[e] = v;
}

int32_t launch_edge_combine(int nnz, const float *a, const int *T, float wa, float wb, float alpha, const float *cs,
                            const int *col_idx, float *out, hipStream_t s)
{
    if (nnz == 0) return FTC_OK;
    hipLaunchKernelGGL(edge_combine_kernel, dim3(ceil_div(nnz, 256)), dim3(256), 0, s, nnz, a, T, wa, wb, alpha, cs,
                       col_idx, out);
    return launch_status("edge_combine");
}

// ---- out = sum_e a[e] * b[e], in a fixed order ----------------------------------------------------
constexpr int DOT_BLOCKS = 1024;

__global__ __launch_bounds__(256) void edge_dot_kernel(int nnz, const float *__restrict__ a, const float *__restrict__ b,
                                                       float *__restrict__ partial)
{
    __shared__ float red[4];
    const int64_t per = (static_cast<int64_t>(nnz) + gridDim.x - 1) / gridDim.x;
    const int64_t lo = per * blockIdx.x, hi = min(static_cast<int64_t>(nnz), lo + per);
    float t = 0.f;
    for (int64_t e = lo + threadIdx.x; e < hi; e += 256) t = fmaf(a[e], b[e], t);
    t = bw_wave_sum(t);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = t;
    __syncthreads();
    if (threadIdx.x == 0) partial[blockIdx.x] = (red[0] + red[1]) + (red[2] + red[3]);
}

__global__ __launch_bounds__(256) void sum_scalar_kernel(int count, const float *__restrict__ partial, float *out)
{
    __shared__ float red[4];
    float t = 0.f;
    for (int i = threadIdx.x; i < count; i += 256) t += partial[i];
    t = bw_wave_sum(t);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = t;
    __syncthreads();
    if (threadIdx.x == 0) *out = (red[0] + red[1]) + (red[2] + red[3]);
}

size_t edge_dot_ws() { return align_up(DOT_BLOCKS * sizeof(float), 256); }

int32_t launch_edge_dot(int nnz, const float *a, const float *b, float *out, void *ws, hipStream_t s)
{
    float *partial = static_cast<float *>(ws);
    hipLaunchKernelGGL(edge_dot_kernel, dim3(DOT_BLOCKS), dim3(256), 0, s, nnz, a, b, partial);
    hipLaunchKernelGGL(sum_scalar_kernel, dim3(1), dim3(256), 0, s, DOT_BLOCKS, partial, out);
    return launch_status("edge_dot");
}

// ---- dH = base + rinv * (q - hn <hn, q>), hn = rinv * h --------------------------------------------
// q is the gradient with respect to the normalised rows, base the part of dH that reaches h through
// the aggregated rows; eight lanes per row.  A row whose norm was clamped (|h| <= 1e-12) is a plain
// scaling: no projection; a row of one element gets nothing through its direction unless clamped.
// base may be dH itself (fp32, in place).
// VEC4: four consecutive elements per lane and step (16-byte loads of q and base; every leading
// dimension a multiple of 4, D too, pointers 16-byte aligned), else element by element.
template <bool VEC4>
__global__ __launch_bounds__(256) void cos_backward_rows_kernel(int n, const void *__restrict__ H, int ld, int dt, int D,
                                                                const float *__restrict__ rinv,
                                                                const float *__restrict__ q, int ldq,
                                                                const float *base, int ldb, void *dH, int lddh,
                                                                int dh_dt)
{
    constexpr int W = VEC4 ? 4 : 1;
    const int sub = threadIdx.x & 7;
    const int64_t row = (static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x) >> 3;
    const bool ok = row < n;
    const float ri = ok ? rinv[row] : 0.f;
    float proj = 0.f;
    // the row has at most 256 elements: 8 lanes x 4 elements x 8 steps, kept in registers between the passes
    float hq[VEC4 ? 8 : 1][W], qq[VEC4 ? 8 : 1][W];
    if (ok) {
        if constexpr (VEC4) {
#pragma unroll
            for (int s = 0; s < 8; ++s) {
                const int k = (s * 8 + sub) * 4;
                if (k < D) {
                    const float4 q4 = *reinterpret_cast<const float4 *>(q + row * ldq + k);
                    qq[s][0] = q4.x; qq[s][1] = q4.y; qq[s][2] = q4.z; qq[s][3] = q4.w;
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        hq[s][e] = load_elem(H, row * ld + k + e, dt) * ri;
                        proj = fmaf(hq[s][e], qq[s][e], proj);
                    }
                }
            }
        } else {
            for (int k = sub; k < D; k += 8) proj = fmaf(load_elem(H, row * ld + k, dt) * ri, q[row * ldq + k], proj);
        }
    }
    proj += __shfl_xor(proj, 1, 64);
    proj += __shfl_xor(proj, 2, 64);
    proj += __shfl_xor(proj, 4, 64);
    const bool clamped = ri >= 0.999e12f;  // the clamp of the row-norm kernel took effect
    if (clamped) proj = 0.f;
    // A one-element row normalises to its sign, whose derivative is zero: q - hn <hn, q> would leave the
    // rounding of hn * hn against 1, multiplied by 1 / |h|.
    const float ri_out = (D == 1 && !clamped) ? 0.f : ri;
    if (ok) {
        if constexpr (VEC4) {
#pragma unroll
            for (int s = 0; s < 8; ++s) {
                const int k = (s * 8 + sub) * 4;
                if (k < D) {
                    const float4 b4 = *reinterpret_cast<const float4 *>(base + row * ldb + k);
                    const float bb[4] = {b4.x, b4.y, b4.z, b4.w};
                    float o[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e) o[e] = bb[e] + ri * (qq[s][e] - hq[s][e] * proj);
                    store_vec<4>(dH, row * lddh + k, dh_dt, o);
                }
            }
        } else {
            for (int k = sub; k < D; k += 8) {
                const float hn = load_elem(H, row * ld + k, dt) * ri;
                store_elem(dH, row * lddh + k, dh_dt, base[row * ldb + k] + ri_out * (q[row * ldq + k] - hn * proj));
            }
        }
    }
}

int32_t launch_cos_backward_rows(int n, const void *H, int ld, int dt, int D, const float *rinv, const float *q, int ldq,
                                 const float *base, int ldb, void *dH, int lddh, int dh_dt, hipStream_t s)
{
    if (n == 0) return FTC_OK;
    const unsigned grid = static_cast<unsigned>((static_cast<int64_t>(n) * 8 + 255) / 256);
    const bool vec4 = D % 4 == 0 && D <= 256 && ld % 4 == 0 && ldq % 4 == 0 && ldb % 4 == 0 && lddh % 4 == 0 &&
                      aligned16(q) && aligned16(base) && aligned16(dH) && aligned16(H);
    if (vec4)
        hipLaunchKernelGGL(cos_backward_rows_kernel<true>, dim3(grid), dim3(256), 0, s, n, H, ld, dt, D, rinv, q, ldq, base,
                           ldb, dH, lddh, dh_dt);
    else
        hipLaunchKernelGGL(cos_backward_rows_kernel<false>, dim3(grid), dim3(256), 0, s, n, H, ld, dt, D, rinv, q, ldq,
                           base, ldb, dH, lddh, dh_dt);
    return launch_status("cos_backward_rows");
}

}  // namespace ftc
