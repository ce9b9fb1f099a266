// Dense update phase Z = X * W for tall-skinny shapes: X is streamed once, W sits in LDS.  All kernels are on the matrix cores but
// for one: 16-bit inputs with d_in <= 256, d_out <= 64 and aligned rows (the benchmark models) keep all of W on chip; few rows are
// split along the contraction (gemm_slice.hip); the rest (fp32, odd widths, rows that are not 16-byte aligned) goes through the
// kernels of gemm_tile.hip, and through gemm_any_kernel for few fp32 columns.
#include "bf16_split.hpp"

namespace ftc {

// fp32 of at most 16 columns, of more rows than gemm_slice.hip takes and fewer than gemm_tile.hip: any width, rows at any alignment of their elements.  Contraction in fp32
// on the matrix cores (v_mfma_f32_16x16x4_f32).  A wave owns a tile of 16 rows of X:
//   A operand  lane l holds X[row0 + l%16][k0 + (l/16) 4 .. + 3], one 16-byte load (64 contiguous bytes per row and step); the
//              j-th product takes element j of every lane, so the contraction
//              index runs in steps of 16 in an order of its own, the same for A and B;
//   B operand  W is staged in LDS in chunks of KC rows, four consecutive k of a column side by side: lane l
//              reads W[k .. k + 3][l%16] as one 16-byte word.
// Bound by the chain of chunks or by reading X.
// One tile per wave, 32 KB of W: two tiles per wave were 10 % slower, 64 KB up to 20 %, 16 KB 5 %.
// 45 000 x 65 -> 7: 0.93 of the time in gemm_tile.hip; up to 65 535 rows (launch_gemm()).
typedef float float4v __attribute__((ext_vector_type(4)));

__global__ __launch_bounds__(256) void gemm_any_kernel(int n, const float *__restrict__ X, int ldx, int d_in,
                                                       const float *__restrict__ W, int d_out, void *__restrict__ Z, int ldz,
                                                       int zdt, Epi epi)
{
    constexpr int STEP = 16, KC = 512, COLS = 16, U = 4, TH = 256;  // contraction indices per step of a wave, of a chunk
    __shared__ __attribute__((aligned(16))) float Ws[KC * COLS];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int m = lane & 15, kb = lane >> 4;
    const int64_t row0 = (static_cast<int64_t>(blockIdx.x) * 4 + wave) * 16;
    const float *x = X + min(row0 + m, static_cast<int64_t>(n) - 1) * ldx;  // clamped: stores are predicated
    // two sums per element, of the even and of the odd products: shorter chains of dependent instructions and of roundings
    float4v acc[2] = {float4v{0.f, 0.f, 0.f, 0.f}, float4v{0.f, 0.f, 0.f, 0.f}};
    typedef float f4 __attribute__((ext_vector_type(4), aligned(4)));  // global loads need no more than the alignment of one element

    auto multiply = [&](const f4 &a, int k) {  // k: first index of the step inside the chunk
        const float4v b = *reinterpret_cast<const float4v *>(&Ws[((k / 4 + kb) * COLS + m) * 4]);
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[j & 1] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[j], b[j], acc[j & 1], 0, 0, 0);
    };

    for (int kc0 = 0; kc0 < d_in; kc0 += KC) {  // uniform
        if (kc0 > 0) __syncthreads();           // the previous chunk has been consumed
        const int kn = min(KC, (d_in - kc0 + STEP - 1) / STEP * STEP);
        for (int t0 = tid; t0 < kn * COLS; t0 += TH * 8) {  // eight loads in flight, unconditional, from clamped addresses
            float w[8];
            bool ok[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const int k = (t0 + j * TH) / COLS, o = (t0 + j * TH) % COLS;
                ok[j] = k < kn && kc0 + k < d_in && o < d_out;
                w[j] = W[ok[j] ? static_cast<int64_t>(kc0 + k) * d_out + o : 0];
            }
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const int k = (t0 + j * TH) / COLS, o = (t0 + j * TH) % COLS;
                if (k < kn) Ws[((k >> 2) * COLS + o) * 4 + (k & 3)] = ok[j] ? w[j] : 0.f;
            }
        }
        __syncthreads();
        int k = 0;
        const int k_end = min(KC, d_in - kc0);
        for (; k + U * STEP <= k_end; k += U * STEP) {
            f4 a[U];
#pragma unroll
            for (int s = 0; s < U; ++s) a[s] = *reinterpret_cast<const f4 *>(x + kc0 + k + s * STEP + kb * 4);
#pragma unroll
            for (int s = 0; s < U; ++s) multiply(a[s], k + s * STEP);
        }
        for (; k < k_end; k += STEP) {
            f4 a;
            if (k + STEP <= k_end) {
                a = *reinterpret_cast<const f4 *>(x + kc0 + k + kb * 4);
            } else {  // nothing beyond d_in is read
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int kk = k + kb * 4 + j;
                    a[j] = kk < k_end ? x[kc0 + kk] : 0.f;
                }
            }
            multiply(a, k);
        }
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int64_t row = row0 + kb * 4 + i;
        if (row < n && m < d_out) store_elem(Z, row * ldz + m, zdt, epi.apply(epi.factor(row), acc[0][i] + acc[1][i]));
    }
}

// fp32 rows of few aligned columns into few: a thread per row, W in LDS.  Bound by reading X and writing Z; the general kernel
// leaves most of its matrix products empty here and stages W anew every 64 rows (10^6 rows, us, there / here: 4 -> 1 41 / 4,
// 4 -> 4 42 / 9, 16 -> 7 44 / 25, 20 -> 4 50 / 18, 32 -> 8 51 / 46).
constexpr int GN_IN = 32;
static bool narrow_shape(int d_in, int d_out) { return (d_in <= GN_IN && d_out <= 8) || (d_in <= 16 && d_out <= 12); }

template <int GN_OUT>
__global__ __launch_bounds__(256) void gemm_narrow_kernel(int n, const float *__restrict__ X, int ldx, int d_in,
                                                          const float *__restrict__ W, int d_out, void *__restrict__ Z, int ldz,
                                                          int zdt, Epi epi)
{
    __shared__ float Ws[GN_IN * GN_OUT];
    for (int t = threadIdx.x; t < GN_IN * GN_OUT; t += 256) {
        const int k = t / GN_OUT, o = t % GN_OUT;
        Ws[t] = k < d_in && o < d_out ? W[k * d_out + o] : 0.f;
    }
    __syncthreads();
    const int64_t row = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
    if (row >= n) return;
    float4 x[GN_IN / 4];
#pragma unroll
    for (int q = 0; q < GN_IN / 4; ++q)
        x[q] = 4 * q < d_in ? *reinterpret_cast<const float4 *>(X + row * ldx + 4 * q) : make_float4(0.f, 0.f, 0.f, 0.f);
    float acc[GN_OUT];
#pragma unroll
    for (int o = 0; o < GN_OUT; ++o) acc[o] = 0.f;
#pragma unroll
    for (int q = 0; q < GN_IN / 4; ++q) {
        if (4 * q >= d_in) break;  // uniform
        const float xk[4] = {x[q].x, x[q].y, x[q].z, x[q].w};
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int o = 0; o < GN_OUT; ++o) acc[o] = fmaf(xk[j], Ws[(4 * q + j) * GN_OUT + o], acc[o]);
    }
    const float f = epi.factor(row);
#pragma unroll
    for (int o = 0; o < GN_OUT; ++o)
        if (o < d_out) store_elem(Z, row * ldz + o, zdt, epi.apply(f, acc[o]));
}

// ------------------------------------------------------------------------------------------------
// Matrix-core version for 16-bit inputs.  The update phase is a dense contraction, so it goes to
// MFMA (v_mfma_f32_16x16x32_{f16,bf16}, fp32 accumulate).  A wave owns tiles of 16 rows of X:
//   A operand  lane l holds X[row0 + l%16][k0 + (l/16)*8 .. +7]: one 16-byte global load, the four
//              lane groups of a row cover 64 contiguous bytes, so X streams in fully used lines;
//   B operand  lane l holds W[k0 + (l/16)*8 .. +7][n0 + l%16]: W is transposed once into LDS
//              (k contiguous, zero padded to multiples of 32 x 16) and read as 16-byte words;
//   C          lane l holds Z[row0 + (l/16)*4 + i][n0 + l%16], i = 0..3.
// The kernel is bound by streaming X from HBM; W (at most 256 x 64) is read once per workgroup.
typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef __bf16 bhalf8 __attribute__((ext_vector_type(8)));

template <class T>
__device__ __forceinline__ float4v mfma16(const uint4 &a, const uint4 &b, float4v c)
{
    if constexpr (std::is_same<T, F16>::value)
        return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(half8, a), __builtin_bit_cast(half8, b), c,
                                                      0, 0, 0);
    else
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bhalf8, a), __builtin_bit_cast(bhalf8, b),
                                                       c, 0, 0, 0);
}

constexpr int GEMM_RT = 2;  // 16-row tiles per wave iteration

template <class T, int KS, int NT>  // KS = ceil(d_in / 32), NT = ceil(d_out / 16)
__global__ __launch_bounds__(256) void gemm_mfma_kernel(int n, const uint16_t *__restrict__ X, int ldx, int d_in,
                                                        const uint16_t *__restrict__ W, int d_out,
                                                        void *__restrict__ Z, int ldz, int zdt, Epi epi,
                                                        int n_tiles, bool vec_store)
{
    constexpr int KP = KS * 32 + 8;  // padded k extent of a W^T row (keeps 16-byte alignment, spreads banks)
    __shared__ __attribute__((aligned(16))) uint16_t Wt[NT * 16 * KP];
    // W is read along its rows (consecutive threads, consecutive columns), all of a thread's loads issued together from clamped
    // addresses: one after the other they cost every workgroup 6 us before its first row (100 000 x 128 -> 32: 16.1 us
    // against 10.6; 2^20 x 128 -> 32: 89 against 78)
    constexpr int PER = NT * 16 * KS * 32 / 256, BATCH = PER <= 16 ? PER : PER % 16 == 0 ? 16 : 8;
    static_assert(PER % BATCH == 0, "whole batches");
    for (int t0 = threadIdx.x; t0 < NT * 16 * KS * 32; t0 += 256 * BATCH) {
        uint16_t wv[BATCH];
#pragma unroll
        for (int j = 0; j < BATCH; ++j) {
            const int k = (t0 + j * 256) / (NT * 16), nn = (t0 + j * 256) % (NT * 16);
            wv[j] = W[(nn < d_out && k < d_in) ? static_cast<size_t>(k) * d_out + nn : 0];
        }
#pragma unroll
        for (int j = 0; j < BATCH; ++j) {
            const int k = (t0 + j * 256) / (NT * 16), nn = (t0 + j * 256) % (NT * 16);
            Wt[nn * KP + k] = (nn < d_out && k < d_in) ? wv[j] : uint16_t(0);
        }
    }
    __syncthreads();
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int m = lane & 15, kb = lane >> 4;
    // B operands stay in registers for the whole kernel
    uint4 breg[KS][NT];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
            breg[ks][nt] = *reinterpret_cast<const uint4 *>(&Wt[(nt * 16 + m) * KP + ks * 32 + kb * 8]);

    constexpr int ZP = NT * 16 + 4;  // row stride of the output patch (16-byte aligned, spreads banks)
    __shared__ __attribute__((aligned(16))) float Zs[4][16 * ZP];
    const int stride = gridDim.x * 4 * GEMM_RT;
    for (int tile0 = (blockIdx.x * 4 + wave) * GEMM_RT; tile0 < n_tiles; tile0 += stride) {
        uint4 a[GEMM_RT][KS];
#pragma unroll
        for (int rt = 0; rt < GEMM_RT; ++rt) {
            const int row = min((tile0 + rt) * 16 + m, n - 1);  // clamped: the store is predicated
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                const int k = ks * 32 + kb * 8;
                if (k < d_in) a[rt][ks] = *reinterpret_cast<const uint4 *>(X + static_cast<size_t>(row) * ldx + k);
                else a[rt][ks] = make_uint4(0u, 0u, 0u, 0u);
            }
        }
#pragma unroll
        for (int rt = 0; rt < GEMM_RT; ++rt) {
            float4v c[NT];
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
                c[nt] = float4v{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int ks = 0; ks < KS; ++ks) c[nt] = mfma16<T>(a[rt][ks], breg[ks][nt], c[nt]);
            }
            if (vec_store) {
                // The accumulators hold columns (lane = column, register = row): written as they are,
                // a 16-bit output would leave in 2-byte pieces, four store instructions per 16 x 16
                // tile.  The tile is turned through LDS instead (each wave has its own patch; LDS
                // operations of one wave execute in order) so that a lane holds 4 NT consecutive
                // columns of one row and the tile leaves in one or two 8- or 16-byte stores per lane.
#pragma unroll
                for (int nt = 0; nt < NT; ++nt)
#pragma unroll
                    for (int i = 0; i < 4; ++i) Zs[wave][(kb * 4 + i) * ZP + nt * 16 + m] = c[nt][i];
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                __builtin_amdgcn_wave_barrier();
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
                const int r = lane >> 2, c0 = (lane & 3) * (4 * NT);
                const int row = (tile0 + rt) * 16 + r;
                float o[4 * NT];
#pragma unroll
                for (int q = 0; q < NT; ++q) {
                    const float4 v = *reinterpret_cast<const float4 *>(&Zs[wave][r * ZP + c0 + 4 * q]);
                    o[4 * q] = v.x; o[4 * q + 1] = v.y; o[4 * q + 2] = v.z; o[4 * q + 3] = v.w;
                }
                if (row < n && c0 < d_out) {
                    const float f = epi.factor(row);
#pragma unroll
                    for (int j = 0; j < 4 * NT; ++j) o[j] = epi.apply(f, o[j]);
                    if constexpr (NT == 1) {
                        store_vec<4>(Z, static_cast<int64_t>(row) * ldz + c0, zdt, reinterpret_cast<float(&)[4]>(o));
                    } else {
#pragma unroll
                        for (int q = 0; q < NT / 2; ++q)
                            store_vec<8>(Z, static_cast<int64_t>(row) * ldz + c0 + 8 * q, zdt,
                                         reinterpret_cast<float(&)[8]>(o[8 * q]));
                    }
                }
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                __builtin_amdgcn_wave_barrier();  // the patch is rewritten by the next tile
            } else {
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) {
                    const int col = nt * 16 + m;
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const int row = (tile0 + rt) * 16 + kb * 4 + i;
                        if (row < n && col < d_out)
                            store_elem(Z, static_cast<int64_t>(row) * ldz + col, zdt,
                                       epi.apply(epi.factor(row), c[nt][i]));
                    }
                }
            }
        }
    }
}

template <class T>
static bool gemm_mfma_t(int n, const void *X, int ldx, int d_in, const void *W, int d_out, void *Z, int ldz,
                        int zdt, Epi epi, hipStream_t s)
{
    const int ks = (d_in + 31) / 32, nt = (d_out + 15) / 16;
    const int n_tiles = (n + 15) / 16;
    int grid = (n_tiles + 4 * GEMM_RT - 1) / (4 * GEMM_RT);
    if (grid > 256 * 8) grid = 256 * 8;
    const uint16_t *x = static_cast<const uint16_t *>(X);
    const uint16_t *w = static_cast<const uint16_t *>(W);
    // whole groups of 4 NT columns per lane, each group 8- or 16-byte aligned in the output
    const int zsize = zdt == FTC_F32 ? 4 : 2;
    const bool vec_store = d_out % (4 * nt) == 0 && aligned16(Z) && (static_cast<int64_t>(ldz) * zsize) % 16 == 0 &&
                           (nt == 1 || nt % 2 == 0);
#define FTC_G(K, N)                                                                                                 if (ks == K && nt == N) {                                                                                           hipLaunchKernelGGL((gemm_mfma_kernel<T, K, N>), dim3(grid), dim3(256), 0, s, n, x, ldx, d_in, w, d_out, Z,                            ldz, zdt, epi, n_tiles, vec_store);                                                                    return true;                                                                                                }
    FTC_G(1, 1) FTC_G(1, 2) FTC_G(2, 1) FTC_G(2, 2) FTC_G(4, 1) FTC_G(4, 2) FTC_G(4, 4) FTC_G(2, 4) FTC_G(1, 4)
    FTC_G(8, 1) FTC_G(8, 2) FTC_G(8, 4) FTC_G(3, 1) FTC_G(3, 2) FTC_G(3, 4)
#undef FTC_G
    return false;
}

// Few rows: where the kernel that splits the contraction (gemm_slice.hip) is ahead of the one that takes the shape otherwise.  us, other / split:
//   16 bits   gemm_mfma_kernel (`on_chip`): fp16 2708 x 256 -> 64 8.2 / 3.7, 2708 x 128 -> 16 3.4 / 2.2, 16 000 x 64 -> 32 3.4 / 3.1, 8000 x 32 -> 32 2.8 / 2.7,
//             4096 x 16 -> 16 2.3 / 2.3; but 24 000 x 64 -> 32 3.6 / 3.6, 16 000 x 32 -> 32 3.0 / 3.1, 6000 x 16 -> 16 2.4 / 2.6
//             gemm_tile.hip: 16 000 x 1433 -> 64 74 / 43, -> 7 25 / 25, 12 000 x 513 -> 128 31 / 28; but 24 000 x 301 -> 7 9.1 / 9.4, 16 000 x 16 -> 128 7.3 / 7.6
//   fp32      gemm_narrow_kernel: 2708 x 16 -> 7 3.7 / 2.8, 16 000 x 16 -> 7 3.8 / 3.7 (24 000 3.8 / 4.2); gemm_any_kernel: 16 000 x 301 -> 16 7.7 / 5.8,
//             24 000 x 513 -> 7 14.9 / 17.0; gemm_tile.hip: 12 000 x 150 -> 64 9.9 / 8.1, 6000 x 513 -> 128 22.7 / 21.6; but 12 000 x 16 -> 32 4.1 / 4.2,
//             16 000 x 150 -> 64 10.2 / 11.0, 8192 x 513 -> 128 23.2 / 25.7
static bool gemm_slice_better(int n, int dt, int d_in, int d_out, bool on_chip)
{
    if (dt != FTC_F32) {
        if (on_chip) return n <= (d_in >= 64 ? 16384 : d_in >= 32 ? 8192 : 4096);
        return n <= (d_out <= 64 ? 16384 : 12288);
    }
    if (d_out <= 16) return n <= 16384;
    if (d_out <= 64) return n <= (d_in >= 32 ? 12288 : 8192);
    // one step of the contraction, or two, are one or two waves', the others have nothing to do: in tiles where the workgroups don't fit the chip at once (us,
    // split / tile: 6000 x 8 -> 500 16.0 / 7.5, 6000 x 32 -> 256 8.6 / 5.8, 4000 x 16 -> 200 7.9 / 5.5, 2000 x 8 -> 500 8.1 / 5.8, 6144 x 48 -> 256 10.3 / 6.8; up to 2000 x
    // 256, 4000 x 130 level).  From 49 to 64 indices the tile is as far ahead, but its two steps one after the other are further from 64 bits (64: 4 %).
    if (d_in <= 48 && static_cast<int64_t>(n) * d_out > 1 << 19) return false;
    return n <= 6144;
}

int32_t launch_gemm(int n, const void *X, int ldx, int dt, int d_in, const void *W, int d_out, void *Z, int ldz,
                    int zdt, Epi epi, hipStream_t s)
{
    if (n == 0) return FTC_OK;
    const int v = dt == FTC_F32 ? 4 : 8;
    // vector loads of X: 16-byte aligned rows, whole vectors
    const bool fast = aligned16(X) && (static_cast<int64_t>(ldx) * elem_size(dt)) % 16 == 0 && d_in % v == 0;
    const bool on_chip = dt != FTC_F32 && fast && d_in <= 256 && d_out <= 64;
    const bool narrow = dt == FTC_F32 && fast && narrow_shape(d_in, d_out);
    const bool few = dt == FTC_F32 && d_in <= SPLIT_FROM;  // fp32 products of a sum this short are not taken in pieces
    if (gemm_slice_better(n, dt, d_in, d_out, on_chip) && !(narrow && d_in < 16) && !few)
        return launch_gemm_slice(n, X, ldx, dt, d_in, W, d_out, Z, ldz, zdt, epi, s);
    if (dt != FTC_F32 && fast) {  // 16-byte row pieces of X: all of W on chip
        const bool done = dt == FTC_F16 ? gemm_mfma_t<F16>(n, X, ldx, d_in, W, d_out, Z, ldz, zdt, epi, s)
                                        : gemm_mfma_t<BF16>(n, X, ldx, d_in, W, d_out, Z, ldz, zdt, epi, s);
        if (done) return launch_status("update_gemm mfma");
    }
    if (narrow) {
        const dim3 grid(static_cast<unsigned>((static_cast<int64_t>(n) + 255) / 256));
        const float *x = static_cast<const float *>(X), *w = static_cast<const float *>(W);
        if (d_out <= 8) hipLaunchKernelGGL(gemm_narrow_kernel<8>, grid, dim3(256), 0, s, n, x, ldx, d_in, w, d_out, Z, ldz, zdt, epi);
        else hipLaunchKernelGGL(gemm_narrow_kernel<12>, grid, dim3(256), 0, s, n, x, ldx, d_in, w, d_out, Z, ldz, zdt, epi);
        return launch_status("update_gemm narrow");
    }
    // Up to 16 fp32 columns both wait for X, gemm_any_kernel in longer chunks, gemm_tile.hip with fewer loads of W.  That one's time over this one's, 5 to
    // 1433 indices into 2, 7, 10, 16 columns: 30 000 rows 1.02 to 1.17, 45 000 0.95 to 1.08, 65 000 0.91 to 1.04, 98 000 0.74 to 0.90, 131 000 0.75 to 1.02, 10^6
    // 0.49 to 0.85.
    if (dt != FTC_F32 || d_out > 16 || n >= 65536 || few) return launch_gemm_tile(n, X, ldx, dt, d_in, W, d_out, Z, ldz, zdt, epi, s);
    hipLaunchKernelGGL(gemm_any_kernel, dim3(static_cast<unsigned>((n + 63) / 64)), dim3(256), 0, s, n, static_cast<const float *>(X), ldx, d_in,
                       static_cast<const float *>(W), d_out, Z, ldz, zdt, epi);
    return launch_status("update_gemm");
}

}  // namespace ftc
