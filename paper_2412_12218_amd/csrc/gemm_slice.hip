// Dense products Z = X W of few rows, on the 16-bit matrix cores (v_mfma_f32_16x16x32): 16-bit inputs as they are, fp32 inputs in
// three exact bf16 pieces (bf16_split.hpp); and dX = G W^T, the same with W transposed (TRANS).  Rows at any alignment of their
// elements, any width.
//
// A workgroup of SW waves owns 16 rows of X and up to 16 NT columns; wave w takes the steps w, w + SW, .. of 32 contraction indices,
// so that 2708 rows occupy 170 compute units, and adds its partial tile to the others' through LDS at the end, the only barrier.
//   A operand  lane l holds X[row0 + l%16][k0 + (l/16) 8 .. +7], loaded at element alignment;
//   B operand  lane l holds W[k0 + (l/16) 8 .. +7][n0 + l%16], eight loads of one element: a workgroup needs every element of W once, so
//              that a copy in LDS would only add a wait.
// A wave whose numbers can't all be taken in pieces does its steps again in fp32.
// Bound by two memory latencies and the launch, not by bytes; from about 10 000 rows by the loads of W, which every 16 rows make anew.
// Sixteen waves from 512 indices on, else four.  Fewer columns a workgroup (down to 16) as long as all fit the chip at once: a short
// wave is worth more than reading X again.  us and error against 64 bits (2-norm), before (W staged in LDS chunk by chunk, products in
// fp32 or on the 16-bit matrix cores, 16 to 64 rows a workgroup) / here:
//   fp16  2708 x 1433 -> 16 9.7 / 6.1 (1.4e-7 / 0.9e-7), -> 32 15.0 / 7.9, 4096 x 1433 -> 64 49.9 / 11.4 (0.9e-7 / 0.9e-7), 1000 x 150 -> 64 9.5 / 2.6
//   fp32  2708 x 1433 -> 16 8.0 / 6.3 (1.5e-7 / 0.8e-7), 8192 x 301 -> 64 13.5 / 8.1 (1.2e-7 / 0.7e-7), 1000 x 1433 -> 128 48.4 / 9.0
// One sum over the partial tiles instead of fours: error of fp16 1433 -> 16 1.0e-7; pairs all the way: fp32 1433 -> 64 14.8 us for 12.6.
#include "bf16_split.hpp"

namespace ftc {

typedef _Float16 gs_half8 __attribute__((ext_vector_type(8)));

// eight elements of one operand, as they come from memory and as the instruction takes them
template <class T>
struct SliceRaw {
    typename std::conditional<T::BYTES == 4, float, uint32_t>::type e[8];
};
template <class T>
__device__ __forceinline__ bool slice_operand(const SliceRaw<T> &r, uint4 (&p)[T::BYTES == 4 ? 3 : 1])
{
    if constexpr (T::BYTES == 4) return split8(r.e, p);
    else {
        p[0] = make_uint4(r.e[0] | r.e[1] << 16, r.e[2] | r.e[3] << 16, r.e[4] | r.e[5] << 16, r.e[6] | r.e[7] << 16);
        return false;
    }
}
template <class T>
__device__ __forceinline__ auto slice_load(const void *base, int64_t i)
{
    if constexpr (T::BYTES == 4) return static_cast<const float *>(base)[i];
    else return static_cast<uint32_t>(static_cast<const uint16_t *>(base)[i]);
}

// one element, and eight in a row, of a W whose type is another than X's: widened
template <class T, class TW>
__device__ __forceinline__ auto slice_w(const void *W, int64_t i)
{
    if constexpr (std::is_same<T, TW>::value) return slice_load<T>(W, i);
    else return std::is_same<TW, F16>::value ? f16_bits_to_f32(slice_load<TW>(W, i)) : bf16_bits_to_f32(slice_load<TW>(W, i));
}
template <class TW>
__device__ __forceinline__ void slice_load8(const void *W, int64_t i, SliceRaw<F32> &r)
{
    if constexpr (TW::BYTES == 4) {
        typedef float f4 __attribute__((ext_vector_type(4), aligned(4)));
        const float *p = static_cast<const float *>(W) + i;
        const f4 x = *reinterpret_cast<const f4 *>(p), y = *reinterpret_cast<const f4 *>(p + 4);
#pragma unroll
        for (int j = 0; j < 4; ++j) { r.e[j] = x[j]; r.e[4 + j] = y[j]; }
    } else {
        typedef uint32_t u4 __attribute__((ext_vector_type(4), aligned(2)));
        const u4 x = *reinterpret_cast<const u4 *>(static_cast<const uint16_t *>(W) + i);
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const uint32_t b = j & 1 ? x[j / 2] >> 16 : x[j / 2] & 0xffffu;
            r.e[j] = std::is_same<TW, F16>::value ? f16_bits_to_f32(b) : bf16_bits_to_f32(b);
        }
    }
}

// TW: the type of W, another than X's only for TRANS, where it is widened.
template <class T, int NT, int SW, bool TRANS, class TW>
__global__ __launch_bounds__(64 * SW) void gemm_slice_kernel(int n, const void *__restrict__ X, int ldx, int d_in, const void *__restrict__ W,
                                                             int w_ld, int d_out, void *__restrict__ Z, int ldz, int zdt, Epi epi)
{
    static_assert(TRANS ? T::BYTES == 4 : std::is_same<T, TW>::value, "types of the products");
    constexpr int COLS = 16 * NT, P = T::BYTES == 4 ? 3 : 1, U = T::BYTES == 4 ? (NT == 4 ? 1 : 2) : (NT == 4 ? 2 : 4);
    __shared__ float part[SW * 16 * COLS];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int m = lane & 15, kb = lane >> 4;
    const int col0 = blockIdx.y * COLS, cols = min(COLS, d_out - col0);
    const int64_t row0 = static_cast<int64_t>(blockIdx.x) * 16;
    const int64_t at = min(row0 + m, static_cast<int64_t>(n) - 1) * ldx;  // clamped: stores are predicated
    split_f32x4 hi[NT], lo[P == 3 ? NT : 1];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) hi[nt] = lo[P == 3 ? nt : 0] = split_f32x4{0.f, 0.f, 0.f, 0.f};
    bool odd = false;
    auto w_index = [&](int k, int o) { return TRANS ? static_cast<int64_t>(o) * w_ld + k : static_cast<int64_t>(k) * w_ld + o; };
    auto product = [&](const uint4 (&a)[P], const SliceRaw<T> (&w)[NT]) {
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            uint4 b[P];
            odd |= slice_operand<T>(w[nt], b);
            if constexpr (P == 3) mfma_split(a, b, hi[nt], lo[nt]);
            else if constexpr (std::is_same<T, F16>::value)
                hi[nt] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(gs_half8, a[0]), __builtin_bit_cast(gs_half8, b[0]), hi[nt], 0, 0, 0);
            else
                hi[nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(split_bf16x8, a[0]), __builtin_bit_cast(split_bf16x8, b[0]), hi[nt], 0, 0, 0);
        }
    };
    // columns of this lane; beyond the last one column 0 is loaded and taken as zero
    int wc[NT];
    bool col_ok[NT];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
        col_ok[nt] = nt * 16 + m < cols;
        wc[nt] = col_ok[nt] ? col0 + nt * 16 + m : 0;
    }
    const int full = d_in / 32;  // whole steps; the rest is the next wave's in turn
    for (int s0 = wave; s0 < full; s0 += SW * U) {
        uint4 a16[U];
        SliceRaw<T> a32[U], w[U][NT];
#pragma unroll
        for (int u = 0; u < U; ++u) {  // the loads of U steps in flight, beyond the last one that one's
            const int k = min(s0 + u * SW, full - 1) * 32 + kb * 8;
            if constexpr (P == 3) {
                typedef float f4 __attribute__((ext_vector_type(4), aligned(4)));
                const float *p = static_cast<const float *>(X) + at + k;
                const f4 x = *reinterpret_cast<const f4 *>(p), y = *reinterpret_cast<const f4 *>(p + 4);
#pragma unroll
                for (int j = 0; j < 4; ++j) { a32[u].e[j] = x[j]; a32[u].e[4 + j] = y[j]; }
            } else {
                typedef uint32_t u4 __attribute__((ext_vector_type(4), aligned(2)));
                const u4 x = *reinterpret_cast<const u4 *>(static_cast<const uint16_t *>(X) + at + k);
                a16[u] = make_uint4(x[0], x[1], x[2], x[3]);
            }
#pragma unroll
            for (int nt = 0; nt < NT; ++nt)
                if constexpr (TRANS) slice_load8<TW>(W, w_index(k, wc[nt]), w[u][nt]);
                else
#pragma unroll
                    for (int j = 0; j < 8; ++j) w[u][nt].e[j] = slice_load<T>(W, w_index(k + j, wc[nt]));
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (u > 0 && s0 + u * SW >= full) break;  // uniform
            uint4 a[P];
            if constexpr (P == 3) odd |= split8(a32[u].e, a);
            else a[0] = a16[u];
#pragma unroll
            for (int nt = 0; nt < NT; ++nt)
#pragma unroll
                for (int j = 0; j < 8; ++j) w[u][nt].e[j] = col_ok[nt] ? w[u][nt].e[j] : 0;
            product(a, w[u]);
        }
    }
    if (d_in % 32 != 0 && full % SW == wave) {  // uniform
        const int k = full * 32 + kb * 8;
        SliceRaw<T> x, w[NT];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const bool in = k + j < d_in;
            const int kk = in ? k + j : d_in - 1;
            const auto v = slice_load<T>(X, at + kk);
            x.e[j] = in ? v : 0;
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
                const auto y = slice_w<T, TW>(W, w_index(kk, wc[nt]));
                w[nt].e[j] = in && col_ok[nt] ? y : 0;
            }
        }
        uint4 a[P];
        odd |= slice_operand<T>(x, a);
        product(a, w);
    }
    if constexpr (P == 3) {
        float zero = 0.f;
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) zero = not_finite(hi[nt] + lo[nt], zero);
        if (__builtin_expect(__builtin_amdgcn_ballot_w64(odd || zero != 0.f) != 0, 0)) {  // this wave's steps in fp32, product j of a step takes the lanes' j-th index
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) hi[nt] = lo[nt] = split_f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
            for (int k0 = wave * 32; k0 < d_in; k0 += SW * 32) {
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    if (k0 + j >= d_in) break;  // uniform
                    const int k = k0 + kb * 8 + j;
                    const bool in = k < d_in;
                    const float v = load_elem(X, at + (in ? k : 0), FTC_F32), x = in ? v : 0.f;
#pragma unroll
                    for (int nt = 0; nt < NT; ++nt) {
                        const float y = slice_w<F32, typename std::conditional<TRANS, TW, F32>::type>(W, w_index(in ? k : 0, wc[nt]));
                        hi[nt] = __builtin_amdgcn_mfma_f32_16x16x4f32(x, in && col_ok[nt] ? y : 0.f, hi[nt], 0, 0, 0);
                    }
                }
            }
        }
    }
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            float v = hi[nt][i];
            if constexpr (P == 3) v += lo[nt][i];
            part[(wave * 16 + kb * 4 + i) * COLS + nt * 16 + m] = v;
        }
    __syncthreads();
    for (int t = tid; t < 16 * COLS; t += 64 * SW) {
        const int64_t row = row0 + t / COLS;
        const int o = t % COLS;
        if (row >= n || o >= cols) continue;
        float v = 0.f;
#pragma unroll
        for (int w = 0; w < SW; w += 4) {  // four at a time: fewer roundings one after the other
            const float *p = part + w * 16 * COLS + t;
            v += (p[0] + p[16 * COLS]) + (p[32 * COLS] + p[48 * COLS]);
        }
        store_elem(Z, row * ldz + col0 + o, zdt, epi.apply(epi.factor(row), v));
    }
}

template <class T, bool TRANS, class TW = T>
static void gemm_slice_t(int n, const void *X, int ldx, int d_in, const void *W, int w_ld, int d_out, void *Z, int ldz, int zdt, Epi epi,
                         hipStream_t s)
{
    if (d_out > GEMM_MOST_COLUMNS) {
        for (int64_t c = 0; c < d_out; c += GEMM_MOST_COLUMNS)
            gemm_slice_t<T, TRANS, TW>(n, X, ldx, d_in, static_cast<const char *>(W) + c * (TRANS ? w_ld : 1) * TW::BYTES, w_ld,
                                       static_cast<int>(d_out - c < GEMM_MOST_COLUMNS ? d_out - c : GEMM_MOST_COLUMNS),
                                       static_cast<char *>(Z) + c * elem_size(zdt), ldz, zdt, epi, s);
        return;
    }
    const int64_t tiles = (static_cast<int64_t>(n) + 15) / 16;
    const bool wide = !TRANS && d_in >= 512;  // sixteen waves (the contraction of dX is at most 504 long)
    int nt = d_out <= 16 ? 1 : d_out <= 32 ? 2 : 4;
    while (nt > 1 && tiles * ((d_out + nt * 8 - 1) / (nt * 8)) <= (wide ? 256 : 1024)) nt /= 2;
    const dim3 grid(static_cast<unsigned>(tiles), static_cast<unsigned>((d_out + nt * 16 - 1) / (nt * 16)));
#define FTC_GS(N, SW)                                                                                                                    \
    hipLaunchKernelGGL((gemm_slice_kernel<T, N, SW, TRANS, TW>), grid, dim3(64 * SW), 0, s, n, X, ldx, d_in, W, w_ld, d_out, Z, ldz, zdt, epi)
    if constexpr (!TRANS) {
        if (wide) {
            if (nt == 1) FTC_GS(1, 16);
            else if (nt == 2) FTC_GS(2, 16);
            else FTC_GS(4, 16);
            return;
        }
    }
    if (nt == 1) FTC_GS(1, 4);
    else if (nt == 2) FTC_GS(2, 4);
    else FTC_GS(4, 4);
#undef FTC_GS
}

int32_t launch_gemm_slice(int n, const void *X, int ldx, int dt, int d_in, const void *W, int d_out, void *Z, int ldz, int zdt, Epi epi,
                          hipStream_t s)
{
    if (dt == FTC_F32) gemm_slice_t<F32, false>(n, X, ldx, d_in, W, d_out, d_out, Z, ldz, zdt, epi, s);
    else if (dt == FTC_F16) gemm_slice_t<F16, false>(n, X, ldx, d_in, W, d_out, d_out, Z, ldz, zdt, epi, s);
    else gemm_slice_t<BF16, false>(n, X, ldx, d_in, W, d_out, d_out, Z, ldz, zdt, epi, s);
    return launch_status("update_gemm slice");
}

// dX = G W^T for G in fp32: W (d_in x d_out) is read transposed, the contraction runs over d_out.
int32_t launch_input_grad_slice(int n, const float *G, int ldg, int d_out, const void *W, int wdt, int d_in, void *dX, int lddx, int dx_dt,
                                hipStream_t s)
{
    const Epi none{0, nullptr};
    if (wdt == FTC_F32) gemm_slice_t<F32, true, F32>(n, G, ldg, d_out, W, d_out, d_in, dX, lddx, dx_dt, none, s);
    else if (wdt == FTC_F16) gemm_slice_t<F32, true, F16>(n, G, ldg, d_out, W, d_out, d_in, dX, lddx, dx_dt, none, s);
    else gemm_slice_t<F32, true, BF16>(n, G, ldg, d_out, W, d_out, d_in, dX, lddx, dx_dt, none, s);
    return launch_status("input_grad slice");
}

}  // namespace ftc
