// dW = X^T G of many rows with more than 32 columns on either side: a contraction over the rows on the bf16 matrix cores.  G (fp32)
// and an fp32 X are taken in three exact bf16 pieces (bf16_split.hpp), an fp16 X in two, a bf16 X as it is: six, five or three
// v_mfma_f32_16x16x32_bf16 for what were eight v_mfma_f32_16x16x4_f32 of twice the time each.
//
// A workgroup owns 16 NA columns of X, 16 NB columns of G and one of `splits` shares of the rows; a step is 32 rows.  A thread loads
// units of two neighbouring columns and eight rows (the next step's while this one is multiplied), takes them apart once for all
// waves and puts the pieces into LDS with the rows of a column side by side, which is how both operands want them (16 bytes a
// lane; columns 80 bytes apart: no bank conflicts).  A wave holds (NA / WA) x (NB / WB) tiles.  The small products of a step are summed
// apart and added once, so a step rounds a sum twice.  Shares, their sums and the ReLU mask: as in weight_grad_kernel (backward.hip).
// Columns and rows beyond the end are zeros in LDS.  A step with numbers that can't be taken in pieces (an infinity times a piece that
// is zero would be NaN) goes through v_mfma_f32_16x16x4_f32 from X and G as they are, and so do all steps of a wave whose sums are not finite.
//
// Bound by the work of taking apart (8 instructions a number, 30 us for 100 000 x 300, 128) next to the products (25 us), two or three
// workgroups a CU; weight_grad_kernel by reading X and G five and two times.  us, there / here, of calls repeated on the same
// inputs, with the sums over the shares (in a training pass, where they are no longer in a cache, 84 and 7 for 78), and error against 64 bits: fp32 100 000 x 300, 128 118 / 78 (2.2e-7 / 1.8e-7), 400 000 x 128, 128 218 / 114, 100 000 x 300, 64 75 / 54, 200 000 x
// 500, 64 199 / 149; fp16 100 000 x 300, 128 115 / 72, 400 000 x 128, 128 197 / 97.  With the mask: fp32 100 000 x 300, 128
// 90, 400 000 x 128, 128 133 (103 and 163 with 12 registers spilled, before the fp32 step was a function of its own).
// Tried: eight waves with a unit each (8 x 8 tiles: 107 us for 78, registers; 1 000 000 x 128, 32 194 for 131).
#include "bf16_split.hpp"

namespace ftc {

// Two neighbouring columns of eight rows, as loaded.
template <class T>
struct PairRaw {
    uint32_t w[T::BYTES == 4 ? 16 : 8];
};

template <class T>
__device__ __forceinline__ float pair_value(const PairRaw<T> &r, int row, int second)
{
    if constexpr (T::BYTES == 4) return __uint_as_float(r.w[2 * row + second]);
    else if constexpr (std::is_same<T, F16>::value) return f16_bits_to_f32(second ? r.w[row] >> 16 : r.w[row] & 0xffffu);
    else return second ? __uint_as_float(r.w[row] & 0xffff0000u) : __uint_as_float(r.w[row] << 16);
}

template <class T>
__device__ __forceinline__ void load_pair(const void *base, int64_t idx, PairRaw<T> &r, int row)
{
    if constexpr (T::BYTES == 4) {
        typedef uint32_t u2 __attribute__((ext_vector_type(2), aligned(4)));
        const u2 v = *reinterpret_cast<const u2 *>(static_cast<const float *>(base) + idx);
        r.w[2 * row] = v[0]; r.w[2 * row + 1] = v[1];
    } else {
        typedef uint32_t u1 __attribute__((aligned(2)));
        r.w[row] = *reinterpret_cast<const u1 *>(static_cast<const uint16_t *>(base) + idx);
    }
}

constexpr int WT_ROWS = 32, WT_STRIDE = WT_ROWS + 8;  // rows of a step; halves between the columns in LDS

template <class T, int NA, int NB, int MASK>
__global__ __launch_bounds__(256, NA * NB >= 64 ? 2 : NA * NB >= 32 ? 3 : 4) void weight_grad_tile_kernel(
    int n, const void *__restrict__ X, int ldx, int d_in, const float *__restrict__ G, int ldg, int d_out, const void *__restrict__ Y,
    int ldy, unsigned limit, float *__restrict__ partial, int ldp, int splits)
{
    constexpr int PX = T::BYTES == 4 ? 3 : std::is_same<T, F16>::value ? 2 : 1;
    constexpr int WB = NB >= 4 ? 2 : 1, WA = 4 / WB;  // waves across
    constexpr int PA = NA / WA, PB = NB / WB;         // tiles of a wave
    static_assert(PA >= 1 && PB >= 1, "every wave has a tile");
    constexpr int XU = NA * 8 * 4, GU = NB * 8 * 4;   // units (two columns, eight rows) of a step
    constexpr int XP = (XU + 255) / 256, GP = (GU + 255) / 256;
    __shared__ __align__(16) uint16_t Xs[PX][NA * 16 * WT_STRIDE];
    __shared__ __align__(16) uint16_t Gs[3][NB * 16 * WT_STRIDE];
    __shared__ int odd_s[2];  // some of this step's numbers can't be taken in pieces
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int m = lane & 15, kb = lane >> 4;
    const int wa = wave / WB * PA, wb = wave % WB * PB;  // this wave's first tiles
    const int a0 = blockIdx.y * (16 * NA), b0 = blockIdx.z * (16 * NB);
    const int64_t per = ((static_cast<int64_t>(n) + splits - 1) / splits + WT_ROWS - 1) / WT_ROWS * WT_ROWS;
    const int64_t r_begin = per * blockIdx.x, r_end = min(static_cast<int64_t>(n), r_begin + per);
    split_f32x4 acc[PA][PB];
#pragma unroll
    for (int i = 0; i < PA; ++i)
#pragma unroll
        for (int j = 0; j < PB; ++j) acc[i][j] = split_f32x4{0.f, 0.f, 0.f, 0.f};
    if (tid < 2) odd_s[tid] = 0;

    PairRaw<T> xr[XP];
    PairRaw<F32> gr[GP];
    PairRaw<F32> yr[MASK == 1 ? GP : 1];
    PairRaw<F16> hr[MASK == 2 ? GP : 1];
    // Eight rows from r0 + k on of the pair of columns from c on; rows beyond the end are the last one.  Where the matrix ends with one
    // column the pair is moved back by it.
    auto load_unit = [&](auto &raw, auto type, const void *base, int64_t ld, int c, int d, int64_t r0, int k, bool full) {
        using E = decltype(type);
        const int64_t row = min(r0 + k, r_end - 1);
        const char *p = static_cast<const char *>(base) + (row * ld + min(c, d - 2)) * E::BYTES;
        const int64_t ldb = ld * E::BYTES;
        const int last = static_cast<int>(min(r_end - 1 - row, static_cast<int64_t>(7)));
#pragma unroll
        for (int j = 0; j < 8; ++j) load_pair<E>(p + (full ? j : min(j, last)) * ldb, 0, raw, j);
    };
    auto load_step = [&](int64_t r0) {
        const bool full = r0 + WT_ROWS <= r_end;
#pragma unroll
        for (int u = 0; u < XP; ++u) {
            const int t = tid + u * 256;
            if (XU % 256 == 0 || t < XU) load_unit(xr[u], T{}, X, ldx, a0 + 2 * (t % (8 * NA)), d_in, r0, t / (8 * NA) * 8, full);
        }
#pragma unroll
        for (int u = 0; u < GP; ++u) {
            const int t = tid + u * 256;
            if (GU % 256 != 0 && t >= GU) continue;
            const int c = b0 + 2 * (t % (8 * NB)), k = t / (8 * NB) * 8;
            load_unit(gr[u], F32{}, G, ldg, c, d_out, r0, k, full);
            if constexpr (MASK == 1) load_unit(yr[u], F32{}, Y, ldy, c, d_out, r0, k, full);
            if constexpr (MASK == 2) load_unit(hr[u], F16{}, Y, ldy, c, d_out, r0, k, full);
        }
    };
    // pieces of a unit's two columns into LDS; columns and rows beyond the end are zero
    auto put = [&](const float (&v0)[8], const float (&v1)[8], auto pieces, uint16_t *s, int t, int cols2, int c0, int d, int64_t r0) {
        constexpr int P = decltype(pieces)::value;
        const int cl = 2 * (t % cols2), c = c0 + cl, k = t / cols2 * 8;
        const bool moved = c + 1 == d;
        const int left = static_cast<int>(min(static_cast<int64_t>(8), r_end - r0 - k));
        bool odd = false;
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            float f[8];
            const int rows = c + q < d ? left : 0;
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const float v = q == 1 || moved ? v1[j] : v0[j];
                f[j] = j < rows ? v : 0.f;
            }
            uint4 p[3];
            if constexpr (P == 1) {
#pragma unroll
                for (int j = 0; j < 8; ++j) odd |= __builtin_amdgcn_classf(f[j], 0x207);  // infinite or NaN: times a piece of G that is zero
                p[0] = make_uint4(bf16_pair(f[0], f[1]), bf16_pair(f[2], f[3]), bf16_pair(f[4], f[5]), bf16_pair(f[6], f[7]));
            } else {
                odd |= split8(f, p);
            }
#pragma unroll
            for (int i = 0; i < P; ++i) *reinterpret_cast<uint4 *>(s + i * (cols2 * 2 * WT_STRIDE) + (cl + q) * WT_STRIDE + k) = p[i];
        }
        return odd;
    };
    // a step in fp32, from X and G as they are; no barrier
    auto plain_step = [&](int64_t r0) {
#pragma unroll 1
        for (int k = 0; k < 8; ++k) {
            const int64_t row = r0 + kb * 8 + k, rc = min(row, r_end - 1);
            float a[PA], b[PB];
#pragma unroll
            for (int i = 0; i < PA; ++i) {
                const int c = a0 + (wa + i) * 16 + m;
                const float v = load_elem(X, rc * ldx + min(c, d_in - 1), T::BYTES == 4 ? FTC_F32 : std::is_same<T, F16>::value ? FTC_F16 : FTC_BF16);
                a[i] = c < d_in && row < r_end ? v : 0.f;
            }
#pragma unroll
            for (int j = 0; j < PB; ++j) {
                const int c = b0 + (wb + j) * 16 + m, cc = min(c, d_out - 1);
                float v = G[rc * ldg + cc];
                if constexpr (MASK == 1) v = static_cast<const float *>(Y)[rc * ldy + cc] > 0.f ? v : 0.f;
                if constexpr (MASK == 2) {
                    const unsigned y = static_cast<const uint16_t *>(Y)[rc * ldy + cc];
                    v = (y != 0u && y <= limit) ? v : 0.f;
                }
                b[j] = c < d_out && row < r_end ? v : 0.f;
            }
#pragma unroll
            for (int i = 0; i < PA; ++i)
#pragma unroll
                for (int j = 0; j < PB; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[i], b[j], acc[i][j], 0, 0, 0);
        }
    };
    if (r_begin < r_end) load_step(r_begin);
    __syncthreads();  // odd_s is cleared before any wave sets it in the first step
    int step = 0;
    bool pieces = false;  // uniform: some steps were taken in pieces
    for (int64_t r0 = r_begin; r0 < r_end; r0 += WT_ROWS, ++step) {  // uniform
        bool odd = false;
#pragma unroll
        for (int u = 0; u < XP; ++u) {
            const int t = tid + u * 256;
            if (XU % 256 != 0 && t >= XU) continue;
            float v0[8], v1[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) { v0[j] = pair_value<T>(xr[u], j, 0); v1[j] = pair_value<T>(xr[u], j, 1); }
            odd |= put(v0, v1, std::integral_constant<int, PX>{}, &Xs[0][0], t, 8 * NA, a0, d_in, r0);
        }
#pragma unroll
        for (int u = 0; u < GP; ++u) {
            const int t = tid + u * 256;
            if (GU % 256 != 0 && t >= GU) continue;
            float v0[8], v1[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                v0[j] = pair_value<F32>(gr[u], j, 0); v1[j] = pair_value<F32>(gr[u], j, 1);
                if constexpr (MASK == 1) {
                    v0[j] = pair_value<F32>(yr[u], j, 0) > 0.f ? v0[j] : 0.f;
                    v1[j] = pair_value<F32>(yr[u], j, 1) > 0.f ? v1[j] : 0.f;
                } else if constexpr (MASK == 2) {
                    const unsigned y0 = hr[u].w[j] & 0xffffu, y1 = hr[u].w[j] >> 16;
                    v0[j] = (y0 != 0u && y0 <= limit) ? v0[j] : 0.f;  // positive, not NaN
                    v1[j] = (y1 != 0u && y1 <= limit) ? v1[j] : 0.f;
                }
            }
            odd |= put(v0, v1, std::integral_constant<int, 3>{}, &Gs[0][0], t, 8 * NB, b0, d_out, r0);
        }
        if (odd) odd_s[step & 1] = 1;
        __syncthreads();
        if (r0 + WT_ROWS < r_end) load_step(r0 + WT_ROWS);
        if (tid == 0) odd_s[(step + 1) & 1] = 0;
        if (!__builtin_amdgcn_readfirstlane(odd_s[step & 1])) {
            pieces = true;
            uint4 b[PB][3];
#pragma unroll
            for (int j = 0; j < PB; ++j)
#pragma unroll
                for (int q = 0; q < 3; ++q) b[j][q] = *reinterpret_cast<const uint4 *>(&Gs[q][((wb + j) * 16 + m) * WT_STRIDE + kb * 8]);
#pragma unroll
            for (int i = 0; i < PA; ++i) {
                asm volatile("" ::: "memory");  // (else all tiles' loads are moved up here, and their registers with them)
                uint4 a[PX];
#pragma unroll
                for (int q = 0; q < PX; ++q) a[q] = *reinterpret_cast<const uint4 *>(&Xs[q][((wa + i) * 16 + m) * WT_STRIDE + kb * 8]);
#pragma unroll
                for (int j = 0; j < PB; ++j) {
                    split_f32x4 small = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int sum = 2; sum >= 1; --sum)
#pragma unroll
                        for (int q = 0; q < PX; ++q)
                            if (sum - q >= 0 && sum - q < 3)
                                small = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(split_bf16x8, a[q]), __builtin_bit_cast(split_bf16x8, b[j][sum - q]), small, 0, 0, 0);
                    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(split_bf16x8, a[0]), __builtin_bit_cast(split_bf16x8, b[j][0]), acc[i][j], 0, 0, 0);
                    acc[i][j] += small;
                }
            }
        } else {
            plain_step(r0);
        }
        __syncthreads();
    }
    float zero = 0.f;
#pragma unroll
    for (int i = 0; i < PA; ++i)
#pragma unroll
        for (int j = 0; j < PB; ++j) zero = not_finite(acc[i][j], zero);
    if (__builtin_expect(pieces && __builtin_amdgcn_ballot_w64(zero != 0.f) != 0, 0)) {  // pieces may have made it so: this wave's sums without them
#pragma unroll
        for (int i = 0; i < PA; ++i)
#pragma unroll
            for (int j = 0; j < PB; ++j) acc[i][j] = split_f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
        for (int64_t r0 = r_begin; r0 < r_end; r0 += WT_ROWS) plain_step(r0);
    }
    float *out = partial + static_cast<size_t>(blockIdx.x) * d_in * ldp;
#pragma unroll
    for (int i = 0; i < PA; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int a = a0 + (wa + i) * 16 + kb * 4 + e;
            if (a >= d_in) continue;
#pragma unroll
            for (int j = 0; j < PB; ++j) {
                const int b = b0 + (wb + j) * 16 + m;
                if (b < d_out) out[static_cast<size_t>(a) * ldp + b] = acc[i][j][e];
            }
        }
}

// The tile, or none: weight_grad_kernel, by the time of a row next to `other`, that kernel's (10^-4 ps, as in its table): padded columns of X
// times those of G times 255, 250 or 170 for 4 x 4, 8 x 4 and 8 x 8 tiles, and 2 or (8 x 8) 4 us for the first step and the sum over
// the shares.  Up to 32 columns on either side and below 32 768 rows it is always the other one (1 000 000 x 128, 32 fp32 134 us there, 131 here;
// 15 000 x 128, 128 17.7 / 18.2).  Of 1926 products (fp32 and fp16, 33 to 500 by 33 to 256 columns, 16 384 to 10^6 rows), each with and
// without the mask, this rule takes 0.84 of weight_grad_kernel's time on average (the best of all four choices 0.81) and in 47 of 3852
// more than 1.03 times, at most 1.17; 8 tiles of X wherever G has more than 64 columns, and no table, 0.87, 623 and 1.52 (500 000 x 33, 200 fp32 with
// the mask 291 / 463 us, 4 x 4 tiles 327; 200 000 x 40, 72 44 / 59, now weight_grad_kernel).
WgPieces weight_grad_pieces(int n, int d_in, int d_out, int64_t other)
{
    if (n < 32768 || d_in <= 32 || d_out <= 32) return {0, 0};
    auto padded = [](int d, int t) { return (static_cast<int64_t>(d) + t - 1) / t * t; };
    struct { WgPieces tile; int64_t cost, us; } const tiles[] = {{{4, 4}, 255, 2}, {{8, 4}, 250, 2}, {{8, 8}, 170, 4}};
    WgPieces best = {0, 0};
    int64_t least = other + other / 20;
    for (const auto &t : tiles) {
        const int64_t cost = padded(d_in, 16 * t.tile.na) * padded(d_out, 16 * t.tile.nb) * t.cost + t.us * 10000000000 / n;
        if (cost < least) {
            least = cost;
            best = t.tile;
        }
    }
    return best;
}

template <class T>
static void wt_launch(WgPieces t, int mask, hipStream_t s, int n, const void *X, int ldx, int d_in, const float *G, int ldg, int d_out,
                      const void *Y, int ldy, unsigned limit, float *partial, int splits)
{
    const dim3 grid(splits, (d_in + 16 * t.na - 1) / (16 * t.na), (d_out + 16 * t.nb - 1) / (16 * t.nb));
#define FTC_WT(A, N, M)                                                                                                           \
    hipLaunchKernelGGL((weight_grad_tile_kernel<T, A, N, M>), grid, dim3(256), 0, s, n, X, ldx, d_in, G, ldg, d_out, Y, ldy, limit, partial, \
                       d_out, splits)
#define FTC_WTN(A, N)                      \
    if (t.na == A && t.nb == N) {          \
        if (mask == 0) FTC_WT(A, N, 0);    \
        else if (mask == 1) FTC_WT(A, N, 1); \
        else FTC_WT(A, N, 2);              \
    }
    FTC_WTN(4, 4) FTC_WTN(8, 4) FTC_WTN(8, 8)
#undef FTC_WTN
#undef FTC_WT
}

void launch_weight_grad_tile(WgPieces t, int n, const void *X, int ldx, int xdt, int d_in, const float *G, int ldg, int d_out, const void *Y,
                             int ldy, int mask, unsigned limit, float *partial, int splits, hipStream_t s)
{
    if (xdt == FTC_F32) wt_launch<F32>(t, mask, s, n, X, ldx, d_in, G, ldg, d_out, Y, ldy, limit, partial, splits);
    else if (xdt == FTC_F16) wt_launch<F16>(t, mask, s, n, X, ldx, d_in, G, ldg, d_out, Y, ldy, limit, partial, splits);
    else wt_launch<BF16>(t, mask, s, n, X, ldx, d_in, G, ldg, d_out, Y, ldy, limit, partial, splits);
}

}  // namespace ftc
