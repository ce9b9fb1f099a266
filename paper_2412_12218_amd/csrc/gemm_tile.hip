// Dense products Z = X W of many rows at any alignment and width on the 16-bit matrix cores (v_mfma_f32_16x16x32), 16-bit
// inputs as they are, fp32 inputs in three exact bf16 pieces (bf16_split.hpp); and dX = G W^T, the same with W transposed (TRANS).
//
// A wave owns 16 rows of X and up to 16 NT columns; a workgroup, four waves, stages a chunk of KC rows of W in LDS, columns
// first, in the operands' layout (eight consecutive k of a column are one 16-byte word), in pieces.
//   A operand  lane l holds X[row0 + l%16][k0 + (l/16) 8 .. +7], loaded at element alignment; the chunk's are all loaded before W is
//              staged, so that a chunk waits for memory once;
//   C          W is the first operand of the instruction (QUADS): lane l holds Z[row0 + l%16][n0 + (l/16) 4 + i], four columns that leave in
//              one store at the alignment of an element.  With X first, a column a lane, us, that way / this: dX fp16 2^20 rows 8 -> 32 48 / 34,
//              fp32 100 000 rows 10 -> 128 29 / 24, Z 300 -> 128 82.5 / 79.3, fp16 179 245 x 18 -> 64 18.1 / 13.7, 400 000 x 301 -> 128 287 / 267; fp32 into
//              at most 16 columns over more than one chunk this way too, but with seven workgroups on some compute units (gemm_tile_t()).
// Where one chunk holds all of W a workgroup walks over the rows and stages it once.
//
// Bound by reading X (and writing Z) up to about 32 columns, then by the chain load, stage, multiply of a chunk, which four workgroups
// on a CU share.  Products and sums are no less exact than on v_mfma_f32_16x16x4_f32, where these products were before: six or one
// instruction for what were eight, so fewer roundings, and the chunks' sums of 16-bit inputs are added up apart.  us and
// error against 64 bits (2-norm), there / here:
//   fp32  100 000 x 300 -> 128 112 / 78 (2.2e-7 / 0.9e-7), 400 000 x 301 -> 128 427 / 342, 100 000 x 500 -> 40 94 / 61, 1 000 000 x 33 -> 2
//         57 / 40, 16 000 x 300 -> 128 40 / 19
//   fp16  100 000 x 300 -> 128 110 / 45 (2.1e-7 / 0.8e-7), 400 000 x 301 -> 128 440 / 180, 179 245 x 18 -> 64 27 / 15, 16 000 x 1433 -> 32 47 / 28
//   bf16  100 000 x 500 -> 40 91 / 35 (1.0e-7 / 0.6e-7), 5000 x 3001 -> 128 176 / 85 (1.3e-7 / 1.1e-7)
// and against 16-bit rows staged in chunks of 256 for 256 rows at a time (aligned rows): fp16 20 000 x 304 -> 64 46 / 11, 100 000 x 1432 -> 16
// 92 / 65, 400 000 x 128 -> 128 189 / 108.  Many 16-bit rows of 256 (192) elements and more into more than 32 columns
// have a kernel of their own since (gemm_rows_kernel).
// Tried: eight waves instead of four (W staged half as often: 300 -> 128 level, 1433 -> 16 12 % slower), the next chunk of X in registers
// (5 to 15 % slower), 128 columns of fp32 (107 us for 78: registers).
#include "bf16_split.hpp"

namespace ftc {

typedef _Float16 gt_half8 __attribute__((ext_vector_type(8)));

template <class T>
struct GemmChunk {
    static constexpr int PIECES = T::BYTES == 4 ? 3 : 1;
    static constexpr int KC = T::BYTES == 4 ? 64 : 128;
};

// 8 elements at idx, elements from `left` on are zero and not read
template <class T>
struct Eight {
    float f[T::BYTES == 4 ? 8 : 1];
    uint4 h;
};
template <class T>
__device__ __forceinline__ void load_eight(const void *base, int64_t idx, int left, Eight<T> &e)
{
    if constexpr (T::BYTES == 4) {
        const float *p = static_cast<const float *>(base) + idx;
        if (left >= 8) {
            typedef float f4 __attribute__((ext_vector_type(4), aligned(4)));
            const f4 a = *reinterpret_cast<const f4 *>(p), b = *reinterpret_cast<const f4 *>(p + 4);
#pragma unroll
            for (int j = 0; j < 4; ++j) { e.f[j] = a[j]; e.f[4 + j] = b[j]; }
        } else {
#pragma unroll
            for (int j = 0; j < 8; ++j) e.f[j] = j < left ? p[j] : 0.f;
        }
    } else {
        const uint16_t *p = static_cast<const uint16_t *>(base) + idx;
        if (left >= 8) {
            typedef uint32_t u4 __attribute__((ext_vector_type(4), aligned(2)));
            const u4 a = *reinterpret_cast<const u4 *>(p);
            e.h = make_uint4(a[0], a[1], a[2], a[3]);
        } else {
            uint32_t w[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) w[j] = j < left ? p[j] : 0u;
            e.h = make_uint4(w[0] | (w[1] << 16), w[2] | (w[3] << 16), w[4] | (w[5] << 16), w[6] | (w[7] << 16));
        }
    }
}

template <class T>
__device__ __forceinline__ float eight_value(const Eight<T> &e, int j)
{
    if constexpr (T::BYTES == 4) return e.f[j];
    else {
        const uint32_t w = j < 2 ? e.h.x : j < 4 ? e.h.y : j < 6 ? e.h.z : e.h.w, b = j & 1 ? w >> 16 : w & 0xffffu;
        return std::is_same<T, F16>::value ? f16_bits_to_f32(b) : bf16_bits_to_f32(b);
    }
}

// TW: the type of W, another than X's only for TRANS.
template <class T, int NT, bool TRANS, bool QUADS, class TW>
__global__ __launch_bounds__(256, NT == 8 ? 2 : NT == 2 && !TRANS ? 5 : 4) void gemm_tile_kernel(int n, const void *__restrict__ X, int ldx, int d_in,
                                                                         const void *__restrict__ W, int w_ld, int d_out,
                                                                         void *__restrict__ Z, int ldz, int zdt, Epi epi, int n_blocks,
                                                                         int neighbours)
{
    static_assert(TRANS ? T::BYTES == 4 : std::is_same<T, TW>::value, "types of the products");
    constexpr int P = GemmChunk<T>::PIECES, KC = GemmChunk<T>::KC, KP = KC + 8, COLS = 16 * NT, STEPS = KC / 32, SB = 2;
    __shared__ __align__(16) uint16_t Ws[P][COLS * KP];
    __shared__ int w_odd;  // some of W can't be taken in pieces
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int m = lane & 15, kb = lane >> 4;
    int first = blockIdx.x, group = blockIdx.y;
    if (TRANS && neighbours) {  // the groups of a block of rows one after the other on one of the eight dies (gridDim.x is a multiple of 8)
        const unsigned id = blockIdx.y * gridDim.x + blockIdx.x, slot = id / 8u;
        group = static_cast<int>(slot % gridDim.y);
        first = static_cast<int>(slot / gridDim.y * 8u + id % 8u);
    }
    const int col0 = group * COLS, cols = min(COLS, d_out - col0);
    const bool whole = d_in <= KC;
    constexpr int WDT = TW::BYTES == 4 ? FTC_F32 : std::is_same<TW, F16>::value ? FTC_F16 : FTC_BF16;
    auto w_index = [&](int k, int o) {
        return TRANS ? static_cast<int64_t>(col0 + o) * w_ld + k : static_cast<int64_t>(k) * w_ld + col0 + o;
    };
    if (P == 3 && tid == 0) w_odd = 0;
    for (int block = first; block < n_blocks; block += gridDim.x) {  // uniform
        const int64_t row0 = (static_cast<int64_t>(block) * 4 + wave) * 16;
        const int64_t at = min(row0 + m, static_cast<int64_t>(n) - 1) * ldx;  // clamped: stores are predicated
        // several sums per element: of the large and of the small products (fp32); of the first and second half of a chunk (16 bits)
        constexpr int TOTAL = P == 3 ? 1 : NT == 8 ? 1 : 2;  // 16 bits: sum over the chunks, the others are the chunk's
        split_f32x4 acc[TOTAL + 1][NT];
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            acc[0][nt] = acc[1][nt] = acc[TOTAL][nt] = split_f32x4{0.f, 0.f, 0.f, 0.f};
        }
        Eight<T> x[STEPS];
        auto load_x = [&](int kc, Eight<T> (&to)[STEPS]) {
#pragma unroll
            for (int s = 0; s < STEPS; ++s)
                if (kc + s * 32 < d_in) load_eight<T>(X, at + kc + s * 32 + kb * 8, d_in - kc - s * 32 - kb * 8, to[s]);
        };
        bool odd = false;
        for (int kc0 = 0; kc0 < d_in; kc0 += KC) {  // uniform
            load_x(kc0, x);
            if (!whole || block == first) {
                __syncthreads();  // the previous chunk has been consumed
                const int k_end = min(KC, (d_in - kc0 + 31) / 32 * 32);
                const int units = k_end / 8 * COLS;
#pragma unroll 1
                for (int t0 = tid; t0 < units; t0 += 256 * SB) {  // consecutive threads: consecutive columns (TRANS: k)
                    float w[SB][P == 3 ? 8 : 1];
                    uint32_t h[SB][P == 3 ? 1 : 8];
#pragma unroll
                    for (int u = 0; u < SB; ++u) {  // all loads of SB units in flight, from clamped addresses
                        const int t = min(t0 + u * 256, units - 1);
                        const int o = TRANS ? t / (k_end / 8) : t % COLS, k = (TRANS ? t % (k_end / 8) : t / COLS) * 8;
                        const int left = o < cols ? d_in - kc0 - k : 0;
                        const int64_t at_w = left > 0 ? w_index(kc0 + k, o) : 0;
                        // The type of W is a template's: with one known at run time only each load was waited for at its branch's end
                        // (dX of 400 000 x 128 from 128 columns, us: 303 / 155, of 100 000 x 301 182 / 92, of 200 000 x 128 from one 31 / 28).
                        if constexpr (TRANS) {
                            if (kc0 + k_end <= d_in) {  // uniform: eight elements of a row of W are there
                                Eight<TW> e;
                                load_eight<TW>(W, at_w, 8, e);
#pragma unroll
                                for (int j = 0; j < 8; ++j) w[u][j] = left > 0 ? eight_value(e, j) : 0.f;
                                continue;
                            }
                        }
#pragma unroll
                        for (int j = 0; j < 8; ++j) {
                            const int64_t i = at_w + (j < left ? static_cast<int64_t>(j) * (TRANS ? 1 : w_ld) : 0);
                            if constexpr (P == 3) {
                                const float v = load_elem(W, i, WDT);
                                w[u][j] = j < left ? v : 0.f;
                            } else {
                                const uint32_t v = static_cast<const uint16_t *>(W)[i];
                                h[u][j] = j < left ? v : 0u;
                            }
                        }
                    }
#pragma unroll
                    for (int u = 0; u < SB; ++u) {
                        const int t = t0 + u * 256;
                        if (u > 0 && t >= units) break;
                        const int o = TRANS ? t / (k_end / 8) : t % COLS, k = (TRANS ? t % (k_end / 8) : t / COLS) * 8;
                        if constexpr (P == 3) {
                            uint4 p[3];
                            if (split8(w[u], p)) w_odd = 1;
#pragma unroll
                            for (int q = 0; q < 3; ++q) *reinterpret_cast<uint4 *>(&Ws[q][o * KP + k]) = p[q];
                        } else {
                            *reinterpret_cast<uint4 *>(&Ws[0][o * KP + k]) = make_uint4(h[u][0] | (h[u][1] << 16), h[u][2] | (h[u][3] << 16),
                                                                                       h[u][4] | (h[u][5] << 16), h[u][6] | (h[u][7] << 16));
                        }
                    }
                }
                __syncthreads();
            }
#pragma unroll
            for (int s = 0; s < STEPS; ++s) {
                if (s > 0 && kc0 + s * 32 >= d_in) break;  // uniform
                uint4 a[3];
                if constexpr (P == 3) odd |= split8(x[s].f, a);
                uint4 b[2][P];  // of this tile of columns and of the next
                auto load_b = [&](int nt) {
#pragma unroll
                    for (int q = 0; q < P; ++q)
                        b[nt & 1][q] = *reinterpret_cast<const uint4 *>(&Ws[q][(nt * 16 + m) * KP + s * 32 + kb * 8]);
                };
                load_b(0);
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) {
                    if (nt + 1 < NT) load_b(nt + 1);
                    asm volatile("" ::: "memory");  // (else all tiles' loads are moved up here, and their registers with them)
                    if constexpr (P == 3) {
                        if constexpr (QUADS) mfma_split(b[nt & 1], a, acc[0][nt], acc[1][nt]);
                        else mfma_split(a, b[nt & 1], acc[0][nt], acc[1][nt]);
                    } else {
                        split_f32x4 &c = acc[TOTAL == 2 ? s >> 1 : 0][nt];
                        const uint4 first = b[nt & 1][0], second = x[s].h;
                        if constexpr (std::is_same<T, F16>::value)
                            c = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(gt_half8, first), __builtin_bit_cast(gt_half8, second), c, 0, 0, 0);
                        else
                            c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(split_bf16x8, first), __builtin_bit_cast(split_bf16x8, second), c, 0, 0, 0);
                    }
                }
            }
            if constexpr (P == 1) {
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) {
                    acc[TOTAL][nt] += TOTAL == 2 ? acc[0][nt] + acc[1][nt] : acc[0][nt];
                    acc[0][nt] = split_f32x4{0.f, 0.f, 0.f, 0.f};
                    if constexpr (TOTAL == 2) acc[1][nt] = acc[0][nt];
                }
            }
        }
        if constexpr (P == 3) {
            float zero = 0.f;
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) zero = not_finite(acc[0][nt] + acc[1][nt], zero);
            // numbers that can't be taken in pieces: the tile again, in fp32, from X and W as they are.  Product j of a step takes the j-th of every
            // lane's eight indices.  Bound by its loads of W, which every wave makes itself.
            if (__builtin_expect(__builtin_amdgcn_ballot_w64(odd || zero != 0.f) != 0 || w_odd, 0)) {
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) acc[0][nt] = acc[1][nt] = split_f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
                for (int k0 = 0; k0 < d_in; k0 += 32) {
                    int k = k0 + kb * 8;
                    asm volatile("" : "+v"(k));  // (else addresses are kept over all of the kernel)
                    Eight<T> xe;
                    load_eight<T>(X, at + (k < d_in ? k : 0), d_in - k, xe);
#pragma unroll
                    for (int nt = 0; nt < NT; ++nt) {
                        const int left = nt * 16 + m < cols ? d_in - k : 0;
                        float b[8];
                        if constexpr (TRANS) {
                            Eight<TW> e;
                            load_eight<TW>(W, left > 0 ? w_index(k, nt * 16 + m) : 0, left, e);
#pragma unroll
                            for (int j = 0; j < 8; ++j) b[j] = eight_value(e, j);
                        } else {
#pragma unroll
                            for (int j = 0; j < 8; ++j) {
                                const float v = load_elem(W, j < left ? w_index(k + j, nt * 16 + m) : 0, WDT);
                                b[j] = j < left ? v : 0.f;
                            }
                        }
#pragma unroll
                        for (int j = 0; j < 8; ++j) {
                            split_f32x4 &c = acc[j & 1][nt];
                            c = QUADS ? __builtin_amdgcn_mfma_f32_16x16x4f32(b[j], xe.f[j], c, 0, 0, 0)
                                      : __builtin_amdgcn_mfma_f32_16x16x4f32(xe.f[j], b[j], c, 0, 0, 0);
                        }
                        asm volatile("" ::: "memory");  // (else all tiles' loads are moved up here, and their registers with them)
                    }
                }
            }
        }
        if constexpr (!QUADS) {
            static_assert(P == 3, "16-bit operands change places");
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int64_t row = row0 + kb * 4 + i;
                if (row >= n) continue;
                const float f = epi.factor(row);
#pragma unroll
                for (int nt = 0; nt < NT; ++nt)
                    if (nt * 16 + m < cols) store_elem(Z, row * ldz + col0 + nt * 16 + m, zdt, epi.apply(f, acc[0][nt][i] + acc[1][nt][i]));
            }
        } else if (row0 + m < n) {
            const int64_t row = row0 + m;
            const float f = epi.factor(row);
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
                const int o = nt * 16 + kb * 4;
                float z[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) z[i] = epi.apply(f, P == 3 ? acc[0][nt][i] + acc[1][nt][i] : acc[TOTAL][nt][i]);
                if (o + 4 <= cols) {
                    store_vec_any<4>(Z, row * ldz + col0 + o, zdt, z);
                } else {
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        if (o + i < cols) store_elem(Z, row * ldz + col0 + o + i, zdt, z[i]);
                }
            }
        }
    }
}

// fp32 products of at most 4 KS indices: KS v_mfma_f32_16x16x4_f32 a tile, lane l holding index l/16 of four; rows, columns, stores and
// `neighbours` as above.  W stays in registers.  Up to SPLIT_FROM indices for the exact products, dX up to FEW_BACK for the time.  Bound by writing Z.  us, in
// pieces / here: 200 000 x 1 -> 128 22.9 / 18.4, 1 000 000 x 4 -> 8 20.2 / 9.9; dX with dW (with input_grad_kernel before) 200 000 x 128 from one column 47.0
// / 44.1 (51.5), 602 932 x 120 from 8 190 / 179 (178), 213 277 x 331 from 8 210 / 197 (205), 100 000 x 300 from 8 68 / 62 (72), 1 000 000 x 128 from 3 300 / 286 (274).
// Tried: an fp32 product a lane and column, whole rows a wave (400 000 x 128 from 7 123 us for 110); non-temporal stores (1 000 000 x 64 from 4
// 155 / 135, but 224 774 x 506 from 2, where rows are no whole lines, 270 / 551).
constexpr int FEW_BACK = 8;

template <int NT, int KS, bool TRANS, class TW>
__global__ __launch_bounds__(256) void gemm_few_kernel(int n, const float *__restrict__ X, int ldx, int d_in, const void *__restrict__ W, int w_ld,
                                                       int d_out, void *__restrict__ Z, int ldz, int zdt, Epi epi, int n_blocks, int neighbours)
{
    constexpr int COLS = 16 * NT;
    constexpr int WDT = TW::BYTES == 4 ? FTC_F32 : std::is_same<TW, F16>::value ? FTC_F16 : FTC_BF16;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int m = lane & 15, kb = lane >> 4;
    int first = blockIdx.x, group = blockIdx.y;
    if (TRANS && neighbours) {
        const unsigned id = blockIdx.y * gridDim.x + blockIdx.x, slot = id / 8u;
        group = static_cast<int>(slot % gridDim.y);
        first = static_cast<int>(slot / gridDim.y * 8u + id % 8u);
    }
    const int col0 = group * COLS, cols = min(COLS, d_out - col0);
    float w[KS][NT];
#pragma unroll
    for (int q = 0; q < KS; ++q)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            const int o = nt * 16 + m, k = q * 4 + kb;
            const bool in = k < d_in && o < cols;
            const int64_t i = TRANS ? static_cast<int64_t>(col0 + o) * w_ld + k : static_cast<int64_t>(k) * w_ld + col0 + o;
            const float v = load_elem(W, in ? i : 0, WDT);
            w[q][nt] = in ? v : 0.f;
        }
    for (int block = first; block < n_blocks; block += gridDim.x) {  // uniform
        const int64_t row = (static_cast<int64_t>(block) * 4 + wave) * 16 + m;
        split_f32x4 c[NT];
#pragma unroll
        for (int q = 0; q < KS; ++q) {
            const int k = q * 4 + kb;
            const float v = X[min(row, static_cast<int64_t>(n) - 1) * ldx + min(k, d_in - 1)], x = k < d_in ? v : 0.f;
#pragma unroll
            for (int nt = 0; nt < NT; ++nt)
                c[nt] = __builtin_amdgcn_mfma_f32_16x16x4f32(w[q][nt], x, q == 0 ? split_f32x4{0.f, 0.f, 0.f, 0.f} : c[nt], 0, 0, 0);
        }
        if (row >= n) continue;
        const float f = epi.factor(row);
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            const int o = nt * 16 + kb * 4;
            float z[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) z[i] = epi.apply(f, c[nt][i]);
            if (o + 4 <= cols) {
                store_vec_any<4>(Z, row * ldz + col0 + o, zdt, z);
            } else {
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if (o + i < cols) store_elem(Z, row * ldz + col0 + o + i, zdt, z[i]);
            }
        }
    }
}

// 16-bit products of long rows, RT tiles of 16 rows a wave: an operand of W that comes from LDS is used RT times and a chunk of W staged for
// 64 RT rows, where one tile a wave (above) waits for both.  A workgroup has 64 RT rows and up to 64 columns, W in chunks of 256 indices (34 KB);
// the groups of 64 columns of the same rows follow one another on one of the eight dies.  Sums of 128 indices
// (SETS = 2: of 64, in pairs) are added up apart, as in the kernel above with 128 (up to 64) columns: the same results.  Registers set the
// workgroups on a compute unit, two (RT = 2: three, 12 registers spilled: 400 000 x 400 -> 33 121 us, 141 with two).  us, by
// gemm_tile_kernel / here (before both, with four tiles a wave too, a launch per 64 columns, other instructions for odd rows): fp16 400 000 x 512 -> 129 718 / 257 (470), -> 65 360 / 192 (292), -> 128 370 / 199 (331), 200 000 x 512 -> 160 353 / 125 (253),
// 1433 -> 128 100 000 rows 311 / 245 (498), 400 000 x 512 -> 40 169 / 133 (149), odd rows 244 / 199 (354).
template <class T, int RT, int SETS>
__global__ __launch_bounds__(256, RT == 4 ? 2 : 3) void gemm_rows_kernel(int n, const void *__restrict__ X, int ldx, int d_in, const uint16_t *__restrict__ W,
                                                           int d_out, void *__restrict__ Z, int ldz, int zdt, Epi epi, int n_batches, int groups)
{
    constexpr int NT = 4, KC = 256, KP = KC + 8, COLS = 16 * NT, SB = 2;
    __shared__ __align__(16) uint16_t Ws[COLS * KP];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int m = lane & 15, kb = lane >> 4;
    const unsigned slot = blockIdx.x / 8u;  // gridDim.x is a multiple of 8 groups
    const int col0 = static_cast<int>(slot % groups) * COLS, cols = min(COLS, d_out - col0);
    const int first = static_cast<int>(slot / groups * 8u + blockIdx.x % 8u), step = static_cast<int>(gridDim.x / groups);
    const bool whole = d_in <= KC;
    for (int batch = first; batch < n_batches; batch += step) {  // uniform
        const int64_t row0 = (static_cast<int64_t>(batch) * 4 + wave) * (16 * RT);
        int64_t at[RT];
        split_f32x4 total[RT][NT], c[SETS][RT][NT];
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) {
            at[rt] = min(row0 + rt * 16 + m, static_cast<int64_t>(n) - 1) * ldx;  // clamped: stores are predicated
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) total[rt][nt] = c[0][rt][nt] = c[SETS - 1][rt][nt] = split_f32x4{0.f, 0.f, 0.f, 0.f};
        }
        for (int kc0 = 0; kc0 < d_in; kc0 += KC) {  // uniform
            if (!whole || batch == first) {
                __syncthreads();  // the previous chunk has been consumed
                const int units = min(KC, (d_in - kc0 + 31) / 32 * 32) / 8 * COLS;
                for (int t0 = tid; t0 < units; t0 += 256 * SB) {
                    uint32_t h[SB][8];
#pragma unroll
                    for (int u = 0; u < SB; ++u) {
                        const int t = t0 + u * 256;
                        const int o = t % COLS, k = t / COLS * 8;
                        const int left = o < cols && t < units ? d_in - kc0 - k : 0;
#pragma unroll
                        for (int j = 0; j < 8; ++j) {
                            const uint32_t v = W[j < left ? static_cast<int64_t>(kc0 + k + j) * d_out + col0 + o : 0];
                            h[u][j] = j < left ? v : 0u;
                        }
                    }
#pragma unroll
                    for (int u = 0; u < SB; ++u) {
                        const int t = t0 + u * 256;
                        if (t < units)
                            *reinterpret_cast<uint4 *>(&Ws[t % COLS * KP + t / COLS * 8]) =
                                make_uint4(h[u][0] | (h[u][1] << 16), h[u][2] | (h[u][3] << 16), h[u][4] | (h[u][5] << 16), h[u][6] | (h[u][7] << 16));
                    }
                }
                __syncthreads();
            }
#pragma unroll
            for (int half = 0; half < 2; ++half) {
                if (half > 0 && kc0 + 128 >= d_in) break;  // uniform
#pragma unroll
                for (int s = half * 4; s < half * 4 + 4; ++s) {
                    if (kc0 + s * 32 >= d_in) break;  // uniform
                    const int k = kc0 + s * 32 + kb * 8;
                    Eight<T> a[RT];
#pragma unroll
                    for (int rt = 0; rt < RT; ++rt) load_eight<T>(X, at[rt] + k, d_in - k, a[rt]);
#pragma unroll
                    for (int nt = 0; nt < NT; ++nt) {
                        if (nt * 16 >= cols) break;  // uniform
                        const uint4 b = *reinterpret_cast<const uint4 *>(&Ws[(nt * 16 + m) * KP + s * 32 + kb * 8]);
#pragma unroll
                        for (int rt = 0; rt < RT; ++rt) {
                            split_f32x4 &v = c[SETS == 2 ? s >> 1 & 1 : 0][rt][nt];
                            if constexpr (std::is_same<T, F16>::value)
                                v = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(gt_half8, b), __builtin_bit_cast(gt_half8, a[rt].h), v, 0, 0, 0);
                            else
                                v = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(split_bf16x8, b), __builtin_bit_cast(split_bf16x8, a[rt].h), v, 0, 0, 0);
                        }
                    }
                }
#pragma unroll
                for (int rt = 0; rt < RT; ++rt)
#pragma unroll
                    for (int nt = 0; nt < NT; ++nt) {
                        total[rt][nt] += SETS == 2 ? c[0][rt][nt] + c[SETS - 1][rt][nt] : c[0][rt][nt];
                        c[0][rt][nt] = c[SETS - 1][rt][nt] = split_f32x4{0.f, 0.f, 0.f, 0.f};
                    }
            }
        }
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) {
            const int64_t row = row0 + rt * 16 + m;
            if (row >= n) continue;
            const float f = epi.factor(row);
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
                const int o = nt * 16 + kb * 4;
                float z[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) z[i] = epi.apply(f, total[rt][nt][i]);
                if (o + 4 <= cols) {
                    store_vec_any<4>(Z, row * ldz + col0 + o, zdt, z);
                } else {
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        if (o + i < cols) store_elem(Z, row * ldz + col0 + o + i, zdt, z[i]);
                }
            }
        }
    }
}

// 16-bit rows into more than 64 columns: from here on in groups of 128, which read X half as often (fp16 301 -> 128, groups of 64 /
// 128: 40 000 rows 24 / 25 us, 400 000 223 / 180; 17 -> 128 40 000 rows 11 / 14).
constexpr int GEMM_TILE_WIDE_ROWS = 65536;

// Where gemm_rows_kernel is ahead: its time over that of gemm_tile_kernel, fp16, aligned rows; odd ones, 66 000 to 10^6 of them, by indices: into 65 to 256 columns 128
// .54 to 1.55; .77 to 1.85, 192 .43 to .94; .66 to 1.14, 256 .39 to .78; .65 to 1.03, 512 .35 to .57; .60 to .94, 1433 .48 to .80; .48 to .80; into 33 to 64 from 100 000
// rows on 192 .77 to 1.09; .81 to .97, 256 .67 to .91; .79 to .92, 768 .67 to .81; .82 to .86, of 66 000 rows 256 to 768 .76 to 1.04; .96 to 1.09.
static bool rows_better(int n, bool aligned, int d_in, int d_out)
{
    return d_out > 64 ? n >= GEMM_TILE_WIDE_ROWS && d_in >= (aligned ? 192 : 256) : d_out > 32 && n >= 98304 && d_in >= 256;
}

template <class T, bool TRANS, class TW = T>
static void gemm_tile_t(int n, const void *X, int ldx, int d_in, const void *W, int w_ld, int d_out, void *Z, int ldz, int zdt, Epi epi,
                        hipStream_t s)
{
    if (d_out > GEMM_MOST_COLUMNS) {
        for (int64_t c = 0; c < d_out; c += GEMM_MOST_COLUMNS)
            gemm_tile_t<T, TRANS, TW>(n, X, ldx, d_in, static_cast<const char *>(W) + c * (TRANS ? w_ld : 1) * TW::BYTES, w_ld,
                                      static_cast<int>(d_out - c < GEMM_MOST_COLUMNS ? d_out - c : GEMM_MOST_COLUMNS),
                                      static_cast<char *>(Z) + c * elem_size(zdt), ldz, zdt, epi, s);
        return;
    }
    if constexpr (T::BYTES == 2 && !TRANS) {
        if (rows_better(n, aligned16(X) && ldx % 8 == 0, d_in, d_out)) {
            const int rt = d_out > 64 ? 4 : 2, groups = (d_out + 63) / 64;
            const int n_batches = static_cast<int>((static_cast<int64_t>(n) + 64 * rt - 1) / (64 * rt));
            int per = d_in <= 256 && n_batches > 1024 / groups + 32 ? 1024 / groups + 32 : n_batches;  // staged once where one chunk holds W
            per = (per + 7) / 8 * 8;
            const dim3 grid(static_cast<unsigned>(per) * static_cast<unsigned>(groups));
            const uint16_t *w = static_cast<const uint16_t *>(W);
            if (rt == 4) hipLaunchKernelGGL((gemm_rows_kernel<T, 4, 1>), grid, dim3(256), 0, s, n, X, ldx, d_in, w, d_out, Z, ldz, zdt, epi, n_batches, groups);
            else hipLaunchKernelGGL((gemm_rows_kernel<T, 2, 2>), grid, dim3(256), 0, s, n, X, ldx, d_in, w, d_out, Z, ldz, zdt, epi, n_batches, groups);
            return;
        }
    }
    const int nt = d_out <= 16 ? 1 : d_out <= 32 ? 2 : d_out <= 64 || T::BYTES == 4 || n < GEMM_TILE_WIDE_ROWS ? 4 : 8;
    const int n_blocks = static_cast<int>((static_cast<int64_t>(n) + 63) / 64);
    const int groups = (d_out + nt * 16 - 1) / (nt * 16);
    // dX of several groups and fewer rows: as many workgroups as the chip holds at once (but 40 a group), which stage W once, and the groups of
    // the same rows together, whose lines of dX are shared (us, 2048 workgroups a group / this; input_grad_kernel before: 100 000 x 128 from 1
    // column 19.8 / 14.4; 17.1, from 10 23.4 / 16.5; 21.9, 200 000 x 128 from 7 30.6 / 23.3; 27.2, 100 000 x 301 from 7 42.6 / 35.6; 36.0, 40 000 x
    // 1433 from 7 122.8 / 83.1; 101.2; 262 144 x 128 from 7 40.9 / 36.3; 37.4; but 400 000 x 128
    // from 64 75.8 / 86.5, from 40 71.3 / 79.9).
    // Products of few indices always do (us, apart / together: 602 932 x 120 from 8 193 / 182, 1 000 000 x 128 from 3 301 / 289, 400 000 x 70 from 5 71.5 / 67.6), and
    // rows that are no whole lines of memory, whose lines two groups share (549 450 x 91 from 10 98 / 82, from 64 142 / 119, 1 153 846 x 91 from 25 293 / 207, 966 183 x
    // 207 from 25 539 / 352, from 100 856 / 669, 454 545 x 330 from 64 383 / 344).
    constexpr int FEW = TRANS ? FEW_BACK : SPLIT_FROM;
    const bool lines = (reinterpret_cast<uintptr_t>(Z) | static_cast<uintptr_t>(ldz) * elem_size(zdt)) % 128 == 0;
    const bool neighbours = TRANS && groups > 1 && (n < 327680 || d_in <= FEW || !lines);
    const int most = !neighbours ? 2048 : groups <= 25 ? 1024 / groups : 40;
    int grid = d_in <= GemmChunk<T>::KC && n_blocks > most ? most : n_blocks;
    if (neighbours) grid = (grid + 7) / 8 * 8;
#define FTC_GT1(N, Q)                                                                                                                      \
    hipLaunchKernelGGL((gemm_tile_kernel<T, N, TRANS, Q, TW>), dim3(grid, groups), dim3(256), 0, s, n, X, ldx, d_in, W, w_ld, d_out, Z, ldz, \
                       zdt, epi, n_blocks, neighbours ? 1 : 0)
#define FTC_GT(N) if (nt == N) FTC_GT1(N, true)
    if constexpr (T::BYTES == 4) {
        if (d_in <= FEW) {
#define FTC_GF1(N, K)                                                                                                                          \
    hipLaunchKernelGGL((gemm_few_kernel<N, K, TRANS, TW>), dim3(grid, groups), dim3(256), 0, s, n, static_cast<const float *>(X), ldx, d_in, W, \
                       w_ld, d_out, Z, ldz, zdt, epi, n_blocks, neighbours ? 1 : 0)
#define FTC_GF(N)                                     \
    if (nt == N) {                                    \
        if (d_in <= 4) FTC_GF1(N, 1);                 \
        else if constexpr (TRANS) FTC_GF1(N, 2);      \
    }
            FTC_GF(1)
            FTC_GF(2)
            FTC_GF(4)
#undef FTC_GF
#undef FTC_GF1
            return;
        }
    }
    if constexpr (T::BYTES == 4 && !TRANS) {
        // A compute unit holds seven workgroups of these.  Where some have seven and the others six, all wait for those with seven, which are ahead with a
        // column a lane (us, a column a lane / four, into 16: 99 000 rows of 300 26.9 / 27.7, of 700 57.6 / 60.2, of 1433 137 / 141, 110 000 of 700 64.3 / 67.5, of 1433
        // 143 / 147); with fewer rows or more they are behind (98 000 of 300 25.7 / 24.7, of 1433 125 / 123, 115 000 of 300 32.2 / 30.3, of 1433 161 / 157, 170 000 225 / 222).
        if (nt == 1 && d_in > GemmChunk<T>::KC && n_blocks > 6 * 256 && n_blocks <= 7 * 256) {
            FTC_GT1(1, false);
            return;
        }
    }
    FTC_GT(1);
    FTC_GT(2);
    FTC_GT(4);
    if constexpr (T::BYTES == 2) FTC_GT(8);
#undef FTC_GT
#undef FTC_GT1
}

int32_t launch_gemm_tile(int n, const void *X, int ldx, int dt, int d_in, const void *W, int d_out, void *Z, int ldz, int zdt, Epi epi,
                         hipStream_t s)
{
    if (dt == FTC_F32) gemm_tile_t<F32, false>(n, X, ldx, d_in, W, d_out, d_out, Z, ldz, zdt, epi, s);
    else if (dt == FTC_F16) gemm_tile_t<F16, false>(n, X, ldx, d_in, W, d_out, d_out, Z, ldz, zdt, epi, s);
    else gemm_tile_t<BF16, false>(n, X, ldx, d_in, W, d_out, d_out, Z, ldz, zdt, epi, s);
    return launch_status("update_gemm tile");
}

// dX = G W^T for G in fp32: W (d_in x d_out) is read transposed, the contraction runs over d_out.  Few results of a contraction of more than
// one chunk go through gemm_slice.hip, where the waves of a workgroup share it (us, here / there: 500 x 64 from 300 columns 13.5 / 3.6, 2708 x 64 from
// 504 23.2 / 16.5, 6000 x 33 from 300 14.5 / 8.5, 16 000 x 16 from 300 10.5 / 7.7; but 2708 x 301 from 128 8.2 / 11.6, 16 000 x 33 from 300
// 16.4 / 17.8; W transposed into a buffer and gemm_any_kernel: 12.9, 18.3, 16.3, 11.2, 15.4, 23.1).
//
// Large dX from up to 16 columns, by input_grad_kernel (backward.hip), which has whole rows of 256 columns in flight.  us, that / here, by columns of dX, from 1, 8, 12
// columns: 220 MB 91 88 / 91, 93 / 99, 94 / 87; 260 MB 70 103 / 95, 108 / 116, 121 / 116, 91 102 / 111, 104 / 118, 114 / 116, 128 92 / 92, 98 / 103, 101 / 92, 207 82 / 91, 88 / 97, 90 / 90;
// 420 MB 91 147 / 167, 165 / 199, 184 / 196, 128 135 / 146, 149 / 165, 164 / 176, 256 125 / 143, 142 / 162, 155 / 150, 366 MB 157 from 16 251 / 276 with dW; 420 MB 506 160 / 170, 170 / 170, 181 / 166; 600 MB 91 205 / 240, 233 / 289,
// 259 / 285, 207 189 / 227, 213 / 249, 221 / 245, 506 214 / 225, 227 / 239, 241 / 239; 420 MB 48 from 4 170 / 158; from 20 600 MB 91 400 / 293, 207 313 / 263.
static bool whole_rows_better(int n, int d_out, int d_in, int dx_dt)
{
    const int64_t all = static_cast<int64_t>(n) * d_in * elem_size(dx_dt);
    return d_in > 64 && (d_out <= 8 ? all >= 250000000 : d_out <= 16 && d_in <= 256 && all >= 350000000);
}

int32_t launch_input_grad(int n, const float *G, int ldg, int d_out, const void *W, int wdt, int d_in, void *dX, int lddx, int dx_dt,
                          hipStream_t s)
{
    if (n == 0) return FTC_OK;
    if (d_out > GemmChunk<F32>::KC && static_cast<int64_t>(n) * d_in <= 1 << 18)
        return launch_input_grad_slice(n, G, ldg, d_out, W, wdt, d_in, dX, lddx, dx_dt, s);
    if (whole_rows_better(n, d_out, d_in, dx_dt)) return launch_input_grad_rows(n, G, ldg, d_out, W, wdt, d_in, dX, lddx, dx_dt, s);
    const Epi none{0, nullptr};
    if (wdt == FTC_F32) gemm_tile_t<F32, true, F32>(n, G, ldg, d_out, W, d_out, d_in, dX, lddx, dx_dt, none, s);
    else if (wdt == FTC_F16) gemm_tile_t<F32, true, F16>(n, G, ldg, d_out, W, d_out, d_in, dX, lddx, dx_dt, none, s);
    else gemm_tile_t<F32, true, BF16>(n, G, ldg, d_out, W, d_out, d_in, dX, lddx, dx_dt, none, s);
    return launch_status("input_grad");
}

}  // namespace ftc
