// AGNN propagation layer in one pass over the edges: edge scores (SDDMM), edge softmax and the
// weighted aggregation (SpMM) fused, so every neighbour row H[j,:] is gathered once per edge
// instead of twice and neither scores nor probabilities travel through HBM.
//
//   out[i,:] = sum_j w_ij H[j,:] / sum_j w_ij,   w_ij = exp(beta * cos(h_i, h_j) - |beta|)
//
// |cos| <= 1, so |beta| is an upper bound of every score of every row: shifting by it instead of
// by the row maximum gives the same softmax (numerator and denominator carry the same factor)
// and makes the pass single-sweep: numerator vector and denominator are plain segmented sums.
// Safe while exp(-2|beta|) is a normal fp32 number (|beta| < 43).
//
// The row norms of the cosine are recomputed from the row slices that are in registers anyway
// (a second DPP reduction in the lane group), so the pass needs no array of inverse norms and no
// random 4-byte gather per edge.
//
// When the caller wants the probabilities the pass also writes the weight of every entry, parked in LDS over the row
// offsets that have been used, and a second kernel divides by the rows' sums: one gather of H per entry instead of the two of
// scores, softmax and aggregation one after the other.
//
// What bounds it: on large graphs the gathers, on graphs whose features lie in the L2s the instructions around them.  Since these
// went (edge_ranges.hpp, and the scalar work of four entries done once instead of by every lane of the group) the layer takes, with
// fix-up, 0.33 ms instead of 0.37 on the R-MAT graph (2^20 nodes, 32 M entries, fp16, 32 columns) and with P 72 us instead of 90 on a
// power-law graph (200 000 nodes, 3.8 M entries).
//
// Work partition, run structure and the handling of rows cut by run / wave boundaries are
// those of the edge-balanced SpMM (spmm_seg.hip): 512 edges per wave (fewer on small graphs) staged in LDS, groups of
// LPR lanes walk contiguous runs, complete rows are stored from registers, the pieces of cut rows are summed
// in edge order by the group that closes the row, and through a carry buffer.  The partial of a cut row is the pair
// (numerator vector, denominator); the division happens once all pieces are added.
#include "edge_ranges.hpp"

namespace ftc {

constexpr int AG_B = 4;    // edges per batch

bool seg_shape(int dtype, int D, int *vec, int *lpr);

static size_t ag_carry_ws(int nnz, int r, int dp)
{
    const size_t n_ranges = static_cast<size_t>(seg_count(nnz, r));
    return align_up(n_ranges * 2 * (dp + 4) * sizeof(float), 256) + align_up(n_ranges * 2 * sizeof(int), 256);
}

size_t agnn_fused_ws(int nnz, int D, bool least)
{
    int vec, lpr, dp = 0;
    if (seg_shape(FTC_F32, D, &vec, &lpr)) dp = vec * lpr;
    if (seg_shape(FTC_F16, D, &vec, &lpr) && vec * lpr > dp) dp = vec * lpr;
    if (dp == 0 || nnz == 0) return 0;
    return ag_carry_ws(nnz, least ? SEG_R : seg_range(nnz, SEG_AGNN), dp);
}

// MODE 0: inference.  1: also write what the backward pass needs (row_z, out32).  2: also write the weight w_ij of every entry
// (edge_w) and row_z; agnn_edge_p_kernel turns the weights into probabilities once every row's sum is known.
//
// Four entries of a group are taken together: the two dot products of each are formed by all lanes, their lane sums and
// what becomes of them (norm, cosine, exponential) by one lane of the quad per entry, and the weights go back to all lanes.
template <class T, int VEC, int LPR, int MODE, int AG_R, bool BIG>
__global__ __launch_bounds__(256) void agnn_fused_kernel(int nnz, int n_ranges, const int *__restrict__ row_ptr,
                                                         const int *__restrict__ col_idx,
                                                         const int *__restrict__ edge_to_row,
                                                         const void *__restrict__ H, uint64_t ldb, int D, float beta,
                                                         void *__restrict__ out, int ldo, int odt,
                                                         float *__restrict__ carry, int *__restrict__ carry_tail_row,
                                                         float *__restrict__ row_z, float *__restrict__ out32,
                                                         int ld32, float *__restrict__ edge_w)
{
    using E = EdgeRange<LPR, AG_R>;
    constexpr bool KEEP = MODE != 0;
    constexpr int NG = E::NG, RUN = E::RUN;
    constexpr int DP = LPR * VEC;
    constexpr int DPZ = DP + 4;  // feature slots, then the denominator
    constexpr int IDX_WORDS = 2 * E::WORDS;
    constexpr int PART_WORDS = NG * DPZ;
    __shared__ __align__(16) int smem[4][IDX_WORDS > PART_WORDS ? IDX_WORDS : PART_WORDS];

    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int g = lane / LPR, sub = lane % LPR, quad = lane & 3;
    const bool odd = lane & 1, upper = lane & 2;
    uint32_t *s_off = reinterpret_cast<uint32_t *>(smem[wave]);
    int *s_row = smem[wave] + E::WORDS;

    const int v = xcd_chunked_block(blockIdx.x, gridDim.x) * 4 + wave;
    if (v >= n_ranges) return;  // (no wave waits for another)
    const int base = v * AG_R;
    const int n_valid = min(AG_R, nnz - base);
    const int prev_row = base > 0 ? edge_to_row[base - 1] : -1;
    const int next_row = nnz - base > AG_R ? edge_to_row[base + AG_R] : -1;
    // row of the first edge after the NEXT range: tells whether a row left open here ends there
    const int far_row = static_cast<int64_t>(base) + 2 * AG_R < nnz ? edge_to_row[base + 2 * AG_R] : -1;
    stage_range<LPR, AG_R, false, BIG>(row_ptr, col_idx, edge_to_row, nullptr, base, n_valid, ldb, nullptr, lane, s_off, s_row,
                                       nullptr);

    const int at = g * E::RUNP;  // the group's run
    const bool live = sub * VEC < D;
    const uint32_t lane_bytes = live ? sub * VEC * T::BYTES : 0;  // lanes beyond the row gather its first piece
    // The exponential is taken in powers of two and the large part of its argument rounded once instead of twice:
    // log2(e) = 1.44269502162933 (its nearest fp32) + 1.92596299e-8.
    const float beta2 = beta * 1.44269504f;
    const float beta2_rest = fmaf(beta, 1.92596299e-8f, fmaf(beta, 1.44269504f, -beta2));
    float acc[VEC], hacc[VEC];
#pragma unroll
    for (int j = 0; j < VEC; ++j) { acc[j] = 0.f; hacc[j] = 0.f; }
    RawVec<T, VEC> xi;  // slice of H[i,:] of the current row, as loaded; zero in lanes beyond the row
    zero_raw(xi);
    float z = 0.f, hz = 0.f, ri = 0.f;
    // MODE 2 sums every other entry apart and joins the halves in the quotient (its two fma round about as often as one sum):
    // that is what makes the output as exact as the three kernels', whose weights were divided by z before they were summed.
    constexpr int ODD = MODE == 2 ? VEC : 1;
    float odds[ODD], odd_z = 0.f;
#pragma unroll
    for (int j = 0; j < ODD; ++j) odds[j] = 0.f;
    auto join_odd = [&]() {  // for a piece of a row
        if constexpr (MODE == 2) {
#pragma unroll
            for (int j = 0; j < VEC; ++j) acc[j] += odds[j];
            z += odd_z;
        }
    };
    bool head_closed = false, first = true;
    int head_row = -1, cur = -1;
    const int first_row = s_row[at];
    const bool left_open = first_row >= 0 && first_row == (g == 0 ? prev_row : s_row[max(at - 5, 0)]);  // the last entry of the run before

    auto put = [&](int row, const float (&o)[VEC]) {
        store_vec_nt<VEC>(out, static_cast<int64_t>(row) * ldo + sub * VEC, odt, o);
        if constexpr (KEEP)
            if (out32) store_vec<VEC>(out32, static_cast<int64_t>(row) * ld32 + sub * VEC, FTC_F32, o);  // unrounded copy
    };
    auto store_row = [&](int row) {
        if constexpr (MODE == 2) z += odd_z;
        if (live) {
            const float inv = __builtin_amdgcn_rcpf(z);  // v_rcp_f32: one ulp, one instruction
            const float rest = fmaf(-z, inv, 1.f) * inv;  // what the reciprocal is short of
            float o[VEC];
#pragma unroll
            for (int j = 0; j < VEC; ++j) {
                if constexpr (MODE == 2) o[j] = fmaf(acc[j], inv, fmaf(odds[j], inv, (acc[j] + odds[j]) * rest));
                else o[j] = acc[j] * inv;
            }
            put(row, o);
        }
        if constexpr (KEEP)
            if (row_z && sub == 0) row_z[row] = z;  // softmax denominator (shifted by |beta|), kept for the backward pass
    };

#pragma unroll 1
    for (int b = 0; b < RUN; b += AG_B) {
        const uint4 o4 = *reinterpret_cast<const uint4 *>(s_off + at + b);
        const int4 r4 = *reinterpret_cast<const int4 *>(s_row + at + b);
        const uint32_t o[AG_B] = {o4.x, o4.y, o4.z, o4.w};
        const int r[AG_B] = {r4.x, r4.y, r4.z, r4.w};
        RawVec<T, VEC> y[AG_B], xs[AG_B];
#pragma unroll
        for (int k = 0; k < AG_B; ++k) load_raw<T, VEC>(row_addr<BIG>(H, o[k], ldb, lane_bytes), 0, y[k]);
        bool need[AG_B];  // a new row starts (the lanes of a group branch together)
#pragma unroll
        for (int k = 0; k < AG_B; ++k) {
            need[k] = r[k] != (k ? r[k - 1] : cur);
            if (need[k]) load_raw<T, VEC>(row_addr<BIG>(H, row_slot<BIG>(max(r[k], 0), ldb), ldb, lane_bytes), 0, xs[k]);
        }
        float ri_mine = ri, dots[AG_B], squares[AG_B];  // ri_mine: of the row of this lane's entry
#pragma unroll
        for (int k = 0; k < AG_B; ++k) {
            if (need[k]) {
#pragma unroll
                for (int w = 0; w < RawVec<T, VEC>::WORDS; ++w) xi.w[w] = live ? xs[k].w[w] : 0u;
                ri = __frsqrt_rn(fmaxf(group_sum_dpp<LPR>(dot_raw<T, VEC>(xi, xi, 0.f)), 1e-24f));  // = 1 / max(||h_i||, 1e-12)
                ri_mine = quad >= k ? ri : ri_mine;
            }
            dots[k] = dot_raw<T, VEC>(xi, y[k], 0.f);
            const float q = dot_raw<T, VEC>(y[k], y[k], 0.f);
            squares[k] = live ? q : 0.f;
        }
        const float rj = __frsqrt_rn(fmaxf(group_sum4<LPR>(squares, odd, upper), 1e-24f));
        const float cosine = ri_mine * rj * group_sum4<LPR>(dots, odd, upper);
        const float wgt = __builtin_amdgcn_exp2f(fmaf(beta2_rest, cosine, fmaf(beta2, cosine, -fabsf(beta2))));
        if constexpr (MODE == 2)
            if (sub < 4) s_off[at + b + sub] = __float_as_uint(wgt);  // these entries' offsets have been used
        const float w4[AG_B] = {quad_lane<0>(wgt), quad_lane<1>(wgt), quad_lane<2>(wgt), quad_lane<3>(wgt)};
#pragma unroll
        for (int k = 0; k < AG_B; ++k) {
            if (need[k]) {  // close the segment of the previous row
                if (cur >= 0) {
                    if (first && left_open) {
                        join_odd();
#pragma unroll
                        for (int j = 0; j < VEC; ++j) hacc[j] = acc[j];
                        hz = z;
                        head_closed = true; head_row = cur;
                    } else {
                        store_row(cur);
                    }
                    first = false;
                }
                cur = r[k];
#pragma unroll
                for (int j = 0; j < VEC; ++j) acc[j] = 0.f;
                z = 0.f;
                if constexpr (MODE == 2) {
#pragma unroll
                    for (int j = 0; j < VEC; ++j) odds[j] = 0.f;
                    odd_z = 0.f;
                }
            }
            float yf[VEC];
            unpack<T, VEC>(y[k], yf);
#pragma unroll
            for (int j = 0; j < VEC; ++j) {
                if constexpr (MODE == 2) {
                    float &a = (k & 1) ? odds[j] : acc[j];
                    a = fmaf(w4[k], yf[j], a);
                } else {
                    acc[j] = fmaf(w4[k], yf[j], acc[j]);
                }
            }
            if (MODE == 2 && (k & 1)) odd_z += w4[k];
            else z += w4[k];
        }
    }
    // the run's last segment
    int open = OPEN_NONE;
    if (cur >= 0) {
        const int right_row = g == NG - 1 ? next_row : s_row[at + E::RUNP];
        if (right_row == cur) {
            join_odd();
            open = first && left_open ? OPEN_THROUGH : OPEN_TAIL;
        } else if (first && left_open) {
            join_odd();
#pragma unroll
            for (int j = 0; j < VEC; ++j) hacc[j] = acc[j];
            hz = z;
            head_closed = true; head_row = cur;
        } else {
            store_row(cur);
        }
    }
    const int from = first_group<LPR>(open, g);
    const bool last_open = g == NG - 1 && open != OPEN_NONE;  // a row that goes on in the next range
    wave_lds_sync();
    if constexpr (MODE == 2) {
        int own = lane;
        asm("" : "+v"(own));  // (else the addresses of the staging loop are kept in registers all the way to here)
#pragma unroll
        for (int j = 0; j < AG_R / 64; ++j) {
            const int i = j * 64 + own;
            if (i < n_valid) edge_w[base + i] = __uint_as_float(s_off[E::slot(i)]);
        }
        wave_lds_sync();
    }
    // Rows cut inside this wave: the group that closes a row adds its pieces, in edge order.  The staged entries are dead, their
    // place is taken by the open pieces.
    float *part = reinterpret_cast<float *>(smem[wave]);
    if (open != OPEN_NONE) {
#pragma unroll
        for (int j = 0; j < VEC; ++j) part[g * DPZ + sub * VEC + j] = acc[j];
        if (sub == 0) part[g * DPZ + DP] = z;
    }
    wave_lds_sync();
    // carried piece: [2 v] of the row that came in from the left, [2 v + 1] of the one left open
    auto store_carry = [&](int slot, const float (&a)[VEC], float az) {
        float *to = carry + (static_cast<size_t>(v) * 2 + slot) * DPZ;
        store_vec<VEC>(to, sub * VEC, FTC_F32, a);
        if (sub == 0) to[DP] = az;
    };
    if (head_closed || (last_open && open == OPEN_THROUGH)) {
        float run[VEC], run_z = 0.f;
#pragma unroll
        for (int j = 0; j < VEC; ++j) run[j] = 0.f;
        for (int q = max(from, 0); q < g; ++q) {
#pragma unroll
            for (int j = 0; j < VEC; ++j) run[j] += part[q * DPZ + sub * VEC + j];
            run_z += part[q * DPZ + DP];
        }
#pragma unroll
        for (int j = 0; j < VEC; ++j) run[j] += head_closed ? hacc[j] : acc[j];
        run_z += head_closed ? hz : z;
        if (from < 0) {
            store_carry(0, run, run_z);
        } else if (head_closed) {
            if (live) {
                float o[VEC];
#pragma unroll
                for (int j = 0; j < VEC; ++j) o[j] = run[j] / run_z;
                put(head_row, o);
            }
            if constexpr (KEEP)
                if (row_z && sub == 0) row_z[head_row] = run_z;
        } else {
            store_carry(1, run, run_z);
        }
    }
    if (last_open && open == OPEN_TAIL) store_carry(1, acc, z);
    if (lane == 63) {
        const int tail = last_open && !(open == OPEN_THROUGH && from < 0) ? cur : -1;
        carry_tail_row[2 * v] = tail;
        carry_tail_row[2 * v + 1] = (tail >= 0 && far_row != tail) ? 1 : 0;  // ends in range v + 1
    }
}

// G lanes (four features each) finish one cut row, 64 / G rows per wave: the kernel is a chain of two dependent
// loads per row (the range's record, then the two pieces), so it is the number of rows in flight that counts.
template <int G>
__global__ __launch_bounds__(256) void agnn_fused_fixup_kernel(int n, int n_ranges, const int *__restrict__ row_ptr,
                                                               const float *__restrict__ carry,
                                                               const int *__restrict__ carry_tail_row, int DP,
                                                               int D, void *__restrict__ out, int ldo, int odt,
                                                               float *__restrict__ row_z, float *__restrict__ out32,
                                                               int ld32, int seg_r)
{
    constexpr int R = 64 / G;  // ranges per wave
    const int DPZ = DP + 4;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int sub = lane % G;
    const int v_mine = (blockIdx.x * 4 + wave) * R + lane / G;
    int2 rec = make_int2(-1, 0);
    if (v_mine < n_ranges) rec = reinterpret_cast<const int2 *>(carry_tail_row)[v_mine];
    // Nearly every open row ends in the next range: numerator and denominator are the head piece of range
    // v + 1 plus the tail piece of range v.  Their addresses depend on v alone, so they are loaded together
    // with the range's record instead of after it.
    {
        const bool ok = v_mine + 1 < n_ranges && sub * 4 < DP;
        const size_t vv = ok ? static_cast<size_t>(v_mine) : 0;
        const float *hv = carry + (vv + 1) * 2 * DPZ;
        const float *tv = carry + (vv * 2 + 1) * DPZ;
        float4 h4 = make_float4(0.f, 0.f, 0.f, 0.f), t4 = h4;
        float spec_z = 1.f;
        if (ok) {
            h4 = *reinterpret_cast<const float4 *>(hv + sub * 4);
            t4 = *reinterpret_cast<const float4 *>(tv + sub * 4);
            spec_z = hv[DP] + tv[DP];
        }
        const int r = rec.x;
        if (ok && r >= 0 && rec.y && sub * 4 < D) {
            const float o[4] = {(h4.x + t4.x) / spec_z, (h4.y + t4.y) / spec_z, (h4.z + t4.z) / spec_z,
                                (h4.w + t4.w) / spec_z};
            if (sub * 4 + 4 <= D) {
                store_vec<4>(out, static_cast<int64_t>(r) * ldo + sub * 4, odt, o);
                if (out32) store_vec<4>(out32, static_cast<int64_t>(r) * ld32 + sub * 4, FTC_F32, o);
            } else {  // widths of 3 and 6: the row's last piece is a short one
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if (sub * 4 + i < D) {
                        store_elem(out, static_cast<int64_t>(r) * ldo + sub * 4 + i, odt, o[i]);
                        if (out32) out32[static_cast<int64_t>(r) * ld32 + sub * 4 + i] = o[i];
                    }
            }
        }
        if (ok && r >= 0 && rec.y && row_z && sub == 0) row_z[r] = spec_z;
    }
    // rows that go on beyond the next range (long rows of a power-law graph): one at a time, by the whole wave
    unsigned long long longs = __builtin_amdgcn_ballot_w64(rec.x >= 0 && !rec.y && sub == 0);
    while (longs) {
        const int src = __ffsll(static_cast<long long>(longs)) - 1;
        longs &= longs - 1;
        const int v = __shfl(v_mine, src, 64), r = __shfl(rec.x, src, 64);
        {
            const int last = (row_ptr[r + 1] - 1) / seg_r;
            // teams of `dl` lanes (one lane per feature) share the ranges of a long row round-robin;
            // team sums are added in team order (fixed by the shape)
            int dl = 1;
            while (dl < D && dl < 64) dl <<= 1;
            const int parts = 64 / dl;
            const int part = lane / dl;
            // denominator: every lane adds all pieces
            float zsum;
            {
                zsum = sum_pieces(carry + DP, 2 * static_cast<size_t>(DPZ), v + 1 + part, last, parts);
                for (int off = 32; off >= dl; off >>= 1) zsum += __shfl_down(zsum, off, 64);
                zsum = __shfl(zsum, 0, 64) + carry[(static_cast<size_t>(v) * 2 + 1) * DPZ + DP];
                if (row_z && lane == 0) row_z[r] = zsum;
            }
            for (int d0 = 0; d0 < D; d0 += 64) {
                const int d = d0 + lane % dl;
                const bool dok = d < D;
                const float *base = carry + (dok ? d : 0);
                float sum = sum_pieces(base, 2 * static_cast<size_t>(DPZ), v + 1 + part, last, parts);
                for (int off = 32; off >= dl; off >>= 1) sum += __shfl_down(sum, off, 64);
                if (lane < dl && dok) {
                    sum += carry[(static_cast<size_t>(v) * 2 + 1) * DPZ + d];
                    store_elem(out, static_cast<int64_t>(r) * ldo + d, odt, sum / zsum);
                    if (out32) out32[static_cast<int64_t>(r) * ld32 + d] = sum / zsum;
                }
            }
        }
    }
    const int64_t row = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
    if (row < n && row_ptr[row] == row_ptr[row + 1]) {
        for (int d = 0; d < D; ++d) store_elem(out, row * ldo + d, odt, 0.f);
        if (out32)
            for (int d = 0; d < D; ++d) out32[row * ld32 + d] = 0.f;
        if (row_z) row_z[row] = 0.f;
    }
}

// p[e] = w[e] / z[row of e], in place, four entries per thread and 64 apart in the wave
__global__ __launch_bounds__(256) void agnn_edge_p_kernel(int nnz, const int *__restrict__ edge_to_row,
                                                          const float *__restrict__ row_z, float *__restrict__ edge_w)
{
    const int64_t e0 = static_cast<int64_t>(blockIdx.x) * 1024 + (threadIdx.x >> 6) * 256 + (threadIdx.x & 63);
    float a[4], z[4];
    int r[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const int64_t e = min(e0 + 64 * k, static_cast<int64_t>(nnz) - 1);
        r[k] = __builtin_nontemporal_load(edge_to_row + e);
        a[k] = edge_w[e];
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) z[k] = row_z[r[k]];
#pragma unroll
    for (int k = 0; k < 4; ++k)
        if (e0 + 64 * k < nnz) __builtin_nontemporal_store(a[k] / z[k], edge_w + e0 + 64 * k);
}

template <class T, int R, bool BIG>
static void launch_agnn_t(int vec, int lpr, unsigned grid, hipStream_t s, int nnz, int n_ranges, const ftc_csr &g,
                          const int *e2r, const void *H, uint64_t ldb, int D, float beta, void *out,
                          int ldo, int odt, float *carry, int *tail_row, float *row_z, float *out32, int ld32,
                          float *edge_w)
{
    constexpr int VM = T::VEC;
#define FTC_AG1(V, L, M)                                                                                              \
    hipLaunchKernelGGL((agnn_fused_kernel<T, V, L, M, R, BIG>), dim3(grid), dim3(256), 0, s, nnz, n_ranges, g.row_ptr, \
                       g.col_idx, e2r, H, ldb, D, beta, out, ldo, odt, carry, tail_row, row_z, out32, ld32, edge_w)
#define FTC_AG(V, L)                         \
    if (edge_w) FTC_AG1(V, L, 2);            \
    else if (row_z || out32) FTC_AG1(V, L, 1); \
    else FTC_AG1(V, L, 0)
    if (vec == VM) {
        if (lpr == 4) { FTC_AG(VM, 4); }
        else if (lpr == 8) { FTC_AG(VM, 8); }
        else if (lpr == 16) { FTC_AG(VM, 16); }
        else { FTC_AG(VM, 32); }
    } else if (vec == VM / 2) {
        FTC_AG(VM / 2, 4);
    } else {
        FTC_AG(VM / 4, 4);
    }
#undef FTC_AG
#undef FTC_AG1
}

// Caller has checked: window index present, seg_shape() accepts (dt, D), rows of H and out 16-byte
// aligned, workspace of agnn_fused_ws(.., least) bytes.
int32_t launch_agnn_fused(const ftc_csr &g, const ftc_windows &w, const void *H, int ld, int dt, int D,
                          float beta, void *out, int ldo, int odt, float *row_z, float *out32, int ld32, float *edge_w, void *ws,
                          size_t ws_bytes, hipStream_t s)
{
    int vec = 0, lpr = 0;
    seg_shape(dt, D, &vec, &lpr);
    const int dp = vec * lpr;
    const int64_t row_bytes = static_cast<int64_t>(ld) * elem_size(dt);
    const bool big = rows_need_64_bits(g.n, row_bytes);  // ranges of SEG_R only: such a matrix has many rows
    const int short_r = big ? SEG_R : seg_range(g.nnz, SEG_AGNN);
    const int r = ws_bytes >= ag_carry_ws(g.nnz, short_r, dp) ? short_r : SEG_R;
    const int n_ranges = static_cast<int>(seg_count(g.nnz, r));
    float *carry = static_cast<float *>(ws);
    int *tail_row = reinterpret_cast<int *>(
        static_cast<char *>(ws) + align_up(static_cast<size_t>(n_ranges) * 2 * (dp + 4) * sizeof(float), 256));
    if (n_ranges > 0) {
        const unsigned grid = static_cast<unsigned>((n_ranges + 3) / 4);
#define FTC_AGR1(T, R, BIG)                                                                                              \
    launch_agnn_t<T, R, BIG>(vec, lpr, grid, s, g.nnz, n_ranges, g, w.edge_to_row, H, static_cast<uint64_t>(row_bytes), D,  \
                             beta, out, ldo, odt, carry, tail_row, row_z, out32, ld32, edge_w)
#define FTC_AGR(T)                             \
    do {                                       \
        if (big) FTC_AGR1(T, SEG_R, true);     \
        else if (r == SEG_R) FTC_AGR1(T, SEG_R, false); \
        else if (r == 256) FTC_AGR1(T, 256, false);     \
        else FTC_AGR1(T, 128, false);          \
    } while (0)
        if (dt == FTC_F32) FTC_AGR(F32);
        else if (dt == FTC_F16) FTC_AGR(F16);
        else FTC_AGR(BF16);
#undef FTC_AGR
#undef FTC_AGR1
        const int32_t st = launch_status("agnn_fused");
        if (st != FTC_OK) return st;
    }
    // lanes per cut row in the fix-up kernel: four features per lane
    int grp = 1;
    while (grp * 4 < dp) grp <<= 1;
    const int64_t blocks_rows = (static_cast<int64_t>(g.n) + 255) / 256;
    const int64_t per_block = 4 * (64 / grp);
    const int64_t blocks_ranges = (n_ranges + per_block - 1) / per_block;
    const unsigned grid2 = static_cast<unsigned>(blocks_rows > blocks_ranges ? blocks_rows : blocks_ranges);
#define FTC_FX(G)                                                                                                    \
    case G:                                                                                                          \
        hipLaunchKernelGGL(agnn_fused_fixup_kernel<G>, dim3(grid2), dim3(256), 0, s, g.n, n_ranges, g.row_ptr, carry, \
                           tail_row, dp, D, out, ldo, odt, row_z, out32, ld32, r);                                   \
        break;
    switch (grp) {
        FTC_FX(1) FTC_FX(2) FTC_FX(4) FTC_FX(8) FTC_FX(16) FTC_FX(32) FTC_FX(64)
    }
#undef FTC_FX
    if (edge_w && g.nnz > 0)
        hipLaunchKernelGGL(agnn_edge_p_kernel, dim3(ceil_div(g.nnz, 1024)), dim3(256), 0, s, g.nnz, w.edge_to_row, row_z,
                           edge_w);
    return launch_status("agnn_fused fixup");
}

}  // namespace ftc
