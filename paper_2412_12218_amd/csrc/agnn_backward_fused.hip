// Backward of the AGNN propagation layer in one pass over the edges (symmetric pattern).
//
// Forward (agnn_fused.hip): y_i = sum_e p_e h_j, p_e = a_e / z_i, a_e = exp(beta c_e - |beta|),
// c_e = <hn_i, hn_j>, z_i = sum_e a_e.  The paper names training (Sections II and V) and gives no
// gradient formulas; these are the derivatives of that definition.  With t_i = sum_e p_e dp_e
// = <dY_i, y_i> and, for the stored entry T(e) = (j, i) that a symmetric pattern holds for every
// e = (i, j), c_T(e) = c_e and a_T(e) = a_e:
//     dp_e = <dY_i, h_j>                 ds_e    = p_e (dp_e - t_i)
//     p_T(e) = a_e / z_j                 ds_T(e) = p_T(e) (<h_i, dY_j> - t_j)
//     dbeta = sum_e ds_e c_e = sum_e ds_e (c_e - m_i)   for any m_i of the row, its ds add up to zero
//     q_i   = beta sum_e (ds_e + ds_T(e)) hn_j        (gradient w.r.t. the normalised row hn_i)
//     agg_i = sum_e p_T(e) dY_j                       (through the aggregated rows)
//     dH_i  = agg_i + (q_i - hn_i <hn_i, q_i>) / |h_i|
// so one sweep that gathers h_j and dY_j once per entry, plus the per-node pair (1 / z_j, t_j),
// yields everything: no edge array (scores, probabilities, transposed index) travels through HBM.
// z comes from the forward pass (row_z of ftc_agnn_layer), t from a row-wise dot product of dY and
// the forward output.  The same row pass copies h_i and dY_i side by side into one matrix HD
// (row i = [h_i | dY_i], each half padded to DP elements): every read that leaves L2 is a 128-byte
// line, so the two 64-byte rows an entry needs cost one line instead of two.
//
// Work partition, runs and the handling of rows cut by run / wave boundaries are those of the
// edge-balanced SpMM (spmm_seg.hip); the partial of a cut row is the pair (q_i, agg_i), 2 * DP slots.  Whoever completes a row
// -- the group that closes it, or the second kernel for rows cut by a range boundary -- applies the derivative of the
// normalisation and writes dH_i: the pairs, 256 bytes a row at D = 32, do not travel through HBM (before: 268 MB written
// and read again by a kernel of its own, next to one for the norms; R-MAT graph, 2^20 nodes, 32 M entries, fp16, D = 32).
#include "edge_ranges.hpp"

namespace ftc {

constexpr int BW_B = 4;  // edges per batch

bool seg_shape(int dtype, int D, int *vec, int *lpr);

// Where dH goes.  `poison`, when not NULL and pointing at a non-zero value, turns every gradient into NaN (the pattern is not
// symmetric).  vec: rows are 16-byte aligned.
struct GradOut {
    void *dH;
    int ld, dt;
    bool vec;
    const int32_t *poison;
    template <int NV>
    __device__ __forceinline__ void store(int64_t row, int k, const float (&o)[NV]) const
    {
        if (vec) {
            store_vec_nt<NV>(dH, row * ld + k, dt, o);
        } else {
#pragma unroll
            for (int j = 0; j < NV; ++j) store_elem(dH, row * ld + k + j, dt, o[j]);
        }
    }
};

// m_i of dbeta = sum ds_e (c_e - m_i): the nearer to the mean of the row's cosines, the less of what z_i and t_i are off by gets into dbeta
// (t_i's error times mean c - m_i).  log(z_i / length) is beta mean c - |beta| to first order, whatever the signs and norms of the features.
// slope = 1 / (beta log2(e)), shift = the sign of beta; where beta is too small for the quotient both are 0, and so is m_i.
// Standard deviation of dbeta's error with m_i = 0, 1/2 and this, 2000 rows of 64 neighbours, D = 32, Y in fp16, beta = 1: signed
// features 2.9e-4 / 3.3e-3 / 1.2e-4, behind a ReLU 7.0e-3 / 3.3e-3 / 1.7e-4; the sweep takes 1 % longer than with a constant.
struct CosineMean {
    float slope, shift;
    explicit CosineMean(float beta)
        : slope(fabsf(beta) < 1e-4f ? 0.f : 0.693147181f / beta), shift(fabsf(beta) < 1e-4f ? 0.f : beta < 0.f ? -1.f : 1.f) {}
    __device__ __forceinline__ float operator()(float inv_z, int length) const
    {
        const float m = fmaf(-__builtin_amdgcn_logf(inv_z * static_cast<float>(length)), slope, shift);
        return slope == 0.f ? 0.f : fminf(fmaxf(m, -1.f), 1.f);
    }
};
__device__ __forceinline__ bool poisoned(const int32_t *flag) { return flag && *flag != 0; }

// 1 / max(|h|, 1e-12) from |h|^2: the hardware's reciprocal root and one Newton step
__device__ __forceinline__ float inverse_norm(float hh)
{
    const float q = fmaxf(hh, 1e-24f);
    const float r = __builtin_amdgcn_rsqf(q);
    const float better = fmaf(0.5f * r, fmaf(-q * r, r, 1.f), r);
    return q < 1e38f ? better : r;  // (an overflowed square keeps its 0)
}

// dH = agg + (q - hn <hn, q>) / |h| for one element; ri = 1 / |h|, t = <hn, q> / |h| (0 where the norm was clamped: the row is a
// plain scaling there)
__device__ __forceinline__ float through_norm(float agg, float q, float h, float ri, float t) { return fmaf(ri, fmaf(-h, t, q), agg); }
__device__ __forceinline__ float projection(float hq, float ri) { return ri >= 0.999e12f ? 0.f : hq * ri * ri; }

// stats[i] = (1 / z_i, <dY_i, Y_i>) and HD[i] = [h_i | dY_i] (element type of H, halves of DP
// elements, zero padded).  Eight lanes per row, 16 bytes of H and dY per lane and step (the caller
// guarantees 16-byte aligned rows of H and dY).  A row without entries gets (0, 0).
template <class T>
__global__ __launch_bounds__(256) void agnn_row_stats_kernel(int n, const void *__restrict__ H,
                                                             const void *__restrict__ dY, int ld,
                                                             const void *__restrict__ Y, int ldy, int ydt, int D, int DP,
                                                             const float *__restrict__ row_z, float2 *__restrict__ stats,
                                                             void *__restrict__ HD)
{
    constexpr int V = T::VEC;  // elements per 16 bytes
    const int sub = threadIdx.x & 7;
    const int64_t row = (static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x) >> 3;
    const bool y_vec = ydt == FTC_F32 && ldy % 4 == 0 && (reinterpret_cast<uintptr_t>(Y) & 15u) == 0;
    float t = 0.f;
    if (row < n) {
        char *dst = static_cast<char *>(HD) + row * 2 * DP * T::BYTES;
        for (int k = sub * V; k < DP; k += 8 * V) {  // DP is a multiple of V
            uint4 h = make_uint4(0u, 0u, 0u, 0u), d = h;
            if (k + V <= D) {
                h = *reinterpret_cast<const uint4 *>(static_cast<const char *>(H) + (row * ld + k) * T::BYTES);
                d = *reinterpret_cast<const uint4 *>(static_cast<const char *>(dY) + (row * ld + k) * T::BYTES);
                float df[V], yf[V];
                load_vec<T>(dY, row * ld + k, df);
                if (y_vec) {
#pragma unroll
                    for (int q = 0; q < V / 4; ++q) {
                        const float4 y4 = *reinterpret_cast<const float4 *>(static_cast<const float *>(Y) + row * ldy + k + 4 * q);
                        yf[4 * q] = y4.x; yf[4 * q + 1] = y4.y; yf[4 * q + 2] = y4.z; yf[4 * q + 3] = y4.w;
                    }
                } else {
#pragma unroll
                    for (int q = 0; q < V; ++q) yf[q] = load_elem(Y, row * ldy + k + q, ydt);
                }
#pragma unroll
                for (int q = 0; q < V; ++q) t = fmaf(df[q], yf[q], t);
            } else if (k < D) {  // a ragged last piece: element by element
                uint32_t hw[4] = {0u, 0u, 0u, 0u}, dw[4] = {0u, 0u, 0u, 0u};
                for (int q = 0; k + q < D; ++q) {
                    if constexpr (T::BYTES == 4) {
                        hw[q] = static_cast<const uint32_t *>(H)[row * ld + k + q];
                        dw[q] = static_cast<const uint32_t *>(dY)[row * ld + k + q];
                    } else {
                        hw[q / 2] |= static_cast<uint32_t>(static_cast<const uint16_t *>(H)[row * ld + k + q]) << (16 * (q & 1));
                        dw[q / 2] |= static_cast<uint32_t>(static_cast<const uint16_t *>(dY)[row * ld + k + q]) << (16 * (q & 1));
                    }
                    t = fmaf(load_elem(dY, row * ld + k + q, T::BYTES == 4 ? FTC_F32 : (std::is_same<T, F16>::value ? FTC_F16 : FTC_BF16)),
                             load_elem(Y, row * ldy + k + q, ydt), t);
                }
                h = make_uint4(hw[0], hw[1], hw[2], hw[3]);
                d = make_uint4(dw[0], dw[1], dw[2], dw[3]);
            }
            *reinterpret_cast<uint4 *>(dst + k * T::BYTES) = h;
            *reinterpret_cast<uint4 *>(dst + (DP + k) * T::BYTES) = d;
        }
    }
    t += __shfl_xor(t, 1, 64);
    t += __shfl_xor(t, 2, 64);
    t += __shfl_xor(t, 4, 64);
    if (row < n && sub == 0) {
        const float z = row_z[row];
        stats[row] = make_float2(z > 0.f ? 1.f / z : 0.f, t);
    }
}

// Four entries of a group are taken together, as in the forward pass: four dot products per entry by all lanes, their
// lane sums and the scalar work by one lane of the quad per entry (which also loads that entry's pair (1 / z_j, t_j)), the two
// coefficients back to all lanes.  Three waves per SIMD: what four have room for spills inside the loop (R-MAT graph, 2^20 nodes,
// 32 M entries, fp16, D = 32, forward and backward of four layers: 5.58 ms before, 5.06 with four waves, 4.87 with three).
template <class T, int VEC, int LPR, int R, bool BIG>
__global__ __launch_bounds__(256, 3) void agnn_backward_fused_kernel(
    int nnz, int n_ranges, const int *__restrict__ row_ptr, const int *__restrict__ col_idx, const int *__restrict__ edge_to_row,
    const void *__restrict__ HD, int D, float beta, const float2 *__restrict__ stats, CosineMean row_mean,
    GradOut grad, float *__restrict__ carry, int *__restrict__ carry_tail_row, float *__restrict__ dbeta_part)
{
    using E = EdgeRange<LPR, R>;
    constexpr int NG = E::NG, RUN = E::RUN;
    constexpr int DP = LPR * VEC;
    constexpr int DP2 = 2 * DP;  // q slots, then agg slots
    constexpr uint64_t ROW = DP2 * T::BYTES;  // bytes of a row of HD
    constexpr int IDX_WORDS = 2 * E::WORDS;
    constexpr int PART_WORDS = NG * DP2;
    __shared__ __align__(16) int smem[4][(IDX_WORDS > PART_WORDS ? IDX_WORDS : PART_WORDS) + PART_WORDS];

    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int g = lane / LPR, sub = lane % LPR, quad = lane & 3;
    const bool odd = lane & 1, upper = lane & 2;
    uint32_t *s_off = reinterpret_cast<uint32_t *>(smem[wave]);
    int *s_row = smem[wave] + E::WORDS;
    // the sums of the row that a group closes first, if it came in from the left: parked here, they are needed at the end only
    float *s_head = reinterpret_cast<float *>(smem[wave] + (IDX_WORDS > PART_WORDS ? IDX_WORDS : PART_WORDS)) + g * DP2 + sub * VEC;

    const int v = xcd_chunked_block(blockIdx.x, gridDim.x) * 4 + wave;
    if (v >= n_ranges) return;  // (no wave waits for another)
    const int base = v * R;
    const int n_valid = min(R, nnz - base);
    const int prev_row = base > 0 ? edge_to_row[base - 1] : -1;
    const int next_row = nnz - base > R ? edge_to_row[base + R] : -1;
    const int far_row = static_cast<int64_t>(base) + 2 * R < nnz ? edge_to_row[base + 2 * R] : -1;
    if (poisoned(grad.poison)) beta = __int_as_float(0x7fc00000);  // every weight is NaN then
    stage_range<LPR, R, false, BIG>(row_ptr, col_idx, edge_to_row, nullptr, base, n_valid, ROW, nullptr, lane, s_off, s_row, nullptr);

    const int at = g * E::RUNP;  // the group's run
    const bool live = sub * VEC < D;
    const uint32_t h_bytes = sub * VEC * T::BYTES, d_bytes = h_bytes + DP * T::BYTES;  // this lane's pieces of a row of HD
    const float beta2 = beta * 1.44269504f;  // powers of two, as in the forward pass
    const float beta2_rest = fmaf(beta, 1.92596299e-8f, fmaf(beta, 1.44269504f, -beta2));
    float acc[2 * VEC];  // [0, VEC): q slice, [VEC, 2 VEC): agg slice
#pragma unroll
    for (int j = 0; j < 2 * VEC; ++j) acc[j] = 0.f;
    // slices of the current row: of H[i,:] and dY[i,:] (for the dot products, ahead of the sums by up to a batch) and of H[i,:]
    // of the row whose sums are in acc
    RawVec<T, VEC> xi, dxi, xc;
    zero_raw(xi);
    zero_raw(dxi);
    zero_raw(xc);
    // of the row of this lane's entry: 1 / |h_i|, the pair (1 / z_i, t_i), the mean of the cosines
    float ri_mine = 0.f, mi_mine = 0.f, dbeta_acc = 0.f;
    float2 si_mine = make_float2(0.f, 0.f);
    bool head_closed = false, first = true;
    int head_row = -1, cur = -1;
    const int first_row = s_row[at];
    const bool left_open = first_row >= 0 && first_row == (g == 0 ? prev_row : s_row[max(at - 5, 0)]);  // the last entry of the run before

    auto load_h = [&](int row, RawVec<T, VEC> &x) { load_raw<T, VEC>(row_addr<BIG>(HD, row_slot<BIG>(max(row, 0), ROW), ROW, h_bytes), 0, x); };
    auto load_d = [&](int row, RawVec<T, VEC> &x) { load_raw<T, VEC>(row_addr<BIG>(HD, row_slot<BIG>(max(row, 0), ROW), ROW, d_bytes), 0, x); };
    // the sums of a complete row become its gradient (all lanes of the group)
    auto store_row = [&](int row, const RawVec<T, VEC> &x, const float (&a)[2 * VEC]) {
        float h[VEC], hq = 0.f, o[VEC];
        unpack<T, VEC>(x, h);
#pragma unroll
        for (int j = 0; j < VEC; ++j) hq = fmaf(h[j], a[j], hq);
        const float r = inverse_norm(group_sum_dpp<LPR>(dot_raw<T, VEC>(x, x, 0.f)));
        const float t = projection(group_sum_dpp<LPR>(hq), r);
#pragma unroll
        for (int j = 0; j < VEC; ++j) o[j] = through_norm(a[VEC + j], a[j], h[j], r, t);
        if (live) grad.store<VEC>(row, sub * VEC, o);
    };

#pragma unroll 1
    for (int b = 0; b < RUN; b += BW_B) {
        const uint4 o4 = *reinterpret_cast<const uint4 *>(s_off + at + b);
        const int4 r4 = *reinterpret_cast<const int4 *>(s_row + at + b);
        const uint32_t o[BW_B] = {o4.x, o4.y, o4.z, o4.w};
        const int r[BW_B] = {r4.x, r4.y, r4.z, r4.w};
        const uint32_t o_mine = s_off[at + b + quad];
        const int r_mine = s_row[at + b + quad];
        RawVec<T, VEC> y[BW_B], dy[BW_B];
#pragma unroll
        for (int k = 0; k < BW_B; ++k) {
            load_raw<T, VEC>(row_addr<BIG>(HD, o[k], ROW, h_bytes), 0, y[k]);
            load_raw<T, VEC>(row_addr<BIG>(HD, o[k], ROW, d_bytes), 0, dy[k]);
        }
        const float2 sj = stats[BIG ? o_mine : o_mine / static_cast<uint32_t>(ROW)];
        bool need[BW_B];  // a new row starts (the lanes of a group branch together)
        int begins = -2;  // the first of them: its slices are loaded ahead
#pragma unroll
        for (int k = BW_B - 1; k >= 0; --k) {
            need[k] = r[k] != (k ? r[k - 1] : cur);
            begins = need[k] ? r[k] : begins;
        }
        RawVec<T, VEC> xs, dxs;
        float2 ss;
        int s0, s1;
        if (begins != -2) {
            load_h(begins, xs);
            load_d(begins, dxs);
            ss = stats[max(begins, 0)];
            s0 = row_ptr[max(begins, 0)];
            s1 = row_ptr[max(begins, 0) + 1];
        }
        float hh[BW_B], squares[BW_B], dp[BW_B], dpt[BW_B];
        ri_mine = quad_lane<3>(ri_mine);  // until a row begins: those of the batch's last entry before
        mi_mine = quad_lane<3>(mi_mine);
        si_mine = make_float2(quad_lane<3>(si_mine.x), quad_lane<3>(si_mine.y));
#pragma unroll
        for (int k = 0; k < BW_B; ++k) {
            if (need[k]) {
                float2 si;
                int length;
                if (r[k] == begins) {
                    xi = xs;
                    dxi = dxs;
                    si = ss;
                    length = s1 - s0;
                } else {
                    load_h(r[k], xi);
                    load_d(r[k], dxi);
                    si = stats[max(r[k], 0)];
                    length = row_ptr[max(r[k], 0) + 1] - row_ptr[max(r[k], 0)];
                }
                const float ri = __frsqrt_rn(fmaxf(group_sum_dpp<LPR>(dot_raw<T, VEC>(xi, xi, 0.f)), 1e-24f));  // 1 / max(|h_i|, 1e-12)
                const float mi = row_mean(si.x, length);
                ri_mine = quad >= k ? ri : ri_mine;
                mi_mine = quad >= k ? mi : mi_mine;
                si_mine.x = quad >= k ? si.x : si_mine.x;
                si_mine.y = quad >= k ? si.y : si_mine.y;
            }
            hh[k] = dot_raw<T, VEC>(xi, y[k], 0.f);
            squares[k] = dot_raw<T, VEC>(y[k], y[k], 0.f);
            dp[k] = dot_raw<T, VEC>(dxi, y[k], 0.f);
            dpt[k] = dot_raw<T, VEC>(xi, dy[k], 0.f);
        }
        const float rj = __frsqrt_rn(fmaxf(group_sum4<LPR>(squares, odd, upper), 1e-24f));
        const float cs = ri_mine * rj * group_sum4<LPR>(hh, odd, upper);
        const float a = __builtin_amdgcn_exp2f(fmaf(beta2_rest, cs, fmaf(beta2, cs, -fabsf(beta2))));
        const float ds = a * si_mine.x * (group_sum4<LPR>(dp, odd, upper) - si_mine.y);
        const float pt = a * sj.x;
        const float dst = pt * (group_sum4<LPR>(dpt, odd, upper) - sj.y);
        const float coef = beta * (ds + dst) * rj;
        // What z_i and t_i are off by enters with what is left of the mean of the row's cosines, not with all of it
        if (r_mine >= 0 && sub < 4) dbeta_acc = fmaf(ds, cs - mi_mine, dbeta_acc);
        const float c4[BW_B] = {quad_lane<0>(coef), quad_lane<1>(coef), quad_lane<2>(coef), quad_lane<3>(coef)};
        const float p4[BW_B] = {quad_lane<0>(pt), quad_lane<1>(pt), quad_lane<2>(pt), quad_lane<3>(pt)};
#pragma unroll
        for (int k = 0; k < BW_B; ++k) {
            if (need[k]) {  // the previous row ends here
                if (cur >= 0) {
                    if (first && left_open) {
                        head_closed = true; head_row = cur;
#pragma unroll
                        for (int j = 0; j < VEC; ++j) { s_head[j] = acc[j]; s_head[DP + j] = acc[VEC + j]; }
                    } else {
                        store_row(cur, xc, acc);
                    }
                    first = false;
                }
                cur = r[k];
                if (r[k] == begins) xc = xs;
                else load_h(r[k], xc);
#pragma unroll
                for (int j = 0; j < 2 * VEC; ++j) acc[j] = 0.f;
            }
            float yf[VEC], dyf[VEC];
            unpack<T, VEC>(y[k], yf);
            unpack<T, VEC>(dy[k], dyf);
#pragma unroll
            for (int j = 0; j < VEC; ++j) {
                acc[j] = fmaf(c4[k], yf[j], acc[j]);
                acc[VEC + j] = fmaf(p4[k], dyf[j], acc[VEC + j]);
            }
        }
    }
    // the run's last segment
    int open = OPEN_NONE;
    if (cur >= 0) {
        const int right_row = g == NG - 1 ? next_row : s_row[at + E::RUNP];
        if (right_row == cur) {
            open = first && left_open ? OPEN_THROUGH : OPEN_TAIL;
        } else if (first && left_open) {
            head_closed = true; head_row = cur;
#pragma unroll
            for (int j = 0; j < VEC; ++j) { s_head[j] = acc[j]; s_head[DP + j] = acc[VEC + j]; }
        } else {
            store_row(cur, xc, acc);
        }
    }
    // the wave's share of dbeta: lanes in a fixed order
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) dbeta_acc += __shfl_xor(dbeta_acc, m, 64);
    if (lane == 0) dbeta_part[v] = dbeta_acc;
    // Rows cut inside this wave: the group that closes a row adds its pieces, in edge order.
    const int from = first_group<LPR>(open, g);
    const bool last_open = g == NG - 1 && open != OPEN_NONE;  // a row that goes on in the next range
    wave_lds_sync();  // the staged entries are dead: their place is taken by the open pieces
    float *part = reinterpret_cast<float *>(smem[wave]) + sub * VEC;
    if (open != OPEN_NONE) {
#pragma unroll
        for (int j = 0; j < VEC; ++j) { part[g * DP2 + j] = acc[j]; part[g * DP2 + DP + j] = acc[VEC + j]; }
    }
    wave_lds_sync();
    // carried piece: [2 v] of the row that came in from the left, [2 v + 1] of the one left open
    auto store_carry = [&](int slot, const float (&x)[2 * VEC]) {
        float q[VEC], ag[VEC];
#pragma unroll
        for (int j = 0; j < VEC; ++j) { q[j] = x[j]; ag[j] = x[VEC + j]; }
        const int64_t to = (static_cast<int64_t>(v) * 2 + slot) * DP2 + sub * VEC;
        store_vec<VEC>(carry, to, FTC_F32, q);
        store_vec<VEC>(carry, to + DP, FTC_F32, ag);
    };
    if (head_closed || (last_open && open == OPEN_THROUGH)) {
        if (head_closed) load_h(head_row, xi);
        float run[2 * VEC];
#pragma unroll
        for (int j = 0; j < 2 * VEC; ++j) run[j] = 0.f;
        for (int q = max(from, 0); q < g; ++q) {
#pragma unroll
            for (int j = 0; j < VEC; ++j) { run[j] += part[q * DP2 + j]; run[VEC + j] += part[q * DP2 + DP + j]; }
        }
#pragma unroll
        for (int j = 0; j < VEC; ++j) {
            run[j] += head_closed ? s_head[j] : acc[j];
            run[VEC + j] += head_closed ? s_head[DP + j] : acc[VEC + j];
        }
        if (from < 0) store_carry(0, run);
        else if (head_closed) store_row(head_row, xi, run);
        else store_carry(1, run);
    }
    if (last_open && open == OPEN_TAIL) store_carry(1, acc);
    if (lane == 63) {
        const int tail = last_open && !(open == OPEN_THROUGH && from < 0) ? cur : -1;
        carry_tail_row[2 * v] = tail;
        carry_tail_row[2 * v + 1] = (tail >= 0 && far_row != tail) ? 1 : 0;  // ends in range v + 1
    }
}

// Sum of the waves' shares in a fixed order by one workgroup of 256 threads.
__device__ __forceinline__ void dbeta_sum(int count, const float *__restrict__ partial, bool poison, float *out)
{
    __shared__ float red[4];
    float t[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    int i = threadIdx.x;
    for (; i + 7 * 256 < count; i += 8 * 256) {
#pragma unroll
        for (int k = 0; k < 8; ++k) t[k] += partial[i + k * 256];
    }
    for (; i < count; i += 256) t[0] += partial[i];
    float s = ((t[0] + t[1]) + (t[2] + t[3])) + ((t[4] + t[5]) + (t[6] + t[7]));
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) s += __shfl_xor(s, m, 64);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) *out = poison ? __int_as_float(0x7fc00000) : (red[0] + red[1]) + (red[2] + red[3]);
}

// Second pass: rows cut by a range boundary, rows without entries (gradient 0) and, in the first workgroup, the sum of dbeta.  As
// in the SpMM's second pass G lanes (four features of q and of agg each) finish a row, 64 / G rows per wave; the long rows of a
// power-law graph, which span more than two ranges, are taken one at a time by the whole wave.
template <class T, int G>
__global__ __launch_bounds__(256) void agnn_backward_fixup_kernel(int n, int n_ranges, const int *__restrict__ row_ptr,
                                                                  const float *__restrict__ carry,
                                                                  const int *__restrict__ carry_tail_row, int D,
                                                                  const void *__restrict__ HD, GradOut grad, int seg_r,
                                                                  const float *__restrict__ dbeta_part, float *__restrict__ dbeta)
{
    constexpr int R = 64 / G, DP = 4 * G, DP2 = 2 * DP;
    const bool poison = poisoned(grad.poison);
    if (blockIdx.x == 0) {
        dbeta_sum(n_ranges, dbeta_part, poison, dbeta);
        return;
    }
    const int block = blockIdx.x - 1;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int sub = lane % G;
    const int v_mine = (block * 4 + wave) * R + lane / G;
    int2 rec = make_int2(-1, 0);
    if (v_mine < n_ranges) rec = reinterpret_cast<const int2 *>(carry_tail_row)[v_mine];
    {
        // nearly every open row ends in the next range: its pieces are loaded together with the range's record
        const bool ok = v_mine + 1 < n_ranges;
        const float *head = carry + (ok ? static_cast<size_t>(v_mine) + 1 : 0) * 2 * DP2 + sub * 4;
        const float *tail = carry + ((ok ? static_cast<size_t>(v_mine) : 0) * 2 + 1) * DP2 + sub * 4;
        float4 hq = make_float4(0.f, 0.f, 0.f, 0.f), ha = hq, tq = hq, ta = hq;
        if (ok) {
            hq = *reinterpret_cast<const float4 *>(head);
            ha = *reinterpret_cast<const float4 *>(head + DP);
            tq = *reinterpret_cast<const float4 *>(tail);
            ta = *reinterpret_cast<const float4 *>(tail + DP);
        }
        const bool mine = ok && rec.x >= 0 && rec.y;
        RawVec<T, 4> x;
        zero_raw(x);
        if (mine) load_raw<T, 4>(HD, static_cast<int64_t>(rec.x) * DP2 + sub * 4, x);
        float h[4];
        unpack<T, 4>(x, h);
        const float q[4] = {hq.x + tq.x, hq.y + tq.y, hq.z + tq.z, hq.w + tq.w};
        const float ag[4] = {ha.x + ta.x, ha.y + ta.y, ha.z + ta.z, ha.w + ta.w};
        float hh = dot_raw<T, 4>(x, x, 0.f), p = 0.f;
#pragma unroll
        for (int i = 0; i < 4; ++i) p = sub * 4 + i < D ? fmaf(h[i], q[i], p) : p;
#pragma unroll
        for (int m = G / 2; m >= 1; m >>= 1) { hh += __shfl_xor(hh, m, 64); p += __shfl_xor(p, m, 64); }
        if (mine) {
            const float ri = inverse_norm(hh), t = projection(p, ri);
            float o[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) o[i] = through_norm(ag[i], q[i], h[i], ri, t);
            if (sub * 4 + 4 <= D) {
                grad.store<4>(rec.x, sub * 4, o);
            } else {
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if (sub * 4 + i < D) store_elem(grad.dH, static_cast<int64_t>(rec.x) * grad.ld + sub * 4 + i, grad.dt, o[i]);
            }
        }
    }
    // rows that go on beyond the next range
    unsigned long long longs = __builtin_amdgcn_ballot_w64(rec.x >= 0 && !rec.y && sub == 0);
    while (longs) {
        const int src = __ffsll(static_cast<long long>(longs)) - 1;
        longs &= longs - 1;
        const int v = __shfl(v_mine, src, 64), r = __shfl(rec.x, src, 64);
        const int last = (row_ptr[r + 1] - 1) / seg_r;  // range holding the row's final entry
        // teams of DL lanes (one per slot) share the row's ranges round-robin; their sums are added in team order: fixed by the
        // shape alone
        constexpr int DL = DP2 < 64 ? DP2 : 64, PARTS = 64 / DL, STEPS = DP2 / DL;
        const int part = lane / DL;
        float sum[STEPS];
#pragma unroll
        for (int st = 0; st < STEPS; ++st) {
            const int d = st * 64 + lane % DL;
            float s = sum_pieces(carry + d, 2 * static_cast<size_t>(DP2), v + 1 + part, last, PARTS);
            for (int off = 32; off >= DL; off >>= 1) s += __shfl_down(s, off, 64);
            sum[st] = s + carry[(static_cast<size_t>(v) * 2 + 1) * DP2 + d];  // meant for the lanes below DL
        }
        // slots [0, DP): q, [DP, 2 DP): agg of the same features.  DP < 64: both in one step, DP lanes apart; else in two steps.
        constexpr int FS = DP < 64 ? 1 : DP / 64;  // steps over the features
        const bool feat = lane < (DP < 64 ? DP : 64);
        float h[FS], hh = 0.f, p = 0.f;
#pragma unroll
        for (int st = 0; st < FS; ++st) {
            const int d = st * 64 + lane;
            h[st] = 0.f;
            if (feat && d < D) {
                RawVec<T, 2> x;  // (an element's pair: rows of HD are padded to whole pieces)
                load_raw<T, 2>(HD, static_cast<int64_t>(r) * DP2 + (d & ~1), x);
                float f[2];
                unpack<T, 2>(x, f);
                h[st] = f[d & 1];
                hh = fmaf(h[st], h[st], hh);
                p = fmaf(h[st], sum[st], p);
            }
        }
#pragma unroll
        for (int m = 32; m >= 1; m >>= 1) { hh += __shfl_xor(hh, m, 64); p += __shfl_xor(p, m, 64); }
        const float ri = inverse_norm(hh), t = projection(p, ri);
#pragma unroll
        for (int st = 0; st < FS; ++st) {
            const int d = st * 64 + lane;
            const float ag = DP < 64 ? __shfl(sum[0], (lane + DP) & 63, 64) : sum[(st + FS) % STEPS];
            if (feat && d < D)
                store_elem(grad.dH, static_cast<int64_t>(r) * grad.ld + d, grad.dt, through_norm(ag, sum[st], h[st], ri, t));
        }
    }
    const int64_t row = static_cast<int64_t>(block) * 256 + threadIdx.x;
    if (row < n && row_ptr[row] == row_ptr[row + 1])
        for (int d = 0; d < D; ++d) store_elem(grad.dH, row * grad.ld + d, grad.dt, poison ? __int_as_float(0x7fc00000) : 0.f);
}

// The fused pass covers the shapes of the edge-balanced kernels whose pair (q, agg) still fits the
// 256 slots of the fix-up kernel.
bool agnn_backward_fused_shape(int dtype, int D)
{
    int vec, lpr;
    return seg_shape(dtype, D, &vec, &lpr) && 2 * vec * lpr <= 256;
}

static size_t bw_dp2(int dtype, int D)
{
    int vec = 0, lpr = 0;
    seg_shape(dtype, D, &vec, &lpr);
    return 2 * static_cast<size_t>(vec) * lpr;
}

static size_t bw_ws(int n, int nnz, int r, size_t dp2)
{
    const size_t n_ranges = static_cast<size_t>(seg_count(nnz, r));
    return align_up(static_cast<size_t>(n) * dp2 * sizeof(float), 256) + align_up(static_cast<size_t>(n) * sizeof(float2), 256) +
           align_up(n_ranges * 2 * dp2 * sizeof(float), 256) + align_up(n_ranges * 2 * sizeof(int), 256) +
           align_up(n_ranges * sizeof(float), 256);
}

// [HD: n x DP2 elements | stats: n float2 | carry | tail rows | dbeta shares], DP2 of the widest element type
size_t agnn_backward_fused_ws(int n, int nnz, int D, bool least)
{
    size_t dp2 = 0;
    if (agnn_backward_fused_shape(FTC_F32, D)) dp2 = bw_dp2(FTC_F32, D);
    if (agnn_backward_fused_shape(FTC_F16, D) && bw_dp2(FTC_F16, D) > dp2) dp2 = bw_dp2(FTC_F16, D);
    if (dp2 == 0) return 0;
    return bw_ws(n, nnz, least ? SEG_R : seg_range(nnz, SEG_AGNN_BACKWARD), dp2);
}

template <class T, int R, bool BIG>
static void launch_bw_t(int vec, int lpr, unsigned grid, hipStream_t s, int nnz, int n_ranges, const ftc_csr &g,
                        const int *e2r, const void *HD, int D, float beta, const float2 *stats, GradOut grad, float *carry,
                        int *tail_row, float *dbeta_part)
{
    constexpr int VM = T::VEC;
#define FTC_BW(V, L)                                                                                                \
    hipLaunchKernelGGL((agnn_backward_fused_kernel<T, V, L, R, BIG>), dim3(grid), dim3(256), 0, s, nnz, n_ranges,   \
                       g.row_ptr, g.col_idx, e2r, HD, D, beta, stats, CosineMean(beta), grad, carry, tail_row, dbeta_part)
    if (vec == VM) {
        if (lpr == 4) FTC_BW(VM, 4);
        else if (lpr == 8) FTC_BW(VM, 8);
        else if (lpr == 16) FTC_BW(VM, 16);
        else if constexpr (T::BYTES == 4) FTC_BW(VM, 32);  // (16-bit pairs of that width are beyond agnn_backward_fused_shape())
    } else if (vec == VM / 2) {
        FTC_BW(VM / 2, 4);
    } else {
        FTC_BW(VM / 4, 4);
    }
#undef FTC_BW
}

template <class T>
static int32_t launch_bw(int vec, int lpr, int r, hipStream_t s, const ftc_csr &g, const int *e2r, const void *H, const void *dY,
                         int ld, int D, float beta, const float *row_z, const void *Y, int ldy, int ydt, GradOut grad, float *dbeta,
                         void *HD, float2 *stats, float *carry, int *tail_row, float *dbeta_part)
{
    const int n = g.n, dp = vec * lpr, n_ranges = static_cast<int>(seg_count(g.nnz, r));
    const unsigned grid_rows8 = static_cast<unsigned>((static_cast<int64_t>(n) * 8 + 255) / 256);
    hipLaunchKernelGGL(agnn_row_stats_kernel<T>, dim3(grid_rows8), dim3(256), 0, s, n, H, dY, ld, Y, ldy, ydt, D, dp, row_z, stats,
                       HD);
    if (n_ranges > 0) {
        const unsigned grid = static_cast<unsigned>((n_ranges + 3) / 4);
#define FTC_BWR(R, BIG) \
    launch_bw_t<T, R, BIG>(vec, lpr, grid, s, g.nnz, n_ranges, g, e2r, HD, D, beta, stats, grad, carry, tail_row, dbeta_part)
        if (rows_need_64_bits(n, 2 * static_cast<int64_t>(dp) * T::BYTES)) FTC_BWR(SEG_R, true);
        else if (r == SEG_R) FTC_BWR(SEG_R, false);
        else if (r == 256) FTC_BWR(256, false);
        else FTC_BWR(128, false);
#undef FTC_BWR
        const int32_t st = launch_status("agnn_backward_fused");
        if (st != FTC_OK) return st;
    }
    const int lanes = dp / 4;  // of a cut row: four features each
    const int64_t blocks_rows = (static_cast<int64_t>(n) + 255) / 256;
    const int64_t blocks_ranges = ceil_div(n_ranges, 4 * (64 / lanes));
    const unsigned grid2 = static_cast<unsigned>((blocks_rows > blocks_ranges ? blocks_rows : blocks_ranges) + 1);
#define FTC_FX(G)                                                                                                          \
    case G:                                                                                                                \
        hipLaunchKernelGGL((agnn_backward_fixup_kernel<T, G>), dim3(grid2), dim3(256), 0, s, n, n_ranges, g.row_ptr, carry, \
                           tail_row, D, HD, grad, r, dbeta_part, dbeta);                                                   \
        break;
    switch (lanes) {
        FTC_FX(1) FTC_FX(2) FTC_FX(4) FTC_FX(8) FTC_FX(16) FTC_FX(32)
    }
#undef FTC_FX
    return launch_status("agnn_backward_fused fixup");
}

// Caller has checked: window index present, agnn_backward_fused_shape(dt, D), rows of H and dY
// 16-byte aligned with the same leading dimension, workspace of agnn_backward_fused_ws() bytes.  pattern_flag: see GradOut.
int32_t launch_agnn_backward_fused(const ftc_csr &g, const ftc_windows &w, const void *H, const void *dY, int ld, int dt,
                                   int D, float beta, const float *row_z, const void *Y, int ldy, int ydt, void *dH,
                                   int lddh, int dh_dt, float *dbeta, const int32_t *pattern_flag, void *ws, size_t ws_bytes,
                                   hipStream_t s)
{
    int vec = 0, lpr = 0;
    seg_shape(dt, D, &vec, &lpr);
    const int dp2 = 2 * vec * lpr, n = g.n;
    const bool big = rows_need_64_bits(n, static_cast<int64_t>(dp2) * elem_size(dt));  // ranges of SEG_R only
    const int short_r = big ? SEG_R : seg_range(g.nnz, SEG_AGNN_BACKWARD);
    const int r = ws_bytes >= bw_ws(n, g.nnz, short_r, dp2) ? short_r : SEG_R;
    const size_t n_ranges = static_cast<size_t>(seg_count(g.nnz, r));
    char *p = static_cast<char *>(ws);
    void *HD = p;
    p += align_up(static_cast<size_t>(n) * dp2 * sizeof(float), 256);
    float2 *stats = reinterpret_cast<float2 *>(p);
    p += align_up(static_cast<size_t>(n) * sizeof(float2), 256);
    float *carry = reinterpret_cast<float *>(p);
    p += align_up(n_ranges * 2 * dp2 * sizeof(float), 256);
    int *tail_row = reinterpret_cast<int *>(p);
    p += align_up(n_ranges * 2 * sizeof(int), 256);
    float *dbeta_part = reinterpret_cast<float *>(p);
    const GradOut grad{dH, lddh, dh_dt, aligned16(dH) && (static_cast<int64_t>(lddh) * elem_size(dh_dt)) % 16 == 0, pattern_flag};
#define FTC_BWT(T) \
    launch_bw<T>(vec, lpr, r, s, g, w.edge_to_row, H, dY, ld, D, beta, row_z, Y, ldy, ydt, grad, dbeta, HD, stats, carry, tail_row, dbeta_part)
    if (dt == FTC_F32) return FTC_BWT(F32);
    if (dt == FTC_F16) return FTC_BWT(F16);
    return FTC_BWT(BF16);
#undef FTC_BWT
}

}  // namespace ftc
