// Sparse neighbour aggregation (SpMM, Section V.A) for narrow feature rows: at most 32 bytes per
// row (D <= 16 for 16-bit features, D <= 8 for fp32), the widths of the GCN hidden and output layers.
//
// The edge-balanced kernel of spmm_seg.hip puts four lanes on a row; with rows this narrow a lane
// then loads 4 or 8 bytes per edge and the per-edge bookkeeping outweighs the arithmetic.  Here a
// SLOT of LPE lanes owns 16 (small graphs: 4) consecutive edges, and each of its lanes loads one 16-byte piece of
// every row (LPE = 1: rows of 16 bytes; LPE = 2: rows of 32 bytes, the two halves in neighbouring
// lanes, so that a load instruction touches one contiguous segment per edge -- two loads per lane
// for the two halves were measured slower than the four-lane layout, 0.35 against 0.30 ms on the
// R-MAT benchmark graph: what costs is the number of separate segments a load instruction touches):
//   - the slot gathers the rows of its edges, eight loads in flight, and accumulates while the
//     output row stays the same; a row that begins and ends inside the slot is stored at once;
//   - the pieces of rows that continue from slot to slot are joined by ONE segmented scan over the
//     wave (data-parallel-primitive moves or lane shuffles, the row beginnings are the segment heads);
//   - the pieces of rows cut by a wave boundary go to the carry buffer of the edge-balanced
//     kernels and are finished by their fix-up kernel, in edge order.
// No floating-point atomics: results are reproducible bit for bit.
//
// The rows of a range come from the row starts inside it, marked as bits in LDS: a lane's 16 edges are 16 bits, the rows before
// them a prefix sum over the wave.  The output scales of these rows are fetched once into LDS: where a row ends nearly every
// step of the loop has a lane that stores, and each would wait for its scale from memory.  Counting starts one by one, 64-bit
// addresses and scales from memory, against this, us (with edge values, R-MAT, 32 M entries): fp16 D = 8 238 / 218, bf16 D = 16
// 277 / 260, fp32 D = 8 265 / 254; power law, 3.8 M entries: 34.3 / 33.6, 47 / 43, 43 / 41.  What remains is the gather (163 and 196
// for 16- and 32-byte rows on the R-MAT graph) and 0.13 to 0.26 GB of ids and values.
#include "edge_ranges.hpp"

namespace ftc {

// Consecutive edges per lane: 16, or 4 on graphs whose ranges of 1024 / 512 edges would leave the chip idle.  fp16, 8 columns,
// us with 16 / 4: 20 / 13 at 9 thousand entries, 20 / 14 at 0.6 M, 23 / 20 at 1.5 M, 35 / 37 at 3.8 M.
constexpr int SL_LONG = 16, SL_SHORT = 4;
static int lane_edges(int nnz) { return nnz >= (1 << 21) ? SL_LONG : SL_SHORT; }

template <int CTRL, int ROW_MASK>
__device__ __forceinline__ int sl_dpp(int v)
{
    return __builtin_amdgcn_update_dpp(0, v, CTRL, ROW_MASK, 0xf, false);
}

// Segmented inclusive scan (sum) of N floats per lane over the lanes of a wave; head != 0 marks the
// first lane of a segment.  Shifts by 1, 2, 4, 8 inside rows of 16 lanes, then lane 15 of a row into
// the next row (rows 1 and 3) and lane 31 into rows 2 and 3; a lane stops taking from the left once
// a head lies in its span.
template <int N>
__device__ __forceinline__ void wave_segmented_sum(float (&x)[N], int head, int lane)
{
#define FTC_STEP(CTRL, ROW_MASK, VALID)                                                          \
    {                                                                                            \
        const int yh = sl_dpp<CTRL, ROW_MASK>(head);                                             \
        _Pragma("unroll") for (int j = 0; j < N; ++j)                                            \
        {                                                                                        \
            const float y = __int_as_float(sl_dpp<CTRL, ROW_MASK>(__float_as_int(x[j])));        \
            if ((VALID) && !head) x[j] += y;                                                     \
        }                                                                                        \
        if (VALID) head |= yh;                                                                   \
    }
    const int r16 = lane & 15;
    FTC_STEP(0x111, 0xf, r16 >= 1)
    FTC_STEP(0x112, 0xf, r16 >= 2)
    FTC_STEP(0x114, 0xf, r16 >= 4)
    FTC_STEP(0x118, 0xf, r16 >= 8)
    FTC_STEP(0x142, 0xa, (lane & 16) != 0)
    FTC_STEP(0x143, 0xc, lane >= 32)
#undef FTC_STEP
}

// Shuffle-based variant of the scan for slots of LPE lanes (a slot's lanes hold different pieces of the
// same rows and share the head flag): Kogge-Stone steps over distances of LPE, 2 LPE, ... lanes.
template <int N, int LPE>
__device__ __forceinline__ void wave_segmented_sum_slots(float (&x)[N], int head, int lane)
{
#pragma unroll
    for (int d = LPE; d < 64; d <<= 1) {
        const int yh = __shfl_up(head, d, 64);
        float y[N];
#pragma unroll
        for (int j = 0; j < N; ++j) y[j] = __shfl_up(x[j], d, 64);
        if (lane >= d) {
            if (!head) {
#pragma unroll
                for (int j = 0; j < N; ++j) x[j] += y[j];
            }
            head |= yh;
        }
    }
}

// Rows of the lane's SL_L consecutive edges (a slot's LPE lanes have the same): rows[k] of edge base + slot SL_L + k of a full range.
// `mark` is LDS of the wave, one bit per edge.  False (wave-uniform) when the range holds more than RANGE / 2 row starts or two rows start at one
// edge, i.e. one is empty: the caller then reads edge_to_row.  All 64 lanes must be active.
template <int SL_L, int LPE>
__device__ __forceinline__ bool slot_rows(const int *__restrict__ row_ptr, int r_first, int n_starts, int base, int lane,
                                          uint32_t *mark, int (&rows)[SL_L])
{
    constexpr int RANGE = 64 * SL_L / LPE;
    static_assert(SL_L == 16 || SL_L == 4, "a slot's marks are half a word or half a byte");
    if (n_starts > RANGE / 2) return false;
    if (lane < RANGE / 32) mark[lane] = 0u;
    wave_lds_sync();
    for (int t = lane; t < n_starts; t += 64) {
        const int p = row_ptr[r_first + 1 + t] - base - 1;  // bit p - 1: a row starts at edge p
        atomicOr(mark + (p >> 5), 1u << (p & 31));
    }
    wave_lds_sync();
    const int slot = lane / LPE;
    const uint32_t mine = SL_L == 16 ? mark[slot >> 1] >> (16 * (slot & 1)) & 0xffffu : mark[slot >> 3] >> (4 * (slot & 7)) & 0xfu;
    const int count = __popc(mine);
    const int upto = wave_inclusive_scan(lane % LPE == 0 ? count : 0);
    if (__builtin_amdgcn_readlane(upto, 63) != n_starts) return false;
    const int before = r_first + upto - count;
#pragma unroll
    for (int k = 0; k < SL_L; ++k) rows[k] = before + __popc(mine & ((1u << k) - 1u));
    return true;
}

// LPE: lanes per edge (1: rows of one 16-byte piece; 2: rows of two pieces, neighbouring lanes load the two
// halves of a row, so a load instruction still touches one contiguous 32-byte segment per edge).
// VALS = false: all edge values are one.
template <class T, int LPE, bool VALS, int SL_L, bool BIG>
__global__ __launch_bounds__(256) void spmm_lane_kernel(int nnz, int n_ranges, const int *__restrict__ row_ptr,
                                                        const int *__restrict__ col_idx,
                                                        const int *__restrict__ edge_to_row,
                                                        const float *__restrict__ vals, const void *__restrict__ X,
                                                        uint64_t ldb, int D, void *__restrict__ out, int ldo, int odt, Epi epi,
                                                        float *__restrict__ carry, int *__restrict__ carry_tail_row,
                                                        int idx_vec, int out_vec)
{
    constexpr int V = T::VEC, DP = V;          // a lane holds one 16-byte piece of its rows
    constexpr int DPT = V * LPE;               // padded row width (carry rows)
    constexpr int RANGE = 64 * SL_L / LPE;     // edges per wave
    constexpr int SL_B = SL_L < 8 ? SL_L : 8;  // gathers issued together
    constexpr int SCALES = 128;
    __shared__ uint32_t s_mark[4][RANGE / 32];
    __shared__ float s_scale[4][SCALES];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int slot = lane / LPE, piece = lane % LPE;
    const int v = xcd_chunked_block(blockIdx.x, gridDim.x) * 4 + wave;
    if (v >= n_ranges) return;  // no workgroup barrier below
    const int base = v * RANGE;
    const int n_valid = min(RANGE, nnz - base);
    const int prev_row = base > 0 ? edge_to_row[base - 1] : -1;
    const int next_row = base + n_valid < nnz ? edge_to_row[base + n_valid] : -1;
    const int far_row = static_cast<int64_t>(base) + 2 * RANGE < nnz ? edge_to_row[base + 2 * RANGE] : -1;
    const int r_first = edge_to_row[base], r_last = edge_to_row[base + n_valid - 1];
    const int e0 = slot * SL_L;
    const bool scales_staged = epi.scale && r_last - r_first < SCALES;
    if (scales_staged)
        for (int t = lane; t <= r_last - r_first; t += 64) s_scale[wave][t] = epi.scale[r_first + t];
    wave_lds_sync();
    auto factor = [&](int row) {
        // (a row that came in from the left began before r_first only if it is r_first: rows here are r_first .. r_last)
        return scales_staged ? s_scale[wave][row - r_first] : epi.factor(row);
    };
    uint32_t c[SL_L];  // where the edges' rows of X begin
    int r[SL_L];
    float a[VALS ? SL_L : 1];
    if (idx_vec && n_valid == RANGE) {
#pragma unroll
        for (int q = 0; q < SL_L / 4; ++q) {
            const int4 c4 = *reinterpret_cast<const int4 *>(col_idx + base + e0 + 4 * q);
            c[4 * q] = row_slot<BIG>(c4.x, ldb); c[4 * q + 1] = row_slot<BIG>(c4.y, ldb);
            c[4 * q + 2] = row_slot<BIG>(c4.z, ldb); c[4 * q + 3] = row_slot<BIG>(c4.w, ldb);
            if constexpr (VALS) {
                const float4 a4 = *reinterpret_cast<const float4 *>(vals + base + e0 + 4 * q);
                a[4 * q] = a4.x; a[4 * q + 1] = a4.y; a[4 * q + 2] = a4.z; a[4 * q + 3] = a4.w;
            }
        }
        // the rows of the lane's edges: from the row starts of the range where that works, else the per-entry stream
        if (!slot_rows<SL_L, LPE>(row_ptr, r_first, r_last - r_first, base, lane, s_mark[wave], r)) {
#pragma unroll
            for (int q = 0; q < SL_L / 4; ++q) {
                const int4 r4 = *reinterpret_cast<const int4 *>(edge_to_row + base + e0 + 4 * q);
                r[4 * q] = r4.x; r[4 * q + 1] = r4.y; r[4 * q + 2] = r4.z; r[4 * q + 3] = r4.w;
            }
        }
    } else {
#pragma unroll
        for (int k = 0; k < SL_L; ++k) {  // padding: rows of their own, never stored, that gather the last entry's row
            const bool ok = e0 + k < n_valid;
            const int at = base + min(e0 + k, n_valid - 1);
            c[k] = row_slot<BIG>(col_idx[at], ldb);
            r[k] = ok ? edge_to_row[at] : -2 - (e0 + k);
            if constexpr (VALS) a[k] = vals[at];
        }
    }
    float one = 1.f;  // fp16 without values: see spmm_seg.hip
    if constexpr (!VALS && std::is_same<T, F16>::value) asm("" : "+v"(one));
    int left;  // row of the edge before the slot's first
    if constexpr (LPE == 1) left = sl_dpp<0x138, 0xf>(r[SL_L - 1]);  // wave_shr:1
    else left = __shfl_up(r[SL_L - 1], LPE, 64);
    if (slot == 0) left = prev_row;

    auto store_row = [&](int row, const float(&s)[DP]) {
        if (row < 0) return;
        const float f = factor(row);
        float o[DP];
#pragma unroll
        for (int j = 0; j < DP; ++j) o[j] = epi.apply(f, s[j]);
        if (out_vec) {  // D == DPT, rows of out 16-byte aligned
#pragma unroll
            for (int j = 0; j < DP; j += 4) {
                const float o4[4] = {o[j], o[j + 1], o[j + 2], o[j + 3]};
                store_vec<4>(out, static_cast<int64_t>(row) * ldo + piece * V + j, odt, o4);
            }
        } else {
#pragma unroll
            for (int j = 0; j < DP; ++j)
                if (piece * V + j < D) store_elem(out, static_cast<int64_t>(row) * ldo + piece * V + j, odt, o[j]);
        }
    };

    float acc[DP], first_piece[DP];
#pragma unroll
    for (int j = 0; j < DP; ++j) { acc[j] = 0.f; first_piece[j] = 0.f; }
    int nb = 0;  // row beginnings inside the slot
#pragma unroll
    for (int h = 0; h < SL_L / SL_B; ++h) {
        RawVec<T, V> y[SL_B];
#pragma unroll
        for (int k = 0; k < SL_B; ++k) load_raw<T, V>(row_addr<BIG>(X, c[h * SL_B + k], ldb, piece * 16), 0, y[k]);
#pragma unroll
        for (int k = 0; k < SL_B; ++k) {
            const int i = h * SL_B + k;
            const int before = i == 0 ? left : r[i - 1];
            if (r[i] != before) {  // a row begins: the piece so far is finished
                if (nb == 0) {
#pragma unroll
                    for (int j = 0; j < DP; ++j) first_piece[j] = acc[j];  // joined with the lanes on the left below
                } else {
                    store_row(before, acc);  // began and ended inside this lane
                }
                ++nb;
#pragma unroll
                for (int j = 0; j < DP; ++j) acc[j] = 0.f;
            }
            float yf[V];
            unpack<T, V>(y[k], yf);
#pragma unroll
            for (int j = 0; j < V; ++j) {
                if constexpr (VALS) acc[j] = fmaf(a[i], yf[j], acc[j]);
                else if constexpr (std::is_same<T, F16>::value) acc[j] = fmaf(one, yf[j], acc[j]);
                else acc[j] += yf[j];
            }
        }
    }
    if (nb == 0) {
#pragma unroll
        for (int j = 0; j < DP; ++j) first_piece[j] = acc[j];
    }
    // one segmented scan joins the lanes' last (or only) pieces
    float incl[DP];
#pragma unroll
    for (int j = 0; j < DP; ++j) incl[j] = acc[j];
    if constexpr (LPE == 1) wave_segmented_sum<DP>(incl, nb > 0 ? 1 : 0, lane);
    else wave_segmented_sum_slots<DP, LPE>(incl, nb > 0 ? 1 : 0, lane);
    // what flows into a slot from the left (every lane takes part in the shift)
    float t[DP];
#pragma unroll
    for (int j = 0; j < DP; ++j) {
        float fl;
        if constexpr (LPE == 1) fl = __int_as_float(sl_dpp<0x138, 0xf>(__float_as_int(incl[j])));  // wave_shr:1
        else fl = __shfl_up(incl[j], LPE, 64);
        if (slot == 0) fl = 0.f;
        t[j] = fl + first_piece[j];
    }
    float *carry_head = carry + (static_cast<size_t>(v) * 2) * DPT + piece * V;
    float *carry_tail = carry + (static_cast<size_t>(v) * 2 + 1) * DPT + piece * V;
    if (nb > 0) {  // the row that was open at the slot's start ends at the slot's first beginning
        if (left == prev_row) {  // it entered the wave from the left: the wave's head piece
#pragma unroll
            for (int j = 0; j < DP; ++j) carry_head[j] = t[j];
        } else {
            store_row(left, t);
        }
    }
    const bool any_begin = __builtin_amdgcn_ballot_w64(nb > 0) != 0ull;
    if (slot == 64 / LPE - 1) {  // the last slot holds the wave's last row
        const int last_row = r[SL_L - 1];
        const bool right_open = n_valid == RANGE && next_row == last_row;
        int tail_out = -1;
        if (!any_begin) {  // one row covers the whole wave (it entered from the left)
#pragma unroll
            for (int j = 0; j < DP; ++j) carry_head[j] = incl[j];
        } else if (right_open) {
#pragma unroll
            for (int j = 0; j < DP; ++j) carry_tail[j] = incl[j];
            tail_out = last_row;
        } else {
            store_row(last_row, incl);  // the last row ends with the wave
        }
        if (piece == 0) {
            carry_tail_row[2 * v] = tail_out;
            carry_tail_row[2 * v + 1] = (tail_out >= 0 && far_row != tail_out) ? 1 : 0;  // ends in range v + 1
        }
    }
}

// Row widths this kernel takes: one or two 16-byte pieces, rows of X at least that long.
bool spmm_lane_shape(int xdt, int D, int ldx)
{
    const int per = xdt == FTC_F32 ? 4 : 8;
    const int lpe = (D + per - 1) / per;
    return D >= 1 && lpe <= 2 && ldx >= lpe * per;
}

static size_t lane_carry_ws(int nnz, int range, int dp)
{
    const size_t n_ranges = static_cast<size_t>(seg_count(nnz, range));
    return align_up(n_ranges * 2 * dp * sizeof(float), 256) + align_up(n_ranges * 2 * sizeof(int), 256);
}

size_t spmm_lane_ws(int nnz, bool least)
{
    if (nnz == 0) return 0;
    return lane_carry_ws(nnz, 64 * (least ? SL_LONG : lane_edges(nnz)) / 2, 16);  // the shorter ranges of LPE = 2
}

template <class T, int L, bool BIG>
static void launch_lane_t(int lpe, unsigned grid, hipStream_t s, int nnz, int n_ranges, const ftc_csr &g, const int *e2r,
                          const float *vals, const void *X, uint64_t ldb, int D, void *out, int ldo, int odt, Epi epi,
                          float *carry, int *tail_row, int idx_vec, int out_vec)
{
#define FTC_LANE(LPE, VALS)                                                                                         \
    hipLaunchKernelGGL((spmm_lane_kernel<T, LPE, VALS, L, BIG>), dim3(grid), dim3(256), 0, s, nnz, n_ranges, g.row_ptr, \
                       g.col_idx, e2r, vals, X, ldb, D, out, ldo, odt, epi, carry, tail_row, idx_vec, out_vec)
    if (lpe == 1) {
        if (vals) FTC_LANE(1, true);
        else FTC_LANE(1, false);
    } else {
        if (vals) FTC_LANE(2, true);
        else FTC_LANE(2, false);
    }
#undef FTC_LANE
}

// Caller has checked: window index present, spmm_lane_shape(), rows of X 16-byte aligned, workspace
// of spmm_lane_ws(.., least) bytes.
int32_t launch_spmm_lane(const ftc_csr &g, const ftc_windows &w, const float *vals, const void *X, int ldx, int xdt,
                         int D, void *out, int ldo, int odt, Epi epi, void *ws, size_t ws_bytes, hipStream_t s)
{
    const int per = xdt == FTC_F32 ? 4 : 8;
    const int lpe = (D + per - 1) / per, dp = per * lpe;
    const int64_t row_bytes = static_cast<int64_t>(ldx) * elem_size(xdt);
    const bool big = rows_need_64_bits(g.n, row_bytes);  // long ranges only: such a matrix has many rows
    const int short_range = 64 * (big ? SL_LONG : lane_edges(g.nnz)) / lpe;
    const int range = ws_bytes >= lane_carry_ws(g.nnz, short_range, dp) ? short_range : 64 * SL_LONG / lpe;
    const bool full = range == 64 * SL_LONG / lpe;
    const int n_ranges = ceil_div(g.nnz, range);
    float *carry = static_cast<float *>(ws);
    int *tail_row = reinterpret_cast<int *>(static_cast<char *>(ws) +
                                            align_up(static_cast<size_t>(n_ranges) * 2 * dp * sizeof(float), 256));
    const int idx_vec = aligned16(g.col_idx) && aligned16(w.edge_to_row) && (!vals || aligned16(vals));
    const int out_vec = D == dp && aligned16(out) && (static_cast<int64_t>(ldo) * elem_size(odt)) % 16 == 0;
    if (n_ranges > 0) {
        const unsigned grid = static_cast<unsigned>((n_ranges + 3) / 4);
#define FTC_LANE1(T, L, BIG)                                                                                             \
    launch_lane_t<T, L, BIG>(lpe, grid, s, g.nnz, n_ranges, g, w.edge_to_row, vals, X, static_cast<uint64_t>(row_bytes), D, \
                             out, ldo, odt, epi, carry, tail_row, idx_vec, out_vec)
#define FTC_LANES(T)                             \
    do {                                         \
        if (big) FTC_LANE1(T, SL_LONG, true);    \
        else if (full) FTC_LANE1(T, SL_LONG, false); \
        else FTC_LANE1(T, SL_SHORT, false);      \
    } while (0)
        if (xdt == FTC_F32) FTC_LANES(F32);
        else if (xdt == FTC_F16) FTC_LANES(F16);
        else FTC_LANES(BF16);
#undef FTC_LANES
#undef FTC_LANE1
        const int32_t st = launch_status("spmm_lane");
        if (st != FTC_OK) return st;
    }
    return launch_seg_fixup(g.n, n_ranges, g.row_ptr, carry, tail_row, dp, D, out, ldo, odt, epi, nullptr, range, s,
                            "spmm_lane fixup");
}

}  // namespace ftc
