// Work-balanced sparse neighbour aggregation (SpMM, Section V.A) on the vector units.
//
// The paper gives one row window to one thread block; on power-law graphs a single window can
// hold 10^5 edges while the median row has two, so here the unit of work is a fixed number of
// EDGES instead.  The window index supplies what makes that possible without searching:
// edge_to_row (`edgeToRow`) tells every edge its output row.
//
//   - A wave owns R consecutive edges (512; 256 or 128 on small graphs, seg_range()).  Their (column, value, row)
//     triples are loaded once, coalesced, into LDS.
//   - The wave is cut into groups of LPR lanes; a group walks a contiguous run of the wave's
//     edges, SEG_B at a time (SEG_B independent 16-byte gathers of X rows in flight per lane),
//     and accumulates in registers while the row stays the same.
//   - A row that lies completely inside one run is stored straight from registers.  A row cut by
//     a run boundary leaves partial sums: those inside one wave are added in edge order by the group that
//     closes the row (all groups at once; one lane per feature walking over the groups took as long as two batches of
//     gathers on short ranges); the pieces that cross a wave boundary go to a small carry buffer and are added, again
//     in edge order, by a second tiny kernel.  No floating-point atomics: results are
//     reproducible bit for bit.
//
// What bounds it: gathers that miss L2 on large graphs (block model, 10^6 nodes, bf16, 64 columns: 0.67 ms, a kernel that only
// gathers these rows 0.58), else the instructions around the gather (edge_ranges.hpp) and, on small graphs, the chain
// index, gather, sum of a wave (GCN layer with 100 000 nodes, fp16 128 -> 32: 44 -> 33 us with the update before it).
#include "edge_ranges.hpp"

namespace ftc {

constexpr int SEG_B = 4;    // edges per batch (gathers in flight per lane)

static int pow2_ceil(int x)
{
    int p = 1;
    while (p < x) p *= 2;
    return p;
}

// Lane layout for a feature width: `vec` elements per lane, `lpr` lanes per row (4..32).
bool seg_shape(int dtype, int D, int *vec, int *lpr)
{
    const int vmax = dtype == FTC_F32 ? 4 : 8;
    for (int v = vmax; v >= vmax / 4 && v >= 1; v /= 2) {
        if (D % v != 0) continue;
        const int l = pow2_ceil(D / v);
        // narrower-than-16-byte lanes exist only in the 4-lane layout (small D)
        if (l >= 4 && l <= (v == vmax ? 32 : 4)) {
            *vec = v;
            *lpr = l;
            return true;
        }
    }
    return false;
}

// The same for any width and any alignment: 16-byte pieces at element alignment; where the width is no multiple of a
// piece the last lane's piece is moved back to end with the row (it then shares columns with its neighbour, both hold
// the same sums).  Rows of at least one piece.
static bool seg_shape_ragged(int dtype, int D, int *vec, int *lpr)
{
    const int v = dtype == FTC_F32 ? 4 : 8;
    const int l = pow2_ceil((D + v - 1) / v);
    if (D < v || l > 32) return false;
    *vec = v;
    *lpr = l < 4 ? 4 : l;
    return true;
}

static size_t seg_carry_ws(int nnz, int r, int dp)
{
    const size_t n_ranges = static_cast<size_t>(seg_count(nnz, r));
    return align_up(n_ranges * 2 * dp * sizeof(float), 256) + align_up(n_ranges * 2 * sizeof(int), 256);
}

// Edges per wave for rows of dp slots: as seg_range() says, as long as the carried pieces stay below 32 MiB and, with the
// flags of the windows, fit the built-in buffer of ftc_spmm_noalloc.
static int spmm_range(int n, int nnz, int dp)
{
    int r = seg_range(nnz, SEG_SPMM);
    while (r < SEG_R && (seg_carry_ws(nnz, r, dp) > (static_cast<size_t>(32) << 20) ||
                         seg_carry_ws(nnz, r, dp) + flag_bytes(n) > NOALLOC_SCRATCH_BYTES))
        r *= 2;
    return r;
}

// Scratch memory of the kernel that takes widths or alignments seg_shape() does not (lane: the kernel for narrow rows), 0 where
// none does: where it would not fit the built-in buffer of ftc_spmm_noalloc (47 columns, 67 M entries; a wider X more) both
// calls stay with the row-wise kernel.
size_t spmm_any_width_ws(int dtype, int D, int n, int nnz, bool lane)
{
    int vec, lpr;
    size_t need = 0;
    if (lane) need = spmm_lane_ws(nnz, false);
    else if (seg_shape_ragged(dtype, D, &vec, &lpr)) need = seg_carry_ws(nnz, spmm_range(n, nnz, vec * lpr), vec * lpr);
    return need + flag_bytes(n) <= NOALLOC_SCRATCH_BYTES ? need : 0;
}

size_t spmm_seg_ws(int n, int nnz, int D, bool least)
{
    if (nnz == 0) return 0;
    size_t need = 0;
    int vec, lpr;
    bool any = false;
    for (const int dt : {FTC_F32, FTC_F16}) {
        size_t k = 0;
        if (seg_shape(dt, D, &vec, &lpr)) {
            any = true;
            k = seg_carry_ws(nnz, least ? SEG_R : spmm_range(n, nnz, vec * lpr), vec * lpr);
        }
        need = k > need ? k : need;
        k = least ? 0 : spmm_any_width_ws(dt, D, n, nnz, false);
        need = k > need ? k : need;
    }
    if (D <= 16) {  // narrow rows may take the lane-per-edge kernel
        const size_t lane = any ? spmm_lane_ws(nnz, least) : least ? 0 : spmm_any_width_ws(FTC_F32, D, n, nnz, true);
        need = lane > need ? lane : need;
    }
    return need;
}

// VALS = false: all edge values are one (vals == NULL): nothing is staged or multiplied for them, which
// also cuts the LDS footprint (more workgroups per CU).  RAGGED: any width from one piece on, any alignment.
template <class T, int VEC, int LPR, bool VALS, int R, bool RAGGED, bool BIG>
__global__ __launch_bounds__(256) void spmm_seg_kernel(int nnz, int n_ranges, const int *__restrict__ row_ptr,
                                                       const int *__restrict__ col_idx,
                                                       const int *__restrict__ edge_to_row,
                                                       const float *__restrict__ vals,
                                                       const void *__restrict__ X, uint64_t ldb, int D,
                                                       void *__restrict__ out, int ldo, int odt, Epi epi,
                                                       float *__restrict__ carry, int *__restrict__ carry_tail_row,
                                                       const uint8_t *__restrict__ dense)
{
    using E = EdgeRange<LPR, R>;
    constexpr int NG = E::NG, RUN = E::RUN;
    constexpr int DP = LPR * VEC;     // padded feature width
    constexpr int IDX_WORDS = (VALS ? 3 : 2) * E::WORDS;
    constexpr int PART_WORDS = NG * DP;
    __shared__ __align__(16) int smem[4][IDX_WORDS > PART_WORDS ? IDX_WORDS : PART_WORDS];

    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int g = lane / LPR, sub = lane % LPR;
    uint32_t *s_off = reinterpret_cast<uint32_t *>(smem[wave]);
    int *s_row = smem[wave] + E::WORDS;
    float *s_val = reinterpret_cast<float *>(smem[wave] + 2 * E::WORDS);  // only with VALS

    const int v = xcd_chunked_block(blockIdx.x, gridDim.x) * 4 + wave;
    if (v >= n_ranges) return;  // (no wave waits for another)
    const int base = v * R;
    const int n_valid = min(R, nnz - base);
    const int prev_row = base > 0 ? edge_to_row[base - 1] : -1;
    const int next_row = nnz - base > R ? edge_to_row[base + R] : -1;
    // row of the first edge after the NEXT range: tells whether a row left open here ends there
    const int far_row = static_cast<int64_t>(base) + 2 * R < nnz ? edge_to_row[base + 2 * R] : -1;
    stage_range<LPR, R, VALS, BIG>(row_ptr, col_idx, edge_to_row, vals, base, n_valid, ldb, dense, lane, s_off, s_row, s_val);

    const int at = g * E::RUNP;  // the group's run
    const bool live = sub * VEC < D;
    // first column of this lane's piece; lanes beyond the row gather its first piece and store nothing
    const int col0 = RAGGED ? min(sub * VEC, D - VEC) : live ? sub * VEC : 0;
    const uint32_t lane_bytes = static_cast<uint32_t>(col0) * T::BYTES;
    float acc[VEC], hacc[VEC];
#pragma unroll
    for (int j = 0; j < VEC; ++j) { acc[j] = 0.f; hacc[j] = 0.f; }
    bool head_closed = false;
    int head_row = -1;
    // an fp16 element is widened by the multiply-add that also takes the value, so without values a one that the compiler
    // does not know takes their place (one instruction per element instead of two)
    float one = 1.f;
    if constexpr (!VALS && std::is_same<T, F16>::value) asm("" : "+v"(one));

    auto store_row = [&](int row, float f, const float (&a)[VEC]) {
        if (live && !(dense && dense[row >> 4])) {
            float o[VEC];
#pragma unroll
            for (int j = 0; j < VEC; ++j) o[j] = epi.apply(f, a[j]);
            if constexpr (RAGGED) store_vec_any<VEC>(out, static_cast<int64_t>(row) * ldo + col0, odt, o);
            else store_vec_nt<VEC>(out, static_cast<int64_t>(row) * ldo + col0, odt, o);
        }
    };

    int cur = s_row[at];
    const bool left_open = cur >= 0 && cur == (g == 0 ? prev_row : s_row[max(at - 5, 0)]);  // the last entry of the run before
    bool first = true;
    float factor = epi.factor(max(cur, 0));  // loaded where the row begins: where it ends nothing has to be waited for
#pragma unroll 1
    for (int b = 0; b < RUN; b += SEG_B) {
        const uint4 o4 = *reinterpret_cast<const uint4 *>(s_off + at + b);
        const int4 r4 = *reinterpret_cast<const int4 *>(s_row + at + b);
        const uint32_t o[SEG_B] = {o4.x, o4.y, o4.z, o4.w};
        const int r[SEG_B] = {r4.x, r4.y, r4.z, r4.w};
        float a[SEG_B];
        if constexpr (VALS) {
            const float4 a4 = *reinterpret_cast<const float4 *>(s_val + at + b);
            a[0] = a4.x; a[1] = a4.y; a[2] = a4.z; a[3] = a4.w;
        } else {
#pragma unroll
            for (int k = 0; k < SEG_B; ++k) a[k] = one;
        }
        RawVec<T, VEC> x[SEG_B];
#pragma unroll
        for (int k = 0; k < SEG_B; ++k) {
            const char *p = row_addr<BIG>(X, o[k], ldb, lane_bytes);
            if constexpr (RAGGED) load_raw_any<T>(p, 0, x[k]);
            else load_raw<T, VEC>(p, 0, x[k]);
        }
#pragma unroll
        for (int k = 0; k < SEG_B; ++k) {
            if (r[k] != cur) {  // the segment of row `cur` ends here
                if (cur >= 0) {
                    if (first && left_open) {
#pragma unroll
                        for (int j = 0; j < VEC; ++j) hacc[j] = acc[j];
                        head_closed = true; head_row = cur;
                    } else {
                        store_row(cur, factor, acc);
                    }
                }
                first = false;
                cur = r[k];
                factor = epi.factor(max(cur, 0));
#pragma unroll
                for (int j = 0; j < VEC; ++j) acc[j] = 0.f;
            }
            float xf[VEC];
            unpack<T, VEC>(x[k], xf);
#pragma unroll
            for (int j = 0; j < VEC; ++j)
                acc[j] = VALS || std::is_same<T, F16>::value ? fmaf(a[k], xf[j], acc[j]) : acc[j] + xf[j];
        }
    }
    // the run's last segment
    int open = OPEN_NONE;
    if (cur >= 0) {
        const int right_row = g == NG - 1 ? next_row : s_row[at + E::RUNP];
        if (right_row == cur) {
            open = first && left_open ? OPEN_THROUGH : OPEN_TAIL;
        } else if (first && left_open) {
#pragma unroll
            for (int j = 0; j < VEC; ++j) hacc[j] = acc[j];
            head_closed = true; head_row = cur;
        } else {
            store_row(cur, factor, acc);
        }
    }
    // Rows cut inside this wave: the group that closes a row adds its pieces, in edge order.
    const int from = first_group<LPR>(open, g);
    const bool last_open = g == NG - 1 && open != OPEN_NONE;  // a row that goes on in the next range
    wave_lds_sync();  // the staged entries are dead: their place is taken by the open pieces
    float *part = reinterpret_cast<float *>(smem[wave]);
    if (open != OPEN_NONE && live) {
#pragma unroll
        for (int j = 0; j < VEC; ++j) part[g * DP + col0 + j] = acc[j];
    }
    wave_lds_sync();
    // carried piece: [2 v] of the row that came in from the left, [2 v + 1] of the one left open
    auto store_carry = [&](int slot, const float (&a)[VEC]) {
        const int64_t to = (static_cast<int64_t>(v) * 2 + slot) * DP + col0;
        if constexpr (RAGGED) {
            if (live) store_vec_any<VEC>(carry, to, FTC_F32, a);
        } else {
            if (live) store_vec<VEC>(carry, to, FTC_F32, a);
        }
    };
    if (head_closed || (last_open && open == OPEN_THROUGH)) {
        float run[VEC];
#pragma unroll
        for (int j = 0; j < VEC; ++j) run[j] = 0.f;
        for (int q = max(from, 0); q < g; ++q) {
#pragma unroll
            for (int j = 0; j < VEC; ++j) run[j] += part[q * DP + col0 + j];
        }
#pragma unroll
        for (int j = 0; j < VEC; ++j) run[j] += head_closed ? hacc[j] : acc[j];
        if (from < 0) store_carry(0, run);
        else if (head_closed) store_row(head_row, epi.factor(head_row), run);
        else store_carry(1, run);
    }
    if (last_open && open == OPEN_TAIL) store_carry(1, acc);
    if (lane == 63) {
        const int tail = last_open && !(open == OPEN_THROUGH && from < 0) ? cur : -1;
        carry_tail_row[2 * v] = tail;
        carry_tail_row[2 * v + 1] = (tail >= 0 && far_row != tail) ? 1 : 0;  // ends in range v + 1
    }
}

// Second pass: rows cut by a wave boundary, and rows without any stored entry.  G lanes (four features
// each) finish one cut row, 64 / G rows per wave: the kernel is a chain of two dependent loads per row (the
// range's record, then the two pieces), so it is the number of rows in flight that counts.  DP is a
// multiple of 4 and the carry buffer 16-byte aligned (both by construction of the first pass).
template <int G>
__global__ __launch_bounds__(256) void spmm_seg_fixup_kernel(int n, int n_ranges, const int *__restrict__ row_ptr,
                                                             const float *__restrict__ carry,
                                                             const int *__restrict__ carry_tail_row, int DP,
                                                             int D, void *__restrict__ out, int ldo, int odt,
                                                             Epi epi, const uint8_t *__restrict__ dense, int seg_r)
{
    constexpr int R = 64 / G;  // ranges per wave
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int sub = lane % G;
    const int v_mine = (blockIdx.x * 4 + wave) * R + lane / G;
    int2 rec = make_int2(-1, 0);
    if (v_mine < n_ranges) rec = reinterpret_cast<const int2 *>(carry_tail_row)[v_mine];
    // Nearly every open row ends in the next range: out = head piece of range v + 1 + tail piece of
    // range v.  Their addresses depend on v alone, so they are loaded together with the range's record
    // instead of after it.
    for (int f0 = 0; f0 < DP; f0 += 4 * G) {
        const int f = f0 + sub * 4;
        const bool ok = v_mine + 1 < n_ranges && f < DP;
        const size_t vv = ok ? static_cast<size_t>(v_mine) : 0;
        float4 h4 = make_float4(0.f, 0.f, 0.f, 0.f), t4 = h4;
        if (ok) {
            h4 = *reinterpret_cast<const float4 *>(carry + (vv + 1) * 2 * DP + f);
            t4 = *reinterpret_cast<const float4 *>(carry + (vv * 2 + 1) * DP + f);
        }
        int r = rec.x;
        if (r >= 0 && dense && dense[r >> 4]) r = -1;
        if (f0 == 0) rec.x = r;
        if (ok && r >= 0 && rec.y) {
            const float fac = epi.factor(r);
            const float o[4] = {h4.x + t4.x, h4.y + t4.y, h4.z + t4.z, h4.w + t4.w};
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (f + i < D) store_elem(out, static_cast<int64_t>(r) * ldo + f + i, odt, epi.apply(fac, o[i]));
        }
    }
    // rows that go on beyond the next range (long rows of a power-law graph): one at a time, by the whole wave
    unsigned long long longs = __builtin_amdgcn_ballot_w64(rec.x >= 0 && !rec.y && sub == 0);
    while (longs) {
        const int src = __ffsll(static_cast<long long>(longs)) - 1;
        longs &= longs - 1;
        const int v = __shfl(v_mine, src, 64), r = __shfl(rec.x, src, 64);
        const int last = (row_ptr[r + 1] - 1) / seg_r;  // wave range holding the row's final edge
        // A hub row can span hundreds of ranges.  The 64 lanes are split into `parts` teams of
        // `dl` lanes (one lane per feature); team p adds the head pieces of ranges v+1+p,
        // v+1+p+parts, ..., then the teams' sums are added in team order.  The
        // order is fixed by the shape alone, so the result is reproducible.
        int dl = 1;
        while (dl < D && dl < 64) dl <<= 1;
        const int parts = 64 / dl;
        const int part = lane / dl;
        for (int d0 = 0; d0 < D; d0 += 64) {
            const int d = d0 + lane % dl;
            const bool dok = d < D;
            const float *base = carry + (dok ? d : 0);
            float sum = sum_pieces(base, 2 * static_cast<size_t>(DP), v + 1 + part, last, parts);
            for (int off = 32; off >= dl; off >>= 1) sum += __shfl_down(sum, off, 64);
            if (lane < dl && dok) {
                sum += carry[(static_cast<size_t>(v) * 2 + 1) * DP + d];
                store_elem(out, static_cast<int64_t>(r) * ldo + d, odt, epi.apply(epi.factor(r), sum));
            }
        }
    }
    const int64_t row = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
    if (row < n && row_ptr[row] == row_ptr[row + 1] && !(dense && dense[row >> 4]))
        for (int d = 0; d < D; ++d) store_elem(out, row * ldo + d, odt, 0.f);
}

int32_t launch_seg_fixup(int n, int n_ranges, const int *row_ptr, const float *carry, const int *tail_row, int dp,
                         int D, void *out, int ldo, int odt, Epi epi, const uint8_t *dense, int seg_r, hipStream_t s,
                         const char *what)
{
    int grp = 1;
    while (grp * 4 < dp && grp < 16) grp <<= 1;  // at most 16 lanes a row: wider rows take several rounds
    const int64_t blocks_rows = (static_cast<int64_t>(n) + 255) / 256;
    const int64_t blocks_ranges = ceil_div(n_ranges, 4 * (64 / grp));
    const unsigned grid2 = static_cast<unsigned>(blocks_rows > blocks_ranges ? blocks_rows : blocks_ranges);
#define FTC_FX(G)                                                                                                  \
    case G:                                                                                                        \
        hipLaunchKernelGGL(spmm_seg_fixup_kernel<G>, dim3(grid2), dim3(256), 0, s, n, n_ranges, row_ptr, carry,    \
                           tail_row, dp, D, out, ldo, odt, epi, dense, seg_r);                                     \
        break;
    switch (grp) {
        FTC_FX(1) FTC_FX(2) FTC_FX(4) FTC_FX(8) FTC_FX(16)
    }
#undef FTC_FX
    return launch_status(what);
}

template <class T, int R, bool BIG>
static void launch_seg_t(int vec, int lpr, bool ragged, hipStream_t s, int n_ranges, const ftc_csr &g, const int *e2r,
                         const float *vals, const void *X, uint64_t ldb, int D, void *out, int ldo, int odt, Epi epi,
                         float *carry, int *tail_row, const uint8_t *dense)
{
    constexpr int VM = T::VEC;
    const dim3 grid(static_cast<unsigned>((n_ranges + 3) / 4));
#define FTC_SEG1(V, L, W, RG)                                                                                          \
    hipLaunchKernelGGL((spmm_seg_kernel<T, V, L, W, R, RG, BIG>), grid, dim3(256), 0, s, g.nnz, n_ranges, g.row_ptr,   \
                       g.col_idx, e2r, vals, X, ldb, D, out, ldo, odt, epi, carry, tail_row, dense)
#define FTC_SEG(V, L, RG)                      \
    do {                                       \
        if (vals) FTC_SEG1(V, L, true, RG);    \
        else FTC_SEG1(V, L, false, RG);        \
    } while (0)
    if (ragged) {
        if (lpr == 4) FTC_SEG(VM, 4, true);
        else if (lpr == 8) FTC_SEG(VM, 8, true);
        else if (lpr == 16) FTC_SEG(VM, 16, true);
        else FTC_SEG(VM, 32, true);
    } else if (vec == VM) {
        if (lpr == 4) FTC_SEG(VM, 4, false);
        else if (lpr == 8) FTC_SEG(VM, 8, false);
        else if (lpr == 16) FTC_SEG(VM, 16, false);
        else FTC_SEG(VM, 32, false);
    } else if (vec == VM / 2) {
        FTC_SEG(VM / 2, 4, false);
    } else {
        FTC_SEG(VM / 4, 4, false);
    }
#undef FTC_SEG
#undef FTC_SEG1
}

template <class T>
static void launch_seg_r(int r, bool big, int vec, int lpr, bool ragged, hipStream_t s, int n_ranges, const ftc_csr &g,
                         const int *e2r, const float *vals, const void *X, uint64_t ldb, int D, void *out, int ldo, int odt,
                         Epi epi, float *carry, int *tail_row, const uint8_t *dense)
{
#define FTC_SEGR(R, BIG) \
    launch_seg_t<T, R, BIG>(vec, lpr, ragged, s, n_ranges, g, e2r, vals, X, ldb, D, out, ldo, odt, epi, carry, tail_row, dense)
    if (big) FTC_SEGR(SEG_R, true);
    else if (r == SEG_R) FTC_SEGR(SEG_R, false);
    else if (r == 256) FTC_SEGR(256, false);
    else FTC_SEGR(128, false);
#undef FTC_SEGR
}

// Caller has checked: window index present; seg_shape() accepts (xdt, D), rows of X and out 16-byte aligned and a workspace of
// spmm_seg_ws(.., least) bytes, or a workspace of spmm_any_width_ws() > 0 bytes.
int32_t launch_spmm_seg(const ftc_csr &g, const ftc_windows &w, const float *vals, const void *X, int ldx,
                        int xdt, int D, void *out, int ldo, int odt, Epi epi, void *ws, size_t ws_bytes,
                        const uint8_t *dense, hipStream_t s)
{
    const bool x16 = aligned16(X) && (static_cast<int64_t>(ldx) * elem_size(xdt)) % 16 == 0;
    const bool o16 = aligned16(out) && (static_cast<int64_t>(ldo) * elem_size(odt)) % 16 == 0;
    // rows of at most 32 bytes: one or two lanes per run of edges instead of four lanes per row
    if (!dense && x16 && spmm_lane_shape(xdt, D, ldx))
        return launch_spmm_lane(g, w, vals, X, ldx, xdt, D, out, ldo, odt, epi, ws, ws_bytes, s);
    int vec = 0, lpr = 0;
    const bool ragged = !(x16 && o16 && seg_shape(xdt, D, &vec, &lpr));
    if (ragged) seg_shape_ragged(xdt, D, &vec, &lpr);
    const int dp = vec * lpr;
    const int64_t row_bytes = static_cast<int64_t>(ldx) * elem_size(xdt);
    const bool big = rows_need_64_bits(g.n, row_bytes);  // ranges of SEG_R only: such a matrix has many rows
    const int short_r = big ? SEG_R : spmm_range(g.n, g.nnz, dp);
    const int r = ws_bytes >= seg_carry_ws(g.nnz, short_r, dp) ? short_r : SEG_R;
    const int n_ranges = static_cast<int>(seg_count(g.nnz, r));
    float *carry = static_cast<float *>(ws);
    int *tail_row = reinterpret_cast<int *>(static_cast<char *>(ws) +
                                            align_up(static_cast<size_t>(n_ranges) * 2 * dp * sizeof(float), 256));
    if (n_ranges > 0) {
        if (xdt == FTC_F32)
            launch_seg_r<F32>(r, big, vec, lpr, ragged, s, n_ranges, g, w.edge_to_row, vals, X, static_cast<uint64_t>(row_bytes), D, out, ldo, odt, epi, carry, tail_row, dense);
        else if (xdt == FTC_F16)
            launch_seg_r<F16>(r, big, vec, lpr, ragged, s, n_ranges, g, w.edge_to_row, vals, X, static_cast<uint64_t>(row_bytes), D, out, ldo, odt, epi, carry, tail_row, dense);
        else
            launch_seg_r<BF16>(r, big, vec, lpr, ragged, s, n_ranges, g, w.edge_to_row, vals, X, static_cast<uint64_t>(row_bytes), D, out, ldo, odt, epi, carry, tail_row, dense);
        const int32_t st = launch_status("spmm_seg");
        if (st != FTC_OK) return st;
    }
    return launch_seg_fixup(g.n, n_ranges, g.row_ptr, carry, tail_row, dp, D, out, ldo, odt, epi, dense, r, s,
                            "spmm_seg fixup");
}

}  // namespace ftc
