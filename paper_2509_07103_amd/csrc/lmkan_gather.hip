// Layers and batches too small for a table to be streamed through LDS: every pass is one launch,
// nothing but the table rows that the samples touch is read, and no scratch memory is used.
//
// The slab kernels pay for the whole table (a 1024 -> 1024 layer: 0.6 GB, 115 us, for a single row)
// and for the passes around them (records, partial sums, zero fills, transposes, the four launches
// of the sort), 5 us each however little there is to do.  Here the inputs are located by the lanes
// that need them, and the rows are gathered from HBM / L2 with 16-byte loads: LPR lanes share a row of
// 4 Q LPR outputs (Q quads of outputs per lane), a wave takes 64 / LPR (row, pair) items at once.
// What bounds the gathers is the texture addresser (four lanes per clock and CU) once the rows come
// from L2, HBM latency and bandwidth for few rows of a large table.
#include <math.h>

#include <type_traits>

#include "lmkan_gather.h"

namespace lmkan {

namespace {

// The outputs of a lane among the 4 Q LPR of a tile: quads at first() and, Q = 2, second().  Float32
// rows arrive in loads that each run along the lanes, 16-bit rows (always Q = 2) in a single one.
template <typename CT, int LPR, int Q>
struct Columns {
    static_assert(sizeof(CT) == 4 || Q == 2, "16-bit rows are read eight outputs at a time");
    static __device__ __forceinline__ int first(int cl) { return sizeof(CT) == 4 ? cl * 4 : cl * 8; }
    static __device__ __forceinline__ int second(int cl) { return sizeof(CT) == 4 ? cl * 4 + 4 * LPR : cl * 8 + 4; }
};

// the coefficients of a lane's outputs in one row, as stored; `step`: distance of the second quad
template <typename CT, int Q>
struct Row {
    uint4 raw;
    __device__ __forceinline__ void load(const CT *p, int64_t) { raw = *reinterpret_cast<const uint4 *>(p); }
    __device__ __forceinline__ void widen(float (&f)[8]) const
    {
        const unsigned w[4] = {raw.x, raw.y, raw.z, raw.w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if constexpr (!std::is_same<CT, bf16_t>::value) {
                typedef _Float16 h2v __attribute__((ext_vector_type(2)));
                const h2v h = __builtin_bit_cast(h2v, w[i]);
                f[2 * i] = (float)h.x;
                f[2 * i + 1] = (float)h.y;
            } else {
                f[2 * i] = __uint_as_float(w[i] << 16);
                f[2 * i + 1] = __uint_as_float(w[i] & 0xffff0000u);
            }
        }
    }
};
template <int Q>
struct Row<float, Q> {
    float4 v[Q];
    __device__ __forceinline__ void load(const float *p, int64_t step)
    {
        v[0] = *reinterpret_cast<const float4 *>(p);
        if constexpr (Q == 2) v[1] = *reinterpret_cast<const float4 *>(p + step);
    }
    __device__ __forceinline__ void widen(float (&f)[4 * Q]) const
    {
#pragma unroll
        for (int q = 0; q < Q; ++q) f[4 * q] = v[q].x, f[4 * q + 1] = v[q].y, f[4 * q + 2] = v[q].z, f[4 * q + 3] = v[q].w;
    }
};

template <typename CT, int Q>
__device__ __forceinline__ void add_row(float (&acc)[4 * Q], float w, const Row<CT, Q> &r)
{
    float f[4 * Q];
    r.widen(f);
#pragma unroll
    for (int i = 0; i < 4 * Q; ++i) acc[i] = fmaf(w, f[i], acc[i]);
}

// element of the table where column `col` of node 0 of pair 0 starts (0 for a column the table lacks:
// what is read there is dropped)
__device__ __forceinline__ int64_t column_offset(const GatherArgs &a, int col)
{
    return col < a.col_limit ? (int64_t)(col >> 6) * a.map.s_tile + (col & 63) : 0;
}

// Four adjacent values of row n of a [B][n_out] tensor from column col on.  Rows of a ragged output
// count start on 4 bytes only, which a 16-byte load allows on this hardware, and its last columns may
// come from the row behind it (the caller drops them); only at the end of the tensor are they read
// one by one.
__device__ __forceinline__ float4 load_row4(const float *base, int64_t n, int col, int n_out, int64_t elems)
{
    typedef float f4u __attribute__((ext_vector_type(4), aligned(4)));
    const int64_t at = n * n_out + col;
    if (at + 4 <= elems) {
        const f4u v = *reinterpret_cast<const f4u *>(base + at);
        return make_float4(v.x, v.y, v.z, v.w);
    }
    float4 r = make_float4(base[at], 0.f, 0.f, 0.f);
    if (at + 1 < elems) r.y = base[at + 1];
    if (at + 2 < elems) r.z = base[at + 2];
    return r;
}

// conv_input_offset in two parts, with 32-bit divisions (rows and inputs of a window fit 32 bits):
// where the window of row n starts, and where its input e lies relative to that
__device__ __forceinline__ int64_t window_start(const ConvGeom &cg, int64_t n)
{
    const unsigned row = (unsigned)n, t = row / (unsigned)cg.OW, img = t / (unsigned)cg.OH;
    const unsigned ox = row - t * cg.OW, oy = t - img * cg.OH;
    return (((int64_t)img * cg.H + oy * cg.stride) * cg.W + ox * cg.stride) * cg.C;
}

__device__ __forceinline__ int64_t input_in_window(const ConvGeom &cg, int e)
{
    const unsigned t = (unsigned)e / (unsigned)cg.C, c = e - t * cg.C, ky = t / (unsigned)cg.kw, kx = t - ky * cg.kw;
    return ((int64_t)ky * cg.W + kx) * cg.C + c;
}

// offsets of the two inputs of pair k relative to the start of a row (or window)
__device__ __forceinline__ void pair_offsets(const GatherArgs &a, int k, int64_t &first, int64_t &second)
{
    first = 2 * k;
    second = first + 1;
    if (a.conv) {
        first = input_in_window(a.cg, 2 * k);
        second = (a.cg.C & 1) ? input_in_window(a.cg, 2 * k + 1) : first + 1;
    }
}

__device__ __forceinline__ float2 input_pair(const GatherArgs &a, int64_t n, int64_t first, int64_t second)
{
    if (!a.conv) return *reinterpret_cast<const float2 *>(a.x + n * a.n_in + first);
    const float *w = a.x + window_start(a.cg, n);
    return make_float2(w[first], w[second]);
}

__device__ __forceinline__ float2 input_pair(const GatherArgs &a, int64_t n, int k)
{
    int64_t first, second;
    pair_offsets(a, k, first, second);
    return input_pair(a, n, first, second);
}

// what the lanes of a wave hand each other through LDS must be written before it is read
__device__ __forceinline__ void wave_lds_fence()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// ---------------------------------------------------------------------------
// Forward.  The pairs of a row are dealt to `spw` slots of a wave (slot = LPR lanes) and `wpr`
// waves; a wave holds NS / spw rows.  Its lanes first locate 64 (row, pair) items (one each, the
// pairs of a row side by side), hand them over through LDS, then every slot walks its items: four
// row pieces, 32 multiply-adds.  The slots and waves of a row are summed in a fixed order.
// ---------------------------------------------------------------------------
template <typename CT, int LPR, int Q, int NW>
__global__ __launch_bounds__(NW * 64) void forward_gather_kernel(GatherArgs a)
{
    constexpr int NS = 64 / LPR;
    __shared__ float4 s_grid[LMKAN_MAX_GRID];
    __shared__ float4 s_w[NW][64];
    __shared__ int64_t s_off[NW][64];
    __shared__ float s_red[NW][LPR][4 * Q];
    stage_intervals(a.tab, s_grid);
    __syncthreads();

    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int slot = lane / LPR, cl = lane % LPR;
    const int ct = blockIdx.x % a.n_ct;
    // (powers of two, given by their logarithms: a division each would cost more than the gathers of a
    // single row)  spw: slots of a wave that share a row, wpr: waves; per_row: items of a row in one
    // chunk; rows_wave: rows of a wave; slot_rows: rows that a slot takes one after the other (one, unless
    // a chunk holds all pairs of a row)
    constexpr int kLogNS = NS == 64 ? 6 : NS == 32 ? 5 : NS == 16 ? 4 : NS == 8 ? 3 : 2;
    const int spw = 1 << a.log_spw, wpr = 1 << a.log_wpr, per_row = 1 << a.log_per_row;
    const int rows_wave = 64 >> a.log_per_row, slot_rows = 1 << (6 - a.log_per_row + a.log_spw - kLogNS);
    const int w = wave & (wpr - 1), q = slot & (spw - 1);
    const int p_item = lane & (per_row - 1);  // the item this lane locates

    const int base = ct * (4 * Q * LPR);
    const int col[2] = {base + Columns<CT, LPR, Q>::first(cl), base + Columns<CT, LPR, Q>::second(cl)};
    const CT *P = static_cast<const CT *>(a.P) + column_offset(a, col[0]);
    // (a second quad past the table repeats the first)
    const int64_t step = col[1] < a.col_limit ? column_offset(a, col[1]) - column_offset(a, col[0]) : 0;
    const int64_t d01 = a.map.s_node, d10 = (int64_t)a.W * a.map.s_node;

    // adds the items of this slot among the located ones (row r of the wave, pairs k0 ...)
    auto walk = [&](float (&acc)[4 * Q], int r, int k0) {
        const int count = min(per_row >> a.log_spw, (a.K - k0 - q + spw - 1) >> a.log_spw);
        const int first = r * per_row + q;
#pragma unroll 2
        for (int t = 0; t < count; ++t) {
            const float4 wv = s_w[wave][first + t * spw];
            const CT *row = P + s_off[wave][first + t * spw];
            Row<CT, Q> r00, r01, r10, r11;
            r00.load(row, step);
            r01.load(row + d01, step);
            r10.load(row + d10, step);
            r11.load(row + d10 + d01, step);
            add_row<CT, Q>(acc, wv.x, r00);
            add_row<CT, Q>(acc, wv.y, r10);
            add_row<CT, Q>(acc, wv.z, r01);
            add_row<CT, Q>(acc, wv.w, r11);
        }
    };
    // sums the slots of a row inside the wave
    auto reduce = [&](float (&acc)[4 * Q]) {
        for (int m = LPR; m < LPR << a.log_spw; m <<= 1)
#pragma unroll
            for (int i = 0; i < 4 * Q; ++i) acc[i] += __shfl_xor(acc[i], m, 64);
    };
    auto store = [&](const float (&acc)[4 * Q], int64_t n) {
        if (q == 0 && n < a.B) {
#pragma unroll
            for (int h = 0; h < Q; ++h)
                if (col[h] < a.n_out) store_outputs(a.out + n * a.n_out + col[h], acc + 4 * h, a.n_out, col[h], false);
        }
    };

    for (int64_t group = blockIdx.x / a.n_ct; group < a.groups; group += gridDim.x / a.n_ct) {
        const int64_t n0 = (group * (NW >> a.log_wpr) + (wave >> a.log_wpr)) * rows_wave;
        const int64_t n_item = n0 + (lane >> a.log_per_row), n_mine = n0 + (slot >> a.log_spw);
        float acc[4 * Q] = {};
        for (int k0 = w * per_row; k0 < a.K; k0 += wpr * per_row) {
            int64_t off = 0;
            float4 wt = make_float4(0.f, 0.f, 0.f, 0.f);
            if (k0 + p_item < a.K && n_item < a.B) {
                const float2 xv = input_pair(a, n_item, k0 + p_item);
                float4 c1, c2;
                const int i1 = locate_cell(s_grid, a.W - 1, xv.x, c1), i2 = locate_cell(s_grid, a.W - 1, xv.y, c2);
                const float u = (xv.x - c1.z) * c1.w, v = (xv.y - c2.z) * c2.w;
                wt = make_float4((1.f - u) * (1.f - v), u * (1.f - v), (1.f - u) * v, u * v);
                off = (int64_t)(i1 * a.W + i2) * a.map.s_node + (int64_t)(k0 + p_item) * a.map.s_pair;
            }
            wave_lds_fence();  // the previous items have been read
            s_w[wave][lane] = wt;
            s_off[wave][lane] = off;
            wave_lds_fence();
            for (int i = 0; i < slot_rows; ++i) {
                const int r = (slot >> a.log_spw) + (i << (kLogNS - a.log_spw));
                if (n0 + r < a.B) walk(acc, r, k0);
                if (slot_rows > 1) {  // the chunk holds the whole row
                    reduce(acc);
                    store(acc, n0 + r);
#pragma unroll
                    for (int e = 0; e < 4 * Q; ++e) acc[e] = 0.f;
                }
            }
        }
        if (slot_rows > 1) continue;
        reduce(acc);
        if (wpr > 1) {  // then the slots of a wave share one row
            if (slot == 0)
#pragma unroll
                for (int e = 0; e < 4 * Q; ++e) s_red[wave][cl][e] = acc[e];
            __syncthreads();
            if (w == 0 && slot == 0) {
                for (int i = 1; i < wpr; ++i)
#pragma unroll
                    for (int e = 0; e < 4 * Q; ++e) acc[e] += s_red[wave + i][cl][e];
                store(acc, n_mine);
            }
            __syncthreads();
        } else {
            store(acc, n_mine);
        }
    }
}

// ---------------------------------------------------------------------------
// Input gradient.  A slot takes a (row, pair): its lanes walk the outputs, each forming the four
// differences of neighbouring corners times gy (differences first: on a smooth table the four dot
// products agree in most digits), the derivatives are summed over the slot's lanes and written as
// one pair.  Every (row, pair) belongs to one slot: no atomics, no clearing (except into the
// overlapping windows of an image, which the caller clears).
// ---------------------------------------------------------------------------
template <int NW>
struct InputShared {
    float4 w[NW][64];  // u, v, 1/h1, 1/h2
    int64_t off[NW][64];
};

template <typename CT, int LPR, int Q, int NW>
__device__ __forceinline__ void input_gather(const GatherArgs &a, int block, const float4 *s_grid, InputShared<NW> &sh)
{
    constexpr int NS = 64 / LPR;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int slot = lane / LPR, cl = lane % LPR;
    // a wave takes `items` = rows_wave x per_row items
    const int per_row = 1 << a.log_per_row, items = a.items, rows_wave = items >> a.log_per_row;
    const int64_t id = (int64_t)block * NW + wave;
    const int64_t n0 = id / a.k_chunks * rows_wave;
    const int k0 = (int)(id % a.k_chunks) * per_row;
    if (n0 >= a.B) return;  // whole wave; no block-wide barrier follows

    if (lane < items) {
        const int64_t n = n0 + (lane >> a.log_per_row);
        const int k = k0 + (lane & (per_row - 1));
        int64_t off = 0;
        float4 wt = make_float4(0.f, 0.f, 0.f, 0.f);
        if (k < a.K && n < a.B) {
            const float2 xv = input_pair(a, n, k);
            float4 c1, c2;
            const int i1 = locate_cell(s_grid, a.W - 1, xv.x, c1), i2 = locate_cell(s_grid, a.W - 1, xv.y, c2);
            wt = make_float4((xv.x - c1.z) * c1.w, (xv.y - c2.z) * c2.w, c1.w, c2.w);
            off = (int64_t)(i1 * a.W + i2) * a.map.s_node + (int64_t)k * a.map.s_pair;
        }
        sh.w[wave][lane] = wt;
        sh.off[wave][lane] = off;
    }
    wave_lds_fence();

    const int64_t d01 = a.map.s_node, d10 = (int64_t)a.W * a.map.s_node;
    for (int e = slot; e < items; e += NS) {
        const int64_t n = n0 + (e >> a.log_per_row);
        const int k = k0 + (e & (per_row - 1));
        const bool on = n < a.B && k < a.K;
        const float4 wt = sh.w[wave][e];
        float d1 = 0.f, d2 = 0.f;
        if (on) {
            const CT *row = static_cast<const CT *>(a.P) + sh.off[wave][e];
            const int64_t elems = a.B * a.n_out;
            float da = 0.f, db = 0.f, dc = 0.f, dd = 0.f;  // P10-P00, P11-P01, P01-P00, P11-P10
#pragma unroll 3 - Q
            for (int base = 0; base < a.n_out; base += 4 * Q * LPR) {
                const int col[2] = {base + Columns<CT, LPR, Q>::first(cl), base + Columns<CT, LPR, Q>::second(cl)};
                // (a quad past the outputs reads the first columns again and counts as zero)
                const int64_t at0 = col[0] < a.n_out ? column_offset(a, col[0]) : 0;
                const int64_t step = col[1] < a.col_limit ? column_offset(a, col[1]) - at0 : 0;
                const CT *p = row + at0;
                Row<CT, Q> r00, r01, r10, r11;
                r00.load(p, step);
                r01.load(p + d01, step);
                r10.load(p + d10, step);
                r11.load(p + d10 + d01, step);
                float g[4 * Q];
#pragma unroll
                for (int h = 0; h < Q; ++h) {
                    const float4 gv = load_row4(a.gy, n, col[h] < a.n_out ? col[h] : 0, a.n_out, elems);
                    g[4 * h] = col[h] < a.n_out ? gv.x : 0.f;
                    g[4 * h + 1] = col[h] + 1 < a.n_out ? gv.y : 0.f;
                    g[4 * h + 2] = col[h] + 2 < a.n_out ? gv.z : 0.f;
                    g[4 * h + 3] = col[h] + 3 < a.n_out ? gv.w : 0.f;
                }
                float c00[4 * Q], c01[4 * Q], c10[4 * Q], c11[4 * Q];
                r00.widen(c00);
                r01.widen(c01);
                r10.widen(c10);
                r11.widen(c11);
#pragma unroll
                for (int i = 0; i < 4 * Q; ++i) {
                    da = fmaf(g[i], c10[i] - c00[i], da);
                    db = fmaf(g[i], c11[i] - c01[i], db);
                    dc = fmaf(g[i], c01[i] - c00[i], dc);
                    dd = fmaf(g[i], c11[i] - c10[i], dd);
                }
            }
            d1 = wt.z * (da * (1.f - wt.y) + db * wt.y);
            d2 = wt.w * (dc * (1.f - wt.x) + dd * wt.x);
        }
#pragma unroll
        for (int m = 1; m < LPR; m <<= 1) {
            d1 += __shfl_xor(d1, m, 64);
            d2 += __shfl_xor(d2, m, 64);
        }
        if (on && cl == 0) {
            if (a.conv) {
                int64_t first, second;
                pair_offsets(a, k, first, second);
                float *w = a.out + window_start(a.cg, n);
                if (a.overlap) {
                    atomicAdd(w + first, d1);
                    atomicAdd(w + second, d2);
                } else {
                    w[first] = d1;
                    w[second] = d2;
                }
            } else {
                *reinterpret_cast<float2 *>(a.out + n * a.n_in + 2 * k) = make_float2(d1, d2);
            }
        }
    }
}

template <typename CT, int LPR, int Q>
__global__ __launch_bounds__(256) void backward_input_gather_kernel(GatherArgs a)
{
    __shared__ float4 s_grid[LMKAN_MAX_GRID];
    __shared__ InputShared<4> sh;
    stage_intervals(a.tab, s_grid);
    __syncthreads();
    input_gather<CT, LPR, Q, 4>(a, blockIdx.x, s_grid, sh);
}

// ---------------------------------------------------------------------------
// Coefficient gradient.  A workgroup takes a pair, 4 Q LPR outputs and a share of the table's nodes.  It
// sorts the samples of the batch by cell in LDS, then every group of LPR lanes takes nodes one
// after the other and sums, over the samples of the (up to) four cells around the node, the node's
// weight times gy.  Every entry of the gradient is written once, zeros included: no zero fill, no
// atomics.  A sample is gathered four times, by the four corners of its cell, and sorted anew for
// every tile, which is what limits this kernel to small batches.
// The counting sort keeps a population per (wave, cell): a sample's rank is what the wave's counter
// held before it, so the order inside a cell follows waves, steps and lanes and does not depend on which
// wave happens to run first: the sums are the same in every run.
// ---------------------------------------------------------------------------
constexpr int kCoefThreads = 512;
constexpr int kCoefWaves = kCoefThreads / 64;
constexpr int kCoefPerFew = 2, kCoefPerMost = 16;  // samples of a thread
constexpr int kCoefMaxBatch = kCoefThreads * kCoefPerMost;

template <int LPR, int Q, int kCoefPer>
__device__ __forceinline__ void coef_gather(const GatherArgs &a, int block, float4 *s_grid, int *s_wave, char *gather_smem)
{
    const int G = a.W - 1, cells = G * G, B = (int)a.B;
    float2 *s_uv = reinterpret_cast<float2 *>(gather_smem);  // [B], by position
    int *s_row = reinterpret_cast<int *>(s_uv + B);          // [B], by position: the sample
    int *s_start = s_row + B;                                // [cells + 1]
    const int even = (cells + 1) & ~1;
    unsigned short *s_off = reinterpret_cast<unsigned short *>(s_start + cells + 1);  // [waves][even]
    int *s_count = reinterpret_cast<int *>(s_off);           // the same memory, two counters to a word
    const int tid = threadIdx.x, wave = tid >> 6;

    const int ct = block % a.coef_ct, k = block / a.coef_ct % a.K, part = block / a.coef_ct / a.K;
    float2 xv[kCoefPer];
    int64_t first, second;
    pair_offsets(a, k, first, second);
#pragma unroll
    for (int j = 0; j < kCoefPer; ++j) {
        const int n = tid + j * kCoefThreads;
        xv[j] = n < B ? input_pair(a, n, first, second) : make_float2(0.f, 0.f);
    }
    stage_intervals(a.tab, s_grid);
    for (int c = tid; c < kCoefWaves * even / 2; c += kCoefThreads) s_count[c] = 0;
    __syncthreads();
    int cell[kCoefPer], rank[kCoefPer];
    float2 uv[kCoefPer];
#pragma unroll
    for (int j = 0; j < kCoefPer; ++j) {
        if (tid + j * kCoefThreads < B) {
            float4 c1, c2;
            const int i1 = locate_cell(s_grid, G, xv[j].x, c1), i2 = locate_cell(s_grid, G, xv[j].y, c2);
            uv[j] = make_float2((xv[j].x - c1.z) * c1.w, (xv[j].y - c2.z) * c2.w);
            cell[j] = i1 * G + i2;
            rank[j] = count_in_order(s_count, wave * even + cell[j], cell[j], cells > 256);
        }
    }
    __syncthreads();
    // populations -> first positions: a run of consecutive cells per thread
    {
        const int per = (cells + kCoefThreads - 1) / kCoefThreads;
        const int c0 = min(cells, tid * per), c1 = min(cells, c0 + per);
        int mine = 0;
        for (int c = c0; c < c1; ++c)
#pragma unroll
            for (int w = 0; w < kCoefWaves; ++w) mine += s_off[w * even + c];
        int incl = mine;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const int t = __shfl_up(incl, d, 64);
            if ((tid & 63) >= d) incl += t;
        }
        if ((tid & 63) == 63) s_wave[wave] = incl;
        __syncthreads();
        int run = incl - mine;
        for (int w = 0; w < wave; ++w) run += s_wave[w];
        for (int c = c0; c < c1; ++c) {
            s_start[c] = run;
#pragma unroll
            for (int w = 0; w < kCoefWaves; ++w) {
                const int count = s_off[w * even + c];
                s_off[w * even + c] = (unsigned short)run;
                run += count;
            }
        }
        if (tid == 0) s_start[cells] = B;
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < kCoefPer; ++j) {
        if (tid + j * kCoefThreads < B) {
            const int pos = s_off[wave * even + cell[j]] + rank[j];
            s_uv[pos] = uv[j];
            s_row[pos] = tid + j * kCoefThreads;
        }
    }
    __syncthreads();

    // groups of LPR lanes: a.spn of them (in one wave) share the samples of a node
    const int per_node = LPR * a.spn, groups = kCoefThreads / per_node;
    const int cl = tid % LPR, share = (tid / LPR) % a.spn;
    const int base = ct * (4 * Q * LPR);
    const int nodes = a.W * a.W;
    const int64_t elems = a.B * a.n_out;
    for (int node = part * groups + tid / per_node; node < nodes; node += a.parts * groups) {
        const int i1 = node / a.W, i2 = node - i1 * a.W;
        float acc[4 * Q] = {};
#pragma unroll
        for (int side = 0; side < 2; ++side) {  // the cells below the node along the first axis, and those above
            const int r = i1 - 1 + side;
            if (r < 0 || r >= G) continue;
            const int mid = s_start[r * G + i2];                      // cells (r, i2 - 1) and (r, i2) are neighbours
            const int begin = i2 > 0 ? s_start[r * G + i2 - 1] : mid;
            const int end = i2 < G ? s_start[r * G + i2 + 1] : mid;
#pragma unroll 4
            for (int p = begin + share; p < end; p += a.spn) {
                const float2 at = s_uv[p];
                const float w = (side == 0 ? at.x : 1.f - at.x) * (p < mid ? at.y : 1.f - at.y);
                // (lanes past n_out repeat the first columns; what they sum is dropped)
                Row<float, Q> g;
#pragma unroll
                for (int h = 0; h < Q; ++h) {
                    const int col = base + cl * 4 + h * 4 * LPR;
                    g.v[h] = load_row4(a.gy, s_row[p], col < a.n_out ? col : 0, a.n_out, elems);
                }
                add_row<float, Q>(acc, w, g);
            }
        }
        for (int m = LPR; m < LPR * a.spn; m <<= 1)
#pragma unroll
            for (int i = 0; i < 4 * Q; ++i) acc[i] += __shfl_xor(acc[i], m, 64);
        if (share != 0) continue;
        float *dst = a.gcoef + ((int64_t)node * a.K + k) * a.n_out;
#pragma unroll
        for (int h = 0; h < Q; ++h) {
            const int col = base + cl * 4 + h * 4 * LPR;
            if (col >= a.n_out) continue;
            if (a.accumulate) {
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if (col + i < a.n_out) dst[col + i] += acc[4 * h + i];
            } else {
                store_outputs(dst + col, acc + 4 * h, a.n_out, col, false);
            }
        }
    }
}

template <int LPR, int Q, int kCoefPer>
__global__ __launch_bounds__(kCoefThreads) void backward_coef_gather_kernel(GatherArgs a)
{
    extern __shared__ __align__(16) char gather_smem[];
    __shared__ float4 s_grid[LMKAN_MAX_GRID];
    __shared__ int s_wave[kCoefWaves];
    coef_gather<LPR, Q, kCoefPer>(a, blockIdx.x, s_grid, s_wave, gather_smem);
}

// Both gradients of a small batch in one launch: each waits for its own loads most of the time (5 us for
// the input gradient, 9 for the coefficient gradient of 256 rows of 16 -> 16), and side by side they
// take as long as the longer one.
template <typename CT, int LPRX, int QX, int LPRP, int QP>
__global__ __launch_bounds__(kCoefThreads) void backward_gather_kernel(GatherArgs a)
{
    extern __shared__ __align__(16) char gather_smem[];
    __shared__ float4 s_grid[LMKAN_MAX_GRID];
    __shared__ int s_wave[kCoefWaves];
    __shared__ InputShared<kCoefWaves> sh;
    if ((int)blockIdx.x < a.coef_blocks) {
        coef_gather<LPRP, QP, kCoefPerFew>(a, blockIdx.x, s_grid, s_wave, gather_smem);
    } else {
        stage_intervals(a.tab, s_grid);
        __syncthreads();
        input_gather<CT, LPRX, QX, kCoefWaves>(a, blockIdx.x - a.coef_blocks, s_grid, sh);
    }
}

// lanes per row, `per_lane` outputs each: as many as the outputs fill, up to sixteen
constexpr int lanes_for(int n_out, int per_lane)
{
    int lpr = 1;
    while (lpr < 16 && lpr * per_lane < n_out) lpr *= 2;
    return lpr;
}

int forward_per_lane(const LayerShape &s) { return s.dtype == LMKAN_F32 ? 4 : 8; }

// eight outputs per lane, so that fewer lanes have to meet at the end of an item; float32 rows of up to 4
// outputs, and of more than 64 (one load per corner and step, two steps in flight): four
constexpr int input_per_lane(bool f32, int n_out) { return f32 && (n_out <= 4 || n_out > 64) ? 4 : 8; }
int backward_input_per_lane(const LayerShape &s) { return input_per_lane(s.dtype == LMKAN_F32, s.n_out); }

// wide layers: tiles of 128 outputs (every tile sorts the batch for itself)
constexpr int coef_per_lane(int n_out) { return n_out > 128 ? 8 : 4; }
int backward_coef_per_lane(const LayerShape &s) { return coef_per_lane(s.n_out); }

int log2_of(int power) { return __builtin_ctz((unsigned)power); }

GatherArgs gather_args(const LayerShape &s, const GridTab &tab, const float *x, const void *coef, const ConvGeom *conv)
{
    GatherArgs a = {};
    a.P = coef;
    a.x = x;
    a.map = coef_map(s);
    a.tab = tab;
    a.B = s.batch;
    a.n_in = s.n_in;
    a.n_out = s.n_out;
    a.K = s.pairs();
    a.W = s.G + 1;
    a.col_limit = s.layout == LMKAN_LAYOUT_PACKED ? s.out_tiles() * LMKAN_PACK_TILE : s.n_out;
    a.conv = conv != nullptr;
    if (conv) a.cg = *conv;
    return a;
}

typedef void (*GatherKernel)(GatherArgs);

template <typename CT, int Q, int NW>
GatherKernel forward_for(int lpr)
{
    switch (lpr) {
    case 1: return forward_gather_kernel<CT, 1, Q, NW>;
    case 2: return forward_gather_kernel<CT, 2, Q, NW>;
    case 4: return forward_gather_kernel<CT, 4, Q, NW>;
    case 8: return forward_gather_kernel<CT, 8, Q, NW>;
    default: return forward_gather_kernel<CT, 16, Q, NW>;
    }
}

template <typename CT, int Q>
GatherKernel backward_input_for(int lpr)
{
    switch (lpr) {
    case 1: return backward_input_gather_kernel<CT, 1, Q>;
    case 2: return backward_input_gather_kernel<CT, 2, Q>;
    case 4: return backward_input_gather_kernel<CT, 4, Q>;
    case 8: return backward_input_gather_kernel<CT, 8, Q>;
    default: return backward_input_gather_kernel<CT, 16, Q>;
    }
}

template <int Q, int PER>
GatherKernel backward_coef_for(int lpr)
{
    switch (lpr) {
    case 1: return backward_coef_gather_kernel<1, Q, PER>;
    case 2: return backward_coef_gather_kernel<2, Q, PER>;
    case 4: return backward_coef_gather_kernel<4, Q, PER>;
    case 8: return backward_coef_gather_kernel<8, Q, PER>;
    default: return backward_coef_gather_kernel<16, Q, PER>;
    }
}

// The kernel for both gradients, with the lanes and outputs per lane of the kernels for one: they change at
// these output counts only.
struct BothGradients {
    GatherKernel kernel;
    int input_lanes, input_per, coef_lanes, coef_per;
};

template <typename CT, int N_OUT>
BothGradients backward_at()
{
    constexpr int px = input_per_lane(sizeof(CT) == 4, N_OUT), pp = coef_per_lane(N_OUT);
    constexpr int lx = lanes_for(N_OUT, px), lp = lanes_for(N_OUT, pp);
    return {backward_gather_kernel<CT, lx, px / 4, lp, pp / 4>, lx, px, lp, pp};
}

template <typename CT>
BothGradients backward_for(int n_out)
{
    return n_out <= 4    ? backward_at<CT, 4>()
           : n_out <= 8  ? backward_at<CT, 8>()
           : n_out <= 16 ? backward_at<CT, 16>()
           : n_out <= 32 ? backward_at<CT, 32>()
           : n_out <= 64 ? backward_at<CT, 64>()
           : n_out <= 128 ? backward_at<CT, 128>()
                          : backward_at<CT, LMKAN_MAX_N_OUT>();
}

size_t coef_gather_lds(const LayerShape &s)
{
    const size_t B = (size_t)s.batch, cells = (size_t)s.G * s.G;
    return B * (sizeof(float2) + sizeof(int)) + (cells + 1) * sizeof(int) +
           kCoefWaves * ((cells + 1) & ~(size_t)1) * sizeof(unsigned short);
}

}  // namespace

void launch_forward_gather(const LayerShape &s, const GridTab &tab, const float *x, const void *coef, float *y,
                           hipStream_t stream, const ConvGeom *conv)
{
    GatherArgs a = gather_args(s, tab, x, coef, conv);
    a.out = y;
    const int per_lane = forward_per_lane(s);
    int lpr = lanes_for(s.n_out, per_lane);
    // Few rows: narrower row pieces (not under 64 bytes) put more CUs to work on a row.
    while (lpr > 4 && s.batch * ((s.n_out + per_lane * lpr - 1) / (per_lane * lpr)) < 128) lpr /= 2;
    a.n_ct = (s.n_out + per_lane * lpr - 1) / (per_lane * lpr);
    const int ns = 64 / lpr;
    // Slots per row: at least so many that the items a wave locates at once hold 16 pairs of a row (128
    // contiguous bytes of x), and until the launch has 4096 waves, as long as a slot keeps four
    // pairs.
    int spr = 1;
    const int64_t rows = s.batch * a.n_ct;
    while (spr < ns && lpr * spr < 16 && lpr * spr < a.K) spr *= 2;
    while (spr < 16 * ns && rows * spr < (int64_t)4096 * ns && a.K >= 8 * spr) spr *= 2;
    const int spw = spr < ns ? spr : ns, wpr = spr / spw;
    const int nw = wpr > 4 ? 16 : 4;
    int per_row = lpr * spw;
    // fewer pairs than that: all of a row in one chunk, and more rows per wave
    while (wpr == 1 && per_row / 2 >= a.K && per_row / 2 >= spw) per_row /= 2;
    a.log_spw = log2_of(spw);
    a.log_wpr = log2_of(wpr);
    a.log_per_row = log2_of(per_row);
    const int64_t rows_block = (int64_t)(nw / wpr) * (64 / per_row);
    a.groups = (s.batch + rows_block - 1) / rows_block;
    // a workgroup goes on to further rows once the chip is full (eight waves per SIMD)
    const int64_t most = 256 * 32 / nw / a.n_ct > 0 ? 256 * 32 / nw / a.n_ct : 1;
    const unsigned grid = (unsigned)((a.groups < most ? a.groups : most) * a.n_ct);
    GatherKernel kernel;
    if (s.dtype == LMKAN_F32)
        kernel = nw == 4 ? forward_for<float, 1, 4>(lpr) : forward_for<float, 1, 16>(lpr);
    else if (s.dtype == LMKAN_F16)
        kernel = nw == 4 ? forward_for<_Float16, 2, 4>(lpr) : forward_for<_Float16, 2, 16>(lpr);
    else
        kernel = nw == 4 ? forward_for<bf16_t, 2, 4>(lpr) : forward_for<bf16_t, 2, 16>(lpr);
    KernelTiming timing(stream, kTimeForward);
    kernel<<<grid, nw * 64, 0, stream>>>(a);
}

// the input gradient's share of the arguments; returns its waves
static int64_t set_input_args(GatherArgs &a, const LayerShape &s, const float *gy, float *gx, const ConvGeom *conv, int lpr,
                              hipStream_t stream)
{
    a.gy = gy;
    a.out = gx;
    // items per wave: 64, fewer (down to one per slot) until the launch has 2048 waves
    a.items = 64;
    while (a.items > 64 / lpr && s.batch * a.K < (int64_t)2048 * a.items) a.items /= 2;
    int per_row = 1;
    while (per_row < a.K && per_row < a.items) per_row *= 2;
    a.log_per_row = log2_of(per_row);
    a.k_chunks = (a.K + per_row - 1) / per_row;
    if (conv) {
        // windows that overlap add into the image; elements no window holds are zero
        const ConvGeom &g = *conv;
        a.overlap = g.stride < g.kh || g.stride < g.kw;
        const bool covered = g.stride == g.kh && g.stride == g.kw && g.OH * g.kh == g.H && g.OW * g.kw == g.W;
        if (!covered) launch_fill_zero(gx, (size_t)g.N * g.H * g.W * g.C, stream);
    }
    return (s.batch + a.items / per_row - 1) / (a.items / per_row) * a.k_chunks;
}

// the coefficient gradient's share; returns its workgroups
static int64_t set_coef_args(GatherArgs &a, const LayerShape &s, const float *gy, float *gcoef, bool accumulate, int lpr,
                             int per_lane)
{
    a.gy = gy;
    a.gcoef = gcoef;
    a.accumulate = accumulate ? 1 : 0;
    a.coef_ct = (s.n_out + per_lane * lpr - 1) / (per_lane * lpr);
    // workgroups that share the nodes of a (pair, tile): each sorts the samples for itself
    const int64_t tiles = (int64_t)a.K * a.coef_ct;
    a.parts = 1;
    while (a.parts < 16 && tiles * a.parts < 512 && s.nodes() * lpr > 2 * a.parts * kCoefThreads) a.parts *= 2;
    // and the lanes of a node's samples, while the nodes leave lanes idle
    a.spn = 1;
    while (a.spn < 64 / lpr && (int64_t)s.nodes() * lpr * a.spn < (int64_t)2 * a.parts * kCoefThreads) a.spn *= 2;
    return tiles * a.parts;
}

void launch_backward_input_gather(const LayerShape &s, const GridTab &tab, const float *x, const void *coef,
                                  const float *gy, float *gx, hipStream_t stream, const ConvGeom *conv)
{
    GatherArgs a = gather_args(s, tab, x, coef, conv);
    const int per_lane = backward_input_per_lane(s), lpr = lanes_for(s.n_out, per_lane);
    const int64_t waves = set_input_args(a, s, gy, gx, conv, lpr, stream);
    const GatherKernel kernel = s.dtype == LMKAN_F32 ? (per_lane == 4 ? backward_input_for<float, 1>(lpr) : backward_input_for<float, 2>(lpr))
                                : s.dtype == LMKAN_F16 ? backward_input_for<_Float16, 2>(lpr)
                                                       : backward_input_for<bf16_t, 2>(lpr);
    KernelTiming timing(stream, kTimeGradInput);
    kernel<<<(unsigned)((waves + 3) / 4), 256, 0, stream>>>(a);
}

void launch_backward_coef_gather(const LayerShape &s, const GridTab &tab, const float *x, const float *gy, float *gcoef,
                                 bool accumulate, hipStream_t stream, const ConvGeom *conv)
{
    GatherArgs a = gather_args(s, tab, x, nullptr, conv);
    const int per_lane = backward_coef_per_lane(s), lpr = lanes_for(s.n_out, per_lane);
    const int64_t blocks = set_coef_args(a, s, gy, gcoef, accumulate, lpr, per_lane);
    const size_t lds = coef_gather_lds(s);
    const bool few = s.batch <= kCoefPerFew * kCoefThreads;
    const GatherKernel kernel =
        per_lane == 4 ? (few ? backward_coef_for<1, kCoefPerFew>(lpr) : backward_coef_for<1, kCoefPerMost>(lpr))
                      : (few ? backward_coef_gather_kernel<16, 2, kCoefPerFew> : backward_coef_gather_kernel<16, 2, kCoefPerMost>);
    if (lds > 60 * 1024) allow_large_lds(reinterpret_cast<const void *>(kernel), 155 * 1024);
    KernelTiming timing(stream, kTimeGradCoef);
    kernel<<<(unsigned)blocks, kCoefThreads, lds, stream>>>(a);
}

// (the LDS of the sort is allocated for the input gradient's workgroups too: only while it leaves room for
// several of them on a CU)
bool backward_gather_shape_ok(const LayerShape &s)
{
    return backward_input_gather_shape_ok(s) && backward_coef_gather_shape_ok(s) &&
           s.batch <= kCoefPerFew * kCoefThreads && coef_gather_lds(s) <= 20 * 1024;
}

void launch_backward_gather(const LayerShape &s, const GridTab &tab, const float *x, const void *coef, const float *gy,
                            float *gx, float *gcoef, bool accumulate, hipStream_t stream, const ConvGeom *conv)
{
    GatherArgs a = gather_args(s, tab, x, coef, conv);
    const BothGradients both = s.dtype == LMKAN_F32   ? backward_for<float>(s.n_out)
                               : s.dtype == LMKAN_F16 ? backward_for<_Float16>(s.n_out)
                                                      : backward_for<bf16_t>(s.n_out);
    const int64_t waves = set_input_args(a, s, gy, gx, conv, both.input_lanes, stream);
    a.coef_blocks = (int)set_coef_args(a, s, gy, gcoef, accumulate, both.coef_lanes, both.coef_per);
    const unsigned grid = (unsigned)(a.coef_blocks + (waves + kCoefWaves - 1) / kCoefWaves);
    KernelTiming timing(stream, kTimeGradInput);
    both.kernel<<<grid, kCoefThreads, coef_gather_lds(s), stream>>>(a);
}

// rows of the table are read 16 bytes at a time
static bool rows_by_16_bytes(const LayerShape &s)
{
    return s.layout == LMKAN_LAYOUT_PACKED || s.n_out % (s.dtype == LMKAN_F32 ? 4 : 8) == 0;
}

// Where the gathers win.  The rules compare a fitted time of the gathering kernel with one of the
// kernels it would replace (microseconds).  The fits are good to a third, so a gather has to promise 15 %
// less.  Over 500 random layers (4 ... 1024 inputs, 2 ... 1024 outputs, 1 ... 200000 rows, grids of 4 to 40, all
// table types) the choice takes 0.6 % longer than the better of the two for the forward pass, 0.8 % for
// grad_x, 8 % for grad_coef (it sorts sparse cells that a gather takes a fourth of the time for); gathering
// always 7, 7 and 8 %, never three times as long.
constexpr double kPromise = 0.85;

static double table_bytes(const LayerShape &s)
{
    return (double)s.nodes() * s.pairs() * s.out_tiles() * LMKAN_PACK_TILE * (s.dtype == LMKAN_F32 ? 4 : 2);
}

// A row piece moves at least a line of `least_line` bytes, and the lanes of a tile load whether the row
// fills it or not.  Lines come at `rate` (bytes per microsecond) while the table sits in the L2s, slower
// the more of it is in the last-level cache, and at what HBM gives beyond that.
static double gather_us(const LayerShape &s, int tile, double least_line, double rate, double falls)
{
    const double item = s.dtype == LMKAN_F32 ? 4 : 2, table = table_bytes(s);
    double line = fmax((s.n_out + 3) / 4 * 4 * item, least_line);
    const double loaded = (s.n_out + tile - 1) / tile * tile * item;
    if (loaded > line) line = (line + loaded) / 2;
    rate = table <= 256e6 ? fmin(rate, fmax(7e6, rate * pow(4e6 / table, falls))) : 5.5e6;
    return 4 + (double)s.batch * s.pairs() * 4 * line / rate;
}

// The slab kernels with the passes around them: what little work takes, the rate of the tile that the
// grid leaves room for (outputs per microsecond), and never less than the table takes from HBM.
static double slab_us(const LayerShape &s, double least, double wide, double half, double fine)
{
    const double rows = (double)s.batch * s.pairs();
    const double work = s.G <= 16 ? rows * ((s.n_out + 63) / 64 * 64) / wide
                                  : rows * ((s.n_out + 31) / 32 * 32) / (s.G <= 34 ? half : fine);
    return fmax(least + work, table_bytes(s) / 4.8e6);
}

bool forward_gather_shape_ok(const LayerShape &s)
{
    // (no slab fits from G = 50 on, and one just does at G = 49, where the two are not weighed; the kernel for few outputs, which
    // takes them beyond G = 34, is three times slower however many rows there are)
    if (!rows_by_16_bytes(s)) return false;
    if (s.G > 48 || (s.n_out > 1 && small_out_shape_ok(s))) return true;
    const int per_lane = forward_per_lane(s), tile = lanes_for(s.n_out, per_lane) * per_lane;
    return gather_us(s, tile, 128, 27e6, 0.25) < kPromise * slab_us(s, 26, 3e6, 2.8e6, 1.8e6);
}

// One output on rows: against the kernel that keeps the pairs' columns of the table in LDS.  A workgroup of it
// fetches a line per node and pair first, which the gathers save while there are few rows; from then on it
// does a pair in a third to a fourth of the time.  (Fitted to 250 random layers of 4 ... 512 pairs, 1 ... 130000
// rows, G of 4 to 30, packed tables, to 30 %.  The choice takes 1.4 % longer than the better of the two,
// at most 7 % longer than the kernel with the columns in LDS; gathering always takes 9 % longer, up to
// 4.4 times as long, and never gathering 81 % longer.)
bool forward_gather_beats_head(const LayerShape &s)
{
    const int chunk = head_pairs_per_chunk(s);
    const double items = (double)s.batch * s.pairs(), lines = (double)chunk * s.nodes();
    const double head = 6.4 + lines / 1480 + 3.3 * ((s.pairs() + chunk - 1) / chunk - 1) + items / 227e3 + items * lines / 5.9e9;
    return gather_us(s, forward_per_lane(s), 128, 27e6, 0.25) < kPromise * head;
}

bool backward_input_gather_shape_ok(const LayerShape &s)
{
    if (!rows_by_16_bytes(s)) return false;
    if (s.n_out > 1 && small_out_shape_ok(s)) return true;
    const int per_lane = backward_input_per_lane(s), tile = lanes_for(s.n_out, per_lane) * per_lane;
    return gather_us(s, tile, 64, 20e6, 0.33) < kPromise * slab_us(s, 38, 3e6, 2.8e6, 1.4e6);
}

// A workgroup sorts the whole batch, every sample is gathered four times (one after the other where
// cells are dense), the gradient is written once; against the sorted stream, whose cost per cell shows on
// sparse tables, more so while few (pair, tile) streams share the chip and meet through atomics.
bool backward_coef_gather_shape_ok(const LayerShape &s)
{
    if (s.batch > kCoefMaxBatch || coef_gather_lds(s) > 155 * 1024) return false;
    const double work = (double)s.batch * s.pairs() * ((s.n_out + 3) / 4 * 4), dense = (double)s.batch / (s.G * s.G);
    const double table = (double)s.nodes() * s.pairs() * s.n_out * 4;
    return 6 + s.batch / 150.0 + 0.2 * dense + work / 1.4e6 + table / 5e6 <
           kPromise * (25 + fmin(table / 1e6, 40 + table / 5e6) + work / 5e6);
}

// (y, gy and the gradient are accessed through 16-byte operations that need 4-byte alignment only)
bool gather_table_aligned(const void *coef) { return (reinterpret_cast<uintptr_t>(coef) & 15) == 0; }

}  // namespace lmkan
