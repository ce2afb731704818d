// Layers with very few outputs: a single output (regression heads), and up to eight outputs where
// the slab kernels do not apply (batches under 256 rows, grids finer than 34 intervals, tables in
// the layout of Alg. 1 whose output count is not a multiple of four).  From two outputs on the
// slab kernels are faster even with most of their 64-output tile empty (256 -> 8, 65536 rows:
// 0.44 ms for both gradients against 2.0 ms here; 256 -> 1: 0.46 against 0.37).
//
// With so few outputs the lanes cannot be outputs: here a lane is a sample and walks over the
// pairs, the preamble records (cell, local coordinates) arriving coalesced along the sample
// axis.  The table of such a layer is small ((G+1)^2 K n_out values) and is gathered from L2.
//   forward:        y[n][j] accumulated in registers over the pairs
//   input gradient: both derivatives of a (sample, pair) come from one lane, written once
//                   into the transposed scratch [n_in][B] (no atomics, no zero fill)
//   coefficient gradient: a workgroup owns a range of pairs whose table slice fits LDS, adds
//                   its samples into that slice with LDS atomics and then adds the slice into
//                   the zero-filled gradient (float32 atomics)
#include <algorithm>

#include "lmkan_kernels.h"

namespace lmkan {

namespace {

constexpr int kSmallMax = kSmallMaxOut;
constexpr int kThreads = 256;

struct SmallArgs {
    const void *P;
    CoefMap map;
    const int32_t *rec_node;
    const float *rec_u;
    const float *rec_v;
    const float *gy;
    float *y;
    float *gx_t;   // transposed scratch [n_in][B]
    float *gP;     // layout of Alg. 1, float32
    GridTab tab;
    int64_t B;
    int n_out;
    int K;
    int W;
    int pairs_per_block;
    int atomic_out;
};

template <typename CT>
__global__ __launch_bounds__(kThreads) void forward_small_kernel(SmallArgs a)
{
    const int64_t n = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    const int k0 = blockIdx.y * a.pairs_per_block;
    const int k1 = min(a.K, k0 + a.pairs_per_block);
    if (n >= a.B) return;
    const CT *P = static_cast<const CT *>(a.P);
    const int64_t d_i1 = (int64_t)a.W * a.map.s_node, d_i2 = a.map.s_node;
    float acc[kSmallMax];
#pragma unroll
    for (int j = 0; j < kSmallMax; ++j) acc[j] = 0.f;
    for (int k = k0; k < k1; ++k) {
        const int64_t o = (int64_t)k * a.B + n;
        const int node = a.rec_node[o];
        const float u = a.rec_u[o], v = a.rec_v[o];
        const float a_lo = 1.0f - u, b_lo = 1.0f - v;
        const float w00 = a_lo * b_lo, w10 = u * b_lo, w01 = a_lo * v, w11 = u * v;
        const CT *row = P + (int64_t)node * a.map.s_node + (int64_t)k * a.map.s_pair;
#pragma unroll
        for (int j = 0; j < kSmallMax; ++j) {
            if (j < a.n_out) {
                acc[j] = fmaf(w00, widen(row[j]), acc[j]);
                acc[j] = fmaf(w10, widen(row[d_i1 + j]), acc[j]);
                acc[j] = fmaf(w01, widen(row[d_i2 + j]), acc[j]);
                acc[j] = fmaf(w11, widen(row[d_i1 + d_i2 + j]), acc[j]);
            }
        }
    }
    float *dst = a.y + n * a.n_out;
#pragma unroll
    for (int j = 0; j < kSmallMax; ++j) {
        if (j < a.n_out) {
            if (a.atomic_out)
                unsafeAtomicAdd(dst + j, acc[j]);
            else
                dst[j] = acc[j];
        }
    }
}

template <typename CT>
__global__ __launch_bounds__(kThreads) void backward_input_small_kernel(SmallArgs a)
{
    __shared__ float s_invh[LMKAN_MAX_GRID];
    for (int i = threadIdx.x; i < a.tab.G; i += blockDim.x) s_invh[i] = a.tab.inv_h[i];
    __syncthreads();
    const int64_t n = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    const int k0 = blockIdx.y * a.pairs_per_block;
    const int k1 = min(a.K, k0 + a.pairs_per_block);
    if (n >= a.B) return;
    const CT *P = static_cast<const CT *>(a.P);
    const int64_t d_i1 = (int64_t)a.W * a.map.s_node, d_i2 = a.map.s_node;
    float g[kSmallMax];
#pragma unroll
    for (int j = 0; j < kSmallMax; ++j) g[j] = j < a.n_out ? a.gy[n * a.n_out + j] : 0.f;
    for (int k = k0; k < k1; ++k) {
        const int64_t o = (int64_t)k * a.B + n;
        const int node = a.rec_node[o];
        const float u = a.rec_u[o], v = a.rec_v[o];
        const CT *row = P + (int64_t)node * a.map.s_node + (int64_t)k * a.map.s_pair;
        float s00 = 0.f, s10 = 0.f, s01 = 0.f, s11 = 0.f;
#pragma unroll
        for (int j = 0; j < kSmallMax; ++j) {
            if (j < a.n_out) {
                s00 = fmaf(g[j], widen(row[j]), s00);
                s10 = fmaf(g[j], widen(row[d_i1 + j]), s10);
                s01 = fmaf(g[j], widen(row[d_i2 + j]), s01);
                s11 = fmaf(g[j], widen(row[d_i1 + d_i2 + j]), s11);
            }
        }
        const int i1 = node / a.W, i2 = node - i1 * a.W;
        const float d1 = s_invh[i1] * ((s10 - s00) * (1.0f - v) + (s11 - s01) * v);
        const float d2 = s_invh[i2] * ((s01 - s00) * (1.0f - u) + (s11 - s10) * u);
        a.gx_t[(int64_t)(2 * k) * a.B + n] = d1;
        a.gx_t[(int64_t)(2 * k + 1) * a.B + n] = d2;
    }
}

// blockIdx.y: range of pairs [k0, k1) whose slice [(G+1)^2][k1-k0][n_out] sits in LDS;
// blockIdx.x: the samples n = blockIdx.x * 256 + tid, stepping by gridDim.x * 256
__global__ __launch_bounds__(kThreads) void backward_coef_small_kernel(SmallArgs a)
{
    extern __shared__ float s_tab[];
    const int k0 = blockIdx.y * a.pairs_per_block;
    const int k1 = min(a.K, k0 + a.pairs_per_block);
    const int kc = k1 - k0;
    const int nodes = a.W * a.W;
    const int slice = nodes * kc * a.n_out;
    for (int i = threadIdx.x; i < slice; i += blockDim.x) s_tab[i] = 0.f;
    __syncthreads();
    const int row_stride = kc * a.n_out;  // one node of the slice
    for (int64_t n = (int64_t)blockIdx.x * kThreads + threadIdx.x; n < a.B; n += (int64_t)gridDim.x * kThreads) {
        float g[kSmallMax];
#pragma unroll
        for (int j = 0; j < kSmallMax; ++j) g[j] = j < a.n_out ? a.gy[n * a.n_out + j] : 0.f;
        for (int k = k0; k < k1; ++k) {
            const int64_t o = (int64_t)k * a.B + n;
            const int node = a.rec_node[o];
            const float u = a.rec_u[o], v = a.rec_v[o];
            const float a_lo = 1.0f - u, b_lo = 1.0f - v;
            const float w00 = a_lo * b_lo, w10 = u * b_lo, w01 = a_lo * v, w11 = u * v;
            float *p = s_tab + node * row_stride + (k - k0) * a.n_out;
#pragma unroll
            for (int j = 0; j < kSmallMax; ++j) {
                if (j < a.n_out) {
                    atomicAdd(p + j, w00 * g[j]);
                    atomicAdd(p + a.W * row_stride + j, w10 * g[j]);
                    atomicAdd(p + row_stride + j, w01 * g[j]);
                    atomicAdd(p + (a.W + 1) * row_stride + j, w11 * g[j]);
                }
            }
        }
    }
    __syncthreads();
    for (int i = threadIdx.x; i < slice; i += blockDim.x) {
        const float v = s_tab[i];
        if (v != 0.f) {
            const int node = i / row_stride, r = i - node * row_stride;
            const int k = k0 + r / a.n_out, j = r - (r / a.n_out) * a.n_out;
            unsafeAtomicAdd(a.gP + (int64_t)node * a.map.s_node + (int64_t)k * a.map.s_pair + j, v);
        }
    }
}

// ---------------------------------------------------------------------------
// One output (a regression head): y[n] = sum_k f_k(x[n][2k], x[n][2k+1]) (Eq. 2 with a single q),
// its input gradient and its coefficient gradient.  With one output the table of a pair is
// (G+1)^2 floats, so the tables of a chunk of pairs (or, for the coefficient gradient, their
// gradient) sit in LDS as float32, [pair][node] with an odd pitch.  A group of `lps` lanes (a
// power of two, up to the whole wave) takes a sample with a lane per pair, so the two inputs of
// its pairs are one contiguous read of the sample's row (and the two derivatives one contiguous
// write), and locates them itself (Alg. 1 "Preamble"): no records are written or read.
//   kHeadForward    the products of a sample meet in a sum over its lanes
//   kHeadGradInput  d/dx1 = gy (1/h1) ((P10 - P00)(1 - v) + (P11 - P01) v), d/dx2 likewise
// A wave has kHeadSamples such steps in flight and asks for the inputs of the next ones before it
// works on those it has.
// ---------------------------------------------------------------------------
enum HeadMode { kHeadForward = 0, kHeadGradInput = 1 };

struct HeadArgs {
    const void *P;
    CoefMap map;           // of P; for kHeadGradCoef of the gradient
    const float *x;
    const float *gy;       // [B] (one output)
    float *y;
    float *gx;             // [B][n_in]
    float *gP;             // float32, layout of Alg. 1
    float *partial;        // coefficient gradient: [workgroups along the samples][nodes][K], or NULL
    GridTab tab;
    int64_t B;
    int n_in;
    int K;
    int W;
    int nodes;
    int pitch;             // LDS floats per pair, odd
    int pairs_per_chunk;   // a multiple of 64 unless one chunk holds every pair
    int lps;               // lanes per sample
    int samples_per_block;
    int atomic_out;        // forward with several chunks: add into the zero-filled y
    int copies;            // coefficient gradient: LDS copies of the chunk's gradient, a power of two
};

constexpr int kHeadSamples = 2;  // steps a wave has in flight
constexpr int kHeadFill = 12;    // table elements a thread has in flight while LDS is filled
constexpr int kHeadThreads = 1024;

template <typename CT, int MODE>
__device__ __forceinline__ void head_body(const HeadArgs &a)
{
    extern __shared__ __align__(16) float head_smem[];
    const int k0 = blockIdx.y * a.pairs_per_chunk;
    const int kc = min(a.K, k0 + a.pairs_per_chunk) - k0;
    float *s_tab = head_smem;
    __shared__ float4 s_grid[LMKAN_MAX_GRID];
    stage_intervals(a.tab, s_grid);
    const int total = kc * a.nodes;
    // element i = node * kc + kl (pairs along the threads: contiguous in the layout of Alg. 1 with
    // one output); a thread's elements lie blockDim.x apart: (node, kl) advance by
    // (step_node, step_kl) with a carry, without a division per element
    const int step_node = (int)blockDim.x / kc, step_kl = (int)blockDim.x - step_node * kc;
    {
        // Every load is unconditional (the node clamped), so that kHeadFill of them are in flight
        // per thread.
        const CT *P = static_cast<const CT *>(a.P);
        int node = (int)threadIdx.x / kc, kl = (int)threadIdx.x - node * kc;
        for (int base = threadIdx.x; base < total; base += blockDim.x * kHeadFill) {
            CT raw[kHeadFill];
            int at[kHeadFill];
#pragma unroll
            for (int u = 0; u < kHeadFill; ++u) {
                const int node_rd = min(node, a.nodes - 1);   // past the end: the same pair of the last node again
                at[u] = kl * a.pitch + node_rd;
                raw[u] = P[(int64_t)node_rd * a.map.s_node + (int64_t)(k0 + kl) * a.map.s_pair];
                node += step_node;
                kl += step_kl;
                if (kl >= kc) {
                    kl -= kc;
                    ++node;
                }
            }
#pragma unroll
            for (int u = 0; u < kHeadFill; ++u) s_tab[at[u]] = widen(raw[u]);  // (a clamped one rewrites an element of the last node)
        }
    }
    __syncthreads();

    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6, waves = blockDim.x >> 6;
    const int per_step = 64 / a.lps;            // samples of a wave step
    const int sub = lane / a.lps, pl = lane - sub * a.lps;
    const int per_round = per_step * kHeadSamples;
    const int64_t n_begin = (int64_t)blockIdx.x * a.samples_per_block;
    const int64_t n_end = min(a.B, n_begin + a.samples_per_block);

    // inputs of (round starting at n, pairs kk ...): lanes past the chunk and samples past the block
    // repeat the last one, every load is in bounds and unconditional, what they yield is dropped
    auto request = [&](int64_t n, int kk, float2 (&xv)[kHeadSamples], float (&g)[kHeadSamples]) {
        const int kl = min(kk + pl, kc - 1);
#pragma unroll
        for (int s = 0; s < kHeadSamples; ++s) {
            const int64_t nn = min(n + s * per_step + sub, n_end - 1);
            xv[s] = *reinterpret_cast<const float2 *>(a.x + nn * a.n_in + 2 * (k0 + kl));
            if constexpr (MODE != kHeadForward) g[s] = a.gy[nn];
        }
    };

    int64_t n = n_begin + (int64_t)wave * per_round;
    float2 xv[kHeadSamples], xv_next[kHeadSamples];
    float g[kHeadSamples] = {}, g_next[kHeadSamples] = {};
    request(n, 0, xv_next, g_next);   // (a wave with no round of its own reads the block's last sample)
    while (n < n_end) {
        float acc[kHeadSamples];
#pragma unroll
        for (int s = 0; s < kHeadSamples; ++s) acc[s] = 0.0f;
        for (int kk = 0; kk < kc; kk += a.lps) {
#pragma unroll
            for (int s = 0; s < kHeadSamples; ++s) {
                xv[s] = xv_next[s];
                g[s] = g_next[s];
            }
            // the step after this one: more pairs of these samples, else the wave's next round
            // (past the end it repeats the block's last sample)
            const bool more = kk + a.lps < kc;
            request(more ? n : n + (int64_t)waves * per_round, more ? kk + a.lps : 0, xv_next, g_next);
            const bool on = kk + pl < kc;
            const int kl = min(kk + pl, kc - 1);
            const float *t_pair = s_tab + kl * a.pitch;
#pragma unroll
            for (int s = 0; s < kHeadSamples; ++s) {
                float4 c1, c2;
                const int i1 = locate_cell(s_grid, a.tab.G, xv[s].x, c1), i2 = locate_cell(s_grid, a.tab.G, xv[s].y, c2);
                const float u = (xv[s].x - c1.z) * c1.w, v = (xv[s].y - c2.z) * c2.w;
                const float a_lo = 1.0f - u, b_lo = 1.0f - v;
                const float *t = t_pair + i1 * a.W + i2;
                const int64_t mine = n + s * per_step + sub;
                if constexpr (MODE == kHeadForward) {
                    float val = (a_lo * b_lo) * t[0];
                    val = fmaf(u * b_lo, t[a.W], val);
                    val = fmaf(a_lo * v, t[1], val);
                    val = fmaf(u * v, t[a.W + 1], val);
                    acc[s] += on ? val : 0.0f;
                } else {
                    const float s00 = g[s] * t[0], s10 = g[s] * t[a.W], s01 = g[s] * t[1], s11 = g[s] * t[a.W + 1];
                    const float d1 = c1.w * ((s10 - s00) * b_lo + (s11 - s01) * v);
                    const float d2 = c2.w * ((s01 - s00) * a_lo + (s11 - s10) * u);
                    if (on && mine < n_end)
                        *reinterpret_cast<float2 *>(a.gx + mine * a.n_in + 2 * (k0 + kl)) = make_float2(d1, d2);
                }
            }
        }
        if constexpr (MODE == kHeadForward) {
#pragma unroll
            for (int s = 0; s < kHeadSamples; ++s) {
                float total_s = acc[s];
                for (int m = a.lps >> 1; m >= 1; m >>= 1) total_s += __shfl_xor(total_s, m, 64);
                const int64_t mine = n + s * per_step + sub;
                if (pl == 0 && mine < n_end) {
                    if (a.atomic_out)
                        unsafeAtomicAdd(a.y + mine, total_s);
                    else
                        a.y[mine] = total_s;
                }
            }
        }
        n += (int64_t)waves * per_round;
    }
}

template <typename CT>
__global__ __launch_bounds__(kHeadThreads) void forward_head_kernel(HeadArgs a)
{
    head_body<CT, kHeadForward>(a);
}

template <typename CT>
__global__ __launch_bounds__(kHeadThreads) void backward_input_head_kernel(HeadArgs a)
{
    head_body<CT, kHeadGradInput>(a);
}

// ---------------------------------------------------------------------------
// The coefficient gradient of one output: gP[corner] += w_corner gy.  The gradient of a chunk of pairs
// sits in LDS, and every pair's copy of it belongs to four lanes of one wave, one lane per corner.  A wave
// executes in lockstep and its LDS instructions in order, so the four lanes read, add and write back
// without atomics: the corners of one sample are four different nodes, and the next sample's reads
// come after this one's writes.  Each lane locates one of four samples; the samples are then handed
// round inside the quad.  Where few pairs leave lanes or LDS idle, a pair has several copies, each with
// samples of its own.  Every workgroup then stores its sums as a partial gradient and
// head_combine_kernel adds the partials up in a fixed order (adding them to the gradient with atomics, as
// a call without room for them does, took 38 us for 256 partials of 148 KB, three times as long).
// (LDS float atomics before this took about 3.5 clocks per lane and CU whatever their addresses: 0.22 ms
// for 256 -> 1 on 65536 rows.  Of the 51 us there 15 go into clearing, staging and writing the
// tables; the rest is bound by the vector port, 100 instructions per four samples and pair: locates further ahead of the chain
// of reads and writes, or several reads in flight, gained 3 % at most.)
// ---------------------------------------------------------------------------
template <int S>
__device__ __forceinline__ float quad_bcast(float v)
{
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), S * 0x55, 0xf, 0xf, true));
}
template <int S>
__device__ __forceinline__ int quad_bcast(int v)
{
    return __builtin_amdgcn_mov_dpp(v, S * 0x55, 0xf, 0xf, true);
}

__global__ __launch_bounds__(kHeadThreads) void backward_coef_head_kernel(HeadArgs a)
{
    extern __shared__ __align__(16) float head_smem[];
    __shared__ float4 s_grid[LMKAN_MAX_GRID];
    const int k0 = blockIdx.y * a.pairs_per_chunk;
    const int kc = min(a.K, k0 + a.pairs_per_chunk) - k0;
    stage_intervals(a.tab, s_grid);
    for (int i = threadIdx.x; i < a.copies * a.pairs_per_chunk * a.pitch; i += blockDim.x) head_smem[i] = 0.0f;
    __syncthreads();

    const int quad = threadIdx.x >> 2, corner = threadIdx.x & 3;
    const int copy = quad / a.pairs_per_chunk, kl = quad - copy * a.pairs_per_chunk;
    const int64_t n_begin = (int64_t)blockIdx.x * a.samples_per_block;
    const int64_t n_end = min(a.B, n_begin + a.samples_per_block);
    if (copy < a.copies && kl < kc) {  // whole quads
        // this lane's corner: weights (flip_u + sign_u u) (flip_v + sign_v v), its node relative to the cell's
        const float sign_u = (corner & 1) ? 1.0f : -1.0f, flip_u = (corner & 1) ? 0.0f : 1.0f;
        const float sign_v = (corner & 2) ? 1.0f : -1.0f, flip_v = (corner & 2) ? 0.0f : 1.0f;
        float *table = head_smem + quad * a.pitch + (corner & 1) * a.W + (corner >> 1);
        const float *xp = a.x + 2 * (k0 + kl);
        const int64_t step = 4 * a.copies;
        int64_t n = n_begin + 4 * copy + corner;  // the sample this lane locates
        auto request = [&](int64_t at, float2 &xv, float &g) {
            const int64_t nn = min(at, n_end - 1);
            xv = *reinterpret_cast<const float2 *>(xp + nn * a.n_in);
            g = a.gy[nn];
        };
        float2 xv;
        float g;
        request(n, xv, g);
        for (; n - corner < n_end; n += step) {
            float2 xv_next;
            float g_next;
            request(n + step, xv_next, g_next);
            float4 c1, c2;
            const int i1 = locate_cell(s_grid, a.tab.G, xv.x, c1), i2 = locate_cell(s_grid, a.tab.G, xv.y, c2);
            int node = i1 * a.W + i2;
            float u = (xv.x - c1.z) * c1.w, v = (xv.y - c2.z) * c2.w;
            if (n >= n_end) node = 0, u = 0.f, v = 0.f, g = 0.f;  // adds zero
            static_for(std::make_integer_sequence<int, 4>{}, [&](auto sc) {
                constexpr int S = decltype(sc)::value;
                const float wu = fmaf(sign_u, quad_bcast<S>(u), flip_u), wv = fmaf(sign_v, quad_bcast<S>(v), flip_v);
                float *t = table + quad_bcast<S>(node);
                *t += wu * wv * quad_bcast<S>(g);
            });
            xv = xv_next;
            g = g_next;
        }
    }
    __syncthreads();
    // element i = node * kc + pair: pairs along the threads, contiguous in the gradient
    const int total = kc * a.nodes;
    const int step_node = (int)blockDim.x / kc, step_kl = (int)blockDim.x - step_node * kc;
    int node = (int)threadIdx.x / kc, kk = (int)threadIdx.x - node * kc;
    for (int i = threadIdx.x; i < total; i += blockDim.x) {
        float v = 0.0f;
        for (int c = 0; c < a.copies; ++c) v += head_smem[(c * a.pairs_per_chunk + kk) * a.pitch + node];
        if (a.partial)
            a.partial[((int64_t)blockIdx.x * a.nodes + node) * a.K + k0 + kk] = v;
        else if (v != 0.0f)
            unsafeAtomicAdd(a.gP + (int64_t)node * a.map.s_node + (int64_t)(k0 + kk) * a.map.s_pair, v);
        node += step_node;
        kk += step_kl;
        if (kk >= kc) {
            kk -= kc;
            ++node;
        }
    }
}

// gP[i] (+)= sum over the partials: 64 elements per workgroup, the partials dealt to its waves, whose
// sums are added in a fixed order
constexpr int kCombineWaves = 16;
__global__ __launch_bounds__(64 * kCombineWaves) void head_combine_kernel(const float *__restrict__ partial,
                                                                          float *__restrict__ gP, int64_t elems,
                                                                          int n_part, int accumulate)
{
    __shared__ float s_sum[kCombineWaves][64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t i = (int64_t)blockIdx.x * 64 + lane;
    float sum = 0.0f;
    if (i < elems)
#pragma unroll 8
        for (int p = wave; p < n_part; p += kCombineWaves) sum += partial[(int64_t)p * elems + i];
    s_sum[wave][lane] = sum;
    __syncthreads();
    if (wave != 0 || i >= elems) return;
    for (int w = 1; w < kCombineWaves; ++w) sum += s_sum[w][lane];
    gP[i] = accumulate ? gP[i] + sum : sum;
}

SmallArgs small_args(const LayerShape &s, const void *coef, const void *records)
{
    const size_t n = (size_t)s.pairs() * (size_t)s.batch;
    SmallArgs a = {};
    a.P = coef;
    a.map = coef_map(s);
    a.rec_node = static_cast<const int32_t *>(records);
    a.rec_u = reinterpret_cast<const float *>(a.rec_node + n);
    a.rec_v = a.rec_u + n;
    a.B = s.batch;
    a.n_out = s.n_out;
    a.K = s.pairs();
    a.W = s.G + 1;
    return a;
}

// enough blocks for 256 CUs: split the pairs when the batch alone gives too few
int pair_split(const LayerShape &s)
{
    const int64_t bblocks = (s.batch + kThreads - 1) / kThreads;
    int split = 1;
    while (bblocks * split < 512 && s.pairs() / (split * 2) >= 8) split *= 2;
    return split;
}

}  // namespace

bool small_out_shape_ok(const LayerShape &s)
{
    return s.n_out <= kSmallMax && (s.n_out == 1 || !slab_backward_input_shape_ok(s));
}

// LDS floats per pair of the one-output forward kernel, and the pairs one workgroup can hold
static int head_pitch(const LayerShape &s) { return s.nodes() | 1; }
static int head_budget() { return (160 * 1024 - LMKAN_MAX_GRID * (int)sizeof(float4)) / (int)sizeof(float); }  // beside the grid
int head_pairs_per_chunk(const LayerShape &s)
{
    int kc = head_budget() / head_pitch(s);
    if (kc >= s.pairs()) return s.pairs();
    return kc & ~63;
}

// One output, rows (not windows), and at least a wave of pairs fits LDS at a time (G <= 24, or few pairs)
bool head_forward_shape_ok(const LayerShape &s)
{
    return s.n_out == 1 && head_pairs_per_chunk(s) > 0;
}

// grid, LDS and per-block share of a launch of head_kernel over at most `max_blocks` workgroups
// per chunk of pairs
static HeadArgs head_args(const LayerShape &s, const GridTab &tab, const float *x, int max_blocks, dim3 *grid,
                          size_t *lds)
{
    HeadArgs a = {};
    a.x = x;
    a.tab = tab;
    a.B = s.batch;
    a.n_in = s.n_in;
    a.K = s.pairs();
    a.W = s.G + 1;
    a.nodes = s.nodes();
    a.pitch = head_pitch(s);
    a.pairs_per_chunk = head_pairs_per_chunk(s);
    const int chunks = (a.K + a.pairs_per_chunk - 1) / a.pairs_per_chunk;
    // a sample takes as many lanes as the chunk has pairs, rounded up to a power of two
    a.lps = 1;
    while (a.lps < 64 && a.lps < a.pairs_per_chunk) a.lps *= 2;
    *lds = (size_t)a.pairs_per_chunk * a.pitch * sizeof(float);
    // every workgroup fills (or clears and later adds out) its LDS copy of the chunk's tables: a
    // workgroup should have at least two rounds of its 16 waves to spread that over
    const int64_t round = (int64_t)(kHeadThreads / 64) * kHeadSamples * (64 / a.lps);
    int64_t per_block = 2 * round;
    if ((s.batch + per_block - 1) / per_block > max_blocks)
        per_block = ((s.batch + max_blocks - 1) / max_blocks + round - 1) / round * round;
    a.samples_per_block = (int)per_block;
    *grid = dim3((unsigned)((s.batch + per_block - 1) / per_block), (unsigned)chunks);
    return a;
}

typedef void (*HeadKernel)(HeadArgs);

static void launch_head(HeadKernel kernel, const HeadArgs &a, dim3 grid, size_t lds, hipStream_t stream,
                        TimedKernel kind, int threads = kHeadThreads)
{
    if (lds > 60 * 1024) allow_large_lds(reinterpret_cast<const void *>(kernel), 160 * 1024 - LMKAN_MAX_GRID * sizeof(float4));
    KernelTiming timing(stream, kind);
    kernel<<<grid, threads, lds, stream>>>(a);
}

void launch_forward_head(const LayerShape &s, const GridTab &tab, const float *x, const void *coef, float *y,
                         hipStream_t stream)
{
    dim3 grid;
    size_t lds;
    HeadArgs a = head_args(s, tab, x, 256, &grid, &lds);   // 256 workgroups fill the chip
    a.P = coef;
    a.map = coef_map(s);
    a.y = y;
    a.atomic_out = grid.y > 1;
    if (a.atomic_out) launch_fill_zero(y, (size_t)s.batch, stream);
    const HeadKernel kernels[3] = {forward_head_kernel<float>, forward_head_kernel<_Float16>,
                                   forward_head_kernel<bf16_t>};
    launch_head(kernels[s.dtype], a, grid, lds, stream, kTimeForward);
}

void launch_backward_input_head(const LayerShape &s, const GridTab &tab, const float *x, const void *coef,
                                const float *gy, float *gx, hipStream_t stream)
{
    dim3 grid;
    size_t lds;
    HeadArgs a = head_args(s, tab, x, 256, &grid, &lds);
    a.P = coef;
    a.map = coef_map(s);
    a.gy = gy;
    a.gx = gx;   // every (sample, pair) is written by exactly one lane: no clearing, no atomics
    const HeadKernel kernels[3] = {backward_input_head_kernel<float>, backward_input_head_kernel<_Float16>,
                                   backward_input_head_kernel<bf16_t>};
    launch_head(kernels[s.dtype], a, grid, lds, stream, kTimeGradInput);
}

// how the coefficient gradient is cut up: copies of the pairs in LDS, samples per workgroup
struct HeadCoefPlan {
    int pairs_per_chunk, copies, threads, chunks;
    int64_t samples_per_block, blocks;
    size_t lds;
};
static HeadCoefPlan head_coef_plan(const LayerShape &s)
{
    HeadCoefPlan p;
    // four lanes per pair: at most 256 pairs and copies of pairs to a workgroup
    const int fit = head_budget() / head_pitch(s);
    p.pairs_per_chunk = std::min(head_pairs_per_chunk(s), 256);
    p.chunks = (s.pairs() + p.pairs_per_chunk - 1) / p.pairs_per_chunk;
    p.copies = 1;
    while (2 * p.copies * p.pairs_per_chunk <= std::min(fit, 256)) p.copies *= 2;
    p.threads = (p.copies * p.pairs_per_chunk * 4 + 63) & ~63;
    p.lds = (size_t)p.copies * p.pairs_per_chunk * head_pitch(s) * sizeof(float);
    // no more workgroups than the chip holds at once, and at least 32 samples to a copy
    const int64_t resident = 256 * std::max(1, std::min((int)(160 * 1024 / (p.lds + 2048)), 2048 / p.threads));
    const int64_t most = std::max<int64_t>(1, std::min<int64_t>(resident / p.chunks, s.batch / (32 * p.copies)));
    p.samples_per_block = ((s.batch + most - 1) / most + 3) & ~(int64_t)3;
    p.blocks = (s.batch + p.samples_per_block - 1) / p.samples_per_block;
    return p;
}

size_t head_partial_bytes(const LayerShape &s)
{
    // (a workgroup whose samples reach few of the nodes adds those few with atomics instead: 4096 rows of
    // 256 -> 1 take 27 us that way, 30 through partials)
    const HeadCoefPlan p = head_coef_plan(s);
    return p.blocks > 1 && 4 * p.samples_per_block >= s.nodes() ? (size_t)p.blocks * s.nodes() * s.pairs() * sizeof(float) : 0;
}

void launch_backward_coef_head(const LayerShape &s, const GridTab &tab, const float *x, const float *gy,
                               float *gcoef, bool accumulate, float *partial, hipStream_t stream)
{
    const HeadCoefPlan p = head_coef_plan(s);
    HeadArgs a = {};
    a.x = x;
    a.tab = tab;
    a.B = s.batch;
    a.n_in = s.n_in;
    a.K = s.pairs();
    a.W = s.G + 1;
    a.nodes = s.nodes();
    a.pitch = head_pitch(s);
    a.pairs_per_chunk = p.pairs_per_chunk;
    a.copies = p.copies;
    a.samples_per_block = (int)p.samples_per_block;
    LayerShape g = s;
    g.layout = LMKAN_LAYOUT_PAPER;
    a.map = coef_map(g);
    a.gy = gy;
    a.gP = gcoef;
    const int64_t elems = (int64_t)s.nodes() * s.pairs();
    // a single workgroup along the samples is its own partial
    if (p.blocks == 1 && !accumulate)
        a.partial = gcoef;
    else
        a.partial = head_partial_bytes(s) > 0 ? partial : nullptr;
    if (!a.partial && !accumulate) launch_fill_zero(gcoef, (size_t)elems, stream);
    launch_head(backward_coef_head_kernel, a, dim3((unsigned)p.blocks, (unsigned)p.chunks), p.lds, stream, kTimeGradCoef,
                p.threads);
    if (a.partial && a.partial != gcoef)
        head_combine_kernel<<<(unsigned)((elems + 63) / 64), 64 * kCombineWaves, 0, stream>>>(a.partial, gcoef, elems,
                                                                                            (int)p.blocks, accumulate ? 1 : 0);
}

void launch_forward_small(const LayerShape &s, const void *coef, float *y, const void *records, hipStream_t stream)
{
    SmallArgs a = small_args(s, coef, records);
    a.y = y;
    const int split = pair_split(s);
    a.pairs_per_block = (a.K + split - 1) / split;
    a.atomic_out = split > 1;
    if (a.atomic_out) launch_fill_zero(y, (size_t)s.batch * s.n_out, stream);
    const dim3 grid((unsigned)((s.batch + kThreads - 1) / kThreads), (unsigned)split);
    KernelTiming timing(stream, kTimeForward);
    switch (s.dtype) {
    case LMKAN_F32: forward_small_kernel<float><<<grid, kThreads, 0, stream>>>(a); break;
    case LMKAN_F16: forward_small_kernel<_Float16><<<grid, kThreads, 0, stream>>>(a); break;
    default: forward_small_kernel<bf16_t><<<grid, kThreads, 0, stream>>>(a); break;
    }
}

void launch_backward_input_small(const LayerShape &s, const GridTab &tab, const void *coef, const float *gy,
                                 float *gx_scratch, const void *records, hipStream_t stream)
{
    SmallArgs a = small_args(s, coef, records);
    a.gy = gy;
    a.gx_t = gx_scratch;
    a.tab = tab;
    const int split = pair_split(s);
    a.pairs_per_block = (a.K + split - 1) / split;
    const dim3 grid((unsigned)((s.batch + kThreads - 1) / kThreads), (unsigned)split);
    KernelTiming timing(stream, kTimeGradInput);
    switch (s.dtype) {
    case LMKAN_F32: backward_input_small_kernel<float><<<grid, kThreads, 0, stream>>>(a); break;
    case LMKAN_F16: backward_input_small_kernel<_Float16><<<grid, kThreads, 0, stream>>>(a); break;
    default: backward_input_small_kernel<bf16_t><<<grid, kThreads, 0, stream>>>(a); break;
    }
}

void launch_backward_coef_small(const LayerShape &s, const void *records, const float *gy, float *gcoef,
                                bool accumulate, hipStream_t stream)
{
    SmallArgs a = small_args(s, nullptr, records);
    a.gy = gy;
    a.gP = gcoef;
    LayerShape g = s;
    g.layout = LMKAN_LAYOUT_PAPER;
    a.map = coef_map(g);
    // pairs per block: the slice must fit 64 KiB of LDS
    const int per_pair = s.nodes() * s.n_out * (int)sizeof(float);
    int kc = (64 * 1024) / per_pair;
    if (kc > a.K) kc = a.K;
    a.pairs_per_block = kc;  // >= 1: (G+1)^2 n_out 4 <= 65^2 * 8 * 4 bytes would not fit, see small_coef_ok
    const int groups = (a.K + kc - 1) / kc;
    int64_t bblocks = (s.batch + kThreads - 1) / kThreads;
    int64_t want = (1024 + groups - 1) / groups;  // about 1024 workgroups in all
    if (bblocks > want) bblocks = want;
    if (!accumulate) launch_fill_zero(gcoef, (size_t)s.nodes() * (size_t)s.pairs() * (size_t)s.n_out, stream);
    const dim3 grid((unsigned)bblocks, (unsigned)groups);
    KernelTiming timing(stream, kTimeGradCoef);
    backward_coef_small_kernel<<<grid, kThreads, (size_t)kc * per_pair, stream>>>(a);
}

bool small_coef_ok(const LayerShape &s)
{
    return small_out_shape_ok(s) && (size_t)s.nodes() * s.n_out * sizeof(float) <= 64 * 1024;
}

}  // namespace lmkan
