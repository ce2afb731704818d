// Device-side pieces shared by every lmKAN kernel: the grid table, the cell
// lookup and the four weights of Alg. 1's preamble, and coefficient decoding.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <utility>

#include "lmkan.h"

namespace lmkan {

// Extended grid (Sec. 3.1, App. B "Edge cases") as float32, passed to kernels by value.
// node[1..G-1] are the real grid points, node[0] / node[G] the ghost points;
// inv_h[i] = 1 / (node[i+1] - node[i]).
struct GridTab {
    float node[LMKAN_MAX_GRID + 1];
    float inv_h[LMKAN_MAX_GRID];
    int G;
};

// Convolution as a fully connected layer on windows (Sec. 5, "lmKAN-based Convolutional Neural
// Networks"): channels-last image x[N][H][W][C], kh x kw window, no padding; row r of the layer =
// output pixel (img, oy, ox), r = (img OH + oy) OW + ox; input e = (ky kw + kx) C + c of that row is
// x[img][oy stride + ky][ox stride + kx][c].  The patches are never written out: every kernel that
// reads x goes through this map.  C == 0 stands for a plain layer on rows x[n][n_in].
struct ConvGeom {
    int N, H, W, C, kh, kw, stride, OH, OW;
};

// offset, in elements, of input e of row n
__host__ __device__ inline int64_t conv_input_offset(const ConvGeom &cg, int64_t n, int e)
{
    const int c = e % cg.C, kx = (e / cg.C) % cg.kw, ky = e / (cg.C * cg.kw);
    const int ox = (int)(n % cg.OW), oy = (int)((n / cg.OW) % cg.OH);
    const int64_t img = n / ((int64_t)cg.OW * cg.OH);
    return ((img * cg.H + (oy * cg.stride + ky)) * cg.W + (ox * cg.stride + kx)) * cg.C + c;
}

// the two inputs of pair k of row n (with an odd channel count they can sit in two pixels)
template <bool CONV>
__device__ inline float2 load_input_pair(const float *__restrict__ x, int64_t n, int n_in, int k, const ConvGeom &cg)
{
    if constexpr (!CONV) {
        return *reinterpret_cast<const float2 *>(x + n * n_in + 2 * k);
    } else {
        const int64_t o0 = conv_input_offset(cg, n, 2 * k);
        const int64_t o1 = (cg.C & 1) ? conv_input_offset(cg, n, 2 * k + 1) : o0 + 1;
        return make_float2(x[o0], x[o1]);
    }
}

// Where coefficient (node, pair k, output tile jt, column jl) lives, in elements:
//   node * s_node + k * s_pair + jt * s_tile + jl,
// and moving one node along the second axis adds s_node, along the first (G+1) * s_node.
// Covers both the layout of Alg. 1 and the packed layout.
struct CoefMap {
    int64_t s_node;
    int64_t s_pair;
    int64_t s_tile;
};

// One record per (sample, pair): Alg. 1's preamble output.
struct Preamble {
    int node;    // i1 * (G+1) + i2 : table node of the cell's lower-left corner
    int cell;    // i1 * G + i2
    float a_lo;  // (node[i1+1] - x1) / h1 : factor of B_{i1}
    float a_hi;  // (x1 - node[i1]) / h1   : factor of B_{i1+1}
    float b_lo;  // same along the second axis
    float b_hi;
    float rh1;   // 1 / h1, 1 / h2 : needed by the input gradient
    float rh2;
};

// App. B Eq. 5 the way Alg. 2 evaluates it: one exponential of -|x|.
__device__ __forceinline__ float sigma(float x)
{
    float t = __expf(-fabsf(x));
    return x > 0.0f ? 1.0f - 0.5f * t : 0.5f * t;
}

// Cell index.  The candidate floor(sigma(x) G) of Sec. 3.1 is corrected against the
// float32 grid table so that the result is exactly "number of real grid points <= x"
// whatever the accuracy of the exponential.  node points to LDS or kernel arguments.
__device__ __forceinline__ int locate(const float *node, int G, float x)
{
    int i = (int)(sigma(x) * (float)G);
    i = min(max(i, 0), G - 1);
    while (i > 0 && x < node[i]) --i;
    while (i < G - 1 && x >= node[i + 1]) ++i;
    return i;
}

__device__ __forceinline__ Preamble preamble(const float *node, const float *inv_h, int G, float x1,
                                             float x2)
{
    Preamble r;
    int i1 = locate(node, G, x1);
    int i2 = locate(node, G, x2);
    r.node = i1 * (G + 1) + i2;
    r.cell = i1 * G + i2;
    r.rh1 = inv_h[i1];
    r.rh2 = inv_h[i2];
    r.a_lo = (node[i1 + 1] - x1) * r.rh1;
    r.a_hi = (x1 - node[i1]) * r.rh1;
    r.b_lo = (node[i2 + 1] - x2) * r.rh2;
    r.b_hi = (x2 - node[i2]) * r.rh2;
    return r;
}

// One interval of the grid as locate_cell() wants it: x belongs to interval i when lo <= x < hi
// (the outer intervals are open ended), u = (x - node) * inv_h.
__device__ __forceinline__ void stage_intervals(const GridTab &tab, float4 *s_grid)
{
    for (int i = threadIdx.x; i < tab.G; i += blockDim.x)
        s_grid[i] = make_float4(i == 0 ? -INFINITY : tab.node[i], i == tab.G - 1 ? INFINITY : tab.node[i + 1],
                                tab.node[i], tab.inv_h[i]);
}

// The interval of x (as locate(): candidate from the exponential, corrected against the table, so
// the index is exact) and its entry.  One 16-byte LDS read unless the candidate was off.
__device__ __forceinline__ int locate_cell(const float4 *s_grid, int G, float x, float4 &cell)
{
    int i = min(max((int)(sigma(x) * (float)G), 0), G - 1);
    cell = s_grid[i];
    while (x < cell.x || x >= cell.y) {
        i += x < cell.x ? -1 : 1;
        if (i < 0 || i >= G) {  // x = +inf: the last interval
            i = G - 1;
            cell = s_grid[i];
            break;
        }
        cell = s_grid[i];
    }
    return i;
}

// Stored coefficient -> float32.
__device__ __forceinline__ float widen(float v) { return v; }
__device__ __forceinline__ float widen(_Float16 v) { return (float)v; }
struct bf16_t {
    uint16_t bits;
};
__device__ __forceinline__ float widen(bf16_t v) { return __uint_as_float((uint32_t)v.bits << 16); }

// ---------------------------------------------------------------------------
// DPP helpers.  row_newbcast:S makes every lane of a 16-lane row read lane S of
// that row.
// ---------------------------------------------------------------------------
template <int S>
__device__ __forceinline__ int row_bcast(int v)
{
    return __builtin_amdgcn_update_dpp(0, v, 0x150 + S, 0xf, 0xf, true);
}

// acc += (w of lane S of this row) * c
template <int S>
__device__ __forceinline__ void fmac_row_bcast(float &acc, float w, float c)
{
    asm("v_fmac_f32_dpp %0, %1, %2 row_newbcast:%3 row_mask:0xf bank_mask:0xf"
        : "+v"(acc)
        : "v"(w), "v"(c), "n"(S));
}

// Counts this lane's sample in a counter of its wave (16 bits, two to an LDS word) and returns how many samples
// the counter held before it: those of earlier calls, and of this call those of lower lanes.  `key` (12 bits,
// `wide` if it has more than 8) tells the counters of the wave apart.
// What an atomic returns depends on the order in which it takes the lanes that meet in a counter, which is the
// hardware's and not documented.  So the lanes with the same key are found by a ballot per bit, the counter is
// read before any of them adds (a wave's LDS operations take place in the order they are issued; the empty
// instructions keep the compiler from exchanging or joining them), and nothing waits in between.
// (Five vector instructions per bit.  One lane adding for all that meet, and handing out what the atomic
// returned, waits for LDS twice per sample: 11 us of a step with 512 pairs x 8192 samples instead of 4.)
__device__ __forceinline__ int count_in_order(int *words, int counter, int key, bool wide)
{
    const uint64_t running = __ballot(true);
    unsigned lo = (unsigned)running, hi = (unsigned)(running >> 32);
    const auto meet = [&](int bit) {
        const unsigned set = (unsigned)__builtin_amdgcn_sbfe(key, bit, 1);  // all ones or zero
        const uint64_t those = __ballot(set != 0);
        lo = __builtin_amdgcn_bitop3_b32(lo, (unsigned)those, set, 0x90);  // lo & ~(those ^ set)
        hi = __builtin_amdgcn_bitop3_b32(hi, (unsigned)(those >> 32), set, 0x90);
    };
#pragma unroll
    for (int bit = 0; bit < 8; ++bit) meet(bit);
    if (wide)
#pragma unroll
        for (int bit = 8; bit < 12; ++bit) meet(bit);
    int *word = &words[counter >> 1];
    const int shift = (counter & 1) * 16;
    const int held = __hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    asm volatile("" : : : "memory");
    (void)__hip_atomic_fetch_add(word, 1 << shift, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    asm volatile("" : : : "memory");
    return ((held >> shift) & 0xffff) + __builtin_amdgcn_mbcnt_hi(hi, __builtin_amdgcn_mbcnt_lo(lo, 0));
}

template <int... Ts, class F>
__device__ __forceinline__ void static_for(std::integer_sequence<int, Ts...>, F &&f)
{
    (f(std::integral_constant<int, Ts>{}), ...);
}

}  // namespace lmkan
