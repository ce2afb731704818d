// The cell-sorted sample stream shared by the backward kernels (lmkan_backward.hip builds it,
// lmkan_backward.hip, lmkan_backward_sparse.hip and lmkan_backward_fused.hip walk it), and the matrix-core pieces they use.
//
// For every pair k the samples are grouped by the cell their two inputs fall in (counting
// sort), every non-empty cell padded to whole chunks of four samples, or to halves of them in a sparse stream.  Inside a cell the
// gradients are small dense contractions over the samples of the cell (Alg. 1's four-term sum,
// differentiated), which is what lets them run on the matrix cores.
#pragma once

#include "lmkan_kernels.h"

namespace lmkan {

typedef float f4v __attribute__((ext_vector_type(4)));
typedef unsigned u2v __attribute__((ext_vector_type(2)));

constexpr int kChunk = 4;    // samples per chunk; a chunk never straddles two cells (sparse streams: half a chunk)
constexpr int kHalf = kChunk / 2;
constexpr int kUnroll = 16;  // chunks per trip of the walking kernels' main loops
constexpr int64_t kMaxSortedBatch = (int64_t)65535 * 4096;
// A wave reads gy rows in the order of the sorted stream, i.e. all over the batch; as long as
// the 64-column slice of gy (256 bytes per sample) fits the L2 of an XCD next to the streams,
// the waves of that XCD share it.  Longer batches are cut into blocks of kBlockSamples samples,
// the stream of a pair is sorted by (block, cell), and all waves of an XCD work on one block
// at a time.
constexpr int kBlockSamples = 8192;  // 2 MiB of gy per block and 64-column tile

__host__ __device__ inline int stream_blocks(int64_t B)
{
    return B > kBlockSamples + kBlockSamples / 2 ? (int)((B + kBlockSamples - 1) / kBlockSamples) : 1;
}

// Entries of the sorted stream a block of the batch may take: every non-empty (block, cell) is
// padded to whole chunks, every block to whole trips of kUnroll chunks, and a trip of padding follows
// (the walking kernels prefetch sample indices and gy from the trip behind the last one).
__host__ __device__ inline int64_t stream_block_entries(int64_t B, int G)
{
    const int64_t samples = stream_blocks(B) > 1 ? kBlockSamples : B;
    constexpr int64_t kTrip = kChunk * kUnroll;
    return (samples + (int64_t)(kChunk - 1) * G * G + kTrip - 1) / kTrip * kTrip + kTrip;
}

// Entries per pair: the blocks, and two more trips at the end that the walking kernels may load from
// (never dereferenced as a sample index)
__host__ __device__ inline int64_t stream_stride(int64_t B, int G)
{
    return stream_blocks(B) * stream_block_entries(B, G) + (int64_t)kChunk * (2 * kUnroll);
}

// One entry of the stream, 16 bytes: the local coordinates of Alg. 1's preamble
// (u, v: the four B-spline products are (1-u)(1-v), u(1-v), (1-u)v, uv), a factor that is 0 for a
// padding entry and 1 or -1 for a sample whose cell's second coordinate i2 is even or odd (which
// pair of accumulators takes which column of nodes, see chunk_fma), and the sample index (bit
// pattern of an int32).  Padding entries repeat the index of a sample of the same cell, so that what
// they multiply is a value the cell sees anyway.
struct SortedStream {
    const f4v *rec;              // [K][S]
    const int32_t *chunk_cell;   // [K][S/4]  i1 << 8 | i2 of the cell each chunk belongs to,
                                 //           non-decreasing inside a block.  Sparse: the lower nodes i1 W + i2 of
                                 //           the cells of either half of each chunk, 16 bits each
    const int32_t *block_chunks; // [K][blocks]  chunks of the block to process (a multiple of kUnroll)
    int64_t S;                   // stream_stride
    int block_stride;            // chunks from the start of a block to that of the next
    int n_blocks;
    bool sparse;                 // cells padded to half chunks, the factor's sign by the parity of the cell's lower node
};

// whether the coefficient gradient alone walks a sparse stream
bool coef_stream_is_sparse(const LayerShape &s);
// records = output of launch_preamble_records; fills the stream in `sorted`
// (sorted_records_bytes()) and returns its description
SortedStream launch_sort(const LayerShape &s, const void *records, void *sorted, bool sparse, hipStream_t stream);
// Number of this workgroup (one wave) such that each XCD has a contiguous run of them: workgroups go to the 8 XCDs
// in turn.  (Any count of workgroups.  With the runs for multiples of eight alone, 1042 -> 800 at G = 12 on 12000
// rows, 6773 waves, took 2218 us and takes 1073, 1026 -> 514 at G = 16 on 8192 rows, 4617 waves, 978 and 628.)
__device__ __forceinline__ int xcd_wave()
{
    const int total = gridDim.x, xcd = blockIdx.x & 7, each = total >> 3, over = total & 7;
    return xcd * each + min(xcd, over) + ((int)blockIdx.x >> 3);
}
// whether the batch is short enough for the 32-bit stream positions and 16-bit grid coordinates
bool sorted_batch_ok(const LayerShape &s);
// waves per (pair, output tile, block) of the coefficient gradient's walk
int stream_run_split(const LayerShape &s);

// gy as the walking kernels gather it: the 64 columns of output tile t of row n start at
// base + t * tile_stride + n * row_stride (bytes).  The gradient as the caller holds it,
// [batch][n_out], is such a view with strides 256 and 4 n_out; but the rows of one tile then sit
// 4 n_out bytes apart, a power-of-two stride for the usual widths, and pile up on a few sets of
// the L2 (a 1 MB tile slice of a 4096-wide layer misses four times in ten).  For wide layers
// launch_gy_tiles copies gy once into [tiles][batch][64] (columns past n_out zero), where a tile
// slice is contiguous; for narrower ones it returns the view of gy itself.
struct GyView {
    const float *base;
    int64_t tile_stride;
    unsigned row_stride;
};
size_t gy_tiles_bytes(const LayerShape &s);
GyView launch_gy_tiles(const LayerShape &s, const float *gy, void *tiles, hipStream_t stream);
bool gy_offsets_fit_32_bits(const LayerShape &s, const GyView &gy);
// whether every node of a gradient counts as shared by the runs (see run_nodes)
bool all_nodes_shared(const LayerShape &s, int n_blocks, int n_sub);
// clears what several runs of a stream add to: nothing, the nodes that runs share, or all
void launch_clear_shared_nodes(const LayerShape &s, const SortedStream &st, int n_sub, float *gcoef, hipStream_t stream);
// coefficient gradient alone (lmkan_backward.hip)
void launch_backward_coef_sorted(const LayerShape &s, const SortedStream &st, const GyView &gy, float *gcoef,
                                 bool accumulate, hipStream_t stream);

struct CoefGradArgs {
    const f4v *rec;
    const int32_t *chunk_cell;
    const int32_t *block_chunks;  // [K][n_blocks]
    GyView gy;
    float *gP;
    CoefMap gmap;  // layout of Alg. 1
    int64_t B;
    int64_t S;     // stream_stride
    int block_stride;  // chunks from one block of the stream to the next
    int n_out;
    int K;
    int G;
    int accumulate;
    int n_blocks;  // locality blocks of the batch
    int n_sub;     // waves per (pair, output tile, block)
    int all_shared;  // every node is added to atomically
};

// its walk of a sparse stream (lmkan_backward_sparse.hip)
void launch_coef_sparse(const CoefGradArgs &a, unsigned waves, unsigned lds, hipStream_t stream);

// input gradient, with the coefficient gradient when gcoef is not NULL (lmkan_backward_fused.hip).
// `partial` is scratch of fused_partial_bytes(); the result goes to gx [batch][n_in], or, when
// gx_transposed is not NULL, to that scratch as [n_in][batch] (for the convolution).
bool fused_backward_applicable(const LayerShape &s, const void *coef, const float *gy, const float *gcoef);
void launch_backward_fused(const LayerShape &s, const GridTab &tab, const SortedStream &st, const void *records,
                           const void *coef, const GyView &gy, float *gx, float *gcoef, bool accumulate,
                           void *partial, float *gx_transposed, hipStream_t stream);

// The coefficient gradient's accumulators of a walk: acc[i][2 h + r] is, for output i of the lane and the
// samples of the lane's group, the sum for node (i1 + r, b) with b = i2 or i2 + 1, whichever has the
// parity h.  The next cell of a row of cells shares its column of nodes i2 + 1, so on a step along the
// row only the column left behind is summed over the groups and added to the ring (flush_column)
// while the other one goes on accumulating: half the lane swaps and LDS traffic of a cell's end, no
// copies of live accumulators.  With four samples per cell the end of a cell is most of the walk: step of
// 2048 -> 2048 (G = 32, 4096 rows, bfloat16) 12.0 -> 11.0 ms, of 256 -> 256 at G = 40 781 -> 734 us; with
// 32 per cell (1024 -> 1024, G = 16) 2.70 -> 2.67 ms.
//
// acc[i][q] += (product q of this group's sample) * gy[i] for the chunk whose products sit in
// quad SUB of every group of `w` (lane 16 g + 4 SUB + q holds product q of group g's sample).
// One MFMA is 16 independent 4x4 outer products, block b = lanes 4b .. 4b+3: the A operand of
// the four blocks of a group is taken from the group's block SUB (broadcast size 4 blocks),
// the B operand is the lane's own gy value, and row q of the result lands in register q of
// the same lane.
template <int SUB>
__device__ __forceinline__ void chunk_fma(f4v (&acc)[4], float w, const f4v &g)
{
    acc[0] = __builtin_amdgcn_mfma_f32_4x4x1f32(w, g.x, acc[0], 2, SUB, 0);
    acc[1] = __builtin_amdgcn_mfma_f32_4x4x1f32(w, g.y, acc[1], 2, SUB, 0);
    acc[2] = __builtin_amdgcn_mfma_f32_4x4x1f32(w, g.z, acc[2], 2, SUB, 0);
    acc[3] = __builtin_amdgcn_mfma_f32_4x4x1f32(w, g.w, acc[3], 2, SUB, 0);
}

// The nodes a walk has touched and not yet written: a ring in LDS, [R][64] floats, node id = i1 W + b in
// slot id mod R.  At cell c = i1 W + i2 the nodes below c are final and the highest one with a sum is
// c + W + 1; nodes are written four at a time, so up to three final ones wait: W + 5 slots.
// The ring's size sets how many waves a CU holds on the fine grids: with two whole rows of the table
// (2 W slots) 9 at G = 32 and 7 at G = 40, now 16 and 13: step of 2048 -> 2048
// (G = 32, 4096 rows, bfloat16) 11.0 -> 10.2 ms, of 256 -> 256 at G = 40 734 -> 654 us.
struct NodeRing {
    float *win;
    int W, R;
    unsigned inv;  // id / R = id inv >> 20 for every node of a table and one row beyond (id R < 2^20)
    __device__ __forceinline__ NodeRing(float *window, int w)
        : win(window), W(w), R(w + 5), inv(((1u << 20) + (unsigned)w + 4u) / ((unsigned)w + 5u))
    {
    }
    __device__ __forceinline__ int slot(int id) const { return id - R * (int)(((unsigned)id * inv) >> 20); }
};
static_assert((LMKAN_MAX_GRID + 2) * (LMKAN_MAX_GRID + 1) * (LMKAN_MAX_GRID + 6) < (1 << 20), "NodeRing::slot");

inline unsigned node_ring_bytes(int G) { return (unsigned)((G + 1 + 5) * LMKAN_PACK_TILE * sizeof(float)); }

// Adds the sums of a column of nodes (the one with parity H; `id` is its node in row i1) to the ring and
// clears its accumulators.  Two rounds of "swap halves of two registers, add": the first pairs row i1
// with row i1 + 1 across the 32-lane halves, the second pairs outputs 0, 1 with 2, 3 across odd and even
// 16-lane rows.
template <int H>
__device__ __forceinline__ void flush_column(f4v (&acc)[4], const NodeRing &ring, int id, int lane)
{
    float z[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        // upper half of row i1's sum <-> lower half of row i1 + 1's
        const u2v s = __builtin_amdgcn_permlane32_swap(__float_as_uint(acc[i][2 * H]),
                                                       __float_as_uint(acc[i][2 * H + 1]), false, false);
        z[i] = __uint_as_float(s.x) + __uint_as_float(s.y);  // lanes 0-31: row i1; lanes 32-63: row i1 + 1
        acc[i][2 * H] = acc[i][2 * H + 1] = 0.f;
    }
    float f[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        // odd rows of z[i] <-> even rows of z[i + 2]
        const u2v s = __builtin_amdgcn_permlane16_swap(__float_as_uint(z[i]), __float_as_uint(z[i + 2]), false, false);
        f[i] = __uint_as_float(s.x) + __uint_as_float(s.y);  // even rows: output i; odd rows: output i + 2
    }
    typedef float f2v __attribute__((ext_vector_type(2)));
    const int slot = lane < 32 ? ring.slot(id) : ring.slot(id + ring.W);
    f2v *p = reinterpret_cast<f2v *>(ring.win + slot * LMKAN_PACK_TILE) + ((lane & 15) * 2 + ((lane >> 4) & 1));
    f2v v = *p;
    v.x += f[0];
    v.y += f[1];
    *p = v;
}

// The walk leaves cell `from` for cell `to` (i1 << 8 | i2; to < 0: it ends).
__device__ __forceinline__ void leave_cell(f4v (&acc)[4], const NodeRing &ring, int from, int to, int lane)
{
    const int c = (from >> 8) * ring.W + (from & 255);
    const int odd = from & 1;
    const bool all = to != from + 1;
    if (all || odd == 0) flush_column<0>(acc, ring, c + odd, lane);
    if (all || odd != 0) flush_column<1>(acc, ring, c + 1 - odd, lane);
}

// The nodes of a run of a pair's stream, i1 W + b: `begin` ... `end` (run_end) are written when the walk has passed them.  A
// cell c (its node i1 W + i2) adds to nodes c, c + 1, c + W, c + W + 1 and cells do not decrease along the stream,
// so nodes from the last cell of the runs before + W + 2 on, and below the first cell of the run behind, are this
// run's alone: own_from ... own_to.  The rest of what it touches it shares with a neighbour and adds atomically
// (launch_clear_shared_nodes has set that to zero).  Every node is in one run's own range or a shared one, also where
// nothing is added.  In a stream of several blocks all nodes are shared, and they count as shared in a small gradient.
// (Clearing the whole gradient and adding all of it atomically moves its bytes three more times: backward of 500 -> 333,
// G = 20, 10000 rows 211 -> 172 us with the clearing, of 256 -> 256, G = 40, 8192 rows 383 -> 337, of 256 -> 512, G = 24,
// 10000 rows 254 -> 170, of 1000 -> 96, G = 30, 9000 rows 281 -> 214.)
// (lower nodes of the first and the last cell of a chunk)
template <bool SPARSE>
__device__ __forceinline__ int first_node(int chunk_cell, int W)
{
    return SPARSE ? chunk_cell & 0xffff : (chunk_cell >> 8) * W + (chunk_cell & 255);
}
template <bool SPARSE>
__device__ __forceinline__ int last_node(int chunk_cell, int W)
{
    return SPARSE ? (int)((unsigned)chunk_cell >> 16) : first_node<false>(chunk_cell, W);
}
struct RunNodes {
    int begin, own_from, own_to;
    __device__ __forceinline__ unsigned own() const { return (unsigned)own_from | (unsigned)own_to << 16; }
};
template <bool SPARSE, typename Cells>
__device__ __forceinline__ RunNodes run_nodes(Cells cell, int n_chunks, bool first_run, bool last_run, bool all_shared, int W)
{
    auto first = [&](int i) { return first_node<SPARSE>(cell[i], W); };
    auto last = [&](int i) { return last_node<SPARSE>(cell[i], W); };
    if (all_shared) return {first(0), 0, 0};
    RunNodes r = {0, 0, W * W};
    if (!first_run) {
        r.own_from = last(-1) + W + 2;
        r.begin = min(first(0), r.own_from);
    }
    // (four nodes are written at a time, from `begin` on: whole groups are owned or shared)
    r.own_from = r.begin + ((r.own_from - r.begin + 3) & ~3);
    if (!last_run) r.own_to = r.begin + (max(min(first(n_chunks), last(n_chunks - 1) + W + 2) - r.begin, 0) & ~3);
    return r;
}
// The first node beyond those of cell `last` (i1 << 8 | i2; SPARSE: its lower node).
// (Through the lower node for both, the compiler ordered the dense and the joint walk differently: 0.2 % slower over 120 layers, 1 %
// at most.)
template <bool SPARSE>
__device__ __forceinline__ int node_beyond(int last, int W)
{
    return SPARSE ? last + W + 2 : ((last >> 8) + 1) * W + (last & 255) + 2;
}
// `end` of a run whose last cell is `last`
template <bool SPARSE>
__device__ __forceinline__ int run_end(unsigned own, int last, int W)
{
    return (int)(own >> 16) == W * W ? W * W : node_beyond<SPARSE>(last, W);
}
static_assert((LMKAN_MAX_GRID + 1) * (LMKAN_MAX_GRID + 1) < 1 << 16, "GradOut::own");

// Chunks of a run, when a block's chunks are dealt to n_sub runs in whole trips
__host__ __device__ inline int run_chunks(int chunks, int n_sub)
{
    return (chunks / kUnroll + n_sub - 1) / n_sub * kUnroll;
}

// Where the nodes of a wave's 64 columns go.  Owned nodes: four per store instruction, group g takes node 4 i + g.
// Shared ones: one atomic instruction per node, lanes on consecutive floats (256 contiguous bytes), sums that are
// zero left out.
struct GradOut {
    float *base;  // first column of the tile, node 0
    int64_t s_node;
    int tile_col;  // first column of the tile
    int n_out;
    bool accumulate;
    unsigned own;  // RunNodes: own_from | own_to << 16 (scalar registers are scarce in the walks)
    __device__ __forceinline__ int own_from() const { return (int)(own & 0xffffu); }
    __device__ __forceinline__ int own_to() const { return (int)(own >> 16); }
};

// Nodes [done, upto) can receive nothing more: they are written and their slots cleared.
// BY_FOUR: a multiple of four of them; ROWS4: n_out is a multiple of four.
template <bool BY_FOUR = false, bool ROWS4 = false>
__device__ __forceinline__ void retire_nodes(const NodeRing &ring, const GradOut &o, int &done, int upto, int lane)
{
    const int g = lane >> 4, l16 = lane & 15;
    for (; done < upto; done += 4) {
        if (done < o.own_from() || done >= o.own_to()) {
            for (int id = done; id < min(done + 4, upto); ++id) {
                float *p = ring.win + ring.slot(id) * LMKAN_PACK_TILE + lane;
                const float v = *p;
                *p = 0.f;
                if (v != 0.f && o.tile_col + lane < o.n_out) unsafeAtomicAdd(o.base + id * o.s_node + lane, v);
            }
        } else {
            int slot = ring.slot(done) + g;
            if (slot >= ring.R) slot -= ring.R;
            f4v *p = reinterpret_cast<f4v *>(ring.win + slot * LMKAN_PACK_TILE) + l16;
            if (BY_FOUR || done + g < upto) {
                const int col = o.tile_col + l16 * 4;
                if (col < o.n_out) {
                    float *dst = o.base + (done + g) * o.s_node + l16 * 4;
                    const f4v v = *p;
                    if (ROWS4 || (o.n_out & 3) == 0) {
                        f4v *d4 = reinterpret_cast<f4v *>(dst);
                        // (past the caches: the gradient of a wave is read by nobody soon, and would push out the
                        // rows of gy that all waves of an XCD gather from: 2048 -> 2048, G = 32: 4290 -> 4130 us,
                        // 1024 -> 1024 at G = 28 1280 -> 1170, with 32 samples per cell no difference)
                        __builtin_nontemporal_store(o.accumulate ? *d4 + v : v, d4);
                    } else if (col + 4 <= o.n_out) {
                        // rows of the gradient start on 4 bytes, which a 16-byte access allows on this hardware (four accesses
                        // of 4 bytes instead: 1000 -> 333, G = 32, 8000 rows 748 us, now 636; 500 -> 333, G = 20 255, now 230)
                        typedef float f4u __attribute__((ext_vector_type(4), aligned(4)));
                        f4u *d4 = reinterpret_cast<f4u *>(dst);
                        const f4u w = {v.x, v.y, v.z, v.w};
                        *d4 = o.accumulate ? *d4 + w : w;
                    } else {
#pragma unroll
                        for (int e = 0; e < 3; ++e)
                            if (col + e < o.n_out) dst[e] = o.accumulate ? dst[e] + v[e] : v[e];
                    }
                }
                *p = f4v{0.f, 0.f, 0.f, 0.f};
            }
        }
    }
}

// Whole groups of four nodes that are final once the walk stands at cell `cell`.
__device__ __forceinline__ void retire_before(const NodeRing &ring, const GradOut &o, int &done, int cell, int lane)
{
    const int c = (cell >> 8) * ring.W + (cell & 255);
    retire_nodes(ring, o, done, done + ((c - done) & ~3), lane);
}

// All four products of this lane's entry, in that order, spread over its quad: r[i] of lane q is product q of the
// entry of the quad's lane i (a 4 x 4 transposition).  One load per lane then serves sixteen chunks.
__device__ __forceinline__ void entry_products(const f4v &e, int lane, float (&r)[4])
{
    const float a0 = 1.0f - e.x, b_lo = 1.0f - e.y, there = __builtin_fabsf(e.z);
    const bool odd = e.z < 0.f;
    const float b0 = (odd ? e.y : b_lo) * there, b1 = (odd ? b_lo : e.y) * there;
    const float p[4] = {a0 * b0, e.x * b0, a0 * b1, e.x * b1};
    auto from = [](float v, auto ctrl) {
        return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), decltype(ctrl)::value, 0xf, 0xf, true));
    };
    constexpr std::integral_constant<int, 0xB1> across1{};   // quad_perm [1,0,3,2]
    constexpr std::integral_constant<int, 0x4E> across2{};   // quad_perm [2,3,0,1]
    const bool q0 = (lane & 1) != 0, q1 = (lane & 2) != 0;
    float t[4];
#pragma unroll
    for (int i = 0; i < 4; i += 2) {
        const float x = from(p[i + 1], across1), y = from(p[i], across1);   // (by all lanes, before anyone chooses)
        t[i] = q0 ? x : p[i];
        t[i + 1] = q0 ? p[i + 1] : y;
    }
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const float x = from(t[i + 2], across2), y = from(t[i], across2);
        r[i] = q1 ? x : t[i];
        r[i + 2] = q1 ? t[i + 2] : y;
    }
}

// product q = (lane & 3) of an entry, in the order of the accumulators: ((1-u)(1-v), u(1-v), (1-u)v, uv)[q]
// for a cell with even i2, the two pairs swapped for an odd one; 0 for padding
__device__ __forceinline__ float entry_product(const f4v &e, int q)
{
    const float a = (q & 1) ? e.x : 1.0f - e.x;
    const float b = ((q & 2) != 0) != (e.z < 0.f) ? e.y : 1.0f - e.y;
    return a * b * __builtin_fabsf(e.z);
}

}  // namespace lmkan
