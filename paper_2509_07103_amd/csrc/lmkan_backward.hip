// Coefficient gradient without atomics.
//
//   gP[a][b][k][j] = sum over samples n whose cell for pair k has (a,b) as a corner of
//                    B_ab(x_n) * gy[n][j]                  (derivative of Alg. 1's sum)
//
// Pass 1 (sort_kernel): for every pair k the samples are grouped by cell with a counting sort, each
// cell padded to whole chunks of four samples, the local coordinates stored next to the sample
// index.  (Sparse streams, coef_stream_is_sparse: cells padded to half a chunk, and pass 2 is the walk of
// lmkan_backward_sparse.hip.)
// Pass 2 (backward_coef_stream_kernel): one wave owns (pair k, 64 outputs) and walks the
// sorted chunks, cell after cell.  The four samples of a chunk go to the four 16-lane
// groups of the wave and a lane covers four adjacent outputs, so gy is read with 16-byte
// loads.  Within a cell the update is a small dense contraction, (4 corners x samples) times
// (samples x outputs), and runs on the matrix cores: one 4x4x1 float32 MFMA (16 blocks)
// multiplies the four products of each group's sample with one gy value per lane, the
// block-broadcast control handing every block of a group the products of that group's sample.
// The 16 partial sums (4 corners x 4 outputs) live in the MFMA accumulators.  When the walk
// leaves a column of nodes its sums are combined across the groups and added into a
// ring of nodes kept in LDS; a node is written to global memory exactly
// once, when the walk has passed it.  Nodes no sample touches are written as exact zeros, so
// no separate zero fill is needed.
#include "lmkan_kernels.h"
#include "lmkan_sorted.h"

namespace lmkan {

namespace {

constexpr int kTile = LMKAN_PACK_TILE;
constexpr int kSortThreads = 1024;

constexpr int kDepth = 8;    // chunks of gy values in flight
static_assert(kUnroll % kDepth == 0, "the gy ring must divide the unrolled trip");

// Counting sort of the samples of every pair by cell, one launch: a workgroup takes the samples of one
// (pair, block).  records_in: [3][K][B] (node, u, v) from the preamble pass.  Per pair k, with
// S = stream_stride and C = stream_block_entries, block b owns the entries [b C, (b + 1) C):
//   rec [K][S]           (u, v, 1 or -1 for an even or odd i2 - sparse: i1 W + i2 -, index) of a sample, 16 bytes;
//                        padding entries are (0, 0, 0, index of a sample of the same cell)
//   chunk_cell [K][S/4]  i1 << 8 | i2 of the cell each chunk belongs to, non-decreasing
//                        inside a block; sparse: i1 W + i2 of the cells of its halves, 16 bits each
//   block_chunks [K][blocks]  chunks of the block to process, a multiple of kUnroll; one trip of
//                        padding entries follows (the walking kernels prefetch into it)
// A thread keeps its samples in registers; LDS holds a population per (wave, cell) (16 bits each).
// A sample's rank is what the counter of its wave and cell held before it, and the wave's samples
// are a run of consecutive ones taken in order, so the order inside a cell is that of the indices:
// sums over a cell repeat in every run.
// The entries go out through LDS, kSortStage stream positions at a time, so that the stores run along
// the stream (16-byte stores all over a block's 130 KB are bound by the L2's requests: 175 us at 64
// pairs x 262144 samples).
// (512 pairs x 8192 samples take 33 us, 64 pairs x 262144 115 us, of which 4 and 8 rank the lanes that meet
// in a cell.  Four launches before this one - a histogram per segment of 4096 samples, block sizes, layout,
// scatter, where a stable order took a pass over each cell's run: 100 and 178 us.)
constexpr int kSortWaves = kSortThreads / 64;
constexpr int kSortPer = 12;  // samples of a thread, at most
constexpr int kSortStage = 4096;  // stream positions that go through LDS at a time
constexpr int kOddCell = 1 << 30;  // a flag beside a sample's index: its cell has an odd i2
static_assert(kMaxSortedBatch < kOddCell, "sample indices leave the bit to the flag");
static_assert(kBlockSamples + kBlockSamples / 2 <= kSortThreads * kSortPer, "a block must fit a workgroup");

__host__ __device__ inline size_t sort_lds_bytes(int G)
{
    const size_t cells = (size_t)G * G, even = (cells + 1) & ~(size_t)1;
    const size_t counts = ((size_t)kSortWaves * even + even) * sizeof(unsigned short);
    const size_t stage = (size_t)kSortStage * 3 * sizeof(float);
    return (cells + 1) * sizeof(int) + (counts > stage ? counts : stage);
}

template <bool SPARSE>
__device__ __forceinline__ void sort_block(const int32_t *__restrict__ rec_node, const float *__restrict__ rec_u,
                                           const float *__restrict__ rec_v, f4v *__restrict__ rec,
                                           int32_t *__restrict__ chunk_cell, int32_t *__restrict__ block_chunks, int64_t B,
                                           int G)
{
    extern __shared__ __align__(16) int s_dyn[];
    __shared__ int s_wave_total[kSortWaves];
    __shared__ int s_last_cell;
    constexpr int kPad = SPARSE ? kHalf : kChunk;
    const int cells = G * G, even = (cells + 1) & ~1;
    int *s_start = s_dyn;                                                             // [cells + 1]
    unsigned short *s_off = reinterpret_cast<unsigned short *>(s_start + cells + 1);  // [waves][even]
    unsigned short *s_total = s_off + kSortWaves * even;                              // [even]
    int *s_count = reinterpret_cast<int *>(s_off);  // the same memory, two counters to a word
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int blk = blockIdx.x, k = blockIdx.y;
    const int blocks = stream_blocks(B);
    const int64_t n0 = (int64_t)blk * kBlockSamples;
    const int count = (int)(blocks > 1 && n0 + kBlockSamples < B ? kBlockSamples : B - n0);
    const int per = (count + kSortThreads - 1) / kSortThreads;
    const int64_t o = (int64_t)k * B + n0;
    const int i0 = wave * per * 64 + lane;  // this thread's samples: i0 + 64 j

    // all loads of the thread first: the pass is bound by the bytes in flight
    int cell[kSortPer], rank[kSortPer];
    unsigned odd = 0;  // bit j: sample j's cell has an odd i2
    float u[kSortPer], v[kSortPer];
#pragma unroll
    for (int j = 0; j < kSortPer; ++j) {
        cell[j] = -1;
        if (j < per && i0 + 64 * j < count) {
            cell[j] = rec_node[o + i0 + 64 * j];
            u[j] = rec_u[o + i0 + 64 * j];
            v[j] = rec_v[o + i0 + 64 * j];
        }
    }
    for (int c = tid; c < kSortWaves * even / 2; c += kSortThreads) s_count[c] = 0;
    if (tid == 0) s_last_cell = 0;
    __syncthreads();
    const unsigned W = G + 1, inv_w = ((1u << 20) + W - 1) / W;  // node / W = node inv_w >> 20 for every node of a table
#pragma unroll
    for (int j = 0; j < kSortPer; ++j) {
        if (cell[j] >= 0) {
            const int i1 = (int)(((unsigned)cell[j] * inv_w) >> 20);
            const int c = cell[j] - i1;  // i1 (G + 1) + i2 -> i1 G + i2
            odd |= ((SPARSE ? cell[j] : cell[j] ^ (i1 & (int)W)) & 1u) << j;  // i2 = node - i1 W
            cell[j] = c;
            rank[j] = count_in_order(s_count, wave * even + c, c, cells > 256);
        }
    }
    __syncthreads();
    // counters -> offsets of a wave's samples inside the cell; padded populations -> first positions
    {
        const int run_cells = (cells + kSortThreads - 1) / kSortThreads;
        const int c0 = min(cells, tid * run_cells), c1 = min(cells, c0 + run_cells);
        int mine = 0;
        for (int c = c0; c < c1; ++c) {
            int run = 0;
#pragma unroll
            for (int w = 0; w < kSortWaves; ++w) {
                const int n = s_off[w * even + c];
                s_off[w * even + c] = (unsigned short)run;
                run += n;
            }
            s_total[c] = (unsigned short)run;
            mine += (run + kPad - 1) / kPad * kPad;
            if (run > 0) atomicMax(&s_last_cell, c);
        }
        int incl = mine;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const int t = __shfl_up(incl, d, 64);
            if (lane >= d) incl += t;
        }
        if (lane == 63) s_wave_total[wave] = incl;
        __syncthreads();
        int run = incl - mine;
        for (int w = 0; w < wave; ++w) run += s_wave_total[w];
        for (int c = c0; c < c1; ++c) {
            s_start[c] = run;
            run += (s_total[c] + kPad - 1) / kPad * kPad;
        }
        if (tid == kSortThreads - 1) s_start[cells] = run;
    }
    __syncthreads();
    const int64_t S = stream_stride(B, G), C = stream_block_entries(B, G);
    f4v *out = rec + (int64_t)k * S + blk * C;
    int32_t *out_cell = chunk_cell + ((int64_t)k * S + blk * C) / kChunk;
    const int last = s_last_cell, real_end = s_start[cells];
    constexpr int kTrip = kUnroll * kChunk;
    const int block_end = (real_end + kTrip - 1) / kTrip * kTrip, fill_end = block_end + kTrip;
#pragma unroll
    for (int j = 0; j < kSortPer; ++j)
        if (cell[j] >= 0) rank[j] += s_start[cell[j]] + s_off[wave * even + cell[j]];  // the stream position
    __syncthreads();
    // the counters make room for the entries on their way out
    float *s_u = reinterpret_cast<float *>(s_off), *s_v = s_u + kSortStage;
    int *s_n = reinterpret_cast<int *>(s_v + kSortStage);
    int last_sample = 0;  // a sample of the block's last cell, for the padding behind it
    for (int base = 0; base < fill_end; base += kSortStage) {
        // (the flagged indices must not be formed ahead of the loop: 64 registers let two workgroups share a CU)
        asm volatile("" : "+v"(odd));
        for (int p = tid; p < kSortStage; p += kSortThreads) s_n[p] = -1;
        __syncthreads();
#pragma unroll
        for (int j = 0; j < kSortPer; ++j) {
            const int p = rank[j] - base;
            if (cell[j] >= 0 && p >= 0 && p < kSortStage) {
                s_u[p] = u[j];
                s_v[p] = v[j];
                s_n[p] = ((int32_t)n0 + i0 + 64 * j) | ((odd >> j & 1u) != 0 ? kOddCell : 0);
            }
        }
        __syncthreads();
        if (real_end > base) last_sample = s_n[min(real_end - base, kSortStage) - kPad];
        for (int p = tid; p < kSortStage && base + p < fill_end; p += kSortThreads) {
            // (the first entry of a chunk, or half chunk, is always a sample, unless it lies past the real ones)
            const int n = s_n[p], first = s_n[p & ~(kPad - 1)];
            f4v e = {0.f, 0.f, 0.f, __int_as_float((first >= 0 ? first : last_sample) & ~kOddCell)};
            if (n >= 0) e = f4v{s_u[p], s_v[p], (n & kOddCell) != 0 ? -1.0f : 1.0f, __int_as_float(n & ~kOddCell)};
            out[base + p] = e;
        }
        __syncthreads();
    }
    // the cell of every chunk, or half chunk: the highest cell whose start is <= its first position (an empty
    // cell shares its start with the next one, so the highest such cell is never empty); chunks past
    // the real ones belong to the block's last cell
    for (int q = tid; q < fill_end / kPad; q += kSortThreads) {
        int c = last;
        if (q * kPad < real_end) {
            int lo = 0, hi = cells - 1;
            while (lo < hi) {
                const int mid = (lo + hi + 1) >> 1;
                if (s_start[mid] <= q * kPad) lo = mid; else hi = mid - 1;
            }
            c = lo;
        }
        if constexpr (SPARSE)
            reinterpret_cast<unsigned short *>(out_cell)[q] = (unsigned short)(c + c / G);
        else
            out_cell[q] = ((c / G) << 8) | (c % G);
    }
    if (tid == 0) block_chunks[(int64_t)k * blocks + blk] = block_end / kChunk;
}

__global__ __launch_bounds__(kSortThreads) void sort_kernel(const int32_t *__restrict__ rec_node, const float *__restrict__ rec_u, const float *__restrict__ rec_v,
                                                           f4v *__restrict__ rec, int32_t *__restrict__ chunk_cell, int32_t *__restrict__ block_chunks, int64_t B, int G)
{
    sort_block<false>(rec_node, rec_u, rec_v, rec, chunk_cell, block_chunks, B, G);
}

// (the same for a sparse stream: cells padded to kPad = kHalf entries, the one value there is)
template <int kPad>
__global__ __launch_bounds__(kSortThreads) void sort_kernel(const int32_t *__restrict__ rec_node, const float *__restrict__ rec_u, const float *__restrict__ rec_v,
                                                           f4v *__restrict__ rec, int32_t *__restrict__ chunk_cell, int32_t *__restrict__ block_chunks, int64_t B, int G)
{
    static_assert(kPad == kHalf, "");
    sort_block<true>(rec_node, rec_u, rec_v, rec, chunk_cell, block_chunks, B, G);
}

template <bool kOffset32>
__global__ __launch_bounds__(64) void backward_coef_stream_kernel(CoefGradArgs a)
{
    extern __shared__ __align__(16) float win[];  // the NodeRing of this wave's columns
    const int lane = threadIdx.x;
    const int g = lane >> 4, l16 = lane & 15;
    const int G = a.G, W = G + 1;

    // Waves that run together on one XCD (ids congruent mod 8) take the same output tile and the
    // same block of the batch, so the piece of gy they all gather from stays in that XCD's L2.
    int id = xcd_wave();
    const int sub = id % a.n_sub;
    id /= a.n_sub;
    const int k = id % a.K;
    id /= a.K;
    const int blk = id % a.n_blocks;
    const int jt = id / a.n_blocks;

    const int col = jt * kTile + l16 * 4;
    const bool col_ok = col < a.n_out;
    typedef __attribute__((address_space(4))) const int32_t *ScalarIntPtr;
    // With one block and one wave per (pair, tile) the wave owns its columns of the gradient and
    // writes every row once.  Otherwise (long batches; too few pairs x tiles to fill the chip)
    // a wave takes a run of whole trips of one block; a run may begin and end anywhere, even
    // inside a cell, and some or all of its nodes are other waves' too (run_nodes).
    bool last_run = true;
    int c_begin = blk * a.block_stride;
    int nch = ((ScalarIntPtr)(a.block_chunks + (int64_t)k * a.n_blocks))[blk];
    if (a.n_sub > 1) {
        const int per = run_chunks(nch, a.n_sub), skip = min(sub * per, nch);
        last_run = skip + per >= nch;
        c_begin += skip;
        nch = min(per, nch - skip);
        if (nch == 0) return;
    }
    ScalarIntPtr cc = (ScalarIntPtr)(a.chunk_cell + (int64_t)k * (a.S / kChunk) + c_begin);

    // entries: lane (g, j) fetches the entry of group g's sample of chunk c + j, sixteen chunks per load (a trip).
    // The texture addresser takes four lanes per clock, so a load costs 16 clocks whatever it brings; with four
    // loads of entries and one of indices per trip it was busy 85 % of the kernel (1024 -> 1024, G = 16).
    const f4v *rec_k = a.rec + (int64_t)k * a.S + (int64_t)c_begin * kChunk;  // wave-uniform
    // The loads of the main loop are written as inline assembly, and so are the waits for them:
    // vector loads return in the order they were issued, and with the cell changes branching
    // inside the loop the compiler sizes its own waits for the worst path it can imagine, which
    // drains the ring of gy values at every step (it emitted vmcnt(0) ... vmcnt(6) where 9 loads
    // may stay in flight).  Every load below is issued at a fixed place of a trip, so the number
    // of younger loads at the point of use is known; loads the compiler adds on the rare paths
    // (row stores, atomics) only add to that number, which keeps the waits safe.
    const unsigned e_off = (unsigned)((l16 * kChunk + g) * sizeof(f4v));
    // (operands are copied into locals first: a name used only as an asm operand is not captured)
    auto load_e = [&](f4v &dst, int chunk) {
        const f4v *base = rec_k + (int64_t)chunk * kChunk;
        const unsigned off = e_off;
        asm volatile("global_load_dwordx4 %0, %1, %2" : "=v"(dst) : "v"(off), "s"(base) : "memory");
    };
    // blocks until at most N loads younger than the one that fills v are outstanding, i.e. until v has landed.
    // The compiler does not know that v is in flight between the load and this wait: were it to copy
    // or move v in between, it would copy stale data and hand the old register to something else for
    // the late load to overwrite.  The comment in the instruction names the register, so that the
    // generated code can be checked (check_codegen.py does, at every build): on every path from a
    // load, the first instruction that touches its destination must be this wait.
    auto landed = [](auto &v, auto nc) {
        asm volatile("s_waitcnt vmcnt(%1) ; landed %0" : "+v"(v) : "n"(decltype(nc)::value) : "memory");
    };

    const unsigned col_bytes = col_ok ? (unsigned)l16 * 16u : 0u;
    const unsigned row_bytes = a.gy.row_stride;
    const char *gy_tile = reinterpret_cast<const char *>(a.gy.base) + (int64_t)jt * a.gy.tile_stride;
    // what a lane keeps of the sixteen samples of a trip: the byte offset of the sample's row when
    // every offset fits 32 bits (one multiply per trip; the broadcast to the group then folds into
    // the add of the lane's column, a single DPP instruction per chunk), else the sample index
    auto row_offset = [&](int n) { return kOffset32 ? (int)__umul24((unsigned)n, row_bytes) : n; };
    auto load_gy = [&](f4v &dst, auto subc, int off16) {
        constexpr int SUB = decltype(subc)::value;
        if constexpr (kOffset32) {
            const unsigned off = (unsigned)row_bcast<SUB>(off16) + col_bytes;
            const char *base = gy_tile;
            asm volatile("global_load_dwordx4 %0, %1, %2" : "=v"(dst) : "v"(off), "s"(base) : "memory");
        } else {
            const char *ptr = gy_tile + ((int64_t)row_bcast<SUB>(off16) * row_bytes + col_bytes);
            asm volatile("global_load_dwordx4 %0, %1, off" : "=v"(dst) : "v"(ptr) : "memory");
        }
    };

    const NodeRing ring(win, W);
    for (int i = lane; i < ring.R * kTile; i += 64) win[i] = 0.0f;
    const RunNodes nodes = run_nodes<false>(cc, nch, sub == 0, last_run, a.all_shared != 0, W);
    const GradOut out{a.gP + (int64_t)k * a.gmap.s_pair + jt * kTile, a.gmap.s_node, jt * kTile, a.n_out, a.accumulate != 0,
                      nodes.own()};

    f4v acc[4];  // [output i of the lane][2 (column parity) + row], see lmkan_sorted.h
#pragma unroll
    for (int i = 0; i < 4; ++i) acc[i] = f4v{0.f, 0.f, 0.f, 0.f};
    int cur_cell = -1;  // (i1 << 8 | i2) of the cell the accumulators belong to
    int done = nodes.begin;  // nodes below have been written, or are not this wave's

    if (nch > 0) {
        // Software pipeline, all through in-order vector loads: at step P of a trip the chunk
        // c + P is consumed and the gy values of chunk c + P + kDepth are requested; the entries of the
        // next trip are requested at its top, their sample indices are needed from the step on that
        // requests its first chunk.  Order of issue in a trip: the entries, then per step one gy load.
        f4v entry;          // of this lane's chunk: on its way from the top of a trip to its middle
        float prod[4];      // products of the trip's entries, chunk 4 j + i in register i and quad j
        f4v gq[kDepth];
        int n_now, n_nxt;
        load_e(entry, 0);
        landed(entry, std::integral_constant<int, 0>{});
        n_now = row_offset(__float_as_int(entry.w));
        static_for(std::make_integer_sequence<int, kDepth>{}, [&](auto dc) {
            constexpr int d = decltype(dc)::value;
            load_gy(gq[d], std::integral_constant<int, d>{}, n_now);
        });
        // cells of a whole trip are fetched one trip ahead (scalar loads return out of order, so
        // every use waits for all of them: keep them few and early)
        int cells_now[kUnroll], cells_nxt[kUnroll];
#pragma unroll
        for (int p = 0; p < kUnroll; ++p) cells_now[p] = cc[p];
        for (int c = 0; c < nch; c += kUnroll) {
#pragma unroll
            for (int p = 0; p < kUnroll; ++p) cells_nxt[p] = cc[c + kUnroll + p];
            entry_products(entry, l16, prod);
            load_e(entry, c + kUnroll);
            static_for(std::make_integer_sequence<int, kUnroll>{}, [&](auto pc) {
                constexpr int P = decltype(pc)::value;
                const int cell_cur = cells_now[P];
                // Younger loads at this point.  A gy value: the 7 gy loads after it, and the load of entries
                // where the top of a trip lies between.  Entries: the gy loads of the steps since.
                if constexpr (P == kUnroll - kDepth) {
                    landed(entry, std::integral_constant<int, kUnroll - kDepth>{});
                    n_nxt = row_offset(__float_as_int(entry.w));  // first needed below
                }
                landed(gq[P % kDepth], std::integral_constant<int, P < kDepth ? kDepth : kDepth - 1>{});
                if (cell_cur != cur_cell) {
                    if (cur_cell >= 0) leave_cell(acc, ring, cur_cell, cell_cur, lane);
                    retire_before(ring, out, done, cell_cur, lane);
                    cur_cell = cell_cur;
                }
                chunk_fma<P / 4>(acc, prod[P % 4], gq[P % kDepth]);
                load_gy(gq[P % kDepth], std::integral_constant<int, (P + kDepth) % kUnroll>{},
                        P + kDepth < kUnroll ? n_now : n_nxt);
            });
            n_now = n_nxt;
#pragma unroll
            for (int p = 0; p < kUnroll; ++p) cells_now[p] = cells_nxt[p];
        }
        // nothing may still be on its way to a register once the compiler is free to reuse it
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    }
    if (cur_cell >= 0) leave_cell(acc, ring, cur_cell, -1, lane);
    retire_nodes(ring, out, done, run_end<false>(out.own, cur_cell, W), lane);
}

// The nodes that run blockIdx.x + 1 of pair blockIdx.y shares with the runs before it start at zero
template <bool SPARSE>
__global__ __launch_bounds__(256) void clear_shared_nodes_kernel(const int32_t *__restrict__ chunk_cell,
                                                                 const int32_t *__restrict__ block_chunks, int64_t S, int n_sub,
                                                                 int W, float *gP, CoefMap gmap, int n_out)
{
    const int k = blockIdx.y, chunks = block_chunks[k], first = ((int)blockIdx.x + 1) * run_chunks(chunks, n_sub);
    if (first >= chunks) return;
    const int32_t *cell = chunk_cell + (int64_t)k * (S / kChunk) + first;
    // (a group of four nodes of a run is shared as a whole)
    const int beyond = node_beyond<SPARSE>(SPARSE ? last_node<true>(cell[-1], W) : cell[-1], W);
    const int from = max(min(first_node<SPARSE>(cell[0], W), beyond) - 3, 0), to = min(beyond + 3, W * W);
    float *out = gP + (int64_t)k * gmap.s_pair;
    for (int id = from + (int)(threadIdx.x >> 6); id < to; id += 4)
        for (int col = threadIdx.x & 63; col < n_out; col += 64) out[id * gmap.s_node + col] = 0.0f;
}

}  // namespace

size_t sorted_records_bytes(const LayerShape &s)
{
    const size_t S = (size_t)stream_stride(s.batch, s.G);
    const size_t per_pair = S * sizeof(f4v) + (S / kChunk + (size_t)stream_blocks(s.batch)) * sizeof(int32_t);
    return ((size_t)s.pairs() * per_pair + 255) & ~(size_t)255;
}

// The cell-sorted paths index stream positions with 32-bit integers and launch a workgroup per block:
// the longest batch they take.  Longer ones go to the generic kernels.
bool sorted_batch_ok(const LayerShape &s)
{
    return s.batch <= kMaxSortedBatch && stream_stride(s.batch, s.G) < ((int64_t)1 << 31);
}

// gy is gathered four columns at a time and the gradient leaves four columns at a time: with a
// ragged output count gy comes from its tile-by-tile copy and the last columns of the gradient are
// stored one by one, which any 4-byte aligned buffers allow
bool sorted_shape_ok(const LayerShape &s) { return sorted_batch_ok(s); }

bool coef_sorted_applicable(const LayerShape &s, const float *gy, const float *gcoef)
{
    if (!sorted_shape_ok(s)) return false;
    if (ragged_outputs(s)) return true;
    return ((reinterpret_cast<uintptr_t>(gy) | reinterpret_cast<uintptr_t>(gcoef)) & 15) == 0;
}

SortedStream launch_sort(const LayerShape &s, const void *records, void *sorted, bool sparse, hipStream_t stream)
{
    const size_t n = (size_t)s.pairs() * (size_t)s.batch;
    const size_t K = (size_t)s.pairs();
    const int32_t *rec_node = static_cast<const int32_t *>(records);
    const float *rec_u = reinterpret_cast<const float *>(rec_node + n);
    const float *rec_v = rec_u + n;
    SortedStream st;
    st.S = stream_stride(s.batch, s.G);
    st.n_blocks = stream_blocks(s.batch);
    st.block_stride = (int)(stream_block_entries(s.batch, s.G) / kChunk);
    f4v *rec = static_cast<f4v *>(sorted);  // 16-byte items first, then the 4-byte ones
    int32_t *chunk_cell = reinterpret_cast<int32_t *>(rec + K * (size_t)st.S);
    int32_t *block_chunks = chunk_cell + K * (size_t)(st.S / kChunk);
    const size_t lds = sort_lds_bytes(s.G);
    typedef void (*Kernel)(const int32_t *, const float *, const float *, f4v *, int32_t *, int32_t *, int64_t, int);
    const Kernel kernel = sparse ? static_cast<Kernel>(sort_kernel<kHalf>) : static_cast<Kernel>(sort_kernel);
    if (lds > 60 * 1024) allow_large_lds(reinterpret_cast<const void *>(kernel), 160 * 1024 - 256);
    kernel<<<dim3((unsigned)st.n_blocks, (unsigned)K), kSortThreads, lds, stream>>>(
        rec_node, rec_u, rec_v, rec, chunk_cell, block_chunks, s.batch, s.G);
    st.rec = rec;
    st.chunk_cell = chunk_cell;
    st.block_chunks = block_chunks;
    st.sparse = sparse;
    return st;
}

// A gradient of fewer than three million entries is cleared as a whole: where the runs meet is in the stream, two loads
// before the first store (7 MB in 4.2 us, its shared nodes alone in 5.0; 17 MB in 6.1 and 5.3, 147 MB in 19.6 and 7.7).
// Adding all of it atomically then costs the walk 1 us at most, and leaves it in the L2 for who reads it next.  The call for this
// gradient alone, all shared -> nodes owned: 128 -> 96, G = 12, 9000 rows 57.5 -> 60.8 us, 358 -> 61, G = 9, 1827 rows 41.6 -> 42.4;
// training steps of 64 -> 64, G = 8, 4096 rows 53.0 -> 54.0, of 358 -> 61 with the regulariser 112.5 -> 113.2.  Added to a gradient
// that is there, when nothing is cleared: 39.2 -> 39.7, 198 -> 65, G = 15, 3016 rows 52.7 -> 53.9, 128 -> 96 56.4 -> 56.3.
bool all_nodes_shared(const LayerShape &s, int n_blocks, int n_sub)
{
    return n_blocks > 1 || (n_sub > 1 && (size_t)s.nodes() * (size_t)s.pairs() * (size_t)s.n_out < 3000000);
}

void launch_clear_shared_nodes(const LayerShape &s, const SortedStream &st, int n_sub, float *gcoef, hipStream_t stream)
{
    LayerShape g = s;
    g.layout = LMKAN_LAYOUT_PAPER;
    if (all_nodes_shared(s, st.n_blocks, n_sub))
        launch_fill_zero(gcoef, (size_t)s.nodes() * (size_t)s.pairs() * (size_t)s.n_out, stream);
    else if (n_sub > 1)
        (st.sparse ? clear_shared_nodes_kernel<true> : clear_shared_nodes_kernel<false>)<<<dim3((unsigned)(n_sub - 1), (unsigned)s.pairs()), 256, 0, stream>>>(
            st.chunk_cell, st.block_chunks, st.S, n_sub, s.G + 1, gcoef, coef_map(g), s.n_out);
}

void launch_backward_coef_sorted(const LayerShape &s, const SortedStream &st, const GyView &gy, float *gcoef,
                                 bool accumulate, hipStream_t stream)
{
    CoefGradArgs a;
    a.rec = st.rec;
    a.chunk_cell = st.chunk_cell;
    a.block_chunks = st.block_chunks;
    a.block_stride = st.block_stride;
    a.gy = gy;
    a.gP = gcoef;
    LayerShape g = s;
    g.layout = LMKAN_LAYOUT_PAPER;
    a.gmap = coef_map(g);
    a.B = s.batch;
    a.S = st.S;
    a.n_out = s.n_out;
    a.K = s.pairs();
    a.G = s.G;
    a.accumulate = accumulate ? 1 : 0;
    const unsigned lds = node_ring_bytes(s.G);
    const int n_sub = stream_run_split(s);
    a.n_blocks = st.n_blocks;
    a.n_sub = n_sub;
    a.all_shared = all_nodes_shared(s, st.n_blocks, n_sub);
    if (!accumulate) launch_clear_shared_nodes(s, st, n_sub, gcoef, stream);
    const unsigned grid = (unsigned)((int64_t)s.pairs() * s.out_tiles() * st.n_blocks * n_sub);
    KernelTiming timing(stream, kTimeGradCoef);
    if (st.sparse)
        launch_coef_sparse(a, grid, lds, stream);
    else if (gy_offsets_fit_32_bits(s, gy))
        backward_coef_stream_kernel<true><<<grid, 64, lds, stream>>>(a);
    else
        backward_coef_stream_kernel<false><<<grid, 64, lds, stream>>>(a);
}

// Runs per (pair, tile, block).  One block: cut the stream when pairs x tiles cannot fill
// 256 CUs x 16 waves.  Several blocks: as many runs as it takes for the pairs of one (tile,
// block) to occupy an XCD (512 waves), so that the XCD works on one block at a time.  A run
// keeps at least four trips.
// A run of one block shares with its neighbours the nodes of about a row of cells at either end and writes the
// others like an uncut stream (run_nodes), so cutting costs little.  Kernel, uncut / cut in two or four: 3900 streams
// (1300 -> 380) at G = 32 with 10 samples per cell 1008 / 972 us with the clearing, 3072 (768 -> 512) at G = 16 with
// 32 390 / 353, 2450 (700 -> 400) at G = 30 with 3 388 / 337, 2500 (1000 -> 300) at G = 24 with 9 341 / 300, 2048 at
// G = 9 with 100 222 / 205, at G = 28 with 5 309 / 240.  With few samples per cell the shared rows weigh more: 3600 streams
// (900 -> 512) at G = 20 with 4 210 / 217, 3072 at G = 28 with 3 382 / 380; those stay whole.
// (While every node of a cut stream was cleared and added atomically, from 1024 to 2048 streams on were better uncut.)
int stream_run_split(const LayerShape &s)
{
    const int64_t streams = (int64_t)s.pairs() * s.out_tiles();
    int n_sub = 1;
    if (stream_blocks(s.batch) == 1) {
        if (streams >= 3072 && s.batch <= (int64_t)4 * s.G * s.G) return 1;
        const int64_t trips = stream_stride(s.batch, s.G) / (kChunk * kUnroll);
        while (streams * n_sub < 4096 && trips / (n_sub * 2) >= 4 && n_sub < 64) n_sub *= 2;
    } else {
        const int64_t trips = kBlockSamples / (kChunk * kUnroll);
        while ((int64_t)s.pairs() * n_sub < 512 && trips / (n_sub * 2) >= 4 && n_sub < 32) n_sub *= 2;
    }
    return n_sub;
}

// 24-bit multiply and 32-bit byte offsets into gy when the tensor is small enough
bool gy_offsets_fit_32_bits(const LayerShape &s, const GyView &gy)
{
    return s.batch < (1 << 24) && gy.row_stride < (1u << 24) &&
           (int64_t)s.batch * gy.row_stride < ((int64_t)1 << 32);
}

namespace {

// out[t][n][c] = gy[n][64 t + c], zero past n_out; one thread per four columns, threads in the
// order of gy's rows
__global__ __launch_bounds__(256) void gy_tiles_kernel(const float *__restrict__ gy, float *__restrict__ out,
                                                       int64_t B, int n_out, int tiles)
{
    const int64_t per_row = (int64_t)tiles * (kTile / 4);
    const int64_t total = B * per_row;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < total; i += (int64_t)gridDim.x * 256) {
        const int64_t n = i / per_row;
        const int r = (int)(i - n * per_row);
        const int t = r / (kTile / 4), c = (r % (kTile / 4)) * 4;
        const int col = t * kTile + c;
        f4v v = {0.f, 0.f, 0.f, 0.f};
        if ((n_out & 3) == 0) {
            if (col < n_out) v = *reinterpret_cast<const f4v *>(gy + n * n_out + col);
        } else {
            // rows of gy do not start on 16 bytes
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (col + e < n_out) v[e] = gy[n * n_out + col + e];
        }
        *reinterpret_cast<f4v *>(out + ((int64_t)t * B + n) * kTile + c) = v;
    }
}

}  // namespace

// Measured: the copy pays from rows of 8 KiB on (at 4096 outputs the gathers' HBM reads fall from
// 62 GB to 18 GB and the coefficient gradient gains 9 %; at 1024 outputs it costs 2 %).
// A ragged output count needs the copy whatever the width: its rows are padded to whole tiles.
static bool gy_tiles_pay(const LayerShape &s) { return (size_t)s.n_out * sizeof(float) >= 8192 || ragged_outputs(s); }

size_t gy_tiles_bytes(const LayerShape &s)
{
    if (!gy_tiles_pay(s)) return 0;
    return ((size_t)s.out_tiles() * (size_t)s.batch * kTile * sizeof(float) + 255) & ~(size_t)255;
}

GyView launch_gy_tiles(const LayerShape &s, const float *gy, void *tiles, hipStream_t stream)
{
    GyView v;
    if (!gy_tiles_pay(s)) {
        v.base = gy, v.tile_stride = kTile * sizeof(float), v.row_stride = (unsigned)s.n_out * sizeof(float);
        return v;
    }
    const int64_t total = s.batch * (int64_t)s.out_tiles() * (kTile / 4);
    const unsigned grid = (unsigned)std::min<int64_t>((total + 255) / 256, 256 * 32);
    gy_tiles_kernel<<<grid, 256, 0, stream>>>(gy, static_cast<float *>(tiles), s.batch, s.n_out, s.out_tiles());
    v.base = static_cast<const float *>(tiles);
    v.tile_stride = s.batch * (int64_t)(kTile * sizeof(float));
    v.row_stride = kTile * sizeof(float);
    return v;
}

}  // namespace lmkan
