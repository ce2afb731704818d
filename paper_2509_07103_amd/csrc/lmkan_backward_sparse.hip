// Coefficient gradient of sparse cells: the walk of lmkan_backward.hip over streams whose cells are padded to two samples.
#include "lmkan_kernels.h"
#include "lmkan_sorted.h"

namespace lmkan {

namespace {

constexpr int kTile = LMKAN_PACK_TILE;
constexpr int kDepth = 8;    // chunks of gy values in flight

// Sparse streams: two samples at a time, one per 32-lane half, so that a column's sums meet in one exchange instead of
// two, from half the accumulators, and cells are padded to two samples.  The price are two exchanges per chunk that deal its
// gy values out: of a chunk's four rows, lanes of group g get outputs 2 (g & 1) and 2 (g & 1) + 1 of their column quad,
// for the chunk's first two samples (`first`, one per half) and its last two.
struct HalfRows {
    float first[2], second[2];
};
// position in its chunk of the entry that group g loads: even groups hold the first two samples
__device__ __forceinline__ int half_position(int g) { return (g & 1) * 2 + (g >> 1); }
__device__ __forceinline__ HalfRows deal_out(const f4v &v)
{
    HalfRows p;
#pragma unroll
    for (int o = 0; o < 2; ++o) {
        // odd rows of output o <-> even rows of output o + 2
        const u2v s = __builtin_amdgcn_permlane16_swap(__float_as_uint(v[o]), __float_as_uint(v[o + 2]), false, false);
        p.first[o] = __uint_as_float(s.x);
        p.second[o] = __uint_as_float(s.y);
    }
    return p;
}
// acc[o][q] += (product q of this half's sample) * (its gy value of output 2 (g & 1) + o); the products sit in quad QUAD of
// the half
template <int QUAD>
__device__ __forceinline__ void half_fma(f4v (&acc)[2], float w, const float (&g)[2])
{
    acc[0] = __builtin_amdgcn_mfma_f32_4x4x1f32(w, g[0], acc[0], 3, QUAD, 0);
    acc[1] = __builtin_amdgcn_mfma_f32_4x4x1f32(w, g[1], acc[1], 3, QUAD, 0);
}

// The two rows of a column in one accumulator, summed over the halves of the wave and cleared: lanes 0-31 get row i1's sum,
// lanes 32-63 row i1 + 1's.
// (A wave issues an instruction every four clocks at most, and written with the builtin the compiler assembled the four
// registers anew around every exchange, a dozen copies to a column.  One operand is tied and exchanged in place, the
// other one copied.  What the matrix instructions before left must have arrived: the wait states are the statement's own.)
template <int H>
__device__ __forceinline__ float sum_halves(f4v &acc)
{
    float z, t, zero, x = acc[2 * H];
    const float y = acc[2 * H + 1];
    asm("s_nop 4\n\tv_mov_b32 %1, %3\n\ts_nop 1\n\tv_permlane32_swap_b32 %2, %1\n\tv_add_f32 %0, %2, %1\n\tv_mov_b32 %2, 0"
        : "=&v"(z), "=&v"(t), "+v"(x)
        : "v"(y));
    asm("v_mov_b32 %0, 0" : "=v"(zero));
    acc[2 * H] = x;
    acc[2 * H + 1] = zero;
    return z;
}

// Adds the sums of the column of nodes `id`, id + W (the one with parity H) to the ring and clears its accumulators.
template <int H>
__device__ __forceinline__ void flush_column(f4v (&acc)[2], const NodeRing &ring, int id, int lane)
{
    typedef float f2v __attribute__((ext_vector_type(2)));
    constexpr int kSlotBytes = LMKAN_PACK_TILE * (int)sizeof(float);
    const int lower = ring.slot(id), up = lower < ring.R - ring.W ? ring.W : ring.W - ring.R;  // to the slot of id + W
    const int at = __mul24(lane >> 5, up * kSlotBytes) + (lane & 15) * 16 + ((lane >> 4) & 1) * 8 + lower * kSlotBytes;
    f2v *p = reinterpret_cast<f2v *>(reinterpret_cast<char *>(ring.win) + at);
    f2v v = *p;
    // (an accumulator is one value of four registers here: cleared in part, it is otherwise assembled anew)
#pragma unroll
    for (int i = 0; i < 2; ++i) asm volatile("" : "+v"(acc[i]));
    v.x += sum_halves<H>(acc[0]);
    v.y += sum_halves<H>(acc[1]);
#pragma unroll
    for (int i = 0; i < 2; ++i) asm volatile("" : "+v"(acc[i]));
    *p = v;
}

// The walk leaves the cell with lower node `from` for that with lower node `to` (< 0: it ends).
// (both columns only where the next cell is not its neighbour; one flag word, since the compiler otherwise derives the two
// conditions in a dozen scalar instructions, and no alternatives, which it would give accumulators of their own)
__device__ __forceinline__ void leave_cell(f4v (&acc)[2], const NodeRing &ring, int from, int to, int lane)
{
    const int odd = from & 1;
    int columns = to == from + 1 ? 1 << odd : 3;
    asm volatile("" : "+s"(columns));
    if ((columns & 1) != 0) flush_column<0>(acc, ring, from + odd, lane);
    if ((columns & 2) != 0) flush_column<1>(acc, ring, from + 1 - odd, lane);
}

// What bounds the walk there are the instructions of its waves, not their sum on the
// vector port: a wave issues one every four clocks at most, of whatever kind, and four waves of a SIMD are what LDS has room
// for (dropping the gradient's stores, or gathering one row of gy for all, changes nothing).  At four samples per cell a chunk
// came to 34 vector and 39 scalar instructions and 8 branches, most of them at the end of a cell; here a cell's end is 15
// vector and as many scalar ones.  Trips of eight chunks, since a chunk holds two cell changes and more than 45 KB of code run
// slower than they gain (2048 -> 2048, G = 32, 4096 rows: 3470 us where the walk of whole chunks takes 3880; sixteen chunks, 67 KB, 1 % longer
// than that one).
constexpr int kSparseTrip = 8;

// TRIP: chunks per trip; ROWS4: n_out is a multiple of four
template <int TRIP, bool ROWS4>
__global__ __launch_bounds__(64) void backward_coef_stream_kernel(CoefGradArgs a)
{
    extern __shared__ __align__(16) float win[];  // the NodeRing of this wave's columns
    static_assert(TRIP == kDepth && kUnroll % TRIP == 0, "the ring of gy values is one trip; runs are whole trips");
    const int lane = threadIdx.x;
    const int g = lane >> 4, l16 = lane & 15;
    const int G = a.G, W = G + 1;

    int id = xcd_wave();
    const int sub = id % a.n_sub;
    id /= a.n_sub;
    const int k = id % a.K;
    id /= a.K;
    const int blk = id % a.n_blocks;
    const int jt = id / a.n_blocks;

    const bool col_ok = jt * kTile + l16 * 4 < a.n_out;
    typedef __attribute__((address_space(4))) const int32_t *ScalarIntPtr;
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

    // entries: lane (g, j) fetches that of its group's sample of chunk c + j, eight chunks per load (the upper half of a
    // group repeats the lower one); loads and waits as in lmkan_backward.hip
    const f4v *rec_k = a.rec + (int64_t)k * a.S + (int64_t)c_begin * kChunk;  // wave-uniform
    const unsigned e_off = (unsigned)(((l16 & 7) * kChunk + half_position(g)) * sizeof(f4v));
    auto load_e = [&](f4v &dst, int chunk) {
        const f4v *base = rec_k + (int64_t)chunk * kChunk;
        const unsigned off = e_off;
        asm volatile("global_load_dwordx4 %0, %1, %2" : "=v"(dst) : "v"(off), "s"(base) : "memory");
    };
    auto landed = [](auto &v, auto nc) {
        asm volatile("s_waitcnt vmcnt(%1) ; landed %0" : "+v"(v) : "n"(decltype(nc)::value) : "memory");
    };
    const unsigned col_bytes = col_ok ? (unsigned)l16 * 16u : 0u;
    const unsigned row_bytes = a.gy.row_stride;
    const char *gy_tile = reinterpret_cast<const char *>(a.gy.base) + (int64_t)jt * a.gy.tile_stride;
    // (the batch is short enough for 32-bit offsets: kSparseRows)
    auto row_offset = [&](int n) { return (int)__umul24((unsigned)n, row_bytes); };
    auto load_gy = [&](f4v &dst, auto subc, int off16) {
        const unsigned off = (unsigned)row_bcast<decltype(subc)::value>(off16) + col_bytes;
        const char *base = gy_tile;
        asm volatile("global_load_dwordx4 %0, %1, %2" : "=v"(dst) : "v"(off), "s"(base) : "memory");
    };

    const NodeRing ring(win, W);
    for (int i = lane; i < ring.R * kTile; i += 64) win[i] = 0.0f;
    const RunNodes nodes = run_nodes<true>(cc, nch, sub == 0, last_run, a.all_shared != 0, W);
    const GradOut out{a.gP + (int64_t)k * a.gmap.s_pair + jt * kTile, a.gmap.s_node, jt * kTile, a.n_out, a.accumulate != 0,
                      nodes.own()};

    f4v acc[2];  // [output of half_fma][2 (parity of the column's node) + row]
    acc[0] = acc[1] = f4v{0.f, 0.f, 0.f, 0.f};
    int cur = nch > 0 ? first_node<true>(cc[0], W) : 0;  // lower node of the cell the accumulators belong to
    int done = nodes.begin;  // nodes below have been written, or are not this wave's
    // whole groups of four nodes that are final once the walk stands at `node`
    auto retire_before = [&](int node) {
        if (node - done >= 4) {
            int from = done;  // (`done` itself must stay in a scalar register)
            done += (node - done) & ~3;
            retire_nodes<true, ROWS4>(ring, out, from, done, lane);
        }
    };
    retire_before(cur);  // (the ring has no room for them and for what the first cell adds to)
    auto enter = [&](int node) {
        if (node != cur) {
            leave_cell(acc, ring, cur, node, lane);
            retire_before(node);
            cur = node;
        }
    };

    if (nch > 0) {
        // Order of issue: the entries of the trip after next at the top of a trip, then one gy load per step, eight steps
        // ahead.  So eight loads are younger than a gy value when its step comes, and eight than the entries of the next
        // trip at the top of a trip.
        f4v coming;         // entries of the next trip, on their way until then
        f4v entry = {};     // of this one
        int n_next = 0;     // row offsets of the next trip's samples
        // (wait and copies are one statement: an assignment behind the wait became a copy ahead of it, of registers that the
        // load had not reached)
        auto take = [&](auto nc) {
            const f4v from = coming;
            float x, y, z, w;
            asm volatile("s_waitcnt vmcnt(%9) ; landed %4\n\tv_mov_b32 %0, %5\n\tv_mov_b32 %1, %6\n\tv_mov_b32 %2, %7\n\t"
                         "v_mov_b32 %3, %8"
                         : "=&v"(x), "=&v"(y), "=&v"(z), "=&v"(w)
                         : "v"(from), "v"(from.x), "v"(from.y), "v"(from.z), "v"(from.w), "n"(decltype(nc)::value)
                         : "memory");
            entry = f4v{x, y, z, 0.f};
            n_next = row_offset(__float_as_int(w));
        };
        float prod[4];
        f4v gq[kDepth];
        load_e(coming, 0);
        take(std::integral_constant<int, 0>{});
        load_e(coming, TRIP);
        static_for(std::make_integer_sequence<int, kDepth>{}, [&](auto dc) {
            constexpr int d = decltype(dc)::value;
            load_gy(gq[d], std::integral_constant<int, d>{}, n_next);
        });
        int cells_now[TRIP], cells_nxt[TRIP];
#pragma unroll
        for (int p = 0; p < TRIP; ++p) cells_now[p] = cc[p];
        for (int c = 0; c < nch; c += TRIP) {
#pragma unroll
            for (int p = 0; p < TRIP; ++p) cells_nxt[p] = cc[c + TRIP + p];
            entry_products(entry, l16, prod);
            take(std::integral_constant<int, kDepth>{});
            load_e(coming, c + 2 * TRIP);
            static_for(std::make_integer_sequence<int, TRIP>{}, [&](auto pc) {
                constexpr int P = decltype(pc)::value;
                landed(gq[P], std::integral_constant<int, kDepth>{});
                const HalfRows rows = deal_out(gq[P]);
                enter(first_node<true>(cells_now[P], W));
                half_fma<P / 4>(acc, prod[P % 4], rows.first);
                enter(last_node<true>(cells_now[P], W));
                half_fma<4 + P / 4>(acc, prod[P % 4], rows.second);
                load_gy(gq[P], pc, n_next);
            });
#pragma unroll
            for (int p = 0; p < TRIP; ++p) cells_now[p] = cells_nxt[p];
        }
        // nothing may still be on its way to a register once the compiler is free to reuse it
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        leave_cell(acc, ring, cur, -1, lane);
    }
    retire_nodes(ring, out, done, run_end<true>(out.own, cur, W), lane);
}

}  // namespace

// Few samples per cell, of a block: the end of a cell outweighs what its chunks pay for it.  Calls for this gradient alone, layers
// drawn, the walk of whole chunks / this one, us:
// - Streams uncut or cut in two or four: 930 -> 966, G = 8, 285 rows (4.5 per cell) 101 / 90 us, 512 -> 512, G = 24, 3455 rows (6) 204 / 192,
//   502 -> 297, G = 17, 1854 rows (6.4) 115 / 98 (up to G = 26 five waves of this walk find room on a SIMD, four of the other);
//   from seven samples on even or the other way (1000 -> 356, G = 13, 1345 rows (8) 127 / 132).
// - The more runs, the fewer samples each has beside the row of cells it shares with its neighbours: in eight 136 -> 570, G = 21, 2449
//   rows (5.6) 106 / 97, but 244 -> 82, G = 17, 2005 rows (6.9) 56 / 58; in sixteen 112 -> 446, G = 45, 5192 rows (2.6) 240 / 236, but
//   272 -> 69, G = 36, 9059 rows (7) 148 / 156; in 32 40 -> 643, G = 43, 5472 rows (3) 212 / 182, but 62 -> 238, G = 35, 5443 rows (4.4) 112 / 123.
// - Where every node is added to, of a small gradient or of several blocks, even to 8 % more (84 -> 33, G = 25, 2925 rows 52 / 56), but for
//   streams of several blocks of four samples per cell at most in few runs (258 -> 26, G = 61, 23701 rows 454 / 420).
// Over 520 layers: 0.988 of the time in the mean, 20 of them 1 % slower and more, 8 % at most (fewer than seven samples of the whole
// batch per cell, whatever the runs: 0.997, 145, 20 %).
constexpr int64_t kSparseRows = 1 << 18;   // rows of gy lie less than 8 KB apart (gy_tiles_pay): offsets of 31 bits
bool coef_stream_is_sparse(const LayerShape &s)
{
    const int64_t cells = (int64_t)s.G * s.G;
    const int n_sub = stream_run_split(s);
    if (s.batch > kSparseRows) return false;
    if (stream_blocks(s.batch) > 1) return n_sub <= 8 && kBlockSamples < 4 * cells;
    if (all_nodes_shared(s, 1, n_sub)) return false;
    const int quarters = 32 - 3 * __builtin_ctz((unsigned)n_sub);   // of a sample per cell; runs are powers of two
    return 4 * s.batch < (quarters < 28 ? quarters : 28) * cells;
}

void launch_coef_sparse(const CoefGradArgs &a, unsigned waves, unsigned lds, hipStream_t stream)
{
    (a.n_out % 4 == 0 ? backward_coef_stream_kernel<kSparseTrip, true> : backward_coef_stream_kernel<kSparseTrip, false>)<<<waves, 64, lds, stream>>>(a);
}

}  // namespace lmkan
