// Pieces shared by the slab-streaming kernels (lmkan_slab.hip, lmkan_slab_f16.hip): kernel
// argument blocks, the LDS-direct load, small DPP helpers.
#pragma once

#include <type_traits>

#include "lmkan_gate.h"
#include "lmkan_kernels.h"
#include "lmkan_split.h"

namespace lmkan {

typedef float f4v __attribute__((ext_vector_type(4)));

constexpr int kSlabTile = LMKAN_PACK_TILE;  // 64 outputs per workgroup tile

struct SlabArgs {
    const void *P;     // float32, or 16-bit storage converted while the slab is filled
    float *y;
    const int32_t *rec_node;
    const float *rec_u;
    const float *rec_v;
    CoefMap map;
    int64_t B;
    int n_out;
    int K;
    int W;             // G + 1
    int nodes;         // W * W
    int col_limit;     // columns >= col_limit do not exist in the coefficient tensor
    int packed;        // 1: packed layout, the slab of (pair, tile) is contiguous
    int pairs_per_split;
    int n_btiles;
    int n_jt;
    int n_split;
    int atomic_out;    // 1: add into y with atomics (split over pairs), 0: plain store
    // Split over pairs without atomics: the workgroups of split 0 store into y, those of split
    // ks > 0 into y_part + (ks - 1) * part_elems, and a later pass adds the parts to y.
    float *y_part;     // NULL: use atomic_out
    int64_t part_elems;
};

// floats between the partial outputs of consecutive pair splits: a whole number of 16-byte pieces
inline int64_t partial_stride(int64_t elems) { return (elems + 3) & ~(int64_t)3; }

// How the splits of a forward launch combine: separate parts when the caller brought room for
// them, atomics on a cleared y otherwise.
inline void finish_split_setup(SlabArgs &a, const LayerShape &s, float *y, float *partials, hipStream_t stream)
{
    a.y_part = a.n_split > 1 ? partials : nullptr;
    a.part_elems = partial_stride((int64_t)s.batch * s.n_out);
    a.atomic_out = a.n_split > 1 && !a.y_part;
    if (a.atomic_out) launch_fill_zero(y, (size_t)s.batch * s.n_out, stream);
}

// four adjacent outputs of a sample leave the registers: one 16-byte store (rows of a ragged output
// count start on 4 bytes only, which such a store allows on this hardware), element by element where
// the row ends before the fourth
__device__ __forceinline__ void store_outputs(float *dst, const float *v, int n_out, int col, bool atomic)
{
    if (atomic) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
            if (col + i < n_out) unsafeAtomicAdd(dst + i, v[i]);
    } else if (col + 4 <= n_out) {
        typedef float f4u __attribute__((ext_vector_type(4), aligned(4)));
        *reinterpret_cast<f4u *>(dst) = f4u{v[0], v[1], v[2], v[3]};
    } else {
#pragma unroll
        for (int i = 0; i < 4; ++i)
            if (col + i < n_out) dst[i] = v[i];
    }
}

// where a forward workgroup of pair split ks stores, and whether it has to add atomically
__device__ __forceinline__ float *forward_out_base(const SlabArgs &a, int ks, bool &atomic)
{
    atomic = a.atomic_out && !a.y_part;
    return (a.y_part && ks > 0) ? a.y_part + (int64_t)(ks - 1) * a.part_elems : a.y;
}

// Tile of this workgroup: consecutive workgroups go to the 8 XCDs in turn, so each XCD is given a
// contiguous run of tiles (those of one slab lie next to each other and share its L2).
__device__ __forceinline__ int xcd_tile()
{
    const int total = gridDim.x, xcd = blockIdx.x & 7, each = total >> 3, over = total & 7;
    return xcd * each + min(xcd, over) + ((int)blockIdx.x >> 3);
}

// Tile of outputs and pair split of workgroup `rest` (workgroups over tiles of samples) of a launch in which the pieces of a row
// that `share` tiles of outputs read lie in one line or two: these tiles lie next to each other as well, so that a line goes to
// one L2.  With the splits next to each other (share = 1) and about as many workgroups for a tile as an XCD has, neighbouring tiles were on
// different XCDs: forward of 256 -> 128, G = 33, 9000 rows 89 -> 81 us; where all of them fit an XCD either way it is the same
// (190 layers drawn, forward, float32 on 16-output tiles: 0.97 of the time in the mean, six of them 1 % slower and more).
__device__ __forceinline__ void place_tile(int share, int rest, int n_split, int n_jt, int &jt, int &ks)
{
    const int group = rest / (share * n_split), width = min(share, n_jt - share * group), in_group = rest - group * share * n_split;
    jt = share * group + in_group % width, ks = in_group / width;
}

__device__ __forceinline__ unsigned lds_address(const void *p)
{
    return (unsigned)(size_t)(__attribute__((address_space(3))) const void *)p;
}

// 16 bytes per lane from global memory (a wave-uniform base and 32 bits of offset per lane) straight into LDS at
// lds_base + lane * 16, for the lanes of `lanes`; none of them is a case too.  Inline assembly on purpose: the
// compiler does not track it, so it cannot make every later LDS read wait for loads that fill the *other* buffer;
// completion is awaited explicitly with s_waitcnt vmcnt(0).  And one statement without a branch the compiler could
// see, so that a fill may stand in the middle of a main loop without cutting it into blocks (each of which would
// be scheduled by itself).  To be used where all lanes of the wave are active.
// m0 is overwritten without being listed as clobbered: it is a reserved register to this
// compiler, which rejects it in a clobber list and never keeps a value in it across
// statements (it sets m0 itself right before any instruction of its own that reads it).
__device__ __forceinline__ void lds_dma16_lanes(const void *gbase, unsigned lane_off, unsigned lds_base, uint64_t lanes)
{
    asm volatile("s_cmp_eq_u64 %3, 0\n\ts_cbranch_scc1 .Labsent%=\n\ts_mov_b32 m0, %2\n\ts_mov_b64 exec, %3\n\t"
                 "global_load_lds_dwordx4 %0, %1\n\ts_mov_b64 exec, -1\n.Labsent%=:"
                 :
                 : "v"(lane_off), "s"(gbase), "s"(lds_base), "s"(lanes)
                 : "memory", "scc");
}

// The same for a chunk of rows of LANES lanes each, however far apart: a load per row, its base row_bytes behind the one
// before.  (The base is counted in fixed registers: 64 bits are added in halves, which an operand cannot name.)
template <int LANES>
__device__ __forceinline__ void lds_dma16_rows(const void *gbase, unsigned lane_off, unsigned lds_base, uint64_t lanes, int64_t row_bytes)
{
    uint64_t left, row;
    asm volatile("s_cmp_eq_u64 %5, 0\n\ts_cbranch_scc1 .Labsent%=\n\ts_mov_b32 m0, %4\n\ts_mov_b64 %0, %5\n\ts_mov_b64 %1, %6\n\t"
                 "s_mov_b64 s[96:97], %3\n.Lrow%=:\n\ts_and_b64 exec, %0, %1\n\tglobal_load_lds_dwordx4 %2, s[96:97]\n\t"
                 "s_andn2_b64 %0, %0, %1\n\ts_cbranch_scc0 .Llast%=\n\ts_lshl_b64 %1, %1, %9\n\t"
                 "s_add_u32 s96, s96, %7\n\ts_addc_u32 s97, s97, %8\n\ts_branch .Lrow%=\n"
                 ".Llast%=:\n\ts_mov_b64 exec, -1\n.Labsent%=:"
                 : "=&s"(left), "=&s"(row)
                 : "v"(lane_off), "s"(gbase), "s"(lds_base), "s"(lanes), "n"((1 << LANES) - 1), "s"((unsigned)row_bytes),
                   "s"((unsigned)((uint64_t)row_bytes >> 32)), "n"(LANES)
                 : "memory", "scc", "s96", "s97");
}

// Four bytes per lane of `lanes` to lds_base + 4 lane: to bring a line into the L2 without a register to receive it
__device__ __forceinline__ void lds_dma4_lanes(const void *gbase, unsigned lane_off, unsigned lds_base, uint64_t lanes)
{
    asm volatile("s_cmp_eq_u64 %3, 0\n\ts_cbranch_scc1 .Labsent%=\n\ts_mov_b32 m0, %2\n\ts_mov_b64 exec, %3\n\t"
                 "global_load_lds_dword %0, %1\n\ts_mov_b64 exec, -1\n.Labsent%=:"
                 :
                 : "v"(lane_off), "s"(gbase), "s"(lds_base), "s"(lanes)
                 : "memory", "scc");
}

// the first n of 64 lanes (n may be zero, negative or more than 64)
__device__ __forceinline__ uint64_t first_lanes(int n)
{
    return n <= 0 ? 0 : n >= 64 ? ~(uint64_t)0 : ((uint64_t)1 << n) - 1;
}

// Slabs of one output tile in the form they are stored in: ROW_BYTES per node, filled by LDS-direct loads of
// 1 KiB (64 lanes x 16 bytes, whole rows), dealt round-robin to the waves.  One code for both layouts: the
// rows of a chunk lie row_bytes apart, columns that do not exist are lanes that never load.  FAR: rows_far_apart.
template <int ROW_BYTES, int WAVES, int MOST_KIB = 80, bool FAR = false>
struct SlabFeed {
    static constexpr int kLanes = ROW_BYTES / 16;   // lanes per row
    static constexpr int kRows = 64 / kLanes;       // rows per chunk
    static constexpr int kMostChunks = (MOST_KIB + WAVES - 1) / WAVES;   // per wave; two slabs share 160 KiB
    const char *tile;
    int64_t pair_bytes, chunk_bytes, row_bytes;
    uint64_t columns;
    unsigned lane_off;
    int nodes, wave;

    template <int ELEMENT>
    __device__ __forceinline__ void init(const void *P, const CoefMap &map, int n_nodes, int col_limit, int first_col, int wave_id,
                                         int lane)
    {
        const int col = first_col + (lane % kLanes) * (16 / ELEMENT);
        tile = static_cast<const char *>(P) + ((int64_t)(first_col >> 6) * map.s_tile + (first_col & 63)) * ELEMENT;
        pair_bytes = map.s_pair * ELEMENT;
        row_bytes = map.s_node * ELEMENT;
        chunk_bytes = row_bytes * kRows;
        lane_off = (FAR ? 0 : (unsigned)(lane / kLanes) * (unsigned)row_bytes) + (unsigned)(lane % kLanes) * 16u;
        columns = __ballot(col < col_limit);
        nodes = n_nodes;
        wave = wave_id;
    }
    __device__ __forceinline__ void issue(unsigned lds_base, int k, bool wanted = true) const
    {
        const char *src = tile + (int64_t)k * pair_bytes;
#pragma unroll
        for (int i = 0; i < kMostChunks; ++i) {
            const int c = wave + i * WAVES;
            const uint64_t lanes = wanted ? first_lanes((nodes - c * kRows) * kLanes) & columns : 0;
            if constexpr (FAR)
                lds_dma16_rows<kLanes>(src + c * chunk_bytes, lane_off, lds_base + c * 1024, lanes, row_bytes);
            else
                lds_dma16_lanes(src + c * chunk_bytes, lane_off, lds_base + c * 1024, lanes);
        }
    }
};

// Layout of Alg. 1: rows lie pairs x outputs elements apart, and the 32 bits of a lane's offset do not reach over a chunk of
// them where that is 3.6e8 or more (float32, four rows a chunk; 7.2e7 with sixteen).  Kernels of their own then load
// row by row: in the others the few scalar instructions more per chunk cost 2 % (a chain of 64-256-256-256-1 on 65536 rows
// 897 -> 917 us).
inline bool rows_far_apart(const LayerShape &s, int rows_per_chunk, int element)
{
    return s.layout != LMKAN_LAYOUT_PACKED &&
           (int64_t)s.pairs() * s.n_out * element * (rows_per_chunk - 1) >= ((int64_t)1 << 32) - 1024;
}
struct FarF32 {   // table type of such a kernel
    float value;
};
template <typename CT>
struct is_far : std::is_same<CT, FarF32> {
};

// The counters of lmkan_gate.h are in LDS.  LDS instructions of a wave execute in order, so a counter moves after the
// reads before it.
// Kernel times with a barrier per pair -> with gate and priorities, 1024 -> 1024, 8192 rows unless stated:
// forward float32 G = 16 945 -> 830 us, G = 20 915 -> 785, G = 28 1293 -> 1130, float16 G = 16 837 -> 750,
// G = 24 910 -> 766, bfloat16 4096 -> 4096 at G = 32, 4096 rows 9100 -> 8130; input gradient float32 G = 16
// 1045 -> 906, G = 20 1377 -> 1167, G = 28 2110 -> 1764; 262144 rows of 128 -> 128, G = 12: 448 -> 425 and
// 570 -> 520.  The gate without the priorities is no gain (994 us instead of 830): the waves that happen to be
// ahead then keep the SIMD until the gate stops them, and the others run alone.
constexpr int kGateBytes = 16;
constexpr int kNowhereBytes = 256;   // what loads for the L2's sake write into

// When a wave does what, in sixteenths of a pair: FILL: the next slab is requested, LANDED: its arrival is waited
// for.  A wave that lags behind gets the SIMD first: its priority falls from quarter to quarter of a pair, and
// steps back up at the start of a pair or (FROM_FILL) at its second quarter, where wait_read has made sure
// that no wave is still in the pair before.
// Which of the two below a kernel takes was measured, all kernels with each (us, early / late; 1024 -> 1024 on 8192 rows unless
// stated).  Early: forward_slab_kernel 815 / 827, forward_lane32_kernel 736 / 750 (float16, G = 24), 114 / 120 (3000 rows of 512 ->
// 512, G = 30), 2022 / 2023 (2048 -> 2048, bfloat16, G = 32).  Late: forward_slab_f16_kernel 861 / 808,
// backward_input_slab_f16_kernel 953 / 905, backward_input_lane32_kernel 1074 / 918 (float16, G = 24) and 1113 / 1077 (bfloat16),
// backward_input_lane32_f32_kernel 1141 / 1110 (G = 20).  Late, though early is no slower: forward_lane32_f32_kernel
// 791 / 810 (G = 20), the 16-output kernels 1090 / 1072 and 1699 / 1725 (forward, input gradient, float32, G = 28).
// backward_input_lane_kernel is late untried: the compiler does not translate its form for rows far apart with early.
template <int FILL, int LANDED, bool FROM_FILL>
struct Pace {
    static constexpr int kFill = FILL, kLanded = LANDED;
    template <int QUARTER>
    static __device__ __forceinline__ void priority()
    {
        __builtin_amdgcn_s_setprio(FROM_FILL ? (4 - QUARTER) % 4 : 3 - QUARTER);
    }
    // for step T of TOTAL
    template <int T, int TOTAL>
    static __device__ __forceinline__ void step_priority()
    {
        if constexpr (T % (TOTAL / 4) == 0) priority<T / (TOTAL / 4)>();
    }
    template <int T, int TOTAL>
    static constexpr bool fill_after = T + 1 == TOTAL * FILL / 16;
    template <int T, int TOTAL>
    static constexpr bool landed_after = T + 1 == TOTAL * LANDED / 16;
};
typedef Pace<4, 12, true> PaceEarly;
typedef Pace<8, 14, false> PaceLate;

struct LdsCounters {
    unsigned landed, read;  // LDS addresses of the counters

    // (a barrier has to follow before the first use)
    __device__ __forceinline__ void init(unsigned lds_addr)
    {
        landed = lds_addr;
        read = lds_addr + 4;
        if (threadIdx.x < 2) *reinterpret_cast<__attribute__((address_space(3))) int *>(lds_addr + threadIdx.x * 4) = 0;
    }
    static __device__ __forceinline__ void arrive(unsigned counter)
    {
        uint64_t exec_before;
        unsigned address, one;   // (set here: nothing of this stays in vector registers over the walk)
        asm volatile("v_mov_b32 %1, %3\n\tv_mov_b32 %2, 1\n\ts_mov_b64 %0, exec\n\ts_mov_b64 exec, 1\n\t"
                     "ds_add_u32 %1, %2\n\ts_mov_b64 exec, %0"
                     : "=&s"(exec_before), "=&v"(address), "=&v"(one)
                     : "s"(counter)
                     : "memory");
    }
    static __device__ __forceinline__ void wait(unsigned counter, int target)
    {
        int v, s;
        asm volatile(".Lpoll%=:\n\tv_mov_b32 %0, %2\n\tds_read_b32 %0, %0\n\ts_waitcnt lgkmcnt(0)\n\t"
                     "v_readfirstlane_b32 %1, %0\n\ts_cmp_ge_i32 %1, %3\n\ts_cbranch_scc1 .Lpassed%=\n\t"
                     "s_sleep 1\n\ts_branch .Lpoll%=\n.Lpassed%=:"
                     : "=&v"(v), "=&s"(s)
                     : "s"(counter), "s"(target)
                     : "memory", "scc");
    }
    __device__ __forceinline__ void arrive_landed() const { arrive(landed); }
    __device__ __forceinline__ void arrive_read() const { arrive(read); }
    __device__ __forceinline__ void until_landed(int n) const { wait(landed, n); }
    __device__ __forceinline__ void until_read(int n) const { wait(read, n); }
    __device__ __forceinline__ void own_landed() const { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }
};
typedef GateOrder<LdsCounters> SlabGate;

// Records of 64 consecutive samples of a pair, from sample n on: scalar base, 32-bit lane offset.  Samples past
// the end of the batch read the record of the last one.  (The limit is kept from the compiler: the offset is
// one instruction, which it would rather keep in a register over the whole walk.)
struct RecordBase {
    int64_t n;
    unsigned last;
    __device__ __forceinline__ RecordBase(int64_t first, int64_t B) : n(min(first, B - 1)), last((unsigned)min((int64_t)63, B - 1 - n)) {}
    __device__ __forceinline__ unsigned lane_index(int lane) const
    {
        unsigned limit = __builtin_amdgcn_readfirstlane(last);
        asm volatile("" : "+s"(limit));
        return min((unsigned)lane, limit);
    }
};

struct GradInArgs {
    const void *P;     // float32, or 16-bit storage converted while the slab is filled
    const float *gy;   // column c of row n at gy[(c >> 6) * gy_tile_stride + n * gy_row_stride + (c & 63)]
    int64_t gy_tile_stride;
    int64_t gy_row_stride;
    float *gx;  // transposed scratch [n_in][ld], zero on entry
    int64_t ld; // row stride of the scratch: B, or B rounded up to 64 with a permuted layout
    const int32_t *rec_node;
    const float *rec_u;
    const float *rec_v;
    CoefMap map;
    GridTab tab;
    int64_t B;
    int n_in;
    int n_out;
    int K;
    int W;
    int nodes;
    int pairs_per_split;
    int n_btiles;
    int n_jt;
    int n_split;
    int col_limit;
    int packed;
    int slab_pitch;    // kernels on the matrix cores: bytes between two grid lines of a slab in LDS
    int tile_share;    // place_tile: the 16-output kernel of float32 tables, the one on the matrix cores
};

// Layouts of a row of the transposed scratch gradient.  The slab kernels leave a set of 64
// samples spread over the lanes so that one atomic instruction holds every other run of 8
// (64-output tiles) or 2 (16-output tiles) samples; stored plainly, the instruction would touch
// 32- or 8-byte pieces with gaps.  Inside each aligned block of 64 samples the row is therefore
// permuted so that each instruction covers 128 contiguous bytes:
//   kScratchOct  (64-output tiles): sample s = 16 g + 8 h + i  sits at 32 h + 8 g + i
//   kScratchQuad (16-output tiles): sample s = 4 g + 2 h + i   sits at 32 h + 2 g + i
// Rows are padded to whole blocks.  The kernels that read the scratch undo the permutation.
enum ScratchLayout { kScratchPlain = 0, kScratchOct = 1, kScratchQuad = 2 };

__host__ __device__ inline int64_t scratch_position(int64_t n, int layout)
{
    if (layout == kScratchPlain) return n;
    const int s = (int)(n & 63);
    const int p = layout == kScratchOct ? ((s & 8) << 2) + ((s >> 4) << 3) + (s & 7)
                                        : ((s & 2) << 4) + ((s >> 2) << 1) + (s & 1);
    return (n & ~(int64_t)63) + p;
}

__host__ __device__ inline int64_t scratch_row_stride(int64_t batch, int layout)
{
    return layout == kScratchPlain ? batch : (batch + 63) & ~(int64_t)63;
}

template <int CTRL>
__device__ __forceinline__ float dpp_move(float v)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, false));
}

// Cross-lane sums of the 64-output input-gradient kernels, in three pieces (see grad_step in
// lmkan_slab.hip).  stage 1, lanes 8 apart: lanes 0-7 of a row keep d/dx1 (t1), lanes 8-15 d/dx2
// (t2).  A DPP add with a bank mask writes only the enabled quarter rows, so no select is needed.
__device__ __forceinline__ float grad_fold_halves(float t1, float t2)
{
    float v;
    asm("v_add_f32_dpp %0, %1, %1 row_ror:8 row_mask:0xf bank_mask:0x3" : "=v"(v) : "v"(t1));
    asm("v_add_f32_dpp %0, %1, %1 row_ror:8 row_mask:0xf bank_mask:0xc" : "+v"(v) : "v"(t2));
    return v;
}

// stage 2, lanes 4 apart: quarter rows 0 and 2 keep the even step (and add what the quarter row
// above holds of it), quarter rows 1 and 3 the odd one
__device__ __forceinline__ float grad_fold_steps(float even, float odd)
{
    float w;
    asm("v_add_f32_dpp %0, %1, %1 row_ror:12 row_mask:0xf bank_mask:0x5" : "=v"(w) : "v"(even));
    asm("v_add_f32_dpp %0, %1, %1 row_ror:4 row_mask:0xf bank_mask:0xa" : "+v"(w) : "v"(odd));
    return w;
}

// stages 3 and 4, lanes 2 and 1 apart: lanes with bit 1 clear keep the first pair of steps
__device__ __forceinline__ float grad_fold_pairs(float first, float second, bool second_half)
{
    const float keep = second_half ? second : first;
    const float send = second_half ? first : second;
    float z = keep + dpp_move<0x4E>(send);  // quad_perm [2,3,0,1]
    z += dpp_move<0xB1>(z);                 // quad_perm [1,0,3,2]
    return z;
}

}  // namespace lmkan
