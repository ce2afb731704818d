// Input gradient of bfloat16 tables on the matrix cores, for the kernels that stream slabs.
//
//   s_c(n, k) = sum_j gy[n][j] P[corner c of the cell of (n, k)][j],   c = 00, 01, 10, 11
//
// is four dot products of a sample: a 4 x TILE matrix times a vector.  A 4x4x4 MFMA multiplies sixteen
// such matrices at once, four outputs deep, but by four columns each, and a sample has one vector.  It is
// given as four: gy split into parts of six significant bits whose sum is gy to the last bit, so that the table needs no
// conversion (the vector pipe spends one beside every multiply-add).  Per instruction 256 multiply-adds
// are of use, in about 9 clocks.
//
// Products of such a part have 14 bits, and sums of eight of them mostly fit float32 without rounding, which is
// what the derivatives ask for: they are differences of neighbouring corners, which agree in most of their digits where a
// table is smooth.  Relative error, 256 -> 256 at G = 24, of tables that are independent from node to node, affine, 2 % apart
// with either sign, 2 % apart with one sign (and a gy of one sign): 9.3e-8, 1.0e-7, 3.4e-7, 3.5e-7; with three parts of
// eight bits and differences every 32 outputs 9.8e-8, 3.1e-7, 1.6e-6, 5.1e-6; on the vector pipe with differences
// every eight outputs 1.1e-7, 5.1e-7, 2.6e-6, 5.2e-6 (every four, G = 16: 1.0e-7, 2.7e-7, 2.0e-6, 2.9e-6).
//
// Lane 4 b + i of a wave reads corner i of sample b as it lies in LDS (16 bytes = 8 outputs = the A operands of two
// MFMAs) and holds part i of that sample's gy (B operand, resident); it receives the sums of part i with all
// four corners.  64 samples of a wave are four sets: sample 4 b + t is block b of set t, so whatever a lane
// has of sample `lane` reaches the four lanes of a block by the DPP broadcast within a quad, and the sums of
// four sets over the parts leave sample `lane` in lane `lane` (a 4 x 4 transposition on the way).
//
// Sixteen lanes read at once: four samples, four corners.  Samples take pieces of their rows in different
// orders (piece j ^ (b & 3) at step j), the corners of one sample lie in different quarters of the banks because
// of the pitch of a grid line in LDS (split_pitch): no two of the sixteen meet on a bank.
#pragma once

#include "lmkan_slab_common.h"

namespace lmkan {

// bytes between two grid lines of a slab in LDS: 128 modulo 256
inline int split_pitch(int W, int row_bytes)
{
    const int line = W * row_bytes;
    return line + ((128 - line) & 255);
}

typedef unsigned u4v __attribute__((ext_vector_type(4)));

typedef unsigned u2v __attribute__((ext_vector_type(2)));

template <typename V>
__device__ __forceinline__ V low_half(u4v v)
{
    return __builtin_bit_cast(V, u2v{v[0], v[1]});
}
template <typename V>
__device__ __forceinline__ V high_half(u4v v)
{
    return __builtin_bit_cast(V, u2v{v[2], v[3]});
}

// gy in four parts of six significant bits, cut off and not rounded; the exponent range is float32's.  of(): a part
// of one value, whatever it is (an infinity or NaN in part 0, zero in the others, so that its products are those of
// the value).  SplitPart: the same for two finite values at a time in few instructions, its constants chosen by the
// lane's part.
struct SplitPart {
    typedef short Vec __attribute__((ext_vector_type(4)));
    static constexpr unsigned kSixBits = 0xfffc0000u;   // of a float32
    static __device__ __forceinline__ unsigned of(float g, int part)
    {
        const bool finite = fabsf(g) < __builtin_inff();
        const unsigned split = SplitPart(part).pair(finite ? g : 0.0f, 0.0f), whole = g != g ? 0x7fc0u : __float_as_uint(g) >> 16;
        return finite ? split & 0xffffu : part == 0 ? whole : 0u;
    }
    unsigned cut1, cut2, cut3, keep;
    explicit __device__ __forceinline__ SplitPart(int part)
        : cut1(part >= 1 ? kSixBits : 0u), cut2(part >= 2 ? kSixBits : 0u), cut3(part >= 3 ? kSixBits : 0u), keep(part < 3 ? 0xfffcfffcu : ~0u)
    {
    }
    __device__ __forceinline__ unsigned pair(float g0, float g1) const
    {
        auto next = [&](unsigned cut) {
            g0 -= __uint_as_float(__float_as_uint(g0) & cut);
            g1 -= __uint_as_float(__float_as_uint(g1) & cut);
        };
        next(cut1), next(cut2), next(cut3);
        return __builtin_amdgcn_perm(__float_as_uint(g1), __float_as_uint(g0), 0x07060302u) & keep;
    }
    static __device__ __forceinline__ void mac(f4v &d, Vec a, Vec b, bool first)
    {
        d = __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(a, b, first ? f4v{0.f, 0.f, 0.f, 0.f} : d, 0, 0, 0);
    }
};

// (w of lane T of this quad) * x, and the same added to acc
template <int T>
__device__ __forceinline__ float split_mul_bcast(float w, float x)
{
    float d;
    asm("v_mul_f32_dpp %0, %1, %2 quad_perm:[%3,%3,%3,%3] row_mask:0xf bank_mask:0xf" : "=v"(d) : "v"(w), "v"(x), "n"(T));
    return d;
}

template <int T>
__device__ __forceinline__ void split_fmac_bcast(float &acc, float w, float x)
{
    asm("v_fmac_f32_dpp %0, %1, %2 quad_perm:[%3,%3,%3,%3] row_mask:0xf bank_mask:0xf" : "+v"(acc) : "v"(w), "v"(x), "n"(T));
}

// lanes with the bit keep b and pass a on, the others keep a and pass b on; XOR: DPP control of the exchange
template <int XOR>
__device__ __forceinline__ float split_exchange(float a, float b, bool bit)
{
    const float keep = bit ? b : a;
    const float send = bit ? a : b;
    return keep + dpp_move<XOR>(send);
}

// The derivatives of the samples in `rows` (bits: lanes) by float32 products, lane j its output of the tile.  An infinite
// entry of the table meets the zeros among the parts of gy and makes the sums above NaN; here it gives the infinity,
// or NaN, that the products themselves give.  gy: first sample of the wave; off, b_lo ... a_hi: as in the walk, of a
// lane's own sample.
__device__ __forceinline__ void split_again(uint64_t rows, const float *gy, int64_t gy_row_stride, int columns, int lane, int off, int pitch,
                                            int row_bytes, float b_lo, float b_hi, float a_lo, float a_hi, float &d1, float &d2)
{
    typedef __attribute__((address_space(3))) const unsigned short *LdsHalf;
    auto of_row = [](float v, int s) { return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), s)); };
#pragma unroll 1
    for (; rows; rows &= rows - 1) {
        const int s = __builtin_ctzll(rows);
        float p[4] = {0.f, 0.f, 0.f, 0.f};
        if (lane < columns) {
            const float g = gy[s * gy_row_stride + lane];
            const unsigned at = (unsigned)__builtin_amdgcn_readlane(off, s) + (unsigned)lane * 2u;
#pragma unroll
            for (int c = 0; c < 4; ++c)
                p[c] = g * __uint_as_float((unsigned)*reinterpret_cast<LdsHalf>(at + (c >> 1) * pitch + (c & 1) * row_bytes) << 16);
        }
        float dif[4] = {p[2] - p[0], p[3] - p[1], p[1] - p[0], p[3] - p[2]};
#pragma unroll
        for (int c = 0; c < 4; ++c)
            for (int apart = 32; apart > 0; apart >>= 1) dif[c] += __shfl_xor(dif[c], apart);
        const float e1 = fmaf(of_row(b_hi, s), dif[1], of_row(b_lo, s) * dif[0]);
        const float e2 = fmaf(of_row(a_hi, s), dif[3], of_row(a_lo, s) * dif[2]);
        if (lane == s) d1 = e1, d2 = e2;
    }
}

// WAVES x 64 samples, TILE outputs (a tile of the packed layout or half of one) per workgroup, slabs of at most SLAB_KIB
template <int TILE, int WAVES, int SLAB_KIB>
__device__ __forceinline__ void backward_input_split(const GradInArgs &a, char *smem)
{
    typedef SplitPart Part;
    typedef Part::Vec Vec;
    typedef PaceLate PACE;   // (its priorities; the fill is spread, see below)
    constexpr int kTileBytes = kSlabTile * 2, kRowB = TILE * 2, kPieces = TILE / 8, kSets = 4, kSteps = kSets * kPieces;
    constexpr int kAhead = 3;                              // LDS reads in flight
    constexpr int kChunks = (SLAB_KIB + WAVES - 1) / WAVES;  // 1 KiB pieces of a slab per wave
    // What bounds this kernel is the fill: a slab serves half the samples that it serves in the forward kernel
    // (four parts of gy take twice the registers of float32).  So the pieces of the next
    // slab are requested one by one over half of a pair, and the lines of the slab after that are brought into the
    // L2 by loads of one word per row.  2048 -> 2048, G = 32, 4096 rows: 3005 us with the fill in one
    // place, 2840 spread, 2600 prefetched, 2500 both (1390 without any fill);
    // with differences every eight outputs 2610.
    constexpr int kFillStep = kSteps / 4 - 1, kFillEvery = kSteps / 8, kLandedStep = kSteps * 7 / 8 - 1;
    static_assert(kFillStep + (kChunks - 1) * kFillEvery < kLandedStep, "the last piece is requested before it is awaited");
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int part = lane & 3, block = lane >> 2, q = block & 3;
    const int W = a.W, pitch = a.slab_pitch;
    const int id = xcd_tile();
    const int btile = id % a.n_btiles;
    const int rest = id / a.n_btiles;
    int ks, jt;
    place_tile(a.tile_share, rest, a.n_split, a.n_jt, jt, ks);
    const int k_begin = ks * a.pairs_per_split;
    const int k_end = min(a.K, k_begin + a.pairs_per_split);
    if (k_begin >= k_end) return;

    // LDS: two slabs, 1/h of the grid, the gate, 256 bytes that nobody reads
    const unsigned slab_bytes = (unsigned)(W * pitch);
    const unsigned base0 = __builtin_amdgcn_readfirstlane(lds_address(smem));
    float *s_invh = reinterpret_cast<float *>(smem + 2 * slab_bytes);
    for (int i = threadIdx.x; i < a.tab.G; i += WAVES * 64) s_invh[i] = a.tab.inv_h[i];
    SlabGate gate;
    gate.init(base0 + 2 * slab_bytes + LMKAN_MAX_GRID * 4);

    // what this lane fetches of a slab: 16 bytes of every chunk, from the node and piece they belong to
    const int first_col = jt * TILE;
    const char *tile = static_cast<const char *>(a.P) + ((int64_t)(first_col >> 6) * a.map.s_tile + (first_col & 63)) * 2;
    unsigned from[kChunks];
    uint64_t lanes[kChunks];
#pragma unroll
    for (int i = 0; i < kChunks; ++i) {
        const int byte = (wave + i * WAVES) * 1024 + lane * 16;
        const int i1 = byte / pitch, in_line = byte - i1 * pitch;
        const int i2 = min(in_line / kRowB, W - 1), piece = (in_line % kRowB) >> 4;
        from[i] = (unsigned)(i1 * W + i2) * (unsigned)(a.map.s_node * 2) + (unsigned)piece * 16u;
        lanes[i] = __ballot(i1 < W && first_col + piece * 8 < a.col_limit);
    }
    auto issue_piece = [&](int i, unsigned lds_base, int k, bool wanted) {
        lds_dma16_lanes(tile + (int64_t)k * a.map.s_pair * 2, from[i], lds_base + (wave + i * WAVES) * 1024, wanted ? lanes[i] : 0);
    };
    // one word of every row of pair k's slab (a row of the packed layout is a line of the L2), dealt to the workgroups that stream it
    const int share = a.n_btiles >= 4 ? 3 : a.n_btiles >= 2 ? 1 : 0;
    const unsigned nowhere = base0 + 2 * slab_bytes + LMKAN_MAX_GRID * 4 + kGateBytes;
    auto prefetch = [&](int k, bool wanted) {
        const char *src = tile + (int64_t)k * a.map.s_pair * 2;
#pragma unroll
        for (int i = 0; i < (SLAB_KIB * 1024 / kRowB + WAVES * 64 - 1) / (WAVES * 64); ++i) {
            const int row = (wave + i * WAVES) * 64;
            lds_dma4_lanes(src + row * kTileBytes, (unsigned)lane * kTileBytes, nowhere,
                           wanted && (wave & share) == (btile & share) ? first_lanes(W * W - row) : 0);
        }
    };

    __syncthreads();  // s_invh and the counters in place before any slab load lands
#pragma unroll
    for (int i = 0; i < kChunks; ++i) issue_piece(i, base0, k_begin, true);
    prefetch(k_begin + 1, k_begin + 1 < k_end);

    const int64_t n_wave = (int64_t)btile * (WAVES * 64) + wave * 64;
    // part `part` of gy of sample n_wave + 4 block + t, outputs first_col + 8 (j ^ q) ... + 7
    u4v gyr[kSets][kPieces];
    bool nan_in_gy = false;   // of sample n_wave + lane
    static_for(std::make_integer_sequence<int, kSets>{}, [&](auto tc) {
        constexpr int t = decltype(tc)::value;
        const float *row = a.gy + min(n_wave + block * 4 + t, a.B - 1) * a.gy_row_stride + (int64_t)(first_col >> 6) * a.gy_tile_stride;
        // (never skipped: what does not exist is read as something that does; samples past the batch are not stored,
        // columns are zeroed)
        float g[kPieces][8];
#pragma unroll
        for (int j = 0; j < kPieces; ++j) {
            const int col = first_col + (j ^ q) * 8;
            const float4 lo = *reinterpret_cast<const float4 *>(row + (col < a.n_out ? col & 63 : first_col & 63));
            const float4 hi = *reinterpret_cast<const float4 *>(row + (col + 4 < a.n_out ? (col & 63) + 4 : first_col & 63));
            g[j][0] = lo.x, g[j][1] = lo.y, g[j][2] = lo.z, g[j][3] = lo.w;
            g[j][4] = hi.x, g[j][5] = hi.y, g[j][6] = hi.z, g[j][7] = hi.w;
        }
        float total = 0.0f;   // of |gy|: not finite where one of them is not
#pragma unroll
        for (int j = 0; j < kPieces; ++j)
#pragma unroll
            for (int i = 0; i < 8; ++i) total += fabsf(g[j][i]);
        const bool finite = total < __builtin_inff();
        if (part == t) nan_in_gy = total != total;
        const Part split(part);
        if (__all(finite)) {
#pragma unroll
            for (int j = 0; j < kPieces; ++j)
#pragma unroll
                for (int i = 0; i < 4; ++i) gyr[t][j][i] = split.pair(g[j][2 * i], g[j][2 * i + 1]);
        } else {
#pragma unroll
            for (int j = 0; j < kPieces; ++j)
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    gyr[t][j][i] = Part::of(g[j][2 * i], part) | Part::of(g[j][2 * i + 1], part) << 16;
        }
#pragma unroll
        for (int j = 0; j < kPieces; ++j) {
            const int col = first_col + (j ^ q) * 8;
            if (col >= a.n_out) gyr[t][j] = u4v{0u, 0u, 0u, 0u};
            if (col + 4 >= a.n_out) gyr[t][j][2] = gyr[t][j][3] = 0u;
        }
        // (one set at a time: the loads of all would be spilled)
#pragma unroll
        for (int j = 0; j < kPieces; ++j) asm volatile("" : "+v"(gyr[t][j]) : : "memory");
    });

    int nx_node = 0;
    float nx_u = 0.f, nx_v = 0.f;
    auto fetch_record = [&](int k) {
        const RecordBase rb(n_wave, a.B);
        const int64_t o = (int64_t)k * a.B + rb.n;
        const unsigned l = rb.lane_index(lane);
        nx_node = (a.rec_node + o)[l];
        nx_u = (a.rec_u + o)[l];
        nx_v = (a.rec_v + o)[l];
    };
    fetch_record(k_begin);
    gate.slab_landed();

    if (n_wave >= a.B) {
        gate.feed_only<WAVES>(k_end - k_begin, [&](int i, bool wanted) {
#pragma unroll
            for (int c = 0; c < kChunks; ++c) issue_piece(c, i & 1 ? base0 + slab_bytes : base0, k_begin + i, wanted);
            prefetch(k_begin + i + 1, k_begin + i + 1 < k_end);
        });
        return;
    }
    const bool valid = n_wave + lane < a.B;
    const float inv_w = 1.0f / (float)W;
    float *gx_wave = a.gx + n_wave;   // transposed scratch [n_in][ld], plain layout
    unsigned piece_off[kPieces];      // of corner `part` and the piece read at step j
#pragma unroll
    for (int j = 0; j < kPieces; ++j) piece_off[j] = (unsigned)((part >> 1) * pitch + (part & 1) * kRowB + (j ^ q) * 16);

    auto add_derivatives = [&](int k, float d1, float d2) {
        if (valid) {
            float *dst = gx_wave + (int64_t)(2 * k) * a.ld;
            unsafeAtomicAdd(dst + (unsigned)lane, d1);
            unsafeAtomicAdd(dst + a.ld + (unsigned)lane, d2);
        }
    };
    for (int k = k_begin; k < k_end; ++k) {
        const int step = k - k_begin;
        const bool more = k + 1 < k_end;
        const unsigned cur = (step & 1) ? base0 + slab_bytes : base0;
        const unsigned nxt = (step & 1) ? base0 : base0 + slab_bytes;
        const int i1 = (int)(((float)nx_node + 0.5f) * inv_w), i2 = nx_node - i1 * W;   // exact for these sizes
        const float rh1 = s_invh[i1], rh2 = s_invh[i2];
        int off = (int)cur + i1 * pitch + i2 * kRowB;
        float b_lo = (1.0f - nx_v) * rh1, b_hi = nx_v * rh1, a_lo = (1.0f - nx_u) * rh2, a_hi = nx_u * rh2;
        // VALU results must not be read through DPP in the next two issue slots
        asm volatile("s_nop 1" : "+v"(b_lo), "+v"(b_hi), "+v"(a_lo), "+v"(a_hi), "+v"(off));
        gate.wait_landed<WAVES>(step);

        u4v ring[kAhead + 1];
        auto request = [&](auto sc) {
            constexpr int s = decltype(sc)::value, t = s / kPieces, j = s % kPieces;
            const unsigned row = (unsigned)__builtin_amdgcn_update_dpp(0, off, t * 0x55, 0xf, 0xf, true);
            ring[s % (kAhead + 1)] = *reinterpret_cast<__attribute__((address_space(3))) const u4v *>(row + piece_off[j]);
        };
        static_for(std::make_integer_sequence<int, kAhead>{}, request);
        f4v d = {0.f, 0.f, 0.f, 0.f};
        float dif_a = 0.f, dif_b = 0.f, dif_c = 0.f, dif_d = 0.f;
        float x1 = 0.f, x2 = 0.f, y1 = 0.f, y2 = 0.f;   // derivatives of the set and of the pair of sets before
        float d1 = 0.f, d2 = 0.f;
        static_for(std::make_integer_sequence<int, kSteps>{}, [&](auto sc) {
            constexpr int s = decltype(sc)::value, t = s / kPieces, j = s % kPieces;
            PACE::step_priority<s, kSteps>();
            u4v p = ring[s % (kAhead + 1)];
            // (the empty statements keep a step's read and its products in their place: without them the compiler
            // requests all of a pair's pieces, halves of a piece apart, and spills them)
            asm volatile("" : "+v"(off), "+v"(p));
            if constexpr (s + kAhead < kSteps) request(std::integral_constant<int, s + kAhead>{});
            Part::mac(d, low_half<Vec>(p), low_half<Vec>(gyr[t][j]), true);
            Part::mac(d, high_half<Vec>(p), high_half<Vec>(gyr[t][j]), false);
            asm volatile("" : "+v"(off), "+v"(d));
            // d[0 ... 3]: this part's sums of eight outputs with corners 00, 01, 10, 11
            if constexpr (j == 0)
                dif_a = d[2] - d[0], dif_b = d[3] - d[1], dif_c = d[1] - d[0], dif_d = d[3] - d[2];
            else
                dif_a += d[2] - d[0], dif_b += d[3] - d[1], dif_c += d[1] - d[0], dif_d += d[3] - d[2];
            if constexpr (j == kPieces - 1) {
                float t1 = split_mul_bcast<t>(b_lo, dif_a), t2 = split_mul_bcast<t>(a_lo, dif_c);
                split_fmac_bcast<t>(t1, b_hi, dif_b);
                split_fmac_bcast<t>(t2, a_hi, dif_d);
                if constexpr ((t & 1) == 0) {
                    x1 = t1, x2 = t2;
                } else {
                    const float z1 = split_exchange<0xB1>(x1, t1, lane & 1), z2 = split_exchange<0xB1>(x2, t2, lane & 1);
                    if constexpr (t == 1) {
                        y1 = z1, y2 = z2;
                    } else {
                        d1 = split_exchange<0x4E>(y1, z1, lane & 2), d2 = split_exchange<0x4E>(y2, z2, lane & 2);
                    }
                }
            }
            if constexpr (s == kFillStep) {
                gate.wait_read<WAVES>(step);
                fetch_record(more ? k + 1 : k);
            }
            if constexpr (s >= kFillStep && (s - kFillStep) % kFillEvery == 0 && (s - kFillStep) / kFillEvery < kChunks)
                issue_piece((s - kFillStep) / kFillEvery, nxt, k + 1, more);
            if constexpr (s == kLandedStep) {
                gate.slab_landed();
                prefetch(k + 2, k + 2 < k_end);
            }
        });
        const uint64_t again = __ballot(valid && !nan_in_gy && (d1 != d1 || d2 != d2));
        if (again)
            split_again(again, a.gy + n_wave * a.gy_row_stride + (int64_t)(first_col >> 6) * a.gy_tile_stride + (first_col & 63), a.gy_row_stride,
                        min(TILE, a.n_out - first_col), lane, off, pitch, kRowB, b_lo, b_hi, a_lo, a_hi, d1, d2);
        gate.slab_read();
        add_derivatives(k, d1, d2);
    }
}

}  // namespace lmkan
