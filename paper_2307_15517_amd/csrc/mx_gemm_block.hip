// MXInt x MXInt product on the integer matrix cores of gfx950, operands in the fragment layout.
//
// Arithmetic (Section 3.2 of the paper, the MXInt dot-product operator): per K-block the mantissa
// products are summed exactly in int32 by one MFMA whose K extent equals the block (32x32x16 for
// block 16, 32x32x32 for block 32, two chained 32x32x32 for block 64); the block's value is that
// integer times 2^(Ea + Eb - (wa-2) - (wb-2)), applied with v_ldexp_f32 and added into an fp32
// accumulator.  The left operand feeds the MFMA "A" side, so in the 32x32 result a lane owns one
// output column n and its 16 registers are 16 rows m: the right operand's block exponent is one
// value per lane, the left operand's is one value per register.
#include <type_traits>

#include "mx_gemm.h"
#include "mx_frag.h"

#ifndef MX_GEMM_BLOCK
#error "compile with -DMX_GEMM_BLOCK=16, 32 or 64"
#endif

namespace mx {
namespace {

typedef v4i_t v4i;
typedef v16i_t v16i;

// ------------------------------------------------------------------------------------------------
// General kernel (M > 8): a workgroup of NW waves owns one 32 x 32 tile of Y, its waves take the K chunks
// round-robin and their partial tiles are added through LDS at the end.  Fragments come straight from global
// memory in lane order, one chunk ahead of the arithmetic.
//
// Bound: vector instruction issue (13824 -> 5120 at 32 rows, 8 by 4 bits, blocks of 16: 24.0 us on the 160 compute units that
// have a tile, whose vector ALUs are active 82 % of their cycles; 75 % at 5120 -> 13824).  Every block of 32 x 32 outputs costs one MFMA (two for block 64) and 16 block sums per lane, each of which
// is scaled and added.  When all block exponents of the chunk lie within [-31, 32] that is two multiply-adds: the sums come
// out of the matrix instruction as floats with a bias (dot_bias), the first takes the bias off and applies the row's
// scale, exactly, the second applies the column's scale and adds.  With a conversion, an integer add for the scale and one
// multiply-add it took 26.9 us (32 x 5120 x 5120 13.3 -> 12.4; 6 by 5 bits 35.6 -> 30.0), as it still does where the bias's
// registers would cost a wave per SIMD (blocks of 64, of 32 with few bits, wide operands).  Otherwise (also for zero blocks,
// whose byte is 0) it is done with ldexp, four instructions.  The row scales and what takes the bias off go through LDS,
// because a lane needs those of 16 rows.
// Waves split K rather than owning larger tiles because the products that arrive here are short in M (the batch of a
// decode step, a short prompt): a 128 x 128 tile per workgroup left most of the chip idle, and the K loop of one wave
// is a serial chain of loads, matrix instructions and scaling.
// ------------------------------------------------------------------------------------------------
// Block sums with a bias where its sixteen registers leave the kernel its waves per SIMD: four with blocks of 16, three with
// blocks of 32, and four without it where both operands are narrow (tests/test_kernel_resources.py holds the built kernels to
// this).
constexpr bool biased_sums(int wa, int wb, int block) {
    return block == 16 ? wa + wb <= (wb == 8 ? 13 : 14) : block == 32 && wa + wb >= 9 && wa + wb <= 14;
}
// LDS of a wave for the rows' exponents, or with the bias for their scales and what takes it off.
constexpr size_t scale_lds(bool biased) { return biased ? 1024 : 512; }

template <int WA, int WB, int B>
__global__ __launch_bounds__(B >= 32 ? 512 : 1024) void gemm_tile_kernel(GemmArgs g) {
    constexpr int kDwA = Piece<WA, B>::kDw, kDwB = Piece<WB, B>::kDw;
    constexpr int kHalfDw = B / 8;       // int8 dwords per lane per block
    constexpr int D = 2 * (kDwA + kDwB + 2) <= 64 ? 2 : 1;               // chunks in registers
    constexpr bool BIASED = biased_sums(WA, WB, B);
    extern __shared__ __attribute__((aligned(16))) uint32_t lds[];       // xe[NW][1 or 2][4][32], red[NW/2][16][64]
    const int nw = (int)blockDim.x >> 6;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int i = lane & 31, h = lane >> 5;
    // workgroup n runs on XCD n % 8: an XCD gets a contiguous range of tiles, row tiles fastest, so that the workgroups
    // that read one column group's records do so behind one L2
    const int64_t total = g.groupsA * g.groupsB, per_xcd = (total + 7) / 8;
    const int64_t lin = (blockIdx.x % 8) * per_xcd + blockIdx.x / 8;
    if (blockIdx.x / 8 >= per_xcd || lin >= total) return;               // whole workgroup, before any barrier
    const int64_t gb = lin / g.groupsA, ga = lin - gb * g.groupsA;
    const int64_t bz = blockIdx.y;
    const uint8_t* Abase = g.A + bz * g.matrixA + ga * g.chunks * g.recordA;
    const uint8_t* Bbase = g.B + bz * g.matrixB + gb * g.chunks * g.recordB;
    const int eadj = g.eadj - Unpack<WA, B>::kScaleLog2 - Unpack<WB, B>::kScaleLog2;
    uint32_t* xe = lds + wave * (int)(scale_lds(BIASED) / 4);
    float* red = reinterpret_cast<float*>(lds + nw * (int)(scale_lds(BIASED) / 4));

    float acc[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[r] = 0.f;
    uint32_t pa[D][kDwA], pb[D][kDwB], ea4[D], eb4[D];
    // chunk t of this wave.  Past the end it is the last chunk again (loaded, not used): no load sits under a condition,
    // so the waits count exactly what is in flight; the record's address is scalar and the lanes' offsets stay put.
    auto fetch = [&](int s, int64_t t) {
        int64_t c = wave + t * nw;
        c = c < g.chunks ? c : g.chunks - 1;
        const uint8_t* ra = Abase + c * g.recordA;
        const uint8_t* rb = Bbase + c * g.recordB;
        load_dwords<kDwB>(rb + lane * (kDwB * 4), pb[s]);
        load_dwords<1>(rb + 64 * (kDwB * 4) + i * 4, &eb4[s]);
        load_dwords<kDwA>(ra + lane * (kDwA * 4), pa[s]);
        load_dwords<1>(ra + 64 * (kDwA * 4) + i * 4, &ea4[s]);
    };
    // exponent bytes rebased to bias 127 and moved up by 32: [96, 159] becomes the bytes whose top bits are 10
    const uint32_t move = (uint32_t)(127 - g.bias + 32) * 0x01010101u, neutral = (uint32_t)g.bias * 0x01010101u;
    const bool arow = ga * 32 + i < g.M, brow = gb * 32 + i < g.N;       // padding rows take a neutral exponent
    const bool upper = ga * 32 + 16 < g.M;                               // rows 16..31 of the tile exist
    // bits of the scales: 2^(Ea - bias) of a row, 2^(Eb - bias + all of eadj but the two biases) of a column
    const uint32_t rowbits = (uint32_t)(127 - g.bias) << 23, colbits = (uint32_t)(127 + g.bias + eadj) << 23;
    v16i bias = dot_bias();
    if constexpr (BIASED) asm volatile("" : "+v"(bias));                 // sixteen registers, not a constant built per block

    const int64_t per_wave = (g.chunks - wave + nw - 1) / nw;           // may be negative: none
    if (per_wave > 0) {
#pragma unroll
        for (int s = 0; s < D; ++s) fetch(s, s);
    }
    for (int64_t t0 = 0; t0 < per_wave; t0 += D) {
#pragma unroll
        for (int s = 0; s < D; ++s) {
            if (t0 + s < per_wave) {                                     // scalar condition: no load depends on it
                const uint32_t ea = arow ? ea4[s] : neutral, eb = brow ? eb4[s] : neutral;
                const uint32_t e2 = h ? ea >> 16 : ea;                   // each lane half writes two of its row's four blocks
                const uint32_t elo = e2 & 0xFFu, ehi = (e2 >> 8) & 0xFFu;
                if constexpr (!BIASED) {
                    xe[(2 * h) * 32 + i] = elo;                          // row exponents as integers -> LDS [block][row]
                    xe[(2 * h + 1) * 32 + i] = ehi;
                }
                const uint32_t off = (((ea + move) ^ 0x80808080u) | ((eb + move) ^ 0x80808080u)) & 0xC0C0C0C0u;
                const bool narrow = __builtin_amdgcn_ballot_w64(off != 0) == 0;
                if constexpr (BIASED) {
                    if (narrow) {                                        // row scales and what takes the bias off
                        const uint32_t slo = (elo << 23) + rowbits, shi = (ehi << 23) + rowbits;
                        xe[(2 * h) * 32 + i] = slo;
                        xe[(2 * h + 1) * 32 + i] = shi;
                        xe[128 + (2 * h) * 32 + i] = slo + kDotBack;
                        xe[128 + (2 * h + 1) * 32 + i] = shi + kDotBack;
                    } else {
                        xe[(2 * h) * 32 + i] = elo;
                        xe[(2 * h + 1) * 32 + i] = ehi;
                    }
                }
                __builtin_amdgcn_wave_barrier();                         // the wave's own LDS writes come first
                auto chunk = [&](auto narrowc, auto upperc) {
                    constexpr bool NARROW = decltype(narrowc)::value;
                    constexpr int NQ = decltype(upperc)::value ? 4 : 2;  // groups of eight rows
                    // one block after the other, pinned: the other waves of the SIMD cover the matrix instruction's
                    // latency, two blocks' sums at a time would not fit the registers next to the prefetched chunk
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        uint32_t fa[kHalfDw], fb[kHalfDw];
                        Unpack<WA, B>::run(pa[s], j, fa);
                        Unpack<WB, B>::run(pb[s], j, fb);
                        const uint32_t* row = xe + j * 32 + 4 * h;
                        if constexpr (NARROW && BIASED) {
                            const v16i d = block_mfma<B>(fa, fb, bias);
                            const float sb = __uint_as_float((((eb >> (8 * j)) & 0xFFu) << 23) + colbits);
                            auto term = [&](int r, float sa, float back) {
                                acc[r] = __builtin_fmaf(__builtin_fmaf(__uint_as_float((uint32_t)d[r]), sa, back), sb, acc[r]);
                            };
#pragma unroll
                            for (int q = 0; q < NQ; ++q) {
                                const float4 sa = *reinterpret_cast<const float4*>(row + 8 * q);
                                const float4 back = *reinterpret_cast<const float4*>(row + 128 + 8 * q);
                                term(4 * q, sa.x, back.x);
                                term(4 * q + 1, sa.y, back.y);
                                term(4 * q + 2, sa.z, back.z);
                                term(4 * q + 3, sa.w, back.w);
                            }
                        } else {
                            const v16i d = block_mfma<B>(fa, fb);
                            const int ebj = (int)((eb >> (8 * j)) & 0xFFu) + eadj + 127;
                            auto term = [&](int r, int e) {
                                if constexpr (NARROW)
                                    acc[r] = __builtin_fmaf((float)d[r], __uint_as_float((uint32_t)(e + ebj) << 23), acc[r]);
                                else acc[r] += __builtin_ldexpf((float)d[r], e + ebj - 127);
                            };
#pragma unroll
                            for (int q = 0; q < NQ; ++q) {
                                const int4 e = *reinterpret_cast<const int4*>(row + 8 * q);
                                term(4 * q, e.x);
                                term(4 * q + 1, e.y);
                                term(4 * q + 2, e.z);
                                term(4 * q + 3, e.w);
                            }
                        }
                        __builtin_amdgcn_sched_barrier(0);
                    }
                };
                // an empty statement that may change the pieces keeps the compiler from unpacking all four blocks ahead
                // of the branch, for both of its sides, in registers it does not have
                auto opaque = [&]() {
#pragma unroll
                    for (int d = 0; d < kDwA; ++d) asm volatile("" : "+v"(pa[s][d]));
#pragma unroll
                    for (int d = 0; d < kDwB; ++d) asm volatile("" : "+v"(pb[s][d]));
                };
                opaque();
                if (narrow) {
                    if (upper) chunk(std::true_type{}, std::true_type{}); else { opaque(); chunk(std::true_type{}, std::false_type{}); }
                } else {
                    opaque();
                    chunk(std::false_type{}, std::true_type{});
                }
                __builtin_amdgcn_wave_barrier();
            }
            fetch(s, t0 + s + D);                                        // the slot is free: refill it
        }
    }

    // partial tiles of the waves, always added in the same order: the upper half of the waves hands over to the lower
    // half, then every output is one thread's sum over the remaining waves
    const int half = nw / 2;
    if (wave >= half) {
#pragma unroll
        for (int r = 0; r < 16; ++r) red[((wave - half) * 16 + r) * 64 + lane] = acc[r];
    }
    __syncthreads();
    if (wave < half) {
#pragma unroll
        for (int r = 0; r < 16; ++r) red[(wave * 16 + r) * 64 + lane] += acc[r];
    }
    __syncthreads();
    float* Y = g.Y + bz * g.batch_stride_y;
    for (int t = threadIdx.x; t < 1024; t += nw * 64) {
        const int r = t >> 6, l = t & 63;
        float s = 0.f;
        for (int w = 0; w < half; ++w) s += red[(w * 16 + r) * 64 + l];
        const int64_t m = ga * 32 + 8 * (r >> 2) + 4 * (l >> 5) + (r & 3);
        const int64_t n = gb * 32 + (l & 31);
        // written once and not read again by this kernel: a streaming store keeps the operands in the L2
        if (m < g.M && n < g.N) __builtin_nontemporal_store(s, &Y[m * g.ldy + n]);
    }
}

// ------------------------------------------------------------------------------------------------
// The form for large products and short K (see large_tiles_faster): a workgroup of four waves owns a 128 x 128 tile, each wave a 64 x 64
// quarter (2 x 2 row groups), so that an unpacked fragment is used twice.  Fragments come straight from global memory in
// lane order.
// ------------------------------------------------------------------------------------------------
template <int WA, int WB, int B>
__global__ __launch_bounds__(256) void gemm_fragment_kernel(GemmArgs g) {
    constexpr int kDwA = Piece<WA, B>::kDw, kDwB = Piece<WB, B>::kDw;
    constexpr int kHalfDw = B / 8;       // int8 dwords per lane per block
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int i = lane & 31, h = lane >> 5;
    const int64_t ga0 = (int64_t)blockIdx.y * 4 + (wave >> 1) * 2;
    const int64_t gb0 = (int64_t)blockIdx.x * 4 + (wave & 1) * 2;
    const int64_t bz = blockIdx.z;
    const uint8_t* Abase = g.A + bz * g.matrixA;
    const uint8_t* Bbase = g.B + bz * g.matrixB;
    const int eadj = g.eadj - Unpack<WA, B>::kScaleLog2 - Unpack<WB, B>::kScaleLog2;

    float acc[2][2][16];
#pragma unroll
    for (int ta = 0; ta < 2; ++ta)
#pragma unroll
        for (int tb = 0; tb < 2; ++tb)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[ta][tb][r] = 0.f;

    for (int64_t c = 0; c < g.chunks; ++c) {
        uint32_t pa[2][kDwA], pb[2][kDwB];
        uint32_t ea[2][16];     // [group][4*gq + r]: the four block exponents of row 8*gq + 4*h + r
        uint32_t eb[2];
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            if (ga0 + t < g.groupsA) {
                const uint8_t* rec = Abase + ((ga0 + t) * g.chunks + c) * g.recordA;
                load_dwords<kDwA>(rec + lane * (kDwA * 4), pa[t]);
                const uint8_t* ex = rec + 64 * (kDwA * 4);
#pragma unroll
                for (int gq = 0; gq < 4; ++gq) load_dwords<4>(ex + (8 * gq + 4 * h) * 4, &ea[t][4 * gq]);
            } else {
#pragma unroll
                for (int d = 0; d < kDwA; ++d) pa[t][d] = 0;
#pragma unroll
                for (int d = 0; d < 16; ++d) ea[t][d] = 0;
            }
            if (gb0 + t < g.groupsB) {
                const uint8_t* rec = Bbase + ((gb0 + t) * g.chunks + c) * g.recordB;
                load_dwords<kDwB>(rec + lane * (kDwB * 4), pb[t]);
                eb[t] = reinterpret_cast<const uint32_t*>(rec + 64 * (kDwB * 4))[i];
            } else {
#pragma unroll
                for (int d = 0; d < kDwB; ++d) pb[t][d] = 0;
                eb[t] = 0;
            }
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            uint32_t fa[2][kHalfDw], fb[2][kHalfDw];
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                Unpack<WA, B>::run(pa[t], j, fa[t]);
                Unpack<WB, B>::run(pb[t], j, fb[t]);
            }
#pragma unroll
            for (int ta = 0; ta < 2; ++ta) {
#pragma unroll
                for (int tb = 0; tb < 2; ++tb) {
                    const v16i d = block_mfma<B>(fa[ta], fb[tb]);
                    const int ebj = (int)((eb[tb] >> (8 * j)) & 0xFFu) + eadj;
#pragma unroll
                    for (int r = 0; r < 16; ++r) {
                        const int e = (int)((ea[ta][r] >> (8 * j)) & 0xFFu) + ebj;
                        acc[ta][tb][r] += __builtin_ldexpf((float)d[r], e);
                    }
                }
            }
        }
    }

    float* Y = g.Y + bz * g.batch_stride_y;
#pragma unroll
    for (int ta = 0; ta < 2; ++ta) {
#pragma unroll
        for (int tb = 0; tb < 2; ++tb) {
            const int64_t n = (gb0 + tb) * 32 + i;
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int64_t m = (ga0 + ta) * 32 + 8 * (r >> 2) + 4 * h + (r & 3);
                // written once and not read again by this kernel: a streaming store keeps the operands in the L2
                if (m < g.M && n < g.N) __builtin_nontemporal_store(acc[ta][tb][r], &Y[m * g.ldy + n]);
            }
        }
    }
}

// ------------------------------------------------------------------------------------------------
// Decode kernel (M <= 8): bound by one pass over the packed right operand.  A workgroup of NW
// waves owns 32 output columns; its waves take the K chunks round-robin, each keeping four fp32
// partial sums per lane (rows 4*h .. 4*h+3), which are added through LDS at the end.
// ------------------------------------------------------------------------------------------------
template <int WA, int WB, int B, int NW>
__global__ __launch_bounds__(NW * 64) void gemv_fragment_kernel(GemmArgs g) {
    constexpr int kDwA = Piece<WA, B>::kDw, kDwB = Piece<WB, B>::kDw;
    constexpr int kHalfDw = B / 8;
    __shared__ float red[NW][4][64];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int i = lane & 31, h = lane >> 5;
    const int64_t gb = blockIdx.x;
    const int64_t bz = blockIdx.y;
    const uint8_t* Abase = g.A + bz * g.matrixA;                       // group 0 holds all M <= 8 rows
    const uint8_t* Bbase = g.B + bz * g.matrixB + gb * g.chunks * g.recordB;
    const int eadj = g.eadj - Unpack<WA, B>::kScaleLog2 - Unpack<WB, B>::kScaleLog2;
    const bool arow = i < g.M;

    float acc[4] = {0.f, 0.f, 0.f, 0.f};
    for (int64_t c = wave; c < g.chunks; c += NW) {
        uint32_t pa[kDwA], pb[kDwB], ea[4], eb;
        const uint8_t* recB = Bbase + c * g.recordB;
        load_dwords<kDwB>(recB + lane * (kDwB * 4), pb);
        eb = reinterpret_cast<const uint32_t*>(recB + 64 * (kDwB * 4))[i];
        const uint8_t* recA = Abase + c * g.recordA;
        if (arow) {
            load_dwords<kDwA>(recA + lane * (kDwA * 4), pa);
        } else {
#pragma unroll
            for (int d = 0; d < kDwA; ++d) pa[d] = 0;
        }
        load_dwords<4>(recA + 64 * (kDwA * 4) + (4 * h) * 4, ea);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            uint32_t fa[kHalfDw], fb[kHalfDw];
            Unpack<WA, B>::run(pa, j, fa);
            Unpack<WB, B>::run(pb, j, fb);
            const v16i d = block_mfma<B>(fa, fb);
            const int ebj = (int)((eb >> (8 * j)) & 0xFFu) + eadj;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int e = (int)((ea[r] >> (8 * j)) & 0xFFu) + ebj;
                acc[r] += __builtin_ldexpf((float)d[r], e);
            }
        }
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) red[wave][r][lane] = acc[r];
    __syncthreads();
    // 256 (r, lane) sums, one per thread of the first four waves
    for (int t = threadIdx.x; t < 256; t += NW * 64) {
        const int r = t >> 6, l = t & 63;
        float s = 0.f;
#pragma unroll
        for (int w = 0; w < NW; ++w) s += red[w][r][l];
        const int64_t m = 4 * (l >> 5) + r;
        const int64_t n = gb * 32 + (l & 31);
        if (m < g.M && n < g.N) g.Y[bz * g.batch_stride_y + m * g.ldy + n] = s;
    }
}

constexpr int kGemvWaves = 8;

// ------------------------------------------------------------------------------------------------
// Streaming decode kernel (M <= 8, K small enough for the activations to sit in LDS): the same
// arithmetic as above, arranged for HBM bandwidth.  The workgroup copies the (tiny) left
// operand's fragments into LDS once; every wave keeps D chunks of its share of the packed right
// operand in flight in registers (a ring that is refilled as soon as a slot has been consumed),
// so the weight stream never waits for the arithmetic.
//   MR: rows per lane half that are computed (1 for M == 1, else 4).
// ------------------------------------------------------------------------------------------------
template <int WA, int WB, int B, int NW, int D, int MR>
__global__ __launch_bounds__(NW * 64) void gemv_stream_kernel(GemmArgs g) {
    constexpr int kDwA = Piece<WA, B>::kDw, kDwB = Piece<WB, B>::kDw;
    constexpr int kHalfDw = B / 8;
    constexpr int XD = 16 * kDwA + 8;            // dwords kept per chunk: 16 lane pieces (rows 0..7, both halves) + 8 rows of exponents
    extern __shared__ __attribute__((aligned(16))) uint32_t xs[];
    float* red = reinterpret_cast<float*>(xs + g.chunks * XD);          // [NW][MR][64]
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int i = lane & 31, h = lane >> 5;
    const int64_t gb = blockIdx.x;
    const int64_t bz = blockIdx.y;
    const uint8_t* Abase = g.A + bz * g.matrixA;
    const uint8_t* Bbase = g.B + bz * g.matrixB + gb * g.chunks * g.recordB;
    const int eadj = g.eadj - Unpack<WA, B>::kScaleLog2 - Unpack<WB, B>::kScaleLog2;
    const int chunks = (int)g.chunks;

    // ring of D chunks of weights per wave; chunk number t of this wave is chunk wave + t*NW, and a
    // chunk number past the end of the column group reads zeros (no branch around a load: the waits
    // the compiler places then count exactly the loads that are in flight)
    const BufRsrc rB = make_rsrc(Bbase, (uint32_t)(chunks * g.recordB));
    uint32_t pb[D][kDwB], eb[D];
    auto fetch = [&](int slot, int t) {
        const uint32_t off = (uint32_t)(wave + t * NW) * (uint32_t)g.recordB;
        buf_load_dwords<kDwB>(rB, off + lane * (kDwB * 4), pb[slot]);
        buf_load_dwords<1>(rB, off + 64 * (kDwB * 4) + i * 4, &eb[slot]);
    };

    // left operand -> LDS (rows 0..7 of row group 0), in units of UD dwords, several loads in flight.
    // Loads return in the order of issue: the first batch of the left operand is requested before the
    // ring of weights, so that it does not wait behind them.
    {
        constexpr int UD = (kDwA % 4 == 0) ? 4 : 1;          // dwords per unit
        constexpr int UPC = XD / UD;                         // units per chunk (XD = 16*kDwA + 8)
        constexpr int UNROLL = 4;
        const int total = chunks * UPC;
        auto batch_load = [&](int base, uint32_t (*v)[UD]) {
#pragma unroll
            for (int u = 0; u < UNROLL; ++u) {
                const int idx = base + u * NW * 64;
                if (idx < total) {
                    const int c = idx / UPC, d = (idx - c * UPC) * UD;
                    const uint8_t* rec = Abase + (int64_t)c * g.recordA;
                    const uint8_t* src;
                    int row;                                  // first row the unit belongs to
                    if (d < 16 * kDwA) {
                        const int l16 = d / kDwA, dd = d - l16 * kDwA;
                        row = l16 & 7;
                        src = rec + ((l16 >> 3) * 32 + row) * (kDwA * 4) + dd * 4;
                    } else {
                        row = d - 16 * kDwA;
                        src = rec + 64 * (kDwA * 4) + row * 4;
                    }
                    // rows >= M feed accumulator rows that are never stored: their slots keep whatever LDS holds
                    if (row < g.M) load_dwords<UD>(src, v[u]);
                }
            }
        };
        auto batch_store = [&](int base, uint32_t (*v)[UD]) {
#pragma unroll
            for (int u = 0; u < UNROLL; ++u) {
                const int idx = base + u * NW * 64;
                if (idx < total) {
#pragma unroll
                    for (int d = 0; d < UD; ++d) xs[idx * UD + d] = v[u][d];
                }
            }
        };
        uint32_t v[UNROLL][UD];
        batch_load(threadIdx.x, v);
#pragma unroll
        for (int u = 0; u < D; ++u) fetch(u, u);
        batch_store(threadIdx.x, v);
        for (int base = threadIdx.x + NW * 64 * UNROLL; base < total; base += NW * 64 * UNROLL) {
            batch_load(base, v);
            batch_store(base, v);
        }
    }
    __syncthreads();

    float acc[MR];
#pragma unroll
    for (int r = 0; r < MR; ++r) acc[r] = 0.f;
    const int per_wave = (chunks - wave + NW - 1) / NW;          // chunks of this wave, wave-uniform (chunks >= NW is not required)
    for (int t0 = 0; t0 < per_wave; t0 += D) {
#pragma unroll
        for (int u = 0; u < D; ++u) {
            const int t = t0 + u;
            const bool live = t < per_wave;                       // scalar condition: no load depends on it
            const int c = wave + t * NW;
            uint32_t fbv[4][kHalfDw];
            uint32_t ebv = 0;
            if (live) {
#pragma unroll
                for (int j = 0; j < 4; ++j) Unpack<WB, B>::run(pb[u], j, fbv[j]);
                ebv = eb[u];
            }
            fetch(u, t + D);                                      // the slot is free: refill it
            if (live) {
                const uint32_t* xc = xs + c * XD;
                uint32_t pa[kDwA], ea[4];
                if (i < 8) {
#pragma unroll
                    for (int d = 0; d < kDwA; ++d) pa[d] = xc[(h * 8 + i) * kDwA + d];
                } else {
#pragma unroll
                    for (int d = 0; d < kDwA; ++d) pa[d] = 0;
                }
#pragma unroll
                for (int r = 0; r < 4; ++r) ea[r] = xc[16 * kDwA + 4 * h + r];
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    uint32_t fa[kHalfDw];
                    Unpack<WA, B>::run(pa, j, fa);
                    const v16i d = block_mfma<B>(fa, fbv[j]);
                    const int ebj = (int)((ebv >> (8 * j)) & 0xFFu) + eadj;
#pragma unroll
                    for (int r = 0; r < MR; ++r) {
                        const int e = (int)((ea[r] >> (8 * j)) & 0xFFu) + ebj;
                        acc[r] += __builtin_ldexpf((float)d[r], e);
                    }
                }
            }
        }
    }
#pragma unroll
    for (int r = 0; r < MR; ++r) red[(wave * MR + r) * 64 + lane] = acc[r];
    __syncthreads();
    for (int t = threadIdx.x; t < MR * 64; t += NW * 64) {
        const int r = t >> 6, l = t & 63;
        float s = 0.f;
#pragma unroll
        for (int w = 0; w < NW; ++w) s += red[(w * MR + r) * 64 + l];
        const int64_t m = 4 * (l >> 5) + r;
        const int64_t n = gb * 32 + (l & 31);
        if (m < g.M && n < g.N) g.Y[bz * g.batch_stride_y + m * g.ldy + n] = s;
    }
}

// Waves of the 32 x 32 form that a compute unit holds (registers): 16 of the kernel with blocks of 16, or of 32 with few bits,
// and 12 of the others.  Not told apart: 8 with blocks of 64 and 7 or 8 bits on both sides, 16 with 8 by 8 bits in blocks of
// 32 and 2 by 2 in blocks of 64.
constexpr int resident_waves(int block, int wa, int wb) { return block == 16 || (block == 32 && wa + wb <= 8) ? 16 : 12; }

// Waves per tile of that form: as many as leave all tiles resident at once.  A workgroup spends most of a short K loop on
// the way to its first records and in its sum over the waves, and only another workgroup's arithmetic covers that.  Two
// workgroups of eight waves on a compute unit instead of one after the other with sixteen: 32 x 13824 x 5120, 8 by 4 bits,
// blocks of 16, 22.9 -> 20.3 us; blocks of 32, four waves where it were eight: 32 x 13824 x 5120 19.0 -> 15.9 us, 40 x 11008
// x 1024 12.7 -> 7.7 us.  Past three (blocks of 64: two) tiles per compute unit two waves win while K is short.  Drawn on
// 14700 random products (M 9 to 4096, N 64 to 14000, K to 14000) timed with every number of waves; six never won.
inline int waves_per_tile(int block, int resident, int64_t chunks, int64_t tiles) {
    if (tiles <= 256) return block == 16 ? 16 : 8;
    if (resident == 16) return tiles <= 512 || (tiles <= 768 && chunks > 40) ? 8 : 4;
    if (tiles <= (block == 32 ? 768 : 512)) return 4;
    return chunks <= (block == 32 || tiles <= 1024 ? 12 : 4) ? 2 : 4;
}

// Which of the two forms for M > 8 is the faster one: the sum that estimates its time (us) is the smaller.  The 128 x 128
// form: every compute unit takes its share of the tiles, a cost per K chunk and one per tile (launch, store).  The 32 x 32
// form: rounds of workgroups (resident_waves), each with the chunks its
// slowest wave takes one after the other and a cost of its own (launch, sum over the waves, store), and the vector work of
// all blocks.  So the split over the waves wins while K is long enough to divide or the tiles are too few to fill the chip,
// and the large tile wins on short K: 32 x 2304 x 5504 x 32 (block 32) 357 us, 1601 us with small tiles; 2064 x 4992 x 160
// 26 and 40 us; 2048 x 4096 x 4096, 8 by 8 bits in blocks of 64, 194 and 261 us, but 6 by 5 bits in blocks of 32 218 and
// 212 us, 8 by 4 bits in blocks of 16 or 32 366 and 274, 202 and 172 us (before the small form's scaling took two instructions
// for three).  The coefficients are least squares over shapes timed in both forms: the large one's over 19159 (M 9 to 32768,
// N 16 to 14000, K 16 to 12000, batch 1 to 32, all widths), the small one's over 14700 (see waves_per_tile); there the choice
// costs 0.1 to 0.3 % against always taking the faster one.  Within 5 % of each other the
// large tile is taken: its scaling is the same for any exponents, the small one's slower outside its narrow range (3363 x
// 8704 x 10368, 8 by 8 bits in blocks of 64, exponents over 60 binades: 1537 us, 2060 with small tiles).
struct FormCost { float base128, step128, chunk128, tile128, base32, step32, round_step32, round32, chunk32; };

inline bool large_tiles_faster(int block, int resident, int64_t chunks, int64_t tiles32, int64_t tiles128, int nw) {
    const FormCost k = block == 16 ? FormCost{1.98f, 0.63f, 2.38f, 2.15f, 1.74f, 0.80f, 0.40f, 2.70f, 0.054f}
                     : block == 32 ? FormCost{1.66f, 0.80f, 2.57f, 2.46f, 1.43f, 0.69f, 0.18f, 3.53f, 0.094f}
                                   : FormCost{1.09f, 0.65f, 3.59f, 3.23f, 0.37f, 1.59f, 0.12f, 3.99f, 0.20f};
    const float c = (float)chunks, steps = (float)ceil_div(chunks, nw);
    const float share128 = (float)ceil_div(tiles128, 256), rounds32 = (float)ceil_div(tiles32, 256 * (resident / nw));
    const float t128 = k.base128 + k.step128 * c + share128 * (k.chunk128 * c + k.tile128);
    const float t32 = k.base32 + k.step32 * steps + rounds32 * (k.round_step32 * steps + k.round32) +
                      k.chunk32 * c * (float)tiles32 / 256.f;
    return t128 < 1.05f * t32;
}

// Chunks in flight per wave: five, and three or two where five do not fit the 128 registers of the 16-wave form (records of
// 20 and more dwords per lane) and would be spilled to memory and read back for every chunk.
// Fewer, which pay in the kernels that quantize their activations (kDotDepth, ring_depth), have not been timed here.
template <int WB, int B, int NW> constexpr int kStreamDepth = NW < 16 || Piece<WB, B>::kDw < 20 ? 5 : Piece<WB, B>::kDw < 24 ? 3 : 2;

template <int WA, int WB, int B, int MR, int NW>
mx_status launch_stream(const GemmArgs& g, int64_t batch, size_t smem, hipStream_t st) {
    auto kern = gemv_stream_kernel<WA, WB, B, NW, kStreamDepth<WB, B, NW>, MR>;
    static std::atomic<uint64_t> done{0};
    if (!allow_dynamic_lds((const void*)kern, 160 * 1024, done)) return MX_ERR_DEVICE;
    dim3 grid((unsigned)g.groupsB, (unsigned)batch);
    hipLaunchKernelGGL(kern, grid, dim3(NW * 64), smem, st, g);
    MX_HIP_LAUNCH_CHECK();
    return MX_OK;
}

template <int WA, int WB, int B>
mx_status launch(const GemmArgs& g, int64_t batch, hipStream_t st) {
    if (g.M <= 8) {
        // streaming kernel when the left operand fits in LDS next to the reduction buffer; 16 waves per
        // workgroup when there are too few column groups to fill the chip with 8
        constexpr int XD = 16 * Piece<WA, B>::kDw + 8;
        const int nw = g.groupsB * batch < 256 ? 16 : 8;
        const size_t smem = (size_t)g.chunks * XD * 4 + (size_t)nw * 4 * 64 * 4;
        if (g.chunks > 0 && (g.chunks + 1024) * g.recordB < (1LL << 31) && smem <= 160 * 1024) {
            if (nw == 16) {
                if (g.M == 1) return launch_stream<WA, WB, B, 1, 16>(g, batch, smem, st);
                return launch_stream<WA, WB, B, 4, 16>(g, batch, smem, st);
            }
            if (g.M == 1) return launch_stream<WA, WB, B, 1, 8>(g, batch, smem, st);
            return launch_stream<WA, WB, B, 4, 8>(g, batch, smem, st);
        }
        dim3 grid((unsigned)g.groupsB, (unsigned)batch);
        hipLaunchKernelGGL((gemv_fragment_kernel<WA, WB, B, kGemvWaves>), grid, dim3(kGemvWaves * 64), 0, st, g);
    } else {
        const int64_t tiles = g.groupsA * g.groupsB * batch;
        constexpr int kResident = resident_waves(B, WA, WB);
        const int nw = waves_per_tile(B, kResident, g.chunks, tiles);
        const bool large = large_tiles_faster(B, kResident, g.chunks, tiles, ceil_div(g.groupsA, 4) * ceil_div(g.groupsB, 4) * batch, nw);
        // a grid dimension holds fewer than 2^32 work items: from 2^24 tiles (a result of 64 GiB) on there are too many
        const bool past_grid = ceil_div(g.groupsA * g.groupsB, 8) * 8 * nw * 64 > 0xffffffffLL;
        if (large || past_grid) {
            dim3 grid((unsigned)ceil_div(g.groupsB, 4), (unsigned)ceil_div(g.groupsA, 4), (unsigned)batch);
            hipLaunchKernelGGL((gemm_fragment_kernel<WA, WB, B>), grid, dim3(256), 0, st, g);
            MX_HIP_LAUNCH_CHECK();
            return MX_OK;
        }
        const size_t smem = (size_t)nw * scale_lds(biased_sums(WA, WB, B)) + (size_t)(nw / 2) * 4096;
        dim3 grid((unsigned)(ceil_div(g.groupsA * g.groupsB, 8) * 8), (unsigned)batch);
        hipLaunchKernelGGL((gemm_tile_kernel<WA, WB, B>), grid, dim3(nw * 64), smem, st, g);
    }
    MX_HIP_LAUNCH_CHECK();
    return MX_OK;
}

#define MX_SW(W_, NAME, ...)                                        \
    switch (W_) {                                                   \
        case 2: { constexpr int NAME = 2; __VA_ARGS__; } break;     \
        case 3: { constexpr int NAME = 3; __VA_ARGS__; } break;     \
        case 4: { constexpr int NAME = 4; __VA_ARGS__; } break;     \
        case 5: { constexpr int NAME = 5; __VA_ARGS__; } break;     \
        case 6: { constexpr int NAME = 6; __VA_ARGS__; } break;     \
        case 7: { constexpr int NAME = 7; __VA_ARGS__; } break;     \
        case 8: { constexpr int NAME = 8; __VA_ARGS__; } break;     \
        default: return MX_ERR_BAD_ARG;                             \
    }

template <int B>
mx_status dispatch_widths(const GemmArgs& g, int wa, int wb, int64_t batch, hipStream_t st) {
    MX_SW(wa, kWA, MX_SW(wb, kWB, return (launch<kWA, kWB, B>(g, batch, st))));
    return MX_ERR_BAD_ARG;
}

}  // namespace

#define MX_CAT2(a, b) a##b
#define MX_CAT(a, b) MX_CAT2(a, b)
mx_status MX_CAT(gemm_block, MX_GEMM_BLOCK)(const GemmArgs& g, int wa, int wb, int64_t batch, hipStream_t st) {
    return dispatch_widths<MX_GEMM_BLOCK>(g, wa, wb, batch, st);
}

}  // namespace mx
