// Attention with both matrix products in MXInt, in one kernel (blocks of 16, operands in the
// bfloat16 form of MX_LAYOUT_MATRIX, see mx_bf16.h).
//
// What is computed, per head (Fig. 1 of the paper: both products of the attention layer take
// quantized operands; Section 3.2: an emulated operator computes on quantized inputs, here the
// probabilities are quantized before the second product like any other operand):
//     S = Q K^T,  P = softmax(scale * S) along the keys (fp32),  P^ = MXInt(P) in blocks of 16 keys,
//     O = P^ V.
// The quantizer scales a block by a power of two chosen from the block's maximum, so P^ needs the
// final row maximum and row sum: the kernel sweeps the keys twice.  Sweep 1 takes S tile by tile
// and keeps a running maximum and sum per query; sweep 2 takes S again (34 GOP at the full size,
// far cheaper than the 537 MB of fp32 scores it replaces), forms P, quantizes it in registers and
// feeds it to the second product.
//
// Register-only hand-over between the products: S is computed transposed, S^T = K Q^T, so that in
// the result a lane holds one query (column) and 16 keys; the rows of the K operand are permuted
// when they are read from LDS (bits 2 and 3 of the row number swapped) so that those 16 keys are
// two whole blocks, elements 8h..8h+7 of each in lane half h -- exactly the operand layout of
// v_mfma_f32_32x32x16_bf16 for O^T = V^T P^T.  The block maximum is completed with the lane of the
// other half (one exchange per block).
//
// Work split: a workgroup of four waves owns 128 queries of one head (a wave: one tile of 32, its
// Q fragments stay in registers), two workgroups per compute unit (few queries: attention_split_kernel); the K (and in
// sweep 2 the V^T) units of one tile of 32 keys are copied global -> LDS with 16-byte direct-to-LDS loads, five
// stages, one barrier per key tile.  Two query tiles per wave (363 registers, one workgroup) were slower, 128 us.
//
// Bound: on real operands the power that they draw, at the full clock vector issue: a matrix instruction takes 8 of its 32
// cycles from the vector ALU, an exponential 8, any other vector instruction 4, an LDS read about 5.  32 heads x 2048 x 2048 x
// 128 takes 125 us, 100 us on operands that are all zero (the same instructions; medians of launches back to back under the
// kernel trace, as all times of this paragraph).  Hence few vector instructions: the exponents of both blocks of a tile are
// computed at once (block_scales).  The LDS reads of a tile's K run a tile ahead, each into the registers that a matrix
// instruction has just freed, so that no instruction waits for them.  Together 131 -> 125 us, on zeros 108 -> 100; 30 heads x 1999
// x 2016 x 96 108 -> 98, 24 x 2040 x 2048 x 80 99 -> 92, 32 x 1500 x 1536 x 64 61.7 -> 55.6, 32 x 900 x 1024 x 128 39.3 -> 37.5.
// V^T straight from global memory instead of through LDS was 3 percent slower.  The second product of a key tile runs one tile
// behind its scores, so that no matrix instruction is left without vector work under it: 16 heads x 2040 queries x 2048 keys x
// 128 7 percent less (where it does not pay: pick_attention).
#include <type_traits>

#include "mx_bf16.h"

namespace mx {
namespace {

typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef int v4i __attribute__((ext_vector_type(4)));
typedef float v16f __attribute__((ext_vector_type(16)));
typedef float v4f __attribute__((ext_vector_type(4)));

struct AttnArgs {
    const uint8_t* Q;
    const uint8_t* K;
    const uint8_t* V;              // V^T: [D x Sk]
    float* O;
    int64_t Sq, Sk, D;
    int64_t matrixQ, matrixK, matrixV;
    int64_t q_tiles;               // row tiles of Q
    int64_t nt;                    // key tiles of 32
    int64_t v_ksteps;              // K steps of the V^T geometry
    int64_t ldo, o_batch_stride;
    int64_t tiles_q, total;        // workgroup tiles per head, and in all
    int32_t parts;                 // column parts per query tile (attention_split_kernel)
    float c;                       // scale * log2(e)
    int32_t wp, bias_p, emax_p;
    int32_t vec;                   // O rows may be stored as float4
    float pair;                    // 0 when two neighbouring queries share the exponents of P, else -inf
    float wide;                    // 0 when P is quantized in blocks of 32 keys (a whole key tile), else -inf
    int32_t join;                  // one of the two
};

// 16 bytes per lane from global memory straight into LDS: lane L's bytes land at lds_addr + 16*L.
// Completion is awaited explicitly with s_waitcnt vmcnt(n) before the barrier that publishes a stage.
__device__ __forceinline__ void copy16_to_lds(const uint8_t* uniform_src, uint32_t lane_offset, uint32_t lds_addr) {
    asm volatile(
        "s_mov_b32 m0, %2\n\t"
        "s_nop 0\n\t"
        "global_load_lds_dwordx4 %0, %1\n\t"
        :
        : "v"(lane_offset), "s"(uniform_src), "s"(lds_addr)
        : "memory", "m0");
}

// s_waitcnt vmcnt(n), every other counter left alone (gfx9 encoding: vmcnt = bits 3:0 and 15:14)
template <int N>
__device__ __forceinline__ void wait_vmcnt() {
    static_assert(N >= 0 && N < 64, "vmcnt is a 6-bit counter");
    __builtin_amdgcn_s_waitcnt(0x0F70 | (N & 15) | ((N >> 4) << 14));
}

// s_waitcnt lgkmcnt(n), every other counter left alone (bits 11:8)
template <int N>
__device__ __forceinline__ void wait_lgkmcnt() {
    static_assert(N >= 0 && N < 16, "lgkmcnt is a 4-bit counter");
    __builtin_amdgcn_s_waitcnt(0xC07F | (N << 8));
}

// A workgroup barrier at which up to N of the wave's newest LDS reads may be under way
template <int N>
__device__ __forceinline__ void step_barrier() {
    wait_lgkmcnt<N>();
    asm volatile("s_barrier" ::: "memory");
}

// The value is computed before this point of the program: an empty volatile statement is ordered with the
// scheduling fences, and so, through it, is the (otherwise freely movable) arithmetic that produces v.
__device__ __forceinline__ void pin(float v) { asm volatile("" ::"v"(v)); }
__device__ __forceinline__ void pin(int v) { asm volatile("" ::"v"(v)); }

// The larger one; __builtin_fmaxf spends an instruction on either operand whose origin the compiler cannot see
__device__ __forceinline__ float max_of(float a, float b) {
    float r;
    asm("v_max_f32 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}

// The integer part of a block's largest log2, between the bounds of the exponent; -200 also for all keys masked, or c = 0 with
// them
__device__ __forceinline__ int block_exponent(const AttnArgs& g, float m) {
    int E;
    asm("v_max_f32 %0, 0xc3480000, %1\n\tv_cvt_flr_i32_f32 %0, %0\n\tv_med3_i32 %0, %0, %2, %3"
        : "=&v"(E) : "v"(m), "v"(-g.bias_p), "s"(g.emax_p));
    return E;
}

// The exponents of the two blocks of 16 keys of a key tile, from the scores s0 and s1 that are the largest of this lane's
// half of either: the quantizer's floor(log2 max) with a = log2 of a probability in place of the probability (exp2 grows with
// the score, so the maximum is taken over the scores).  Out: t[b], a mantissa q of block b stands for q * 2^t[b], and off[b],
// so that 2^(c * score + off[b]) is the probability in units of that.  One exchange between the lane halves turns two
// half maxima into one whole one per lane (lower half: block 0, upper half: block 1), so that what follows is done
// once for both; with an exchange per block and everything done twice it took 19 instructions more.
__device__ __forceinline__ void block_scales(const AttnArgs& g, float s0, float s1, float c, float mrow, int wm2, float (&off)[2],
                                             int (&t)[2]) {
    const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(s0), __float_as_uint(s1), false, false);
    float m = __builtin_fmaf(max_of(__uint_as_float(sw[0]), __uint_as_float(sw[1])), c, -mrow);
    int join = g.join;
    asm("" : "+s"(join));                                 // a scalar branch
    if (join) {
        // two-row blocks: queries 2t and 2t+1 (neighbouring lanes) share the exponent, the larger of the two
        // log-probabilities; one-row blocks add -inf to the neighbour's and keep their own
        m = __builtin_fmaxf(m, g.pair + __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(
                                            0, __builtin_bit_cast(int, m), 0xB1, 0xF, 0xF, true)));
        // blocks of 32: the tile's two runs of 16 keys are one block (the same trick: + 0 or + -inf)
        const auto both = __builtin_amdgcn_permlane32_swap(__float_as_uint(m), __float_as_uint(m), false, false);
        m = __builtin_fmaxf(m, g.wide + __builtin_fmaxf(__uint_as_float(both[0]), __uint_as_float(both[1])));
    }
    const int E = block_exponent(g, m);
    const int tm = E - wm2;
    const auto tb = __builtin_amdgcn_permlane32_swap(tm, tm, false, false);
#pragma unroll
    for (int b = 0; b < 2; ++b) {
        t[b] = (int)tb[b];
        off[b] = -(float)t[b] - mrow;
    }
}

// The same where a lane holds half of one block, its other half 16 lanes away (attention_short_kernel).
__device__ __forceinline__ void block_scale(const AttnArgs& g, float s, float c, float mrow, int wm2, float& off, int& t) {
    const auto sw = __builtin_amdgcn_permlane16_swap(__float_as_uint(s), __float_as_uint(s), false, false);
    float m = __builtin_fmaf(max_of(__uint_as_float(sw[0]), __uint_as_float(sw[1])), c, -mrow);
    if (g.join) {
        m = __builtin_fmaxf(m, g.pair + __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(
                                            0, __builtin_bit_cast(int, m), 0xB1, 0xF, 0xF, true)));
        const auto both = __builtin_amdgcn_permlane32_swap(__float_as_uint(m), __float_as_uint(m), false, false);
        m = __builtin_fmaxf(m, g.wide + __builtin_fmaxf(__uint_as_float(both[0]), __uint_as_float(both[1])));
    }
    t = block_exponent(g, m) - wm2;
    off = -(float)t - mrow;
}

constexpr int kAttnStages = 5;

// KS: K steps of 32 along the head dimension (2 or 4); DT: tiles of 32 along the head dimension of V; LAG: the second product
// runs one key tile behind the scores (see pick_attention).  A wave owns one tile of 32 queries; at most 256 registers and
// 80 KiB of LDS, so that two workgroups share a compute unit and their waves fill each other's waits.
template <int KS, int DT, int RND, bool LAG>
__global__ __launch_bounds__(256, 2) void attention_bf16_kernel(AttnArgs g) {
    constexpr int S = kAttnStages;
    constexpr int NK = 2 * KS;                          // matrix instructions (16 elements) along the head dimension
    constexpr int STAGE = (KS + DT) * kBfUnitBytes;     // K units, then V^T units
    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];

    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int i = lane & 31, h = lane >> 5;
    // Workgroup n runs on XCD n % 8, each with its own L2: every XCD gets one contiguous range of
    // (head, query tile) pairs, so that the workgroups resident on it share the K and V of few heads.
    const int64_t per_xcd = (g.total + 7) / 8;
    const int64_t lin = (blockIdx.x % 8) * per_xcd + blockIdx.x / 8;
    if (lin >= g.total) return;
    const int64_t bz = lin / g.tiles_q, bq = lin - bz * g.tiles_q;
    const uint8_t* Qbase = g.Q + bz * g.matrixQ;
    const uint8_t* Kbase = g.K + bz * g.matrixK;
    const uint8_t* Vbase = g.V + bz * g.matrixV;
    const uint32_t lane16 = lane * 16;
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void*)smem;

    // the wave's Q fragments (right operand of S^T = K Q^T): lane 32h + i holds query i, elements 8h..8h+7.
    // A negative scale is carried by the operand (sign bits flipped: every product and sum changes
    // sign exactly), so that below the largest score is the largest argument of exp.
    const int64_t qt = bq * 4 + wave;
    const int flip = g.c < 0.f ? (int)0x80008000u : 0;
    const float c = __builtin_fabsf(g.c);
    v4i qf[NK];
    {
        const int64_t rt = qt < g.q_tiles ? qt : g.q_tiles - 1;       // tiles past the matrix re-read its last tile (never stored)
#pragma unroll
        for (int kk = 0; kk < NK; ++kk) {
            qf[kk] = *reinterpret_cast<const v4i*>(Qbase + (rt * KS + (kk >> 1)) * kBfUnitBytes + (kk & 1) * 1024 + lane16);
#pragma unroll
            for (int d = 0; d < 4; ++d) qf[kk][d] ^= flip;
        }
    }

    // K rows are read permuted (bits 2 and 3 of the row swapped): result register r of lane 32h + i is
    // then key 16*(r/8) + 8h + r%8 of the tile.
    const int sig = (i & 0x13) | ((i & 4) << 1) | ((i & 8) >> 1);
    const int koff = (32 * h + sig) * 16;

    float m_run = -__builtin_inff(), l_run = 0.f;       // sweep 1: running maximum and sum of this lane's keys
    float mrow = 0.f;                                   // sweep 2: row maximum + log2(row sum), in the exp2 domain
    v16f o[DT];
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[dt][r] = 0.f;
    const float qmax = (float)((1 << (g.wp - 1)) - 1);
    const int wm2 = g.wp - 2;

    // scores of two consecutive key tiles live in two register sets: while the arithmetic on one tile's
    // scores runs on the vector units, the matrix cores take the next tile's.  With LAG the second product runs one tile
    // behind: P^ of a tile is multiplied with its V under the arithmetic on the tile after it.
    v16f s[2];
    v4i pf[2][2];                                       // P^ of the tile in set 0 / 1, two fragments of 16 keys
    v4i vf[DT][2];                                      // V^T of the tile before, replaced by this tile's piece by piece

    auto sweep = [&](auto pvc) {
        constexpr bool PV = decltype(pvc)::value;
        // 1 KiB pieces of a key tile that this wave copies: of K, and of V^T (the last one twice rather than a branch)
        constexpr int KP = KS / 2, VP = PV ? (2 * DT + 3) / 4 : 0;
        static_assert(KS % 2 == 0, "the four waves share the pieces of K evenly");
        constexpr int NL = KP + VP;                     // copies in flight per tile step
        constexpr int NREAD = NK + (PV && LAG ? 2 * DT : 0);   // LDS reads of a step that the next step's work needs
        const uint8_t* ksrc = Kbase + wave * 1024;
        const uint8_t* vsrc[VP + 1];
        int vdst[VP + 1];
#pragma unroll
        for (int q = 0; q < VP; ++q) {
            const int t = q * 4 + wave < 2 * DT ? q * 4 + wave : 2 * DT - 1;
            vsrc[q] = Vbase + (t >> 1) * g.v_ksteps * kBfUnitBytes + (t & 1) * 1024;
            vdst[q] = KS * kBfUnitBytes + t * 1024;
        }
        // Copies are always issued in full, past the last key tile that tile again, so that the
        // number of copies in flight is the same at every step and the vmcnt waits stay exact.
        const int nt = (int)g.nt;
        int k_next = 0, v_next = 0;
        auto issue_k = [&](uint32_t slot) {
#pragma unroll
            for (int q = 0; q < KP; ++q) copy16_to_lds(ksrc + q * 4096, lane16, lds0 + slot + wave * 1024 + q * 4096);
            ksrc += ++k_next < nt ? KS * kBfUnitBytes : 0;
        };
        auto issue_v = [&](uint32_t slot) {
            ++v_next;
#pragma unroll
            for (int q = 0; q < VP; ++q) {
                copy16_to_lds(vsrc[q], lane16, lds0 + slot + vdst[q]);
                vsrc[q] += v_next < nt ? kBfUnitBytes : 0;
            }
        };
        // S^T of a key tile into register set `set`: matrix instruction kk = 0 .. NK-1 one at a time (the caller slots
        // vector work between them), each followed by the read of the tile after it into the registers it has freed
        v4i kf[NK];
        auto read_k = [&](int kk, uint32_t slot) {
            kf[kk] = *reinterpret_cast<const v4i*>(smem + slot + (kk >> 1) * kBfUnitBytes + (kk & 1) * 1024 + koff);
        };
        auto score_mfma = [&](int kk, auto setc) {
            constexpr int set = decltype(setc)::value;
            v16f zero;
#pragma unroll
            for (int r = 0; r < 16; ++r) zero[r] = 0.f;
            s[set] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(v8bf, kf[kk]), __builtin_bit_cast(v8bf, qf[kk]),
                                                             kk == 0 ? zero : s[set], 0, 0, 0);
        };
        auto out_mfma = [&](int m, auto setc) {           // consecutive ones never share an accumulator (DT > 1)
            constexpr int set = decltype(setc)::value;
            const int b = m / DT, dt = m % DT;
            o[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(v8bf, vf[dt][b]),
                                                            __builtin_bit_cast(v8bf, pf[set][b]), o[dt], 0, 0, 0);
        };
        auto read_v = [&](int m, uint32_t slot) {
            const int b = m / DT, dt = m % DT;
            vf[dt][b] = *reinterpret_cast<const v4i*>(smem + slot + (KS + dt) * kBfUnitBytes + b * 1024 + lane16);
        };
        // One key tile: tile kt's scores are in set kt % 2, tile kt+1's are started into the other set, and (sweep 2)
        // tile kt-1's P^ V is added.  RAG: keys past Sk are masked (only the last tile can have them).
        // The instruction order is written out and pinned: one matrix instruction, then its share of the
        // vector work (given as numbered units), so that both pipes stay busy.
        auto body = [&](int kt, uint32_t s0, uint32_t s2, uint32_t s3, auto setc, auto ragc) {
            constexpr int set = decltype(setc)::value;
            constexpr bool RAG = decltype(ragc)::value;
            const auto nset = std::integral_constant<int, set ^ 1>{};
            // What is awaited is K of tile kt+2 and V of tile kt; in flight stay the copies of the two newest steps.  The
            // barrier publishes them.  LDS reads of tile kt-1's step may be under way at it, none from before (reads return in
            // order), so K's slot of tile kt and V's of tile kt-2 are free for the copies of this step.
            wait_vmcnt<2 * NL>();
            step_barrier<(NREAD < 15 ? NREAD : 15)>();
            if constexpr (PV && !LAG) {
#pragma unroll
                for (int m = 0; m < 2 * DT; ++m) read_v(m, s0);
            }
            __builtin_amdgcn_sched_barrier(0);
            auto next_score = [&](int kk) {
                score_mfma(kk, nset);
                __builtin_amdgcn_sched_barrier(0);        // the read takes the registers that the instruction has freed
                read_k(kk, s2);
                if (kk == 0) {
                    issue_k(s0);
                    if constexpr (PV) issue_v(s3);
                }
            };
            const int valid = (int)(g.Sk - (int64_t)kt * 32) - 8 * h;   // this lane's key 16*b + e is real iff 16*b + e < valid
            auto masked = [&](int r) { return RAG && 16 * (r >> 3) + (r & 7) >= valid; };
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (!PV) {
                // The exponentials are taken against the running maximum, tile by tile: the terms that dominate the sum then have
                // arguments near 0, which are not rounded, and a lane's sum depends on its own query alone.  Against an older
                // maximum while a tile stays within 2^20 of it the search is saved in most tiles (0 to 3 percent: 32 x 2048 x 2048 x
                // 128 124 us for 125, on zeros 97 for 100), but those arguments have rounding errors of up to 2^-20, log2 of the
                // sum as much again.
                // Units: 0 = tile maximum and the new running maximum, 1..4 = four exponentials each, 5 = the running sum.
                constexpr int NU = 6;
                float m_old, m_use, sum;
                auto unit = [&](int u) {
                    if (u == 0) {
                        float sm = -__builtin_inff();
#pragma unroll
                        for (int r = 0; r < 16; ++r) sm = __builtin_fmaxf(sm, masked(r) ? -__builtin_inff() : s[set][r]);
                        m_old = m_run;
                        m_run = __builtin_fmaxf(m_run, sm * c);
                        m_use = m_run == -__builtin_inff() ? 0.f : m_run;
                        sum = 0.f;
                        pin(m_use);
                    } else if (u < 5) {
#pragma unroll
                        for (int r = 4 * (u - 1); r < 4 * u; ++r) {
                            float arg = __builtin_fmaf(s[set][r], c, -m_use);
                            if (masked(r)) arg = -__builtin_inff();   // also when c is 0
                            sum += __builtin_amdgcn_exp2f(arg);
                        }
                        pin(sum);
                    } else {
                        l_run = l_run * __builtin_amdgcn_exp2f(m_old - m_use) + sum;
                        pin(l_run);
                    }
                };
#pragma unroll
                for (int m = 0; m < NK; ++m) {
                    next_score(m);
#pragma unroll
                    for (int x = m * NU / NK; x < (m + 1) * NU / NK; ++x) unit(x);
                    __builtin_amdgcn_sched_barrier(0);
                }
            } else {
                // The tile is two blocks of 16 keys, this lane's half of each: the arithmetic of mx_quantize on P, the
                // mantissas being round(2^(a - E + w - 2)).  Units: 0 = half-block maxima, the exponents; 1..8 = two elements
                // each, packed into their operand register.
                constexpr int NU = 9;
                float off[2];
                int t[2];
                auto unit = [&](int u) {
                    if (u == 0) {
                        float sm[2];
#pragma unroll
                        for (int b = 0; b < 2; ++b) {
                            sm[b] = -__builtin_inff();
#pragma unroll
                            for (int e = 0; e < 8; ++e) sm[b] = __builtin_fmaxf(sm[b], masked(8 * b + e) ? -__builtin_inff() : s[set][8 * b + e]);
                        }
                        block_scales(g, sm[0], sm[1], c, mrow, wm2, off, t);
                        pin(off[0]);
                        pin(off[1]);
                    } else {
                        const int b = (u - 1) >> 2, d = (u - 1) & 3;
                        float el[2];
#pragma unroll
                        for (int x = 0; x < 2; ++x) {
                            const int r = 8 * b + 2 * d + x;
                            float arg = __builtin_fmaf(s[set][r], c, off[b]);
                            if (masked(r)) arg = -__builtin_inff();
                            const float sc = __builtin_amdgcn_exp2f(arg);
                            float v = RND == MX_RNE ? __builtin_rintf(sc) : __builtin_truncf(sc);
                            v = __builtin_fminf(v, qmax);                     // probabilities are not negative
                            el[x] = __builtin_ldexpf(v, t[b]);                // an exact bfloat16 number
                        }
                        // the upper halves of two fp32 values
                        pf[set][b][d] = (int)__builtin_amdgcn_perm(__float_as_uint(el[1]), __float_as_uint(el[0]), 0x07060302u);
                        pin(pf[set][b][d]);
                    }
                };
                if constexpr (!LAG) {
                    unit(0);
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int m = 0; m < NK; ++m) {
                        next_score(m);
#pragma unroll
                        for (int x = 1 + m * (NU - 1) / NK; x < 1 + (m + 1) * (NU - 1) / NK; ++x) unit(x);
                        __builtin_amdgcn_sched_barrier(0);
                    }
#pragma unroll
                    for (int m = 0; m < 2 * DT; ++m) out_mfma(m, setc);
                    __builtin_amdgcn_sched_barrier(0);
                    return;
                }
                // matrix instructions in turn: the second product of the tile before (each followed by the read of this
                // tile's V into the registers it has freed) and the next tile's scores; vector work under all of them
                constexpr int NO = 2 * DT, NM = NO + NK;
                int mo = 0, mk = 0;
#pragma unroll
                for (int m = 0; m < NM; ++m) {
                    if ((m + 1) * NO / NM > mo) {
                        out_mfma(mo, nset);
                        __builtin_amdgcn_sched_barrier(0);
                        read_v(mo, s0);
                        ++mo;
                    } else {
                        next_score(mk);
                        ++mk;
                    }
#pragma unroll
                    for (int x = m * NU / NM; x < (m + 1) * NU / NM; ++x) unit(x);
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
        };

        if constexpr (PV && LAG) {                        // no tile before the first one: adds zeros
#pragma unroll
            for (int b = 0; b < 2; ++b) {
                pf[1][b] = v4i{0, 0, 0, 0};
#pragma unroll
                for (int dt = 0; dt < DT; ++dt) vf[dt][b] = v4i{0, 0, 0, 0};
            }
        }
        // tile step j copies K of tile j+5 and V of tile j+3; the steps before the first one, and K of two tiles ahead of them
        issue_k(0);
        issue_k(STAGE);
#pragma unroll
        for (int st = 0; st < 3; ++st) {
            issue_k((st + 2) * STAGE);
            if constexpr (PV) issue_v(st * STAGE);
        }
        wait_vmcnt<3 * NL>();
        step_barrier<0>();
#pragma unroll
        for (int kk = 0; kk < NK; ++kk) read_k(kk, 0);
#pragma unroll
        for (int kk = 0; kk < NK; ++kk) {
            score_mfma(kk, std::integral_constant<int, 0>{});
            read_k(kk, STAGE);
        }
        wait_lgkmcnt<NK>();                               // tile 0 has been read
        __builtin_amdgcn_sched_barrier(0);
        // tiles in pairs (the register sets alternate); the last one or two tiles take the masking form.  slot[x]: where tile
        // kt+x lies
        int kt = 0;
        uint32_t slot[S] = {0, STAGE, 2 * STAGE, 3 * STAGE, 4 * STAGE};
        while (kt + 2 < nt) {
            body(kt, slot[0], slot[2], slot[3], std::integral_constant<int, 0>{}, std::false_type{});
            body(kt + 1, slot[1], slot[3], slot[4], std::integral_constant<int, 1>{}, std::false_type{});
            kt += 2;
            const uint32_t t0 = slot[0], t1 = slot[1];
            slot[0] = slot[2]; slot[1] = slot[3]; slot[2] = slot[4]; slot[3] = t0; slot[4] = t1;
        }
        body(kt, slot[0], slot[2], slot[3], std::integral_constant<int, 0>{}, std::true_type{});
        if (kt + 1 < nt) {
            body(kt + 1, slot[1], slot[3], slot[4], std::integral_constant<int, 1>{}, std::true_type{});
            if constexpr (PV && LAG) {
#pragma unroll
                for (int m = 0; m < 2 * DT; ++m) out_mfma(m, std::integral_constant<int, 1>{});
            }
        } else if constexpr (PV && LAG) {
#pragma unroll
            for (int m = 0; m < 2 * DT; ++m) out_mfma(m, std::integral_constant<int, 0>{});
        }
        wait_vmcnt<0>();                                  // the clamped tail copies must not outlive the stage's next use
        __syncthreads();
    };

    sweep(std::false_type{});
    // row statistics: the two lane halves hold disjoint keys of the same query
    {
        const float mo = __shfl_xor(m_run, 32, 64), lo = __shfl_xor(l_run, 32, 64);
        const float mf = __builtin_fmaxf(m_run, mo);     // finite: there is at least one key
        // The halves may differ in the last place of the sum, in which either half's own product is not rounded.  (What has to
        // be one value for a block, its exponent, comes from one half: block_scales.)
        const float other = lo * __builtin_amdgcn_exp2f(mo - mf);
        mrow = mf + __builtin_amdgcn_logf(__builtin_fmaf(l_run, __builtin_amdgcn_exp2f(m_run - mf), other));
    }
    sweep(std::true_type{});

    // O^T registers: register r of lane 32h + i is element 8*(r/4) + 4h + r%4 of the tile's 32, query i
    float* O = g.O + bz * g.o_batch_stride;
    auto store = [&](auto vecc) {
        constexpr bool VEC = decltype(vecc)::value;
        const int64_t row = qt * 32 + i;
        if (row < g.Sq) {
#pragma unroll
            for (int dt = 0; dt < DT; ++dt)
#pragma unroll
                for (int gq = 0; gq < 4; ++gq) {
                    const int d = dt * 32 + 8 * gq + 4 * h;
                    if (d < (int)g.D) {                      // D is a multiple of 16: four elements or none
                        float* dst = O + row * g.ldo + d;
                        if constexpr (VEC) {
                            *reinterpret_cast<float4*>(dst) = make_float4(o[dt][4 * gq], o[dt][4 * gq + 1],
                                                                          o[dt][4 * gq + 2], o[dt][4 * gq + 3]);
                        } else {
#pragma unroll
                            for (int j = 0; j < 4; ++j) dst[j] = o[dt][4 * gq + j];
                        }
                    }
                }
        }
    };
    if (g.vec) store(std::true_type{}); else store(std::false_type{});
}

// ------------------------------------------------------------------------------------------------
// Few queries (decoding, chunks of a prompt, few heads): a workgroup of eight waves owns 32 queries of one head and 32*DTW
// columns of the result; its waves take the key tiles round-robin in both sweeps, with operands straight from global
// memory (the layout is the lane order), and meet twice: for the row statistics between the sweeps and for the sum of
// their partial results at the end, both in wave order through LDS.  The arithmetic on a key tile is that of the kernel
// above.
// ------------------------------------------------------------------------------------------------
constexpr int kSplitWaves = 8;
constexpr int kSplitPitch = 65;                         // floats per result register of 64 lanes, skewed over the banks

// The waves' partial results, one tile of 32 columns after the other: every output is one thread's sum over the waves.  Two
// buffers: the next tile is written while slower threads still read this one.
template <int DTW>
__device__ __forceinline__ void add_waves(const AttnArgs& g, const v16f (&o)[DTW], float* red, int wave, int lane, int64_t bz, int64_t qt,
                                          int part) {
    constexpr int NW = kSplitWaves, PITCH = kSplitPitch;
    float* O = g.O + bz * g.o_batch_stride;
#pragma unroll
    for (int dt = 0; dt < DTW; ++dt) {
        float* buf = red + (dt & 1) * NW * 16 * PITCH;
#pragma unroll
        for (int r = 0; r < 16; ++r) buf[(wave * 16 + r) * PITCH + lane] = o[dt][r];
        __syncthreads();
        for (int t = threadIdx.x; t < 1024; t += NW * 64) {
            // register r of lane 32h + i is element 8*(r/4) + 4h + r%4 of the tile's 32, query i
            const int q = t >> 5, e = t & 31, r = 4 * (e >> 3) + (e & 3), l = 8 * (e & 4) + q;
            float sum = 0.f;
#pragma unroll
            for (int w = 0; w < NW; ++w) sum += buf[(w * 16 + r) * PITCH + l];
            const int64_t row = qt * 32 + q;
            const int d = (part * DTW + dt) * 32 + e;
            if (row < g.Sq && d < (int)g.D) O[row * g.ldo + d] = sum;
        }
    }
}

template <int KS, int DTW, int RND>
__global__ __launch_bounds__(kSplitWaves * 64) void attention_split_kernel(AttnArgs g) {
    constexpr int NW = kSplitWaves, NK = 2 * KS;
    __shared__ float stat[2][NW][64];
    extern __shared__ __attribute__((aligned(16))) float red[];       // [1 or 2][NW][16][kSplitPitch]
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int i = lane & 31, h = lane >> 5;
    // an XCD gets one contiguous range of (head, query tile, column part): those of a head share its K and V in the L2
    const int64_t per_xcd = (g.total + 7) / 8;
    const int64_t lin = (blockIdx.x % 8) * per_xcd + blockIdx.x / 8;
    if (blockIdx.x / 8 >= per_xcd || lin >= g.total) return;          // whole workgroup, before any barrier
    const int part = (int)(lin % g.parts);
    const int64_t tq = lin / g.parts, bz = tq / g.tiles_q, qt = tq - bz * g.tiles_q;
    const uint8_t* Kbase = g.K + bz * g.matrixK;
    const uint8_t* Vbase = g.V + bz * g.matrixV + (int64_t)part * DTW * g.v_ksteps * kBfUnitBytes;
    const uint32_t lane16 = lane * 16;

    // the wave's Q fragments and the permuted K rows: as in the kernel above
    const int flip = g.c < 0.f ? (int)0x80008000u : 0;
    const float c = __builtin_fabsf(g.c);
    v4i qf[NK];
#pragma unroll
    for (int kk = 0; kk < NK; ++kk) {
        qf[kk] = *reinterpret_cast<const v4i*>(g.Q + bz * g.matrixQ + (qt * KS + (kk >> 1)) * kBfUnitBytes + (kk & 1) * 1024 + lane16);
#pragma unroll
        for (int d = 0; d < 4; ++d) qf[kk][d] ^= flip;
    }
    const int sig = (i & 0x13) | ((i & 4) << 1) | ((i & 8) >> 1);
    const uint32_t koff = (32 * h + sig) * 16;

    v4i kf[NK];
    auto fetch_k = [&](int64_t kt) {                    // past the end: the last tile again (loaded, not used)
        kt = kt < g.nt ? kt : g.nt - 1;
#pragma unroll
        for (int kk = 0; kk < NK; ++kk)
            kf[kk] = *reinterpret_cast<const v4i*>(Kbase + (kt * KS + (kk >> 1)) * kBfUnitBytes + (kk & 1) * 1024 + koff);
    };
    v16f s;
    auto scores = [&]() {
#pragma unroll
        for (int r = 0; r < 16; ++r) s[r] = 0.f;
#pragma unroll
        for (int kk = 0; kk < NK; ++kk)
            s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(v8bf, kf[kk]), __builtin_bit_cast(v8bf, qf[kk]), s, 0, 0, 0);
    };
    // only the last key tile can hold keys past Sk; this lane's key 16*b + e is real iff 16*b + e < valid
    const bool ragged = (g.Sk & 31) != 0;
    const int valid = (int)(g.Sk - (g.nt - 1) * 32) - 8 * h;

    float m_run = -__builtin_inff(), l_run = 0.f;
    fetch_k(wave);
    for (int64_t kt = wave; kt < g.nt; kt += NW) {
        scores();
        fetch_k(kt + NW);
        auto tile = [&](auto ragc) {
            constexpr bool RAG = decltype(ragc)::value;
            auto masked = [&](int r) { return RAG && 16 * (r >> 3) + (r & 7) >= valid; };
            float sm = -__builtin_inff();
#pragma unroll
            for (int r = 0; r < 16; ++r) sm = __builtin_fmaxf(sm, masked(r) ? -__builtin_inff() : s[r]);
            const float m_old = m_run;
            m_run = __builtin_fmaxf(m_run, sm * c);
            const float m_use = m_run == -__builtin_inff() ? 0.f : m_run;
            float sum = 0.f;
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                float arg = __builtin_fmaf(s[r], c, -m_use);
                if (masked(r)) arg = -__builtin_inff();               // also when c is 0
                sum += __builtin_amdgcn_exp2f(arg);
            }
            l_run = l_run * __builtin_amdgcn_exp2f(m_old - m_use) + sum;
        };
        if (ragged && kt == g.nt - 1) tile(std::true_type{}); else tile(std::false_type{});
    }

    // row statistics: the waves, and the two lane halves of each, hold disjoint keys of the same query
    fetch_k(wave);                                      // the second sweep's first tile, under the exchange
    stat[0][wave][lane] = m_run;
    stat[1][wave][lane] = l_run;
    __syncthreads();
    float mrow;
    {
        float mf = -__builtin_inff();
#pragma unroll
        for (int w = 0; w < NW; ++w) mf = __builtin_fmaxf(mf, __builtin_fmaxf(stat[0][w][i], stat[0][w][32 + i]));
        float l = 0.f;                                  // mf is finite: there is at least one key
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            l += stat[1][w][i] * __builtin_amdgcn_exp2f(stat[0][w][i] - mf);
            l += stat[1][w][32 + i] * __builtin_amdgcn_exp2f(stat[0][w][32 + i] - mf);
        }
        mrow = mf + __builtin_amdgcn_logf(l);           // the same value in both halves and in every wave
    }

    v16f o[DTW];
#pragma unroll
    for (int dt = 0; dt < DTW; ++dt)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[dt][r] = 0.f;
    const float qmax = (float)((1 << (g.wp - 1)) - 1);
    const int wm2 = g.wp - 2;
    v4i vf[DTW][2];
    auto fetch_v = [&](int64_t kt) {
        kt = kt < g.nt ? kt : g.nt - 1;
#pragma unroll
        for (int dt = 0; dt < DTW; ++dt)
#pragma unroll
            for (int b = 0; b < 2; ++b)
                vf[dt][b] = *reinterpret_cast<const v4i*>(Vbase + (dt * g.v_ksteps + kt) * kBfUnitBytes + b * 1024 + lane16);
    };
    fetch_v(wave);
    for (int64_t kt = wave; kt < g.nt; kt += NW) {
        scores();
        fetch_k(kt + NW);
        v4i pf[2];
        auto tile = [&](auto ragc) {
            constexpr bool RAG = decltype(ragc)::value;
            auto masked = [&](int r) { return RAG && 16 * (r >> 3) + (r & 7) >= valid; };
            float sm[2], off[2];
            int t[2];
#pragma unroll
            for (int b = 0; b < 2; ++b) {
                sm[b] = -__builtin_inff();
#pragma unroll
                for (int e = 0; e < 8; ++e) sm[b] = __builtin_fmaxf(sm[b], masked(8 * b + e) ? -__builtin_inff() : s[8 * b + e]);
            }
            block_scales(g, sm[0], sm[1], c, mrow, wm2, off, t);
#pragma unroll
            for (int b = 0; b < 2; ++b) {
                float el[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    float arg = __builtin_fmaf(s[8 * b + e], c, off[b]);
                    if (masked(8 * b + e)) arg = -__builtin_inff();
                    const float sc = __builtin_amdgcn_exp2f(arg);
                    float v = RND == MX_RNE ? __builtin_rintf(sc) : __builtin_truncf(sc);
                    v = __builtin_fminf(v, qmax);                     // probabilities are not negative
                    el[e] = __builtin_ldexpf(v, t[b]);                // an exact bfloat16 number
                }
#pragma unroll
                for (int d = 0; d < 4; ++d)                           // the upper halves of two fp32 values
                    pf[b][d] = (int)__builtin_amdgcn_perm(__float_as_uint(el[2 * d + 1]), __float_as_uint(el[2 * d]), 0x07060302u);
            }
        };
        if (ragged && kt == g.nt - 1) tile(std::true_type{}); else tile(std::false_type{});
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int dt = 0; dt < DTW; ++dt)
                o[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(v8bf, vf[dt][b]), __builtin_bit_cast(v8bf, pf[b]), o[dt], 0, 0, 0);
        fetch_v(kt + NW);
    }

    add_waves<DTW>(g, o, red, wave, lane, bz, qt, part);
}

// ------------------------------------------------------------------------------------------------
// Few queries and 17 to 64 key tiles: the split kernel with the scores kept.  A workgroup of eight waves owns 32 queries of one
// head and 32*DTW columns of the result, its waves take the key tiles round-robin, at most T each, and hold the scores of
// all of them in registers between the row statistics and the second product: K is read and multiplied once.
//
// Bound: vector issue, about 900 cycles per key tile of which an exponential is 8, and the K and V^T of a head that one
// compute unit loads.  With the scores taken again in a second sweep 32 heads x 100 queries x 2048 keys x 128 took 21.4 us, 16.5 this
// way, 32 x 512 x 2048 x 128 43.3 and 33.1, 24 x 700 x 2048 x 128 58.8 and 44.5.
// A wave requests one tile of K ahead and one or two of V^T, the first under the exchange of the row statistics (two of K and
// four of V^T: 32 x 1 x 1936 x 128 13.2 for 12.7 us, 32 x 100 x 2048 x 128 16.7 for 16.2, 4 percent over 40 random shapes).
// Loads past the last key tile are out of the buffer's range: they read zeros and touch no memory, so none sits under a
// condition.
// ------------------------------------------------------------------------------------------------
template <int KS, int DTW, int T, int RND>
__global__ __launch_bounds__(kSplitWaves * 64, 2) void attention_kept_kernel(AttnArgs g) {
    constexpr int NW = kSplitWaves, NK = 2 * KS, RV = DTW == 1 ? 2 : 1;
    __shared__ float stat[2][NW][64];
    extern __shared__ __attribute__((aligned(16))) float red[];       // [1 or 2][NW][16][kSplitPitch]
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int i = lane & 31, h = lane >> 5;
    // an XCD gets one contiguous range of (head, query tile, column part): those of a head share its K and V in the L2
    const int64_t per_xcd = (g.total + 7) / 8;
    const int64_t lin = (blockIdx.x % 8) * per_xcd + blockIdx.x / 8;
    if (blockIdx.x / 8 >= per_xcd || lin >= g.total) return;          // whole workgroup, before any barrier
    const int part = (int)(lin % g.parts);
    const int64_t tq = lin / g.parts, bz = tq / g.tiles_q, qt = tq - bz * g.tiles_q;
    const int nt = (int)g.nt, v_row = (int)g.v_ksteps * kBfUnitBytes;
    const BufRsrc rK = make_rsrc(g.K + bz * g.matrixK, (uint32_t)(nt * KS * kBfUnitBytes));
    const BufRsrc rV = make_rsrc(g.V + bz * g.matrixV + (int64_t)part * DTW * v_row, (uint32_t)(DTW * v_row));
    constexpr uint32_t kNowhere = 0x40000000u;          // past the end of either buffer
    const uint32_t lane16 = lane * 16;

    // The wave's Q fragments and the permuted K rows: as in attention_bf16_kernel.  A scale of zero is a Q of zeros, so that a
    // masked score of -inf stays one.
    const int flip = g.c < 0.f ? (int)0x80008000u : 0, keep = g.c == 0.f ? 0 : -1;
    const float c = g.c == 0.f ? 1.f : __builtin_fabsf(g.c);
    v4i qf[NK];
#pragma unroll
    for (int kk = 0; kk < NK; ++kk) {
        qf[kk] = *reinterpret_cast<const v4i*>(g.Q + bz * g.matrixQ + (qt * KS + (kk >> 1)) * kBfUnitBytes + (kk & 1) * 1024 + lane16);
#pragma unroll
        for (int d = 0; d < 4; ++d) qf[kk][d] = (qf[kk][d] ^ flip) & keep;
    }
    const int sig = (i & 0x13) | ((i & 4) << 1) | ((i & 8) >> 1);
    const uint32_t koff = (32 * h + sig) * 16;

    v4i kf[NK];
    auto fetch_k = [&](int t) {
        const int kt = wave + t * NW;
        const uint32_t at = koff + (kt < nt ? (uint32_t)(kt * KS * kBfUnitBytes) : kNowhere);
#pragma unroll
        for (int kk = 0; kk < NK; ++kk)
            kf[kk] = __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(rK, at + kk * 1024, 0, 0));
    };
    v4i vf[RV][DTW][2];
    auto fetch_v = [&](int slot, int t) {
        const int kt = wave + t * NW;
        const uint32_t at = lane16 + (kt < nt ? (uint32_t)(kt * kBfUnitBytes) : kNowhere);
#pragma unroll
        for (int dt = 0; dt < DTW; ++dt)
#pragma unroll
            for (int b = 0; b < 2; ++b)
                vf[slot][dt][b] = __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(rV, at + (uint32_t)(dt * v_row) + b * 1024, 0, 0));
    };
    // only the last key tile can hold keys past Sk; this lane's key 16*b + e is real iff 16*b + e < valid
    const bool ragged = (g.Sk & 31) != 0;
    const int valid = (int)(g.Sk - (g.nt - 1) * 32) - 8 * h;

    v16f s[T];
    float m_run = -__builtin_inff(), l_run = 0.f;
    fetch_k(0);
#pragma unroll
    for (int t = 0; t < T; ++t) {
        const int kt = wave + t * NW;
        if (kt >= nt) break;
#pragma unroll
        for (int r = 0; r < 16; ++r) s[t][r] = 0.f;
#pragma unroll
        for (int kk = 0; kk < NK; ++kk)
            s[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(v8bf, kf[kk]), __builtin_bit_cast(v8bf, qf[kk]), s[t], 0, 0, 0);
        if (t + 1 < T) fetch_k(t + 1);
        if (ragged && kt == nt - 1) {
#pragma unroll
            for (int r = 0; r < 16; ++r) s[t][r] = 16 * (r >> 3) + (r & 7) >= valid ? -__builtin_inff() : s[t][r];
        }
        float sm = s[t][0];
#pragma unroll
        for (int r = 1; r < 16; ++r) sm = __builtin_fmaxf(sm, s[t][r]);
        const float m_old = m_run;
        m_run = __builtin_fmaxf(m_run, sm * c);
        const float m_use = m_run == -__builtin_inff() ? 0.f : m_run;          // no key in this lane's tiles so far
        float sum = 0.f;
#pragma unroll
        for (int r = 0; r < 16; ++r) sum += __builtin_amdgcn_exp2f(__builtin_fmaf(s[t][r], c, -m_use));
        l_run = l_run * __builtin_amdgcn_exp2f(m_old - m_use) + sum;
    }

    // row statistics: the waves, and the two lane halves of each, hold disjoint keys of the same query
#pragma unroll
    for (int t = 0; t < RV; ++t) fetch_v(t, t);
    stat[0][wave][lane] = m_run;
    stat[1][wave][lane] = l_run;
    __syncthreads();
    float mrow;
    {
        float mf = -__builtin_inff();
#pragma unroll
        for (int w = 0; w < NW; ++w) mf = __builtin_fmaxf(mf, __builtin_fmaxf(stat[0][w][i], stat[0][w][32 + i]));
        float l = 0.f;                                  // mf is finite: there is at least one key
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            l += stat[1][w][i] * __builtin_amdgcn_exp2f(stat[0][w][i] - mf);
            l += stat[1][w][32 + i] * __builtin_amdgcn_exp2f(stat[0][w][32 + i] - mf);
        }
        mrow = mf + __builtin_amdgcn_logf(l);           // the same value in both halves and in every wave
    }

    v16f o[DTW];
#pragma unroll
    for (int dt = 0; dt < DTW; ++dt)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[dt][r] = 0.f;
    const float qmax = (float)((1 << (g.wp - 1)) - 1);
    const int wm2 = g.wp - 2;
#pragma unroll
    for (int t = 0; t < T; ++t) {
        if (wave + t * NW >= nt) break;
        float sm[2], off[2];
        int te[2];
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            sm[b] = s[t][8 * b];
#pragma unroll
            for (int e = 1; e < 8; ++e) sm[b] = __builtin_fmaxf(sm[b], s[t][8 * b + e]);
        }
        block_scales(g, sm[0], sm[1], c, mrow, wm2, off, te);
        v4i pf[2];
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            float el[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const float sc = __builtin_amdgcn_exp2f(__builtin_fmaf(s[t][8 * b + e], c, off[b]));
                float v = RND == MX_RNE ? __builtin_rintf(sc) : __builtin_truncf(sc);
                v = __builtin_fminf(v, qmax);                     // probabilities are not negative
                el[e] = __builtin_ldexpf(v, te[b]);               // an exact bfloat16 number
            }
#pragma unroll
            for (int d = 0; d < 4; ++d)                           // the upper halves of two fp32 values
                pf[b][d] = (int)__builtin_amdgcn_perm(__float_as_uint(el[2 * d + 1]), __float_as_uint(el[2 * d]), 0x07060302u);
        }
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int dt = 0; dt < DTW; ++dt)
                o[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(v8bf, vf[t % RV][dt][b]), __builtin_bit_cast(v8bf, pf[b]), o[dt], 0, 0, 0);
        if (t + RV < T) fetch_v(t % RV, t + RV);
    }
    add_waves<DTW>(g, o, red, wave, lane, bz, qt, part);
}

// ------------------------------------------------------------------------------------------------
// Decoding, one to sixteen queries and up to 64 key tiles: attention_kept_kernel on 16 x 16 results, so that the vector work on a
// key tile is half of what 32 queries take.  A workgroup of eight waves owns all queries of one head and 32*DTW columns of the
// result.
//
// S^T of a tile of 32 keys is two results of 16 keys x 16 queries, the K rows of which are read so that lane 16g + j holds keys
// 8g .. 8g+7 of query j: the operand of O^T = V^T P^T, and one half of one block of 16 keys, so that a lane has one exponent.
//
// Bound: the serial chain of one workgroup.  Of 11.2 us for 32 heads x 1 query x 1936 keys x 128 a launch that does next to nothing
// takes 3.6; the loads of a compute unit, K of a head and 32 columns of V^T in each of the four workgroups that share it, take
// 4.4 (0.6 MB at 64 bytes per cycle); what is left is the waits between the tiles of a wave and its two meetings with the
// others, which nothing tells apart (vector ALUs of the busy units active 38 percent, matrix cores 10).  Against the kernels that
// it took the place of (scores taken twice, for 1000 heads 128 queries per workgroup): 15.7 -> 11.2 us, 8 x 1 x 2048 x 64 12.2 -> 7.3,
// 32 x 8 x 1024 x 128 10.4 -> 7.4, 32 x 3 x 512 x 128 7.3 -> 5.4, 1000 x 1 x 512 x 128 72 -> 45.  Sixteen waves: 4 to 10 percent more.
// ------------------------------------------------------------------------------------------------
template <int KS, int DTW, int T, int RND>
__global__ __launch_bounds__(kSplitWaves * 64, 2) void attention_short_kernel(AttnArgs g) {
    constexpr int NW = kSplitWaves;
    __shared__ float stat[2][NW][16];
    extern __shared__ __attribute__((aligned(16))) float red[];       // [1 or 2][NW][8][kSplitPitch]
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int j = lane & 15, o8 = lane >> 4;
    // an XCD gets one contiguous range of (head, column part): those of a head share its K and V in the L2
    const int64_t per_xcd = (g.total + 7) / 8;
    const int64_t lin = (blockIdx.x % 8) * per_xcd + blockIdx.x / 8;
    if (blockIdx.x / 8 >= per_xcd || lin >= g.total) return;          // whole workgroup, before any barrier
    const int part = (int)(lin % g.parts);
    const int64_t bz = lin / g.parts;
    const int nt = (int)g.nt, v_row = (int)g.v_ksteps * kBfUnitBytes;
    const BufRsrc rK = make_rsrc(g.K + bz * g.matrixK, (uint32_t)(nt * KS * kBfUnitBytes));
    const BufRsrc rV = make_rsrc(g.V + bz * g.matrixV + (int64_t)part * DTW * v_row, (uint32_t)(DTW * v_row));
    constexpr uint32_t kNowhere = 0x40000000u;          // past the end of either buffer
    // 16 bytes of row r, elements 8*o8 .. 8*o8+7 of a unit's 32
    const uint32_t oct = (o8 >> 1) * 1024 + (o8 & 1) * 512;

    // a scale below zero or of zero: as in attention_kept_kernel
    const int flip = g.c < 0.f ? (int)0x80008000u : 0, keep = g.c == 0.f ? 0 : -1;
    const float c = g.c == 0.f ? 1.f : __builtin_fabsf(g.c);
    v4i qf[KS];
#pragma unroll
    for (int kk = 0; kk < KS; ++kk) {
        qf[kk] = *reinterpret_cast<const v4i*>(g.Q + bz * g.matrixQ + kk * kBfUnitBytes + oct + j * 16);
#pragma unroll
        for (int d = 0; d < 4; ++d) qf[kk][d] = (qf[kk][d] ^ flip) & keep;
    }
    const uint32_t koff = oct + (8 * (j >> 2) + (j & 3)) * 16;

    v4i kf[2 * KS];                                     // the first and the second four keys of every eight
    auto fetch_k = [&](int t) {
        const int kt = wave + t * NW;
        const uint32_t at = koff + (kt < nt ? (uint32_t)(kt * KS * kBfUnitBytes) : kNowhere);
#pragma unroll
        for (int kk = 0; kk < 2 * KS; ++kk)
            kf[kk] = __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(rK, at + (kk >> 1) * kBfUnitBytes + (kk & 1) * 64, 0, 0));
    };
    v4i vf[2 * DTW];
    auto fetch_v = [&](int t) {
        const int kt = wave + t * NW;
        const uint32_t at = oct + j * 16 + (kt < nt ? (uint32_t)(kt * kBfUnitBytes) : kNowhere);
#pragma unroll
        for (int x = 0; x < 2 * DTW; ++x)
            vf[x] = __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(rV, at + (uint32_t)((x >> 1) * v_row) + (x & 1) * 256, 0, 0));
    };
    // only the last key tile can hold keys past Sk; this lane's key e is real iff e < valid
    const bool ragged = (g.Sk & 31) != 0;
    const int valid = (int)(g.Sk - (g.nt - 1) * 32) - 8 * o8;

    float s[T][8];
    float m_run = -__builtin_inff(), l_run = 0.f;
    fetch_k(0);
#pragma unroll
    for (int t = 0; t < T; ++t) {
        const int kt = wave + t * NW;
        if (kt >= nt) break;
        v4f d[2];
#pragma unroll
        for (int x = 0; x < 2; ++x) {
            d[x] = v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int kk = 0; kk < KS; ++kk)
                d[x] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(v8bf, kf[2 * kk + x]), __builtin_bit_cast(v8bf, qf[kk]), d[x], 0, 0, 0);
        }
        if (t + 1 < T) fetch_k(t + 1);
#pragma unroll
        for (int e = 0; e < 8; ++e) s[t][e] = d[e >> 2][e & 3];
        if (ragged && kt == nt - 1) {
#pragma unroll
            for (int e = 0; e < 8; ++e) s[t][e] = e >= valid ? -__builtin_inff() : s[t][e];
        }
        float sm = s[t][0];
#pragma unroll
        for (int e = 1; e < 8; ++e) sm = __builtin_fmaxf(sm, s[t][e]);
        const float m_old = m_run;
        m_run = __builtin_fmaxf(m_run, sm * c);
        const float m_use = m_run == -__builtin_inff() ? 0.f : m_run;          // no key in this lane's tiles so far
        float sum = 0.f;
#pragma unroll
        for (int e = 0; e < 8; ++e) sum += __builtin_amdgcn_exp2f(__builtin_fmaf(s[t][e], c, -m_use));
        l_run = l_run * __builtin_amdgcn_exp2f(m_old - m_use) + sum;
    }

    // row statistics: the four lane groups of a wave, then the waves, hold disjoint keys of the same query
    fetch_v(0);
#pragma unroll
    for (int step = 16; step <= 32; step *= 2) {
        const float mo = __shfl_xor(m_run, step, 64), lo = __shfl_xor(l_run, step, 64);
        const float mf = __builtin_fmaxf(m_run, mo), m_use = mf == -__builtin_inff() ? 0.f : mf;
        l_run = l_run * __builtin_amdgcn_exp2f(m_run - m_use) + lo * __builtin_amdgcn_exp2f(mo - m_use);
        m_run = mf;
    }
    if (lane < 16) {
        stat[0][wave][j] = m_run;
        stat[1][wave][j] = l_run;
    }
    __syncthreads();
    float mrow;
    {
        float mf = -__builtin_inff();
#pragma unroll
        for (int w = 0; w < NW; ++w) mf = __builtin_fmaxf(mf, stat[0][w][j]);
        float l = 0.f;                                  // mf is finite: there is at least one key
#pragma unroll
        for (int w = 0; w < NW; ++w) l += stat[1][w][j] * __builtin_amdgcn_exp2f(stat[0][w][j] - mf);
        mrow = mf + __builtin_amdgcn_logf(l);           // the same value in every lane group and wave
    }

    v4f o[2 * DTW];
#pragma unroll
    for (int x = 0; x < 2 * DTW; ++x) o[x] = v4f{0.f, 0.f, 0.f, 0.f};
    const float qmax = (float)((1 << (g.wp - 1)) - 1);
    const int wm2 = g.wp - 2;
#pragma unroll
    for (int t = 0; t < T; ++t) {
        if (wave + t * NW >= nt) break;
        float sm = s[t][0], off;
#pragma unroll
        for (int e = 1; e < 8; ++e) sm = __builtin_fmaxf(sm, s[t][e]);
        int te;
        block_scale(g, sm, c, mrow, wm2, off, te);
        float el[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const float sc = __builtin_amdgcn_exp2f(__builtin_fmaf(s[t][e], c, off));
            float v = RND == MX_RNE ? __builtin_rintf(sc) : __builtin_truncf(sc);
            v = __builtin_fminf(v, qmax);                         // probabilities are not negative
            el[e] = __builtin_ldexpf(v, te);                      // an exact bfloat16 number
        }
        v4i pf;
#pragma unroll
        for (int d = 0; d < 4; ++d)                               // the upper halves of two fp32 values
            pf[d] = (int)__builtin_amdgcn_perm(__float_as_uint(el[2 * d + 1]), __float_as_uint(el[2 * d]), 0x07060302u);
#pragma unroll
        for (int x = 0; x < 2 * DTW; ++x)
            o[x] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(v8bf, vf[x]), __builtin_bit_cast(v8bf, pf), o[x], 0, 0, 0);
        if (t + 1 < T) fetch_v(t + 1);
    }

    // the waves' partial results as in add_waves: 32 columns are two results of 16 columns x 16 queries, of which register r of
    // lane 16g + j is column 4g + r of query j
    float* O = g.O + bz * g.o_batch_stride;
#pragma unroll
    for (int dt = 0; dt < DTW; ++dt) {
        float* buf = red + (dt & 1) * NW * 8 * kSplitPitch;
#pragma unroll
        for (int r = 0; r < 8; ++r) buf[(wave * 8 + r) * kSplitPitch + lane] = o[2 * dt + (r >> 2)][r & 3];
        __syncthreads();
        for (int t = threadIdx.x; t < 512; t += NW * 64) {
            const int q = t >> 5, e = t & 31, r = 4 * (e >> 4) + (e & 3), l = 16 * ((e >> 2) & 3) + q;
            const int d = (part * DTW + dt) * 32 + e;
            if (q < g.Sq && d < (int)g.D) {
                float sum = 0.f;
#pragma unroll
                for (int w = 0; w < NW; ++w) sum += buf[(w * 8 + r) * kSplitPitch + l];
                O[q * g.ldo + d] = sum;
            }
        }
    }
}

// One of the kernels for few queries: a workgroup per 32 queries and column part.
mx_status launch_few(AttnArgs& g, void (*kern)(AttnArgs), std::atomic<uint64_t>& done, int smem, int64_t batch, int parts, hipStream_t st) {
    if (!allow_dynamic_lds((const void*)kern, smem, done)) return MX_ERR_DEVICE;
    g.tiles_q = g.q_tiles;
    g.parts = parts;
    g.total = g.tiles_q * batch * parts;
    if (g.total > 0x7fffff00LL) return MX_ERR_UNSUPPORTED;
    dim3 grid((unsigned)(ceil_div(g.total, 8) * 8));
    hipLaunchKernelGGL(kern, grid, dim3(kSplitWaves * 64), smem, st, g);
    MX_HIP_LAUNCH_CHECK();
    return MX_OK;
}
constexpr int few_lds(int dtw, int regs) { return (dtw == 1 ? 1 : 2) * kSplitWaves * regs * kSplitPitch * 4; }

template <int KS, int DTW>
mx_status launch_attention_split(AttnArgs& g, int64_t batch, int parts, int rnd, hipStream_t st) {
    static std::atomic<uint64_t> done[2];
    auto kern = rnd == MX_RNE ? attention_split_kernel<KS, DTW, MX_RNE> : attention_split_kernel<KS, DTW, MX_RTZ>;
    return launch_few(g, kern, done[rnd == MX_RNE], few_lds(DTW, 16), batch, parts, st);
}

template <int KS, int DTW, int T>
mx_status launch_attention_kept(AttnArgs& g, int64_t batch, int parts, int rnd, hipStream_t st) {
    static std::atomic<uint64_t> done[2];
    auto kern = rnd == MX_RNE ? attention_kept_kernel<KS, DTW, T, MX_RNE> : attention_kept_kernel<KS, DTW, T, MX_RTZ>;
    return launch_few(g, kern, done[rnd == MX_RNE], few_lds(DTW, 16), batch, parts, st);
}

template <int KS, int DTW, int T>
mx_status launch_attention_short(AttnArgs& g, int64_t batch, int parts, int rnd, hipStream_t st) {
    static std::atomic<uint64_t> done[2];
    auto kern = rnd == MX_RNE ? attention_short_kernel<KS, DTW, T, MX_RNE> : attention_short_kernel<KS, DTW, T, MX_RTZ>;
    return launch_few(g, kern, done[rnd == MX_RNE], few_lds(DTW, 8), batch, parts, st);
}

template <int KS, int DTW>
mx_status pick_short(AttnArgs& g, int64_t batch, int parts, int rnd, hipStream_t st) {
    if (g.nt <= 2 * kSplitWaves) return launch_attention_short<KS, DTW, 2>(g, batch, parts, rnd, st);
    if (g.nt <= 4 * kSplitWaves) return launch_attention_short<KS, DTW, 4>(g, batch, parts, rnd, st);
    return launch_attention_short<KS, DTW, 8>(g, batch, parts, rnd, st);
}

template <int KS, int DT, bool LAG>
mx_status launch_attention(AttnArgs& g, int64_t batch, int rnd, hipStream_t st) {
    constexpr int smem = kAttnStages * (KS + DT) * kBfUnitBytes;
    static_assert(smem * 2 <= 160 * 1024, "LDS budget of one compute unit");
    auto k0 = attention_bf16_kernel<KS, DT, MX_RNE, LAG>;
    auto k1 = attention_bf16_kernel<KS, DT, MX_RTZ, LAG>;
    static std::atomic<uint64_t> done0{0}, done1{0};
    if (!allow_dynamic_lds((const void*)k0, smem, done0) || !allow_dynamic_lds((const void*)k1, smem, done1))
        return MX_ERR_DEVICE;
    g.tiles_q = ceil_div(g.Sq, 128);
    g.total = g.tiles_q * batch;
    if (g.total > 0x7fffff00LL) return MX_ERR_UNSUPPORTED;
    dim3 grid((unsigned)(ceil_div(g.total, 8) * 8));
    hipLaunchKernelGGL(rnd == MX_RNE ? k0 : k1, grid, dim3(256), smem, st, g);
    MX_HIP_LAUNCH_CHECK();
    return MX_OK;
}

template <int KS, int DTW>
mx_status pick_kept(AttnArgs& g, int64_t batch, int parts, int rnd, hipStream_t st) {
    if constexpr (KS == 4)
        if (g.nt <= 4 * kSplitWaves) return launch_attention_kept<KS, DTW, 4>(g, batch, parts, rnd, st);
    return launch_attention_kept<KS, DTW, 8>(g, batch, parts, rnd, st);
}

// Heads of more than 64 elements, see pick_attention.
bool keeps_scores(const AttnArgs& g, int64_t groups, int64_t batch) {
    const int64_t rounds = ceil_div(groups, 256);
    if (g.nt <= 16 || g.nt > 64) return false;
    if (rounds <= 3) return rounds <= 2 || g.nt >= 24;
    return rounds <= 5 && g.nt >= 40 && ceil_div(g.Sq, 128) * batch > 256;
}

// The split kernel takes one round of workgroups in a time that hardly depends on the number of keys while they are few,
// the 128-query workgroups one tile of keys at a time for as long whether there is one of them or 256: with one round
// the split kernel is the faster one (8 heads x 512 queries x 2048 keys x 128: 70 us, 22 us split) from the second key tile
// on (100 heads x 55 queries x 128, 32 keys: 6.5 and 7.2 us, 64 keys: 0.94 of the time and less), with two from ten key tiles on (16 x 1024 x 256 x 128: 15.0 and 16.3 us, 16 x 1024 x 320 x 96: 16.6
// and 15.1 us, 32 x 512 x 2048 x 128: 74 and 45 us), with three from about forty (24 x 1024 x 960 x 128: 38.6 and 39.6 us,
// 24 x 1024 x 2048 x 128: 75 and 64 us), beyond that no more (16 x 2040 x 2048 x 128: 71 and 81 us).
// With room for it every 32 columns of the result get a workgroup of their own, which
// repeats the scores and saves registers, V and the sum (32 heads, one query, 1936 keys: 16.8 against 20.0 us); with more
// than one such workgroup per compute unit that costs more than it saves (32 x 100 x 2048 x 128: 35 against 22 us).
// Up to sixteen queries take attention_short_kernel up to 64 key tiles (52 random shapes of 8 to 2000 heads, 2 to 64 key tiles: 0.55
// to 1.02 of the time of what the rules below pick).  64 is where its forms end, eight tiles per wave in 98 to 136 registers; one
// for more keys would fit the registers but has not been built, so they take the scores twice.
// The scores are kept (attention_kept_kernel) from 17 key tiles on where heads have more than 64 elements: in one round of
// workgroups always (us, scores taken twice and kept: 17 tiles 10.8 and 10.0, 32 tiles 14.9 and 12.5, 54 tiles 18.8 and 15.6), in two as
// well (297 workgroups x 17 tiles 19.8 and 17.9, 360 x 62 40.3 and 31.6; up to 16 tiles, 405 x 12, 16.7 and 17.3), in three from
// 24 tiles on against the 128-query workgroups (744 x 41 43.1 and 34.3, 540 x 30 33.9 and 30.5, 713 x 21 27.6 and 27.9), in four and five
// from 40 on if there are more than 256 of those (988 x 42 61.5 and 44.3, 1088 x 47 67.4 and 61.2; 961 x 30 34.9 and 36.7, six
// rounds 1335 x 47 69.3 and 72.4).  Heads of up to 64 elements in one round from 33 tiles on (209 x 46 12.2 and 11.3; 232 x 17
// 7.1 and 7.9): with fewer, two workgroups of the other form share a compute unit.
// The second product of the 128-query form runs one key tile behind its scores (LAG), but not for one or two key tiles, where
// the additional round of it costs more or as much (54 heads x 1828 x 64 x 48: 12.5 and 13.4 us, 32 x 2000 x 64 x 128 15.4
// either way), nor for heads of 33 to 64 elements once a compute unit has more than four workgroups to take: the lag needs 139
// registers for 126, three workgroups at a time for four (106 x 3866 x 128 x 64: 61 and 65 us, 500 x 258 x 352 x 64 43.1 and 44.0, 106 x
// 3866 x 512 x 64 127 and 129; even from 24 to 32 key tiles: 106 x 3866 x 768 x 64 171 and 171, 300 x 512 x 800 x 48 68.3 and 67.2).
// With fewer workgroups the lag pays: 64 x 1024 x 512 x 64 26.1 and 25.0.
template <int KS, int DT>
mx_status pick_attention(AttnArgs& g, int64_t batch, int rnd, hipStream_t st) {
    const int64_t groups = g.q_tiles * batch;
    if (g.Sq <= 16 && g.nt <= 8 * kSplitWaves)
        return groups * DT <= 256 ? pick_short<KS, 1>(g, batch, DT, rnd, st) : pick_short<KS, DT>(g, batch, 1, rnd, st);
    if (KS == 2 ? groups <= 256 && g.nt > 32 && g.nt <= 64 : keeps_scores(g, groups, batch)) {
        if (groups * DT <= 256) return pick_kept<KS, 1>(g, batch, DT, rnd, st);
        return pick_kept<KS, DT>(g, batch, 1, rnd, st);
    }
    if (groups * DT <= 256) return launch_attention_split<KS, 1>(g, batch, DT, rnd, st);
    const int64_t rounds = ceil_div(groups, DT <= 2 ? 512 : 256);      // two workgroups of at most 128 registers share a compute unit
    if (groups <= 768 && g.nt >= (rounds == 1 ? 2 : rounds == 2 ? 10 : 40))
        return launch_attention_split<KS, DT>(g, batch, 1, rnd, st);
    if (g.nt <= 2 || (KS == 2 && DT == 2 && groups > 4096 && g.nt <= 32)) return launch_attention<KS, DT, false>(g, batch, rnd, st);
    return launch_attention<KS, DT, true>(g, batch, rnd, st);
}

}  // namespace

bool matrix_format_ok(const mx_format& f);

}  // namespace mx

using namespace mx;

extern "C" mx_status mx_attention(int64_t batch, int64_t Sq, int64_t Sk, int64_t D, const void* Q_packed, mx_format fq,
                                  const void* K_packed, mx_format fk, const void* Vt_packed, mx_format fv, mx_format fp,
                                  float scale, int32_t layout, float* O, int64_t ldo, int64_t o_batch_stride,
                                  void* stream) {
    if (!format_ok_quant(fq) || !format_ok_quant(fk) || !format_ok_quant(fv) || !format_ok_quant(fp))
        return MX_ERR_BAD_ARG;
    if (fq.block != fk.block || fq.exp_bits != fk.exp_bits || fp.block % fv.block != 0 || fp.exp_bits != fv.exp_bits)
        return MX_ERR_BAD_ARG;
    if (layout != MX_LAYOUT_FRAGMENT && layout != MX_LAYOUT_MATRIX) return MX_ERR_BAD_ARG;
    if (batch < 0 || Sq < 0 || Sk < 1 || D < 1 || D % fq.block != 0 || Sk % fp.block != 0 || ldo < D) return MX_ERR_BAD_ARG;
    if (!(scale == scale) || __builtin_isinf(scale)) return MX_ERR_BAD_ARG;
    // two-row blocks: whole pairs of queries (Q, P), of keys (K), of columns of V (the rows of V^T)
    if (((fq.block_rows == 2 || fp.block_rows == 2) && Sq % 2 != 0) || (fk.block_rows == 2 && Sk % 2 != 0) ||
        (fv.block_rows == 2 && D % 2 != 0))
        return MX_ERR_BAD_ARG;
    // built for the bfloat16 form of the matrix layout, which is declared with blocks of 16.  The packed operands carry
    // their exponents inside the elements, so their block shape (one or two rows) makes no difference here; P's does:
    // its blocks are 16 keys, or 32 (one key tile of the kernel).
    if (layout != MX_LAYOUT_MATRIX || !matrix_format_ok(fq) || !matrix_format_ok(fk) || !matrix_format_ok(fv) ||
        !matrix_format_ok(fp))
        return MX_ERR_UNSUPPORTED;
    if (fq.block != 16 || fv.block != 16 || (fp.block != 16 && fp.block != 32) || D > 128) return MX_ERR_UNSUPPORTED;
    if (batch == 0 || Sq == 0) return MX_OK;
    if (!Q_packed || !K_packed || !Vt_packed || !O || ((uintptr_t)O & 3)) return MX_ERR_BAD_ARG;
    if (batch > 1 && o_batch_stride < (Sq - 1) * ldo + D) return MX_ERR_BAD_ARG;      // heads would overlap
    if (((uintptr_t)Q_packed & 255) || ((uintptr_t)K_packed & 255) || ((uintptr_t)Vt_packed & 255)) return MX_ERR_BAD_ARG;
    const BfGeom gq = bf_geom(Sq, D), gk = bf_geom(Sk, D), gv = bf_geom(D, Sk);
    AttnArgs g;
    g.Q = (const uint8_t*)Q_packed; g.K = (const uint8_t*)K_packed; g.V = (const uint8_t*)Vt_packed; g.O = O;
    g.Sq = Sq; g.Sk = Sk; g.D = D;
    g.matrixQ = gq.matrix; g.matrixK = gk.matrix; g.matrixV = gv.matrix;
    g.q_tiles = gq.row_tiles; g.nt = gk.row_tiles; g.v_ksteps = gv.ksteps;
    g.ldo = ldo; g.o_batch_stride = o_batch_stride;
    g.tiles_q = g.total = 0; g.parts = 1;
    g.c = scale * 1.4426950408889634f;
    g.wp = fp.mant_bits; g.bias_p = (1 << (fp.exp_bits - 1)) - 1;
    g.emax_p = ((1 << fp.exp_bits) - 1) - g.bias_p;
    g.vec = (((uintptr_t)O & 15) == 0 && ldo % 4 == 0 && o_batch_stride % 4 == 0) ? 1 : 0;
    g.pair = fp.block_rows == 2 ? 0.f : -__builtin_inff();
    g.wide = fp.block == 32 ? 0.f : -__builtin_inff();
    g.join = fp.block_rows == 2 || fp.block == 32;
    const int dt = (int)ceil_div(D, 32);
    hipStream_t st = (hipStream_t)stream;
    if (gq.ksteps == 2)
        return dt == 1 ? pick_attention<2, 1>(g, batch, fp.rounding, st) : pick_attention<2, 2>(g, batch, fp.rounding, st);
    return dt == 3 ? pick_attention<4, 3>(g, batch, fp.rounding, st) : pick_attention<4, 4>(g, batch, fp.rounding, st);
}
