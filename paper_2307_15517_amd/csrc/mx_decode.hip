// Decode-time linear layer in one launch (mx_linear, 1..8 activation rows, weights in the fragment layout).
//
// Arithmetic (Section 3.2 of the paper: quantize the input, then the MXInt dot-product operator -- exact
// integer block dots, the two shared exponents applied once per block; format of Section 4.1): the fp32
// activations are quantized with the arithmetic of mx_quantize on their way into on-chip memory, the block
// dots are taken with one int8 MFMA per block, each block's integer is scaled by
// 2^(Ea + Eb - (wa-2) - (wb-2)) and added into an fp32 accumulator.  mx_linear uses this kernel for three
// to eight rows; one and two rows go to the dot-product kernel of mx_gemv_dot.hip, which needs no exchange
// between workgroups.
//
// Work split: the path is bound by one pass over the packed weights, so every compute unit has to stream.  A workgroup
// owns a few neighbouring column groups of 32 (NW) and a K slice, which KS waves per column group divide among them; it
// quantizes its own slice of the activations into LDS, every wave keeps one to four weight records in flight, and the KS
// partial tiles are added through LDS in wave order.  With more than one K slice the partial sums go to the caller's
// workspace and the workgroup that arrives last at the columns' counter adds them in slice order, so the result does
// not depend on the order of arrival.
//
// What a call takes beyond the pass over the weights (8 rows, 8 by 4 bits, blocks of 16, 5120 -> 5120, 5120 -> 13824 and
// 13824 -> 5120: 10.3, 14.7 and 15.3 us; timed on copies of this kernel with the part left out): the exchange between slices,
// three dependent trips to memory, 2.4, 1.9 and 1.6 us (so few slices); quantizing, which every workgroup of a slice repeats,
// 1.5, 1.5 and 3.2 (so wide workgroups); scaling the block sums 1.5, 2.6 and 2.8.  Without all three it takes 5.0, 8.5 and
// 8.3 us, the time of a bare read of the same bytes.  choose_split weighs the first two with the number of workgroups.
// Eight elements per quantizer item (four, and a row found in a loop, before) and waves that divide the slice inside the
// workgroup (slices that meet through memory, before): 12.0 -> 9.5 us, 17.0 -> 14.9 and 17.4 -> 15.0; 5 rows, 6 by 5 bits,
// blocks of 32, 11008 -> 4096 17.2 -> 13.3; 3 rows 768 -> 3072 6.8 -> 4.4.  The 16 x 16 results, of which all elements are used,
// are 0.4 us of 17 of that with blocks of 16 and nothing with blocks of 32.
#include <type_traits>

#include "mx_decode.h"
#include "mx_frag.h"

namespace mx {
namespace {

constexpr int64_t kTargetPairs = 2560;     // (column group, K slice) pairs that the workspace is sized for
constexpr int64_t kMinSlice = 4;           // and records per such slice at least

struct DecodeArgs {
    const float* x;
    int64_t x_stride;
    const uint8_t* B;        // packed weights [groups][chunks] records
    float* Y;
    int64_t ldy;
    uint32_t* counters;      // one per workgroup column: zero on entry, zero again on exit
    float* partial;          // [ksplit][M][32*groups]
    int32_t M, N, K;
    int32_t groups, columns, chunks, ksplit;       // columns of workgroups, K slices
    int32_t slice, part;     // records per slice and per wave
    int32_t recordB;
    int32_t wa, bias, emax, rounding;
    int32_t eadj;            // -bias - (wa-2) - (wb-2)
};

// Weight records a wave keeps in flight: about eight dwords a lane, or one record where it has more (up to 32), requested
// once its activations are quantized.  More of them, or earlier ones, only stand in the way of the activations, which every workgroup waits for first: with five records
// requested ahead of the quantizer 8 rows by 8 and 4 bits, blocks of 16, 5120 -> 5120, 5120 -> 13824 and 13824 -> 5120 took
// 9.9, 14.9 and 15.8 us, with two ahead of it 9.0, 13.9 and 14.9, with two after it 8.9, 13.5 and 14.5 (three 9.1, 14.1, 14.3,
// one 8.9, 14.7, 15.4); 5 rows by 6 and 5 bits, blocks of 32, 4096 -> 4096, 4096 -> 11008 and 11008 -> 4096 five 8.6, 13.0 and 13.1, two
// 7.9, 12.5 and 11.7, one 7.4, 12.4 and 11.0.
constexpr int ring_depth(int wb, int block) {
    const int dw = block * wb / 16;
    return dw <= 2 ? 4 : dw <= 4 ? 2 : 1;
}
constexpr int waves_per_simd(int wb, int block) {
    const int regs = ring_depth(wb, block) * (block * wb / 16 + 1) + (block == 16 ? 65 : block == 32 ? 78 : 110);
    return regs <= 128 ? 4 : regs <= 168 ? 3 : 2;
}

// Grid: (columns of workgroups) x (K slices).  Wave kw * NW + g of a workgroup streams the records of column group
// NW * column + g that belong to part kw of the slice; all share the quantized activations of the slice (LDS).
// Up to eight rows: one int8 MFMA per block (two for block 64), 32 columns at a time (block_mfma16).
template <int B> constexpr int kZeroDw = ((48 + 1) * (B / 8) + 3) & ~3;     // what a lane without codes reads for a record
template <int WB, int B, int NW, int KS>
__global__ __launch_bounds__(NW * KS * 64, waves_per_simd(WB, B))
void linear_splitk_kernel(DecodeArgs a) {
    constexpr int kDwB = Piece<WB, B>::kDw, D = ring_depth(WB, B);
    constexpr int kHalfDw = B / 8;                       // int8 dwords of a half block
    constexpr int MP = 8;                                 // rows with a slot in LDS
    constexpr int MR = 4;                                 // accumulators per lane: rows row0 .. row0 + 3
    constexpr int T = NW * KS * 64;
    extern __shared__ __attribute__((aligned(16))) uint32_t lds[];
    __shared__ int is_last;
    __shared__ uint32_t wide_any[NW * KS];

    const int gq = (int)(blockIdx.x % (unsigned)a.columns), ks = (int)(blockIdx.x / (unsigned)a.columns);
    const int c0 = ks * a.slice;
    const int nc = (a.chunks - c0 < a.slice) ? a.chunks - c0 : a.slice;     // records of this slice, >= 1
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int h = lane >> 5, row = lane & 7;
    const int col = 16 * h + (lane & 15);                 // this lane's column of the results, inside the group
    const int row0 = 4 * ((lane >> 4) & 1);               // and the first of its four rows
    const bool arow = ((lane >> 3) & 1) == ((lane >> 4) & 1);     // the left operand's lane carries codes
    const int kw = wave / NW;                             // this wave's part of the slice
    const int gb = gq * NW + wave - kw * NW;              // this wave's column group
    const bool wave_live = gb < a.groups;                 // wave-uniform

    // LDS: x8[slice*4 blocks][2 halves][8 rows][kHalfDw], xe[slice*4 blocks][8 rows] (bits of 2^Ea), zeros for the other
    // lanes of the left operand
    uint32_t* x8 = lds;
    uint32_t* xe = x8 + MP * a.slice * 4 * 2 * kHalfDw;
    uint32_t* none = xe + MP * a.slice * 4;
    for (int d = (int)threadIdx.x; d < kZeroDw<B>; d += T) none[d] = 0;

    const int w0 = kw * a.part;                           // first record of the wave inside the slice
    const int nw = nc - w0 < 0 ? 0 : nc - w0 < a.part ? nc - w0 : a.part;   // its records, none in the parts past a short slice

    // ring of D records of this wave's column group; a record past the slice reads zeros without touching
    // memory, so no load sits under a condition and the waits stay exact
    const uint8_t* Bbase = a.B + ((int64_t)(wave_live ? gb : 0) * a.chunks + c0 + (nw > 0 ? w0 : 0)) * a.recordB;
    const BufRsrc rB = make_rsrc(Bbase, wave_live ? (uint32_t)(nw * a.recordB) : 0u);
    uint32_t pb[D][kDwB], eb[D];
    auto fetch = [&](int slot, int t) {
        const uint32_t off = (uint32_t)t * (uint32_t)a.recordB;
        buf_load_dwords<kDwB>(rB, off + lane * (kDwB * 4), pb[slot]);
        buf_load_dwords<1>(rB, off + 64 * (kDwB * 4) + col * 4, &eb[slot]);
    };

    bool wide = false;                                    // an exponent of the activations outside [-63, 64]

    // ---- activations of this slice: fp32 -> MXInt (the arithmetic of mx_quantize) -> int8 in LDS.
    // One item is eight consecutive elements of a row, a half block or a part of one; consecutive lanes take consecutive
    // items, so a block is B/8 neighbouring lanes and its maximum takes log2(B/8) DPP steps.  Loads return in the order of
    // issue: the weights are requested after them.
    {
        const int per_row = nc * 4 * B;                    // elements of a row in this slice
        const float qmax = (float)((1 << (a.wa - 1)) - 1);
        const int64_t k0 = (int64_t)c0 * 4 * B;
        constexpr int XU = 4, XR = 2;                      // items per thread requested at first, and at a time after that
        constexpr float kMagic = 12582912.0f;              // 1.5 * 2^23: adding it rounds to an integer, ties to even
        // item -> (row, first element inside the slice), advanced without divisions
        const int step_m = (8 * T) / per_row, step_e = 8 * T - step_m * per_row;
        int m_it = (int)(8 * threadIdx.x) / per_row, e_it = (int)(8 * threadIdx.x) - m_it * per_row;
        auto advance = [&]() {
            m_it += step_m; e_it += step_e;
            if (e_it >= per_row) { e_it -= per_row; ++m_it; }
        };
        auto item_load = [&](int m, int e, float4 (&v)[2]) {
            v[0] = v[1] = make_float4(0.f, 0.f, 0.f, 0.f);
            if (m < a.M && k0 + e < a.K) {                  // K is a multiple of the block
                const float4* src = reinterpret_cast<const float4*>(a.x + (int64_t)m * a.x_stride + k0 + e);
                v[0] = src[0]; v[1] = src[1];
            }
        };
        auto item_store = [&](auto rndc, int m, int e, const float4 (&v)[2]) {
            const float x[8] = {v[0].x, v[0].y, v[0].z, v[0].w, v[1].x, v[1].y, v[1].z, v[1].w};
            auto max4 = [](const float4& f) {
                return __float_as_uint(__builtin_fmaxf(__builtin_fmaxf(__builtin_fabsf(f.x), __builtin_fabsf(f.y)),
                                                       __builtin_fmaxf(__builtin_fabsf(f.z), __builtin_fabsf(f.w))));
            };
            uint32_t ab = max4(v[0]), o = max4(v[1]);
            ab = o > ab ? o : ab;
            o = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)ab, 0xB1, 0xF, 0xF, true);  ab = o > ab ? o : ab;   // lane ^ 1
            if (B >= 32) { o = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)ab, 0x4E, 0xF, 0xF, true); ab = o > ab ? o : ab; }    // lane ^ 2
            if (B >= 64) { o = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)ab, 0x141, 0xF, 0xF, true); ab = o > ab ? o : ab; }   // 7 - lane within 8
            if (m >= a.M) return;                          // after the cross-lane steps: every lane of a block takes part in them
            const int ef = (int)(ab >> 23);
            int E = ef == 0 ? -127 : ef - 127;
            E = E < -a.bias ? -a.bias : E;
            E = E > a.emax ? a.emax : E;
            const int shift = (a.wa - 2) - E;
            // round(x * 2^shift), clamped: the sum with kMagic holds the integer in its low mantissa bits (a
            // value beyond the clamp, however large, ends at the clamp as well), its low byte is the int8 code
            uint32_t z[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                float sc = __builtin_ldexpf(x[k], shift);
                if (decltype(rndc)::value != MX_RNE) sc = __builtin_truncf(sc);
                z[k] = __float_as_uint(__builtin_fminf(__builtin_fmaxf(sc + kMagic, kMagic - qmax), kMagic + qmax));
            }
            uint32_t word[2];
#pragma unroll
            for (int k = 0; k < 2; ++k)
                word[k] = __builtin_amdgcn_perm(z[4 * k + 1], z[4 * k], 0x0C0C0400u) | __builtin_amdgcn_perm(z[4 * k + 3], z[4 * k + 2], 0x04000C0Cu);
            const int blk = e / B, p = e - blk * B;         // block of the slice, position inside it (B is a power of two)
            const int hh = p / (B / 2), d = (p - hh * (B / 2)) >> 2;
            // 2^Ea; a block of zeros takes 1, its sums are zero whatever the scale
            const int ebits = ab == 0 ? 127 : E + 127;
            wide |= (uint32_t)(ebits - (127 - 63)) > 127u;
            *reinterpret_cast<uint2*>(x8 + ((blk * 2 + hh) * 8 + m) * kHalfDw + d) = make_uint2(word[0], word[1]);
            if (p == 0) xe[blk * 8 + m] = (uint32_t)ebits << 23;
        };
        // every thread runs the same number of rounds (the DPP steps need whole blocks of lanes)
        const int rounds = (a.M * per_row + 8 * T - 1) / (8 * T);
        auto load_items = [&](auto& xv, auto& mm, auto& ee) {
            for (auto& v : xv) {
                const int u = (int)(&v - &xv[0]);
                mm[u] = m_it; ee[u] = e_it;
                item_load(m_it, e_it, v);
                advance();
            }
        };
        float4 xv[XU][2];
        int mm[XU], ee[XU];
        load_items(xv, mm, ee);
        auto quantize = [&](auto rndc) {
#pragma unroll
            for (int u = 0; u < XU; ++u)
                if (u < rounds) item_store(rndc, mm[u], ee[u], xv[u]);
#pragma unroll 1
            for (int r = XU; r < rounds; r += XR) {
                float4 yv[XR][2];
                int ym[XR], ye[XR];
                load_items(yv, ym, ye);
#pragma unroll
                for (int u = 0; u < XR; ++u)
                    if (r + u < rounds) item_store(rndc, ym[u], ye[u], yv[u]);
            }
        };
        if (a.rounding == MX_RNE) quantize(std::integral_constant<int, MX_RNE>{});
        else quantize(std::integral_constant<int, MX_RTZ>{});
    }
#pragma unroll
    for (int u = 0; u < D; ++u) fetch(u, u);
    const bool wide_wave = __builtin_amdgcn_ballot_w64(wide) != 0;
    if (lane == 0) wide_any[wave] = wide_wave;
    __syncthreads();
    uint32_t rows_wide = 0;
#pragma unroll
    for (int w = 0; w < NW * KS; ++w) rows_wide |= wide_any[w];

    float acc[MR];
#pragma unroll
    for (int r = 0; r < MR; ++r) acc[r] = 0.f;
    const int per_wave = wave_live ? nw : 0;
    const bool rows_narrow = __builtin_amdgcn_readfirstlane(rows_wide) == 0;
    const bool bcol = (int64_t)gb * 32 + col < a.N;           // columns past N take a neutral exponent
    const uint32_t neutral = (uint32_t)a.bias * 0x01010101u, move = (uint32_t)(127 - a.bias + 32) * 0x01010101u;
    const int eadj = a.eadj - Unpack<WB, B>::kScaleLog2;      // of an exponent byte of the weights
    const uint32_t colbits = (uint32_t)(127 + eadj) << 23;
    v4i_t bias = {(int)kDotBias, (int)kDotBias, (int)kDotBias, (int)kDotBias};
    asm volatile("" : "+v"(bias));                            // four registers, not a constant built per block
    const uint32_t* xa = arow ? x8 + w0 * (64 * kHalfDw) + (h * 8 + row) * kHalfDw : none;
    const int xstep = arow ? 64 * kHalfDw : 0;
    const uint32_t* xs = xe + w0 * 32 + row0;
    for (int t0 = 0; t0 < per_wave; t0 += D) {
#pragma unroll
        for (int u = 0; u < D; ++u) {
            const int c = t0 + u;                             // record inside the wave's part
            const bool live = c < per_wave;                   // scalar condition: no load depends on it
            uint32_t fb[4][kHalfDw];
            uint32_t ebv = 0;
            if (live) {
#pragma unroll
                for (int j = 0; j < 4; ++j) Unpack<WB, B>::run(pb[u], j, fb[j]);
                ebv = bcol ? eb[u] : neutral;
            }
            fetch(u, c + D);                                  // the slot is free: refill it
            if (!live) continue;
            uint32_t fa[4][kHalfDw];
            uint4 ea[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
#pragma unroll
                for (int q = 0; q < kHalfDw; ++q) fa[j][q] = xa[j * 16 * kHalfDw + q];
                ea[j] = *reinterpret_cast<const uint4*>(xs + j * 8);
            }
            xa += xstep;
            xs += 32;
            v4i_t d[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) d[j] = block_mfma16<B>(fa[j], fb[j], bias);
            const bool narrow = rows_narrow && __builtin_amdgcn_ballot_w64((((ebv + move) ^ 0x80808080u) & 0xC0C0C0C0u) != 0) == 0;
            if (narrow) {
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const float sb = __uint_as_float((((ebv >> (8 * j)) & 0xFFu) << 23) + colbits);
                    auto term = [&](int r, uint32_t sa) {
                        const float t = __builtin_fmaf(__uint_as_float((uint32_t)d[j][r]), __uint_as_float(sa), __uint_as_float(sa + kDotBack));
                        acc[r] = __builtin_fmaf(t, sb, acc[r]);
                    };
                    term(0, ea[j].x); term(1, ea[j].y); term(2, ea[j].z); term(3, ea[j].w);
                }
            } else {
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int ebj = (int)((ebv >> (8 * j)) & 0xFFu) + eadj - 127;
                    auto term = [&](int r, uint32_t sa) {
                        acc[r] += __builtin_ldexpf((float)(d[j][r] - (int)kDotBias), (int)(sa >> 23) + ebj);
                    };
                    term(0, ea[j].x); term(1, ea[j].y); term(2, ea[j].z); term(3, ea[j].w);
                }
            }
        }
    }

    if constexpr (KS > 1) {                                   // the parts of the slice, in their order
        float* part = reinterpret_cast<float*>(none + kZeroDw<B>);
        if (kw > 0) {
#pragma unroll
            for (int r = 0; r < MR; ++r) part[((wave - NW) * MR + r) * 64 + lane] = acc[r];
        }
        __syncthreads();
        if (kw == 0) {
#pragma unroll
            for (int k = 0; k < KS - 1; ++k)
#pragma unroll
                for (int r = 0; r < MR; ++r) acc[r] += part[((k * NW + wave) * MR + r) * 64 + lane];
        }
    }

    // ---- a wave's 32 sums per row: the result, or with several K slices this slice's partial sums.  The
    // partial sums are written and read with device-coherent accesses (they pass between workgroups that may
    // sit behind different L2 caches), so no cache has to be written back or invalidated as a whole.
    const int64_t np = (int64_t)a.groups * 32;
    const int64_t n = (int64_t)gb * 32 + col;
    // buffer accesses with the device-scope bit: written through / read at the level every compute unit shares
    constexpr int kDeviceScope = 0x10;
    const BufRsrc rP = make_rsrc(a.partial, (uint32_t)((int64_t)a.ksplit * a.M * np * 4));
    auto put = [&](int m, float s) {
        if (m >= a.M || !wave_live || kw > 0) return;
        if (a.ksplit == 1) { if (n < a.N) a.Y[(int64_t)m * a.ldy + n] = s; }
        else __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(s), rP, (uint32_t)((((int64_t)ks * a.M + m) * np + n) * 4), 0, kDeviceScope);
    };
#pragma unroll
    for (int r = 0; r < 4; ++r) put(row0 + r, acc[r]);
    if (a.ksplit == 1) return;

    // ---- the K slices of this workgroup column: whoever arrives last adds the partial sums in slice order.
    // Order: this thread's partial sums have been written through (the wait), then every thread's (the barrier),
    // then the arrival is counted; the last workgroup reads after it has seen every arrival.
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    if (threadIdx.x == 0) {
        const uint32_t old = __hip_atomic_fetch_add(a.counters + gq, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        is_last = old == (uint32_t)(a.ksplit - 1);
    }
    __syncthreads();
    if (!is_last) return;
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
    // A thread owns up to OPT outputs of the workgroup's columns.  The loads of all of them, eight or sixteen slices at
    // a time, are requested before the first addition (one trip to memory for up to sixteen slices, not one per output
    // or per slice); the additions run in slice order whatever the order of arrival was.  A thread without an output
    // reads the first partial sum and drops it.
    const uint32_t kstride = (uint32_t)(a.M * np * 4);
    constexpr int OPT = (MP * NW * 32 + T - 1) / T;
    uint32_t off0[OPT];
    int64_t col_n[OPT];
    int row_m[OPT];
    float s[OPT];
#pragma unroll
    for (int o = 0; o < OPT; ++o) {
        const int t = (int)threadIdx.x + o * T;
        const int m = t / (NW * 32), col = t - m * (NW * 32);
        const int64_t nn = (int64_t)gq * (NW * 32) + col;
        const bool on = m < a.M && nn < np;
        row_m[o] = on ? m : -1;
        col_n[o] = nn;
        off0[o] = on ? (uint32_t)(((int64_t)m * np + nn) * 4) : 0u;
        s[o] = 0.f;
    }
    auto add_slices = [&](auto kbc) {                     // KB slices per trip
        constexpr int KB = decltype(kbc)::value;
        for (int k0 = 0; k0 < a.ksplit; k0 += KB) {
            uint32_t v[OPT][KB];
#pragma unroll
            for (int o = 0; o < OPT; ++o)
#pragma unroll
                for (int u = 0; u < KB; ++u) {
                    const int k = k0 + u < a.ksplit ? k0 + u : a.ksplit - 1;     // a repeated load instead of a branch
                    v[o][u] = __builtin_amdgcn_raw_buffer_load_b32(rP, off0[o] + (row_m[o] >= 0 ? (uint32_t)k * kstride : 0u), 0, kDeviceScope);
                }
#pragma unroll
            for (int o = 0; o < OPT; ++o)
#pragma unroll
                for (int u = 0; u < KB; ++u)
                    if (k0 + u < a.ksplit) s[o] += __uint_as_float(v[o][u]);
        }
    };
    if (a.ksplit <= 8) add_slices(std::integral_constant<int, 8>{});
    else add_slices(std::integral_constant<int, 16>{});
#pragma unroll
    for (int o = 0; o < OPT; ++o)
        if (row_m[o] >= 0 && col_n[o] < a.N) a.Y[(int64_t)row_m[o] * a.ldy + col_n[o]] = s[o];
    if (threadIdx.x == 0) __hip_atomic_store(a.counters + gq, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// LDS of a workgroup: per record of the slice the codes and scales of eight rows, the zeros, the partial tiles.
constexpr int64_t record_lds(int block) { return (4 * 2 * 8 * (block / 8) + 4 * 8) * 4; }
constexpr int64_t slice_lds(int block, int64_t slice, int groups, int parts) {
    return slice * record_lds(block) + (((48 + 1) * (block / 8) + 3) & ~3) * 4 + (int64_t)(parts - 1) * groups * 4 * 64 * 4;
}
constexpr int kMaxLds = 72 * 1024;

// Column groups of a workgroup, parts of its slice, K slices and the records per part.
struct DecodeSplit { int groups, parts, slices, part; };

// The waves per SIMD that choose_split counts on.  Its coefficients were fitted with them, on kernels whose rings of weight
// records took 25 to 165 registers.  The kernels have room for as many or more, but the split says in what order a row's sums are
// added, so it does not follow the ring.  With waves_per_simd in their place 18 percent of the sizes of 512 to 13824 with
// blocks of 32 and 8 bits, or of 64, are split otherwise, to no one side's gain (3 and 8 rows, that way and this: 8 bits, blocks of 32,
// 11008 -> 4096 11.5 and 12.2 us, 12.0 and 12.5, 5504 -> 2860 8.9 and 9.2, 7.5 and 8.3; 2 bits, blocks of 64, 5120 -> 12643 11.2 and 11.9,
// 11.2 and 14.3).
constexpr int split_waves(int wb, int block) {
    if (block == 64) return wb == 2 ? 3 : 2;
    return block == 32 && wb == 8 ? 3 : 4;
}

// The split that takes the least of: the items a thread quantizes and the records a wave streams, per round of resident
// workgroups; the waves of the fullest compute unit with the bytes they stream; the exchange between slices and the
// partial sums a thread adds there; all of it on average over three to eight rows.  It does not look at the number of rows
// of the call: the split says in what order a row's sums are added, so a sequence gets the same bits in a batch of three as
// in one of eight.  That costs nothing (130 random shapes of 3 to 8 rows: 0.998 of the time with the split that the rule
// takes for each number alone; 5 rows 5120 -> 5120 9.8 us for 9.45, 8 rows 11008 -> 4096 13.8 either way).
// (4, 2), (2, 4), (1, 8) and (1, 4) are the best of nine forms over 3300 random shapes (3 to 8 rows, K and N 256 to 14000,
// all blocks), 0.6 % above always the best of the nine.  The coefficients (us) are least squares over 2800 shapes, every
// number of slices timed in each form.
// No more than `most` slices: the workspace holds the partial sums of that many.
DecodeSplit choose_split(int chunks, int groups, int block, int wb, int record, int most) {
    static constexpr int counts[] = {1, 2, 3, 4, 5, 6, 8, 10, 12, 16, 20, 24, 32, 48, 64};
    DecodeSplit best = {0, 0, 0, 0};
    float least = 0.f;
    const int resident_waves = 4 * split_waves(wb, block), record_bytes = (int)record_lds(block);
    // Every call comes through here: two divisions per split and the rest in shifts and multiplications, 0.27 to 0.43 us of host
    // time at 80 to 216 chunks by 128 to 432 groups; 0.7 to 1.0 us with a division for each quotient.
    static constexpr unsigned inverse[5] = {0, 65536, 32768, 21846, 16384};      // of 1 to 4, in 2^-16, rounded up
    auto weigh = [&](auto nwc, auto ksc) {
        constexpr int NW = decltype(nwc)::value, KS = decltype(ksc)::value, WAVES = NW * KS;
        const int columns = (groups + NW - 1) / NW, turns = (chunks + KS - 1) / KS;
        const int fixed_lds = (int)slice_lds(block, 0, NW, KS), by_regs = resident_waves / WAVES;
        int before = 0;
        for (int count : counts) {
            const int n = count < most ? count : most;
            const int part = (int)((unsigned)(turns + n - 1) / (unsigned)n);
            if (part != before) {
                before = part;
                const int slice = part * KS < chunks ? part * KS : chunks, slices = (int)((unsigned)(turns + part - 1) / (unsigned)part);
                if (slice > kMaxLds / record_bytes || slice * record_bytes + fixed_lds > kMaxLds) continue;
                const int lds = slice * record_bytes + fixed_lds + 1024;
                const int by_lds = 4 * lds <= 160 * 1024 ? 4 : 3 * lds <= 160 * 1024 ? 3 : 2;      // a workgroup takes no more than 72 KiB
                const int resident = by_lds < by_regs ? by_lds : by_regs;      // workgroups on a compute unit
                const int share = (columns * slices + 255) >> 8;     // of the fullest compute unit
                const int rounds = (int)((unsigned)(share + resident - 1) * inverse[resident] >> 16);       // exact below 2^15
                const unsigned per_row = (unsigned)(slice * block) / 2;
                unsigned items = 0;
                for (unsigned rows = 3; rows <= 8; ++rows) items += (rows * per_row + WAVES * 64 - 1) / (WAVES * 64);
                const float t = (float)rounds * ((0.45f / 6.f) * (float)(int)items + 0.07f * (float)part) +
                                (float)share * (0.25f * WAVES) * (0.315f + 4e-5f * (float)part * (float)record) +
                                (slices > 1 ? 1.55f + (0.088f * 5.5f / (2 * KS)) * (float)slices : 0.f);
                if (best.parts == 0 || t < least) { least = t; best = {NW, KS, slices, part}; }
            }
            if (n == most) break;
        }
    };
    weigh(std::integral_constant<int, 4>{}, std::integral_constant<int, 2>{});
    weigh(std::integral_constant<int, 2>{}, std::integral_constant<int, 4>{});
    weigh(std::integral_constant<int, 1>{}, std::integral_constant<int, 8>{});
    weigh(std::integral_constant<int, 1>{}, std::integral_constant<int, 4>{});
    return best;
}

template <int WB, int B, int NW, int KS>
mx_status launch_form(const DecodeArgs& a, hipStream_t st) {
    const size_t smem = (size_t)slice_lds(B, a.slice, NW, KS);
    auto kern = linear_splitk_kernel<WB, B, NW, KS>;
    static std::atomic<uint64_t> done{0};
    if (smem > kMaxLds) return MX_ERR_UNSUPPORTED;            // choose_split stays below it
    if (smem > 64 * 1024 && !allow_dynamic_lds(reinterpret_cast<const void*>(kern), kMaxLds, done)) return MX_ERR_DEVICE;
    hipLaunchKernelGGL(kern, dim3((unsigned)((int64_t)a.columns * a.ksplit)), dim3(NW * KS * 64), smem, st, a);
    MX_HIP_LAUNCH_CHECK();
    return MX_OK;
}

template <int WB, int B>
mx_status launch_decode(const DecodeArgs& a, const DecodeSplit& s, hipStream_t st) {
    if (s.groups == 4) return launch_form<WB, B, 4, 2>(a, st);
    if (s.groups == 2) return launch_form<WB, B, 2, 4>(a, st);
    if (s.parts == 4) return launch_form<WB, B, 1, 4>(a, st);
    return launch_form<WB, B, 1, 8>(a, st);
}

template <int B>
mx_status dispatch_wb(const DecodeArgs& a, int wb, const DecodeSplit& s, hipStream_t st) {
    switch (wb) {
        case 2: return launch_decode<2, B>(a, s, st);
        case 3: return launch_decode<3, B>(a, s, st);
        case 4: return launch_decode<4, B>(a, s, st);
        case 5: return launch_decode<5, B>(a, s, st);
        case 6: return launch_decode<6, B>(a, s, st);
        case 7: return launch_decode<7, B>(a, s, st);
        case 8: return launch_decode<8, B>(a, s, st);
    }
    return MX_ERR_BAD_ARG;
}

}  // namespace

// How mx_linear splits the weights of an M x K by N x K product over workgroups.  `ok` is false when the
// one-launch kernel does not take the shape (the caller then quantizes and multiplies in two launches).
DecodePlan decode_plan(int64_t M, int64_t K, int64_t N, int block, int wb) {
    DecodePlan p;
    p.ok = false; p.ksplit = 1; p.partial_floats = 0;
    const FragGeom gb = frag_geom(N, K, block, wb);
    if (M < 1 || M > 8 || K <= 0 || gb.groups > kDecodeMaxGroups || gb.chunks > (1 << 20)) return p;
    if ((gb.chunks + 1024) * (int64_t)gb.record >= (1LL << 31)) return p;       // 32-bit ring offsets
    // the most K slices a call uses, which its workspace is sized for
    int64_t ksplit = (kTargetPairs + gb.groups / 2) / gb.groups;
    ksplit = ksplit < 1 ? 1 : ksplit;
    int64_t slice = ceil_div(gb.chunks, ksplit);
    slice = slice < kMinSlice ? kMinSlice : slice;
    slice = slice > (56 * 1024) / record_lds(block) ? (56 * 1024) / record_lds(block) : slice;
    slice = slice > gb.chunks ? gb.chunks : slice;
    ksplit = ceil_div(gb.chunks, slice);                                         // every slice holds a record
    if (ksplit > kDecodeMaxSplit) return p;
    p.ok = true; p.ksplit = (int32_t)ksplit;
    p.partial_floats = ksplit > 1 ? ksplit * M * gb.groups * 32 : 0;
    return p;
}

mx_status linear_decode(const float* x, int64_t M, int64_t K, int64_t row_stride, mx_format fx, void* workspace,
                        const void* B_packed, int64_t N, mx_format fb, float* Y, int64_t ldy, hipStream_t st) {
    const DecodePlan p = decode_plan(M, K, N, fb.block, fb.mant_bits);
    if (!p.ok) return MX_ERR_UNSUPPORTED;
    const FragGeom gb = frag_geom(N, K, fb.block, fb.mant_bits);
    DecodeArgs a;
    a.x = x; a.x_stride = row_stride; a.B = (const uint8_t*)B_packed; a.Y = Y; a.ldy = ldy;
    a.counters = reinterpret_cast<uint32_t*>(workspace);
    a.partial = reinterpret_cast<float*>((uint8_t*)workspace + kDecodeCounterBytes);
    a.M = (int32_t)M; a.N = (int32_t)N; a.K = (int32_t)K;
    a.groups = (int32_t)gb.groups;
    const DecodeSplit s = choose_split((int)gb.chunks, a.groups, fb.block, fb.mant_bits, gb.record, p.ksplit);
    if (s.parts == 0) return MX_ERR_UNSUPPORTED;              // not reached: `most` slices of the smallest form fit the LDS
    a.columns = (a.groups + s.groups - 1) / s.groups;
    a.chunks = (int32_t)gb.chunks; a.part = s.part; a.ksplit = s.slices;
    a.slice = s.part * s.parts < a.chunks ? s.part * s.parts : a.chunks;
    a.recordB = gb.record;
    a.wa = fx.mant_bits;
    a.bias = (1 << (fx.exp_bits - 1)) - 1;
    a.emax = ((1 << fx.exp_bits) - 1) - a.bias;
    a.rounding = fx.rounding;
    a.eadj = -a.bias - (fx.mant_bits - 2) - (fb.mant_bits - 2);
    switch (fb.block) {
        case 16: return dispatch_wb<16>(a, fb.mant_bits, s, st);
        case 32: return dispatch_wb<32>(a, fb.mant_bits, s, st);
        case 64: return dispatch_wb<64>(a, fb.mant_bits, s, st);
    }
    return MX_ERR_UNSUPPORTED;
}

}  // namespace mx
