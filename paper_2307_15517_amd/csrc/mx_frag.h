// Device helpers shared by the kernels that read MX_LAYOUT_FRAGMENT operands: lane pieces, their
// unpacking to int8, and the exact per-block integer product on the matrix cores (Section 3.2 of the
// paper: mantissa products are summed as integers inside a block, the shared exponents come after).
#pragma once

#include "mx_common.h"

namespace mx {

typedef int v4i_t __attribute__((ext_vector_type(4)));
typedef int v16i_t __attribute__((ext_vector_type(16)));

// dwords of one lane piece: four half blocks of B/2 elements, W bits each
template <int W, int B> struct Piece { static constexpr int kDw = B * W / 16; };

template <int NDW>
__device__ __forceinline__ void load_dwords(const uint8_t* p, uint32_t* out) {
    if constexpr (NDW % 4 == 0) {
#pragma unroll
        for (int d = 0; d < NDW / 4; ++d) {
            uint4 v = reinterpret_cast<const uint4*>(p)[d];
            out[4 * d] = v.x; out[4 * d + 1] = v.y; out[4 * d + 2] = v.z; out[4 * d + 3] = v.w;
        }
    } else if constexpr (NDW % 2 == 0) {
#pragma unroll
        for (int d = 0; d < NDW / 2; ++d) {
            uint2 v = reinterpret_cast<const uint2*>(p)[d];
            out[2 * d] = v.x; out[2 * d + 1] = v.y;
        }
    } else {
#pragma unroll
        for (int d = 0; d < NDW; ++d) out[d] = reinterpret_cast<const uint32_t*>(p)[d];
    }
}

// Half-block j of a lane piece -> B/2 int8 in B/8 dwords, in element order.  Every code lands in the top W bits of its
// byte, i.e. the bytes come out multiplied by 2^(8-W) (kScaleLog2), which the exponent offset takes back: no sign
// extension, only shifts and masks.
//   W = 4: the nibbles of every group of 8 elements are stored e0 e4 e1 e5 e2 e6 e3 e7: two masks.
//   other W < 8: four codes (4W <= 28 bits) are brought to bit 0, the upper two moved to bit 16, and then both halves
//   are spread the same way: seven instructions for four elements.  One code at a time with sign extension took ten;
//   five rows decoding against 5-bit weights in blocks of 32 (4096 -> 11008) took 15.8 us that way, 14.2 us this way,
//   2048 x 4096 x 4096 with 6 by 5 bits 269 against 212 us (block 32).
template <int W, int B> struct Unpack {
    static constexpr int kScaleLog2 = 8 - W;
    __device__ __forceinline__ static void run(const uint32_t* piece, int j, uint32_t* out) {
        constexpr int kOut = B / 8;
        if constexpr (W == 8) {
#pragma unroll
            for (int d = 0; d < kOut; ++d) out[d] = piece[j * kOut + d];
        } else if constexpr (W == 4) {
#pragma unroll
            for (int d = 0; d < kOut / 2; ++d) {
                const uint32_t x = piece[j * (kOut / 2) + d];
                out[2 * d] = (x << 4) & 0xF0F0F0F0u;
                out[2 * d + 1] = x & 0xF0F0F0F0u;
            }
        } else {
            constexpr uint32_t kTop = ((0xFFu << (8 - W)) & 0xFFu) * 0x01010101u;
#pragma unroll
            for (int d = 0; d < kOut; ++d) {
                const int bit = (j * (B / 2) + d * 4) * W, dw = bit >> 5, sh = bit & 31;
                uint32_t x = piece[dw] >> sh;
                if (sh + 4 * W > 32) x = __builtin_amdgcn_alignbit(piece[dw + 1], piece[dw], sh);
                const uint32_t y = (x & 0xFFFFu) | ((x << (16 - 2 * W)) & 0xFFFF0000u);       // codes at bits 0, W, 16, 16 + W
                out[d] = (((y << (16 - 2 * W)) & 0xFF00FF00u) | ((y << (8 - W)) & 0x00FF00FFu)) & kTop;
            }
        }
    }
};

// Exact int32 dot products of one block, added to z: D (32x32) = A half-blocks x B half-blocks + z.
template <int B>
__device__ __forceinline__ v16i_t block_mfma(const uint32_t* a, const uint32_t* b, v16i_t z) {
    if constexpr (B == 16) {
        const long la = (long)(((uint64_t)a[1] << 32) | a[0]);
        const long lb = (long)(((uint64_t)b[1] << 32) | b[0]);
        return __builtin_amdgcn_mfma_i32_32x32x16_i8(la, lb, z, 0, 0, 0);
    } else {
#pragma unroll
        for (int s = 0; s < B / 32; ++s) {
            v4i_t va = {(int)a[4 * s], (int)a[4 * s + 1], (int)a[4 * s + 2], (int)a[4 * s + 3]};
            v4i_t vb = {(int)b[4 * s], (int)b[4 * s + 1], (int)b[4 * s + 2], (int)b[4 * s + 3]};
            z = __builtin_amdgcn_mfma_i32_32x32x32_i8(va, vb, z, 0, 0, 0);
        }
        return z;
    }
}
template <int B>
__device__ __forceinline__ v16i_t block_mfma(const uint32_t* a, const uint32_t* b) {
    return block_mfma<B>(a, b, v16i_t{0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0});
}

// The same for up to eight rows in a 16 x 16 result of which every element is used: half the matrix cycles and a quarter
// of the result registers of the 32 x 32 form.  Lane 32h + 16c + i of a record carries half h of column 16c + i; the
// instruction takes it as K range 2h + c of its column i.  Its rows 0..7 are the activations in the lanes with c = 0 and
// zeros in the others, rows 8..15 the reverse, so element (8c + r, i) is row r against column 16c + i.
template <int B>
__device__ __forceinline__ v4i_t block_mfma16(const uint32_t* a, const uint32_t* b, v4i_t z) {
    if constexpr (B == 16) {
        const long la = (long)(((uint64_t)a[1] << 32) | a[0]);
        const long lb = (long)(((uint64_t)b[1] << 32) | b[0]);
        return __builtin_amdgcn_mfma_i32_16x16x32_i8(la, lb, z, 0, 0, 0);
    } else {
#pragma unroll
        for (int s = 0; s < B / 32; ++s) {
            v4i_t va = {(int)a[4 * s], (int)a[4 * s + 1], (int)a[4 * s + 2], (int)a[4 * s + 3]};
            v4i_t vb = {(int)b[4 * s], (int)b[4 * s + 1], (int)b[4 * s + 2], (int)b[4 * s + 3]};
            z = __builtin_amdgcn_mfma_i32_16x16x64_i8(va, vb, z, 0, 0, 0);
        }
        return z;
    }
}

// Block dots as fp32 without a conversion.  The integer accumulator starts at the bit pattern of 1.5 * 2^23, so the sum d
// comes out as the bit pattern of the float 1.5 * 2^23 + d (|d| <= 2^20 < 2^22).  With s = 2^k, (1.5 * 2^23 + d) * s -
// 1.5 * 2^23 * s is d * s in one fused multiply-add, exact since d * s fits the 24 bits of a float; both s and
// -1.5 * 2^23 * s are bit patterns that integer adds build.
constexpr uint32_t kDotBias = 0x4B400000u;
constexpr uint32_t kDotBack = 0x80000000u + (23u << 23) + 0x00400000u;     // bits of -1.5 * 2^23 * s = bits of s + this
__device__ __forceinline__ v16i_t dot_bias() {
    v16i_t z;
#pragma unroll
    for (int r = 0; r < 16; ++r) z[r] = (int)kDotBias;
    return z;
}

}  // namespace mx
