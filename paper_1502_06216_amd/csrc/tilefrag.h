// MFMA fragments of the fused 2D tile arithmetic, shared by the tile kernels
// (gibbs2d.hip) and the one-block kernel (small2d.hip): the same products in
// the same order, hence the same bits.
#pragma once

#include "epilogue.h"

namespace jko {

// One 16 x 16 fragment of Z = X K1_1^T: xr is this lane's halo row (lane & 15)
// and kr / khr, klr this lane's factor row (FP32, or bfloat16 hi and lo), each
// offset by the lane's first k: 4 (lane >> 4) in FP32, 8 (lane >> 4) split.
// L: k extent, a multiple of 16 (FP32) or 32 (split).
template <bool SPLIT>
__device__ __forceinline__ f4 z_frag(const float* xr, const float* kr, const uint16_t* khr, const uint16_t* klr,
                                     int L) {
    if constexpr (SPLIT) {
        f4 acc = f4{0.f, 0.f, 0.f, 0.f};
        for (int c0 = 0; c0 < L; c0 += 32) {
            bf8 ah, al;
            split_bf16(*reinterpret_cast<const f4*>(xr + c0), *reinterpret_cast<const f4*>(xr + c0 + 4), ah, al);
            const bf8 bh = __builtin_bit_cast(bf8, *reinterpret_cast<const u16x8*>(khr + c0));
            const bf8 bl = __builtin_bit_cast(bf8, *reinterpret_cast<const u16x8*>(klr + c0));
            acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(al, bh, acc, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah, bl, acc, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah, bh, acc, 0, 0, 0);
        }
        return acc;
    } else {
        // even and odd k-chunks go to two accumulators (independent MFMA chains)
        f4 acc0 = f4{0.f, 0.f, 0.f, 0.f}, acc1 = f4{0.f, 0.f, 0.f, 0.f};
        int c0 = 0;
        for (; c0 + 16 < L; c0 += 32) {
            const f4 a0 = *reinterpret_cast<const f4*>(xr + c0);
            const f4 b0 = *reinterpret_cast<const f4*>(kr + c0);
            const f4 a1 = *reinterpret_cast<const f4*>(xr + c0 + 16);
            const f4 b1 = *reinterpret_cast<const f4*>(kr + c0 + 16);
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                acc0 = __builtin_amdgcn_mfma_f32_16x16x4f32(a0[s], b0[s], acc0, 0, 0, 0);
                acc1 = __builtin_amdgcn_mfma_f32_16x16x4f32(a1[s], b1[s], acc1, 0, 0, 0);
            }
        }
        if (c0 < L) {
            const f4 a0 = *reinterpret_cast<const f4*>(xr + c0);
            const f4 b0 = *reinterpret_cast<const f4*>(kr + c0);
#pragma unroll
            for (int s = 0; s < 4; ++s) acc0 = __builtin_amdgcn_mfma_f32_16x16x4f32(a0[s], b0[s], acc0, 0, 0, 0);
        }
        return acc0 + acc1;
    }
}

// One of the two accumulators of an FP32 fragment alone: the chunks c0 = first,
// first + 32, ...; z_frag is the sum of the one from 0 and the one from 16.
__device__ __forceinline__ f4 z_half(const float* xr, const float* kr, int first, int L) {
    f4 acc = f4{0.f, 0.f, 0.f, 0.f};
    for (int c0 = first; c0 < L; c0 += 32) {
        const f4 a = *reinterpret_cast<const f4*>(xr + c0);
        const f4 b = *reinterpret_cast<const f4*>(kr + c0);
#pragma unroll
        for (int s = 0; s < 4; ++s) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a[s], b[s], acc, 0, 0, 0);
    }
    return acc;
}

// One k-chunk (16 in FP32, 32 split) of a 16 x 16 fragment of Y^T = Z^T K1_0^T,
// added to acc; the pointers as above, already at the chunk.  Z is zr, or zr +
// z2 (the two accumulators of an FP32 fragment).
template <bool SPLIT>
__device__ __forceinline__ f4 y_chunk(const float* zr, const float* kr, const uint16_t* khr, const uint16_t* klr,
                                      f4 acc, const float* z2 = nullptr) {
    if constexpr (SPLIT) {
        bf8 ah, al;
        split_bf16(*reinterpret_cast<const f4*>(zr), *reinterpret_cast<const f4*>(zr + 4), ah, al);
        const bf8 bh = __builtin_bit_cast(bf8, *reinterpret_cast<const u16x8*>(khr));
        const bf8 bl = __builtin_bit_cast(bf8, *reinterpret_cast<const u16x8*>(klr));
        acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(al, bh, acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah, bl, acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah, bh, acc, 0, 0, 0);
    } else {
        f4 a = *reinterpret_cast<const f4*>(zr);
        if (z2) a += *reinterpret_cast<const f4*>(z2);
        const f4 b = *reinterpret_cast<const f4*>(kr);
#pragma unroll
        for (int s = 0; s < 4; ++s) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a[s], b[s], acc, 0, 0, 0);
    }
    return acc;
}

}  // namespace jko
