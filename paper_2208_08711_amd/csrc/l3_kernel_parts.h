/*
 * Parts shared by the decoder and the encoder kernels of the L3 library, written on the
 * primitives of l3_gfx950.h: the custom Paeth predictor (arxiv 2208.08711 Section 4.2) on
 * packed pairs of 16-bit fields, and the order in which workgroups take work.
 * Device code only; every translation unit gets its own copy.
 */
#ifndef L3_KERNEL_PARTS_H
#define L3_KERNEL_PARTS_H

#include "l3_gfx950.h"

namespace {

/* Section 4.2, custom Paeth filter, on NP registers of two pixels at once.  Value-wise the
 * nearest of TL, TR, T to TL + TR - T is: with lo = min(TL,TR), hi = max(TL,TR), dl = T - lo,
 * dh = hi - T: lo if dl >= 2 dh, else hi if dh >= 2 dl, else T.  The stated tie order
 * (TL, TR, T) only ever chooses between equal values, except T against a neighbour, where
 * the neighbour wins: that is the ">=".
 * The decoder and the encoder are bound by the number of their vector instructions; this takes 9
 * a register (11 with integer masks: a multiply-add and a shift for each, three selects).
 * A field holds the pixel as a 16-bit float from 1024 to 1279: bits 0x6400 | pixel, so that nothing
 * is converted.  All values are whole numbers of at most 11 bits, which 16-bit floats hold
 * exactly.  n_lo = (2 dh > dl) and n_hi = (2 dl > dh) are one multiply-add each, clamped to
 * 0..1, and the prediction is lo + dh + n_lo * dl - n_hi * dh: T where both hold, hi where
 * n_hi does not (then n_lo holds or dl is 0), lo where n_lo does not (then n_hi holds or dh is
 * 0).  In the first and last column of a patch, where the prediction is T, a third operand of the
 * minimum and of the maximum makes lo = 0 and hi = 1919: then dl = T is 1024..1279, dh = 1919 - T
 * is 640..895, both n hold and the sum is T, whatever the outer neighbours hold (0, or another
 * patch's pixel).  The registers are worked on in lockstep so that dependent instructions are
 * not adjacent.
 * Measured together with the shorter record walk of the decoder's open_row (the decoder's write-out as
 * it was), before and after on one card: 32 images of 2048x1024 81.3 -> 77.9 us a call, 8 of 3840x2160
 * planar 78.9 -> 75.0, 32 of 1920x1080 planar 84.2 -> 79.3, 256 photographs 59.3 -> 56.9.  Calls that
 * leave the SIMDs with one wave or less wait for the longer chain instead: 4 of 2048x1024 35.7 -> 36.5, one of
 * 1920x1080 20.2 -> 20.4, 16 fused windows of 768x768 54.2 -> 54.2.  Written as inline assembly those
 * lost more: behind that the compiler puts wait states. */
constexpr uint32_t kPixelBias = 0x64006400u;          /* 1024 in both fields: a pixel of value 0 */
constexpr uint32_t kPredictLow = 0x0000u;             /* 0, border fields' third operand of the minimum */
constexpr uint32_t kPredictHigh = 0x677Fu;            /* 1919, of the maximum */
constexpr uint32_t kPredictNoLimitLow = 0x67FFu;      /* 2047 and 0: all other fields */
constexpr uint32_t kPredictNoLimitHigh = 0x0000u;
/* The third operands for a register that holds pixels x and x + 2 of a patch of pw columns. */
__device__ __forceinline__ void predict_limits(uint32_t x, uint32_t pw, uint32_t& least, uint32_t& most) {
    const bool edge_lo = x == 0 || x + 1 == pw, edge_hi = x + 3 == pw;
    least = (edge_lo ? kPredictLow : kPredictNoLimitLow) | ((edge_hi ? kPredictLow : kPredictNoLimitLow) << 16);
    most = (edge_lo ? kPredictHigh : kPredictNoLimitHigh) | ((edge_hi ? kPredictHigh : kPredictNoLimitHigh) << 16);
}
template <int NP>
__device__ __forceinline__ void predict_pairs_biased(const uint32_t (&TL)[NP], const uint32_t (&TR)[NP],
                                                     const uint32_t (&T)[NP], const uint32_t (&least)[NP],
                                                     const uint32_t (&most)[NP], uint32_t (&pred)[NP]) {
    uint32_t lo[NP], hi[NP], dl[NP], dh[NP], n_lo[NP], n_hi[NP];
#pragma unroll
    for (int j = 0; j < NP; ++j) lo[j] = pk_min3_f16(TL[j], TR[j], least[j]);
#pragma unroll
    for (int j = 0; j < NP; ++j) hi[j] = pk_max3_f16(TL[j], TR[j], most[j]);
#pragma unroll
    for (int j = 0; j < NP; ++j) dl[j] = pk_sub_f16(T[j], lo[j]);
#pragma unroll
    for (int j = 0; j < NP; ++j) dh[j] = pk_sub_f16(hi[j], T[j]);
#pragma unroll
    for (int j = 0; j < NP; ++j) n_lo[j] = pk_twice_exceeds_f16(dh[j], dl[j]);
#pragma unroll
    for (int j = 0; j < NP; ++j) n_hi[j] = pk_twice_exceeds_f16(dl[j], dh[j]);
#pragma unroll
    for (int j = 0; j < NP; ++j) pred[j] = pk_add_f16(lo[j], dh[j]);
#pragma unroll
    for (int j = 0; j < NP; ++j) pred[j] = pk_fma_f16(n_lo[j], dl[j], pred[j]);
#pragma unroll
    for (int j = 0; j < NP; ++j) pred[j] = pk_fnma_f16(n_hi[j], dh[j], pred[j]);
}

/* Which (image, unit) a workgroup takes.  The grid is one-dimensional, a multiple of 8
 * long, and the hardware hands consecutive workgroups to the 8 XCDs in turn (workgroup L
 * runs on XCD L mod 8).  Work item number (L mod 8) * grid/8 + L / 8 therefore gives every
 * XCD one contiguous eighth of the (image, unit) sequence: neighbouring strips, whose
 * streams and output rows share cache lines, meet in the same L2. */
__device__ __forceinline__ bool take_work(uint32_t units_per_image, uint32_t images, uint32_t& image,
                                          uint32_t& unit) {
    const uint32_t eighth = gridDim.x >> 3;
    const uint32_t item = (blockIdx.x & 7u) * eighth + (blockIdx.x >> 3);
    image = item / units_per_image;
    unit = item - image * units_per_image;
    return image < images;
}

}  // namespace

#endif
