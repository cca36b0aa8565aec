/*
 * gfx950 encoder of the L3 format: interleaved 8-bit RGB in device memory ->
 * L3 files in device memory, byte for byte what l3_encode_cpu produces.
 *
 * arxiv 2208.08711, Section 4.2, encoding direction: per patch and channel, the
 * custom Paeth filter (rows after the first: pixel minus the nearest of the three
 * upper neighbours to TL + TR - T, taken from the ORIGINAL row above, so every
 * pixel of the patch is independent), then row-wise base-delta (row minimum as
 * base, minimal width, deltas packed).  Section 4.3: patches concatenated, their
 * offsets recorded in three arrays behind a 13-byte header.
 *
 * Patch sizes 32, 64 and 128 (the ones the paper's rule picks) take two or three kernels (few strips: one):
 *   strip    a workgroup of three waves (one per channel) owns a strip of adjacent
 *            patches, 4 pixels per lane as two packed pairs of 16-bit fields: per
 *            four rows it filters, reduces their min and max over the patch's lanes, packs
 *            the deltas with LDS atomic OR into a small ring per patch and streams the
 *            finished 16-byte granules to a fixed-size slot of a workspace; the
 *            patch's byte size goes to a table;
 *   layout   one workgroup per image: exclusive prefix sum of the patch sizes ->
 *            header, offset arrays, file length (this is where a scan belongs: the
 *            addends are all known); only in calls with very many patches or with an image on
 *            the plain route, otherwise the next kernel does this too;
 *   compact  copies every slot to its place in the file.
 * Calls of few strips take one kernel instead, which shares a strip's rows among waves (the chained
 * route, if all files have room for the longest stream).
 * Any other patch size up to 128 takes the plain route: measure (one wave per patch
 * and channel walks the rows for the sizes), layout, pack (walks them again and
 * writes the bits).  The forward filter needs no row recurrence: the row above is
 * the original one, kept in registers, with lane shifts for the neighbours.
 */
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdlib>
#include <cstring>
#include <new>
#include <type_traits>

#include "l3_ctx.h"
#include "l3_gfx950.h"
#include "l3_kernel_parts.h"

namespace {

constexpr int kMaxPatch = 128;                       /* two pixels per lane */

struct L3EncodeDesc {
    const uint8_t* rgb;
    uint8_t* file;
    uint64_t row_stride;
    uint64_t file_cap;
    uint32_t width, height;
    uint32_t tiles_x, tiles_y;
    uint32_t patch;
    uint32_t sizes_base;     /* first entry of this image in the sizes scratch */
    uint32_t status_index;
    uint32_t strips_x;       /* strip route: wave strips per patch row */
    uint64_t slots_base;     /* strip route: byte offset of this image's first slot in the workspace */
};

__device__ __forceinline__ int nearest_upper(int tl, int t, int tr) {
    /* distances to TL + TR - T: |TR - T| for TL, |TL - T| for TR, |TL + TR - 2T| for T;
     * ties: TL, then TR, then T */
    const int d_tl = abs(tr - t), d_tr = abs(tl - t), d_t = abs(tl + tr - 2 * t);
    if (d_tl <= d_tr && d_tl <= d_t) return tl;
    return d_tr <= d_t ? tr : t;
}

__device__ __forceinline__ int wave_min(int v) {
#pragma unroll
    for (int s = 32; s >= 1; s >>= 1) v = min(v, __shfl_xor(v, s));
    return v;
}
__device__ __forceinline__ int wave_max(int v) {
#pragma unroll
    for (int s = 32; s >= 1; s >>= 1) v = max(v, __shfl_xor(v, s));
    return v;
}

/* Walks the rows of patch (c, ty, tx).  PACK = false: returns the patch's size in
 * bits.  PACK = true: also ORs every field into `bits` (LDS, zeroed by the caller). */
template <bool PACK>
__device__ uint32_t walk_patch(const L3EncodeDesc& d, uint32_t c, uint32_t tx, uint32_t ty,
                               uint32_t* bits) {
    const uint32_t lane = threadIdx.x;
    const uint32_t n = d.patch;
    const uint32_t x0 = tx * n, y0 = ty * n;
    const uint32_t pw = min(n, d.width - x0), ph = min(n, d.height - y0);
    const bool has0 = lane < pw, has1 = lane + 64 < pw;          /* pixels lane and lane + 64 */
    const uint8_t* src = d.rgb + (size_t)y0 * d.row_stride + (size_t)x0 * 3 + c;

    int up0 = 0, up1 = 0;           /* the original row above */
    uint32_t pos = 0;               /* bit position of the current row's record */
    int next0 = has0 ? src[3 * (size_t)lane] : 0;             /* the row after, already travelling */
    int next1 = has1 ? src[3 * (size_t)(lane + 64)] : 0;
    for (uint32_t r = 0; r < ph; ++r) {
        const int cur0 = next0, cur1 = next1;
        if (r + 1 < ph) {
            const uint8_t* row = src + (size_t)(r + 1) * d.row_stride;
            next0 = has0 ? row[3 * (size_t)lane] : 0;
            next1 = has1 ? row[3 * (size_t)(lane + 64)] : 0;
        }
        int v0, v1;
        if (r == 0) {
            v0 = cur0;              /* first row raw, taken as unsigned */
            v1 = cur1;
        } else {
            /* neighbours of pixel `lane`: lanes -1/+1; of pixel `lane + 64`: the same
             * lanes' second pixels, with lanes 63 and 0 joining the halves */
            const int l0 = __shfl_up(up0, 1), r0 = __shfl_down(up0, 1);
            const int l1 = __shfl_up(up1, 1), r1 = __shfl_down(up1, 1);
            const int first1 = __shfl(up1, 0), last0 = __shfl(up0, 63);
            const int tl0 = l0, tr0 = lane == 63 ? first1 : r0;
            const int tl1 = lane == 0 ? last0 : l1, tr1 = r1;
            const bool edge0 = lane == 0 || lane + 1 == pw;
            const bool edge1 = lane + 64 + 1 == pw;
            const int p0 = edge0 ? up0 : nearest_upper(tl0, up0, tr0);
            const int p1 = edge1 ? up1 : nearest_upper(tl1, up1, tr1);
            v0 = (int)(int8_t)(uint8_t)(cur0 - p0);   /* later rows taken as signed bytes */
            v1 = (int)(int8_t)(uint8_t)(cur1 - p1);
        }
        int lo = 1 << 20, hi = -(1 << 20);
        if (has0) { lo = v0; hi = v0; }
        if (has1) { lo = min(lo, v1); hi = max(hi, v1); }
        lo = wave_min(lo);
        hi = wave_max(hi);
        const uint32_t range = (uint32_t)(hi - lo);
        const uint32_t width = range ? 32u - (uint32_t)__builtin_clz(range) : 0u;
        if (PACK) {
            if (lane == 0) {
                const uint32_t rec = width | (((uint32_t)lo & 0xFFu) << 4);
                const uint32_t sh = pos & 31u;
                atomicOr(&bits[pos >> 5], rec << sh);
                if (sh > 20) atomicOr(&bits[(pos >> 5) + 1], rec >> (32u - sh));
            }
            if (width) {
                if (has0) {
                    const uint32_t b = pos + 12 + lane * width, sh = b & 31u;
                    const uint32_t dlt = (uint32_t)(v0 - lo);
                    atomicOr(&bits[b >> 5], dlt << sh);
                    if (sh + width > 32) atomicOr(&bits[(b >> 5) + 1], dlt >> (32u - sh));
                }
                if (has1) {
                    const uint32_t b = pos + 12 + (lane + 64) * width, sh = b & 31u;
                    const uint32_t dlt = (uint32_t)(v1 - lo);
                    atomicOr(&bits[b >> 5], dlt << sh);
                    if (sh + width > 32) atomicOr(&bits[(b >> 5) + 1], dlt >> (32u - sh));
                }
            }
        }
        pos += 12 + pw * width;
        up0 = cur0;
        up1 = cur1;
    }
    return pos;
}


/* ---- the strip route: N in {32, 64, 128} ------------------------------------ */

template <int N>
struct StripGeom {
    static constexpr int LPT = N / 4;              /* lanes per patch, 4 pixels each */
    static constexpr int TPW = 64 / LPT;           /* patches per wave */
    static constexpr int P = 4;                    /* rows of a period: filtered, reduced and packed together */
    static constexpr int RING = 8 * N;             /* ring bytes per patch and channel */
    static constexpr int RING_WORDS = RING / 4 + 4; /* + a word that stands for word 0 of the next lap (and padding to 16 bytes) */
    /* the longest patch stream, rounded up to whole 16-byte granules */
    static constexpr uint32_t SLOT = ((uint32_t)N * (12 + 8 * N) / 8 + 1 + 15) / 16 * 16;
    /* A flush round takes one granule per lane of the patch, 4N bytes; P rows add at most
     * 4N + 6, so the stream's unflushed part may grow by 6 bytes a period over the patch's
     * N / 4 periods, beside a partial granule.  The ring holds that and the period being
     * packed; FINAL_ROUNDS rounds empty it behind the last row. */
    static constexpr int PERIOD_MAX = P * (12 + 8 * N) / 8;
    static constexpr int BACKLOG = 15 + (N / P) * (PERIOD_MAX - LPT * 16);
    static constexpr int FINAL_ROUNDS = (BACKLOG + PERIOD_MAX + 15 + LPT * 16 - 1) / (LPT * 16);
    static_assert(RING >= BACKLOG + PERIOD_MAX + 1 + 8, "ring holds a period behind the backlog");
    static_assert((RING & (RING - 1)) == 0, "ring size is a power of two");
};

__host__ __device__ constexpr uint32_t strip_slot_bytes(uint32_t n) {
    return n == 32 ? StripGeom<32>::SLOT : n == 64 ? StripGeom<64>::SLOT : StripGeom<128>::SLOT;
}

/* max((low half of a) - b, 0) in both 16-bit halves: v_pk_sub_u16 with clamp */
__device__ __forceinline__ uint32_t pk_sub_u16_sat_from_low(uint32_t a, uint32_t b) {
    const unsigned short low = (unsigned short)a;
    return __builtin_bit_cast(uint32_t, __builtin_elementwise_sub_sat((u16x2){low, low}, __builtin_bit_cast(u16x2, b)));
}
/* both halves of v shifted left by the halves of `by`, modulo 16 */
__device__ __forceinline__ uint32_t pk_lshl_b16(uint32_t by, uint32_t v) {
    return __builtin_bit_cast(uint32_t, (u16x2)(__builtin_bit_cast(u16x2, v) << (__builtin_bit_cast(u16x2, by) & (u16x2){15, 15})));
}
__device__ __forceinline__ uint32_t pk_min_u16(uint32_t a, uint32_t b) {
    return __builtin_bit_cast(uint32_t, __builtin_elementwise_min(__builtin_bit_cast(u16x2, a),
                                                                  __builtin_bit_cast(u16x2, b)));
}
template <int CTRL>
__device__ __forceinline__ uint32_t dpp_move(uint32_t v) {
    /* every lane has a source lane under these controls, so the "old" value is never used */
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xF, 0xF, true);
}
constexpr int kDppXor1 = 0xB1, kDppXor2 = 0x4E;                  /* quad_perm [1,0,3,2], [2,3,0,1] */
constexpr int kDppHalfMirror = 0x141, kDppMirror = 0x140;        /* inside 8 and 16 lanes */

__device__ __forceinline__ uint32_t pk_max_i16(uint32_t a, uint32_t b) {
    return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(s16x2, a),
                                                                  __builtin_bit_cast(s16x2, b)));
}

/* Row minima of four rows over the LPT lanes of a patch (both 16-bit fields separately), all at
 * once: while lanes are folded onto each other, the two lanes of a pair take different rows, so
 * that after two such steps one register holds all four rows and the remaining steps are paid
 * once instead of four times.  In lane i of the patch the result is that of row
 * reduced_row<LPT>(i); the order of the rows is turned round in every other quad, so that the
 * mirrors inside 8 and 16 lanes bring equal rows together.  22 instructions for four rows with
 * the way back at N = 128 instead of 40 for four separate butterflies. */
template <int LPT>
__device__ __forceinline__ uint32_t reduced_row(uint32_t lane) {
    const uint32_t turned = (lane & 4u) ? 3u : 0u;
    return LPT == 32 ? ((lane >> 4) & 1u) + 2u * ((lane ^ turned) & 1u) : ((lane ^ turned) & 3u);
}
template <int CTRL>
__device__ __forceinline__ uint32_t fold_two_rows(uint32_t a, uint32_t b, bool second) {
    const uint32_t keep = second ? b : a, send = second ? a : b;
    return pk_min_u16(keep, dpp_move<CTRL>(send));
}
template <int LPT>
__device__ __forceinline__ uint32_t patch_min_of_rows(const uint32_t (&v)[4], uint32_t my_row) {
    uint32_t m;
    if constexpr (LPT == 32) {
        /* the swap of neighbouring 16-lane rows between two registers is the first such step */
        const auto p = __builtin_amdgcn_permlane16_swap(v[0], v[1], false, false);
        const auto q = __builtin_amdgcn_permlane16_swap(v[2], v[3], false, false);
        const uint32_t v01 = pk_min_u16((uint32_t)p[0], (uint32_t)p[1]);
        const uint32_t v23 = pk_min_u16((uint32_t)q[0], (uint32_t)q[1]);
        m = fold_two_rows<kDppXor1>(v01, v23, (my_row & 2u) != 0);
        m = pk_min_u16(m, dpp_move<kDppXor2>(m));
    } else {
        const uint32_t v01 = fold_two_rows<kDppXor1>(v[0], v[1], (my_row & 1u) != 0);
        const uint32_t v23 = fold_two_rows<kDppXor1>(v[2], v[3], (my_row & 1u) != 0);
        m = fold_two_rows<kDppXor2>(v01, v23, (my_row & 2u) != 0);
    }
    m = pk_min_u16(m, dpp_move<kDppHalfMirror>(m));
    if (LPT >= 16) m = pk_min_u16(m, dpp_move<kDppMirror>(m));
    return m;
}
/* The way back: value of row i in every lane of the patch. */
template <int LPT>
__device__ __forceinline__ void rows_to_all_lanes(uint32_t v, uint32_t (&row)[4]) {
    /* the turned quads (banks 1 and 3 of a 16-lane row) back in order */
    v = (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, LPT == 32 ? kDppXor1 : 0x1B /* quad_perm [3,2,1,0] */, 0xF, 0xA, false);
    if constexpr (LPT == 32) {
        const auto p = __builtin_amdgcn_permlane16_swap(v, v, false, false);
        row[0] = dpp_move<0x00>((uint32_t)p[0]);      /* quad_perm [0,0,0,0] */
        row[1] = dpp_move<0x00>((uint32_t)p[1]);
        row[2] = dpp_move<0x55>((uint32_t)p[0]);      /* quad_perm [1,1,1,1] */
        row[3] = dpp_move<0x55>((uint32_t)p[1]);
    } else {
        row[0] = dpp_move<0x00>(v);
        row[1] = dpp_move<0x55>(v);
        row[2] = dpp_move<0xAA>(v);
        row[3] = dpp_move<0xFF>(v);
    }
}

/* What a lane knows of its four pixels, columns 4 xl .. 4 xl + 3 of a patch of pw columns from image
 * column x0 on (pw = 0: a lane without a patch). */
struct StripLane {
    uint32_t xpix, nvalid;          /* the first of the columns; how many exist */
    /* registers of two 16-bit fields: E = pixels (0, 2), O = pixels (1, 3) */
    uint32_t validE, validO, keepE, keepO, nowhere;
    uint32_t least[2], most[2];     /* the predictor's limits: see predict_pairs_biased */
    /* The lane's 12 bytes of a row.  A lane at the right edge of the image owns fewer than
     * 4 pixels and must not read past the row: it reads the 12 bytes that END at its last
     * pixel and shifts them down when it takes them (what then sits above the valid bytes is
     * masked later).  Only waves with such a lane shift.  A lane without pixels reads the start
     * of the row, so that no load is conditional.  Images narrower than 4 pixels go byte by
     * byte; there all pixels are lane 0's. */
    bool wide, ragged_wave;
    uint32_t shift, lane_at, row_bytes;

    __device__ __forceinline__ StripLane(uint32_t width, uint32_t x0, uint32_t pw, uint32_t xl) {
        xpix = 4 * xl;
        nvalid = pw > xpix ? min(4u, pw - xpix) : 0u;
        validE = (nvalid > 0 ? 0x0000FFFFu : 0u) | (nvalid > 2 ? 0xFFFF0000u : 0u);
        validO = (nvalid > 1 ? 0x0000FFFFu : 0u) | (nvalid > 3 ? 0xFFFF0000u : 0u);
        predict_limits(xpix, pw, least[0], most[0]);
        predict_limits(xpix + 1, pw, least[1], most[1]);
        keepE = validE & 0x00FF00FFu;
        keepO = validO & 0x00FF00FFu;
        nowhere = ~(validE | validO);       /* fields that neither register has a pixel for */
        wide = width >= 4;
        ragged_wave = wide && __builtin_amdgcn_ballot_w64(nvalid != 0 && nvalid != 4) != 0;
        const uint32_t back = wide && nvalid ? 3 * (4 - nvalid) : 0;              /* bytes to step back: 0, 3, 6, 9 */
        shift = back;
        lane_at = nvalid ? (x0 + xpix) * 3 - back : 0u;            /* below 3 * 2^24 */
        row_bytes = width * 3;
    }

    /* The residual byte r is looked at as t = r ^ K, K = 0 in the first row (raw,
     * unsigned) and 0x80 after it (signed byte + 128), so that the unsigned minimum of t
     * is the row minimum of Section 4.2; what is kept is u = t ^ 0xFF, whose maximum gives
     * the row minimum.  Fields of pixels that do not exist read 0xFFFF: neither the unsigned
     * minimum nor the signed maximum takes them.  These are K ^ 0xFF in the fields. */
    __device__ __forceinline__ void first_row_key(uint32_t& kE, uint32_t& kO) const {
        kE = ~validE | keepE;
        kO = ~validO | keepO;
    }
    __device__ __forceinline__ void later_row_key(uint32_t& kE, uint32_t& kO) const {
        kE = ~validE | (keepE & 0x007F007Fu);
        kO = ~validO | (keepO & 0x007F007Fu);
    }

    __device__ __forceinline__ u32x3 load(const uint8_t* row) const { return wide ? load_wide(row) : load_narrow(row); }
    __device__ __forceinline__ u32x3 load_wide(const uint8_t* row) const {
        uint32_t at = lane_at;
        L3_KEEP_VGPR(at);      /* stays the load's 32-bit offset */
        return load_u32x3(reinterpret_cast<global_const_u8*>((uintptr_t)row) + at);
    }
    __device__ __forceinline__ u32x3 load_narrow(const uint8_t* row) const {
        global_const_u8* base = reinterpret_cast<global_const_u8*>((uintptr_t)row);
        uint32_t b[9];
#pragma unroll
        for (uint32_t k = 0; k < 9; ++k) b[k] = base[min(k, row_bytes - 1)];
        u32x3 v;
        v.x = b[0] | (b[1] << 8) | (b[2] << 16) | (b[3] << 24);
        v.y = b[4] | (b[5] << 8) | (b[6] << 16) | (b[7] << 24);
        v.z = b[8];
        return v;
    }
    __device__ __forceinline__ void shift_down(u32x3& v) const {
        const uint32_t words = shift >> 2, bits = (shift & 3u) * 8;
        const uint32_t a0 = words == 0 ? v.x : (words == 1 ? v.y : v.z);
        const uint32_t a1 = words == 0 ? v.y : (words == 1 ? v.z : 0u);
        const uint32_t a2 = words == 0 ? v.z : 0u;
        v.x = __builtin_amdgcn_alignbit(a1, a0, bits);
        v.y = __builtin_amdgcn_alignbit(a2, a1, bits);
        v.z = a2 >> bits;
    }

    /* Section 4.2 stage 1 on the original row above; leaves u and the lane's own part of the
     * row's extremes: (minimum of u, ~(maximum of u)), so that both go on as minima. */
    __device__ __forceinline__ uint32_t filter(const uint32_t (&above)[2], const uint32_t (&cur)[2], uint32_t kE,
                                               uint32_t kO, uint32_t& uE, uint32_t& uO) const {
        const uint32_t from_left = dpp_from_lower_lane(above[1]);
        const uint32_t from_right = dpp_from_upper_lane(above[0]);
        uint32_t TL[2], TR[2], pred[2];
        TL[0] = __builtin_amdgcn_alignbit(above[1], from_left, 16);
        TR[0] = above[1];
        TL[1] = above[0];
        TR[1] = __builtin_amdgcn_alignbit(from_right, above[0], 16);
        predict_pairs_biased<2>(TL, TR, above, least, most, pred);
        const uint32_t rE = __builtin_bit_cast(uint32_t, (u16x2)(__builtin_bit_cast(u16x2, cur[0]) -
                                                                 __builtin_bit_cast(u16x2, pred[0])));
        const uint32_t rO = __builtin_bit_cast(uint32_t, (u16x2)(__builtin_bit_cast(u16x2, cur[1]) -
                                                                 __builtin_bit_cast(u16x2, pred[1])));
        uE = __builtin_amdgcn_bitop3_b32(rE, keepE, kE, 0x6A);           /* (r & keep) ^ k */
        uO = __builtin_amdgcn_bitop3_b32(rO, keepO, kO, 0x6A);
        const uint32_t a = pk_min_u16(uE, uO);
        const uint32_t b = ~pk_max_i16(uE, uO) | nowhere;
        return pk_min_u16(__builtin_amdgcn_perm(b, a, 0x05040100u),      /* (a.lo, b.lo) */
                          __builtin_amdgcn_perm(b, a, 0x07060302u));     /* (a.hi, b.hi) */
    }
};

/* channel C of pixel i is byte 3 i + C of the lane's 12 bytes; biased as the predictor takes
 * it (the bias goes again with the subtraction of the prediction) */
template <int C>
__device__ __forceinline__ void take_channel(const u32x3 raw, uint32_t pixel_bias, uint32_t (&cur)[2]) {
    if (C == 0) {
        cur[0] = __builtin_amdgcn_perm(raw.y, raw.x, 0x0C060C00u);   /* bytes 0, 6 */
        cur[1] = __builtin_amdgcn_perm(raw.z, raw.x, 0x0C050C03u);   /* bytes 3, 9 */
    } else if (C == 1) {
        cur[0] = __builtin_amdgcn_perm(raw.y, raw.x, 0x0C070C01u);   /* bytes 1, 7 */
        cur[1] = __builtin_amdgcn_perm(raw.z, raw.y, 0x0C060C00u);   /* bytes 4, 10 */
    } else {
        cur[0] = __builtin_amdgcn_perm(raw.z, raw.x, 0x0C040C02u);   /* bytes 2, 8 */
        cur[1] = __builtin_amdgcn_perm(raw.z, raw.y, 0x0C070C01u);   /* bytes 5, 11 */
    }
    cur[0] |= pixel_bias;
    cur[1] |= pixel_bias;
}

/* Steps 1-2 of stage 2 for four rows at once, from the lanes' parts of their extremes: in every
 * lane, for row my_row, its least t, its largest u and its width.  (Each in a register of its own, not the last
 * two packed here: the strip kernel then gets the shorter code, 2 images of 3001x2000 55.5 us, packed here 56.1; 24 of 640x480
 * at N = 64 38.6 and 39.6.) */
struct RowExtremes {
    uint32_t tmin, umax, width;
    __device__ __forceinline__ uint32_t packed() const { return umax | (width << 16); }
    /* the row's record: 4-bit width, 8-bit base; K as above */
    __device__ __forceinline__ uint32_t record(uint32_t K) const { return width | ((tmin ^ K) << 4); }
};
template <int LPT>
__device__ __forceinline__ RowExtremes extremes_of_my_row(const uint32_t (&lane_part)[4], uint32_t my_row) {
    const uint32_t m = patch_min_of_rows<LPT>(lane_part, my_row);
    RowExtremes e;
    const uint32_t umin = m & 0xFFFFu;
    e.tmin = (m >> 16) & 0xFFu;
    e.umax = e.tmin ^ 0xFFu;
    const uint32_t range = (e.umax - umin) & 0xFFu;      /* masked: lanes without a patch hold no minimum */
    e.width = 31u - (uint32_t)__builtin_clz(2u * range + 1u);
    return e;
}

/* Steps 3-4 of stage 2 for one row, given its largest u in the low half and its width in
 * the high half: deltas t - tmin = umax - u, 0 where no pixel exists; the lane's four deltas
 * as one field of 4 w bits.  (d0 | d1 << w, d2 | d3 << w) first, then the lower field moves up to the
 * upper one (not the upper one down: that takes three instructions more; 32 images of 2048x1024
 * 172.4 -> 171.6 us with this): the four deltas are then the bits from 16 - 2 w on, below them zeros, and
 * go to the stream by as much sooner, at bit (xpix + 2) w - 4 behind the start of the row's record, which may be up
 * to 4 bits ahead of it.  w = 0 shifts a field of zeros. */
__device__ __forceinline__ uint32_t delta_field(uint32_t extremes, uint32_t uE, uint32_t uO) {
    const uint32_t w = extremes >> 16;
    const uint32_t dE = pk_sub_u16_sat_from_low(extremes, uE), dO = pk_sub_u16_sat_from_low(extremes, uO);
    const uint32_t pair = dE | (dO << w);
    const uint32_t up_by = (uint32_t)(16 - 2 * (int)w);     /* and nothing in the upper half */
    return pk_lshl_b16(up_by, pair);
}

/* One strip: TPW adjacent patches of one patch row, channel C. */
template <int N, int C>
__device__ __forceinline__ void encode_strip(const L3EncodeDesc& d, uint32_t* __restrict__ sizes,
                                             uint8_t* __restrict__ slots, uint32_t* ring_words) {
    using G = StripGeom<N>;
    constexpr int LPT = G::LPT, TPW = G::TPW, P = G::P, RING = G::RING;

    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t g = lane / LPT, xl = lane % LPT;
    const uint32_t ty = blockIdx.x / d.strips_x, strip = blockIdx.x - ty * d.strips_x;
    const uint32_t tx = strip * TPW + g;
    const bool active = tx < d.tiles_x;
    const uint32_t x0 = tx * N, y0 = ty * N;
    const uint32_t pw = active ? min((uint32_t)N, d.width - x0) : 0u;
    const uint32_t ph = min((uint32_t)N, d.height - y0);
    const uint32_t patches = d.tiles_x * d.tiles_y;
    const uint32_t k = C * patches + ty * d.tiles_x + tx;               /* index in the offset arrays */
    uint8_t* const slot = slots + d.slots_base + (uint64_t)k * G::SLOT;

    const StripLane ln(d.width, x0, pw, xl);
    const uint8_t* src = d.rgb + (size_t)y0 * d.row_stride;   /* start of the image row, walks down; scalar */
    uint32_t kE, kO;
    ln.first_row_key(kE, kO);
    const uint32_t my_row = reduced_row<LPT>(lane);                     /* see patch_min_of_rows */
    uint32_t krow = my_row == 0 ? 0u : 0x80u;                           /* K of that row in the first period */

    uint64_t row_stride = d.row_stride;
    L3_KEEP_SGPR(row_stride);               /* kept in registers, not reloaded every row */
    /* rows first .. first + P - 1 of the patch from `row` on; rows that do not exist (of the
     * last period) repeat the last one */
    u32x3 ahead[P];
    auto load_rows = [&](const uint8_t* row, uint32_t exist) {
#pragma unroll
        for (int i = 0; i < P; ++i) ahead[i] = ln.load(row + min((uint32_t)i, exist - 1) * row_stride);
    };

    uint32_t* const ring = ring_words + g * G::RING_WORDS;
    const uint32_t ring_lds = lds_address_of(ring);
    {
        u32x4 zero = {0, 0, 0, 0};
        for (uint32_t i = xl; i < G::RING_WORDS / 4; i += LPT) reinterpret_cast<u32x4*>(ring)[i] = zero;
    }
    wave_lds_fence();

    /* ORs `value` (at most 32 bits) into the ring at bit `pos`.  The upper part may land in
     * the word behind the ring, which stands for word 0 of the next lap: the flush folds
     * it in. */
    uint32_t word_bits = __builtin_ctz(RING / 4);
    L3_KEEP_SGPR(word_bits);   /* unknown to the compiler: a bit-field extract and a shift-add, not three instructions */
    auto put = [&](uint32_t value, uint32_t pos) {
        const uint32_t w0 = __builtin_amdgcn_ubfe(pos, 5, word_bits);
        const uint32_t lo = value << (pos & 31u);
        const uint32_t hi = (value >> 1) >> (~pos & 31u);
        lds_or_pair(ring_lds + 4 * w0, lo, hi);
    };

    uint32_t rowpos = 0;       /* bit position of the next row record in the patch stream */
    uint32_t flushed = 0;      /* granules already in the slot */
    /* writes granules [flushed, end) of the stream to the slot and clears them in the ring, at
     * most one per lane of the patch */
    auto flush = [&](uint32_t end) {
        wave_lds_fence();
        const uint32_t upto = min(end, flushed + LPT);
        const uint32_t gi = flushed + xl;
        if (active && gi < upto) {
            const uint32_t at = (gi * 16) & (RING - 1);
            u32x4* cell = reinterpret_cast<u32x4*>(reinterpret_cast<uint8_t*>(ring) + at);
            u32x4 v = *cell;
            const u32x4 zero = {0, 0, 0, 0};
            *cell = zero;
            if (at == 0) {                  /* what the previous lap left for this granule's first word */
                v.x |= ring[RING / 4];
                ring[RING / 4] = 0;
            }
            *reinterpret_cast<global_u32x4*>((uintptr_t)(slot + (size_t)gi * 16)) = v;
        }
        flushed = max(flushed, upto);
        wave_lds_fence();
    };

    /* the original row above the period; zeros above the first row predict 0 */
    uint32_t up[2] = {kPixelBias, kPixelBias};
    uint32_t pixel_bias = kPixelBias;
    L3_KEEP_SGPR(pixel_bias);

    /* packs one row and moves rowpos to the next record */
    auto pack_row = [&](uint32_t extremes, uint32_t uE, uint32_t uO) {
        const uint32_t w = extremes >> 16;
        /* (up to 4 bits ahead of the stream: the ring's last word, zeros)
         * lanes without pixels add zeros to their own ring */
        put(delta_field(extremes, uE, uO), rowpos - 4 + (ln.xpix + 2) * w);
        rowpos += 12 + pw * w;
    };

    /* Periods of P rows.  A row's range takes a reduction over the patch's lanes and then a few
     * scalar-like steps; done row by row every lane works those out for itself (101 vector
     * instructions a row in all, which is what bounds this kernel), done for four rows at once
     * the steps are shared (see patch_min_of_rows; about 75, and 70 with what pack_row saved
     * later).  By this step alone a call with 32 images of 2048x1024 went from 198 to 173 us, one with
     * one of 1920x1080 from 40.7 to 34.9 us.  The rows of the next period are asked for as soon as
     * this one's channel bytes are taken out of their registers; the granules the previous period
     * completed are written out right behind those loads, so that neither is waited for before a
     * whole period of arithmetic has passed. */
    static_assert(P == 4, "patch_min_of_rows takes four rows");
    load_rows(src, ph);
    /* issue priorities as in the decoder: lowered by quarters of the rows, an older
     * workgroup of a CU a little sooner; workgroups ahead of the launch's last round keep
     * the top priority */
    const uint32_t wg = blockIdx.y * gridDim.x + blockIdx.x, wgs = gridDim.x * gridDim.y;
    const uint32_t last_round_from = wgs > 2048u ? wgs - 2048u : 0u;
    const uint32_t age_rank = min(7u, ((wg - min(wg, last_round_from)) >> 3) / 32u);
    const uint32_t drop_at[3] = {wg < last_round_from ? 0x7FFFFFFFu : (ph * (8u + age_rank) + 31u) / 32u,
                                 (ph * (16u + age_rank) + 31u) / 32u, (ph * (24u + age_rank) + 31u) / 32u};
    uint32_t next_drop = drop_at[0], stage = 0;
    const bool writes_record = active && (LPT == 32 ? (xl & 14u) == 0 : xl < 4);
    __builtin_amdgcn_s_setprio(3);
    for (uint32_t r = 0; r < ph; r += P) {
        const uint32_t rows = min((uint32_t)P, ph - r);
        if (r >= next_drop) {
            ++stage;
            next_drop = stage == 1 ? drop_at[1] : (stage == 2 ? drop_at[2] : 0x7FFFFFFFu);
            if (stage == 1) __builtin_amdgcn_s_setprio(2);
            else if (stage == 2) __builtin_amdgcn_s_setprio(1);
            else __builtin_amdgcn_s_setprio(0);
        }
        uint32_t cur[P][2];
        if (ln.ragged_wave) {
#pragma unroll
            for (int i = 0; i < P; ++i) ln.shift_down(ahead[i]);
        }
#pragma unroll
        for (int i = 0; i < P; ++i) {
            take_channel<C>(ahead[i], pixel_bias, cur[i]);
            L3_KEEP_VGPR(cur[i][0]);
            L3_KEEP_VGPR(cur[i][1]);
        }
        __builtin_amdgcn_sched_barrier(0);
        src += P * row_stride;
        if (r + P < ph) load_rows(src, ph - (r + P));
        if (r > 0) flush(rowpos >> 7);

        uint32_t uE[P], uO[P], lane_part[P], extremes[P];
        lane_part[0] = ln.filter(up, cur[0], kE, kO, uE[0], uO[0]);
        if (r == 0) ln.later_row_key(kE, kO);
#pragma unroll
        for (int i = 1; i < P; ++i) lane_part[i] = ln.filter(cur[i - 1], cur[i], kE, kO, uE[i], uO[i]);
        up[0] = cur[P - 1][0];
        up[1] = cur[P - 1][1];

        /* stage 2, steps 1-2, for all rows at once: every lane works on row my_row */
        const RowExtremes mine = extremes_of_my_row<LPT>(lane_part, my_row);
        const uint32_t my_rec = mine.record(krow);
        krow = 0x80u;
        /* a row that does not exist packs nothing: no u is below 0, and its width is 0 */
        const bool exists = my_row < rows;
        rows_to_all_lanes<LPT>(exists ? mine.packed() : 0u, extremes);

        uint32_t my_at = rowpos;
        pack_row(extremes[0], uE[0], uO[0]);
#pragma unroll
        for (int i = 1; i < P; ++i) {
            my_at = my_row == (uint32_t)i ? rowpos : my_at;
            pack_row(extremes[i], uE[i], uO[i]);
        }
        if (writes_record && exists) put(my_rec, my_at);
    }
    rowpos -= 12 * ((P - ph % P) % P);           /* the records of rows that do not exist */
    const uint32_t bytes = (rowpos + 7) / 8;
#pragma unroll
    for (int i = 0; i < G::FINAL_ROUNDS; ++i) flush((bytes + 15) / 16);
    if (active && xl == 0) sizes[d.sizes_base + k] = bytes;
}

template <int N>
__device__ __forceinline__ void strip_block(const L3EncodeDesc& d, uint32_t* __restrict__ sizes,
                                            uint8_t* __restrict__ slots) {
    __shared__ __attribute__((aligned(16))) uint32_t rings[3][StripGeom<N>::TPW * StripGeom<N>::RING_WORDS];
    if (d.patch != N || blockIdx.x >= d.strips_x * d.tiles_y) return;
    const uint32_t c = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (c == 0) encode_strip<N, 0>(d, sizes, slots, rings[0]);
    else if (c == 1) encode_strip<N, 1>(d, sizes, slots, rings[1]);
    else encode_strip<N, 2>(d, sizes, slots, rings[2]);
}

/* Descriptors either in a device table (any batch size) or, for small batches, inside
 * the kernel arguments: no upload to wait for, so consecutive calls run back to back.  Two capacities, so
 * that small batches do not carry a large argument block.  (Batches of 33 to 256 images went through the
 * table before; with the arguments marshalled column by column as well, 256 photographs 161 -> 142 us a
 * call, of which the kernels take 135; the block alone left the call to the host, 162.) */
constexpr int kArgDescsSmall = 32, kArgDescs = 256;
template <int CAP>
struct EncodePack { L3EncodeDesc d[CAP]; };
static_assert(sizeof(EncodePack<kArgDescs>) + 64 <= 32768, "kernel argument segment");

template <int N>
__global__ __launch_bounds__(192) void l3_encode_strip_kernel(const L3EncodeDesc* __restrict__ descs,
                                                              uint32_t* __restrict__ sizes,
                                                              uint8_t* __restrict__ slots) {
    strip_block<N>(descs[blockIdx.y], sizes, slots);
}
template <int N, int CAP>
__global__ __launch_bounds__(192) void l3_encode_strip_kernel_args(const EncodePack<CAP> pack,
                                                                   uint32_t* __restrict__ sizes,
                                                                   uint8_t* __restrict__ slots) {
    strip_block<N>(pack.d[blockIdx.y], sizes, slots);
}

/* The fixed part of the file's header. */
__device__ __forceinline__ void write_fixed_header(const L3EncodeDesc& d) {
    uint8_t* f = d.file;
    f[0] = 0x4C; f[1] = 0x33; f[2] = 0x00; f[3] = 0x01;
    for (int b = 0; b < 4; ++b) {
        f[4 + b] = (uint8_t)(d.width >> (8 * b));
        f[8 + b] = (uint8_t)(d.height >> (8 * b));
    }
    f[12] = (uint8_t)d.patch;
}

/* The same where there is room for it, and what the caller is told about the file. */
__device__ __forceinline__ void write_header(const L3EncodeDesc& d, uint64_t need, uint64_t header,
                                             uint64_t* __restrict__ file_len, uint32_t* __restrict__ status) {
    file_len[d.status_index] = need;
    uint32_t st = 0;
    if (need > d.file_cap) st |= 1u;                       /* output capacity too small: nothing packed */
    if (need - header > 0xFFFFFFFFull) st |= 2u;           /* data section beyond 32-bit offsets */
    if (status) status[d.status_index] = st;
    if (header <= d.file_cap) write_fixed_header(d);
}

/* How a workgroup of the compaction shares its slots: a slot of a 128-pixel patch (up to 16.6 KB)
 * takes all four waves, one of a 64-pixel patch one wave, and of the 32-pixel ones (0.8 KB
 * on photographs, less than one granule per lane) a wave takes four, so that its loads travel
 * together. */
template <int N>
struct CompactGeom {
    static constexpr int WAVE_SLOTS = N == 32 ? 4 : 1;                      /* slots a wave works on */
    static constexpr int LANES = N == 128 ? 256 : 64;                       /* threads on a slot */
    static constexpr int SLOTS = N == 128 ? 1 : 4 * WAVE_SLOTS;             /* slots of a workgroup */
    static_assert(SLOTS <= 16, "offsets inside a workgroup are a scan over one 16-lane row");
};

/* Which calls lay their files out in the compaction itself (OWN_LAYOUT below).  A workgroup then reads
 * all patch sizes of its image, so what is read grows with the square of the patches and with
 * the number of images; the layout kernel's time grows with the largest image only (2.5 us, and
 * 3.5 us for every 1000 of its patches).  The reads come out of the L2 at 10 TB/s at N = 128, 13 at
 * N = 64 and, where a workgroup copies 16 slots behind them, 40 at N = 32.  So they are counted 4, 3
 * and 1 times by patch size, and taken where ten million of them a microsecond are done sooner
 * than the layout kernel.  A call with the layout kernel against one without, on one card:
 *   N = 128   32 images of 384 patches (all channels) 202.5 / 200.5 us, 1 of 4095 92.6 / 77.6, 2 of 4095
 *             153.6 / 143.8, 4 of 2700 196 / 197, 16 of 1587 407.6 / 410.5, 16 of 4095 977 / 1074
 *   N = 64    8 of 4095 156.1 / 146.2, 32 of 1587 223.1 / 223.7, 16 of 4095 287.8 / 291.7, 64 1004 / 1076
 *   N = 32    256 of 540 180.7 / 178.1, 64 of 4095 307.4 / 304.2, 128 555.7 / 555.7, 256 1057 / 1070
 * and on another, images of whole patches: N = 128, 3 of 4095 188.7 / 197.0; N = 64, 16 258.4 / 262.4; N = 32, 165
 * 620.4 / 631.6.
 * Images of more than kOwnLayoutPatches patches keep the layout kernel (one of 12288 32-pixel patches
 * would take 36.5 instead of 82.6 us without, so that bound could lie higher). */
constexpr uint32_t kOwnLayoutPatches = 4096;
/* counted as above, for one image; 32-bit and without a division: a batch is planned image by image */
constexpr uint32_t own_layout_reads(uint32_t n, uint32_t patches) {
    constexpr uint32_t s32 = CompactGeom<32>::SLOTS, s64 = CompactGeom<64>::SLOTS;
    static_assert(CompactGeom<128>::SLOTS == 1 && 4ull * kOwnLayoutPatches * kOwnLayoutPatches <= 0xFFFFFFFFull, "");
    return n == 32 ? patches * ((patches + s32 - 1) / s32) : n == 64 ? 3 * patches * ((patches + s64 - 1) / s64) : 4 * patches * patches;
}
constexpr bool own_layout_pays(uint32_t max_patches, uint64_t reads) {
    return max_patches <= kOwnLayoutPatches && reads <= 36000ull * (max_patches + 700);
}

/* Copies the slots of the strip route to their places in the file.
 * OWN_LAYOUT: every workgroup works out where its slots go: it adds up all patch sizes of the
 * image and those ahead of its own (a few loads per thread, out of the L2), instead of waiting
 * for a kernel of one workgroup per image that does so once for all (5 to 9 us, of which a call
 * with one image has nothing to hide behind).  Otherwise the layout kernel runs first and the
 * offsets are read from the header.  The rule is own_layout_pays. */
template <int N, bool OWN_LAYOUT>
__device__ __forceinline__ void compact_block(const L3EncodeDesc& d, const uint32_t* __restrict__ sizes,
                                              const uint8_t* __restrict__ slots,
                                              uint64_t* __restrict__ file_len, uint32_t* __restrict__ status) {
    using G = CompactGeom<N>;
    const uint32_t patches = d.tiles_x * d.tiles_y, total = 3 * patches;
    const uint32_t first = blockIdx.x * G::SLOTS;
    if (d.patch != N || first >= total) return;
    const uint64_t header = 13 + 12ull * patches;
    const uint32_t lane = threadIdx.x & 63u, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t* const image_sizes = sizes + d.sizes_base;
    uint8_t* const table = d.file + 13;                   /* the three offset arrays */

    /* lane j of every wave: size and offset of the workgroup's slot j */
    const uint32_t k = first + lane;
    const bool mine = lane < (uint32_t)G::SLOTS && k < total;
    const uint32_t size = mine ? image_sizes[k] : 0u;
    uint32_t offset = 0;
    uint64_t need;
    if (OWN_LAYOUT) {
        uint32_t all = 0, ahead = 0;                      /* at most 4096 * 16.6 KB */
        for (uint32_t i = threadIdx.x; i < total; i += 256) {
            const uint32_t s = image_sizes[i];
            all += s;
            ahead += i < first ? s : 0u;
        }
#pragma unroll
        for (int step = 32; step >= 1; step >>= 1) {
            all += (uint32_t)__shfl_xor((int)all, step);
            ahead += (uint32_t)__shfl_xor((int)ahead, step);
        }
        __shared__ uint32_t parts[4][2];
        if (lane == 0) {
            parts[wave][0] = all;
            parts[wave][1] = ahead;
        }
        __syncthreads();
        all = parts[0][0] + parts[1][0] + parts[2][0] + parts[3][0];
        ahead = parts[0][1] + parts[1][1] + parts[2][1] + parts[3][1];
        uint32_t upto = size;                             /* inclusive scan of the first 16 lanes */
        if (G::SLOTS > 1) {
#pragma unroll
            for (int step = 1; step < 16; step <<= 1) {
                const uint32_t from = (uint32_t)__shfl_up((int)upto, step);
                upto += lane >= (uint32_t)step ? from : 0u;
            }
        }
        offset = ahead + upto - size;
        need = header + all;
        if (wave == 0 && mine && header <= d.file_cap)
            *reinterpret_cast<global_u32_any*>((uintptr_t)(table + 4 * (size_t)k)) = offset;
        if (first == 0 && threadIdx.x == 0) write_header(d, need, header, file_len, status);
    } else {
        need = file_len[d.status_index];
    }
    if (need > d.file_cap || need - header > 0xFFFFFFFFull) return;
    if (!OWN_LAYOUT && mine)
        offset = *reinterpret_cast<global_const_u32_any*>((uintptr_t)(table + 4 * (size_t)k));

    /* Bound by memory: 32 images of 2048x1024 move 330 MB in 57 us, 256 photographs of 39 million
     * pixels 180 MB in 40 us (the layout kernel and this one took 57 and 54 us before, with one
     * 64-thread workgroup per slot of the photographs).  Measured slower: aligned stores with the
     * slot read at any alignment instead (64 us with four granules per lane in flight), that
     * many in flight otherwise (60 us), non-temporal stores (a call with 32 images in turn with
     * others 176.5 instead of 171.6 us), non-temporal slot stores in the strip kernel (62 us here). */
    const uint32_t me = N == 128 ? threadIdx.x : lane;
    const uint8_t* from[G::WAVE_SLOTS];
    uint8_t* to[G::WAVE_SLOTS];
    uint32_t whole[G::WAVE_SLOTS], tail[G::WAVE_SLOTS];
    u32x4 v[G::WAVE_SLOTS];
    uint8_t last[G::WAVE_SLOTS];
#pragma unroll
    for (int j = 0; j < G::WAVE_SLOTS; ++j) {
        const uint32_t nth = N == 128 ? 0u : wave * G::WAVE_SLOTS + j;
        const uint32_t bytes = (uint32_t)__builtin_amdgcn_readlane((int)size, (int)nth);
        from[j] = slots + d.slots_base + (uint64_t)(first + nth) * strip_slot_bytes(N);
        to[j] = d.file + header + (uint32_t)__builtin_amdgcn_readlane((int)offset, (int)nth);
        whole[j] = bytes / 16;
        tail[j] = bytes & 15u;
        if (me < whole[j]) v[j] = *reinterpret_cast<global_const_u32x4*>((uintptr_t)(from[j] + 16 * me));
        if (me < tail[j]) last[j] = from[j][16 * whole[j] + me];
    }
#pragma unroll
    for (int j = 0; j < G::WAVE_SLOTS; ++j) {
        if (me < whole[j])
            *reinterpret_cast<global_u32x4_any*>((uintptr_t)(to[j] + 16 * me)) = v[j];
        for (uint32_t i = me + G::LANES; i < whole[j]; i += G::LANES)
            *reinterpret_cast<global_u32x4_any*>((uintptr_t)(to[j] + 16 * i)) =
                *reinterpret_cast<global_const_u32x4*>((uintptr_t)(from[j] + 16 * i));
        if (me < tail[j]) to[j][16 * whole[j] + me] = last[j];
    }
}
template <int N, bool OWN_LAYOUT>
__global__ __launch_bounds__(256) void l3_encode_compact_kernel(const L3EncodeDesc* __restrict__ descs,
                                                                const uint32_t* __restrict__ sizes,
                                                                const uint8_t* __restrict__ slots,
                                                                uint64_t* __restrict__ file_len,
                                                                uint32_t* __restrict__ status) {
    compact_block<N, OWN_LAYOUT>(descs[blockIdx.y], sizes, slots, file_len, status);
}
template <int N, bool OWN_LAYOUT, int CAP>
__global__ __launch_bounds__(256) void l3_encode_compact_kernel_args(const EncodePack<CAP> pack,
                                                                     const uint32_t* __restrict__ sizes,
                                                                     const uint8_t* __restrict__ slots,
                                                                     uint64_t* __restrict__ file_len,
                                                                     uint32_t* __restrict__ status) {
    compact_block<N, OWN_LAYOUT>(pack.d[blockIdx.y], sizes, slots, file_len, status);
}

/* ---- the chained route: N in {32, 64, 128}, room for the longest file ---------- */

/* One kernel for calls of few strips whose files all have room for the longest stream there is
 * (l3_encode_bound).  The strip kernel walks a strip's rows in one wave a channel, which is what such a call
 * waits for, and the copy behind it waits for all of them.  Here a workgroup encodes one channel of a
 * strip, that is patches that follow one another in the file: a wave takes R of the strip's rows (the
 * filter needs the original row above, not a decoded one), keeps their residuals in registers and works out
 * the rows' widths; with the waves' bit counts in LDS every wave knows where its rows begin and packs them
 * into the unit's bytes in LDS.  Where those go in the file depends on the sizes of all units ahead of
 * it in the image: each unit publishes its size as soon as it is known, ahead of packing, and adds up what
 * the units ahead published (a decoupled look-back, Merrill and Garland 2016), 512 of them a round trip.
 *
 * Which image a workgroup works for follows from its number, but the image's units are taken in the
 * order of a ticket, so that all units that one waits for are already with running workgroups, and those
 * wait for smaller tickets only: every wait ends, whatever else runs on the GPU.  Images are taken in
 * the order of workgroups, spread over the XCDs: with an eighth of the images on each as in the other kernels
 * units look for others that have only just begun (256 photographs 207 us a call instead of 158).
 *
 * What bounds it (one image of 1920x1080: 15.9 us, 18.9 and 5.3 before) is a chain of round trips, the
 * ticket, the rows, the look and the stores, with some 5 us of arithmetic between; the look costs 2 us of
 * it.  Which calls take it: see chained_pays.  Measured the same or slower: 16 rows a wave at N = 32 and 64 (4
 * photographs 14.9 us, 11.7 with 8), 8 at N = 128 (32 images of 2048x1024 182 us, 177 with 16), the first look
 * ahead of all packing instead of in its middle (183 us). */
template <int N>
struct UnitGeom {
    static constexpr int LPT = N / 4;              /* lanes per patch, 4 pixels each */
    static constexpr int TPW = 64 / LPT;           /* patches of a unit */
    static constexpr int R = N == 128 ? 16 : 8;    /* rows of a wave */
    static constexpr int WAVES = N / R, THREADS = 64 * WAVES;
    static constexpr int Q = R / 4;                /* fours of rows, reduced together */
    /* the unit's bytes in LDS: from word LEAD on (a lane's field may begin 4 bits ahead of the first
     * record, with zeros there), and room for the word behind the last */
    static constexpr int LEAD = 4;
    static constexpr int WORDS = TPW * (N * (12 + 8 * N) / 8) / 4;
    static constexpr int ALL_WORDS = (LEAD + WORDS + 2 + 3) / 4 * 4;
    static_assert(WORDS * 4 == TPW * (N * (12 + 8 * N) / 8), "whole words");
    static_assert(WAVES <= 16 && R % 4 == 0, "fours of rows, and a workgroup of at most 1024 threads");
};

/* What a unit tells the others, one 64-bit word (cell) each: the number of the launch, whether the value
 * includes all units ahead in the image, and a number of bytes.  A cell with another number is from an
 * earlier launch.  The host counts a context's launches and passes each its number; the images of a launch
 * have their units' cells one behind the other.
 * Tickets are taken from a word that holds the launch's number and the image's next unit.  An image has two
 * such words, for even and odd numbers, and each launch makes the other ones ready for the next, also those of
 * images that it has not itself: nothing is cleared between launches, and words that anything has disturbed are
 * right again a launch later.  (One word that is raised to the launch's number and then taken from does the same with
 * two accesses a workgroup, which queue up at the word, some 10 ns each: one image of 1920x1080 23.1 us instead of 19.4, one
 * of 3840x1500 at N = 32 77.7 instead of 57.0.)  After 2^35 launches, 5 us apart two days, all are cleared and
 * numbers begin again. */
constexpr int kCellValueBits = 28;
constexpr uint64_t kChainMaxBytes = (1ull << kCellValueBits) - 1;
constexpr uint64_t kCellWhole = 1ull << kCellValueBits;
constexpr int kNumberShift = kCellValueBits + 1;
constexpr uint64_t kLastNumber = ~0ull >> kNumberShift;
/* Many workgroups add to a ticket: a cache line each, also apart from the one that is made ready (beside each other 2
 * images of 1920x1080 27.5 us, so 26.3). */
struct __attribute__((aligned(128))) L3Ticket { uint64_t next; };   /* number << 29 | the image's next unit */
struct L3ChainWord {
    L3Ticket ticket[2];                                 /* of even and odd numbers */
    uint64_t gave_up;                                   /* the last launch in which a unit of the image was not written */
};

/* Calls that take this route: few units, N = 32 ones counted by two thirds (four waves, not eight).  Every
 * unit reads all three channels' bytes, and with many in flight those no longer meet in a cache (32 images of
 * 2048x1024 fetch 547 MB instead of 219), which the strip kernel and the copy then do better; 4 a CU
 * is where they draw level.  An image of so many patches that they would need the layout kernel
 * between them (own_layout_pays) is worth it up to 12 a CU.  A call by the strip kernel / by this (units):
 *   N = 32    1 of 64x64 (6) 16.5 / 11.4 us, 1 photograph (72) 18.7 / 11.2, 16 (1056) 22.9 / 17.9, 4 of 1024x720 (1104) 24.7 / 20.7;
 *             with the layout kernel 1 of 3840x1500 (2115) 107.7 / 56.7
 *   N = 64    1 of 1920x1080 (408) 27.5 / 19.1, 2 (816) 32.4 / 26.2; with the layout kernel 1 of 2816x2048 (1056) 50.9 / 37.7
 *   N = 128   1 of 2048x1024 (192) 39.3 / 15.8, 4 (768) 42.9 / 32.4, 1 of 3840x2160 (765) 42.7 / 39.5
 * and beyond the line, measured when this kernel was a few percent slower,
 *   N = 32    6 of 1024x720 (1656) 28.9 / 27.5, 8 (2208) 29.6 / 32.9, 32 74.6 / 96.2
 *   N = 64    3 of 1920x1080 (1224) 32.9 / 33.5, 4 (1632) 38.9 / 40.4, 32 182.8 / 249.5
 *   N = 128   8 of 2048x1024 (1536) 58.5 / 51.5, 16 (3072) 94.9 / 95.1, 2 of 3840x2160 (1530) 59.8 / 63.7 */
constexpr uint32_t kMostChainUnits = 3072;
/* The units of one image also wait for one another, at their ticket and in their looks: long images are the
 * strip kernel's sooner.  (At N = 128, where a unit is twice the work, they are not before the 1024 above.)
 *   N = 32    1 of 1200x1000 (480) 20.9 / 18.3, 2 of 1000x1300 (984, 492 each) 23.9 / 24.2, 2 of 1100x1150 (1080, 540 each) 23.8 / 25.7
 *   N = 64    1 of 1920x1408 (528) 25.9 / 23.0, 1 of 2100x1600 (675) 26.9 / 26.9, 1 of 2400x1600 (750) 27.3 / 27.9,
 *             1 of 2048x2048 (768) 26.1 / 28.7, 1 of 2560x1900 (900) 30.4 / 33.4
 *   N = 128   1 of 4096x2304 (864) 49.0 / 41.9, 1 of 4096x2560 (960) 49.7 / 44.6 */
constexpr uint32_t kMostUnitsOfOne[2] = {480, 640};
constexpr bool chained_pays(const uint32_t (&strips)[3], uint64_t images, bool own_layout) {
    if (own_layout && (3 * strips[0] > kMostUnitsOfOne[0] || 3 * strips[1] > kMostUnitsOfOne[1])) return false;
    const uint64_t two_thirds = 3 * images * (2ull * strips[0] + 3ull * strips[1] + 3ull * strips[2]);   /* of units, times 3 */
    return two_thirds <= 3ull * (own_layout ? 1024 : kMostChainUnits) && 3 * images * strips[0] <= kMostChainUnits;
}
static_assert(kMostChainUnits * (uint64_t)UnitGeom<128>::WORDS * 4 <= kChainMaxBytes, "an image's bytes fit a cell");
constexpr uint32_t kMostChainImages = kMostChainUnits / 3;      /* no image has fewer than three units */
/* How often a unit looks for the ones ahead before it gives up (each look is a round trip to memory,
 * about a microsecond: a second in all).  By the order of tickets it cannot happen; if it did, the unit would
 * not be written and its image's status word would say so. */
constexpr uint32_t kMaxLooks = 1u << 20;
constexpr uint32_t kStatusGaveUp = 4u;

/* The status word is cleared by the image's unit 0, which may be the one that the others wait for in vain.  So who
 * gives up first leaves the launch's number in the image's word and then sets the bit, and unit 0 first clears and
 * then looks for that number: one of the two sees the other.  Each waits for its first access's answer. */
__device__ __forceinline__ void give_up(L3ChainWord* word, uint64_t number, uint32_t* status) {
    uint64_t before = agent_exchange_u64(&word->gave_up, number);
    L3_WAIT_FOR(before);
    if (status) atomicOr(status, kStatusGaveUp);
}

/* The cells of the 512 units that end `behind` units ahead of `unit`, in the lanes of a wave; `cell` is
 * the unit's own, those of the units ahead lie in front of it. */
struct ChainLook {
    static constexpr int W = 8;
    uint64_t c[W];
    __device__ __forceinline__ void at(const uint64_t* cell, uint32_t unit, uint64_t number, uint32_t lane, uint32_t behind) {
#pragma unroll
        for (int j = 0; j < W; ++j) {
            const uint32_t back = behind + 64 * j + lane;          /* units between this one and that */
            c[j] = number << kNumberShift | kCellWhole;             /* ahead of the image: nothing, and all of it */
            if (back < unit) c[j] = agent_load_u64(cell - 1 - back);
        }
    }
};
/* Bytes of the units ahead, given the first look at them; false if it gave up. */
__device__ __forceinline__ bool bytes_ahead(ChainLook look, const uint64_t* cell, uint32_t unit, uint64_t number,
                                            uint32_t lane, uint32_t& ahead) {
    uint32_t sum = 0, behind = 0, looks = 0;
    bool whole = false, ok = true;
    for (;;) {
        uint32_t part = 0;
        bool missing = false;
#pragma unroll
        for (int j = 0; j < ChainLook::W; ++j) {
            const bool there = look.c[j] >> kNumberShift == number;
            const uint64_t have = __builtin_amdgcn_ballot_w64(there);
            const uint64_t full = __builtin_amdgcn_ballot_w64(there && (look.c[j] & kCellWhole) != 0);
            const uint64_t upto = full ? full ^ (full - 1) : ~0ull;   /* the nearest that holds all ahead of it, and those nearer */
            if (!whole && !missing) {
                missing = (have & upto) != upto;
                part += upto >> lane & 1u ? (uint32_t)(look.c[j] & kChainMaxBytes) : 0u;
                whole = !missing && full != 0;
            }
        }
        if (missing) {
            ok = ++looks < kMaxLooks;
        } else {
            sum += part;
            behind += 64 * ChainLook::W;
        }
        if (whole || !ok) break;
        look.at(cell, unit, number, lane, behind);
    }
#pragma unroll
    for (int step = 32; step >= 1; step >>= 1) sum += (uint32_t)__shfl_xor((int)sum, step);
    ahead = sum;
    return ok;
}

template <int N>
__device__ __forceinline__ void encode_unit(const L3EncodeDesc& d, const uint32_t unit, const uint32_t units,
                                            const uint64_t number, L3ChainWord* __restrict__ word, uint64_t* __restrict__ cell,
                                            uint64_t* __restrict__ file_len, uint32_t* __restrict__ status) {
    using G = UnitGeom<N>;
    constexpr int LPT = G::LPT, TPW = G::TPW, R = G::R, Q = G::Q, WAVES = G::WAVES;
    __shared__ __attribute__((aligned(16))) uint32_t stream[G::ALL_WORDS];
    __shared__ uint32_t wave_bits[WAVES][TPW];
    __shared__ uint32_t place[2];               /* the unit's offset in the data section; 1: known */

    const uint32_t lane = threadIdx.x & 63u, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t g = lane / LPT, xl = lane % LPT;
    const uint32_t channel_units = d.strips_x * d.tiles_y;
    const uint32_t c = unit / channel_units, in_channel = unit - c * channel_units;
    const uint32_t ty = in_channel / d.strips_x, strip = in_channel - ty * d.strips_x;
    const uint32_t tx = strip * TPW + g;
    const bool active = tx < d.tiles_x;
    const uint32_t x0 = tx * N, y0 = ty * N;
    const uint32_t pw = active ? min((uint32_t)N, d.width - x0) : 0u;
    const uint32_t ph = min((uint32_t)N, d.height - y0);
    const StripLane ln(d.width, x0, pw, xl);

    /* rows first .. first + R - 1 of the patch and the one above them; rows that do not exist repeat
     * the last one */
    const uint32_t first = wave * R;
    u32x3 raw[R + 1];
    {
        const uint8_t* row = d.rgb + (size_t)(y0 + min(first - min(first, 1u), ph - 1)) * d.row_stride;
        const uint64_t row_stride = d.row_stride;
        const auto load_all = [&](auto load) {
#pragma unroll
            for (int i = 0; i <= R; ++i) {
                raw[i] = load(row);
                row += first + i > 0 && first + i < ph ? row_stride : 0;      /* row i + 1 of these is row first + i */
            }
        };
        if (ln.wide) load_all([&](const uint8_t* r) { return ln.load_wide(r); });
        else load_all([&](const uint8_t* r) { return ln.load_narrow(r); });
    }
    {
        const u32x4 zero = {0, 0, 0, 0};
        for (uint32_t i = threadIdx.x; i < G::ALL_WORDS / 4; i += G::THREADS) reinterpret_cast<u32x4*>(stream)[i] = zero;
    }
    if (ln.ragged_wave) {
#pragma unroll
        for (int i = 0; i <= R; ++i) ln.shift_down(raw[i]);
    }
    uint32_t cur[R + 1][2], pixel_bias = kPixelBias;
    L3_KEEP_SGPR(pixel_bias);
    if (c == 0) {
#pragma unroll
        for (int i = 0; i <= R; ++i) take_channel<0>(raw[i], pixel_bias, cur[i]);
    } else if (c == 1) {
#pragma unroll
        for (int i = 0; i <= R; ++i) take_channel<1>(raw[i], pixel_bias, cur[i]);
    } else {
#pragma unroll
        for (int i = 0; i <= R; ++i) take_channel<2>(raw[i], pixel_bias, cur[i]);
    }

    /* Section 4.2: filter, and the rows' widths, four rows at a time */
    const uint32_t my_row = reduced_row<LPT>(lane);                 /* see patch_min_of_rows */
    uint32_t kE, kO, krow = 0x80u;
    ln.later_row_key(kE, kO);
    if (wave == 0) {                 /* zeros above the patch's first row predict 0; it is looked at as unsigned */
        cur[0][0] = cur[0][1] = kPixelBias;
        ln.first_row_key(kE, kO);
        krow = my_row == 0 ? 0u : 0x80u;
    }
    uint32_t uE[R], uO[R], mine[Q], my_rec[Q], my_widths = 0;
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        uint32_t part[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            part[i] = ln.filter(cur[4 * q + i], cur[4 * q + i + 1], kE, kO, uE[4 * q + i], uO[4 * q + i]);
            if (q == 0 && i == 0) ln.later_row_key(kE, kO);
        }
        const RowExtremes m = extremes_of_my_row<LPT>(part, my_row);
        my_rec[q] = m.record(krow);
        krow = 0x80u;
        /* a row that does not exist packs nothing: no u is below 0, and its width is 0 */
        mine[q] = first + 4 * q + my_row < ph ? m.packed() : 0u;
        my_widths += mine[q] >> 16;
    }

    /* how many bits the wave's rows of each patch take, and from the other waves' where they begin */
    uint32_t widths[4];
    rows_to_all_lanes<LPT>(my_widths, widths);
    const uint32_t exist = ph - min(ph, first) < (uint32_t)R ? ph - min(ph, first) : (uint32_t)R;
    const uint32_t bits = active ? 12 * exist + pw * (widths[0] + widths[1] + widths[2] + widths[3]) : 0u;
    if (xl == 0) wave_bits[wave][g] = bits;
    __syncthreads();
    uint32_t before = 0, patch_bits = 0;
#pragma unroll
    for (uint32_t w = 0; w < (uint32_t)WAVES; ++w) {
        const uint32_t b = wave_bits[w][g];
        before += w < wave ? b : 0u;
        patch_bits += b;
    }
    const uint32_t patch_bytes = (patch_bits + 7) / 8;
    uint32_t patch_at = 0, unit_bytes = 0;       /* the patch's first byte in the unit; the unit's bytes */
#pragma unroll
    for (int p = 0; p < TPW; ++p) {
        patch_at = g == (uint32_t)p ? unit_bytes : patch_at;
        unit_bytes += (uint32_t)__builtin_amdgcn_readlane((int)patch_bytes, p * LPT);
    }
    const bool looks_back = wave == WAVES - 1;   /* the wave with the fewest rows */
    if (looks_back && lane == 0)
        agent_store_u64(cell, number << kNumberShift | (unit == 0 ? kCellWhole : 0u) | unit_bytes);
    /* behind the size that the others wait for */
    uint32_t cleared = 0;
    if (unit == 0 && threadIdx.x == 0 && status) cleared = agent_exchange_u32(&status[d.status_index], 0);

    /* the deltas of all rows into the unit's bytes */
    const uint32_t stream_lds = lds_address_of(stream);
    auto put = [&](uint32_t value, uint32_t pos) {
        const uint32_t lo = value << (pos & 31u);
        const uint32_t hi = (value >> 1) >> (~pos & 31u);
        lds_or_pair(stream_lds + (pos >> 5) * 4, lo, hi);
    };
    /* Zeros that all lanes put into one word queue up there.  So lanes without a patch put theirs into words of
     * their own, and rows that do not exist are left out where a four of them has none: images whose last row of patches is short
     * or whose last strip has few patches waited for these zeros (at N = 128 2 of 2500x1700 51.1 us, 40.0
     * so, 2 of 1920x1080 30.6 and 22.1, 32 of 300x300 40.0 and 25.2). */
    uint32_t rowpos = 32 * G::LEAD + (active ? 8 * patch_at + before : 32 * lane);
    const bool writes_record = active && (LPT == 32 ? (xl & 14u) == 0 : xl < 4);
    ChainLook look;
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        if (q == Q / 2 && looks_back) look.at(cell, unit, number, lane, 0);
        if (first + 4 * q >= ph) continue;
        uint32_t extremes[4], my_at = rowpos;
        rows_to_all_lanes<LPT>(mine[q], extremes);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const uint32_t w = extremes[i] >> 16;
            if (i) my_at = my_row == (uint32_t)i ? rowpos : my_at;
            put(delta_field(extremes[i], uE[4 * q + i], uO[4 * q + i]), rowpos - 4 + (ln.xpix + 2) * w);
            rowpos += 12 + pw * w;
        }
        if (writes_record && first + 4 * q + my_row < ph) put(my_rec[q], my_at);
    }

    if (looks_back) {
        uint32_t ahead;
        const bool known = bytes_ahead(look, cell, unit, number, lane, ahead);
        if (lane == 0) {
            if (known && unit) agent_store_u64(cell, number << kNumberShift | kCellWhole | (ahead + unit_bytes));
            place[0] = ahead;
            place[1] = known;
        }
    }
    __syncthreads();
    const uint32_t patches = d.tiles_x * d.tiles_y;
    const uint64_t header = 13 + 12ull * patches;
    const uint32_t at = place[0];
    if (!place[1]) {
        if (threadIdx.x == 0) {
            give_up(word, number, status ? &status[d.status_index] : nullptr);
            if (unit == units - 1) file_len[d.status_index] = 0;
        }
        return;
    }
    if (wave == 0 && xl == 0 && active)          /* Section 4.3, the offset array of channel c */
        *reinterpret_cast<global_u32_any*>((uintptr_t)(d.file + 13 + 4 * (size_t)(c * patches + ty * d.tiles_x + tx))) = at + patch_at;
    if (threadIdx.x == 0) {
        if (unit == 0) write_fixed_header(d);
        if (unit == units - 1) file_len[d.status_index] = header + at + unit_bytes;
    }
    uint8_t* const to = d.file + header + at;
    const uint32_t whole = unit_bytes / 16, tail = unit_bytes & 15u;
    const uint32_t* const from = stream + G::LEAD;
    for (uint32_t i = threadIdx.x; i < whole; i += G::THREADS)
        *reinterpret_cast<global_u32x4_any*>((uintptr_t)(to + 16 * (size_t)i)) = reinterpret_cast<const u32x4*>(from)[i];
    if (threadIdx.x < tail)
        to[16 * (size_t)whole + threadIdx.x] = reinterpret_cast<const uint8_t*>(from)[16 * (size_t)whole + threadIdx.x];
    if (unit == 0 && threadIdx.x == 0 && status) {
        L3_WAIT_FOR(cleared);
        if (agent_load_u64(&word->gave_up) == number) atomicOr(&status[d.status_index], kStatusGaveUp);
    }
}

template <int N, class Descs>
__device__ __forceinline__ void chain_block(const Descs& descs, uint32_t units_per_image, L3ChainWord* __restrict__ words,
                                            uint64_t* __restrict__ cells, uint64_t number, uint32_t slots,
                                            uint64_t* __restrict__ file_len, uint32_t* __restrict__ status) {
    const uint32_t image = blockIdx.x / units_per_image;      /* in dispatch order: see encode_unit */
    /* what the rows' addresses wait for is read while the ticket travels */
    L3EncodeDesc d = descs[image];
    L3_KEEP_SGPR(d.rgb);
    L3_KEEP_SGPR(d.file);
    L3_KEEP_SGPR(d.row_stride);
    L3_KEEP_SGPR(d.width);
    L3_KEEP_SGPR(d.height);
    L3_KEEP_SGPR(d.tiles_x);
    L3_KEEP_SGPR(d.tiles_y);
    L3_KEEP_SGPR(d.strips_x);
    L3_KEEP_SGPR(d.patch);
    L3_KEEP_SGPR(d.status_index);
    L3_KEEP_SGPR(words);
    __shared__ uint64_t taken;
    if (threadIdx.x == 0) {
        taken = agent_add_u64(&words[image].ticket[number & 1].next, 1);
        if (blockIdx.x == image * units_per_image)
            agent_store_u64(&words[image].ticket[~number & 1].next, (number + 1) << kNumberShift);
    }
    if (blockIdx.x == 0)
        for (uint32_t i = gridDim.x / units_per_image + threadIdx.x; i < slots; i += blockDim.x)
            agent_store_u64(&words[i].ticket[~number & 1].next, (number + 1) << kNumberShift);
    if (d.patch != N) return;
    __syncthreads();
    const uint32_t low = __builtin_amdgcn_readfirstlane((uint32_t)taken);
    const uint32_t high = __builtin_amdgcn_readfirstlane((uint32_t)(taken >> 32));
    const uint32_t unit = low & (uint32_t)(kCellWhole * 2 - 1);
    const uint32_t units = 3 * d.strips_x * d.tiles_y;
    if (((uint64_t)high << 32 | low) >> kNumberShift != number) {      /* a disturbed word */
        if (threadIdx.x == 0) give_up(&words[image], number, status ? &status[d.status_index] : nullptr);
        return;
    }
    if (unit < units)
        encode_unit<N>(d, unit, units, number, &words[image], cells + (size_t)image * units_per_image + unit, file_len, status);
}
template <int N>
__global__ __launch_bounds__(UnitGeom<N>::THREADS) void l3_encode_chain_kernel(
    const L3EncodeDesc* __restrict__ descs, uint32_t units_per_image, L3ChainWord* __restrict__ words,
    uint64_t* __restrict__ cells, uint64_t number, uint32_t slots, uint64_t* __restrict__ file_len,
    uint32_t* __restrict__ status) {
    chain_block<N>(descs, units_per_image, words, cells, number, slots, file_len, status);
}
template <int N, int CAP>
__global__ __launch_bounds__(UnitGeom<N>::THREADS) void l3_encode_chain_kernel_args(
    const EncodePack<CAP> pack, uint32_t units_per_image, L3ChainWord* __restrict__ words,
    uint64_t* __restrict__ cells, uint64_t number, uint32_t slots, uint64_t* __restrict__ file_len,
    uint32_t* __restrict__ status) {
    chain_block<N>(pack.d, units_per_image, words, cells, number, slots, file_len, status);
}
__global__ void l3_encode_clear_kernel(L3ChainWord* __restrict__ words, uint64_t* __restrict__ cells) {
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < kMostChainImages) {
        words[i].ticket[0].next = 2ull << kNumberShift;       /* the first launch behind this has the number 2 */
        words[i].ticket[1].next = words[i].gave_up = 0;
    }
    if (i < kMostChainUnits) cells[i] = 0;
}

/* ---- the plain route: any other N up to 128 -------------------------------- */

__global__ __launch_bounds__(64) void l3_encode_measure_kernel(const L3EncodeDesc* __restrict__ descs,
                                                               uint32_t* __restrict__ sizes) {
    const L3EncodeDesc& d = descs[blockIdx.y];
    const uint32_t patches = d.tiles_x * d.tiles_y;
    const uint32_t k = blockIdx.x;
    if (k >= 3 * patches || d.patch == 32 || d.patch == 64 || d.patch == 128) return;
    const uint32_t c = k / patches, i = k - c * patches;
    const uint32_t bits = walk_patch<false>(d, c, i % d.tiles_x, i / d.tiles_x, nullptr);
    if (threadIdx.x == 0) sizes[d.sizes_base + k] = (bits + 7) / 8;
}

/* One workgroup per image: offsets = exclusive prefix sum of the patch sizes. */
__device__ __forceinline__ void layout_block(const L3EncodeDesc& d, const uint32_t* __restrict__ sizes,
                                             uint64_t* __restrict__ file_len,
                                             uint32_t* __restrict__ status) {
    const uint32_t patches = d.tiles_x * d.tiles_y, total = 3 * patches;
    const uint64_t header = 13 + 12ull * patches;
    const bool header_fits = header <= d.file_cap;
    __shared__ uint64_t scan[256];
    __shared__ uint64_t carry;
    if (threadIdx.x == 0) carry = 0;
    __syncthreads();
    for (uint32_t first = 0; first < total; first += 256) {
        const uint32_t k = first + threadIdx.x;
        const uint64_t mine = k < total ? sizes[d.sizes_base + k] : 0;
        scan[threadIdx.x] = mine;
        __syncthreads();
        for (uint32_t step = 1; step < 256; step <<= 1) {       /* inclusive scan of the chunk */
            const uint64_t add = threadIdx.x >= step ? scan[threadIdx.x - step] : 0;
            __syncthreads();
            scan[threadIdx.x] += add;
            __syncthreads();
        }
        const uint64_t offset = carry + scan[threadIdx.x] - mine;
        if (k < total && header_fits && offset <= 0xFFFFFFFFull)
            *reinterpret_cast<global_u32_any*>((uintptr_t)(d.file + 13 + 4 * (size_t)k)) = (uint32_t)offset;
        __syncthreads();
        if (threadIdx.x == 255) carry += scan[255];
        __syncthreads();
    }
    if (threadIdx.x == 0) write_header(d, header + carry, header, file_len, status);
}
__global__ __launch_bounds__(256) void l3_encode_layout_kernel(const L3EncodeDesc* __restrict__ descs,
                                                               const uint32_t* __restrict__ sizes,
                                                               uint64_t* __restrict__ file_len,
                                                               uint32_t* __restrict__ status) {
    layout_block(descs[blockIdx.x], sizes, file_len, status);
}
template <int CAP>
__global__ __launch_bounds__(256) void l3_encode_layout_kernel_args(const EncodePack<CAP> pack,
                                                                    const uint32_t* __restrict__ sizes,
                                                                    uint64_t* __restrict__ file_len,
                                                                    uint32_t* __restrict__ status) {
    layout_block(pack.d[blockIdx.x], sizes, file_len, status);
}

__global__ __launch_bounds__(64) void l3_encode_pack_kernel(const L3EncodeDesc* __restrict__ descs,
                                                            const uint32_t* __restrict__ sizes,
                                                            const uint64_t* __restrict__ file_len) {
    const L3EncodeDesc& d = descs[blockIdx.y];
    const uint32_t patches = d.tiles_x * d.tiles_y;
    const uint32_t k = blockIdx.x;
    if (k >= 3 * patches || d.patch == 32 || d.patch == 64 || d.patch == 128) return;
    const uint64_t need = file_len[d.status_index];
    if (need > d.file_cap || need - (13 + 12ull * patches) > 0xFFFFFFFFull) return;

    L3_DYNAMIC_LDS(uint32_t, bits);      /* sized by the host for the largest patch of the launch */
    const uint32_t bytes = sizes[d.sizes_base + k];
    const uint32_t words = (bytes + 3) / 4 + 1;
    for (uint32_t i = threadIdx.x; i < words; i += 64) bits[i] = 0;
    __syncthreads();
    const uint32_t c = k / patches, i = k - c * patches;
    (void)walk_patch<true>(d, c, i % d.tiles_x, i / d.tiles_x, bits);
    __syncthreads();

    const uint32_t offset = *reinterpret_cast<global_const_u32_any*>((uintptr_t)(d.file + 13 + 4 * (size_t)k));
    uint8_t* dst = d.file + 13 + 12 * (size_t)patches + offset;
    const uint32_t whole = bytes / 4;
    for (uint32_t w = threadIdx.x; w < whole; w += 64)
        *reinterpret_cast<global_u32_any*>((uintptr_t)(dst + 4 * (size_t)w)) = bits[w];
    const uint32_t tail = bytes - 4 * whole;
    if (threadIdx.x < tail) dst[4 * (size_t)whole + threadIdx.x] = (uint8_t)(bits[whole] >> (8 * threadIdx.x));
}

}  // namespace

/* Workspace of l3_encode_batch: descriptor table (pinned + device) and patch sizes. */
struct L3EncodeState {
    L3EncodeDesc* h_descs = nullptr;  /* pinned: kStage staging tables of desc_cap entries each */
    hipEvent_t staged[4] = {};        /* the upload from staging table i has left it */
    bool staged_pending[4] = {};
    int next_stage = 0;
    L3EncodeDesc* d_descs = nullptr;
    size_t desc_cap = 0;
    uint32_t* d_sizes = nullptr;
    size_t sizes_cap = 0;
    uint8_t* d_slots = nullptr;      /* strip route: one fixed-size slot per patch and channel */
    size_t slots_cap = 0;
    L3ChainWord* d_words = nullptr;  /* chained route: words of kMostChainImages images, and behind them kMostChainUnits cells */
    uint64_t chain_number = 0;       /* of its last launch; 0: not cleared yet, no launch has it or 1 */
    uint32_t chain_slots = 32;       /* images whose words every launch makes ready: the most a call has had, or twice that */
    hipEvent_t done = nullptr;       /* the last call's kernels have finished */
    bool pending = false;
    hipStream_t last_stream = nullptr;
};

void l3_encode_state_free(L3EncodeState* s) {
    if (!s) return;
    if (s->pending) (void)hipEventSynchronize(s->done);
    if (s->done) (void)hipEventDestroy(s->done);
    for (int i = 0; i < 4; ++i)
        if (s->staged[i]) (void)hipEventDestroy(s->staged[i]);
    if (s->h_descs) (void)hipHostFree(s->h_descs);
    if (s->d_descs) (void)hipFree(s->d_descs);
    if (s->d_sizes) (void)hipFree(s->d_sizes);
    if (s->d_slots) (void)hipFree(s->d_slots);
    if (s->d_words) (void)hipFree(s->d_words);
    delete s;
}

extern "C" l3_status l3_encode_batch(l3_ctx* ctx, const l3_encode_item* items, int n,
                                     uint64_t* d_file_len, uint32_t* d_status, void* stream_v) {
    if (!ctx || n < 0 || (n > 0 && (!items || !d_file_len))) return L3_ERR_INVALID_ARG;
    if (n == 0) return L3_OK;
    hipStream_t stream = static_cast<hipStream_t>(stream_v);
    DeviceGuard guard(ctx->device);
    if (!guard.ok) return L3_ERR_DEVICE;

    size_t total_patches = 0, slot_bytes = 0;
    uint32_t max_patches = 0, max_n = 1;
    uint32_t strip_units[3] = {0, 0, 0};   /* largest grid of the strip route per N = 32, 64, 128 */
    uint32_t strip_slots[3] = {0, 0, 0};   /* most slots of an image, likewise */
    uint64_t layout_reads = 0;             /* see own_layout_pays */
    bool any_plain = false, chained = true;
    for (int i = 0; i < n; ++i) {
        const l3_encode_item& it = items[i];
        if (!it.d_rgb || !it.d_file || it.width == 0 || it.height == 0 ||
            it.row_stride < (size_t)it.width * 3)
            return L3_ERR_INVALID_ARG;
        const uint32_t np = it.patch ? it.patch : l3_default_patch(it.width, it.height);
        if (np > kMaxPatch) return L3_ERR_UNSUPPORTED;
        if (np > max_n) max_n = np;
        if (it.width > (1u << 24) || it.height > (1u << 24)) return L3_ERR_UNSUPPORTED;
        const uint64_t p = (uint64_t)((it.width + np - 1) / np) * ((it.height + np - 1) / np);
        if (3 * p > 0x7FFFFFFFull) return L3_ERR_UNSUPPORTED;
        total_patches += (size_t)(3 * p);
        if (3 * p > max_patches) max_patches = (uint32_t)(3 * p);
        if (np == 32 || np == 64 || np == 128) {
            const uint32_t cls = np == 32 ? 0 : np == 64 ? 1 : 2;
            const uint32_t tpw = 256 / np, tiles_x = (it.width + np - 1) / np;
            const uint64_t units = (uint64_t)((tiles_x + tpw - 1) / tpw) * ((it.height + np - 1) / np);
            if (units > strip_units[cls]) strip_units[cls] = (uint32_t)units;
            if (3 * p > strip_slots[cls]) strip_slots[cls] = (uint32_t)(3 * p);
            if (3 * p <= kOwnLayoutPatches) layout_reads += own_layout_reads(np, (uint32_t)(3 * p));
            slot_bytes += (size_t)(3 * p) * strip_slot_bytes(np);
            /* what l3_encode_bound gives: every row at 12 + 8 bits a pixel, a byte of padding a patch */
            const uint64_t bound = 13 + 12 * p + 3 * ((uint64_t)it.width * it.height + 2 * (uint64_t)it.height * tiles_x + p);
            chained &= it.file_cap >= bound;
        } else {
            any_plain = true;
        }
    }
    if (total_patches > 0xFFFFFFFFull) return L3_ERR_UNSUPPORTED;
    const bool own_layout = own_layout_pays(max_patches, layout_reads) && !any_plain;
    chained &= !any_plain && chained_pays(strip_units, (uint64_t)n, own_layout);

    if (!ctx->enc) {
        ctx->enc = new (std::nothrow) L3EncodeState;
        if (!ctx->enc) return L3_ERR_DEVICE;
        if (hipEventCreateWithFlags(&ctx->enc->done, hipEventDisableTiming) != hipSuccess) return L3_ERR_DEVICE;
    }
    L3EncodeState* st = ctx->enc;
    /* The workspace (size table, slots, descriptor table) is shared by consecutive calls.
     * On the device a call is ordered after the previous one; the host waits for the
     * previous call only before it frees or overwrites something that call still reads. */
    auto wait_previous = [&]() -> bool {
        if (st->pending && hipEventSynchronize(st->done) != hipSuccess) return false;
        st->pending = false;
        return true;
    };
    if (st->pending && stream != st->last_stream &&
        hipStreamWaitEvent(stream, st->done, 0) != hipSuccess)
        return L3_ERR_DEVICE;
    const bool by_args = n <= kArgDescs && !any_plain;
    constexpr int kStage = 4;
    int stage = 0;
    if (!by_args) {
        if ((size_t)n > st->desc_cap) {
            if (!wait_previous()) return L3_ERR_DEVICE;      /* its uploads and kernels read the old tables */
            size_t cap = 64;
            while (cap < (size_t)n) cap *= 2;
            if (st->h_descs) (void)hipHostFree(st->h_descs);
            if (st->d_descs) (void)hipFree(st->d_descs);
            st->h_descs = nullptr;
            st->d_descs = nullptr;
            st->desc_cap = 0;
            for (int i = 0; i < kStage; ++i) st->staged_pending[i] = false;
            if (hipHostMalloc(reinterpret_cast<void**>(&st->h_descs), kStage * cap * sizeof(L3EncodeDesc),
                              hipHostMallocDefault) != hipSuccess ||
                hipMalloc(reinterpret_cast<void**>(&st->d_descs), cap * sizeof(L3EncodeDesc)) != hipSuccess)
                return L3_ERR_DEVICE;
            st->desc_cap = cap;
        }
        /* the staging table about to be rewritten: its last upload must have left it */
        stage = st->next_stage;
        st->next_stage = (stage + 1) % kStage;
        if (!st->staged[stage] &&
            hipEventCreateWithFlags(&st->staged[stage], hipEventDisableTiming) != hipSuccess)
            return L3_ERR_DEVICE;
        if (st->staged_pending[stage] && hipEventSynchronize(st->staged[stage]) != hipSuccess)
            return L3_ERR_DEVICE;
        st->staged_pending[stage] = false;
    }
    /* The chained kernels count on words that earlier launches left in the workspace.  What a capturing
     * stream records runs later, or again, or never, and is not seen by `done`: such a call takes the
     * strip kernels, which find nothing in the workspace but what they wrote themselves.  (Their part of it is
     * sized by every call, so that a call that has been made once can be captured; the words are there from the first
     * call on, whatever it takes, so that later ones do not allocate.) */
    if (chained || !st->d_words) {
        hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
        const bool asked = hipStreamIsCapturing(stream, &capture) == hipSuccess;
        if (!asked) (void)hipGetLastError();
        const bool ordinary = asked && capture == hipStreamCaptureStatusNone;
        if (ordinary && !st->d_words &&
            hipMalloc(reinterpret_cast<void**>(&st->d_words),
                      kMostChainImages * sizeof(L3ChainWord) + kMostChainUnits * sizeof(uint64_t)) != hipSuccess) {
            (void)hipGetLastError();        /* the strip kernels do without */
            st->d_words = nullptr;
        }
        chained &= ordinary && st->d_words != nullptr;
        const uint32_t images = chained ? (uint32_t)n : 0u;
        if (ordinary && st->d_words &&
            (st->chain_number == 0 || st->chain_number + 3 > kLastNumber || images > st->chain_slots)) {
            while (st->chain_slots < images) st->chain_slots *= 2;
            st->chain_number = 0;                       /* until the clear is enqueued and all calls are behind it */
            hipLaunchKernelGGL(l3_encode_clear_kernel, dim3((kMostChainUnits + 255) / 256), dim3(256), 0, stream,
                               st->d_words, reinterpret_cast<uint64_t*>(st->d_words + kMostChainImages));
            if (hipGetLastError() != hipSuccess || hipEventRecord(st->done, stream) != hipSuccess) return L3_ERR_DEVICE;
            st->pending = true;
            st->last_stream = stream;
            st->chain_number = 1;
        }
    }
    if (total_patches > st->sizes_cap) {
        if (!wait_previous()) return L3_ERR_DEVICE;
        size_t cap = 4096;
        while (cap < total_patches) cap *= 2;
        if (st->d_sizes) (void)hipFree(st->d_sizes);
        st->d_sizes = nullptr;
        st->sizes_cap = 0;
        if (hipMalloc(reinterpret_cast<void**>(&st->d_sizes), cap * sizeof(uint32_t)) != hipSuccess)
            return L3_ERR_DEVICE;
        st->sizes_cap = cap;
    }
    if (slot_bytes > st->slots_cap) {
        if (!wait_previous()) return L3_ERR_DEVICE;
        if (st->d_slots) (void)hipFree(st->d_slots);
        st->d_slots = nullptr;
        st->slots_cap = 0;
        if (hipMalloc(reinterpret_cast<void**>(&st->d_slots), slot_bytes) != hipSuccess)
            return L3_ERR_DEVICE;
        st->slots_cap = slot_bytes;
    }

    EncodePack<kArgDescs> pack;              /* the first kArgDescsSmall of it are the smaller block */
    const EncodePack<kArgDescsSmall>& small_pack = reinterpret_cast<const EncodePack<kArgDescsSmall>&>(pack);
    const bool small = n <= kArgDescsSmall;
    L3EncodeDesc* const table = by_args ? pack.d : st->h_descs + (size_t)stage * st->desc_cap;
    size_t base = 0, slots_base = 0;
    for (int i = 0; i < n; ++i) {
        const l3_encode_item& it = items[i];
        L3EncodeDesc& d = table[i];
        const uint32_t np = it.patch ? it.patch : l3_default_patch(it.width, it.height);
        d.rgb = it.d_rgb;
        d.file = it.d_file;
        d.row_stride = it.row_stride;
        d.file_cap = it.file_cap;
        d.width = it.width;
        d.height = it.height;
        d.tiles_x = (it.width + np - 1) / np;
        d.tiles_y = (it.height + np - 1) / np;
        d.patch = np;
        d.sizes_base = (uint32_t)base;
        d.status_index = (uint32_t)i;
        d.strips_x = 0;
        d.slots_base = 0;
        if (np == 32 || np == 64 || np == 128) {
            const uint32_t tpw = 256 / np;
            d.strips_x = (d.tiles_x + tpw - 1) / tpw;
            d.slots_base = slots_base;
            slots_base += 3 * (size_t)d.tiles_x * d.tiles_y * strip_slot_bytes(np);
        }
        base += 3 * (size_t)d.tiles_x * d.tiles_y;
    }
    if (by_args) {
        const int block = small ? kArgDescsSmall : kArgDescs;
        std::memset(&pack.d[n], 0, (size_t)(block - n) * sizeof(L3EncodeDesc));
    } else {
        if (hipMemcpyAsync(st->d_descs, table, (size_t)n * sizeof(L3EncodeDesc), hipMemcpyHostToDevice,
                           stream) != hipSuccess ||
            hipEventRecord(st->staged[stage], stream) != hipSuccess)
            return L3_ERR_DEVICE;
        st->staged_pending[stage] = true;
    }
    if (chained) {
        uint64_t* const cells = reinterpret_cast<uint64_t*>(st->d_words + kMostChainImages);
        const auto encode = [&](auto n_tag, uint32_t strips) {
            constexpr int N = decltype(n_tag)::value;
            if (!strips) return;
            const uint32_t units = 3 * strips;
            const uint64_t number = ++st->chain_number;
            const dim3 grid(units * (uint32_t)n);
            if (by_args && small)
                hipLaunchKernelGGL((l3_encode_chain_kernel_args<N, kArgDescsSmall>), grid, dim3(UnitGeom<N>::THREADS), 0, stream,
                                   small_pack, units, st->d_words, cells, number, st->chain_slots, d_file_len, d_status);
            else if (by_args)
                hipLaunchKernelGGL((l3_encode_chain_kernel_args<N, kArgDescs>), grid, dim3(UnitGeom<N>::THREADS), 0, stream, pack,
                                   units, st->d_words, cells, number, st->chain_slots, d_file_len, d_status);
            else
                hipLaunchKernelGGL(l3_encode_chain_kernel<N>, grid, dim3(UnitGeom<N>::THREADS), 0, stream, st->d_descs,
                                   units, st->d_words, cells, number, st->chain_slots, d_file_len, d_status);
        };
        encode(std::integral_constant<int, 32>(), strip_units[0]);
        encode(std::integral_constant<int, 64>(), strip_units[1]);
        encode(std::integral_constant<int, 128>(), strip_units[2]);
    } else if (by_args) {
        const uint32_t m = (uint32_t)n;
        const auto launch = [&](const auto& descs, auto cap_tag) {
            constexpr int CAP = decltype(cap_tag)::value;
            if (strip_units[0])
                hipLaunchKernelGGL((l3_encode_strip_kernel_args<32, CAP>), dim3(strip_units[0], m), dim3(192), 0, stream,
                                   descs, st->d_sizes, st->d_slots);
            if (strip_units[1])
                hipLaunchKernelGGL((l3_encode_strip_kernel_args<64, CAP>), dim3(strip_units[1], m), dim3(192), 0, stream,
                                   descs, st->d_sizes, st->d_slots);
            if (strip_units[2])
                hipLaunchKernelGGL((l3_encode_strip_kernel_args<128, CAP>), dim3(strip_units[2], m), dim3(192), 0, stream,
                                   descs, st->d_sizes, st->d_slots);
            if (!own_layout)
                hipLaunchKernelGGL(l3_encode_layout_kernel_args<CAP>, dim3(m), dim3(256), 0, stream, descs, st->d_sizes,
                                   d_file_len, d_status);
            const auto compact = [&](auto n_tag, uint32_t most) {
                constexpr int N = decltype(n_tag)::value;
                const dim3 grid((most + CompactGeom<N>::SLOTS - 1) / CompactGeom<N>::SLOTS, m);
                if (most && own_layout)
                    hipLaunchKernelGGL((l3_encode_compact_kernel_args<N, true, CAP>), grid, dim3(256), 0, stream, descs,
                                       st->d_sizes, st->d_slots, d_file_len, d_status);
                else if (most)
                    hipLaunchKernelGGL((l3_encode_compact_kernel_args<N, false, CAP>), grid, dim3(256), 0, stream, descs,
                                       st->d_sizes, st->d_slots, d_file_len, d_status);
            };
            compact(std::integral_constant<int, 32>(), strip_slots[0]);
            compact(std::integral_constant<int, 64>(), strip_slots[1]);
            compact(std::integral_constant<int, 128>(), strip_slots[2]);
        };
        if (small) launch(small_pack, std::integral_constant<int, kArgDescsSmall>());
        else launch(pack, std::integral_constant<int, kArgDescs>());
    } else {
        const size_t lds_bytes = ((size_t)max_n * (12 + 8 * (size_t)max_n) + 31) / 32 * 4 + 8;
        for (int first = 0; first < n; first += 65535) {
            const uint32_t m = (uint32_t)(n - first < 65535 ? n - first : 65535);
            const L3EncodeDesc* dd = st->d_descs + first;
            if (strip_units[0])
                hipLaunchKernelGGL(l3_encode_strip_kernel<32>, dim3(strip_units[0], m), dim3(192), 0, stream,
                                   dd, st->d_sizes, st->d_slots);
            if (strip_units[1])
                hipLaunchKernelGGL(l3_encode_strip_kernel<64>, dim3(strip_units[1], m), dim3(192), 0, stream,
                                   dd, st->d_sizes, st->d_slots);
            if (strip_units[2])
                hipLaunchKernelGGL(l3_encode_strip_kernel<128>, dim3(strip_units[2], m), dim3(192), 0, stream,
                                   dd, st->d_sizes, st->d_slots);
            if (any_plain)
                hipLaunchKernelGGL(l3_encode_measure_kernel, dim3(max_patches, m), dim3(64), 0, stream, dd,
                                   st->d_sizes);
        }
        if (!own_layout)
            hipLaunchKernelGGL(l3_encode_layout_kernel, dim3((uint32_t)n), dim3(256), 0, stream, st->d_descs,
                               st->d_sizes, d_file_len, d_status);
        for (int first = 0; first < n; first += 65535) {
            const uint32_t m = (uint32_t)(n - first < 65535 ? n - first : 65535);
            const L3EncodeDesc* dd = st->d_descs + first;
            const auto compact = [&](auto n_tag, uint32_t most) {
                constexpr int N = decltype(n_tag)::value;
                const dim3 grid((most + CompactGeom<N>::SLOTS - 1) / CompactGeom<N>::SLOTS, m);
                if (most && own_layout)
                    hipLaunchKernelGGL((l3_encode_compact_kernel<N, true>), grid, dim3(256), 0, stream, dd,
                                       st->d_sizes, st->d_slots, d_file_len, d_status);
                else if (most)
                    hipLaunchKernelGGL((l3_encode_compact_kernel<N, false>), grid, dim3(256), 0, stream, dd,
                                       st->d_sizes, st->d_slots, d_file_len, d_status);
            };
            compact(std::integral_constant<int, 32>(), strip_slots[0]);
            compact(std::integral_constant<int, 64>(), strip_slots[1]);
            compact(std::integral_constant<int, 128>(), strip_slots[2]);
            if (any_plain)
                hipLaunchKernelGGL(l3_encode_pack_kernel, dim3(max_patches, m), dim3(64), lds_bytes, stream,
                                   dd, st->d_sizes, d_file_len);
        }
    }
    if (hipGetLastError() != hipSuccess || hipEventRecord(st->done, stream) != hipSuccess) {
        st->chain_number = 0;       /* which launches ran is not known: the words are cleared again */
        return L3_ERR_DEVICE;
    }
    st->pending = true;
    st->last_stream = stream;
    return L3_OK;
}
