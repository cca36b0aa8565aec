/*
 * The kernels' predictor on packed 16-bit floats (predict_pairs_biased) against the definition
 * (arxiv 2208.08711 Section 4.2: the nearest of top-left, top-right, top to TL + TR - T, ties in
 * that order; the first and last column predict T), every TL, TR and T from 0 to 255.
 * usage: predictor <first T> <end T>.  Test infrastructure.
 */
#include <hip/hip_runtime.h>

#include "l3_gfx950.h"
#include "../../../paper_2208_08711_amd/csrc/l3_kernel_parts.h"

#include <cstdio>
#include <cstdlib>

static int nearest(int tl, int tr, int t) {
    const int p = tl + tr - t;
    int best = tl;
    if (std::abs(tr - p) < std::abs(best - p)) best = tr;
    if (std::abs(t - p) < std::abs(best - p)) best = t;
    return best;
}

int main(int argc, char** argv) {
    if (argc != 3) return 2;
    const uint32_t pw = 9;
    uint32_t inner_least, inner_most, first_least, first_most, last_least, last_most;
    predict_limits(1, pw, inner_least, inner_most);        /* columns 1 and 3 of 9 */
    predict_limits(0, pw, first_least, first_most);        /* columns 0 and 2 */
    predict_limits(6, pw, last_least, last_most);          /* columns 6 and 8 */
    for (int t = std::atoi(argv[1]); t < std::atoi(argv[2]); ++t)
        for (int tl = 0; tl < 256; ++tl)
            for (int tr = 0; tr < 256; ++tr) {
                const uint32_t u = 255u - (uint32_t)t;     /* the upper fields: neighbours exchanged, another T */
                /* register 2: the outer neighbours of columns 0 and 8 are the 0 of a wave's end in
                 * one field and another patch's pixel in the other */
                const uint32_t both_l = kPixelBias | (uint32_t)tl | ((uint32_t)tr << 16);
                const uint32_t both_r = kPixelBias | (uint32_t)tr | ((uint32_t)tl << 16);
                const uint32_t both_t = kPixelBias | (uint32_t)t | (u << 16);
                const uint32_t TL[3] = {both_l, both_l & 0xFFFF0000u, both_l}, TR[3] = {both_r, both_r, both_r & 0x0000FFFFu};
                const uint32_t T[3] = {both_t, both_t, both_t};
                const uint32_t least[3] = {inner_least, first_least, last_least}, most[3] = {inner_most, first_most, last_most};
                uint32_t pred[3];
                predict_pairs_biased<3>(TL, TR, T, least, most, pred);
                const uint32_t lower = (uint32_t)nearest(tl, tr, t), upper = (uint32_t)nearest(tr, tl, (int)u);
                const uint32_t want[3] = {kPixelBias | lower | (upper << 16), kPixelBias | (uint32_t)t | (upper << 16),
                                          kPixelBias | lower | (u << 16)};
                for (int j = 0; j < 3; ++j)
                    if (pred[j] != want[j]) {
                        std::printf("register %d: TL %d TR %d T %d: %08x, expected %08x\n", j, tl, tr, t, pred[j], want[j]);
                        return 1;
                    }
            }
    std::printf("ok\n");
    return 0;
}
