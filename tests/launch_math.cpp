// Host checks of the launch arithmetic that kernels and host code share (csrc/msda_internal.h), by
// brute force: prints "failures: 0" when every check holds.
#include <cstdio>
#include <initializer_list>
#include <vector>

#include "msda_internal.h"

int main() {
    int failures = 0;
    // strip_pixel is a permutation of a level's pixels that keeps every eighth of the rows (the band that one XCD
    // takes, as set_bands cuts the levels) in its own places, and that runs over an eighth in strips of at most
    // kStripRows rows, column by column
    for (int H : {1, 2, 7, 8, 9, 13, 15, 16, 23, 25, 38, 50, 100, 151, 1000})
        for (int W : {1, 2, 5, 8, 33, 1048}) {
            if ((int64_t)H * W >= msda::kStripMaxPixels) continue;
            std::vector<int> seen(H * W, 0);
            bool ok = true;
            int prev = -1;  // the pixel before
            for (int r = 0; r < H * W; ++r) {
                const int px = msda::strip_pixel(r, H, W);
                ok = ok && px >= 0 && px < H * W && ++seen[px] == 1;
                auto band = [&](int row) { return (8 * row + 4) / H; };
                ok = ok && band(px / W) == band(r / W);
                if (prev >= 0) {  // one row down, or to the strip's top row one column on, or to a new strip's first column
                    const int dr = px / W - prev / W, dc = px % W - prev % W;
                    const bool down = dr == 1 && dc == 0, on = dc == 1 && dr <= 0 && -dr < msda::kStripRows;
                    ok = ok && (down || on || px % W == 0);
                }
                prev = px;
            }
            if (!ok) {
                ++failures;
                std::printf("strip_pixel %d x %d\n", H, W);
            }
        }
    // small_div over its range, with the reciprocal off by up to two units in the last place
    for (int d : {1, 2, 3, 4, 5, 6, 7, 9, 12, 16, 31, 127, 128, 1000, 4097, 65535, 1048575})
        for (int ulps = -2; ulps <= 2; ++ulps) {
            const float inv = (1.f / (float)d) * (1.f + (float)ulps * 5.9604645e-8f);
            for (int j = 0; j < (1 << 20); j += d < 64 ? 1 : 7)
                for (int e : {j, j / d * d, j / d * d + d - 1}) {
                    if (e >= (1 << 20)) continue;
                    if (msda::small_div(e, inv) != e / d) {
                        if (failures++ < 10) std::printf("small_div %d / %d\n", e, d);
                    }
                }
        }
    // the fold's rows and channels that are not there: past grad_out's end as 32-bit byte offsets, alone and together
    // and at the second 16 bytes of a lane, up to the largest problem that the binned path takes
    for (int64_t elems : {int64_t(4), int64_t(96), int64_t(1) << 20, (int64_t(1) << 28) + 36, msda::kMaxLaunchElems - 4}) {
        msda::Params p = {};
        p.n_batch = p.Lq = p.M = 1;
        p.D = (int)elems;
        const int64_t nothing = msda::fold_nothing(p);
        for (int64_t row : {int64_t(0), elems - 4, nothing})
            for (int64_t ch : {int64_t(0), int64_t(28), nothing})
                for (int64_t more : {0, 4}) {
                    if (row != nothing && ch != nothing) continue;
                    for (int bytes : {2, 4}) {
                        const uint32_t at = (uint32_t)(row + ch) * (uint32_t)bytes + (uint32_t)(more * bytes);
                        if ((int64_t)at < elems * bytes) {
                            ++failures;
                            std::printf("fold marker: %lld elements, row %lld + channel %lld + %lld\n", (long long)elems,
                                        (long long)row, (long long)ch, (long long)more);
                        }
                    }
                }
    }
    std::printf("failures: %d\n", failures);
    return failures != 0;
}
