// Launch shape and work arrangement of the gather kernels (forward and bwd_kernel): which workgroup
// takes which heads and queries. Host code without a GPU call; the kernels' side of it is
// block_work and strip_pixel in msda_internal.h.
#include "msda_internal.h"

namespace msda {

namespace {

// The arrangement of block_work. Query eighths when there are at least half as many queries as value
// pixels (self-attention over the maps: a query's reference point follows the query order, so an
// eighth of the queries reads a band of every level, and an XCD's L2 holds the bands of several
// slabs at once). Slab ranges otherwise (cross-attention: a query samples anywhere in its slab, so
// the working set is the slab, and fewer slabs per L2 is better). Measured with both arrangements:
// the forward 6 % faster at the DETR-encoder shape, 5-16 % at the Swin shape and 10-22 % at the
// BEV-temporal shape with eighths; 4 % (BEV-spatial) and 40 % (DETR-decoder) slower with them.
bool xcd_split(const Params& p) {
#if defined(MSDA_ABLATE_SLAB_RANGES) || defined(MSDA_ABLATE_NO_XCD_REMAP) || defined(MSDA_ABLATE_HEAD_FASTEST)
    (void)p;
    return false;
#elif defined(MSDA_ABLATE_QUERY_EIGHTHS)
    (void)p;
    return true;
#else
    return 2 * (int64_t)p.Lq >= p.S;
#endif
}

// Whether the query eighths follow the rows of the maps instead of the query index: for
// self-attention over the maps (as many queries as value pixels, query q at pixel q in level-major
// order). With eighths of the query index, the XCDs that hold the coarse levels' queries read every
// level over the whole map; with bands of rows every XCD reads one band of each level. Same-box A/B:
// Swin-feature shape forward 256 -> 238 us, backward 841 -> 820 us; DETR-encoder and one-level
// BEV shapes within 1 %. If the queries are in another order only the speed changes.
bool xcd_bands(const Params& p) {
#ifdef MSDA_ABLATE_INDEX_EIGHTHS
    (void)p;
    return false;
#else
    return p.Lq == p.S;
#endif
}

}  // namespace

// The chunk ranges of the band arrangement: row h of level l is in band floor(8 (h + 1/2) / H_l), and a query
// chunk goes with the band of its first query.
void set_bands(Params& p) {
    const int64_t qpb = p.q_per_block;
    auto first_chunk = [&](int64_t q) { return (int)((q + qpb - 1) / qpb); };
    for (int l = 0; l < kMaxLevels; ++l)
        for (int x = 0; x <= 8; ++x) p.band_c[l][x] = 0;
    for (int l = 0; l < p.L; ++l) {
        const int64_t H = p.H[l], W = p.W[l], s = p.start[l];
        for (int x = 0; x < 8; ++x) {
            // first row whose band is at least x: 8 h + 4 >= x H
            int64_t r0 = (x * H - 4 + 7) / 8;
            if (x * H - 4 <= 0) r0 = 0;
            p.band_c[l][x] = first_chunk(s + r0 * W);
        }
        p.band_c[l][8] = first_chunk(s + H * W);
    }
    p.band_cap = 0;
    for (int x = 0; x < 8; ++x) {
        int n = 0;
        for (int l = 0; l < p.L; ++l) n += p.band_c[l][x + 1] - p.band_c[l][x];
        p.band_count[x] = n;
        if (n > p.band_cap) p.band_cap = n;
    }
}

GatherLaunch plan_gather(Params& p, int ppw, int elem_bytes) {
    const int64_t chunks4 = (p.Lq + kWaves * ppw - 1) / (kWaves * ppw);
    const int waves = (int64_t)p.n_batch * p.M * chunks4 < kSmallGrid ? 1 : kWaves;
    // Strips of rows where the queries are the pixels (as many queries as pixels; if they are in
    // another order only the speed changes), and two heads per workgroup where two heads' rows of
    // one pixel are one 128-byte cache line. Forward / backward us before and after, same box:
    // Swin-feature shape fp16 188 / 853 -> 151 / 811, BEV-temporal fp16 207 / 792 -> 186 / 751,
    // DETR-encoder fp32 91 / 300 -> 89 / 293 (its 128-byte rows hit the cache more often, and its
    // loads run at 0.7 of the cache's rate). Strips of 16 rows were 2-5 % slower, of 4 rows 1-15 %
    // in the backward; workgroups of 8 or 16 waves were slower. Not for rows longer than a line, which gain as
    // much as the order costs (fp32 forward us with strips and without: 40 channels, 6 samples 85.6 / 82.6; 48
    // channels, 16 samples 29.9 / 28.9; 64 channels, 24 samples 34.2 / 33.6), nor for queries of fewer samples (48 channels,
    // 1 sample 59.2 / 54.5; 32 channels, 2 samples 22.9 / 21.9; fp16, 32 channels, 1 sample 13.4 / 12.5), against
    // fp16 of 16 channels, 4 samples 103.1 / 122.7 and 32 channels, 8 samples 48.0 / 52.8.
    p.strips = waves > 1 && p.Lq == p.S && p.S < kStripMaxPixels && p.D * elem_bytes <= kStripMaxRowBytes &&
               p.K >= kStripMinSamples;
    for (int l = 0; l < p.L; ++l)
        if (p.H[l] > kStripMaxRows) p.strips = 0;
    p.head_group = waves > 1 && p.M % 2 == 0 && p.D * elem_bytes == 64 ? 2 : 1;
    p.groups = p.M / p.head_group;
    p.n_groups = p.n_batch * p.groups;
    p.head_waves = waves / p.head_group;
    p.q_per_block = p.head_waves * ppw;
    const int qchunks = (p.Lq + p.q_per_block - 1) / p.q_per_block;
    // a grid too small to fill the chip splits each query's samples over up to k_split_max
    // work items, as long as a part keeps kSplitMinSamples samples
    int ks = 1;
    while (2 * ks <= p.k_split_max && 2 * ks * kSplitMinSamples <= p.K &&
           (int64_t)p.n_batch * p.M * qchunks * p.head_waves * 2 * ks <= kSplitWaves)
        ks *= 2;
    p.k_split = ks;
    p.chunks = qchunks * ks;
    p.num_blocks = p.n_groups * p.chunks;
    if (p.num_blocks == 0) return {0, waves};
    const int64_t split_grid = 8 * (int64_t)p.n_groups * ((p.chunks + 7) / 8);
    p.xcd_split = xcd_split(p) && split_grid <= INT32_MAX;
    p.xcd_bands = 0;
    int64_t band_grid = 0;
    if (p.xcd_split && ks == 1 && xcd_bands(p)) {
        set_bands(p);
        band_grid = 8 * (int64_t)p.n_groups * p.band_cap;
        p.xcd_bands = band_grid <= INT32_MAX;
    }
    return {p.xcd_bands ? (int)band_grid : p.xcd_split ? (int)split_grid : (p.num_blocks + 7) / 8 * 8, waves};
}

}  // namespace msda
