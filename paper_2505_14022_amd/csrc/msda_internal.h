// Internal interface between the C ABI (msda_api.cpp) and the HIP kernels (msda_*.hip).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "msda.h"

// Ablation builds (never the product library): each MSDA_ABLATE_* macro, set on the compiler
// command line by microbench/ablation.py, replaces one design choice with a complete, correct
// alternative, so that the choice can be timed and counted against the product build.
// The query order (strips) and the head pairs are those of the product in all of them but LDS_STAGE, whose
// forward takes one head and the query index where a level is staged.
//   MSDA_ABLATE_NO_XCD_REMAP    workgroup b runs work item b on every shape (no XCD-aware arrangement)
//   MSDA_ABLATE_HEAD_FASTEST    work items in (batch, query chunk, head) order instead of slab-major
//                               (slab ranges on every shape)
//   MSDA_ABLATE_SLAB_RANGES     slab ranges per XCD on every shape (no query eighths)
//   MSDA_ABLATE_QUERY_EIGHTHS   query eighths per XCD on every shape
//   MSDA_ABLATE_INDEX_EIGHTHS   query eighths by query index also where there are as many queries as
//                               value pixels (no bands of rows)
//   MSDA_ABLATE_NO_KSPLIT       small backward grids keep each query chunk's samples in one workgroup
//   MSDA_ABLATE_VEC1            one channel per lane (D lanes per query) instead of 16-byte pieces
//   MSDA_ABLATE_NO_DPP          lane-group sums and maxima by ds_bpermute shuffles instead of DPP
//   MSDA_ABLATE_PLAIN_STORES    outputs written with ordinary stores instead of nontemporal ones
//   MSDA_ABLATE_ONE_STREAM      the owner-computes backward on the caller's stream alone
//   MSDA_ABLATE_FOLD_ONE_QUEUE  one work-queue counter for the fold instead of one per XCD
//   MSDA_ABLATE_LDS_STAGE       the forward stages the largest level that fits 32 KB in LDS

namespace msda {

constexpr int kMaxLevels = MSDA_MAX_LEVELS;

// Largest per-launch tensor, in elements. Element offsets of value / grad_value rows are kept in
// 32 bits, and kOOBElem (= this limit) marks a corner that lies off the map: scaled to bytes it
// is past the end of every buffer resource, so the hardware returns zero for the load and drops
// the atomic.
constexpr int64_t kMaxLaunchElems = int64_t(1) << 29;
constexpr int64_t kMaxIndex = (int64_t(1) << 31) - 1;

// Waves of a workgroup of the gather kernels, or one where that many workgroups would leave CUs idle: a
// wave's work does not depend on the other waves of its workgroup, and at the DETR-decoder shape
// (160 four-wave workgroups) one-wave workgroups spread the grad_value atomics over all CUs.
constexpr int kWaves = 4;
constexpr int kSmallGrid = 1024;
#ifndef MSDA_KSPLIT_WAVES
#define MSDA_KSPLIT_WAVES 4096
#endif
constexpr int64_t kSplitWaves = MSDA_KSPLIT_WAVES;  // waves a sample split may grow the grid to
#ifndef MSDA_KSPLIT_MIN
#define MSDA_KSPLIT_MIN 4
#endif
constexpr int kSplitMinSamples = MSDA_KSPLIT_MIN;

// Owner-computes grad_value: limits of the binned path.
constexpr int kHistMax = 15872;      // bins of one (n, m) slab counted in LDS (62 KB)
constexpr int kTileFloats = 3200;    // LDS floats of one tile accumulator with its margin (12.5 KB per wave)
constexpr int kBinnedMaxD = 355;     // channels per head handled by the binned path (1x1 tiles)
constexpr int kChunkRecords = 512;   // records folded by one accumulate work item
// Threads per workgroup of the counting / scatter passes (512 or 1024, with four times the samples
// per workgroup and so fewer bin atomics, made the backward 3-14 % slower), and their samples.
constexpr int kBinBlock = 256;
constexpr int kCountQueries = 16 * kBinBlock;
constexpr int kStripRows = 8;        // rows of a strip of the gather kernels' query order
constexpr int64_t kStripMaxPixels = int64_t(1) << 20;  // maps of this many pixels, or of more than
constexpr int kStripMaxRows = 1 << 17;                 // this many rows, keep the index order (small_div)
constexpr int kStripMaxRowBytes = 128;  // as do calls of longer value rows,
constexpr int kStripMinSamples = 4;     // or of fewer samples per query and head
constexpr int kScanTiles = 256;      // tiles per workgroup in the scan passes (one per thread)
constexpr int kAtomicMaxSamples = 16384;  // problems this small take the atomic grad_value path
// Bytes of the static device scratch of msda_backward_noalloc (per GPU, held until the process ends).
constexpr size_t kStaticScratchBytes = size_t(128) << 20;

// j / d for 0 <= j < 2^20 and 1 <= d, given inv = 1 / d within an ulp or two: the distance of
// (j + 1/2) / d to the next integer, at least 1 / (2 d), is more than the rounding errors move it.
// (An integer division by a number known only at run time takes about twenty instructions.)
__host__ __device__ inline int small_div(int j, float inv) { return (int)(((float)j + 0.5f) * inv); }

// 1 / x, within an ulp on the GPU.
__host__ __device__ inline float fast_rcp(float x) {
#ifdef __HIP_DEVICE_COMPILE__
    return __builtin_amdgcn_rcpf(x);
#else
    return 1.f / x;
#endif
}

// Pixel (row-major) at place r of a level's query order, for levels of less than 2^20 pixels and at most 2^17 rows. The
// order runs over each eighth of the rows (the band that one XCD takes, row h in band floor(8 (h + 1/2) / H))
// in strips of rows, as few of equal height as leave at most kStripRows rows a strip, and column by column within
// a strip. Cutting the strips at the bands keeps an XCD's queries in its rows: with strips of 8 rows across the
// bands, 79, 56, 39 and 23 % of the queries of the four DETR levels were in their XCD's band (99, 97, 86 and
// 47 % in index order), and the DETR-encoder forward moved 203 MB and bwd_kernel 271; 186 and 253 so, with the
// same requests to L2.
__host__ __device__ inline int strip_pixel(int r, int H, int W) {
    const int h = small_div(r, fast_rcp((float)W));               // the row that place r has in row-major order,
    const int x = small_div(8 * h + 4, fast_rcp((float)H));       // and the band, whose rows have the same places
    const int r0 = (x * H + 3) >> 3, n = (((x + 1) * H + 3) >> 3) - r0;
    const int strips = (n + kStripRows - 1) / kStripRows, high = small_div(n + strips - 1, fast_rcp((float)strips));
    const int top = small_div(h - r0, fast_rcp((float)high)) * high;  // of the strip, within the band
    const int rows = n - top < high ? n - top : high, rem = r - (r0 + top) * W;
    const int col = small_div(rem, fast_rcp((float)rows));
    return (r0 + top + rem - col * rows) * W + col;
}

// Everything one launch needs, passed by value as the kernel argument.
struct Params {
    const void* value;     // [n_batch, S, M, D] dtype (already offset to the first batch item)
    const float* loc;      // [n_batch, Lq, M, L, P, 2]
    const float* attn;     // [n_batch, Lq, M, L, P]
    const float* ref;      // [n_batch, Lq, L, 2]          (fused entry points)
    const float* pix_offsets;  // [n_batch, Lq, M, L, P, 2] (fused entry points, pixels)
    const float* logits;   // [n_batch, Lq, M, L*P]        (fused entry points)
    void* out;             // [n_batch, Lq, M*D] dtype                       (forward)
    const void* grad_out;  // [n_batch, Lq, M*D] dtype                       (backward)
    float* grad_value;     // [n_batch, S, M, D] fp32                        (backward)
    float* grad_loc;       // [n_batch, Lq, M, L, P, 2]                      (backward)
    float* grad_attn;      // [n_batch, Lq, M, L, P]                         (backward)
    int* reset;            // backward: a counter that bwd_kernel zeroes for the kernels after it (or null)
    int prologue_grads;    // backward: grad_loc / grad_attn hold grad_offsets / grad_logits instead
    int stream_grads;      // backward: grad_loc / grad_attn are read by no later kernel of the call
    uint32_t value_bytes;  // size of the value buffer resource
    uint32_t gv_bytes;     // size of the grad_value buffer resource
    int n_batch, S, M, D, Lq, L, P, K;  // K = L*P samples per (query, head)
    float inv_P;           // 1 / P
    int q_per_block;       // queries of one (n, m) handled by one workgroup
    int chunks;            // work items per slab: ceil(Lq / q_per_block) * k_split
    int strips;            // query order of the gather kernels: strips of rows (strip_pixel) or the query index
    int head_group;        // heads that one workgroup of the gather kernels takes together (divides M)
    int groups;            // M / head_group
    int n_groups;          // n_batch * groups: slab groups
    int head_waves;        // waves of a workgroup per head (head_group * head_waves waves in all)
    int k_split;           // bwd_kernel: a query chunk's samples are split over k_split work items
    int k_split_max;       // set by the launcher: the largest k_split it accepts (0 or 1: none)
    int xcd_split;         // forward / bwd_kernel work arrangement (tile_of): 1 query eighths, 0 slab ranges
    int xcd_bands;         // with xcd_split: the eighths are bands of rows: XCD x takes the query chunks
                           // whose first query lies in the x-th eighth of the rows of its level
    int band_cap;          // with xcd_bands: work slots per slab and XCD
    int band_count[8];     // with xcd_bands: query chunks of one slab that XCD x takes
    int band_c[kMaxLevels][9];  // with xcd_bands: XCD x's chunks of level l are [band_c[l][x], band_c[l][x+1])
    int num_blocks;        // n_batch * M * chunks (the launch grid may be larger: see tile_of)
    int H[kMaxLevels], W[kMaxLevels], start[kMaxLevels];
    int stage_level;       // forward, MSDA_ABLATE_LDS_STAGE only: level staged in LDS (-1: none)
    int stage_chunks;      // forward, MSDA_ABLATE_LDS_STAGE only: query chunks per workgroup

    // ---- binned grad_value (owner-computes); filled by plan_binned() ----
    int tile_lh[kMaxLevels];    // log2 of the tile height at level l
    int tile_lw[kMaxLevels];    // log2 of the tile width at level l
    int tiles_x[kMaxLevels];    // tiles per tile-row at level l
    int tile_base[kMaxLevels];  // first tile of level l within a slab
    int tile_bins[kMaxLevels];  // bins per tile at level l (4, or 11 with the interior class split by row)
    int bin_base[kMaxLevels];   // first bin of level l within a slab
    int tiles_per_slab;
    int bins_per_slab;
    int n_bins;                 // n_slabs * bins_per_slab
    int n_slabs;                // n_batch * M
    int n_tiles;                // n_slabs * tiles_per_slab
    int n_samples;              // n_batch * Lq * M * K
    int one_launch;             // the whole batch is in this launch
    int slab_bins;              // binning in one launch, a workgroup per (slab, level)
    int item_records;           // with slab_bins: visible records of a tile per work item (kChunkRecords else)
    int ch_blocks;              // with slab_bins: work items per descriptor, blocks of 32 channels (0: one, of all)
    int max_items;              // capacity of `items`
    int scan_blocks;            // ceil(n_tiles / kScanTiles)
    int deterministic;          // grad_value summed in an order fixed by the inputs (bitwise reproducible)
    int* counts;                // [n_bins]            samples per bin (tile, class)
    int* queue;                 // [8 * 64]            fold work queue counters, 256 B apart (zeroed with counts)
    int* scan_done;             // [1]                 workgroups of the scan's first pass done, or with slab_bins
                                //                     the number of work items (zeroed with counts)
    int* item_desc;             // [max_items * 16]    fold work item descriptors (slab_bins: [n_tiles * 16], of tiles)
    int* offsets;               // [n_bins + 1]        exclusive prefix of counts
    int* cursor;                // [n_bins]            fill position per bin
    int* tile_chunks;           // [n_tiles + 1]       exclusive prefix of work items per tile
    int* items;                 // [max_items]         work item -> tile (slab_bins: tile and chunk of its records)
    int* block_sums;            // [2 * scan_blocks]
    int* records;               // [n_samples][4]      {grad_out row, a, h_im, w_im} per sample, sorted by bin
    int* chunk_hist;            // [n_slabs * chunks][bins_per_slab] (deterministic) records per counting
                                //                     workgroup and bin, then their prefix over workgroups
    float* partials;            // [max_items][64][D]  (deterministic) sums of the work items of split tiles
};

// Workgroup -> (slab group, query chunk); false: no work. A slab group is p.head_group heads of a batch item, in
// (batch, head) order. Workgroup b of G runs on XCD b % 8 (the dispatcher deals workgroups
// to the eight XCDs in turn); with i = b / 8, XCD x takes its work in one of two arrangements:
//  * query eighths (p.xcd_split): the x-th eighth of every slab group's query chunks, group after group. The
//    grid is 8 * groups * ceil(chunks / 8); a workgroup past the end of its eighth exits. With
//    p.xcd_bands the eighths are bands of rows instead: XCD x takes the chunks whose first query lies
//    in the x-th eighth of the rows of its level (at most p.band_cap per group; the grid is
//    8 * groups * band_cap and a workgroup past the end of its band exits).
//  * slab ranges: the contiguous range [x*G/8, (x+1)*G/8) of the work items in slab-major order, so
//    that each slab's rows are read through one XCD's L2. The grid is a multiple of 8.
__host__ __device__ inline bool block_work(const Params& p, uint32_t b, uint32_t G, int& slab, int& chunk) {
    if (p.xcd_bands) {
        const int x = (int)(b & 7u), i = (int)(b >> 3);
        slab = i / p.band_cap;
        int k = i - slab * p.band_cap;
        if (slab >= p.n_groups || k >= p.band_count[x]) return false;
        chunk = -1;
        for (int l = 0; l < p.L; ++l) {
            const int c0 = p.band_c[l][x], n = p.band_c[l][x + 1] - c0;
            if (k < n) {
                chunk = c0 + k;
                break;
            }
            k -= n;
        }
        return chunk >= 0;
    }
    if (p.xcd_split) {
        const int x = (int)(b & 7u), i = (int)(b >> 3);
        const int per = (p.chunks + 7) >> 3;
        slab = i / per;
        chunk = (int)(((int64_t)x * p.chunks) >> 3) + (i - slab * per);
        return slab < p.n_groups && chunk < (int)(((int64_t)(x + 1) * p.chunks) >> 3);
    }
#ifndef MSDA_ABLATE_NO_XCD_REMAP
    const uint32_t w = (b & 7u) * (G >> 3) + (b >> 3);
#else
    const uint32_t w = b;
    (void)G;
#endif
    if (w >= (uint32_t)p.num_blocks) return false;
#ifndef MSDA_ABLATE_HEAD_FASTEST
    slab = (int)(w / (uint32_t)p.chunks);
    chunk = (int)(w - (uint32_t)slab * (uint32_t)p.chunks);
#else
    // work items ordered (batch, query chunk, head group): the heads of one chunk are consecutive
    const int nc = (int)(w / (uint32_t)p.groups);
    const int n = nc / p.chunks;
    chunk = nc - n * p.chunks;
    slab = n * p.groups + (int)(w - (uint32_t)nc * (uint32_t)p.groups);
#endif
    return true;
}

// Element offset that stands, in the fold, for a grad_out row that is not there and for channels past D: grad_out's
// number of elements. A row and a channel of which one or both are this lie past grad_out's end, and below
// 2^30 elements, so that their byte offset in 32 bits does not wrap round to its start.
__host__ __device__ inline int fold_nothing(const Params& p) { return p.n_batch * p.Lq * p.M * p.D; }

struct Tile {
    int n, m, q0;  // slab (n, m) and the first query (place in the query order) of this wave
    int part;      // which of the p.k_split parts of the queries' samples this workgroup takes
};

// The work of wave `wave` of a workgroup that takes `chunk` of `slab`. The heads of one slab group share cache
// lines, so the waves of a workgroup take the same queries of all of them.
__host__ __device__ inline Tile wave_work(const Params& p, int ppw, int slab, int chunk, int wave) {
    const int hg = wave >= p.head_waves ? 1 : 0;  // head_group is 1 or 2
    Tile t;
    t.n = slab / p.groups;
    t.m = (slab - t.n * p.groups) * p.head_group + hg;
    t.part = 0;
    if (p.k_split > 1) {
        // the parts of one query chunk are consecutive work items
        t.part = chunk % p.k_split;
        chunk /= p.k_split;
    }
    t.q0 = chunk * p.q_per_block + (wave - hg * p.head_waves) * ppw;
    return t;
}

// Launch shape of a gather kernel of `ppw` queries per wave: fills the arrangement fields of `p` for its
// n_batch and k_split_max (host code).
struct GatherLaunch {
    int grid;   // workgroups (0: nothing to do)
    int waves;  // waves per workgroup
};
GatherLaunch plan_gather(Params& p, int ppw, int elem_bytes);

// The chunk ranges of the band arrangement (p.xcd_bands) for p.q_per_block queries per chunk: fills
// p.band_c, p.band_count and p.band_cap from the level table (host code).
void set_bands(Params& p);

hipError_t launch_forward(const Params& p, msda_dtype_t dtype, hipStream_t stream);
// The forward with locations and weights computed from ref / offsets / logits.
hipError_t launch_forward_fused(const Params& p, msda_dtype_t dtype, hipStream_t stream);
// loc and attn of every sample from ref / offsets / logits (the backward's prologue).
hipError_t launch_prologue(const Params& p, float* loc, float* attn, hipStream_t stream);
// grad_offsets, grad_logits and (if non-null) grad_ref from the sampling's grad_loc / grad_attn.
hipError_t launch_prologue_grad(const Params& p, const float* attn, const float* grad_loc,
                                const float* grad_attn, float* grad_offsets, float* grad_logits,
                                float* grad_ref, hipStream_t stream);
// grad_loc / grad_attn; with `atomic_grad_value` the same kernel also scatters grad_value with
// fp32 atomics (grad_value must be zero beforehand). With p.prologue_grads set, the kernel writes the
// prologue's gradients instead (grad_offsets into p.grad_loc, grad_logits into p.grad_attn); that
// needs prologue_grads_in_kernel(p, dtype).
hipError_t launch_backward_grads(const Params& p, msda_dtype_t dtype, bool atomic_grad_value, hipStream_t stream);
// True when the backward kernel holds all L*P samples of a (query, head) at once, so that it can
// form the softmax chain rule of the fused entry points itself.
bool prologue_grads_in_kernel(const Params& p, msda_dtype_t dtype);
// grad_ref from grad_offsets (grad_loc = grad_offsets * (W_l, H_l), summed over heads and points).
hipError_t launch_ref_grad_from_offsets(const Params& p, const float* grad_offsets, float* grad_ref,
                                        hipStream_t stream);
// Zeroes the counters at the head of the binned path's workspace; enqueued before
// launch_backward_value_binned (on its stream or on one that it waits for).
hipError_t launch_binned_reset(const Params& p, hipStream_t stream);
// grad_value by binning samples per destination tile and accumulating each tile once.
hipError_t launch_backward_value_binned(const Params& p, msda_dtype_t dtype, hipStream_t stream);
hipError_t launch_zero(float* ptr, int64_t n, hipStream_t stream);

// Compute units of the device `stream` belongs to (the current device for the null stream),
// cached per device; -1 on error.
int device_cu_count(hipStream_t stream);

// Device address of the static scratch array (kStaticScratchBytes) on `device`, looked up on the
// first call for that device; no allocation.
hipError_t static_scratch(int device, void** ptr);

// True for the sparse or small problems that msda_backward runs on fp32 atomics when it has no workspace.
bool atomics_suffice(const Params& p);
// True when fp32 atomics are expected to beat the binned grad_value path: not beyond atomics_suffice.
bool prefer_atomic(const Params& p);
// Chooses tile sizes for the binned grad_value path and fills the geometry fields of `p`.
// Returns false if the path does not apply (then grad_value uses atomics).
bool plan_binned(Params& p);
// Workspace bytes of the binned path for the geometry in `p` (after plan_binned).
size_t binned_workspace_bytes(const Params& p);
// Points the workspace fields of `p` into `ws`.
void bind_workspace(Params& p, void* ws);

}  // namespace msda
