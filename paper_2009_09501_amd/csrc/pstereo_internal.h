// Internal interface between the C ABI layer and the gfx950 kernels.
#pragma once

#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "pstereo.h"

namespace pstereo {

// Everything one frame's kernels need, passed by value as a kernel argument.
struct FrameDesc {
    const uint8_t* frame;    // RGB24 [h][w][3]
    uint8_t* out_l;          // RGB24 outputs, any may be null
    uint8_t* out_r;
    uint8_t* out_a;
    const uint8_t* depth_in; // external depth map (u8 [h][w]) or null
    uint8_t* out_df;         // optional filtered-depth dump
    uint8_t* out_d0;         // optional raw-depth dump
    uint8_t* out_h;          // optional half side-by-side frame, RGB24 [h][w][3]
    uint32_t* stats;         // per block: mean R | G << 8 | B << 16 | edge << 24
    uint2* binfo;            // per block: {stats, region depth}
    int32_t* labels;         // per block: region label
    uint8_t* df;             // filtered depth scratch, u8 [h][w] (4-byte aligned)
    // strip-parallel region grouping (rstrip > 0): strip-local components are
    // merged across strip boundaries through a list of slots; binfo then
    // holds {statistics, slot of the block's component}
    uint32_t* rlist;         // per slot: the strip's entry, then final label << 9 | background << 8 | depth
    uint32_t* rhdr;          // per strip: slots, joins, then the join bits of its first row
    int rstrip;              // block rows per strip, 0 = single-workgroup grouping
    int w, h;
    int K, gw, gh;           // depth block size and grid
    int B, T, g, tau, r;     // method parameters
    int aligned;             // w % 4 == 0 and every RGB24 pointer 4-byte aligned
    int gather;              // reconstruct by the Fig. 3 gather instead of the warp and fill
    // block-iterative inpainting (ipc != null): the warp leaves, per view, a
    // word of tag and colour per pixel and the marks of the tiles with holes
    // for the sweeps and the final composition
    uint32_t* ipc;           // tag << 24 | colour, [2][h][w]
    uint32_t* ipf;           // tiles that hold a hole, [2][tiles]
    uint32_t* ipn;           // pixels the last sweep of each launch filled
    // end-of-depth-map signal (pipelined calls): the grouping's last kernel
    // stores sig_value to *sig when it is done (null: no signal)
    unsigned long long* sig;
    unsigned long long sig_value;
    // start-of-filter mark (pipelined calls): the depth filter stores
    // mark_value to *mark as it starts, i.e. once everything before it on
    // its stream is done (null: no mark)
    unsigned long long* mark;
    unsigned long long mark_value;
    // start-of-warp mark (three-stage pipelined calls): the warp stores
    // wmark_value to *wmark as it starts (null: no mark)
    unsigned long long* wmark;
    unsigned long long wmark_value;
};

// Launch shape of the warp kernel (one image row per workgroup).
struct WarpShape {
    int threads;        // workgroup size (multiple of 64, <= 1024)
    int quads;          // quads (4 px) per lane: 1, 2 or 4
    size_t lds_bytes;   // dynamic LDS per workgroup
};

// One kernel launch of a frame: every kernel takes a single FrameDesc.
struct LaunchSpec {
    const void* func;
    dim3 grid, block;
    size_t lds;
};

// Launch specifications (kernels_depth.hip, kernels_render.hip); func is null
// for an unsupported combination.
bool warp_shape(int w, WarpShape* out);
// The fewest quads per lane (1, 2, 4) that keep the lanes of a row within
// cap (else four quads per lane, up to 1024 lanes).
bool warp_shape_cap(int w, int cap, WarpShape* out);
LaunchSpec spec_blockstats(const FrameDesc& f);
LaunchSpec spec_regions(const FrameDesc& f);
// Strip-parallel grouping: strips, merge, per-block resolution.
int strip_rows(int gw, int gh);
int strip_lanes(int gw, int rows);
constexpr int kRegionSlots = 4096;  // slots the merge holds in LDS
// Blocks of a grid grouped whole on one workgroup (k_rg_small): four a lane,
// whose 64-block words are a lane each of one wave.  (Eight a lane, two words:
// 850x480, 6420 blocks, 33.6 us a frame where strips take 29.8.)
constexpr int kSmallBlocks = 4096;
constexpr int kMaxStrips = 64;
// 64-column pieces of the rows that one of the merge's 16 waves' strips start
// with, a lane each: at most 62, for 17 one-row strips of 1921 to 1927 columns
// (two strips of 31 pieces; a wider row leaves 16 rows, one strip a wave).
constexpr int kMaxPieces = 62;
constexpr int kStripHdrBits = 2;    // header word of the first join bits (2048 columns: 64 words)
constexpr int kStripHdrWords = 66;
LaunchSpec spec_rg_strip(const FrameDesc& f);
LaunchSpec spec_rg_merge(const FrameDesc& f);
LaunchSpec spec_rg_final(const FrameDesc& f);
LaunchSpec spec_cbf(const FrameDesc& f);
int cbf_tile_rows(long long tiles32);  // from the number of 64 x 32 tiles
// Filter tile rows for blocks of 2 px, whatever the launch: 16 / 32 / 48 rows
// take 281 / 276 / 275 us for a batch of 128 frames of 512x256 px at radius 2
// (8192 tiles of 32 rows), 365 / 370 / 383 for 140 at radius 3.
constexpr int kCbfRows2 = 16;
LaunchSpec spec_warp(const FrameDesc& f, const WarpShape& ws);
// Block-iterative inpainting: reset (before the warp), the sweeps in launches
// of kInpaintSweeps, composition once launch `last` has filled nothing in its
// last sweep (*done, in pinned host memory: 1 composed, 2 not done).
constexpr int kMaxSweeps = 4096;
constexpr int kInpaintSweeps = 8;
size_t inpaint_flags(int w, int h);
hipError_t launch_inpaint_reset(const FrameDesc& f, hipStream_t s);
hipError_t launch_inpaint_sweeps(const FrameDesc& f, int n, hipStream_t s);
hipError_t launch_inpaint_final(const FrameDesc& f, int last, uint32_t* done, hipStream_t s);
// Fig. 3 gather in place of the warp and the fill (one row per workgroup).
bool gather_fits(int w);
LaunchSpec spec_gather(const FrameDesc& f);

// Launch one spec on a stream (hipSuccess or the launch error).
inline hipError_t launch(const LaunchSpec& ls, const FrameDesc& f, hipStream_t s) {
    if (!ls.func) return hipErrorInvalidValue;
    FrameDesc arg = f;
    void* args[] = {&arg};
    return hipLaunchKernel(ls.func, ls.grid, ls.block, args, ls.lds, s);
}
// The same with the kernel's own start and stop times recorded into two
// events (timestamps of the dispatch itself, no marker packets around it).
inline hipError_t launch_timed(const LaunchSpec& ls, const FrameDesc& f, hipStream_t s, hipEvent_t start,
                               hipEvent_t stop) {
    if (!ls.func) return hipErrorInvalidValue;
    FrameDesc arg = f;
    void* args[] = {&arg};
    return hipExtLaunchKernel(ls.func, ls.grid, ls.block, args, ls.lds, s, start, stop, 0);
}
size_t regions_lds_bytes(int nb);
size_t merge_lds_bytes(int nb);  // the merge's, its fallback's or a small grid's, the largest
// Store v to *p (system-scope release) once everything before it on s is done.
hipError_t launch_signal(unsigned long long* p, unsigned long long v, hipStream_t s);
// Concurrency probe of two idle streams: a bounded wait on wait_on for a
// store of token to w[0] from post_on; w[1] receives 1 if the store was seen
// while waiting, 2 if not (the streams ran one after the other).
hipError_t launch_probe(unsigned long long* w, unsigned long long token, hipStream_t wait_on, hipStream_t post_on);
hipError_t prepare_depth_kernels();
hipError_t prepare_render_kernels();

// Accessors of the opaque context for the other C ABI files: its device, the
// batch object it keeps for pstereo_synthesize_batch, and its last-error text.
int ctx_device(const pstereo_ctx* c);
pstereo_batch** ctx_batch(pstereo_ctx* c);
void ctx_set_error(pstereo_ctx* c, const char* msg);

}  // namespace pstereo
