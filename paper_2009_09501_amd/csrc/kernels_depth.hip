// gfx950 kernels of the depth map: block statistics and region grouping (one
// frame per launch); the stage bodies live in body_depth.h.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "body_depth.h"

namespace pstereo {

template <int K, bool ALIGNED, int RW>
__global__ void __launch_bounds__(256) k_blockstats(FrameDesc f) {
    __shared__ uint32_t lds[BsTile<K, RW>::kLdsWords];
    const int gx = gridDim.x;
    const int tile = xcd_tile(blockIdx.y * gx + blockIdx.x, gx * gridDim.y);
    const int ty = tile / gx;
    bs_tile<K, ALIGNED, RW>(f, tile - ty * gx, ty, threadIdx.x, lds, true);
}

__global__ void __launch_bounds__(256) k_blockstats_k2(FrameDesc f) {
    bs_tile_k2(f, blockIdx.x, blockIdx.y, threadIdx.x, true);
}

// The signal of a finished depth map (pipelined calls; the kernel is one
// workgroup): every wave waits until its stores are acknowledged, then one
// lane's system-scope release store (which writes the L2 back first) sets the
// word a stream's wait-value packet polls, so the kernels that packet releases
// read the whole depth map from any XCD.
__device__ __forceinline__ void signal_done(const FrameDesc& f) {
    if (!f.sig) return;
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    if (threadIdx.x == 0) __hip_atomic_store(f.sig, f.sig_value, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

__global__ void __launch_bounds__(kRegionThreads) k_regions(FrameDesc f) {
    extern __shared__ uint32_t lds[];
    regions_body(f, lds);
    signal_done(f);
}

__global__ void __launch_bounds__(kStripLanes) k_rg_small(FrameDesc f) {
    extern __shared__ uint32_t lds[];
    rg_small_body(f, lds);
    signal_done(f);
}

__global__ void __launch_bounds__(kStripLanes) k_rg_strip(FrameDesc f) {
    __shared__ uint32_t lds[rg_strip_lds_words()];
    rg_strip_body(f, blockIdx.x, blockDim.x, lds);
}

__global__ void __launch_bounds__(kStripLanes) k_rg_merge(FrameDesc f) {
    extern __shared__ uint32_t lds[];
    rg_merge_body(f, lds);
    signal_done(f);
}

__global__ void __launch_bounds__(256) k_rg_final(FrameDesc f) { rg_final_block(f, blockIdx.x * 256 + threadIdx.x); }

// Whether two streams run beside each other.  k_probe_wait, launched on one
// stream, waits -- bounded in wall-clock time (s_memrealtime counts at
// 100 MHz) and in iterations, so it always ends -- for k_probe_post, launched
// on the other stream after it, to store `token` to w[0]; it then stores 1 to
// w[1] if it saw that store, 2 if its time ran out.  Streams that share a
// hardware queue run the two one after the other, so the wait runs out.
__global__ void __launch_bounds__(64) k_probe_wait(unsigned long long* w, unsigned long long token,
                                                   unsigned long long limit_ticks) {
    if (threadIdx.x != 0) return;
    const uint64_t t0 = __builtin_amdgcn_s_memrealtime();
    unsigned long long seen = 2;
    for (int i = 0; i < (1 << 16); ++i) {
        if (__hip_atomic_load(&w[0], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM) == token) {
            seen = 1;
            break;
        }
        if (__builtin_amdgcn_s_memrealtime() - t0 > limit_ticks) break;
        __builtin_amdgcn_s_sleep(2);
    }
    __hip_atomic_store(&w[1], seen, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

__global__ void __launch_bounds__(64) k_probe_post(unsigned long long* w, unsigned long long token) {
    if (threadIdx.x == 0) __hip_atomic_store(&w[0], token, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// The end of the kernels before it on its stream, as a word a wait-value
// packet polls: it runs once they are done and their stores written back.
__global__ void __launch_bounds__(64) k_signal(unsigned long long* p, unsigned long long v) {
    if (threadIdx.x == 0) __hip_atomic_store(p, v, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

// ---------------------------------------------------------------------------
// host-side launch helpers

template <int K, bool A>
static LaunchSpec bs_spec(const FrameDesc& f) {
    // 32-row tiles also for 32 px blocks (one frame; a batch, whose launch is
    // longer, keeps 64 rows there): 7680x4320 32.8 -> 31.6 us
    constexpr int RW = K <= 32 ? 8 : 16;
    constexpr int TH = BsTile<K, RW>::TH;
    return {reinterpret_cast<const void*>(&k_blockstats<K, A, RW>),
            dim3((f.w + kBsTileW - 1) / kBsTileW, (f.h + TH - 1) / TH), dim3(256), 0};
}

template <bool A>
static LaunchSpec bs_k(const FrameDesc& f) {
    switch (f.K) {
        case 2:
            return {reinterpret_cast<const void*>(&k_blockstats_k2),
                    dim3((f.w + kBsTileW - 1) / kBsTileW, (f.h + 63) / 64), dim3(256), 0};
        case 4: return bs_spec<4, A>(f);
        case 8: return bs_spec<8, A>(f);
        case 16: return bs_spec<16, A>(f);
        case 32: return bs_spec<32, A>(f);
        case 64: return bs_spec<64, A>(f);
        default: return {nullptr, dim3(), dim3(), 0};
    }
}

LaunchSpec spec_blockstats(const FrameDesc& f) { return f.aligned ? bs_k<true>(f) : bs_k<false>(f); }

size_t regions_lds_bytes(int nb) { return regions_lds_bytes_c(nb); }
// What the merge kernels run on a grid of nb blocks: the merge or the loops it
// falls back to, and in a batch a small grid's grouping.
static constexpr size_t merge_lds_words(int nb) {
    return std::max(std::max(rg_merge_lds_words(nb), regions_loops_lds_words(nb)), rg_small_lds_words());
}
size_t merge_lds_bytes(int nb) { return merge_lds_words(nb) * 4; }
static_assert(merge_lds_words(PSTEREO_MAX_BLOCKS) * 4 < regions_lds_bytes_c(PSTEREO_MAX_BLOCKS) - 12 * 1024 &&
                  merge_lds_words(PSTEREO_MAX_BLOCKS) * 4 <= kMaxLds,
              "no room for tables that only regions_body has");

LaunchSpec spec_regions(const FrameDesc& f) {
    if (f.gw * f.gh <= kSmallBlocks)
        return {reinterpret_cast<const void*>(&k_rg_small), dim3(1), dim3(kStripLanes), rg_small_lds_words() * 4};
    return {reinterpret_cast<const void*>(&k_regions), dim3(1), dim3(kRegionThreads), regions_lds_bytes(f.gw * f.gh)};
}

// Rows per strip: about one block per lane (two for rows wider than the
// workgroup), 0 when a row does not fit a strip or one workgroup groups the
// whole grid.  Narrow grids take strips of six rows (unless that makes more
// than kMaxStrips): the unions inside a strip walk its rows one after the
// other, which joining more strips does not.  Measured, strips of 2 / 4 / 6 /
// 8 / 12 rows: 850x480 (107x60 blocks) 32.3 / 31.4 / 31.3 / 31.7 / 31.6 us a
// frame, 720x576 (90x72) 29.0 / 28.4 / 28.3 / 28.4 / 28.6, 960x540 (120x68)
// 29.2 / 28.4 / 28.7 / 29.1 / 28.8.
static constexpr int strip_rows_of(int gw, int gh) {
    if (gw < 1 || gw > kStripBlocks || gw * gh <= kSmallBlocks) return 0;
    if (gw > kStripLanes) return 1;
    return std::min(kStripLanes / gw, std::max(6, (gh + kMaxStrips - 1) / kMaxStrips));
}
int strip_rows(int gw, int gh) { return strip_rows_of(gw, gh); }

// Over every grid of up to PSTEREO_MAX_BLOCKS blocks that takes strips: what
// the strips and the merge assume of them.  (For one row count, strips and
// pieces grow with gh, so the grids just before the count changes are enough.)
static constexpr bool strips_fit() {
    for (int gw = 1; gw <= kStripBlocks; ++gw) {
        const int top = PSTEREO_MAX_BLOCKS / gw;
        for (int gh = std::min(top, 6 * kMaxStrips);; gh = std::min(top, (gh / kMaxStrips + 1) * kMaxStrips)) {
            if (const int rows = strip_rows_of(gw, gh)) {
                const int strips = (gh + rows - 1) / rows;
                const int pieces = (strips + kStripWaves - 1) / kStripWaves * ((gw + 63) / 64);
                if (strips > kMaxStrips || pieces > kMaxPieces || rows * gw > kStripBlocks || rows > kStripLanes) return false;
            }
            if (gh >= top) break;
        }
    }
    return true;
}
static_assert(strips_fit(), "strips within the merge's tables, their pieces a lane each, entries within a slot's bits");
static_assert(kMaxPieces <= 64 && kMaxStrips <= 64, "a lane a strip and a lane a piece");
static_assert(kStripHdrWords >= kStripHdrBits + kStripBlocks / 32, "a join bit a column");

int strip_lanes(int gw, int rows) { return std::min(kStripLanes, (gw * rows + 63) / 64 * 64); }

LaunchSpec spec_rg_strip(const FrameDesc& f) {
    return {reinterpret_cast<const void*>(&k_rg_strip), dim3((f.gh + f.rstrip - 1) / f.rstrip),
            dim3(strip_lanes(f.gw, f.rstrip)), 0};
}

LaunchSpec spec_rg_merge(const FrameDesc& f) {
    return {reinterpret_cast<const void*>(&k_rg_merge), dim3(1), dim3(kStripLanes), merge_lds_bytes(f.gw * f.gh)};
}

LaunchSpec spec_rg_final(const FrameDesc& f) {
    return {reinterpret_cast<const void*>(&k_rg_final), dim3((f.gw * f.gh + 255) / 256), dim3(256), 0};
}

hipError_t launch_probe(unsigned long long* w, unsigned long long token, hipStream_t wait_on, hipStream_t post_on) {
    // 300 us: far beyond the start-up latency of a kernel on an idle stream
    hipLaunchKernelGGL(k_probe_wait, dim3(1), dim3(64), 0, wait_on, w, token, 30000ull);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_probe_post, dim3(1), dim3(64), 0, post_on, w, token);
    return hipGetLastError();
}

hipError_t launch_signal(unsigned long long* p, unsigned long long v, hipStream_t s) {
    hipLaunchKernelGGL(k_signal, dim3(1), dim3(64), 0, s, p, v);
    return hipGetLastError();
}

hipError_t prepare_depth_kernels() {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&k_regions),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)kMaxLds);
    if (e != hipSuccess) return e;
    if ((e = hipFuncSetAttribute(reinterpret_cast<const void*>(&k_rg_small),
                                 hipFuncAttributeMaxDynamicSharedMemorySize, (int)kMaxLds)) != hipSuccess)
        return e;
    return hipFuncSetAttribute(reinterpret_cast<const void*>(&k_rg_merge), hipFuncAttributeMaxDynamicSharedMemorySize,
                               (int)kMaxLds);
}

}  // namespace pstereo
