// gfx950 kernels of the stereo rendering (one frame per launch): the depth
// filter on tiles of 64 x 16, 32 or 48 px and the per-row warp; the bodies live
// in body_render.h.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>

#include "body_render.h"

namespace pstereo {

// The warp's start mark (three-stage pipelined calls), stored by the first
// lane of the first workgroup: the kernel runs only once all earlier work on
// its stream is done.
__device__ __forceinline__ void warp_start_mark(const FrameDesc& f) {
    if (f.wmark && blockIdx.x == 0 && threadIdx.x == 0)
        __hip_atomic_store(f.wmark, f.wmark_value, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

template <int R, bool ALIGNED, CbfKind KIND, int TH>
__global__ void __launch_bounds__(256) k_cbf(FrameDesc f) {
    __shared__ uint32_t lds[CbfTile<R, TH, KIND == CbfKind::kBlocks2>::kLdsWords];
    // the start mark of a pipelined call: this kernel runs only once all
    // earlier work on its stream is done (a system-scope store that a
    // stream's wait-value packet polls; it publishes no data)
    if (f.mark && blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0)
        __hip_atomic_store(f.mark, f.mark_value, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
    const int gx = gridDim.x;
    const int tile = xcd_tile(blockIdx.y * gx + blockIdx.x, gx * gridDim.y);
    const int ty = tile / gx;
    cbf_tile<R, ALIGNED, KIND, TH>(f, tile - ty * gx, ty, threadIdx.x, lds, true);
}

// Rows blockIdx.x, blockIdx.x + gridDim.x, ...: a grid of at most a few
// workgroups per CU walks the rows, loading each next row during the current
// one.  IP: block-iterative inpainting follows (a kernel of its own: the words
// it leaves take a dozen registers more, two of seven waves per SIMD).
template <bool ALIGNED, int Q, bool IP>
__global__ void __launch_bounds__(512) k_warp(FrameDesc f) {
    extern __shared__ uint32_t lds[];
    warp_start_mark(f);
    warp_rows<ALIGNED, Q, IP>(f, blockIdx.x, f.h, gridDim.x, threadIdx.x, blockDim.x, lds);
}

// Rows needing four quads per lane (wider than 4096 px): one row per
// workgroup of up to 1024 lanes (a second row's prefetched share would not
// fit the register budget).
template <bool ALIGNED, bool IP>
__global__ void __launch_bounds__(1024) k_warp_wide(FrameDesc f) {
    extern __shared__ uint32_t lds[];
    warp_start_mark(f);
    warp_row<ALIGNED, 4, IP>(f, blockIdx.x, threadIdx.x, blockDim.x, lds, true);
}

template <bool ALIGNED>
__global__ void __launch_bounds__(256) k_gather(FrameDesc f) {
    extern __shared__ uint32_t lds[];
    warp_start_mark(f);
    gather_row<ALIGNED>(f, blockIdx.x, threadIdx.x, blockDim.x, lds);
}

// Counters and tile marks back to zero before a frame's warp.
__global__ void __launch_bounds__(256) k_inpaint_reset(FrameDesc f, int nflag) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i < kMaxSweeps / kIpSweeps) f.ipn[i] = 0;
    if (i < nflag) f.ipf[i] = 0;
}

// Tags of filled pixels back to 0 (every kIpCycle launches).
__global__ void __launch_bounds__(256) k_inpaint_settle(FrameDesc f, int launch) {
    if (f.ipn[launch - 1] == 0) return;
    const size_t n = 2 * (size_t)f.w * f.h;
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (size_t)gridDim.x * 256) {
        const uint32_t w = f.ipc[i];
        if (w >> 24 && w >> 24 != kIpHole) f.ipc[i] = w & 0xFFFFFFu;
    }
}

// Words other lanes or workgroups may store meanwhile: whole, in one access.
__device__ __forceinline__ uint32_t load_word(const uint32_t* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
}
__device__ __forceinline__ void store_word(uint32_t* p, uint32_t v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
}

// Sweeps kIpSweeps n + 1 .. kIpSweeps (n + 1) of the block-iterative
// inpainting (Jacobi: a hole with at least two 8-neighbours undamaged before
// the sweep takes their per-channel mean rounded half up) on one marked tile
// of one view.  The tile is loaded with a halo of kIpSweeps px, so all of the
// launch's sweeps run in LDS: a halo pixel at distance d is right up to sweep
// kIpSweeps - d, which is all the tile's own pixels need.  Only those are
// written back, while other workgroups may load them: a word goes from hole
// to {sweep, colour} once, in one store, and both say the same whether a
// workgroup computes the pixel itself or reads it.  ipn[n] counts the pixels
// the last sweep filled; once it is 0 no later sweep fills any.
//
// One sweep per launch over every pixel of the frame moved 8 bytes a pixel 24
// times (1920x1080: 24.7 us each, 593 us a frame); three launches of eight
// sweeps on the tiles that hold holes take about 17 us each (bound by the LDS
// reads of the tiles fullest of holes; 512 or 1024 lanes a tile, or tiles of
// 16 or 64 rows, came out within 3 % at 1920x1080 and slower at 3840x2160).
__global__ void __launch_bounds__(256) k_inpaint_sweeps(FrameDesc f, int n) {
    if (n > 0 && f.ipn[n - 1] == 0) return;
    constexpr int S = kIpSweeps, RW = kIpW + 2 * S, RH = kIpH + 2 * S;
    constexpr uint32_t kOutside = 254u;
    __shared__ uint32_t reg[RW * RH];
    __shared__ uint16_t list[RW * RH];
    __shared__ uint32_t nlist, nlast, nleft;
    const int W = f.w, H = f.h, t = threadIdx.x, lane = t & 63;
    uint32_t* flag = f.ipf + gridDim.x * blockIdx.y + blockIdx.x;
    if (*flag == 0) return;
    const int ntx = (W + kIpW - 1) / kIpW;
    const int ty = blockIdx.x / ntx, tx = blockIdx.x - ty * ntx;
    const int x0 = tx * kIpW - S, y0 = ty * kIpH - S;
    uint32_t* words = f.ipc + (size_t)W * H * blockIdx.y;
    if (t == 0) nlist = nlast = nleft = 0;
    __syncthreads();
    const uint32_t tag0 = 1u + (uint32_t)(S * (n % kIpCycle));  // tag of this launch's first sweep
    constexpr int N = RW * RH / 256;
    static_assert(RW * RH % 256 == 0, "whole passes");
    uint32_t w[N];
#pragma unroll
    for (int k = 0; k < N; ++k) {
        const int i = t + 256 * k, ly = i / RW, lx = i - ly * RW;
        const int x = x0 + lx, y = y0 + ly;
        w[k] = (unsigned)x < (unsigned)W && (unsigned)y < (unsigned)H ? load_word(&words[(size_t)y * W + x]) : kOutside << 24;
    }
#pragma unroll
    for (int k = 0; k < N; ++k) {
        const int i = t + 256 * k, ly = i / RW, lx = i - ly * RW;
        const uint32_t tag = w[k] >> 24;
        uint32_t local = tag >= kOutside ? tag : tag - tag0 < (uint32_t)S ? tag - tag0 + 1u : 0u;
        reg[i] = (local << 24) | (w[k] & 0xFFFFFFu);
        // the region's rim has no neighbours here; it stays as it is
        const bool hole = tag == kIpHole && lx > 0 && lx < RW - 1 && ly > 0 && ly < RH - 1;
        const unsigned long long m = __ballot(hole);
        if (m) {
            uint32_t o = 0;
            if (lane == 0) o = atomicAdd(&nlist, (uint32_t)__popcll(m));
            o = __builtin_amdgcn_readfirstlane(o);
            if (hole) list[o + __popcll(m & ((1ull << lane) - 1ull))] = (uint16_t)i;
        }
    }
    __syncthreads();
    const int nl = (int)nlist;
    for (uint32_t s = 1; s <= (uint32_t)S; ++s) {
        for (int i = t; i < nl; i += 256) {
            const int p = list[i];
            if (load_word(&reg[p]) >> 24 != kIpHole) continue;
            constexpr int off[8] = {-RW - 1, -RW, -RW + 1, -1, 1, RW - 1, RW, RW + 1};
            uint32_t nb[8], cnt = 0, s02 = 0, s1 = 0;
#pragma unroll
            for (int k = 0; k < 8; ++k) nb[k] = load_word(&reg[p + off[k]]);
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                if (nb[k] >> 24 >= s) continue;
                ++cnt;
                s02 += nb[k] & 0x00FF00FFu;  // two 16-bit sums of at most 8 x 255
                s1 += (nb[k] >> 8) & 0xFFu;
            }
            if (cnt < 2) continue;
            const uint32_t h = cnt >> 1;
            const uint32_t r = div_small_quotient((s02 & 0xFFFFu) + h, cnt), g = div_small_quotient(s1 + h, cnt),
                           b = div_small_quotient((s02 >> 16) + h, cnt);
            store_word(&reg[p], (s << 24) | r | (g << 8) | (b << 16));
        }
        __syncthreads();
    }
    uint32_t last = 0, left = 0;
    for (int i = t; i < nl; i += 256) {
        const int p = list[i], ly = p / RW, lx = p - ly * RW;
        const int x = x0 + lx, y = y0 + ly;
        if (lx < S || lx >= S + kIpW || ly < S || ly >= S + kIpH) continue;
        const uint32_t v = reg[p], s = v >> 24;
        if (s == kIpHole) {
            left = 1;
        } else {
            store_word(&words[(size_t)y * W + x], ((tag0 + s - 1u) << 24) | (v & 0xFFFFFFu));
            last += s == (uint32_t)S;
        }
    }
    if (last) atomicAdd(&nlast, last);
    if (left) atomicOr(&nleft, 1u);
    __syncthreads();
    if (t == 0) {
        if (nlast) atomicAdd(&f.ipn[n], nlast);
        if (!nleft) *flag = 0;
    }
}

// The views from the inpainted colours (pixels never filled keep their own
// source pixel), then the anaglyph and the half side-by-side frame -- if the
// sweeps are done: ipn[last] = 0.  *done (host memory) receives 1 then, else
// 2 and nothing is written.
template <bool ALIGNED>
__global__ void __launch_bounds__(256) k_inpaint_final(FrameDesc f, int last, uint32_t* done) {
    const bool ready = f.ipn[last] == 0;
    if (blockIdx.x == 0 && threadIdx.x == 0)
        __hip_atomic_store(done, ready ? 1u : 2u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    if (!ready) return;
    const int W = f.w;
    const int q = blockIdx.x * 256 + threadIdx.x;
    const int qw = (W + 3) >> 2;
    if (q >= qw * f.h) return;
    const int y = q / qw, x0 = 4 * (q - y * qw);
    const size_t o = (size_t)y * W + x0;
    const uint32_t* pl = f.ipc + o;
    const uint32_t* pr = pl + (size_t)W * f.h;
    uint32_t cl[4] = {0, 0, 0, 0}, cr[4] = {0, 0, 0, 0};
    const int n = min(4, W - x0);
    if (ALIGNED || n == 4) {
        uint4 l, r;
        __builtin_memcpy(&l, pl, 16);
        __builtin_memcpy(&r, pr, 16);
        cl[0] = l.x, cl[1] = l.y, cl[2] = l.z, cl[3] = l.w;
        cr[0] = r.x, cr[1] = r.y, cr[2] = r.z, cr[3] = r.w;
    } else {
#pragma unroll
        for (int j = 0; j < 3; ++j)
            if (j < n) {
                cl[j] = pl[j];
                cr[j] = pr[j];
            }
    }
    if (max(max(max(cl[0], cl[1]), max(cl[2], cl[3])), max(max(cr[0], cr[1]), max(cr[2], cr[3]))) >= kIpHole << 24) {
        uint32_t src[4];
        quad_colours(load_quad_words<ALIGNED>(f.frame + o * 3, n), src);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if (cl[j] >> 24 == kIpHole) cl[j] = src[j];
            if (cr[j] >> 24 == kIpHole) cr[j] = src[j];
        }
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        cl[j] &= 0xFFFFFFu;
        cr[j] &= 0xFFFFFFu;
    }
    store_quad_views<ALIGNED>(f, y, x0, cl, cr);
}

// ---------------------------------------------------------------------------
// host-side launch helpers

// The plain path: up to 512 lanes per row (two quads per lane from 2048 px)
// before four quads per lane.
bool warp_shape(int w, WarpShape* out) { return warp_shape_cap(w, 512, out); }

bool warp_shape_cap(int w, int cap, WarpShape* out) {
    const int quads = (w + 3) / 4;
    int q = 1;
    while (q < 4 && (quads + q - 1) / q > cap) q *= 2;
    int threads = ((quads + q - 1) / q + 63) / 64 * 64;
    if (threads > 1024) return false;
    const size_t lds = warp_lds_bytes(w, threads, q);
    if (lds > kMaxLds) return false;
    out->threads = threads;
    out->quads = q;
    out->lds_bytes = lds;
    return true;
}

template <int R, bool A, CbfKind KIND, int TH>
static LaunchSpec cbf_launch(const FrameDesc& f) {
    return {reinterpret_cast<const void*>(&k_cbf<R, A, KIND, TH>),
            dim3((f.w + kTileW - 1) / kTileW, (f.h + TH - 1) / TH), dim3(256), 0};
}

template <int R, bool A, int TH>
static LaunchSpec cbf_th(const FrameDesc& f) {
    return f.K >= 8 && !f.depth_in && !f.out_df && !f.out_d0 ? cbf_launch<R, A, CbfKind::kPlain, TH>(f)
                                                             : cbf_launch<R, A, CbfKind::kAny, TH>(f);
}

// Tile height of a filter launch.  Up to about six 32-row tiles per CU (1536;
// eight are resident) the kernel is one round of workgroups and lasts as long
// as its slowest tile, so 16-row tiles, half as long, win although they read
// and convert a quarter more halo; with dozens per CU a tile's set-up and halo
// decide, and 48 rows win although only six fit a CU.  Measured, 16 / 32 / 48
// rows: 640x360 5.9 / 8.2 / 9.9 us, 1920x1080 10.4 / 10.9 / 12.3, 2240x1260
// (1400 tiles of 32) 12.0 / 12.8 / 12.6, 2560x1440 (1800) 13.9 / 13.9 / 14.1,
// 3840x2160 (4080) 24.0 / 21.1 / 21.5, 7680x4320 (16200) 67.0 / 52.6 / 49.6.
constexpr int kShortTiles = 1536, kTallTiles = 8192;

int cbf_tile_rows(long long tiles32) { return tiles32 <= kShortTiles ? 16 : tiles32 <= kTallTiles ? 32 : 48; }

template <int R, bool A>
static LaunchSpec cbf_spec(const FrameDesc& f) {
    // (an external depth map needs no blocks, whatever their size)
    if (f.K == 2 && !f.depth_in) return cbf_launch<R, A, CbfKind::kBlocks2, kCbfRows2>(f);
    switch (cbf_tile_rows((long long)((f.w + kTileW - 1) / kTileW) * ((f.h + 31) / 32))) {
        case 16: return cbf_th<R, A, 16>(f);
        case 48: return cbf_th<R, A, 48>(f);
        default: return cbf_th<R, A, 32>(f);
    }
}

template <bool A>
static LaunchSpec cbf_r(const FrameDesc& f) {
    switch (f.r) {
        case 0: return cbf_spec<0, A>(f);
        case 1: return cbf_spec<1, A>(f);
        case 2: return cbf_spec<2, A>(f);
        case 3: return cbf_spec<3, A>(f);
        default: return {nullptr, dim3(), dim3(), 0};
    }
}

LaunchSpec spec_cbf(const FrameDesc& f) { return f.aligned ? cbf_r<true>(f) : cbf_r<false>(f); }

// The row kernels by alignment, quads per lane (1, 2, 4) and inpainting.
constexpr int kWarpFns = 12;
static const void* warp_fn(bool aligned, int quads, bool ip) {
    static const void* const fns[kWarpFns] = {
        (const void*)&k_warp<false, 1, false>,   (const void*)&k_warp<false, 1, true>,
        (const void*)&k_warp<false, 2, false>,   (const void*)&k_warp<false, 2, true>,
        (const void*)&k_warp_wide<false, false>, (const void*)&k_warp_wide<false, true>,
        (const void*)&k_warp<true, 1, false>,    (const void*)&k_warp<true, 1, true>,
        (const void*)&k_warp<true, 2, false>,    (const void*)&k_warp<true, 2, true>,
        (const void*)&k_warp_wide<true, false>,  (const void*)&k_warp_wide<true, true>};
    return fns[(aligned ? 6 : 0) + (quads == 1 ? 0 : quads == 2 ? 2 : 4) + (ip ? 1 : 0)];
}
// Waves per SIMD their registers allow, read at preparation (every context
// stores the same values).
static std::atomic<int> g_warp_waves[kWarpFns];

LaunchSpec spec_warp(const FrameDesc& f, const WarpShape& ws) {
    const void* fn = warp_fn(f.aligned, ws.quads, f.ipc != nullptr);
    if (ws.quads == 4) return {fn, dim3(f.h), dim3(ws.threads), ws.lds_bytes};
    // resident workgroups per CU by LDS, lanes and registers (a workgroup's
    // waves spread over the 4 SIMDs), times 256 CUs; every workgroup gets a
    // row.  At 1920x1080 the scalar registers allow seven waves a SIMD where
    // the vector ones alone would allow eight: three workgroups a CU, and a
    // grid of four made the rest wait for a second round (768 workgroups 9.9
    // us, 1024 11.1, 540 11.9).  Of workgroups of one or two waves, four or two
    // take the place of one of four (1x60000 65 -> 36 us, 100x20000 28 -> 17,
    // 500x9000 19.6 -> 17.6); of three waves, more than one a SIMD do not all
    // fit (690x12000 32 -> 40)
    int waves_simd = 8;
    for (int i = 0; i < kWarpFns; ++i)
        if (warp_fn(i >= 6, i % 6 < 2 ? 1 : i % 6 < 4 ? 2 : 4, i & 1) == fn)
            waves_simd = g_warp_waves[i].load(std::memory_order_relaxed);
    const int waves = ws.threads / 64;
    const int by_regs = std::max(1, waves < 4 ? 4 / waves * waves_simd : waves_simd / ((waves + 3) / 4));
    const int by_lds = std::max(1, (int)(kMaxLds / std::max<size_t>(ws.lds_bytes, 1)));
    const int by_lanes = std::max(1, 2048 / ws.threads);
    const int resident = std::min(std::min(by_lds, by_lanes), by_regs) * 256;
    return {fn, dim3(std::min(f.h, resident)), dim3(ws.threads), ws.lds_bytes};
}

bool gather_fits(int w) { return gather_lds_bytes(w) <= kMaxLds; }

static int inpaint_tiles(int w, int h) { return ((w + kIpW - 1) / kIpW) * ((h + kIpH - 1) / kIpH); }

size_t inpaint_flags(int w, int h) { return 2 * (size_t)inpaint_tiles(w, h); }

hipError_t launch_inpaint_reset(const FrameDesc& f, hipStream_t s) {
    const int nflag = (int)inpaint_flags(f.w, f.h), n = std::max(nflag, kMaxSweeps / kIpSweeps);
    hipLaunchKernelGGL(k_inpaint_reset, dim3((n + 255) / 256), dim3(256), 0, s, f, nflag);
    return hipGetLastError();
}

hipError_t launch_inpaint_sweeps(const FrameDesc& f, int n, hipStream_t s) {
    if (n > 0 && n % kIpCycle == 0) hipLaunchKernelGGL(k_inpaint_settle, dim3(2048), dim3(256), 0, s, f, n);
    hipLaunchKernelGGL(k_inpaint_sweeps, dim3(inpaint_tiles(f.w, f.h), 2), dim3(256), 0, s, f, n);
    return hipGetLastError();
}

hipError_t launch_inpaint_final(const FrameDesc& f, int last, uint32_t* done, hipStream_t s) {
    const long long quads = (long long)((f.w + 3) / 4) * f.h;
    const dim3 grid((unsigned)((quads + 255) / 256));
    if (f.aligned) hipLaunchKernelGGL(k_inpaint_final<true>, grid, dim3(256), 0, s, f, last, done);
    else hipLaunchKernelGGL(k_inpaint_final<false>, grid, dim3(256), 0, s, f, last, done);
    return hipGetLastError();
}

LaunchSpec spec_gather(const FrameDesc& f) {
    const void* fn = f.aligned ? reinterpret_cast<const void*>(&k_gather<true>)
                               : reinterpret_cast<const void*>(&k_gather<false>);
    return {fn, dim3(f.h), dim3(256), gather_lds_bytes(f.w)};
}

hipError_t prepare_render_kernels() {
    hipError_t e;
    for (int i = 0; i < kWarpFns; ++i) {
        const void* fn = warp_fn(i >= 6, i % 6 < 2 ? 1 : i % 6 < 4 ? 2 : 4, i & 1);
        if ((e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kMaxLds)) != hipSuccess)
            return e;
        // one-wave workgroups without LDS: as many per CU as the registers
        // (vector and scalar) let run
        int waves = 0;
        if ((e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&waves, fn, 64, 0)) != hipSuccess) return e;
        g_warp_waves[i].store(std::min(8, std::max(1, waves / 4)), std::memory_order_relaxed);
    }
    if ((e = hipFuncSetAttribute(reinterpret_cast<const void*>(&k_gather<true>),
                                 hipFuncAttributeMaxDynamicSharedMemorySize, (int)kMaxLds)) != hipSuccess)
        return e;
    return hipFuncSetAttribute(reinterpret_cast<const void*>(&k_gather<false>),
                               hipFuncAttributeMaxDynamicSharedMemorySize, (int)kMaxLds);
}

}  // namespace pstereo
