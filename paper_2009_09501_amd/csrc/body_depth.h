// Device bodies of the depth-map stages: block statistics and region grouping
// (used by the per-frame kernels and by the persistent batch kernel).
//
// The depth map follows the paper's conversion scheme (Section 3, Fig. 1:
// the depth map is the first of the six components; Section 4: it is the
// "iterative" stage) built from block colour and edge cues (Section 2 and
// Table 1: edge / region-boundary information, block processing).  The exact
// cues, thresholds and region-depth rule are the library's readings.
#pragma once
#include <hip/hip_runtime.h>

#include <type_traits>

#include "device_common.h"

namespace pstereo {

// ---------------------------------------------------------------------------
// block statistics: per K x K block, rounded mean colour and edge flag.
//
// Tiles of 256 px x 4 RW rows on 256 lanes (four waves): wave w covers the RW
// rows [RW w, RW w + RW) of the tile (RW = 8 for blocks up to 16 px, 16 for
// larger ones, so that a block lies in one tile) and lane l the quad of
// pixels 4l .. 4l+3 in each of them, so every load instruction of a wave
// reads 768 contiguous bytes of one row; a lane issues all RW + 1 of its rows
// (its RW and the one below, for the vertical luma steps) before using any.
// Sums and luma come from byte dot products in registers; the horizontal step
// into the next quad takes that quad's first luma from the next lane (the
// tile's last lane loads the next tile's first pixel); the lanes of one block
// combine by lane shuffles, and blocks taller than a wave's rows add the
// waves' shares in LDS.
constexpr int kBsTileW = 256;  // px: 64 quads, one per lane of a wave

// Rows per wave of a block-statistics tile by default (the tile is four
// waves tall).
__host__ __device__ constexpr int bs_default_rw(int K) { return K <= 16 ? 8 : 16; }

// A 256 x 4 RWT px tile for blocks of K px (4 RWT >= K: a block never spans
// two tiles).
template <int K, int RWT = bs_default_rw(K)>
struct BsTile {
    static_assert(4 * RWT >= K && (RWT == 4 || RWT == 8 || RWT == 16), "block-statistics tile rows");
    static constexpr int RW = RWT;                                         // rows per wave
    static constexpr int TH = 4 * RW;                                      // tile rows
    static constexpr int QB = K / 4;                                       // lanes per block
    static constexpr int NBR = K >= RW ? 1 : RW / K;                       // block rows per wave
    static constexpr int kBlocks = (kBsTileW / K) * (TH / K);              // blocks per tile (K >= 4)
    static constexpr bool kCross = K > RW;                                 // blocks span waves
    static constexpr int kLdsWords = kCross ? 4 * kBlocks : 1;             // r, g, b, edge per block
};

// Tile rows of the block statistics for block size K (2 px blocks: 64).
__host__ __device__ constexpr int bs_tile_rows(int K) { return K <= 2 ? 64 : K <= 16 ? 32 : 64; }
// The same with a tuned height (0 = the default; else 16, 32 or 64, raised
// to K so that a block never spans two tiles; 2 px blocks keep 64).
__host__ __device__ constexpr int bs_tile_rows_tuned(int K, int rows) {
    return K <= 2 || rows == 0 ? bs_tile_rows(K) : (rows > K ? rows : K);
}

// Rounded mean sum / cnt of a block of cnt pixels, (sum + cnt / 2) / cnt: a
// shift for a whole K x K block (cnt = K * K, a power of two), the division
// only for blocks cut by the frame's right or bottom edge.
template <int K>
__device__ __forceinline__ uint32_t block_mean(uint32_t sum, uint32_t cnt) {
    constexpr uint32_t kFull = (uint32_t)(K * K);
    constexpr int kShift = __builtin_ctz(kFull);
    if (cnt == kFull) return (sum + kFull / 2) >> kShift;
    return (sum + cnt / 2) / cnt;
}

// Luma of the four pixels of a quad held in three dwords.
__device__ __forceinline__ void bs_quad_luma(uint3 q, uint32_t (&Y)[4]) {
    constexpr uint32_t wlo = 77u | (150u << 8) | (29u << 16);
    Y[0] = __builtin_amdgcn_udot4(q.x, wlo, 128u, false) >> 8;
    Y[1] = __builtin_amdgcn_udot4(__builtin_amdgcn_alignbyte(q.y, q.x, 3), wlo, 128u, false) >> 8;
    Y[2] = __builtin_amdgcn_udot4(__builtin_amdgcn_alignbyte(q.z, q.y, 2), wlo, 128u, false) >> 8;
    Y[3] = __builtin_amdgcn_udot4(q.z, wlo << 8, 128u, false) >> 8;
}

// One 256 x 4 RWT tile (tile_x, tile_y) on 256 lanes t = 0..255.  lds:
// BsTile<K, RWT>::kLdsWords words.  Inactive lane groups (active == false) do no
// memory work but pass the same barriers (blocks spanning waves only).
template <int K, bool ALIGNED, int RWT = bs_default_rw(K)>
__device__ __forceinline__ void bs_tile(const FrameDesc& f, int tile_x, int tile_y, int t, uint32_t* lds,
                                        bool active) {
    using T = BsTile<K, RWT>;
    constexpr int QB = T::QB, NBR = T::NBR, RW = T::RW;
    constexpr uint32_t wlo = 77u | (150u << 8) | (29u << 16);
    const int wave = t >> 6, lane = t & 63;
    const int W = f.w, H = active ? f.h : 0;
    const int x0 = tile_x * kBsTileW + 4 * lane;
    const int y0 = tile_y * T::TH + RW * wave;
    const int n = min(4, W - x0);  // pixels of the lane's quad inside the image (<= 0: none)
    const uint32_t g = (uint32_t)f.g;
    if (T::kCross)
        for (int i = t; i < T::kLdsWords; i += 256) lds[i] = 0;

    // every row's loads in flight before any is used
    const uint8_t* p0 = f.frame + ((size_t)y0 * W + x0) * 3;
    const size_t stride = (size_t)W * 3;
    uint3 v[RW + 1];
    uint32_t nx[RW];  // the tile's last lane: the next tile's first pixel per row
#pragma unroll
    for (int k = 0; k <= RW; ++k) {
        v[k] = make_uint3(0u, 0u, 0u);
        if (y0 + k < H && n > 0) v[k] = load_quad_words<ALIGNED>(p0 + k * stride, n);
    }
    const bool edge_lane = lane == 63 && x0 + 4 < W;
#pragma unroll
    for (int k = 0; k < RW; ++k) {
        nx[k] = 0u;
        if (edge_lane && y0 + k < H) {
            const uint8_t* q = p0 + k * stride + 12;
            nx[k] = ALIGNED ? *reinterpret_cast<const uint32_t*>(q)
                            : (uint32_t)q[0] | ((uint32_t)q[1] << 8) | ((uint32_t)q[2] << 16);
        }
    }

    // a step from pixel j to the right exists when j + 1 is in the image;
    // a pixel exists when j < n
    uint32_t sr[NBR], sg[NBR], sb[NBR], em[NBR];
#pragma unroll
    for (int i = 0; i < NBR; ++i) sr[i] = sg[i] = sb[i] = em[i] = 0u;
    // FULL: the wave's rows and the row below all lie inside the image (the
    // common case), so no row needs a bounds test
    auto rows = [&](auto full) {
        constexpr bool FULL = decltype(full)::value;
        uint32_t Yc[4];
        bs_quad_luma(v[0], Yc);
#pragma unroll
        for (int k = 0; k < RW; ++k) {
            const int br = (k * NBR) / RW;  // block row of row k inside the wave
            const int y = y0 + k;
            uint32_t Yb[4];
            bs_quad_luma(v[k + 1], Yb);  // the row below (zero past the image)
            const uint32_t yn_lane = (uint32_t)__shfl_down((int)Yc[0], 1);  // pixel x0 + 4 from the next lane
            if (FULL || y < H) {
                sr[br] = __builtin_amdgcn_udot4(v[k].x, 0x01000001u, sr[br], false);
                sr[br] = __builtin_amdgcn_udot4(v[k].y, 0x00010000u, sr[br], false);
                sr[br] = __builtin_amdgcn_udot4(v[k].z, 0x00000100u, sr[br], false);
                sg[br] = __builtin_amdgcn_udot4(v[k].x, 0x00000100u, sg[br], false);
                sg[br] = __builtin_amdgcn_udot4(v[k].y, 0x01000001u, sg[br], false);
                sg[br] = __builtin_amdgcn_udot4(v[k].z, 0x00010000u, sg[br], false);
                sb[br] = __builtin_amdgcn_udot4(v[k].x, 0x00010000u, sb[br], false);
                sb[br] = __builtin_amdgcn_udot4(v[k].y, 0x00000100u, sb[br], false);
                sb[br] = __builtin_amdgcn_udot4(v[k].z, 0x01000001u, sb[br], false);
                const uint32_t Yn = lane == 63 ? __builtin_amdgcn_udot4(nx[k], wlo, 128u, false) >> 8 : yn_lane;
                const uint32_t Yr[4] = {Yc[1], Yc[2], Yc[3], Yn};
                uint32_t dh[4], dv[4];
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const bool h_ok = ALIGNED ? (j < 3 || x0 + 4 < W) : (j < n && x0 + j + 1 < W);
                    const bool v_ok = (ALIGNED || j < n) && (FULL || y + 1 < H);
                    dh[j] = h_ok ? __builtin_amdgcn_sad_u16(Yr[j], Yc[j], 0u) : 0u;
                    dv[j] = v_ok ? __builtin_amdgcn_sad_u16(Yb[j], Yc[j], 0u) : 0u;
                }
                em[br] = max(max(max(em[br], dh[0]), max(dh[1], dh[2])),
                             max(max(dh[3], dv[0]), max(max(dv[1], dv[2]), dv[3])));
            }
#pragma unroll
            for (int j = 0; j < 4; ++j) Yc[j] = Yb[j];
        }
    };
    if (y0 + RW < H) rows(std::true_type{});
    else rows(std::false_type{});

    const int bx = x0 / K;  // the lane's block column (x0 >= 0)
    if (!T::kCross) {
        // K <= 16: a block lies in one wave, QB lanes wide; two 16-bit sums
        // per register (QB * K * 4 * 255 < 2^16)
#pragma unroll
        for (int br = 0; br < NBR; ++br) {
            uint32_t rg = sr[br] | (sg[br] << 16), be = sb[br] | ((em[br] > g ? 1u : 0u) << 16);
#pragma unroll
            for (int o = 1; o < QB; o <<= 1) {
                rg += (uint32_t)__shfl_xor((int)rg, o);
                be += (uint32_t)__shfl_xor((int)be, o);
            }
            const int by = (y0 + br * K) / K;
            if (active && lane % QB == 0 && bx < f.gw && by < f.gh && n > 0) {
                const uint32_t cnt = (uint32_t)((min(bx * K + K, W) - bx * K) * (min(by * K + K, H) - by * K));
                f.stats[by * f.gw + bx] = block_mean<K>(rg & 0xFFFFu, cnt) | (block_mean<K>(rg >> 16, cnt) << 8) |
                                          (block_mean<K>(be & 0xFFFFu, cnt) << 16) | ((be >> 16) ? 1u << 24 : 0u);
            }
        }
    } else {
        // blocks taller than RW: the wave's RW rows of its blocks, then across
        // waves (32-bit sums)
        uint32_t r = sr[0], gg = sg[0], b = sb[0], e = em[0] > g ? 1u : 0u;
#pragma unroll
        for (int o = 1; o < QB; o <<= 1) {
            r += (uint32_t)__shfl_xor((int)r, o);
            gg += (uint32_t)__shfl_xor((int)gg, o);
            b += (uint32_t)__shfl_xor((int)b, o);
            e |= (uint32_t)__shfl_xor((int)e, o);
        }
        __syncthreads();  // the LDS sums are zero
        constexpr int BC = kBsTileW / K;  // block columns per tile
        const int blk = (lane / QB) + BC * ((wave * RW) / K);
        if (lane % QB == 0) {
            atomicAdd(&lds[4 * blk + 0], r);
            atomicAdd(&lds[4 * blk + 1], gg);
            atomicAdd(&lds[4 * blk + 2], b);
            if (e) atomicOr(&lds[4 * blk + 3], 1u);
        }
        __syncthreads();
        if (t < T::kBlocks) {
            const int cbx = tile_x * BC + t % BC, cby = tile_y * (T::TH / K) + t / BC;
            if (active && cbx < f.gw && cby < f.gh) {
                const uint32_t cnt =
                    (uint32_t)((min(cbx * K + K, W) - cbx * K) * (min(cby * K + K, H) - cby * K));
                f.stats[cby * f.gw + cbx] = block_mean<K>(lds[4 * t + 0], cnt) |
                                            (block_mean<K>(lds[4 * t + 1], cnt) << 8) |
                                            (block_mean<K>(lds[4 * t + 2], cnt) << 16) | (lds[4 * t + 3] << 24);
            }
        }
    }
}

// Block statistics for blocks of 2 x 2 px (frames of at most 2^17 pixels,
// so this path is never the bulk of the work): 256 x 64 px tiles on 256
// lanes; lane t takes blocks t, t + 256, ... of the tile's 128 x 32 blocks,
// reading pixels bytewise and the luma steps to the right and below
// directly.  No barriers.
__device__ __forceinline__ void bs_tile_k2(const FrameDesc& f, int tile_x, int tile_y, int t, bool active) {
    if (!active) return;
    const int W = f.w, H = f.h;
    constexpr int BC = kBsTileW / 2, BR = 64 / 2;
    for (int i = t; i < BC * BR; i += 256) {
        const int bx = tile_x * BC + i % BC, by = tile_y * BR + i / BC;
        if (bx >= f.gw || by >= f.gh) continue;
        uint32_t sr = 0, sg = 0, sb = 0, cnt = 0, edge = 0;
        for (int dy = 0; dy < 2; ++dy) {
            for (int dx = 0; dx < 2; ++dx) {
                const int x = 2 * bx + dx, y = 2 * by + dy;
                if (x >= W || y >= H) continue;
                const uint8_t* p = f.frame + ((size_t)y * W + x) * 3;
                sr += p[0];
                sg += p[1];
                sb += p[2];
                ++cnt;
                const int Y = luma(p[0], p[1], p[2]);
                if (x + 1 < W && iabs(luma(p[3], p[4], p[5]) - Y) > f.g) edge = 1;
                if (y + 1 < H) {
                    const uint8_t* q = p + (size_t)W * 3;
                    if (iabs(luma(q[0], q[1], q[2]) - Y) > f.g) edge = 1;
                }
            }
        }
        f.stats[by * f.gw + bx] = ((sr + cnt / 2) / cnt) | (((sg + cnt / 2) / cnt) << 8) |
                                  (((sb + cnt / 2) / cnt) << 16) | (edge << 24);
    }
}

// ---------------------------------------------------------------------------
// region grouping, one workgroup of 1024 lanes per frame.
//
// Links join right / down neighbours that are both non-edge blocks and whose
// mean colours differ by at most tau (sum of absolute channel differences).
// A region is a connected component of the link graph; its label is its
// smallest block index.  Lane t owns the 32 contiguous blocks [32t, 32t+32).
//
//  1. link and edge bits of every block into LDS bitmaps;
//  2. row segments (maximal runs of right-linked blocks): a block-wide prefix
//     max of segment starts gives each block its segment; the parent array
//     starts as one star per segment;
//  3. lock-free union-find over the down links, only where the pair of
//     segments changes along the row; roots hook by a fixed pseudo-random
//     priority, so trees stay shallow whatever the order of the unions;
//  4. the smallest block index of every tree (atomic minimum at its root) is
//     the label; the parent array is then reused as the per-label block
//     count / background key and as the per-label lowest block row.
constexpr int kRegionThreads = 1024;
constexpr int kRegionPer = PSTEREO_MAX_BLOCKS / kRegionThreads;  // 32 blocks per lane

__device__ __forceinline__ uint32_t lds_load(const uint32_t* p) { return __atomic_load_n(p, __ATOMIC_RELAXED); }
__device__ __forceinline__ void lds_store(uint32_t* p, uint32_t v) { __atomic_store_n(p, v, __ATOMIC_RELAXED); }

// Bijective 32-bit mix: distinct blocks get distinct hooking priorities.
__device__ __forceinline__ uint32_t hook_prio(uint32_t x) {
    x *= 0x9E3779B1u;
    x ^= x >> 16;
    x *= 0x85EBCA6Bu;
    x ^= x >> 13;
    return x;
}

// LDS index of block b in the parent array: one pad word every 32 blocks, so
// the 64 lanes of a wave, each at its own run of 32 blocks, hit 64 distinct
// banks instead of one.
__device__ __forceinline__ uint32_t pidx(uint32_t b) { return b + (b >> 5); }

__device__ __forceinline__ uint32_t uf_find_s(uint32_t* parent, uint32_t x) {
    while (true) {
        const uint32_t p = lds_load(&parent[pidx(x)]);
        if (p == x) return x;
        const uint32_t gp = lds_load(&parent[pidx(p)]);
        if (gp != p) lds_store(&parent[pidx(x)], gp);
        x = gp;
    }
}

__device__ __forceinline__ void uf_unite_s(uint32_t* parent, uint32_t a, uint32_t b) {
    while (true) {
        a = uf_find_s(parent, a);
        b = uf_find_s(parent, b);
        if (a == b) return;
        if (hook_prio(a) > hook_prio(b)) { const uint32_t t = a; a = b; b = t; }
        if (atomicCAS(&parent[pidx(a)], a, b) == a) return;
    }
}

// Exact floor(n / d) for n, d < 2^16 from m = ceil(2^32 / d) (d >= 2): the
// product overshoots n / d by less than n / 2^32 < 1 / d, which never carries
// past the next integer.
__device__ __forceinline__ uint32_t div_u16(uint32_t n, uint32_t m, uint32_t d) {
    return d == 1 ? n : __umulhi(n, m);
}

// Region grouping of one frame on a whole 1024-lane workgroup; lds: the
// regions_lds_bytes(gw * gh) bytes of dynamic LDS.
//
// Lane t owns the 32 contiguous blocks [32t, 32t + 32).  Row segments (runs
// of right-linked blocks) are formed by a prefix-max scan, rows are joined by
// union-find in LDS only where the pair of segments changes along a row, and
// the label of a component (its smallest block index, always a segment start)
// is found at the root.  The label's own word then collects the lowest block
// row + 1 (low half, atomicMax) and the block count (high half, atomicAdd,
// after the rows); the lane owning the label block turns that into the
// region's depth.  Edge blocks are components of their own.
__device__ __forceinline__ void regions_body(const FrameDesc& f, uint32_t* lds) {
    const int gw = f.gw, gh = f.gh, nb = gw * gh;
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    constexpr int NW = kRegionThreads / 64;
    uint32_t* parent = lds;                           // pidx(nb) words
    uint32_t* lrb = parent + pidx((uint32_t)nb) + 1;  // right-link bits, word j = blocks 32j..32j+31
    uint32_t* ldb = lrb + kRegionThreads;             // down-link bits
    uint32_t* eb = ldb + kRegionThreads;              // edge bits
    uint32_t* scan = eb + kRegionThreads;             // NW words
    uint32_t* misc = scan + NW;                       // [0]: background key
    uint32_t* binfo_w = reinterpret_cast<uint32_t*>(f.binfo);

    // 1. block statistics into LDS (strided, coalesced loads, all in flight),
    // and the statistics half of the block table
    {
        uint32_t sv[kRegionPer];
#pragma unroll
        for (int i = 0; i < kRegionPer; ++i) {
            const int b = i * kRegionThreads + t;
            sv[i] = b < nb ? f.stats[b] : 0u;
        }
#pragma unroll
        for (int i = 0; i < kRegionPer; ++i) {
            const int b = i * kRegionThreads + t;
            if (b < nb) {
                parent[pidx(b)] = sv[i];
                binfo_w[2 * b] = sv[i];
            }
        }
    }
    if (t == 0) misc[0] = 0;
    __syncthreads();

    // 2. edge / right-link / down-link bits of the owned blocks, branch-free
    // from LDS (lane t's words sit 33 apart: distinct banks across a wave).
    // Blocks past the grid read as edges.
    const int b0 = t * kRegionPer;
    const int nown = max(0, min(kRegionPer, nb - b0));
    const uint32_t own_mask = nown >= 32 ? 0xFFFFFFFFu : ((1u << nown) - 1u);
    uint32_t* own = parent + 33 * t;  // own[i] = parent[pidx(b0 + i)] for i < 32
    int B0 = b0;
    const uint32_t gwm = gw > 1 ? (uint32_t)((0x100000000ull + (uint32_t)gw - 1) / (uint32_t)gw) : 0u;
    const uint32_t row0 = div_u16((uint32_t)min(b0, nb - 1 > 0 ? nb - 1 : 0), gwm, (uint32_t)gw);
    uint32_t emask = 0, lr = 0, ld = 0;
    {
        constexpr uint32_t kPast = 0xFF000000u;
        // bit i: block b0 + i ends its row (then it has no right neighbour);
        // a run of 32 blocks crosses at most one row end when gw >= 32
        uint32_t rowend = 0;
        if (gw >= kRegionPer) {
            const int wrap = (int)((row0 + 1) * (uint32_t)gw) - b0;  // next row's first block, from b0
            if (wrap >= 1 && wrap <= kRegionPer) rowend = 1u << (wrap - 1);
        } else {
            for (int i = 0; i < kRegionPer; ++i)
                if ((b0 + i + 1) % gw == 0) rowend |= 1u << i;
        }
        // two halves of 16 blocks: 33 loads in flight per half
#pragma unroll
        for (int h = 0; h < kRegionPer; h += 16) {
            // unconditional loads from clamped (in-range) indices, then a
            // select: no branch per load
            uint32_t sv[17], dv[16];
            const int last = nb - 1;
#pragma unroll
            for (int i = 0; i <= 16; ++i) {
                const int b = b0 + h + i;
                const uint32_t v = parent[pidx((uint32_t)min(b, last))];
                sv[i] = b <= last ? v : kPast;
            }
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                const int b = b0 + h + i + gw;
                const uint32_t v = parent[pidx((uint32_t)min(b, last))];
                dv[i] = b <= last ? v : kPast;
            }
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                const uint32_t sb = sv[i];
                const bool e = (sb >> 24) != 0;
                const bool row_end = (rowend >> (h + i)) & 1u;
                const bool rok = !row_end && !(sv[i + 1] >> 24) &&
                                 (int)__builtin_amdgcn_sad_u8(sb, sv[i + 1], 0u) <= f.tau;
                const bool dok = !(dv[i] >> 24) && (int)__builtin_amdgcn_sad_u8(sb, dv[i], 0u) <= f.tau;
                emask |= (uint32_t)e << (h + i);
                lr |= (uint32_t)(!e && rok) << (h + i);
                ld |= (uint32_t)(!e && dok) << (h + i);
            }
        }
    }
    emask = (uint32_t)opaque((int)(emask | ~own_mask));  // kept as one mask, not 32 flags
    lr &= own_mask;
    ld &= own_mask;
    lrb[t] = lr;
    ldb[t] = ld;
    eb[t] = emask;
    __syncthreads();

    B0 = opaque(b0);
    // 3. segments: start(b) = b is not right-linked from b - 1 (a row's first
    // block never is: the last block of a row has no right link)
    const uint32_t prev_lr = t > 0 ? lrb[t - 1] : 0u;
    const uint32_t linked_from_left = (lr << 1) | (prev_lr >> 31);
    const uint32_t starts = ~linked_from_left & own_mask;
    const int last_start = starts ? B0 + 31 - __clz(starts) : -1;
    int incl = last_start;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int v = __shfl_up(incl, o);
        if (lane >= o) incl = max(incl, v);
    }
    if (lane == 63) scan[wave] = (uint32_t)(incl + 1);
    __syncthreads();
    int carry = __shfl_up(incl, 1);
    if (lane == 0) carry = -1;
    for (int v = 0; v < wave; ++v) carry = max(carry, (int)scan[v] - 1);
    const int seg_in = carry;   // segment start of block b0 when b0 is not a start
#pragma unroll
    for (int i = 0; i < kRegionPer; ++i) {
        if ((starts >> i) & 1u) carry = B0 + i;
        if (i < nown) own[i] = (uint32_t)carry;
    }
    __syncthreads();

    B0 = opaque(b0);
    // 4. unions across rows, only where the pair of segments changes along
    // the row: skip b when b - 1 is in the same segment, also links down, and
    // the blocks below b - 1 and b are right-linked too (then b and the block
    // below it are already joined through b - 1).  Block b0 - 1 belongs to
    // the previous lane; its bits are read from the shared bitmaps.
    {
        const int c0 = B0 + gw;  // first block below the owned run
        uint32_t below_lr = 0;
        if (ld) {
            const int w = c0 >> 5, sh = c0 & 31;
            const uint32_t lo = lrb[w];
            const uint32_t hi = (w + 1 < kRegionThreads) ? lrb[w + 1] : 0u;
            below_lr = sh ? (lo >> sh) | (hi << (32 - sh)) : lo;  // bit i = right link of block c0 + i
        }
        uint32_t todo = ld & ~((ld & lr & below_lr) << 1);
        if ((todo & 1u) && t > 0 && ((ldb[t - 1] & prev_lr) >> 31)) {
            const int c = B0 - 1 + gw;  // below block b0 - 1 (exists: b0 - 1 links down)
            if ((lrb[c >> 5] >> (c & 31)) & 1u) todo &= ~1u;
        }
        while (todo) {
            const int i = __ffs(todo) - 1;
            todo &= todo - 1;
            uf_unite_s(parent, (uint32_t)(B0 + i), (uint32_t)(B0 + i + gw));
        }
    }
    __syncthreads();

    B0 = opaque(b0);
    // 5. labels of the segment starts: root, then the smallest start index of
    // the tree collected at the root as 0x10000 | min, then published in the
    // start's own word for the blocks of later lanes in the same segment
    uint32_t lab[kRegionPer];  // root, then label of each segment start; then label of each owned block
#pragma unroll
    for (int i = 0; i < kRegionPer; ++i) lab[i] = ((starts >> i) & 1u) ? uf_find_s(parent, opaque(b0) + i) : 0u;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kRegionPer; ++i)
        if (((starts >> i) & 1u) && lab[i] == (uint32_t)(B0 + i)) own[i] = 0xFFFFFFFFu;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kRegionPer; ++i)
        if ((starts >> i) & 1u) atomicMin(&parent[pidx(lab[i])], 0x10000u | (uint32_t)(B0 + i));
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kRegionPer; ++i)
        if ((starts >> i) & 1u) lab[i] = parent[pidx(lab[i])] & 0xFFFFu;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kRegionPer; ++i)
        if ((starts >> i) & 1u) own[i] = lab[i];
    __syncthreads();
    {
        uint32_t cur = (nown && !(starts & 1u)) ? parent[pidx(seg_in)] : 0u;
#pragma unroll
        for (int i = 0; i < kRegionPer; ++i) {
            if ((starts >> i) & 1u) cur = lab[i];
            lab[i] = cur;
        }
    }
    // piece ends: last owned block of a run of equal labels
    uint32_t pend = 0;
#pragma unroll
    for (int i = 0; i < kRegionPer; ++i)
        if (i + 1 < kRegionPer && lab[i + 1] != lab[i]) pend |= 1u << i;
    pend = (pend | (1u << (nown > 0 ? nown - 1 : 0))) & own_mask;
    // label blocks owned here (the component's smallest block)
    uint32_t lown = 0;
#pragma unroll
    for (int i = 0; i < kRegionPer; ++i)
        if (lab[i] == (uint32_t)(B0 + i)) lown |= 1u << i;
    lown &= own_mask;
    __syncthreads();

    B0 = opaque(b0);
    // 6. per non-edge label: lowest row + 1, then the block count
#pragma unroll
    for (int i = 0; i < kRegionPer; ++i)
        if ((lown >> i) & 1u) own[i] = 0;
    __syncthreads();
    const uint32_t nonedge_end = pend & ~emask;
#pragma unroll
    for (int i = 0; i < kRegionPer; ++i)
        if ((nonedge_end >> i) & 1u)
            atomicMax(&parent[pidx(lab[i])], div_u16((uint32_t)(B0 + i), gwm, (uint32_t)gw) + 1u);
    __syncthreads();
    {
        // a piece is one edge block or all non-edge; its length is the
        // distance to the previous piece end
        int prev = -1;
#pragma unroll
        for (int i = 0; i < kRegionPer; ++i) {
            if ((pend >> i) & 1u) {
                if (!((emask >> i) & 1u)) atomicAdd(&parent[pidx(lab[i])], (uint32_t)(i - prev) << 16);
                prev = i;
            }
        }
    }
    __syncthreads();

    B0 = opaque(b0);
    // 7. background = the largest non-edge region, ties to the smaller label
    // (largest key (count << 16) | (0xFFFF - label)); each non-edge label's
    // word becomes its region depth: the ramp at its lowest row
    {
        uint32_t best = 0;
        const uint32_t lne = lown & ~emask;
#pragma unroll
        for (int i = 0; i < kRegionPer; ++i) {
            if ((lne >> i) & 1u) {
                const uint32_t w = own[i];
                best = max(best, (w & 0xFFFF0000u) | (0xFFFFu - (uint32_t)(B0 + i)));
                own[i] = (uint32_t)ramp((int)(w & 0xFFFFu) - 1, gh);
            }
        }
#pragma unroll
        for (int o = 32; o >= 1; o >>= 1) best = max(best, (uint32_t)__shfl_xor((int)best, o));
        if (lane == 0 && best) atomicMax(&misc[0], best);
    }
    __syncthreads();
    const uint32_t bgkey = misc[0];
    const uint32_t bg = bgkey ? 0xFFFFu - (bgkey & 0xFFFFu) : 0xFFFFFFFFu;

    B0 = opaque(b0);
    // 8. block depth: edge and background blocks follow the row ramp, any
    // other block takes its region's depth; packed (label << 8 | depth)
    {
        auto pack = [&](int i, int rr) {
            const bool own_ramp = ((emask >> i) & 1u) || lab[i] == bg;
            const int d = own_ramp ? rr : (int)parent[pidx(lab[i])];
            lab[i] = (lab[i] << 8) | (uint32_t)d;
        };
        if (gw >= kRegionPer) {
            // at most two rows: the ramps of both, picked per block
            const int r0 = ramp((int)row0, gh), r1 = ramp((int)row0 + 1, gh);
            const int wrap = (int)((row0 + 1) * (uint32_t)gw) - b0;
#pragma unroll
            for (int i = 0; i < kRegionPer; ++i)
                if (i < nown) pack(i, i < wrap ? r0 : r1);
        } else {
#pragma unroll
            for (int i = 0; i < kRegionPer; ++i)
                if (i < nown) pack(i, ramp((int)div_u16((uint32_t)(B0 + i), gwm, (uint32_t)gw), gh));
        }
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kRegionPer; ++i)
        if (i < nown) own[i] = lab[i];
    __syncthreads();
#pragma unroll 8
    for (int i = 0; i < kRegionPer; ++i) {
        const int b = i * kRegionThreads + t;
        if (b < nb) {
            const uint32_t v = parent[pidx(b)];
            binfo_w[2 * b + 1] = (v & 255u) | kResolved;
            f.labels[b] = (int32_t)(v >> 8);
        }
    }
}

__host__ __device__ constexpr size_t regions_lds_bytes_c(int nb) {
    return (size_t)(nb + nb / 32 + 1 + 3 * kRegionThreads + kRegionThreads / 64 + 4) * 4;
}

// ---------------------------------------------------------------------------
// Strip-parallel region grouping.  The same components and labels as
// regions_body, computed in two launches (plus a per-block pass on request):
//   strips: one workgroup per strip of rstrip block rows (at most
//     kStripBlocks blocks, two per lane) finds the strip-local components by
//     union-find in LDS over horizontal runs of linked blocks (a root is
//     hooked under the smaller root, so every root is its component's
//     smallest block).  Its non-edge components, in block order, are the
//     first entries of the strip's own part of the slot list (from the index
//     of its first block on, so no strip waits for another's count); each
//     block gets {statistics, slot}, and the strip's header the number of
//     slots and one bit per column whose down link joins the strip above;
//   merge: one workgroup joins slots across strip boundaries (union-find over
//     the slots numbered strip by strip, so in label order, again rooted at
//     the smallest), sums counts and takes the lowest row per merged
//     component, picks the background and replaces each slot's list entry by
//     its final label and depth.  With more than kRegionSlots slots it runs
//     regions_loops instead, for the whole frame;
//   final (only for the per-block dump): one lane per block turns its slot
//     into the final label and depth.  The depth filter resolves the depths
//     it needs from the slot list itself.
//
// Both kernels are one chain of short dependent steps on at most a few CUs, so
// what counts is the number of memory round trips and barriers.  With fixed
// list parts per strip (no atomic counters, one round of loads before the
// merge's second), counts by row pieces, scans inside the vector unit and the
// joins hooked at once (1920x1080, between first and last in-kernel time
// stamp): strips 7.1 -> 4.6 us, merge 6.7 -> 6.0.

constexpr int kStripLanes = 1024;
constexpr int kStripBlocks = 2048;

// A strip's entry of the slot list: its local root (block in the strip), its
// non-edge blocks - 1 and its lowest block row in the strip.
static_assert(kStripBlocks <= 1 << 11 && kStripLanes <= 1 << 10, "slot entry: 11 + 11 + 10 bits");
__device__ __forceinline__ uint32_t slot_pack(uint32_t root, uint32_t cnt, uint32_t row) {
    return root | ((cnt - 1u) << 11) | (row << 22);
}

__device__ __forceinline__ uint32_t ufl_find(uint32_t* par, uint32_t x) {
    while (true) {
        const uint32_t p = lds_load(&par[x]);
        if (p == x) return x;
        const uint32_t gp = lds_load(&par[p]);
        if (gp != p) lds_store(&par[x], gp);
        x = gp;
    }
}

// Join the sets of a and b, hooking the larger root under the smaller.
__device__ __forceinline__ void ufl_unite(uint32_t* par, uint32_t a, uint32_t b) {
    while (true) {
        a = ufl_find(par, a);
        b = ufl_find(par, b);
        if (a == b) return;
        if (a < b) { const uint32_t t = a; a = b; b = t; }
        if (atomicCAS(&par[a], a, b) == a) return;
    }
}

__device__ __forceinline__ bool linked(uint32_t s, uint32_t n, int tau) {
    return !((s | n) >> 24) && (int)__builtin_amdgcn_sad_u8(s, n, 0u) <= tau;
}

// Inclusive sum or maximum over the lanes of a wave by lane moves inside the
// vector unit (within rows of 16 lanes, then from row to row): six short
// instructions where shuffles through LDS take six LDS round trips (0.3 us of
// a kernel whose whole chain is 5 us).
template <int CTRL, int ROWS>
__device__ __forceinline__ uint32_t dpp_or_0(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, ROWS, 0xF, false);
}
template <typename Op>
__device__ __forceinline__ uint32_t wave_scan(uint32_t v, Op op) {
    v = op(v, dpp_or_0<0x111, 0xF>(v));  // row_shr 1, 2, 4, 8
    v = op(v, dpp_or_0<0x112, 0xF>(v));
    v = op(v, dpp_or_0<0x114, 0xF>(v));
    v = op(v, dpp_or_0<0x118, 0xF>(v));
    v = op(v, dpp_or_0<0x142, 0xA>(v));  // lane 15 of rows 0, 2 to rows 1, 3
    v = op(v, dpp_or_0<0x143, 0xC>(v));  // lane 31 to rows 2, 3
    return v;
}
__device__ __forceinline__ uint32_t wave_scan_add(uint32_t v) {
    return wave_scan(v, [](uint32_t a, uint32_t b) { return a + b; });
}
__device__ __forceinline__ uint32_t wave_scan_max(uint32_t v) {
    return wave_scan(v, [](uint32_t a, uint32_t b) { return max(a, b); });
}

constexpr int kStripWaves = kStripLanes / 64;
__host__ __device__ constexpr size_t rg_strip_lds_words() {
    return 6 * kStripBlocks + kStripBlocks / 32 + kStripLanes + 2 * (2 * kStripWaves) + 2 * kStripWaves;
}

// One strip on NT lanes (whole waves; at least half of its blocks).
__device__ __forceinline__ void rg_strip_body(const FrameDesc& f, int strip, int NT, uint32_t* lds) {
    const int gw = f.gw, gh = f.gh, SR = f.rstrip, NW = NT >> 6;
    const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int r0 = strip * SR;
    const int rows = min(SR, gh - r0);
    const int n = rows * gw, base = r0 * gw;
    const int nload = (r0 + rows < gh ? rows + 1 : rows) * gw;
    uint32_t* st = lds;                      // statistics of the strip and the row below
    uint32_t* sa = st + 2 * kStripBlocks;    // statistics of the row above the strip
    uint32_t* par = sa + kStripBlocks;       // union-find
    uint32_t* cnt = par + kStripBlocks;      // per root: non-edge blocks
    uint32_t* row = cnt + kStripBlocks;      // per root: lowest local row
    uint32_t* starts = row + kStripBlocks;   // run-start bits, 32 blocks per word
    uint32_t* lastw = starts + kStripBlocks / 32 + 64 * wave;  // per wave: see below
    unsigned long long* rmask =              // root bits, 64 blocks per word
        reinterpret_cast<unsigned long long*>(starts + kStripBlocks / 32 + kStripLanes);
    uint32_t* rcnt = reinterpret_cast<uint32_t*>(rmask + 2 * kStripWaves);  // their counts | joins << 16
    const uint32_t gwm = gw > 1 ? (uint32_t)((0x100000000ull + (uint32_t)gw - 1) / (uint32_t)gw) : 0u;
    uint32_t* hdr = f.rhdr + strip * kStripHdrWords;

    for (int j = t; j < nload; j += NT) st[j] = f.stats[base + j];
    if (r0 > 0)
        for (int j = t; j < gw; j += NT) sa[j] = f.stats[base - gw + j];
    for (int j = t; j < n; j += NT) {
        par[j] = j;
        cnt[j] = 0;
        row[j] = 0;
    }
    __syncthreads();

    // horizontal runs: block j starts a run unless it is right-linked from
    // j - 1 in the same row; the start bits of a wave's 64 consecutive blocks
    // come from one ballot.  (A lane has a second block only in rows of more
    // than 1024 blocks.)
    const int NK = n > NT ? 2 : 1;
    int xk[2] = {0, 0}, yk[2] = {0, 0};
    uint32_t sk[2] = {0u, 0u};
    bool dk[2] = {false, false};  // down link inside the strip
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        if (k >= NK) break;
        const int j = t + k * NT;
        const bool in = j < n;
        yk[k] = in ? (int)div_u16((uint32_t)j, gwm, (uint32_t)gw) : 0;
        xk[k] = in ? j - yk[k] * gw : 0;
        sk[k] = in ? st[j] : 1u << 24;
        dk[k] = in && j + gw < n && linked(sk[k], st[j + gw], f.tau);
        const bool start = in && (xk[k] == 0 || !linked(st[j - 1], sk[k], f.tau));
        const unsigned long long m = __ballot(start);
        if (lane == 0 && j < n) {
            starts[j >> 5] = (uint32_t)m;
            starts[(j >> 5) + 1] = (uint32_t)(m >> 32);
        }
    }
    __syncthreads();
    // the start of block i's run: the last start bit at or before i (every
    // row's first block is one).  Each wave keeps, in its own slice, the last
    // start at or before the end of every 32-block word (a max-scan over the
    // words, n <= 2048), so a lookup reads at most two words
    {
        const uint32_t word = lane < ((n + 31) >> 5) ? starts[lane] : 0u;
        lastw[lane] = wave_scan_max(word ? (uint32_t)(lane * 32 + 32 - __clz(word)) : 0u) - 1u;
    }
    auto run_of = [&](int i) -> uint32_t {
        const int w = i >> 5;
        const uint32_t m = starts[w] & ((((uint32_t)1u << (i & 31)) << 1) - 1u);
        return m ? (uint32_t)(w * 32 + 31 - __clz(m)) : lastw[w - 1];
    };

    // unions between runs along the down links inside the strip, one per
    // place where the pair of runs above and below changes
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        if (k >= NK) break;
        const int j = t + k * NT;
        if (!dk[k]) continue;
        if (xk[k] > 0 && linked(st[j - 1], sk[k], f.tau) && linked(st[j - 1 + gw], st[j + gw], f.tau) &&
            linked(st[j - 1], st[j - 1 + gw], f.tau))
            continue;
        ufl_unite(par, run_of(j), run_of(j + gw));
    }
    __syncthreads();

    // roots (= smallest block of each component, its first run's start); per
    // root the non-edge count and lowest row, one pair of atomics per piece
    // of a row's consecutive blocks with one root in a wave; the bits of the
    // non-edge roots and of the joins with the strip above -- the down links
    // from the row above into the first row, except where block x - 1 links
    // the same pair of components (right links in both rows and a down link)
    uint32_t root[2] = {0u, 0u};
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        const int j = t + k * NT;
        unsigned long long rm = 0;
        if (k < NK) {
            const bool ne = !(sk[k] >> 24);
            root[k] = ne ? ufl_find(par, run_of(j)) : 0xFFFFFFFFu;
            const uint32_t left = (uint32_t)__shfl_up((int)root[k], 1);
            const bool head = ne && (lane == 0 || xk[k] == 0 || left != root[k]);
            const unsigned long long heads = __ballot(head), stop = heads | ~__ballot(ne);
            if (head) {
                const unsigned long long m = lane < 63 ? stop >> (lane + 1) : 0ull;
                const uint32_t len = m ? (uint32_t)__ffsll((long long)m) : 64u - (uint32_t)lane;
                atomicAdd(&cnt[root[k]], len);
                atomicMax(&row[root[k]], (uint32_t)yk[k]);
            }
            rm = __ballot(ne && root[k] == (uint32_t)j);
        }
        unsigned long long jm = 0;
        if (r0 > 0 && k * NT + 64 * wave < gw) {
            bool c = j < gw && linked(sa[j], st[j], f.tau);
            if (c && j > 0 && linked(sa[j - 1], st[j - 1], f.tau) && linked(sa[j - 1], sa[j], f.tau) &&
                linked(st[j - 1], st[j], f.tau))
                c = false;
            jm = __ballot(c);
            if (lane == 0) reinterpret_cast<unsigned long long*>(hdr + kStripHdrBits)[k * NW + wave] = jm;
        }
        if (lane == 0) {
            rmask[k * NW + wave] = rm;
            rcnt[k * NW + wave] = (uint32_t)__popcll(rm) | ((uint32_t)__popcll(jm) << 16);
        }
    }
    __syncthreads();
    // slots in block order: the roots before a root's 64-block word, then
    // those before it in the word
    const uint32_t own = lane < 2 * NW ? rcnt[lane] : 0u;
    const uint32_t incl = wave_scan_add(own);
    const uint32_t before = (incl - own) & 0xFFFFu;
    if (t == 63) *reinterpret_cast<uint2*>(hdr) = make_uint2(incl & 0xFFFFu, incl >> 16);
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        if (k >= NK) break;
        const int j = t + k * NT;
        const bool ne = !(sk[k] >> 24);
        const uint32_t r = ne ? root[k] : 0u;
        const uint32_t s = (uint32_t)base + (uint32_t)__shfl((int)before, (int)(r >> 6)) +
                           (uint32_t)__popcll(rmask[r >> 6] & ((1ull << (r & 63u)) - 1ull));
        if (j < n) f.binfo[base + j] = make_uint2(sk[k], ne ? s : 0u);
        if (ne && r == (uint32_t)j) f.rlist[s] = slot_pack(r, cnt[j], row[j]);
    }
}

// LDS of the merge of a grid of nb blocks: its tables, then the joins, 16 bits
// each and at most one a block, so that every grid's fit.  (Past a list of 8192
// the frame went to one workgroup as a whole: 512x64 blocks with 32 slots and
// 15,872 joins 127 -> 62 us a frame, 1000x32 with 15,500 131 -> 64.)
static_assert(PSTEREO_MAX_BLOCKS <= 1 << 16 && kRegionSlots <= 1 << 16, "block and slot indices of 16 bits");
__host__ __device__ constexpr size_t rg_merge_lds_words(int nb) {
    return 4 * (size_t)kRegionSlots + kMaxStrips + 4 + (size_t)(nb + 1) / 2;
}

// Region grouping of a whole frame on one 1024-lane workgroup in loops over
// its blocks, for launches that rarely come to it (more components than the
// merge holds): the same components, labels and depths as regions_body, whose
// 32 blocks a lane in registers set the registers of the kernel around it.
// With that body the merge took 128 VGPRs, 21 more spilled, and with it as a
// function called from there 540 bytes of scratch a lane; with this one 70 and
// none: 3840x2160 66.0 (67.5 called) -> 64.7 us a frame, 1920x1080 38.2 (39.9)
// -> 37.3.  Runs are joined by hooks and shortened paths, twice, before any
// search, and labels stay in registers, two to each (region grouping of a
// frame that comes here, with regions_body / every link by search and labels
// re-read / now: random blocks of 1024x128 px with half of them linked 114 /
// 120 / 92 us, a comb of those 103 / 101 / 86, a checkerboard of 240 x 135
// blocks 74 / 69 / 57).  lds: regions_loops_lds_words(gw * gh) words.
__host__ __device__ constexpr size_t regions_loops_lds_words(int nb) { return (size_t)nb + 1; }

__device__ __forceinline__ void regions_loops(const FrameDesc& f, uint32_t* lds) {
    const int gw = f.gw, gh = f.gh, nb = gw * gh;
    const int t = threadIdx.x, lane = t & 63;
    uint32_t* par = lds;
    uint32_t* misc = par + nb;  // [0]: background key
    const uint32_t gwm = gw > 1 ? (uint32_t)((0x100000000ull + (uint32_t)gw - 1) / (uint32_t)gw) : 0u;
    auto row_of = [&](int b) { return (int)div_u16((uint32_t)b, gwm, (uint32_t)gw); };
    if (t == 0) misc[0] = 0;
    // kU blocks of each lane at a time, so that their reads are in flight
    // together; bit i of a lane's masks is its block t + 1024 i
    constexpr int kU = 8, kN = kRegionPer;
    static_assert(kN == 32 && kN % kU == 0, "a bit a block of the lane");
    const int last = nb - 1;
    auto block = [&](int i) { return t + i * kRegionThreads; };

    // each block under the start of its run of the row (in a run longer than
    // the wave's 64 blocks first under the block before them)
    uint32_t runs_on = 0, solid = 0;  // the run starts before the wave's blocks; no edge block
    for (int i = 0; i * kRegionThreads < nb; i += kU) {
        uint32_t s[kU], left[kU];
#pragma unroll
        for (int k = 0; k < kU; ++k) {
            const int b = min(block(i + k), last);
            s[k] = f.stats[b];
            left[k] = f.stats[max(b - 1, 0)];
        }
#pragma unroll
        for (int k = 0; k < kU; ++k) {
            const int b = block(i + k);
            const bool runs = b < nb && b != row_of(min(b, last)) * gw && linked(left[k], s[k], f.tau);
            const unsigned long long m = ~__ballot(runs) & (((1ull << lane) << 1) - 1ull);
            if (b >= nb) continue;
            par[b] = (uint32_t)(m ? b - lane + 63 - __clzll((long long)m) : b - lane - 1);
            runs_on |= (uint32_t)!m << (i + k);
            solid |= (uint32_t)!(s[k] >> 24) << (i + k);
        }
    }
    __syncthreads();
    // the paths of the blocks in `which` down to their roots, by all lanes
    // together: a block goes to where its parent points, and those above it
    // take that step with it
    auto shorten = [&](uint32_t which) {
        for (int i = 0; i * kRegionThreads < nb; i += kU) {
            if (!((which >> i) & 0xFFu)) continue;
            uint32_t p[kU];
#pragma unroll
            for (int k = 0; k < kU; ++k) p[k] = lds_load(&par[min(block(i + k), last)]);
            for (bool more = true; more;) {
                uint32_t g[kU];
#pragma unroll
                for (int k = 0; k < kU; ++k) g[k] = lds_load(&par[p[k]]);
                more = false;
#pragma unroll
                for (int k = 0; k < kU; ++k) {
                    if (g[k] == p[k] || !((which >> (i + k)) & 1u)) continue;
                    lds_store(&par[block(i + k)], g[k]);
                    p[k] = g[k];
                    more = true;
                }
            }
        }
    };
    shorten(runs_on);
    __syncthreads();

    // links down, but for those that the blocks to the left have joined: the
    // run below is hooked under the smallest run that it links to, by one
    // atomic minimum a link
    uint32_t down = 0;
    for (int i = 0; i * kRegionThreads + gw < nb; i += kU) {
        uint32_t s[kU], left[kU], below[kU], bl[kU];
#pragma unroll
        for (int k = 0; k < kU; ++k) {
            const int b = min(block(i + k), last - gw);
            const int l = max(b - 1, 0);
            s[k] = f.stats[b];
            left[k] = f.stats[l];
            below[k] = f.stats[b + gw];
            bl[k] = f.stats[l + gw];
        }
#pragma unroll
        for (int k = 0; k < kU; ++k) {
            const int b = block(i + k);
            if (b + gw >= nb || !linked(s[k], below[k], f.tau)) continue;
            const bool row0 = b == row_of(b) * gw;
            const bool above_runs = !row0 && linked(left[k], s[k], f.tau);
            const bool below_runs = !row0 && linked(bl[k], below[k], f.tau);
            if (above_runs && below_runs && linked(left[k], bl[k], f.tau)) continue;
            // (only the words of run starts change here)
            const uint32_t ra = above_runs ? par[b] : (uint32_t)b, rb = below_runs ? par[b + gw] : (uint32_t)(b + gw);
            atomicMin(&par[rb], ra);
            down |= 1u << (i + k);
        }
    }
    __syncthreads();
    const uint32_t mine = t <= last ? 0xFFFFFFFFu >> (kN - 1 - (last - t) / kRegionThreads) : 0u;
    shorten(mine);
    __syncthreads();
    // a run that links to several keeps the smallest: once more root under
    // root for the links whose roots differ, then by search
    for (int i = 0; i * kRegionThreads < nb; i += kU) {
        if (!((down >> i) & 0xFFu)) continue;
        uint32_t ra[kU], rb[kU];
#pragma unroll
        for (int k = 0; k < kU; ++k) {
            ra[k] = lds_load(&par[min(block(i + k), last)]);
            rb[k] = lds_load(&par[min(block(i + k) + gw, last)]);
        }
#pragma unroll
        for (int k = 0; k < kU; ++k) {
            if (!((down >> (i + k)) & 1u)) continue;
            if (ra[k] == rb[k]) down &= ~(1u << (i + k));
            else atomicMin(&par[max(ra[k], rb[k])], min(ra[k], rb[k]));
        }
    }
    __syncthreads();
    shorten(mine);
    __syncthreads();
    for (; down; down &= down - 1) {
        const int b = block(__ffs(down) - 1);
        if (lds_load(&par[b]) != lds_load(&par[b + gw])) ufl_unite(par, (uint32_t)b, (uint32_t)(b + gw));
    }
    __syncthreads();

    // labels, kept in 16 bits a block
    uint32_t root[kN / 2];
#pragma unroll
    for (int i = 0; i < kN; i += kU) {
        if (i * kRegionThreads >= nb) break;
        uint32_t p[kU];
#pragma unroll
        for (int k = 0; k < kU; ++k) p[k] = lds_load(&par[min(block(i + k), last)]);
        for (bool more = true; more;) {
            uint32_t g[kU];
#pragma unroll
            for (int k = 0; k < kU; ++k) g[k] = lds_load(&par[p[k]]);
            more = false;
#pragma unroll
            for (int k = 0; k < kU; ++k) {
                more |= g[k] != p[k];
                p[k] = g[k];
            }
        }
#pragma unroll
        for (int k = 0; k < kU; ++k) {
            if (block(i + k) < nb) f.labels[block(i + k)] = (int32_t)p[k];
            root[(i + k) / 2] = k & 1 ? root[(i + k) / 2] | (p[k] << 16) : p[k];
        }
    }
    auto root_of = [&](int i) { return i & 1 ? root[i / 2] >> 16 : root[i / 2] & 0xFFFFu; };
    __syncthreads();
    for (int b = t; b < nb; b += kRegionThreads) par[b] = 0;
    __syncthreads();
    // per non-edge label the lowest row + 1 (low half), then the block count
    // (high half), by pieces of a row
    uint32_t heads = 0;
#pragma unroll
    for (int i = 0; i < kN; ++i) {
        if (i * kRegionThreads >= nb) break;
        const int b = min(block(i), last), y = row_of(b);
        const uint32_t r = root_of(i), left = (uint32_t)__shfl_up((int)r, 1);
        if (((solid >> i) & 1u) && (lane == 0 || b == y * gw || left != r)) {
            atomicMax(&par[r], (uint32_t)y + 1u);
            heads |= 1u << i;
        }
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kN; ++i) {
        if (i * kRegionThreads >= nb) break;
        const bool head = (heads >> i) & 1u;
        const unsigned long long stop = __ballot(head) | ~__ballot((solid >> i) & 1u);
        if (head) {
            const unsigned long long m = lane < 63 ? stop >> (lane + 1) : 0ull;
            atomicAdd(&par[root_of(i)], (m ? (uint32_t)__ffsll((long long)m) : 64u - (uint32_t)lane) << 16);
        }
    }
    __syncthreads();
    // background = the largest non-edge component, ties to the smaller label;
    // each non-edge label's word becomes its depth
    uint32_t best = 0;
    for (int i = 0; i * kRegionThreads < nb; i += kU) {
        uint32_t w[kU];
#pragma unroll
        for (int k = 0; k < kU; ++k) w[k] = par[min(block(i + k), last)];
#pragma unroll
        for (int k = 0; k < kU; ++k) {
            const int b = block(i + k);
            if (b >= nb || !w[k]) continue;  // 0: not a non-edge label
            best = max(best, (w[k] & 0xFFFF0000u) | (0xFFFFu - (uint32_t)b));
            par[b] = (uint32_t)ramp((int)(w[k] & 0xFFFFu) - 1, gh);
        }
    }
    best = wave_scan_max(best);
    if (lane == 63 && best) atomicMax(&misc[0], best);
    __syncthreads();
    const uint32_t bg = 0xFFFFu - (misc[0] & 0xFFFFu);
#pragma unroll
    for (int i = 0; i < kN; i += kU) {
        if (i * kRegionThreads >= nb) break;
        uint32_t s[kU], dep[kU];
#pragma unroll
        for (int k = 0; k < kU; ++k) {
            s[k] = f.stats[min(block(i + k), last)];
            dep[k] = par[root_of(i + k)];
        }
#pragma unroll
        for (int k = 0; k < kU; ++k) {
            const int b = block(i + k);
            if (b >= nb) break;
            if ((s[k] >> 24) || root_of(i + k) == bg) dep[k] = (uint32_t)ramp(row_of(b), gh);
            f.binfo[b] = make_uint2(s[k], dep[k] | kResolved);
        }
    }
}


__device__ __forceinline__ void rg_merge_body(const FrameDesc& f, uint32_t* lds) {
    const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int gw = f.gw, gh = f.gh, SR = f.rstrip;
    const int nstrip = (gh + SR - 1) / SR, per = SR * gw;  // blocks per strip
    uint32_t* par = lds;
    uint32_t* lab = par + kRegionSlots;   // label of a strip-local component | its place in the slot list << 16
    uint32_t* cnt = lab + kRegionSlots;
    uint32_t* row = cnt + kRegionSlots;
    uint32_t* first = row + kRegionSlots;   // per strip: its first slot - the place of that in the list
    uint32_t* misc = first + kMaxStrips;    // [0]: background key
    uint16_t* joins = reinterpret_cast<uint16_t*>(misc + 4);  // blocks that join the strip above theirs

    // A wave takes strips wave, wave + 16, ..., and the rows they start with in
    // pieces of 64 columns (lane l knows the l-th of at most kMaxPieces).  One
    // round of loads brings the counts of all strips, the first 64 slots of the
    // wave's strips and the join bits of its pieces.
    const uint2 hd =
        lane < nstrip ? *reinterpret_cast<const uint2*>(f.rhdr + lane * kStripHdrWords) : make_uint2(0u, 0u);
    const uint32_t own = hd.x;
    const int nc = (gw + 63) >> 6;
    const int li = lane / nc, lc = lane - li * nc, ls = wave + kStripWaves * li;
    const unsigned long long* hbits = reinterpret_cast<const unsigned long long*>(f.rhdr + kStripHdrBits);
    const unsigned long long bits = ls > 0 && ls < nstrip ? hbits[ls * (kStripHdrWords / 2) + lc] : 0ull;
    constexpr int SW = kMaxStrips / kStripWaves;  // strips per wave
    uint32_t ent[SW];
#pragma unroll
    for (int i = 0; i < SW; ++i) {
        const int s = wave + kStripWaves * i;
        ent[i] = s < nstrip && s * per + lane < gw * gh ? f.rlist[s * per + lane] : 0u;
    }
    // the joins as one flat list, so that a lane has about one of them: those
    // of the strips above, then of the strip's earlier pieces and columns
    const uint32_t nj = (uint32_t)__popcll(bits), upto = wave_scan_add(nj) - nj;
    const uint32_t jall = wave_scan_add(hd.y);
    const int njoins = (int)__builtin_amdgcn_readlane(jall, 63);
    const uint32_t jpos = (uint32_t)__shfl((int)(jall - hd.y), min(ls, 63)) + upto - (uint32_t)__shfl((int)upto, lane - lc);
    const int npiece = wave < nstrip ? ((nstrip - 1 - wave) / kStripWaves + 1) * nc : 0;
    const uint32_t pblk = (uint32_t)(ls * per + 64 * lc);
    for (int q = 0; q < npiece; ++q) {
        const uint32_t lo = __builtin_amdgcn_readlane((uint32_t)bits, q);
        const uint32_t hi = __builtin_amdgcn_readlane((uint32_t)(bits >> 32), q);
        const unsigned long long m = ((unsigned long long)hi << 32) | lo;
        const uint32_t o = __builtin_amdgcn_readlane(jpos, q) + lanes_below(m);
        if ((m >> lane) & 1ull) joins[o] = (uint16_t)(__builtin_amdgcn_readlane(pblk, q) + (uint32_t)lane);
    }
    // slot numbers: strip s's slots follow those of the strips above it
    const uint32_t incl = wave_scan_add(own);
    const uint32_t before = incl - own;
    const int ns = (int)__builtin_amdgcn_readlane(incl, 63);
    if (ns > kRegionSlots) {
        // too many strip-local components: group the whole frame here
        __syncthreads();  // the list is written over
        regions_loops(f, lds);
        return;
    }
    if (t < kMaxStrips) first[t] = before - (uint32_t)(t * per);
    if (t == 0) misc[0] = 0;
#pragma unroll
    for (int i = 0; i < SW; ++i) {
        const int s = wave + kStripWaves * i;
        if (s >= nstrip) break;
        const uint32_t o = __builtin_amdgcn_readlane(before, s), c = __builtin_amdgcn_readlane(own, s);
        for (uint32_t p = lane; p < c; p += 64) {
            const uint32_t e = p < 64 ? ent[i] : f.rlist[s * per + p];
            par[o + p] = o + p;
            lab[o + p] = ((uint32_t)(s * per) + (e & 2047u)) | (((uint32_t)(s * per) + p) << 16);
            cnt[o + p] = ((e >> 11) & 2047u) + 1u;
            row[o + p] = (uint32_t)(s * SR) + (e >> 22);
        }
    }
    __syncthreads();

    // A region that spans the frame is a chain of one slot per strip, and
    // lock-free unions along it walk ever longer paths, so first every slot is
    // hooked at once under the smallest slot above it that it joins (one
    // atomic minimum per join, no search), then every path is shortened by
    // all lanes together, and only joins whose two roots still differ are
    // united by search.  (1920x1080: 3.2 us of searches -> 1.9 in all.)
    const uint32_t perm = (uint32_t)((0x100000000ull + (uint32_t)per - 1) / (uint32_t)per);
    auto join_slots = [&](uint32_t blk, uint32_t& a, uint32_t& b) {
        const uint32_t s = div_u16(blk, perm, (uint32_t)per);
        b = f.binfo[blk].y + first[s];
        a = f.binfo[blk - gw].y + first[s - 1];
    };
    uint32_t ja = 0, jb = 0;
    if (t < njoins) {
        join_slots(joins[t], ja, jb);
        atomicMin(&par[jb], ja);
    }
    __syncthreads();
    for (int s = t; s < ns; s += kStripLanes) {
        // lanes of one path double its steps together; a racing step only
        // reads a shorter path
        uint32_t p = lds_load(&par[s]);
        while (true) {
            const uint32_t g = lds_load(&par[p]);
            if (g == p) break;
            lds_store(&par[s], g);
            p = g;
        }
    }
    __syncthreads();
    if (t < njoins) ufl_unite(par, ja, jb);
    // a lane's joins past the first, four at a time, so that their loads are
    // in flight together; of a row of joins between the same two slots only
    // the first is left
    for (int o = t + kStripLanes; o < njoins; o += 4 * kStripLanes) {
        uint32_t a[4], b[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) join_slots(joins[min(o + u * kStripLanes, njoins - 1)], a[u], b[u]);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const uint32_t pair = (a[u] << 16) | b[u], left = (uint32_t)__shfl_up((int)pair, 1);
            if (lane == 0 || left != pair) ufl_unite(par, a[u], b[u]);
        }
    }
    __syncthreads();

    // merged component totals at the roots (the root holds the smallest label)
    constexpr int SL = kRegionSlots / kStripLanes;  // slots per lane
    uint32_t root[SL];
#pragma unroll
    for (int i = 0; i < SL; ++i) {
        const int s = t + i * kStripLanes;
        if (s >= ns) break;
        root[i] = ufl_find(par, s);
        if (root[i] != (uint32_t)s) {
            atomicAdd(&cnt[root[i]], cnt[s]);
            atomicMax(&row[root[i]], row[s]);
        }
    }
    __syncthreads();
    // background = the largest component, ties to the smaller label
    uint32_t best = 0;
#pragma unroll
    for (int i = 0; i < SL; ++i) {
        const int s = t + i * kStripLanes;
        if (s >= ns) break;
        if (root[i] == (uint32_t)s) best = max(best, (cnt[s] << 16) | (0xFFFFu - (uint32_t)s));
    }
    best = wave_scan_max(best);
    if (lane == 63 && best) atomicMax(&misc[0], best);
    __syncthreads();
    const uint32_t bg = 0xFFFFu - (misc[0] & 0xFFFFu);
#pragma unroll
    for (int i = 0; i < SL; ++i) {
        const int s = t + i * kStripLanes;
        if (s >= ns) break;
        const uint32_t r = root[i];
        f.rlist[lab[s] >> 16] = ((lab[r] & 0xFFFFu) << 9) | ((r == bg ? 1u : 0u) << 8) | (uint32_t)ramp((int)row[r], gh);
    }
}

// ---------------------------------------------------------------------------
// Region grouping of a small grid (at most kSmallBlocks) on one workgroup of
// 1024 lanes, in one launch: the same components, labels and depths as
// regions_body, with the strips' and the merge's means.  Lane t has blocks t,
// t + 1024, ...; a block's parent is first the start of its row run (ballots
// and a scan over the grid's 64-block words), runs are hooked under the
// smallest run above them that they link to, paths are shortened by all lanes
// together and only links whose roots still differ are united by search.
// One launch less than strips and merge, and no tables between them: 640x360
// (3600 blocks) 24.6 -> 22.9 us a frame, 320x180 (920) 23.2 -> 20.1; with
// eight blocks a lane 850x480 (6420) took 33.6 where strips take 29.8.
__host__ __device__ constexpr size_t rg_small_lds_words() {
    return 4 * (size_t)kSmallBlocks + 2 * kSmallBlocks / 64 + 4;
}

__device__ __forceinline__ void rg_small_body(const FrameDesc& f, uint32_t* lds) {
    const int gw = f.gw, gh = f.gh, n = gw * gh;
    const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
    constexpr int N = kSmallBlocks, NB = N / kStripLanes, NWORD = N / 64;  // 64-block words
    static_assert(NWORD == 64, "a word a lane");
    uint32_t* st = lds;
    uint32_t* par = st + N;
    uint32_t* cnt = par + N;
    uint32_t* row = cnt + N;
    unsigned long long* starts = reinterpret_cast<unsigned long long*>(row + N);
    uint32_t* misc = row + N + 2 * NWORD;  // [0]: background key
    const uint32_t gwm = gw > 1 ? (uint32_t)((0x100000000ull + (uint32_t)gw - 1) / (uint32_t)gw) : 0u;

    uint32_t s[NB];
#pragma unroll
    for (int k = 0; k < NB; ++k) {
        const int j = t + k * kStripLanes;
        s[k] = j < n ? f.stats[j] : 1u << 24;
    }
#pragma unroll
    for (int k = 0; k < NB; ++k) {
        const int j = t + k * kStripLanes;
        st[j] = s[k];
        cnt[j] = 0;
        row[j] = 0;
    }
    if (t == 0) misc[0] = 0;
    __syncthreads();

    // row runs and the links down that change the pair of runs
    int x[NB], y[NB];
    uint32_t down = 0;  // bit k: block k unites its run with the one below
    unsigned long long sw[NB];
#pragma unroll
    for (int k = 0; k < NB; ++k) {
        const int j = t + k * kStripLanes;
        const bool in = j < n;
        y[k] = in ? (int)div_u16((uint32_t)j, gwm, (uint32_t)gw) : 0;
        x[k] = in ? j - y[k] * gw : 0;
        const uint32_t left = x[k] > 0 ? st[j - 1] : 1u << 24;
        const uint32_t below = in && j + gw < n ? st[j + gw] : 1u << 24;
        const uint32_t bl = in && x[k] > 0 && j + gw < n ? st[j + gw - 1] : 1u << 24;
        const bool from_left = linked(left, s[k], f.tau), dn = linked(s[k], below, f.tau);
        if (dn && !(from_left && linked(bl, below, f.tau) && linked(left, bl, f.tau))) down |= 1u << k;
        sw[k] = __ballot(!in || !from_left);
        if (lane == 0) starts[k * kStripWaves + wave] = sw[k];
    }
    __syncthreads();
    // last run start at or before the end of every word (index + 1): lane l
    // holds word l
    const unsigned long long word = starts[lane];
    const uint32_t last = wave_scan_max(word ? (uint32_t)(64 * lane + 64 - __clzll(word)) : 0u);
    uint32_t run[NB];
#pragma unroll
    for (int k = 0; k < NB; ++k) {
        const int w = k * kStripWaves + wave;
        const unsigned long long m = sw[k] & (((1ull << lane) << 1) - 1ull);
        const uint32_t before = w > 0 ? __builtin_amdgcn_readlane(last, w - 1) - 1u : 0u;
        run[k] = m ? (uint32_t)(64 * w + 63 - __clzll(m)) : before;
        par[t + k * kStripLanes] = run[k];
    }
    __syncthreads();

    // the joined runs above and below; from here on only run starts matter
    uint32_t rb[NB];
#pragma unroll
    for (int k = 0; k < NB; ++k) rb[k] = ((down >> k) & 1u) ? par[t + k * kStripLanes + gw] : 0u;
    __syncthreads();
#pragma unroll
    for (int k = 0; k < NB; ++k)
        if ((down >> k) & 1u) atomicMin(&par[rb[k]], run[k]);
    __syncthreads();
#pragma unroll
    for (int k = 0; k < NB; ++k) {
        const int j = t + k * kStripLanes;
        if (run[k] != (uint32_t)j || j >= n) continue;
        uint32_t q = lds_load(&par[j]);
        while (true) {
            const uint32_t g = lds_load(&par[q]);
            if (g == q) break;
            lds_store(&par[j], g);
            q = g;
        }
    }
    __syncthreads();
    uint32_t qa[NB], qb[NB];
#pragma unroll
    for (int k = 0; k < NB; ++k) {
        qa[k] = lds_load(&par[run[k]]);
        qb[k] = ((down >> k) & 1u) ? lds_load(&par[rb[k]]) : qa[k];
    }
#pragma unroll
    for (int k = 0; k < NB; ++k)
        if (qa[k] != qb[k]) ufl_unite(par, qa[k], qb[k]);
    __syncthreads();

    // per root the block count and lowest row, by pieces of a row
    uint32_t root[NB];
#pragma unroll
    for (int k = 0; k < NB; ++k) {
        const bool ne = !(s[k] >> 24);
        root[k] = ne ? ufl_find(par, run[k]) : 0xFFFFFFFFu;
        const uint32_t left = (uint32_t)__shfl_up((int)root[k], 1);
        const bool head = ne && (lane == 0 || x[k] == 0 || left != root[k]);
        const unsigned long long stop = __ballot(head) | ~__ballot(ne);
        if (head) {
            const unsigned long long m = lane < 63 ? stop >> (lane + 1) : 0ull;
            atomicAdd(&cnt[root[k]], m ? (uint32_t)__ffsll((long long)m) : 64u - (uint32_t)lane);
            atomicMax(&row[root[k]], (uint32_t)y[k]);
        }
    }
    __syncthreads();
    // background = the largest component, ties to the smaller label
    uint32_t best = 0;
#pragma unroll
    for (int k = 0; k < NB; ++k) {
        const int j = t + k * kStripLanes;
        if (root[k] == (uint32_t)j) best = max(best, (cnt[j] << 16) | (0xFFFFu - (uint32_t)j));
    }
    best = wave_scan_max(best);
    if (lane == 63 && best) atomicMax(&misc[0], best);
    __syncthreads();
    const uint32_t bg = 0xFFFFu - (misc[0] & 0xFFFFu);
#pragma unroll
    for (int k = 0; k < NB; ++k) {
        const int j = t + k * kStripLanes;
        if (j >= n) continue;
        const bool ne = !(s[k] >> 24);
        const int r = ne && root[k] != bg ? (int)row[root[k]] : y[k];
        f.binfo[j] = make_uint2(s[k], (uint32_t)ramp(r, gh) | kResolved);
        f.labels[j] = ne ? (int32_t)root[k] : j;
    }
}

// One block per lane: final label and depth from the block's slot (nothing to
// do after the single-workgroup grouping).
__device__ __forceinline__ void rg_final_block(const FrameDesc& f, int b) {
    const int gw = f.gw, gh = f.gh;
    if (b >= gw * gh) return;
    const uint2 e = f.binfo[b];
    if (e.y & kResolved) return;
    const int by = b / gw;
    const uint32_t v = (e.x >> 24) ? ((uint32_t)b << 9) | 256u : f.rlist[e.y];
    const uint32_t d = ((v >> 8) & 1u) ? (uint32_t)ramp(by, gh) : (v & 255u);
    f.binfo[b].y = d | kResolved;
    f.labels[b] = (int32_t)(v >> 9);
}

}  // namespace pstereo
