// Device bodies of the stereo rendering: filtered depth, then both views
// (used by the per-frame kernels and by the persistent batch kernel).
//
//   k_cbf   pixel depth (from the block tables) and its cross-bilateral
//           filter guided by luma (Section 3: filtered depth map; Section 4:
//           GPU cross-bilateral filtering), on 64 x 16, 64 x 32 or 64 x 48
//           pixel tiles with a halo in LDS.  Windows whose depths are all equal take the exact
//           shortcut; the other quads are compacted into a workgroup list so
//           that only they pay for the weighted sum.  Output: filtered depth,
//           one byte per pixel, in a scratch buffer.
//   k_warp  one image row per workgroup: left / right frame reconstruction
//           (Section 4, Fig. 3 code: depth -> shift, threshold T, half the
//           stereo base per view) as a forward warp whose z-buffer is an LDS
//           atomic max on (depth << 24 | RGB) -- the nearer source wins and
//           its colour travels in the key; then inpainting of the holes
//           (Section 3: post-processed frames) from the nearer valid pixel
//           of the row, found with wave ballots; then anaglyph composition
//           (Fig. 3 code: red from the left view, green and blue from the
//           right) and RGB24 stores.
#pragma once
#include <hip/hip_runtime.h>

#include <climits>

#include "device_common.h"

namespace pstereo {

// Distinct squared distances dx^2 + dy^2 inside a (2r+1)^2 window, r <= 3.
__host__ __device__ constexpr int k_value(int i) {
    return i == 0 ? 0 : i == 1 ? 1 : i == 2 ? 2 : i == 3 ? 4 : i == 4 ? 5 : i == 5 ? 8
         : i == 6 ? 9 : i == 7 ? 10 : i == 8 ? 13 : 18;
}
__host__ __device__ constexpr int k_index(int k) {
    return k == 0 ? 0 : k == 1 ? 1 : k == 2 ? 2 : k == 4 ? 3 : k == 5 ? 4 : k == 8 ? 5
         : k == 9 ? 6 : k == 10 ? 7 : k == 13 ? 8 : 9;
}
__host__ __device__ constexpr int k_count(int r) { return r == 0 ? 1 : r == 1 ? 3 : r == 2 ? 6 : 10; }

// Product weights ws(k) * wr(|d|) of the cross-bilateral filter for every
// distinct squared distance k (k_index order) and signed luma difference
// d = -255..255.  In LDS row k holds 512 u16 entries, entry d + 255 (the last
// one unused), two to a word; the table for radius r is the prefix of
// k_count(r) rows.  Indexed by the signed difference, a tap's entry sits at
// byte offset 2 Yq + (510 - 2 Yp) of its row (doubled luma), one add per tap.
__host__ __device__ constexpr uint32_t cbf_w(int k, int j) {
    return j < 511 ? spatial_w(k_value(k)) * range_w(j < 255 ? 255 - j : j - 255) : 0u;
}
// The range weight is 0 from |d| = kRangeTaps on, so only words kCbfW0 ..
// kCbfW0 + kCbfWords - 1 of a row are non-zero; global memory holds just
// those, in kCbfCopies copies that successive workgroups take in turn (every
// workgroup reads the table, and one copy would sit in few L2 channels).
constexpr int kRangeTaps = 43;
constexpr int kCbfW0 = (255 - (kRangeTaps - 1)) / 2;             // 106
constexpr int kCbfWords = (255 + (kRangeTaps - 1)) / 2 + 1 - kCbfW0;  // 43
constexpr int kCbfCopies = 32;
static_assert(range_w(kRangeTaps) == 0 && range_w(kRangeTaps - 1) != 0, "range weight support");
struct CbfWeightTable {
    uint32_t w[kCbfCopies][10 * kCbfWords];
};
__host__ __device__ constexpr CbfWeightTable make_cbf_weights() {
    CbfWeightTable t{};
    for (int k = 0; k < 10; ++k)
        for (int i = 0; i < kCbfWords; ++i) {
            const int j = 2 * (kCbfW0 + i);
            t.w[0][k * kCbfWords + i] = cbf_w(k, j) | cbf_w(k, j + 1) << 16;
        }
    for (int c = 1; c < kCbfCopies; ++c)
        for (int i = 0; i < 10 * kCbfWords; ++i) t.w[c][i] = t.w[0][i];
    return t;
}
__device__ const CbfWeightTable kCbfWeights = make_cbf_weights();

// Depth -> (left offset, right offset) of the Fig. 3 rule with the rounding
// reading: P = round(B*m/255), m = D when D > T (crossed) else 255 - D
// (uncrossed); the left view moves by ceil(P/2), the right view by floor(P/2),
// in opposite directions.  Packed as (oL & 0xFFFF) | (oR << 16).
__device__ __forceinline__ uint32_t shift_entry(int d, int B, int T) {
    const bool crossed = d > T;
    const int m = crossed ? d : 255 - d;
    const int P = (B * m + 127) / 255;
    const int a = (P + 1) >> 1, b = P >> 1;
    const int oL = crossed ? a : -a;
    const int oR = crossed ? -b : b;
    return ((uint32_t)oL & 0xFFFFu) | ((uint32_t)oR << 16);
}

typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));

// Packed-integer helpers (single gfx950 instructions).
__device__ __forceinline__ uint32_t dot2_u16(uint32_t a, uint32_t b, uint32_t c) {
    return __builtin_amdgcn_udot2(__builtin_bit_cast(u16x2, a), __builtin_bit_cast(u16x2, b), c, false);
}
__device__ __forceinline__ uint32_t perm(uint32_t hi, uint32_t lo, uint32_t sel) { return __builtin_amdgcn_perm(hi, lo, sel); }
__device__ __forceinline__ uint32_t alignbyte(uint32_t hi, uint32_t lo, uint32_t s) { return __builtin_amdgcn_alignbyte(hi, lo, s); }

// The four RGB24 pixels of a quad held in three dwords, as four R | G << 8 |
// B << 16 words (top byte zero).
__device__ __forceinline__ void quad_colours(uint3 v, uint32_t (&c)[4]) {
    c[0] = v.x & 0xFFFFFFu;
    c[1] = alignbyte(v.y, v.x, 3) & 0xFFFFFFu;
    c[2] = alignbyte(v.z, v.y, 2) & 0xFFFFFFu;
    c[3] = v.z >> 8;
}

// Luma of the four pixels of an aligned quad, doubled, as u16 pairs
// (2Y0 | 2Y1 << 16, 2Y2 | 2Y3 << 16).  Luma = byte 1 of 77R + 150G + 29B + 128.
__device__ __forceinline__ void quad_luma2(uint3 v, uint32_t& y01, uint32_t& y23) {
    constexpr uint32_t wlo = 77u | (150u << 8) | (29u << 16);  // R, G, B in bytes 0..2
    constexpr uint32_t whi = wlo << 8;                         // R, G, B in bytes 1..3
    const uint32_t r0 = __builtin_amdgcn_udot4(v.x, wlo, 128u, false);
    const uint32_t r1 = __builtin_amdgcn_udot4(alignbyte(v.y, v.x, 3), wlo, 128u, false);
    const uint32_t r2 = __builtin_amdgcn_udot4(alignbyte(v.z, v.y, 2), wlo, 128u, false);
    const uint32_t r3 = __builtin_amdgcn_udot4(v.z, whi, 128u, false);
    y01 = perm(r1, r0, 0x0c050c01u) << 1;
    y23 = perm(r3, r2, 0x0c050c01u) << 1;
}

// Region depth of a block in row by from its {statistics, region} entry: the
// entry holds the depth itself (kResolved) after the single-workgroup
// grouping, else its component's slot; edge blocks and the background follow
// the row ramp, other blocks take their merged component's depth.
__device__ __forceinline__ uint32_t block_depth(const FrameDesc& f, int by, uint2 e) {
    if (e.y & kResolved) return e.y & 255u;
    const uint32_t v = (e.x >> 24) ? 256u : f.rlist[e.y];
    return ((v >> 8) & 1u) ? (uint32_t)ramp(by, f.gh) : (v & 255u);
}

// The search key of a block in the filter's staged table (second word of its
// entry): its region depth when it is a non-edge block, else kNoCandidate,
// which stays above every candidate's key (distance << 16 | index << 8 |
// depth, distance <= 765) with any index or distance added and does not
// overflow.
constexpr uint32_t kNoCandidate = 0xFC000000u;

// Raw depth of the four pixels of a quad: the region depth of their block, or
// for an edge block that of the non-edge 3x3 neighbour block whose mean colour
// is nearest (L1), first strict minimum in raster order; with no candidate
// the ramp of the block row.  col[j] = R | G << 8 | B << 16 of pixel j; the
// L1 distance to a block mean (stats word, edge byte zero for candidates) is
// one v_sad_u8.  The blocks come from a table staged in LDS: tab holds the
// blocks from (bx_lo, by_lo) on, bp entries a row, {statistics, search key},
// and covers every block the lookup can touch; K = 1 << ks.
__device__ __forceinline__ void quad_depth_tab(const FrameDesc& f, int x0, int yy, int ks, const uint2* tab,
                                               int bx_lo, int by_lo, int bp, const uint32_t (&col)[4],
                                               uint32_t (&D)[4]) {
    const int by = yy >> ks;
    const uint2* at = tab + (__umul24(by - by_lo, bp) + ((x0 >> ks) - bx_lo));
    const uint2 own = *at;
    if (!(own.x >> 24)) {
#pragma unroll
        for (int j = 0; j < 4; ++j) D[j] = own.y;
        return;
    }
    // branch-free: per pixel the minimum of (distance << 16) + (k << 8 |
    // depth) over the candidates k in raster order (distance <= 765), so
    // that ties go to the first -- one v_sad_hi_u8 per candidate; a
    // non-candidate's key starts at kNoCandidate
    uint32_t best[4] = {0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu};
#pragma unroll
    for (int k = 0; k < 9; ++k) {
        const uint2 c = at[(k / 3 - 1) * bp + (k % 3 - 1)];
        const uint32_t tag = c.y | ((uint32_t)k << 8);
#pragma unroll
        for (int j = 0; j < 4; ++j) best[j] = min(best[j], __builtin_amdgcn_sad_hi_u8(col[j], c.x, tag));
    }
    // the ramp of the block row only where a pixel found no candidate (rare)
    bool none = false;
#pragma unroll
    for (int j = 0; j < 4; ++j) none |= best[j] >= kNoCandidate;
    uint32_t fallback = 0;
    if (none) fallback = (uint32_t)ramp(by, f.gh);
#pragma unroll
    for (int j = 0; j < 4; ++j) D[j] = best[j] >= kNoCandidate ? fallback : (best[j] & 255u);
}

// The same for blocks of 2 px, of which a quad spans two.
__device__ __forceinline__ void quad_depth_tab2(const FrameDesc& f, int x0, int yy, const uint2* tab, int bx_lo,
                                                int by_lo, int bp, const uint32_t (&col)[4], uint32_t (&D)[4]) {
    const int by = yy >> 1;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const uint2* at = tab + (__umul24(by - by_lo, bp) + ((x0 >> 1) + h - bx_lo));
        const uint2 own = *at;
        D[2 * h] = D[2 * h + 1] = own.y;
        if (!(own.x >> 24)) continue;
        uint32_t best[2] = {0xFFFFFFFFu, 0xFFFFFFFFu};
#pragma unroll
        for (int k = 0; k < 9; ++k) {
            const uint2 c = at[(k / 3 - 1) * bp + (k % 3 - 1)];
            const uint32_t tag = c.y | ((uint32_t)k << 8);
#pragma unroll
            for (int j = 0; j < 2; ++j) best[j] = min(best[j], __builtin_amdgcn_sad_hi_u8(col[2 * h + j], c.x, tag));
        }
        uint32_t fallback = 0;
        if (max(best[0], best[1]) >= kNoCandidate) fallback = (uint32_t)ramp(by, f.gh);
#pragma unroll
        for (int j = 0; j < 2; ++j) D[2 * h + j] = best[j] >= kNoCandidate ? fallback : (best[j] & 255u);
    }
}

// ---------------------------------------------------------------------------
// k_cbf: 64 x TH pixel tiles (TH = 16, 32 or 48 by the launch's size), 256 lanes;
// lane = one quad in every 16th tile row.  LDS holds, for the tile and a
// 4 px / R row halo, doubled luma and raw depth as u16 pairs (two dwords per
// quad).  A window of quad x0 reads the six dwords of columns x0-4 .. x0+7 per
// row.
//
// Bound: small frames, the serial chain of one workgroup (staging, luma and
// depth, window tests, filter); 4K and up, VALU issue (7.3 M wave
// instructions a 4K frame, 12 us of the 20.7) plus the last round's tail.
// With the taps free of image-bounds tests, the block table loaded first, the
// slot flag in the entry instead of a control word (whose load waited for the
// whole frame tile) and 32-bit offsets: 640x360 13.2 -> 7.2 us, 1920x1080 14.5
// -> 11.7, 1920x1080 of an external depth map at R = 3 31.5 -> 20.3, 3840x2160
// 25.5 -> 23.5, 7680x4320 64.7 -> 58.5; with the plain form, staging loads
// free of branches (behind which the compiler waited for each) and a work
// list without atomics 5.7, 10.3, -, 20.7 and (48 rows) 49.3.  512 lanes per
// 32-row tile (twice the waves, each with its own set-up) took 27.7 us at 4K.
constexpr int kTileQ = 16;                   // quads per tile row
constexpr int kTileW = 4 * kTileQ;           // 64 px
constexpr int kTileH = 32;                   // rows (default)
constexpr int kTileQuads = kTileQ + 2;       // quads per LDS row: one extra each side
constexpr int kRowWords = 2 * kTileQuads;    // 36 dwords per LDS row and plane

// Window of a pixel pair at an even LDS column c0: the words from the one
// holding column c0 - R through the one holding c0 + 1 + R.
template <int R>
struct CbfPairWin {
    static constexpr int kW0 = (R + 1) >> 1;  // words before c0's word
    static constexpr int kWords = (2 * kW0 + 1 + R) / 2 + 1;
};

// Doubled luma of a pixel outside the image: kRangeTaps above the largest
// luma, so its difference from every guide pixel has range weight 0 and the
// pixel drops out of both sums with no test (its entries run up to 42 past a
// table row: the zero head of the next row, or the table's zero tail).
constexpr uint32_t kLumaOut = 2u * (255 + kRangeTaps);
constexpr int kWtabTail = 32;  // words of zeros after the table's last row
static_assert(kLumaOut / 2 + 255 < 512 + 2 * kWtabTail, "outside pixels read zeros");

// c + w * (half HI of d): one v_mad_u32_u16, which reads the low half of w and
// picks the half of d (from C the compiler masks w and shifts d first).
template <int HI>
__device__ __forceinline__ uint32_t mad_half(uint16_t w, uint32_t d, uint32_t c) {
    uint32_t r;
    if constexpr (HI) asm("v_mad_u32_u16 %0, %1, %2, %3 op_sel:[0,1,0,0]" : "=v"(r) : "v"(w), "v"(d), "v"(c));
    else asm("v_mad_u32_u16 %0, %1, %2, %3" : "=v"(r) : "v"(w), "v"(d), "v"(c));
    return r;
}

// Filtered depth of the two pixels of a pair.  yw / dw: the window words of
// each of the 2R + 1 rows, luma doubled and raw depth as u16 pairs; pixel j
// sits at window column 2 kW0 + j, so every tap's word and half are
// compile-time constants.  Taps go in pairs (c, c + 1) of one word (c even),
// so the weighted depth sum and the weight sum each take one dot2 per pair on
// the word as stored; a row's odd tap out takes a multiply-add of its half.
// The pixel's own weight is a constant, and that between the two pixels is
// read once (it depends on the absolute luma difference).  Straight-line:
// pixels outside the image carry kLumaOut (weight 0), so no tap is tested and
// all table reads can be in flight.  R = 2: 172 VALU and 64 LDS instructions
// for the two pixels, 191 and 66 (and two 32-bit products in the divisions)
// with every tap in a pair and looked up; the stage by events 21.3 -> 20.7 us
// at 3840x2160, 49.5 -> 48.6 at 7680x4320.
template <int R>
__device__ __forceinline__ void cbf_pair(const uint32_t (&yw)[2 * R + 1][CbfPairWin<R>::kWords],
                                         const uint32_t (&dw)[2 * R + 1][CbfPairWin<R>::kWords],
                                         const uint16_t* wtab, uint32_t (&df)[2]) {
    constexpr int PW = CbfPairWin<R>::kWords;
    const uint8_t* wt = reinterpret_cast<const uint8_t*>(wtab);
    uint16_t mutual = 0;  // the weight between the two pixels
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const int pc = 2 * CbfPairWin<R>::kW0 + j;
        // byte offset of a tap's weight in its table row: 2 Yq + (510 - 2 Yp)
        // (a pixel past the row's end, never stored, counts as luma 255)
        const uint32_t base = 510u - min((yw[R][pc >> 1] >> (16 * (pc & 1))) & 0xFFFFu, 510u);
        uint32_t acc = 0, wsum = 0;
        auto weight = [&](int dx, int dy, uint32_t y2) -> uint16_t {
            if (dx == 0 && dy == 0) return spatial_w(0) * range_w(0);
            if (dy == 0 && dx == -1 && j == 1) return mutual;
            const uint16_t w = *reinterpret_cast<const uint16_t*>(wt + k_index(dx * dx + dy * dy) * 1024 + (y2 + base));
            if (dy == 0 && dx == 1 && j == 0) mutual = w;
            return w;
        };
#pragma unroll
        for (int dy = -R; dy <= R; ++dy) {
            const uint32_t(&yr)[PW] = yw[dy + R];
            const uint32_t(&dr)[PW] = dw[dy + R];
#pragma unroll
            for (int dx = -R - ((pc - R) & 1); dx <= R; dx += 2) {
                const int c = pc + dx;  // even
                const uint32_t y = yr[c >> 1], dd = dr[c >> 1];
                if (dx < -R) {
                    const uint16_t w = weight(dx + 1, dy, y >> 16);
                    acc = mad_half<1>(w, dd, acc);
                    wsum = mad_half<0>(w, 1u, wsum);
                } else if (dx + 1 > R) {
                    const uint16_t w = weight(dx, dy, y & 0xFFFFu);
                    acc = mad_half<0>(w, dd, acc);
                    wsum = mad_half<0>(w, 1u, wsum);
                } else {
                    const uint32_t wp = weight(dx, dy, y & 0xFFFFu) | ((uint32_t)weight(dx + 1, dy, y >> 16) << 16);
                    acc = dot2_u16(wp, dd, acc);
                    wsum = dot2_u16(wp, 0x00010001u, wsum);
                }
            }
        }
        df[j] = div_small_quotient(acc + (wsum >> 1), wsum);
    }
}

// A tile of 64 x TH px (TH a multiple of 16) on 256 lanes; K2: of blocks of
// 2 px.
template <int R, int TH = kTileH, bool K2 = false>
struct CbfTile {
    static constexpr int NT = 256;
    static_assert(16 * TH % NT == 0, "whole passes over the tile's quads");
    static constexpr int TR = TH + 2 * R;  // LDS rows incl. halo
    static constexpr int NK = k_count(R);
    // tY, tD: TR * kRowWords words each; wtab: NK * 512 u16 and its zero tail;
    // work: 16 TH u16, a quarter per wave; nwork: 4 words
    // block table of the tile, its halo and one ring of neighbours, uint2
    // each: at most 12 blocks a row (16 entries) by TH / 8 + 4 for blocks of
    // 8 px and more, 20 by TH / 4 + 4 for 4 px, 38 by TH / 2 + 6 for 2 px
    static constexpr int kBlkPitch = K2 ? 38 : 20;
    static constexpr int kBlkEntries = kBlkPitch * (K2 ? TH / 2 + 6 : TH / 4 + 4);
    static constexpr int kTabOff = 2 * TR * kRowWords;
    static constexpr int kWorkOff = kTabOff + NK * 256 + kWtabTail;
    static constexpr int kBlkOff = (kWorkOff + 8 * TH + 4 + 1) & ~1;  // 8-byte aligned
    static constexpr int kLdsWords = kBlkOff + 2 * kBlkEntries;
    static constexpr int NQ = (TR * kTileQuads + NT - 1) / NT;  // quads per lane incl. halo
};

// What a filter launch has to provide for: plain (generated depth, blocks of
// 8 px and more, no depth dumps -- nearly every call), blocks of 2 px, or any
// other.  The plain form drops the options' tests: 3840x2160 22.9 -> 21.8 us.
// Blocks of 2 px take a form of their own for their larger table (looked up in
// global memory, with their slots, 128 frames of 512x256 px at radius 2 took
// 422 us a batch and one 72; from the table 275 and 49).
enum class CbfKind { kPlain, kBlocks2, kAny };

// One 64 x TH tile (tile_x, tile_y) on 256 lanes t = 0..255 (four whole
// waves).  lds: CbfTile<R, TH>::kLdsWords words.  Inactive lane groups do no
// memory work but pass the same three barriers.
template <int R, bool ALIGNED, CbfKind KIND = CbfKind::kAny, int TH = kTileH>
__device__ __forceinline__ void cbf_tile(const FrameDesc& f, int tile_x, int tile_y, int t, uint32_t* lds,
                                         bool active) {
    constexpr int S = 2 * R + 1;
    constexpr bool K2 = KIND == CbfKind::kBlocks2, PLAIN = KIND == CbfKind::kPlain;
    using T = CbfTile<R, TH, K2>;
    constexpr int NT = T::NT;
    constexpr int TR = T::TR;
    constexpr int NK = T::NK;
    uint32_t* tY = lds;
    uint32_t* tD = tY + TR * kRowWords;
    uint16_t* wtab = reinterpret_cast<uint16_t*>(lds + T::kTabOff);
    uint16_t* work = reinterpret_cast<uint16_t*>(lds + T::kWorkOff);
    constexpr int kWavePart = 16 * TH / (NT / 64);
    int* nwork = reinterpret_cast<int*>(work + 16 * TH);  // per wave
    uint2* btab = reinterpret_cast<uint2*>(lds + T::kBlkOff);

    const uint8_t* depth_in = PLAIN ? nullptr : f.depth_in;
    uint8_t* out_df = PLAIN ? nullptr : f.out_df;
    uint8_t* out_d0 = PLAIN ? nullptr : f.out_d0;
    const int W = f.w, H = active ? f.h : 0;
    const int tx0 = tile_x * kTileW, ty0 = tile_y * TH;

    // the tile's block table: its blocks, those of the halo and one ring of
    // neighbours (clipped to the grid plus one ring outside it, whose entries
    // are marked as edge blocks), bp entries a row.  A lane's first entry is
    // loaded before anything else, so that the slot it leads to can be looked
    // up while the frame arrives
    const int ks = __builtin_ctz((unsigned)f.K);
    const int bx_lo = max(-1, ((tx0 - 4) >> ks) - 1);
    const int by_lo = max(-1, ((ty0 - R) >> ks) - 1), by_hi = min(f.gh, ((ty0 + TH - 1 + R) >> ks) + 1);
    const bool wide = PLAIN || (!K2 && ks >= 3);
    const int bp = wide ? 16 : T::kBlkPitch;
    const bool table = !depth_in && active;
    const int nbt = bp * (by_hi - by_lo + 1);
    auto entry_pos = [&](int i, int& bx, int& by) {
        const int r = wide ? i >> 4 : i / T::kBlkPitch;
        by = by_lo + r;
        bx = bx_lo + (i - r * bp);
    };
    auto entry_load = [&](int bx, int by) {  // the nearest block of the grid
        return f.binfo[__umul24(min(max(by, 0), f.gh - 1), f.gw) + min(max(bx, 0), f.gw - 1)];
    };
    auto entry_store = [&](int i, int bx, int by, uint2 e) {
        // outside the grid: an edge block; an edge block is never a candidate
        const bool in = (unsigned)by < (unsigned)f.gh && (unsigned)bx < (unsigned)f.gw;
        const uint32_t d = !in || (e.x >> 24) ? kNoCandidate : block_depth(f, by, e);
        btab[i] = make_uint2(in ? e.x : 1u << 24, d);
    };
    // a lane's first entries, all of them for blocks of 2 px and 8 px and more
    constexpr int NB = K2 ? (T::kBlkEntries + NT - 1) / NT : 1;
    static_assert(16 * (TH / 8 + 4) <= NT, "one pass for blocks of 8 px and more");
    int bx0[NB], by0[NB];
    uint2 e0[NB];
    if (table) {
#pragma unroll
        for (int k = 0; k < NB; ++k) {
            entry_pos(t + NT * k, bx0[k], by0[k]);
            e0[k] = entry_load(bx0[k], by0[k]);
        }
    }

    // the frame loads of all of a lane's quads of the tile and its halo.
    // Quads outside the image read the nearest one inside: their luma is
    // replaced below and their depths, those of a quad the window holds anyway
    // where it is consulted, change no test.  Addresses are the tile's first
    // row (uniform) and a 32-bit offset.
    constexpr int NQ = T::NQ;
    const int yb = max(ty0 - R, 0);
    const size_t row0 = (size_t)yb * W;
    const uint8_t* frame0 = f.frame + 3 * row0;
    const int xl = (W - 1) & ~3;  // the row's last quad
    uint3 vq[NQ];
    uint32_t dq[NQ];
    if (active) {
#pragma unroll
        for (int k = 0; k < NQ; ++k) {
            const int i = t + NT * k;
            if (NT * (k + 1) > TR * kTileQuads && i >= TR * kTileQuads) break;
            const int tr = i / kTileQuads, tq = i - tr * kTileQuads;
            const int yy = min(max(ty0 - R + tr, 0), H - 1), x0 = min(max(tx0 - 4 + 4 * tq, 0), xl);
            const uint32_t o = __umul24(yy - yb, W) + x0;
            vq[k] = load_quad_words<ALIGNED>(frame0 + 3u * o, W - x0);
            if (depth_in) dq[k] = load_quad_bytes<false>(depth_in + row0 + o, W - x0);
        }
    }

    // the non-zero words of the weight table: lane t holds word t of every row
    uint32_t wq[NK];
    {
        const uint32_t* src = kCbfWeights.w[(blockIdx.x + blockIdx.y) % kCbfCopies];
        const int i = min(max(t - kCbfW0, 0), kCbfWords - 1);
        const bool nz = i == t - kCbfW0;
#pragma unroll
        for (int k = 0; k < NK; ++k) wq[k] = src[k * kCbfWords + i];
#pragma unroll
        for (int k = 0; k < NK; ++k) wq[k] = nz ? wq[k] : 0u;
    }

    if (table) {
#pragma unroll
        for (int k = 0; k < NB; ++k)
            if (t + NT * k < nbt) entry_store(t + NT * k, bx0[k], by0[k], e0[k]);
        if (!PLAIN && !K2)
            for (int i = t + NT; i < nbt; i += NT) {
                int bx, by;
                entry_pos(i, bx, by);
                entry_store(i, bx, by, entry_load(bx, by));
            }
    }
#pragma unroll
    for (int k = 0; k < NK; ++k) reinterpret_cast<uint32_t*>(wtab)[k * 256 + t] = wq[k];
    if (t < kWtabTail) reinterpret_cast<uint32_t*>(wtab)[NK * 256 + t] = 0;
    __syncthreads();

    auto store_df = [&](int x0_, int y_, uint32_t df4) {
        const uint32_t o = __umul24(y_ - yb, W) + x0_;
        store_quad_bytes<ALIGNED>(f.df + row0 + o, df4, W - x0_);
        if (out_df) store_quad_bytes<false>(out_df + row0 + o, df4, W - x0_);
    };

    // a tile whose windows all lie in non-edge blocks of one region depth is
    // that depth (blocks of 8 px and more: at most 10 x 8 blocks under the
    // windows, one per lane in two steps)
    bool uniform = false;
    if (!depth_in && wide && !out_d0) {
        const int cx = min((max(tx0 - R, 0) >> ks) + (t & 15), min(tx0 + kTileW - 1 + R, W - 1) >> ks) - bx_lo;
        const int b0 = max(ty0 - R, 0) >> ks, b1 = min(ty0 + TH - 1 + R, H - 1) >> ks;
        const uint32_t c = btab[((ty0 >> ks) - by_lo) * bp + (tx0 >> ks) - bx_lo].y;
        uint32_t bad = 0;
        for (int b = b0 + ((t >> 4) & 3); b <= b1; b += 4) {
            const uint2 e = btab[(b - by_lo) * bp + cx];
            bad |= (e.x >> 24) | (e.y ^ c);
        }
        uniform = !__ballot(bad != 0);
        if (uniform) {
#pragma unroll
            for (int half = 0; half < 16 * TH / NT; ++half) {
                const int x0 = tx0 + 4 * (t & (kTileQ - 1)), y = ty0 + (t >> 4) + NT / 16 * half;
                if (x0 < W && y < H) store_df(x0, y, perm(c, c, 0u));
            }
        }
    }

    // doubled luma + raw depth of the tile and its halo (columns tx0-4 ..
    // tx0+67)
#pragma unroll
    for (int k = 0; k < NQ; ++k) {
        const int i = t + NT * k;
        if ((NT * (k + 1) > TR * kTileQuads && i >= TR * kTileQuads) || uniform || !active) break;
        const int tr = i / kTileQuads, tq = i - tr * kTileQuads;
        const int yo = ty0 - R + tr, xo = tx0 - 4 + 4 * tq;
        const int yy = min(max(yo, 0), H - 1), x0 = min(max(xo, 0), xl);
        const int n = W - x0;
        uint32_t y01, y23, col[4], D[4];
        quad_luma2(vq[k], y01, y23);
        if (yy != yo || x0 != xo) y01 = y23 = kLumaOut * 0x10001u;
        if (!ALIGNED && n < 4) {
            if (n < 2) y01 = (y01 & 0xFFFFu) | (kLumaOut << 16);
            y23 = n < 3 ? kLumaOut * 0x10001u : (y23 & 0xFFFFu) | (kLumaOut << 16);
        }
        if (depth_in) {
#pragma unroll
            for (int j = 0; j < 4; ++j) D[j] = (dq[k] >> (8 * j)) & 255u;
        } else {
            quad_colours(vq[k], col);
            if (K2) quad_depth_tab2(f, x0, yy, btab, bx_lo, by_lo, bp, col, D);
            else quad_depth_tab(f, x0, yy, ks, btab, bx_lo, by_lo, bp, col, D);
        }
        if (!ALIGNED) {
#pragma unroll
            for (int j = 1; j < 4; ++j) if (j >= n) D[j] = 0;
        }
        if (out_d0 && yy == yo && x0 == xo && tr >= R && tr < R + TH && tq >= 1 && tq <= kTileQ)
            store_quad_bytes<false>(out_d0 + (size_t)yy * W + x0, D[0] | (D[1] << 8) | (D[2] << 16) | (D[3] << 24), n);
        tY[tr * kRowWords + 2 * tq] = y01;
        tY[tr * kRowWords + 2 * tq + 1] = y23;
        tD[tr * kRowWords + 2 * tq] = D[0] | (D[1] << 16);
        tD[tr * kRowWords + 2 * tq + 1] = D[2] | (D[3] << 16);
    }
    __syncthreads();

    const int qx = t & (kTileQ - 1);
    const int wave = t >> 6;
    uint32_t nlist = 0;  // quads in this wave's part of the work list
#pragma unroll
    for (int half = 0; half < 16 * TH / NT; ++half) {
        const int ty = (t >> 4) + NT / 16 * half;
        const int x0 = tx0 + 4 * qx, y = ty0 + ty;
        bool needs = false;
        if (x0 < W && y < H && !uniform) {
            // exact shortcut: all in-window depths (columns x0-R .. x0+3+R,
            // rows inside the image) equal -> the normalised weighted sum is
            // that depth.  With blocks of 8 px or more the window's pixels
            // inside the image lie in at most 2 x 2 blocks: when those are
            // non-edge blocks of one region depth the window is uniform
            // (four table reads); else the depths are compared pixel by pixel
            // (a window over non-edge blocks of different depths holds pixels
            // of each -- every block under it holds a window pixel -- so it
            // is not uniform and goes to the filter without the pixel test:
            // the block-row steps of the background ramp are most of these)
            uint32_t c = 0, bad = 1, sure = 0;
            if (!depth_in && wide) {
                const int bxa = max(x0 - R, 0) >> ks, bxb = min(x0 + 3 + R, W - 1) >> ks;
                const int bya = max(y - R, 0) >> ks, byb = min(y + R, H - 1) >> ks;
                const uint2 e00 = btab[16 * (bya - by_lo) + (bxa - bx_lo)], e01 = btab[16 * (bya - by_lo) + (bxb - bx_lo)];
                const uint2 e10 = btab[16 * (byb - by_lo) + (bxa - bx_lo)], e11 = btab[16 * (byb - by_lo) + (bxb - bx_lo)];
                c = e00.y;
                const uint32_t edge = (e00.x | e01.x | e10.x | e11.x) >> 24;
                const uint32_t differ = (e01.y ^ c) | (e10.y ^ c) | (e11.y ^ c);
                bad = edge | differ;
                sure = !edge && differ;
            }
            if (bad && !sure) {
                c = tD[(ty + R) * kRowWords + 2 * qx + 2] & 0xFFFFu;
                bad = 0;
                const uint32_t splat = c | (c << 16);
#pragma unroll
                for (int i = 0; i < S; ++i) {
                    // (rows outside the image hold the depths of the nearest
                    // row inside, which the window holds too)
                    const int base = (ty + i) * kRowWords + 2 * qx;
#pragma unroll
                    for (int k = (4 - R) >> 1; k <= (7 + R) >> 1; ++k) {
                        const uint32_t mask = ((2 * k >= 4 - R) ? 0xFFFFu : 0u) | ((2 * k + 1 <= 7 + R) ? 0xFFFF0000u : 0u);
                        bad |= (tD[base + k] ^ splat) & mask;
                    }
                }
            }
            if (!bad) {
                store_df(x0, y, perm(c, c, 0u));
            } else {
                needs = true;
            }
        }
        // compact the quads that need the full filter, each wave into its own
        // part of the list
        const unsigned long long m = __ballot(needs);
        if (needs) work[kWavePart * wave + nlist + lanes_below(m)] = (uint16_t)(t + NT * half);
        nlist += (uint32_t)__popcll(m);
    }
    if ((t & 63) == 0) nwork[wave] = nlist;
    __syncthreads();
    // the full filter: two lanes per listed quad, two pixels each (half the
    // serial length of one lane per quad); the even lane of a pair takes its
    // partner's two results by a lane shuffle and stores all four.  All lanes
    // share the four parts of the list
    constexpr int PW = CbfPairWin<R>::kWords;
    const int n0 = nwork[0], n1 = n0 + nwork[1], n2 = n1 + nwork[2];
    const int nw2 = 2 * (n2 + nwork[3]);
    for (int i0 = 0; i0 < nw2; i0 += NT) {
        const int i = i0 + t;
        const bool on = i < nw2;
        const int k = i >> 1;
        const int at = k < n1 ? (k < n0 ? k : k - n0 + kWavePart)
                              : (k < n2 ? k - n1 + 2 * kWavePart : k - n2 + 3 * kWavePart);
        const int q = on ? work[at] : 0;
        const int hf = i & 1;
        const int qx_ = q & (kTileQ - 1), ty_ = q / kTileQ;
        const int x0_ = tx0 + 4 * qx_, y_ = ty0 + ty_;
        uint32_t df2[2] = {0u, 0u};
        if (on) {
            // the pair's first pixel is LDS column 4 qx + 4 + 2 hf
            const int wb = 2 * qx_ + 2 + hf - CbfPairWin<R>::kW0;
            uint32_t yw[S][PW], dw[S][PW];
#pragma unroll
            for (int r = 0; r < S; ++r) {
                const int base = (ty_ + r) * kRowWords + wb;
#pragma unroll
                for (int k = 0; k < PW; ++k) { yw[r][k] = tY[base + k]; dw[r][k] = tD[base + k]; }
            }
            cbf_pair<R>(yw, dw, wtab, df2);
        }
        const uint32_t other = (uint32_t)__shfl_xor((int)(df2[0] | (df2[1] << 8)), 1);
        if (on && !hf) {
            store_df(x0_, y_, df2[0] | (df2[1] << 8) | (other << 16));
        }
    }
}

// ---------------------------------------------------------------------------
// k_warp: one image row per workgroup.  Lane t owns the quads t, t + NT,
// t + 2 NT, ... (Q of them), so the lanes of a wave always touch consecutive
// quads: coalesced global traffic.  Quad iteration qi of wave w covers the
// 256-pixel chunk c = qi * NW + w, and chunks follow each other along the
// row, which is what the hole search walks.  The z-buffer index of pixel x is
// swizzled to x + x / 32 so that the four pixels of the lanes' quads spread
// over all LDS banks.
__device__ __forceinline__ int kidx(int x) { return x + (x >> 5); }

// 1 if k != 0, else 0, as one v_min_u32 (the optimiser would turn min(k, 1)
// back into a compare and a select through VCC).
__device__ __forceinline__ uint32_t nonzero_bit(uint32_t k) {
    uint32_t r;
    asm("v_min_u32 %0, %1, 1" : "=v"(r) : "v"(k));
    return r;
}

// kidx(x) held as one value, so that the word address is formed from it in
// one shift-add instead of the two shifted terms the optimiser distributes
// it into.
__device__ __forceinline__ int kidx_held(int x) {
    int k = kidx(x);
    asm("" : "+v"(k));
    return k;
}

// Per-byte mean of two packed colours, rounded half up, with no carries
// between bytes: (a | b) - ((a ^ b) >> 1) per byte.
__device__ __forceinline__ uint32_t avg_bytes(uint32_t a, uint32_t b) {
    return (a | b) - (((a ^ b) >> 1) & 0x7F7F7F7Fu);
}

// Two packed R | G << 8 | B << 16 pixels to 6 bytes at an even address.
__device__ __forceinline__ void store_px2_u16(uint8_t* p, uint32_t c0, uint32_t c1) {
    uint16_t* q = reinterpret_cast<uint16_t*>(p);
    q[0] = (uint16_t)c0;
    q[1] = (uint16_t)(((c0 >> 16) & 0xFFu) | ((c1 & 0xFFu) << 8));
    q[2] = (uint16_t)(c1 >> 8);
}

__device__ __forceinline__ void store_px_bytes(uint8_t* p, uint32_t c) {
    p[0] = (uint8_t)c;
    p[1] = (uint8_t)(c >> 8);
    p[2] = (uint8_t)(c >> 16);
}

// The outputs of four pixels x0..x0+3 of row y from their left / right view
// colours (R | G << 8 | B << 16): left and right views, the anaglyph (red
// from the left view, green and blue from the right), and the half
// side-by-side frame when requested (half column p = mean of view columns 2p,
// 2p + 1 rounded up per byte; left view in the first floor(W/2) columns,
// right view after them).  ALIGNED: W % 4 == 0 and 4-byte aligned buffers,
// four pixels = three dwords.
template <bool ALIGNED>
__device__ __forceinline__ void store_quad_views(const FrameDesc& f, int y, int x0, const uint32_t* cl,
                                                 const uint32_t* cr) {
    const int W = f.w;
    const int n = min(4, W - x0);
    const size_t off = ((size_t)y * W + x0) * 3;
    if (ALIGNED || n == 4) {
        // both views packed once; in the three dwords of a quad the red bytes
        // sit at fixed places, so the anaglyph is one bit-field insert per
        // dword
        const uint3 lp = make_uint3(perm(cl[1], cl[0], 0x04020100u), perm(cl[2], cl[1], 0x05040201u),
                                    perm(cl[3], cl[2], 0x06050402u));
        const uint3 rp = make_uint3(perm(cr[1], cr[0], 0x04020100u), perm(cr[2], cr[1], 0x05040201u),
                                    perm(cr[3], cr[2], 0x06050402u));
        auto store3 = [&](uint8_t* out, uint3 v) {
            if (ALIGNED) *reinterpret_cast<uint3*>(out + off) = v;
            else store_96(out + off, v);
        };
        if (f.out_l) store3(f.out_l, lp);
        if (f.out_r) store3(f.out_r, rp);
        if (f.out_a) {
            constexpr uint32_t m0 = 0xFF0000FFu, m1 = 0x00FF0000u, m2 = 0x0000FF00u;
            store3(f.out_a,
                   make_uint3((lp.x & m0) | (rp.x & ~m0), (lp.y & m1) | (rp.y & ~m1), (lp.z & m2) | (rp.z & ~m2)));
        }
    } else {
        // the quad a row of another width ends with: byte stores of its pixels
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            if (j >= n) continue;
            if (f.out_l) store_px_bytes(f.out_l + off + 3 * j, cl[j]);
            if (f.out_r) store_px_bytes(f.out_r + off + 3 * j, cr[j]);
            if (f.out_a) store_px_bytes(f.out_a + off + 3 * j, (cl[j] & 0xFFu) | (cr[j] & 0xFFFF00u));
        }
    }
    if (f.out_h) {
        const int hw = W >> 1;
        const uint32_t l0 = avg_bytes(cl[0], cl[1]), l1 = avg_bytes(cl[2], cl[3]);
        const uint32_t r0 = avg_bytes(cr[0], cr[1]), r1 = avg_bytes(cr[2], cr[3]);
        const int p0 = x0 >> 1;
        uint8_t* row = f.out_h + (size_t)y * W * 3;
        if (ALIGNED) {
            // W % 4 == 0: both pairs exist, and both halves start at even
            // byte offsets
            store_px2_u16(row + (size_t)p0 * 3, l0, l1);
            store_px2_u16(row + (size_t)(hw + p0) * 3, r0, r1);
        } else {
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                const int xa = x0 + 2 * k;
                if (xa >= W) break;
                const int pc = p0 + k;
                const bool pair = xa + 1 < W;
                const uint32_t lm = pair ? (k ? l1 : l0) : cl[2 * k];
                const uint32_t rm = pair ? (k ? r1 : r0) : cr[2 * k];
                if (pc < hw) store_px_bytes(row + (size_t)pc * 3, lm);
                store_px_bytes(row + (size_t)(hw + pc) * 3, rm);
            }
        }
    }
}

// LDS of the warp of one row: both z-buffers (kidx-padded), the shift
// table, the zero-key tag, the row's filtered depth, and per chunk (Q x 64
// lanes' quads) the keys at its valid extremes.
__host__ __device__ constexpr size_t warp_lds_bytes(int w, int threads, int q) {
    return (size_t)(2 * (((w + 3) & ~3) + ((w + 3) & ~3) / 32 + 1) * 4 + 256 * 4 + ((w + 3) & ~3) +
                    8 * q * (threads / 64) * 4 + 4);
}

// A lane's share of one image row: the frame bytes of its Q quads (three
// raw dwords per quad) and their filtered depths.
template <bool ALIGNED, int Q>
struct WarpRowIn {
    static constexpr int kPerQuad = 3;
    uint32_t c[kPerQuad * Q];
    uint32_t dq[Q];
};

template <bool ALIGNED, int Q>
__device__ __forceinline__ void warp_load(const FrameDesc& f, int y, int t, int NT, WarpRowIn<ALIGNED, Q>& in) {
    constexpr int P = WarpRowIn<ALIGNED, Q>::kPerQuad;
    const int W = f.w;
    const uint8_t* drow = f.df + (size_t)y * W;
    // the lane's first quad of the row; its next quads a uniform 12 NT bytes
    // apart
    const uint8_t* q0 = f.frame + ((size_t)y * W + 4 * t) * 3;
#pragma unroll
    for (int qi = 0; qi < Q; ++qi) {
        const int x0 = 4 * (qi * NT + t);
#pragma unroll
        for (int j = 0; j < P; ++j) in.c[P * qi + j] = 0;
        in.dq[qi] = 0;
        if (x0 >= W) continue;
        const uint3 v = load_quad_words<ALIGNED>(q0 + (size_t)qi * 12 * NT, W - x0);
        in.c[P * qi] = v.x;
        in.c[P * qi + 1] = v.y;
        in.c[P * qi + 2] = v.z;
        in.dq[qi] = load_quad_bytes<ALIGNED>(drow + x0, W - x0);
    }
}

// The warp's standing LDS state for rows of width W: the shift table, and
// both z-buffers zero.  Each row's validity pass zeroes the words of x < W;
// the padding words past the row, where out-of-row targets land, are never
// read at this width, so the state holds from row to row of one frame (rows
// of another width need a fresh preparation).  A barrier must follow before
// the first row.
__device__ __forceinline__ void warp_prepare(const FrameDesc& f, int W, int t, int NT, uint32_t* lds) {
    const int KW = kidx((W + 3) & ~3) + 1;
    uint32_t* lut = lds + 2 * KW;
    for (int d = t; d < 256; d += NT) lut[d] = shift_entry(d, f.B, f.T);
    for (int i = t; i < 2 * KW; i += NT) lds[i] = 0;
    if (t == 0) lut[256] = 0;  // the zero-key tag
}

// Key of the last (LAST) or first valid pixel of a quad: mask m (bit j =
// pixel j valid) over keys k[0..3]; 0 when none.
template <bool LAST>
__device__ __forceinline__ uint32_t quad_extreme_key(uint32_t m, const uint32_t* k) {
    uint32_t r = 0;
#pragma unroll
    for (int jj = 0; jj < 4; ++jj) {
        const int j = LAST ? jj : 3 - jj;
        if ((m >> j) & 1u) r = k[j];
    }
    return r;
}

// The key of the last (LAST) or first valid pixel of a wave's chunk, read
// back from the view's z-buffer: any = ballot of the lanes whose quad holds a
// valid pixel, m = the lane's quad mask, c0 = the chunk's first pixel; 0 when
// the chunk has none.  Uniform: one lane's mask, one broadcast LDS read.
template <bool LAST>
__device__ __forceinline__ uint32_t chunk_extreme_key(unsigned long long any, uint32_t m, const uint32_t* key,
                                                      int c0) {
    if (!any) return 0u;
    const int src = LAST ? 63 - __clzll(any) : __ffsll((long long)any) - 1;
    const uint32_t ms = __builtin_amdgcn_readlane(m, src);
    const int j = LAST ? 31 - __clz(ms) : __ffs(ms) - 1;
    return key[kidx(c0 + 4 * src + j)];
}

// Hole fill of one view's quad: pixel j with valid bit clear takes the
// nearer valid pixel on either side of the row, the smaller depth winning
// and ties going left (LEFT_TIES, the left view) or right; with a valid
// pixel on one side only that one; with none, the source pixel (need bit j).
// k: the quad's keys; ex / ef: key of the nearest valid pixel before / after
// the quad, hx / hf: whether it exists.  Returns the four colours.
template <bool LEFT_TIES>
__device__ __forceinline__ void fill_quad(uint32_t m, uint32_t own, const uint32_t* k, uint32_t ex, bool hx,
                                          uint32_t ef, bool hf, uint32_t* c, uint32_t& need) {
    uint32_t lk[4], rk[4], lh = 0, rh = 0;
    uint32_t run = ex;
    bool has = hx;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        lk[j] = run;
        if (has) lh |= 1u << j;
        if ((m >> j) & 1u) { run = k[j]; has = true; }
    }
    run = ef;
    has = hf;
#pragma unroll
    for (int j = 3; j >= 0; --j) {
        rk[j] = run;
        if (has) rh |= 1u << j;
        if ((m >> j) & 1u) { run = k[j]; has = true; }
    }
    // branch-free per pixel: an invalid pixel's key is 0, which is also its
    // colour when neither side has a valid pixel
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const bool valid = (m >> j) & 1u;
        const bool a = (lh >> j) & 1u, b = (rh >> j) & 1u;
        const uint32_t ka = lk[j], kb = rk[j];
        const bool nearer_b = LEFT_TIES ? (kb >> 24) < (ka >> 24) : (kb >> 24) <= (ka >> 24);
        const uint32_t fill = b && (!a || nearer_b) ? kb : (a ? ka : 0u);
        const uint32_t v = valid ? k[j] : fill;
        if (!valid && !a && !b && ((own >> j) & 1u)) need |= 1u << j;
        c[j] = v & 0xFFFFFFu;
    }
}

// One view's colours of a lane's quad after the hole fill (fill_quad), for
// the views whose wave has a hole; the nearest valid keys outside the quad
// come from the wave's lanes (shuffles, run on all lanes) or from the other
// chunks' published extremes (entry words pw (last) and pw + 1 (first),
// flag bit pbit).
template <bool LEFT_TIES>
__device__ __forceinline__ void fill_view(uint32_t qv, uint32_t oq, const uint32_t* k, unsigned long long any,
                                          unsigned long long below, unsigned long long above, int lane,
                                          const uint32_t* pub, int ch, int NC, int pw, uint32_t pbit, uint32_t* c,
                                          uint32_t& need) {
    if (!__ballot((oq & ~qv) != 0)) {
#pragma unroll
        for (int j = 0; j < 4; ++j) c[j] = k[j] & 0xFFFFFFu;
        return;
    }
    const unsigned long long lb = any & below, la = any & above;
    uint32_t ex = (uint32_t)__shfl((int)quad_extreme_key<true>(qv, k), lb ? 63 - __clzll(lb) : lane);
    uint32_t ef = (uint32_t)__shfl((int)quad_extreme_key<false>(qv, k), la ? __ffsll(la) - 1 : lane);
    bool hx = lb != 0, hf = la != 0;
    if (oq & ~qv) {
        for (int o = ch - 1; o >= 0 && !hx; --o)
            if (pub[8 * o + 4] & pbit) {
                ex = pub[8 * o + pw];
                hx = true;
            }
        for (int o = ch + 1; o < NC && !hf; ++o)
            if (pub[8 * o + 4] & pbit) {
                ef = pub[8 * o + pw + 1];
                hf = true;
            }
    }
    fill_quad<LEFT_TIES>(qv, oq, k, ex, hx, ef, hf, c, need);
}

// Block-iterative inpainting: tiles of kIpW x kIpH px, kIpSweeps sweeps a
// launch.  A pixel's word is its colour below a tag: 0 as warped, kIpHole a
// hole, else 1 + (sweep - 1) % (kIpSweeps * kIpCycle) of the sweep that filled
// it (tags return to 0 every kIpCycle launches).
constexpr int kIpW = 64, kIpH = 32;
constexpr int kIpSweeps = kInpaintSweeps;
constexpr int kIpCycle = 31;
constexpr uint32_t kIpHole = 255u;
static_assert(1 + kIpSweeps * kIpCycle < 254 && kMaxSweeps % kIpSweeps == 0, "tags fit beside the hole and the outside");

// Image row y on NT lanes t = 0..NT-1 (whole waves) from the lane's loaded
// share `in`; when next_y >= 0 the share of row next_y is loaded into `next`
// while this row is resolved.  lds: warp_lds_bytes(w, NT, Q) bytes in the
// state warp_prepare leaves, which the row restores.  Two barriers; inactive
// lane groups do no memory work but pass them too.
template <bool ALIGNED, int Q, bool IP = false>
__device__ __forceinline__ void warp_row_body(const FrameDesc& f, int y, int t, int NT, uint32_t* lds, bool active,
                                              const WarpRowIn<ALIGNED, Q>& in, int next_y,
                                              WarpRowIn<ALIGNED, Q>& next) {
    const int W = active ? f.w : 0;
    // wave: the same for all lanes of a wave (whole waves), held uniform
    const int lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6), NW = NT >> 6;
    const int NC = Q * NW;  // chunks per row
    const int W4 = (W + 3) & ~3;
    const int KW = kidx(W4) + 1;
    uint32_t* keyL = lds;
    uint32_t* keyR = keyL + KW;
    const uint32_t* lut = keyR + KW;                                  // 256 entries
    uint32_t* ztag = keyR + KW + 256;                                 // y + 1 if a source of row y has key 0
    uint8_t* drow_l = reinterpret_cast<uint8_t*>(ztag + 1);           // the row's filtered depth, W4 bytes
    uint32_t* pub = reinterpret_cast<uint32_t*>(drow_l + W4);         // per chunk: 8 words

    // ---- forward warp of the row's pixels into both views; the key carries
    // the depth above the colour, so the atomic max keeps the nearer source
    // and its colour
    // a target outside the row lands on a padding word (x in [W, W4]: the
    // word of x = W4 is a spare one past the row), which nothing reads, so
    // the atomics need no branch
    bool zero_key = false;
#pragma unroll
    for (int qi = 0; qi < Q; ++qi) {
        const int x0 = 4 * (qi * NT + t);
        if (x0 >= W) continue;
        const int n = ALIGNED ? 4 : min(4, W - x0);
        uint32_t c[4];
        quad_colours(make_uint3(in.c[3 * qi], in.c[3 * qi + 1], in.c[3 * qi + 2]), c);
        const uint32_t dq = in.dq[qi];
        *reinterpret_cast<uint32_t*>(drow_l + x0) = dq;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if (!ALIGNED && j >= n) continue;
            const int x = x0 + j;
            const uint32_t d = (dq >> (8 * j)) & 255u;
            const uint32_t lv = lut[d];
            const int xl = (int)min((unsigned)(x + (int)(int16_t)(lv & 0xFFFFu)), (unsigned)W4);
            const int xr = (int)min((unsigned)(x + (int)(int16_t)(lv >> 16)), (unsigned)W4);
            const uint32_t key = (d << 24) | c[j];
            zero_key |= key == 0;
            atomicMax(&keyL[kidx_held(xl)], key);
            atomicMax(&keyR[kidx_held(xr)], key);
        }
    }
    if (__ballot(zero_key) && (t & 63) == 0) *ztag = (uint32_t)y + 1u;
    __syncthreads();

    // the next row's share is loaded while this row is resolved
    if (next_y >= 0) warp_load<ALIGNED, Q>(f, next_y, t, NT, next);

    // ---- validity, and the z-buffers back to zero: a landed source has a
    // non-zero key, except a black source of depth 0, whose key is 0; such a
    // source is the only one that can land on a zero key, so in a row that
    // has one (the tag) zero keys check the depth at their depth-0 source
    // position directly
    uint32_t kl[4 * Q], kr[4 * Q];
    uint32_t vL = 0, vR = 0, own = 0;  // bit 4 qi + j
#pragma unroll
    for (int qi = 0; qi < Q; ++qi) {
        const int x0 = 4 * (qi * NT + t);
        // aligned rows hold whole quads only
        const bool quad_in = x0 < W;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int x = x0 + j;
            const int i = 4 * qi + j;
            kl[i] = 0;
            kr[i] = 0;
            if (ALIGNED ? quad_in : x < W) {
                kl[i] = keyL[kidx(x)];
                kr[i] = keyR[kidx(x)];
                own |= 1u << i;
            }
        }
    }
    // the valid bits once every read is out
#pragma unroll
    for (int i = 0; i < 4 * Q; ++i) {
        vL |= nonzero_bit(kl[i]) << i;
        vR |= nonzero_bit(kr[i]) << i;
    }
    // the lane's z-buffer words back to zero (after the chunk's extreme keys
    // are read back below: the words of a chunk are this wave's alone, and
    // its LDS accesses complete in order)
    auto clear_own = [&]() {
#pragma unroll
        for (int qi = 0; qi < Q; ++qi) {
            const int x0 = 4 * (qi * NT + t);
            const bool quad_in = x0 < W;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                if (ALIGNED ? quad_in : x0 + j < W) {
                    keyL[kidx(x0 + j)] = 0;
                    keyR[kidx(x0 + j)] = 0;
                }
            }
        }
    };
    if (*ztag == (uint32_t)y + 1u && __ballot((own & ~(vL & vR)) != 0)) {
        const uint32_t lv0 = lut[0];
        const int o0[2] = {(int)(int16_t)(lv0 & 0xFFFFu), (int)(int16_t)(lv0 >> 16)};
        const uint32_t* d32 = reinterpret_cast<const uint32_t*>(drow_l);
        const int nd = W4 >> 2;
#pragma unroll
        for (int qi = 0; qi < Q; ++qi) {
            const int x0 = 4 * (qi * NT + t);
#pragma unroll
            for (int v = 0; v < 2; ++v) {
                uint32_t& vm = v ? vR : vL;
                const uint32_t z = (own & ~vm) >> (4 * qi) & 15u;
                if (!z) continue;
                // the four sources x0 + j - o0 are consecutive bytes
                const int b = x0 - o0[v];
                const int i0 = b >> 2;
                const uint32_t w0 = d32[min(max(i0, 0), nd - 1)], w1 = d32[min(max(i0 + 1, 0), nd - 1)];
                const uint32_t bytes = alignbyte(w1, w0, (uint32_t)(b & 3));
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    if (((z >> j) & 1u) && (unsigned)(b + j) < (unsigned)W && !((bytes >> (8 * j)) & 255u))
                        vm |= 1u << (4 * qi + j);
            }
        }
    }
    if constexpr (IP) {
        // block-iterative inpainting follows: leave one word a pixel and the
        // marks of the tiles that hold a hole, no row fill
        const size_t plane = (size_t)f.w * f.h;
        const int ntx = (W + kIpW - 1) / kIpW, ntile = ntx * ((f.h + kIpH - 1) / kIpH);
#pragma unroll
        for (int qi = 0; qi < Q; ++qi) {
            const int x0 = 4 * (qi * NT + t);
            const uint32_t oq = (own >> (4 * qi)) & 15u;
            if (!oq) continue;
#pragma unroll
            for (int v = 0; v < 2; ++v) {
                const uint32_t* k = v ? &kr[4 * qi] : &kl[4 * qi];
                const uint32_t holes = oq & ~((v ? vR : vL) >> (4 * qi));
                uint32_t w[4];
#pragma unroll
                for (int j = 0; j < 4; ++j) w[j] = ((holes >> j) & 1u) ? kIpHole << 24 : k[j] & 0xFFFFFFu;
                uint32_t* dst = f.ipc + plane * v + (size_t)y * W + x0;
                if (oq == 15u) {
                    __builtin_memcpy(dst, w, 16);
                } else {
#pragma unroll
                    for (int j = 0; j < 3; ++j)
                        if ((oq >> j) & 1u) dst[j] = w[j];
                }
                if (holes) f.ipf[ntile * v + y / kIpH * ntx + x0 / kIpW] = 1u;
            }
        }
        clear_own();
        __syncthreads();  // the z-buffers and the row depth are free again
        return;
    }
    // per chunk: ballot of the quads holding a valid pixel; the keys at the
    // chunk's extremes go to LDS for the other chunks
    unsigned long long anyL[Q], anyR[Q];
#pragma unroll
    for (int qi = 0; qi < Q; ++qi) {
        const uint32_t ql = (vL >> (4 * qi)) & 15u, qr = (vR >> (4 * qi)) & 15u;
        anyL[qi] = __ballot(ql != 0);
        anyR[qi] = __ballot(qr != 0);
        const int c0 = 4 * (qi * NT + 64 * wave);  // the chunk's first pixel
        const uint32_t a = chunk_extreme_key<true>(anyL[qi], ql, keyL, c0);
        const uint32_t b = chunk_extreme_key<false>(anyL[qi], ql, keyL, c0);
        const uint32_t c = chunk_extreme_key<true>(anyR[qi], qr, keyR, c0);
        const uint32_t d = chunk_extreme_key<false>(anyR[qi], qr, keyR, c0);
        if (lane == 0) {
            uint32_t* p = pub + 8 * (qi * NW + wave);
            p[0] = a;
            p[1] = b;
            p[2] = c;
            p[3] = d;
            p[4] = (anyL[qi] ? 1u : 0u) | (anyR[qi] ? 2u : 0u);
        }
    }
    clear_own();
    __syncthreads();

    // ---- hole filling from the nearest valid keys: inside the quad, in the
    // chunk through the ballots (shuffles run on all lanes of the wave), else
    // in the other chunks; then the anaglyph and the stores
    const unsigned long long below = (1ull << lane) - 1ull;
    const unsigned long long above = ~((2ull << lane) - 1ull);
#pragma unroll
    for (int qi = 0; qi < Q; ++qi) {
        const int x0 = 4 * (qi * NT + t);
        const uint32_t ql = (vL >> (4 * qi)) & 15u, qr = (vR >> (4 * qi)) & 15u;
        const uint32_t oq = (own >> (4 * qi)) & 15u;
        uint32_t cl[4], cr[4], needL = 0, needR = 0;
        const int ch = qi * NW + wave;
        fill_view<true>(ql, oq, &kl[4 * qi], anyL[qi], below, above, lane, pub, ch, NC, 0, 1u, cl, needL);
        fill_view<false>(qr, oq, &kr[4 * qi], anyR[qi], below, above, lane, pub, ch, NC, 2, 2u, cr, needR);
        if (needL | needR) {
            // a view row without any valid pixel keeps the source pixels
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                if (!(((needL | needR) >> j) & 1u)) continue;
                const uint8_t* p = f.frame + ((size_t)y * W + x0 + j) * 3;
                const uint32_t src = p[0] | ((uint32_t)p[1] << 8) | ((uint32_t)p[2] << 16);
                if ((needL >> j) & 1u) cl[j] = src;
                if ((needR >> j) & 1u) cr[j] = src;
            }
        }
        if (x0 < W) store_quad_views<ALIGNED>(f, y, x0, cl, cr);
    }
}

// LDS bytes of the gather row: the shift table and the row's source colours.
__host__ __device__ constexpr size_t gather_lds_bytes(int w) {
    return (size_t)(256 + ((w + 3) & ~3) + (((w + 3) & ~3) >> 5) + 1) * 4;  // 256 + kidx(W4) + 1 words
}

// Image row y by the Fig. 3 gather (Section 4): each destination pixel reads
// the filtered depth at its own position and copies the source pixel its
// view's offset points back to (its own source pixel when that lies outside
// the row); no occlusion test, no holes.  The source row's colours are staged
// in LDS (padded every 32 words) so the gathers are LDS reads.
template <bool ALIGNED>
__device__ __forceinline__ void gather_row(const FrameDesc& f, int y, int t, int NT, uint32_t* lds) {
    const int W = f.w;
    uint32_t* lut = lds;           // 256 entries
    uint32_t* rowc = lut + 256;    // source colours, kidx-indexed
    for (int d = t; d < 256; d += NT) lut[d] = shift_entry(d, f.B, f.T);
    const uint8_t* src = f.frame + (size_t)y * W * 3;
    for (int x0 = 4 * t; x0 < W; x0 += 4 * NT) {
        uint32_t c[4];
        quad_colours(load_quad_words<ALIGNED>(src + (size_t)x0 * 3, W - x0), c);
#pragma unroll
        for (int j = 0; j < 4; ++j) rowc[kidx(x0 + j)] = c[j];
    }
    __syncthreads();
    const uint8_t* drow = f.df + (size_t)y * W;
    for (int x0 = 4 * t; x0 < W; x0 += 4 * NT) {
        const uint32_t dq = load_quad_bytes<ALIGNED>(drow + x0, W - x0);
        uint32_t cl[4], cr[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int x = x0 + j;
            const uint32_t lv = lut[(dq >> (8 * j)) & 255u];
            int xl = x - (int)(int16_t)(lv & 0xFFFFu);
            int xr = x - (int)(int16_t)(lv >> 16);
            if ((unsigned)xl >= (unsigned)W) xl = x;
            if ((unsigned)xr >= (unsigned)W) xr = x;
            cl[j] = x < W ? rowc[kidx(xl)] : 0u;
            cr[j] = x < W ? rowc[kidx(xr)] : 0u;
        }
        store_quad_views<ALIGNED>(f, y, x0, cl, cr);
    }
}

// One image row (the single-row form used by the batch kernels), from and
// to any LDS contents.
template <bool ALIGNED, int Q, bool IP = false>
__device__ __forceinline__ void warp_row(const FrameDesc& f, int y, int t, int NT, uint32_t* lds, bool active) {
    WarpRowIn<ALIGNED, Q> in, unused;
    if (active) {
        warp_load<ALIGNED, Q>(f, y, t, NT, in);
    } else {
#pragma unroll
        for (int i = 0; i < WarpRowIn<ALIGNED, Q>::kPerQuad * Q; ++i) in.c[i] = 0;
#pragma unroll
        for (int i = 0; i < Q; ++i) in.dq[i] = 0;
    }
    warp_prepare(f, active ? f.w : 0, t, NT, lds);
    __syncthreads();
    warp_row_body<ALIGNED, Q, IP>(f, y, t, NT, lds, active, in, -1, unused);
}

// Rows y0, y0 + step, ... below y_end of the frame, the LDS state prepared
// once, each row's loads issued during the previous row (one or two quads per
// lane: a second row's share of four would not fit the registers).
template <bool ALIGNED, int Q, bool IP = false>
__device__ __forceinline__ void warp_rows(const FrameDesc& f, int y0, int y_end, int step, int t, int NT,
                                          uint32_t* lds) {
    static_assert(Q < 4, "four quads per lane take one row at a time");
    if (y0 >= y_end) return;
    WarpRowIn<ALIGNED, Q> cur, nxt;
    warp_load<ALIGNED, Q>(f, y0, t, NT, cur);
    warp_prepare(f, f.w, t, NT, lds);
    __syncthreads();
    for (int y = y0; y < y_end; y += step) {
        const int ny = y + step < y_end ? y + step : -1;
        warp_row_body<ALIGNED, Q, IP>(f, y, t, NT, lds, true, cur, ny, nxt);
        cur = nxt;
    }
}

}  // namespace pstereo
